// Host check of what wd_set_gauge allocates, frees and launches: runtime.cpp over
// stand-ins for the HIP calls and the launchers that it makes there.  The 12-real
// float64 form exists for links that pass the check and for no others: links off
// the group cost no allocation, now or on the next call, and no more memory at the
// peak than the form they keep.  Exit code 0 on success.
#include "runtime.cpp"

static size_t live = 0, peak = 0;
static int mallocs = 0, frees = 0, syncs = 0;
static bool no_memory = false;
static std::map<void *, size_t> sizes;
static double deviation = 0.0;  // of the links that come in
static void *ingest12 = nullptr, *lo12 = nullptr;
static int lo_after_sync = 0;

extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
    if (no_memory) return hipErrorOutOfMemory;
    ++mallocs;
    *p = calloc(1, n);
    sizes[*p] = n;
    live += n;
    if (live > peak) peak = live;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    ++frees;
    live -= sizes.at(p);
    sizes.erase(p);
    free(p);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t) {
    memset(p, v, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    ++syncs;
    lo_after_sync = 0;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
}

namespace wd {
void launch_ingest(const double *, void *g64, void *g12, unsigned long long *maxbits, const Geom &g,
                   hipStream_t) {
    // the word of the deviation lies behind the tiles, in the same allocation
    if (maxbits) {
        const size_t ofs = (char *)maxbits - (char *)g64;
        if (ofs < gauge_bytes(WD_F64, g.V) || ofs + 8 > sizes.at(g64)) abort();
        memcpy(maxbits, &deviation, sizeof deviation);
    }
    ingest12 = g12;
}
void launch_gauge_lo(const void *, void *o, int form, int, hipStream_t) {
    if (form == kLinkF64R12) lo12 = o;
    ++lo_after_sync;
}
void servers_forget(wd_lattice *) {}
}  // namespace wd

static int fails = 0;
static void expect(bool ok, const char *what) {
    if (!ok) {
        ++fails;
        printf("not so: %s\n", what);
    }
}

// one call on links of the given deviation
static void set(wd_lattice *lat, double dev) {
    static double U[2];
    deviation = dev;
    mallocs = frees = syncs = 0;
    ingest12 = lo12 = nullptr;
    peak = live;
    expect(wd_set_gauge(lat, U, nullptr) == WD_OK, "the call succeeds");
    expect(lo_after_sync == 0, "every launch is waited for");
}

int main() {
    const int32_t dims[4] = {4, 4, 4, 4};
    wd_lattice *lat = nullptr;
    if (wd_create_lattice(dims, 1, &lat) != WD_OK) return 1;
    const size_t g18 = wd::gauge_bytes(WD_F64, 256) + 256;
    const size_t g12 = wd::gauge_bytes(wd::kLinkF64R12, 256);
    int reals = 0;
    double dev = 0.0;
    auto form = [&] {
        wd_lattice_links_info(lat, &reals, &dev);
        return reals;
    };
    set(lat, 1e-9);
    expect(mallocs == 1 && frees == 0 && peak == g18 && form() == 18 && dev == 1e-9,
           "first links, off the group: the 18-real form and nothing else");
    set(lat, INFINITY);
    expect(mallocs == 0 && frees == 0 && peak == g18 && form() == 18, "again: no allocation");
    set(lat, 1e-16);
    expect(mallocs == 1 && live == g18 + g12 && lo12 == lat->gauge12 && lo12 && form() == 12,
           "links in the group: the 12-real form, written from the 18");
    set(lat, 2e-16);
    expect(mallocs == 0 && frees == 0 && ingest12 == lat->gauge12 && ingest12 && !lo12 &&
               syncs == 1 && form() == 12,
           "again: written on ingest, no allocation, one synchronisation");
    set(lat, 2e-14);
    expect(mallocs == 0 && frees == 1 && live == g18 && form() == 18, "off the group: dropped");
    no_memory = true;
    set(lat, 0.0);
    expect(live == g18 && form() == 18, "no memory for 12 reals: 18 are kept");
    no_memory = false;
    set(lat, 0.0);
    expect(live == g18 + g12 && form() == 12, "memory again");
    setenv("WD_LINKS64_12", "0", 1);
    set(lat, 0.0);
    expect(live == g18 && form() == 18 && dev == -1.0 && !ingest12, "WD_LINKS64_12=0");
    wd_destroy_lattice(lat);
    expect(live == 0, "everything is freed");
    printf(fails ? "FAIL %d\n" : "OK\n", fails);
    return fails ? 1 : 0;
}
