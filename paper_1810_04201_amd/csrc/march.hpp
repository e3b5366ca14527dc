// What the stencils on internal fields share: hops that load their operands,
// the LDS images of a marching workgroup and its launch shape, and the
// residual update done where a stencil forms A p.
#pragma once

#include <cstdlib>

#include "hops.hpp"


// hops per scheduling group (see k_dslash): with two marching workgroups
// per CU, float64 groups of 3 measured 1-2% faster than 1 (2 and 6 within
// 0.3% of 3)
#ifndef WD_GROUP_F64
#define WD_GROUP_F64 3
#endif
#ifndef WD_GROUP_LO
#define WD_GROUP_LO 2
#endif
// non-temporal forward links / outputs in the marching stencil (measured:
// streaming the outputs past the caches keeps more of the slices the
// neighbouring columns read; the links are re-read by the backward hops)
#ifndef WD_NT_LINK
#define WD_NT_LINK 0
#endif
// non-temporal forward t links: each is read once (the next slice's
// backward hop reuses it from registers), so streaming it past L2 leaves
// room for the faces neighbouring columns read (-1% time)
#ifndef WD_NT_LINK_T
#define WD_NT_LINK_T 1
#endif
#ifndef WD_NT_OUT
#define WD_NT_OUT 1
#endif
// binary16 hops (12-real links) with their link products on packed halves
// (v_dot2_f32_f16) instead of float32 operands: 48^3 x 96 binary16 stencil
// 0.63 -> 0.56 ms, its r-updating form 0.82 -> 0.79 ms
#ifndef WD_F16_DOT2
#define WD_F16_DOT2 1
#endif
// the marching stencil's fused r update: load r at the start of the step
// (its latency hidden behind the hops) instead of after them; per
// precision bit: 1 float64, 2 float32, 4 binary16
#ifndef WD_XR_PREFETCH
#define WD_XR_PREFETCH 1
#endif
// the prefetched r loaded non-temporally: read once per iteration (-1%)
#ifndef WD_NT_RLOAD
#define WD_NT_RLOAD 1
#endif


namespace wd {

// one hop: project the neighbour spinor, multiply by the link, rebuild, add
template <int MU, int S, bool BWD, int PREC, int LF = PREC>
__device__ __forceinline__ void hop(const void *gauge, const FieldRef &in, int nbr_entry,
                                    int link_site, bool negate,
                                    cx<typename Spinor<PREC>::R> acc[12]) {
    using R = typename Spinor<PREC>::R;
    if constexpr (PREC == WD_F16 && LF == WD_F16 && WD_F16_DOT2) {
        h2_t q[12];
        float sc;
        Spinor<WD_F16>::load_raw(in, nbr_entry, q, sc);
        h2_t h0[3], h1[3];
        project_h2<MU, S>(q, h0, h1);
        h2_t u[9];
        Link<WD_F16>::load_h2<false>(gauge, MU, link_site, u);
        cx<float> w0[3], w1[3];
        su3_mul_h2<BWD>(u, h0, w0);
        su3_mul_h2<BWD>(u, h1, w1);
        // the antiperiodic boundary sign rides on the site scale
        accumulate_s<MU, S>(MU == 3 && negate ? -sc : sc, w0, w1, acc);
        return;
    }
    cx<R> p[12];
    Spinor<PREC>::load(in, nbr_entry, p);
    cx<R> h0[3], h1[3];
    project<MU, S>(p, h0, h1);
    if (MU == 3) {
        // antiperiodic boundary: a select, not a branch, so that the
        // compiler keeps each hop's arithmetic next to its loads
        const R sg = negate ? R(-1) : R(1);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            h0[c] = scale(sg, h0[c]);
            h1[c] = scale(sg, h1[c]);
        }
    }
    cx<R> u[9];
    Link<LF>::load(gauge, MU, link_site, u);
    cx<R> w0[3], w1[3];
    su3_mul<BWD>(u, h0, w0);
    su3_mul<BWD>(u, h1, w1);
    accumulate<MU, S>(w0, w1, acc);
}

// LDS image of a workgroup's part of a brick slice: its tiles copied
// verbatim (a part is a multiple of 64 sites and starts at a multiple of
// 64), so the field accessors read it with the field's own tile arithmetic.
template <int PREC>
__host__ __device__ inline size_t slice_bytes(int sites) {
    return (size_t)(sites >> 6) * Spinor<PREC>::kTileBytes;
}

// field view of an LDS slice image
__device__ __forceinline__ FieldRef lds_view(const FieldRef &f, const char *img) {
    FieldRef v = f;
    v.data = (void *)img;
    return v;
}

typedef __attribute__((address_space(3))) void lds_void;

// Asynchronous copy of the slice whose first tile is tile0 into the LDS image
// img: wave w copies tile w, plane by plane, each lane 16 bytes (4 for the
// binary16 scales) straight from memory into LDS (the wave's LDS target is
// uniform, lane k lands at k * size past it).  Completion is tracked by the
// vector memory counter.
template <int PREC>
__device__ __forceinline__ void slice_copy(const FieldRef &f, int tile0, char *img) {
    constexpr size_t TB = Spinor<PREC>::kTileBytes;
    constexpr int NP = PREC == WD_F64 ? 12 : (PREC == WD_F32 ? 6 : 3);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    const char *src = (const char *)f.data + (size_t)(tile0 + w) * TB;
    char *dst = img + (size_t)w * TB;
#pragma unroll
    for (int k = 0; k < NP; ++k)
        __builtin_amdgcn_global_load_lds((const void *)(src + k * 1024 + lane * 16),
                                         (lds_void *)(dst + k * 1024), 16, 0, 0);
    if (PREC == WD_F16)
        __builtin_amdgcn_global_load_lds((const void *)(src + NP * 1024 + lane * 4),
                                         (lds_void *)(dst + NP * 1024), 4, 0, 0);
}

// The same for a part that starts at any entry: lane l copies entry first + l
// to place tid of the image (lanes past the part repeat its last entry).
template <int PREC>
__device__ __forceinline__ void slice_copy_ragged(const FieldRef &f, int entry, char *img) {
    constexpr size_t TB = Spinor<PREC>::kTileBytes;
    constexpr int NP = PREC == WD_F64 ? 12 : (PREC == WD_F32 ? 6 : 3);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    char *dst = img + (size_t)w * TB;
#pragma unroll
    for (int k = 0; k < NP; ++k)
        __builtin_amdgcn_global_load_lds((const void *)tile_elem(f.data, TB, entry, k),
                                         (lds_void *)(dst + k * 1024), 16, 0, 0);
    if constexpr (PREC == WD_F16)
        __builtin_amdgcn_global_load_lds((const void *)Spinor<WD_F16>::scale_ptr(f, entry),
                                         (lds_void *)(dst + NP * 1024), 4, 0, 0);
}

// Keeps a site's result where it is: a store that only some lanes do would
// otherwise draw the whole step's arithmetic behind its branch, and every
// operand would be spilled.
template <typename R>
__device__ __forceinline__ void pin(cx<R> v[12]) {
#pragma unroll
    for (int k = 0; k < 12; ++k) asm volatile("" : "+v"(v[k].re), "+v"(v[k].im));
}

// Wait until this wave's outstanding copies have landed in LDS.  Before the
// barrier that ends the step a lane reads them at its own place alone (PartLane),
// which its own wave filled, so no barrier is needed here: with one, the waves of a workgroup met twice per slice and
// idled together (both forms timed in turn: the 12-source float32 solve on
// 24^3 x 48 1.023 times as fast, a 48^3 x 12 slab pass 1.019; single launches at
// 48^3 x 96 differ by less than their runs do).  Binary16 keeps the barrier: its plain stencil
// measured equal without it (0.55 ms), its r-updating iteration slower (1.97 ->
// 2.15 ms).
template <int PREC>
__device__ __forceinline__ void copy_landed() {
    __builtin_amdgcn_s_waitcnt(0);
    if constexpr (PREC == WD_F16) {
        __syncthreads();
    } else {
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
    }
}

// one spatial hop of the marching stencil: the neighbour comes from the LDS
// image when it lies in this workgroup's part of the slice (wvol sites from
// sbase), else (a brick face, or another part of the slice) from memory
template <int MU, int S, bool BWD, int PREC, int LF = PREC>
__device__ __forceinline__ void hop_s(const void *gauge, const FieldRef &in, const FieldRef &cur,
                                      int sbase, int wvol, int nbr, int link_site,
                                      cx<typename Spinor<PREC>::R> acc[12]) {
    using R = typename Spinor<PREC>::R;
    const int d = nbr - sbase;
    if constexpr (PREC == WD_F16 && LF == WD_F16 && WD_F16_DOT2) {
        h2_t q[12];
        float sc;
        if ((unsigned)d < (unsigned)wvol)
            Spinor<WD_F16>::load_raw(cur, d, q, sc);
        else
            Spinor<WD_F16>::load_raw(in, nbr, q, sc);
        h2_t h0[3], h1[3];
        project_h2<MU, S>(q, h0, h1);
        h2_t u[9];
        Link<WD_F16>::load_h2<WD_NT_LINK && !BWD>(gauge, MU, link_site, u);
        cx<float> w0[3], w1[3];
        su3_mul_h2<BWD>(u, h0, w0);
        su3_mul_h2<BWD>(u, h1, w1);
        accumulate_s<MU, S>(sc, w0, w1, acc);
        return;
    }
    cx<R> p[12];
    // the compiler merges the two loads into one flat load on the selected
    // pointer (LDS or memory); separate LDS-typed and global loads measured
    // four times slower in float64 (both paths' registers live at once)
    if ((unsigned)d < (unsigned)wvol)
        Spinor<PREC>::load(cur, d, p);
    else
        Spinor<PREC>::load(in, nbr, p);
    cx<R> h0[3], h1[3];
    project<MU, S>(p, h0, h1);
    cx<R> u[9];
    Link<LF>::template load<WD_NT_LINK && !BWD>(gauge, MU, link_site, u);
    cx<R> w0[3], w1[3];
    su3_mul<BWD>(u, h0, w0);
    su3_mul<BWD>(u, h1, w1);
    accumulate<MU, S>(w0, w1, acc);
}

// r -= alpha q at site i of one rhs (r in F64, or F32 beside an F32/F16
// stencil), in the compute type of the stencil; returns |r|^2 in float64.
// The same arithmetic as the stand-alone update of the solver, on the
// stencil's unrounded q.  xr_site_r: with r already loaded into v.
template <int PREC>
__device__ __forceinline__ double xr_site_r(const XrArgs &a, int rhs, int i,
                                            typename Spinor<PREC>::R alpha,
                                            const cx<typename Spinor<PREC>::R> q[12],
                                            cx<typename Spinor<PREC>::R> v[12],
                                            bool mine = true) {
    constexpr int PX = xr_prec_of(PREC);
    double nrm = 0.0;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        v[k] = {v[k].re - alpha * q[k].re, v[k].im - alpha * q[k].im};
        nrm += (double)v[k].re * (double)v[k].re + (double)v[k].im * (double)v[k].im;
    }
    if (mine) Spinor<PX>::template store<WD_NT_OUT>(rhs_view(a.r, rhs), i, v);
    return nrm;
}

template <int PREC>
__device__ __forceinline__ double xr_site(const XrArgs &a, int rhs, int i,
                                          typename Spinor<PREC>::R alpha,
                                          const cx<typename Spinor<PREC>::R> q[12],
                                          bool mine = true) {
    constexpr int PX = xr_prec_of(PREC);
    using R = typename Spinor<PREC>::R;
    cx<R> v[12];
    Spinor<PX>::load(rhs_view(a.r, rhs), i, v);
    return xr_site_r<PREC>(a, rhs, i, alpha, q, v, mine);
}

// WD_TCHUNK overrides the marching stencil's chunk length (tuning)
static int env_chunk() {
    static const int env = [] {
        const char *e = getenv("WD_TCHUNK");
        return e ? atoi(e) : 0;
    }();
    return env;
}
static int tm_chunk(const Geom &g, int nrhs) { return tm_chunk_len(g, nrhs, env_chunk()); }

// WD_SITE_KERNEL=1 forces the one-lane-per-site stencils on internal fields (tuning)
static const bool g_force_site_kernel = [] {
    const char *e = getenv("WD_SITE_KERNEL");
    return e && atoi(e) != 0;
}();

// hops per scheduling group (see k_dslash)
template <int PREC>
struct HopGroup {
    static constexpr int value = PREC == WD_F64 ? WD_GROUP_F64 : WD_GROUP_LO;
};

// LDS a workgroup may use on the current device
static size_t max_lds_per_block() {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return 65536;
    return (size_t)v;
}

// dynamic LDS above 64 KiB must be allowed per kernel once
template <typename K>
static void allow_lds(K kernel, size_t bytes) {
    if (bytes > 65536)
        (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)bytes);
}

// launch shape of a marching stencil over slices of n sites (entries)
struct March {
    PartShape p;
    int tch, ncols, chunks;
    dim3 grid, bs;
    size_t lds;
    bool ok;  // the form runs on this geometry
};

template <int PREC>
static March march_of(const Geom &g, int n, int nrhs) {
    static const size_t cap = max_lds_per_block();
    March m{};
    if (!marches(n) || g_force_site_kernel) return m;
    m.p = geom_part(g, n, PREC);
    m.lds = 2 * slice_bytes<PREC>(m.p.threads);
    m.ok = m.lds + 64 <= cap;
    // Binary16 with 12-real links rounds differently in the first slice of a chunk
    // (its t hop is projected in float32) and in the others: on slices that are no
    // whole tiles, where solves took one lane per site before they marched, the
    // length is that of one rhs, so that a batch is its single solves bit for bit.
    const bool as_single = PREC == WD_F16 && m.p.ragged && !g.f16_links8;
    m.tch = tm_chunk(g, (as_single ? 1 : nrhs) * m.p.nsub);
    m.ncols = g.V / (g.L[3] * g.bvol);
    // chunks of one slice that do not all fit the chip at once, where chunks of
    // two do: those (each chunk pays for a slice before its first and one after
    // its last; 16^3 x 32 float64, one workgroup a CU: stencil 26.4 -> 24.9 us,
    // CG iteration 85.0 -> 80.8).  Not in binary16: the rule depends on nrhs, and a
    // batch would no longer be its single calls.
    const int at_once = 256 * (int)(cap / m.lds);
    const int parts = m.ncols * m.p.nsub * nrhs;
    const int wgs = wgs_at_once(PREC, m.p.threads, m.lds);
    // Where two float64 workgroups share a CU, no length whose workgroups are under
    // four fifths of what fits at once: some CUs have one of them and others two,
    // and the launch lasts as long as two (24 x 8 x 8 x 24 with 3 rhs 22.0 us in
    // chunks of one slice, 288 of 512 workgroups in chunks of two 26.0; 12^3 x 36 with
    // 2 rhs 24.1 and 26.6; but 24^3 x 4 with 3 rhs, 432 of 512, 34.0 and 31.2).
    auto uneven = [&](int c) {
        return PREC == WD_F64 && wgs == 512 &&
               5 * parts * ((g.L[3] + c - 1) / c) < 4 * wgs;
    };
    if (PREC != WD_F16 && env_chunk() <= 0 && m.tch == 1 && parts * g.L[3] > at_once &&
        parts * ((g.L[3] + 1) / 2) <= at_once && !uneven(2))
        m.tch = 2;
    // (not in binary16, whose steps are too short for the count: 24^3 x 48 38 us
    // at one and two slices, 40 at three, which it ranks first; nor from one
    // slice in float32, the same: 18^3 x 36 x 2 38 us, 40 at three)
    if ((PREC == WD_F64 || (PREC == WD_F32 && m.tch > 1)) && env_chunk() <= 0) {
        const int c = balanced_chunk(g.L[3], parts, wgs, m.tch, chunk_gain(PREC, nrhs));
        if (!uneven(c)) m.tch = c;
    }
    m.chunks = (g.L[3] + m.tch - 1) / m.tch;
    m.grid = dim3(m.ncols * m.chunks * m.p.nsub * nrhs);
    m.bs = dim3(m.p.threads);
    return m;
}

// Whether a plain application over slices that are no whole tiles marches: a
// solve's reducing stencils always do, and plain ones give the same bits in both
// forms.  Few sites over all rhs last as long as one workgroup's chain, in which
// parts that leave lanes idle and chunks that read two slices more weigh most.
// Float64, marching against one lane per site: 6^4 7.8 and 8.5 us; 14^4 12.6 and
// 12.1, 6^3 x 20 x 12 12.6 and 11.6; 14^4 x 2 18.2 and 19.4, but 10^4 x 12, few sites
// of each rhs, 25.9 and 22.4.  Float32: 14^4 8.4 and 7.0, 18^4 x 4 40.0 and 35.5,
// 14^3 x 28 x 12 70 and 67; 18^3 x 36 22.5 and 24.2, 18^4 x 12 92 and 94, 18^3 x 36 x 12
// 177 and 250.  Binary16: see launch_canon_out.
template <int PREC>
static bool ragged_marches(const Geom &g, int nrhs) {
    const int64_t n = (int64_t)g.V * nrhs;
    if (PREC == WD_F64) return n < 32768 || (n >= 65536 && g.V >= 16384);
    return PREC == WD_F32 && (g.V >= 196608 || n >= (1 << 20));
}

}  // namespace wd
