// The stencil of Eq. (1) applied straight to canonical spinors (wd_apply):
// out = in - kappa * (hops) read from and written to the caller's
// [rhs][V][24] float64 arrays, in place of an import into internal tiles, the
// stencil on them and an export.  Float64 and float32; the float32 operator
// rounds each component as it reads it, exactly as the import does.  The links
// are the resident internal forms.
//
// Bound by memory: links and two spinors per site, 768 bytes in float64 where
// the three passes moved 1536.  48^3 x 96 3.52 -> 1.94 ms (4.2 TB/s of those
// 768 bytes), 24^3 x 48 237 -> 118 us, 16^3 x 32 52.8 -> 26.8; 18^3 x 36, whose
// bricks are no whole tiles and whose links have 18 reals, 115 -> 47 us; 8^4 33 ->
// 8.2 us a call.  Float32 takes this form on
// small lattices only: its image would be float64 too, and reading float64
// faces costs it more than the import (24^3 x 48, 12 rhs: 1.64 ms against
// 1.18 for import and launch_dslash_canon).
#include "apply.hpp"

#include "hops.hpp"

namespace wd {

// ------------------------------------------------------------------ sites

// a site of a brick column: its coordinates fix its canonical index in a time
// slice and the steps to its six neighbours in both orders, the same in
// every slice
struct ColSite {
    int lex;        // canonical index within a time slice
    int d[6];       // internal index step to x+, x-, y+, y-, z+, z-
    int dl[6];      // canonical index step
};

__device__ __forceinline__ ColSite col_site(const Geom &g, int col, int loc) {
    const int bx = col % g.ncx;
    const int q = col / g.ncx;
    const int by = q % g.ncy, bz = q / g.ncy;
    const int xl = loc % g.tx;
    const int r = loc / g.tx;
    const int yl = r % g.ty, zl = r / g.ty;
    const int x = bx * g.tx + xl, y = by * g.ty + yl, z = bz * g.tz + zl;
    const int Lx = g.L[0], Ly = g.L[1], Lz = g.L[2];
    ColSite c;
    c.lex = x + Lx * (y + Ly * z);
    const int cx = g.L[3] * g.bvol;
    nbr_dir(0, xl, g.tx, bx, g.ncx, 1, cx, c.d[0], c.d[1]);
    nbr_dir(0, yl, g.ty, by, g.ncy, g.tx, g.ncx * cx, c.d[2], c.d[3]);
    nbr_dir(0, zl, g.tz, bz, g.ncz, g.tx * g.ty, g.ncx * g.ncy * cx, c.d[4], c.d[5]);
    c.dl[0] = x == Lx - 1 ? 1 - Lx : 1;
    c.dl[1] = x == 0 ? Lx - 1 : -1;
    c.dl[2] = y == Ly - 1 ? Lx * (1 - Ly) : Lx;
    c.dl[3] = y == 0 ? Lx * (Ly - 1) : -Lx;
    c.dl[4] = z == Lz - 1 ? Lx * Ly * (1 - Lz) : Lx * Ly;
    c.dl[5] = z == 0 ? Lx * Ly * (Lz - 1) : -Lx * Ly;
    return c;
}

__device__ __forceinline__ const char *canon_site(const double2 *f, int64_t site) {
    return (const char *)f + site * kSiteBytes;
}

// a spinor of 12 consecutive complex float64 (memory or LDS image), in the
// compute type
template <typename R>
__device__ __forceinline__ void load12(const char *p, cx<R> v[12]) {
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const d2_t d = *(const d2_t *)(p + 16 * k);
        v[k] = {(R)d.x, (R)d.y};
    }
}

// ------------------------------------------------------------------ one lane per site

// For lattices too small to fill the chip: every load is issued from one
// wave's program without a barrier, so the launch lasts a few memory
// latencies.
template <int PREC, bool DAG, int LF>
__global__ void __launch_bounds__(kApplySiteBlock, 1)
    k_apply_site(Geom g, const void *__restrict__ gauge, const double2 *__restrict__ in,
                 double2 *__restrict__ out, double kappa_d, int nrhs) {
    using R = typename Spinor<PREC>::R;
    const int lb = logical_block();
    const int sb = lb / nrhs;
    const int rhs = lb - sb * nrhs;
    const int i = sb * kApplySiteBlock + (int)threadIdx.x;
    if (i >= g.V) return;
    in += (size_t)rhs * g.V * 12;
    out += (size_t)rhs * g.V * 12;
    const int Lt = g.L[3], V3 = g.V / Lt;
    const int ct = i / g.bvol, loc = i - ct * g.bvol;
    const int col = ct / Lt, t = ct - col * Lt;
    const ColSite s = col_site(g, col, loc);
    const int lex = s.lex + t * V3;
    const int tp = t == Lt - 1 ? 1 - Lt : 1, tm = t == 0 ? Lt - 1 : -1;
    cx<R> acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = {R(0), R(0)};
    constexpr int SF = DAG ? +1 : -1;
    constexpr int SB = -SF;
    // one hop: the neighbour, its link, the projection
    auto fwd = [&](auto mu, int l, bool neg) {
        constexpr int MU = decltype(mu)::value;
        cx<R> p[12], u[9];
        load12<R>(canon_site(in, l), p);
        Link<LF>::load(gauge, MU, i, u);
        hop_p<MU, SF, false>(p, u, neg, acc);
    };
    auto bwd = [&](auto mu, int j, int l, bool neg) {
        constexpr int MU = decltype(mu)::value;
        cx<R> p[12], u[9];
        load12<R>(canon_site(in, l), p);
        Link<LF>::load(gauge, MU, j, u);
        hop_p<MU, SB, true>(p, u, neg, acc);
    };
    fwd(Int<0>{}, lex + s.dl[0], false);
    bwd(Int<0>{}, i + s.d[1], lex + s.dl[1], false);
    fwd(Int<1>{}, lex + s.dl[2], false);
    bwd(Int<1>{}, i + s.d[3], lex + s.dl[3], false);
    fwd(Int<2>{}, lex + s.dl[4], false);
    bwd(Int<2>{}, i + s.d[5], lex + s.dl[5], false);
    fwd(Int<3>{}, lex + tp * V3, g.antiperiodic && t == Lt - 1);
    bwd(Int<3>{}, i + tm * g.bvol, lex + tm * V3, g.antiperiodic && t == 0);
    cx<R> c[12];
    load12<R>(canon_site(in, lex), c);
    const R kappa = (R)kappa_d;
#pragma unroll
    for (int k = 0; k < 12; ++k) c[k] = c[k] - scale(kappa, acc[k]);
    d2_t *o = (d2_t *)canon_site(out, lex);
#pragma unroll
    for (int k = 0; k < 12; ++k) o[k] = d2_t{(double)c[k].re, (double)c[k].im};
}

// ------------------------------------------------------------------ marching

// LDS image of a workgroup's part of a time slice: one canonical spinor per
// site, 208 bytes apart (13 elements of 16 bytes, an odd number, so that
// 16 lanes reading one component of consecutive sites meet 16 different
// bank groups).  A tile of 64 sites is 13 KiB.
constexpr int kImgSite = 208;
static_assert(kImgTile == 64 * kImgSite, "image tile");

typedef __attribute__((address_space(3))) void lds_void;

// The marching stencil of dslash.hip on canonical spinors: one workgroup per
// brick column, chunk of time slices, part of the brick slice (w sites, the
// last one maybe fewer) and rhs, one lane per site, two LDS images.  The
// copies of a slice write the image linearly, lane after lane, so each wave
// gathers its 64 sites with 13 instructions whose lanes read consecutive
// memory (every 13th element is padding and repeats its neighbour), and the
// results leave through the same tile in the same order.  Lanes past the part
// repeat its last site, stores included.
template <bool DAG, int LF>
__global__ void __launch_bounds__(kApplyPart, 2)
    k_apply_tm(Geom g, const void *__restrict__ gauge, const double2 *__restrict__ in,
               double2 *__restrict__ out, double kappa_d, int nrhs, int tchunk, int ncols, int w) {
    using R = double;
    extern __shared__ __align__(16) char lds[];
    const int nsub = (g.bvol + w - 1) / w;
    const int lb = logical_block();
    const int cb = lb / nrhs;
    const int rhs = lb - cb * nrhs;
    in += (size_t)rhs * g.V * 12;
    out += (size_t)rhs * g.V * 12;
    const int cc = cb / nsub;
    const int h = cb - cc * nsub;
    const int chunk = cc / ncols;
    const int col = cc - chunk * ncols;
    const int Lt = g.L[3], bvol = g.bvol, V3 = g.V / Lt;
    const int n = bvol - h * w < w ? bvol - h * w : w;  // sites of this part
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const PartLane pl = part_lane(tid, n);
    int l = pl.l;
    ColSite s = col_site(g, col, h * w + l);
    const int t0 = chunk * tchunk;
    const int t1 = t0 + tchunk < Lt ? t0 + tchunk : Lt;
    const int cbase = col * Lt * bvol + h * w;
    constexpr int SF = DAG ? +1 : -1;
    constexpr int SB = -SF;
    const R kappa = (R)kappa_d;

    // element of a slice (16 bytes each) that this lane copies in each of the
    // 13 instructions of its wave's tile
    int src[13];
#pragma unroll
    for (int j = 0; j < 13; ++j) {
        const int e = j * 64 + lane, site = e / 13, k = e - site * 13;
        src[j] = __shfl(s.lex, site, 64) * 12 + (k < 12 ? k : 11);
    }
    const int imgbytes = (int)(blockDim.x >> 6) * kImgTile;
    const int wtile = __builtin_amdgcn_readfirstlane(tid >> 6) * kImgTile;
    auto copy = [&](int t, char *img) {
        const double2 *f = in + (size_t)t * V3 * 12;
#pragma unroll
        for (int j = 0; j < 13; ++j)
            __builtin_amdgcn_global_load_lds((const void *)(f + (unsigned)src[j]),
                                             (lds_void *)(img + wtile + j * 1024), 16, 0, 0);
    };

    // prologue: slice t0, and the backward t hop from t0 - 1
    copy(t0, lds);
    cx<R> cw0[3], cw1[3];
    auto carry = [&](const cx<R> p[12], const cx<R> u[9], R sg) {
        cx<R> h0[3], h1[3];
        project<3, SB>(p, h0, h1);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            h0[k] = scale(sg, h0[k]);
            h1[k] = scale(sg, h1[k]);
        }
        su3_mul<true>(u, h0, cw0);
        su3_mul<true>(u, h1, cw1);
    };
    {
        const int tprev = t0 == 0 ? Lt - 1 : t0 - 1;
        cx<R> p[12], u[9];
        load12<R>(canon_site(in, (int64_t)tprev * V3 + s.lex), p);
        Link<LF>::load(gauge, 3, cbase + tprev * bvol + l, u);
        carry(p, u, g.antiperiodic && t0 == 0 ? R(-1) : R(1));
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    for (int t = t0; t < t1; ++t) {
        const bool odd = (t - t0) & 1;
        const char *cur = lds + (odd ? imgbytes : 0);
        char *nxt = lds + (odd ? 0 : imgbytes);
        const int tn = t + 1 < Lt ? t + 1 : 0;
        // the steps are the same in every slice, and the compiler would keep
        // every address built from them across the loop (over 100 registers,
        // spilled): make them opaque here
#pragma unroll
        for (int k = 0; k < 6; ++k) asm volatile("" : "+v"(s.d[k]), "+v"(s.dl[k]));
        asm volatile("" : "+v"(s.lex), "+v"(l));
#pragma unroll
        for (int j = 0; j < 13; ++j) asm volatile("" : "+v"(src[j]));
        copy(tn, nxt);
        const int i = cbase + t * bvol + l;
        const double2 *ft = in + (size_t)t * V3 * 12;
        cx<R> acc[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = {R(0), R(0)};
        // a neighbour inside the part from the image, else from memory; one
        // load on the selected address (see dslash.hip)
        auto nbr = [&](int dir, cx<R> p[12]) {
            const int d = l + s.d[dir];
            const char *a = (unsigned)d < (unsigned)n ? cur + d * kImgSite
                                                      : canon_site(ft, s.lex + s.dl[dir]);
            load12<R>(a, p);
        };
        auto fwd = [&](auto mu) {
            constexpr int MU = decltype(mu)::value;
            cx<R> p[12], u[9];
            nbr(2 * MU, p);
            Link<LF>::load(gauge, MU, i, u);
            hop_p<MU, SF, false>(p, u, false, acc);
        };
        auto bwd = [&](auto mu) {
            constexpr int MU = decltype(mu)::value;
            cx<R> p[12], u[9];
            nbr(2 * MU + 1, p);
            Link<LF>::load(gauge, MU, i + s.d[2 * MU + 1], u);
            hop_p<MU, SB, true>(p, u, false, acc);
        };
        // after each pair of hops the sum is made opaque: the compiler
        // otherwise moves the arithmetic of all hops behind the loads of the
        // last one and spills.  Pairs against single hops: 48^3 x 96 2.02
        // against 2.04 ms, 18^3 x 36 (12-real links) 48.5 against 50.5 us.
        auto fence = [&] {
#pragma unroll
            for (int k = 0; k < 12; ++k) asm volatile("" : "+v"(acc[k].re), "+v"(acc[k].im));
            __builtin_amdgcn_sched_barrier(0);
        };
        fwd(Int<0>{});
        bwd(Int<0>{});
        fence();
        fwd(Int<1>{});
        bwd(Int<1>{});
        fence();
        fwd(Int<2>{});
        bwd(Int<2>{});
        fence();
        cx<R> ut[9];
        Link<LF>::template load<true>(gauge, 3, i, ut);
        // this wave's copy of the next slice has landed: until the barrier that
        // ends the step a lane reads its own place of it
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
        {
            cx<R> nx[12];
            load12<R>(nxt + pl.place * kImgSite, nx);
            hop_p<3, SF, false>(nx, ut, g.antiperiodic && t == Lt - 1, acc);
        }
        accumulate<3, SB>(cw0, cw1, acc);
        cx<R> c[12];
        load12<R>(cur + l * kImgSite, c);
        carry(c, ut, R(1));
#pragma unroll
        for (int k = 0; k < 12; ++k) c[k] = c[k] - scale(kappa, acc[k]);
        __syncthreads();  // the current image is free
        // out through this wave's tile of it, as the copies came in: lane
        // after lane, so that a store instruction fills whole lines
        char *tile = (char *)cur + wtile;
#pragma unroll
        for (int k = 0; k < 12; ++k)
            *(d2_t *)(tile + lane * kImgSite + 16 * k) = d2_t{c[k].re, c[k].im};
        wave_lds_sync();
        d2_t *fo = (d2_t *)out + (size_t)t * V3 * 12;
#pragma unroll
        for (int j = 0; j < 13; ++j) {
            const d2_t v = *(const d2_t *)(tile + (j * 64 + lane) * 16);
            if ((j * 64 + lane) % 13 < 12) fo[(unsigned)src[j]] = v;
        }
        wave_lds_sync();
    }
}

template <int PREC, int LF>
static void launch_site(const Geom &g, const void *gauge, double kappa, int dagger, int nrhs,
                        const double2 *in, double2 *out, hipStream_t s) {
    const dim3 grid(blocks_for(g.V, kApplySiteBlock) * nrhs), bs(kApplySiteBlock);
    if (dagger)
        hipLaunchKernelGGL((k_apply_site<PREC, true, LF>), grid, bs, 0, s, g, gauge, in, out,
                           kappa, nrhs);
    else
        hipLaunchKernelGGL((k_apply_site<PREC, false, LF>), grid, bs, 0, s, g, gauge, in, out,
                           kappa, nrhs);
}

template <int LF>
static void launch_march(const Geom &g, const void *gauge, double kappa, int dagger, int nrhs,
                         const double2 *in, double2 *out, hipStream_t s) {
    const ApplyShape a = apply_shape(g, nrhs);
    const int threads = (a.w + 63) / 64 * 64;
    const dim3 grid(a.ncols * a.nchunks * a.nsub * nrhs), bs(threads);
    const size_t lds = apply_lds(threads);
    auto go = [&](auto k) {
        (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
        hipLaunchKernelGGL(k, grid, bs, lds, s, g, gauge, in, out, kappa, nrhs, a.tchunk, a.ncols,
                           a.w);
    };
    if (dagger)
        go(k_apply_tm<true, LF>);
    else
        go(k_apply_tm<false, LF>);
}

bool apply_direct_ok(const Geom &g, int prec, int nrhs, const double *in, const double *out) {
    if ((((uintptr_t)in | (uintptr_t)out) & 15) != 0) return false;
    // fields that share memory: through an import, which reads all of `in` first
    const size_t n = (size_t)g.V * nrhs * 24;
    if ((uintptr_t)in < (uintptr_t)(out + n) && (uintptr_t)out < (uintptr_t)(in + n)) return false;
    return prec == WD_F64 || (prec == WD_F32 && !apply_march(g, nrhs));
}

void launch_apply(const Geom &g, const void *gauge, const void *g12, double kappa, int prec,
                  int dagger, int nrhs, const double *in, double *out, hipStream_t s) {
    const double2 *ci = (const double2 *)in;
    double2 *co = (double2 *)out;
    const bool march = apply_march(g, nrhs);
    if (prec == WD_F32) {
        launch_site<WD_F32, WD_F32>(g, gauge, kappa, dagger, nrhs, ci, co, s);
    } else if (g12) {
        if (march)
            launch_march<kLinkF64R12>(g, g12, kappa, dagger, nrhs, ci, co, s);
        else
            launch_site<WD_F64, kLinkF64R12>(g, g12, kappa, dagger, nrhs, ci, co, s);
    } else {
        if (march)
            launch_march<WD_F64>(g, gauge, kappa, dagger, nrhs, ci, co, s);
        else
            launch_site<WD_F64, WD_F64>(g, gauge, kappa, dagger, nrhs, ci, co, s);
    }
}

}  // namespace wd
