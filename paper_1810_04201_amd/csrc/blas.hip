// Field kernels of the CG solve (Sec. 2.2): gauge and spinor packing between
// the canonical interleaved layout and the internal planes, precision
// conversion, the vector updates of the CG iteration (x += alpha p with
// p = r + beta p in one pass; the unfused x/r update with the |r|^2
// reduction and p update), the float64 true residual, and norms.
// All of them stream their operands once; the reductions are the
// deterministic block reduction of device.hpp.
#include "hops.hpp"

namespace wd {

static constexpr int kBS = 256;  // gauge kernels (one lane per site)

// ------------------------------------------------------------------ reduction phase 2

// Fixed-order sum of the nb partials of an rhs, then the finaliser.  The order
// does not depend on nrhs (thread t sums partials t + 4jT, t + (4j+1)T,
// t + (4j+2)T, t + (4j+3)T into four running sums, T = 1024; a butterfly inside
// each wave; the 16 waves in order), so a batched solve reproduces the
// single-rhs solves bit for bit.  A block per rhs: 12 of them over 3456
// partials each took one block 24 us.  RED_TRUE tests the states of all rhs
// (a reliable update whose gate was off wrote no partials), so one block does
// them all.
constexpr int kFinalizeThreads = 1024;

__global__ void __launch_bounds__(kFinalizeThreads) k_finalize(RedArgs red, int nb) {
    if (red.mode == RED_TRUE) {
        const bool off = gate_off(Gate{red.st, red.ctl.nrhs, GATE_TRIGGER});
        __syncthreads();  // the states are read before any is written
        if (off) return;
    }
    constexpr int T = kFinalizeThreads, NW = T / 64;
    __shared__ double sm[NW * 12];
    const int nrhs = red.ctl.nrhs;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const double *P = red.partials;
    for (int r = blockIdx.x; r < nrhs; r += gridDim.x) {
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
        int b = tid;
        for (; b + 3 * T < nb; b += 4 * T) {
            a0 += P[(size_t)b * nrhs + r];
            a1 += P[(size_t)(b + T) * nrhs + r];
            a2 += P[(size_t)(b + 2 * T) * nrhs + r];
            a3 += P[(size_t)(b + 3 * T) * nrhs + r];
        }
        for (; b < nb; b += T) a0 += P[(size_t)b * nrhs + r];
        double v = (a0 + a1) + (a2 + a3);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0) sm[w * 12 + r] = v;
    }
    __syncthreads();
    for (int r = blockIdx.x + tid * gridDim.x; r < nrhs; r += kFinalizeThreads * gridDim.x) {
        double t = 0.0;
        for (int k = 0; k < NW; ++k) t += sm[k * 12 + r];
        if (red.mode != RED_NONE) finalize_state(red.st[r], red.ctl, red.mode, t);
    }
}

void launch_finalize(const RedArgs &red, int nb, hipStream_t s) {
    if (red.deferred) return;
    hipLaunchKernelGGL(k_finalize, dim3(red.mode == RED_TRUE ? 1 : red.ctl.nrhs),
                       dim3(kFinalizeThreads), 0, s, red, nb);
}

// ------------------------------------------------------------------ gauge

// Gauge ingest: canonical [s][mu][a][b][re,im] (lexicographic s) -> F64-18 tiles
// in brick order, and in the same pass (CHECK) the F64-12 tiles (g12 given) and
// the largest deviation of a row 2 from conj(row 0 x row 1): per block in LDS,
// then one atomic maximum on the bit pattern (non-negative doubles order like
// their patterns).  Bound by memory: 1536 bytes per site where a pass each for
// the tiles, the check and the 12-real form moved 2688 (24^3 x 48: 168 + 98 + 82
// us, in one pass 213).
template <bool CHECK>
__global__ void __launch_bounds__(kBS) k_ingest(const double2 *__restrict__ canon,
                                                void *__restrict__ g, void *__restrict__ g12,
                                                Geom geo, unsigned long long *maxbits) {
    __shared__ double wmax[kBS / 64];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    double e = 0.0;
    if (i < geo.V) {
        int x, y, z, t;
        coords_of(geo, i, x, y, z, t);
        const double2 *src = canon + (size_t)lex_of(geo, x, y, z, t) * 36;
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) {
            cx<double> u[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                double2 d = src[mu * 9 + k];
                u[k] = {d.x, d.y};
            }
            Link<WD_F64>::store(g, mu, i, u);
            if constexpr (CHECK) {
                if (g12) Link<kLinkF64R12>::store(g12, mu, i, u);
                cx<double> r[9];
#pragma unroll
                for (int k = 0; k < 6; ++k) r[k] = u[k];
                reconstruct_row2(r);
#pragma unroll
                for (int j = 6; j < 9; ++j) {
                    const double dr = u[j].re - r[j].re, di = u[j].im - r[j].im;
                    const double d = sqrt(dr * dr + di * di);
                    if (!(d <= e)) e = d == d ? d : INFINITY;
                }
            }
        }
    }
    if constexpr (CHECK) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) e = fmax(e, __shfl_xor(e, off, 64));
        if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = e;
        __syncthreads();
        if (threadIdx.x == 0) {
            double m = wmax[0];
            for (int w = 1; w < (int)(blockDim.x >> 6); ++w) m = fmax(m, wmax[w]);
            atomicMax(maxbits, (unsigned long long)__double_as_longlong(m));
        }
    }
}

// F64-18 -> the compressed forms: 12 reals (rows 0 and 1, rounded to nearest
// even), or the 8-real binary16 form
template <int PREC>
__global__ void k_gauge_lo(const void *__restrict__ g, void *__restrict__ o, int V) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= V) return;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        cx<double> u[9];
        Link<WD_F64>::load(g, mu, i, u);
        Link<PREC>::store(o, mu, i, u);
    }
}

void launch_ingest(const double *canon, void *g64, void *g12, unsigned long long *maxbits,
                   const Geom &geo, hipStream_t s) {
    const dim3 gr(blocks_for(geo.V, kBS)), bs(kBS);
    if (maxbits)
        hipLaunchKernelGGL(k_ingest<true>, gr, bs, 0, s, (const double2 *)canon, g64, g12, geo,
                           maxbits);
    else
        hipLaunchKernelGGL(k_ingest<false>, gr, bs, 0, s, (const double2 *)canon, g64, nullptr,
                           geo, maxbits);
}

void launch_gauge_lo(const void *g64, void *glo, int form, int V, hipStream_t s) {
    const dim3 gr(blocks_for(V, kBS)), bs(kBS);
    if (form == WD_F32)
        hipLaunchKernelGGL(k_gauge_lo<WD_F32>, gr, bs, 0, s, g64, glo, V);
    else if (form == WD_F16)
        hipLaunchKernelGGL(k_gauge_lo<WD_F16>, gr, bs, 0, s, g64, glo, V);
    else if (form == kLinkF64R12)
        hipLaunchKernelGGL(k_gauge_lo<kLinkF64R12>, gr, bs, 0, s, g64, glo, V);
    else if (form == kLinkF16R8)
        hipLaunchKernelGGL(k_gauge_lo<kLinkF16R8>, gr, bs, 0, s, g64, glo, V);
}

// even-odd: links of the parity-p sites in the half layout and format PREC
template <int PREC>
__global__ void k_gauge_split(const void *__restrict__ g, void *__restrict__ o, int p, Geom geo) {
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    if (h >= geo.V / 2) return;
    const int i = site_of_half(geo, h, p);
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        cx<double> u[9];
        Link<WD_F64>::load(g, mu, i, u);
        Link<PREC>::store(o, mu, h, u);
    }
}

void launch_gauge_split(const void *g64, void *half, int form, int p, const Geom &geo,
                        hipStream_t s) {
    const dim3 gr(blocks_for(geo.V / 2, kBS)), bs(kBS);
    const int prec = form;
    if (form == kLinkF64R12)
        hipLaunchKernelGGL(k_gauge_split<kLinkF64R12>, gr, bs, 0, s, g64, half, p, geo);
    else if (prec == WD_F64)
        hipLaunchKernelGGL(k_gauge_split<WD_F64>, gr, bs, 0, s, g64, half, p, geo);
    else if (prec == WD_F32)
        hipLaunchKernelGGL(k_gauge_split<WD_F32>, gr, bs, 0, s, g64, half, p, geo);
    else if (form == kLinkF16R8)
        hipLaunchKernelGGL(k_gauge_split<kLinkF16R8>, gr, bs, 0, s, g64, half, p, geo);
    else
        hipLaunchKernelGGL(k_gauge_split<WD_F16>, gr, bs, 0, s, g64, half, p, geo);
}

// ------------------------------------------------------------------ spinors

template <int PREC>
__device__ __forceinline__ void load_as_double(const FieldRef &f, int i, cx<double> v[12]) {
    cx<typename Spinor<PREC>::R> t[12];
    Spinor<PREC>::load(f, i, t);
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = {(double)t[k].re, (double)t[k].im};
}

template <int PREC>
__device__ __forceinline__ void store_from_double(const FieldRef &f, int i, const cx<double> v[12]) {
    using R = typename Spinor<PREC>::R;
    cx<R> t[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) t[k] = {(R)v[k].re, (R)v[k].im};
    Spinor<PREC>::store(f, i, t);
}

// Every field kernel below runs a grid of site_blocks(V) x nrhs workgroups:
// lane = site of the rhs blockIdx.y, so gating by the solver state is
// uniform over a workgroup.
static dim3 field_grid(const FieldRef &f) { return dim3(site_blocks(f.V), f.nrhs); }

// A field goes out through LDS, a wave's tile at a time (export_tile): a lane
// writing its own site spreads every store over 64 places 192 bytes apart.
// 48^3 x 96 out of float64 898 -> 781 us, out of float32 641 -> 587, binary16
// 633 -> 494; two rhs of 18^3 x 36 in binary16 30 -> 17.
// A half field comes in the same way, 12 lanes to a site (208 bytes apart there,
// so that the lanes that then read a component of one site each meet different
// banks): 30^3 x 60 into float32 90 -> 64 us.  A whole field's import reads per
// lane: its 64 sites are rows of consecutive memory that the cache holds whole
// until the lanes have read them (48^3 x 96 into float64 770 us, through LDS 779;
// 24^3 x 48 x 12 into float32 421 and 428).
constexpr int kImportWave = 64 * 208;

// src: the canonical field; lex: the lane's own site in it; img: the wave's
// kImportWave bytes of LDS
__device__ __forceinline__ void gather_site(const double2 *src, int64_t lex, char *img,
                                            cx<double> v[12]) {
    typedef __attribute__((address_space(3))) void lds_void;
    const int lane = threadIdx.x & 63;
    const int lo = (int)(uint32_t)lex, hi = (int)(lex >> 32);
#pragma unroll
    for (int j = 0; j < 13; ++j) {
        const int e = j * 64 + lane, site = e / 13, k = e - site * 13;
        const int64_t st = ((int64_t)__shfl(hi, site, 64) << 32) | (uint32_t)__shfl(lo, site, 64);
        __builtin_amdgcn_global_load_lds((const void *)(src + st * 12 + (k < 12 ? k : 11)),
                                         (lds_void *)(img + j * 1024), 16, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const d2_t d = *(const d2_t *)(img + lane * 208 + k * 16);
        v[k] = {d.x, d.y};
    }
}

// canonical [rhs][s][12][re,im] (lexicographic s) <-> internal site i of rhs, or
// (HALF) entry h of a half field of parity p: site site_of_half(h, p), f.V = V / 2.
// DIRECT: each lane its own site, also where buffers are aligned to a double only.
template <bool HALF>
__device__ __forceinline__ int64_t canon_index(const Geom &geo, int r, int i, int p) {
    int x, y, z, t;
    coords_of(geo, HALF ? site_of_half(geo, i, p) : i, x, y, z, t);
    return (int64_t)r * geo.V + lex_of(geo, x, y, z, t);
}

template <int PREC, bool HALF, bool DIRECT>
__global__ void __launch_bounds__(kSiteBlock) k_import(const double2 *__restrict__ canon,
                                                       FieldRef f, int p, Geom geo) {
    __shared__ __align__(16) char img[kSiteBlock / 64][DIRECT ? 16 : kImportWave];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool mine = i < f.V;
    const int r = blockIdx.y;
    const int64_t lex = canon_index<HALF>(geo, r, mine ? i : f.V - 1, p);
    cx<double> v[12];
    if constexpr (DIRECT) {
#pragma unroll
        for (int k = 0; k < 12; ++k) v[k] = {canon[lex * 12 + k].x, canon[lex * 12 + k].y};
    } else {
        gather_site(canon, lex, img[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)], v);
    }
    if (mine) store_from_double<PREC>(rhs_view(f, r), i, v);
}

template <int PREC, bool HALF, bool DIRECT>
__global__ void __launch_bounds__(kSiteBlock) k_export(FieldRef f, double2 *__restrict__ canon,
                                                       int p, Geom geo) {
    typedef __attribute__((address_space(3))) void lds_void;
    constexpr int TB = (int)Spinor<PREC>::kTileBytes;
    __shared__ __align__(16) char img[kSiteBlock / 64][DIRECT ? 16 : TB];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool mine = i < f.V;
    const int r = blockIdx.y;
    const FieldRef fr = rhs_view(f, r);
    if constexpr (DIRECT) {
        if (!mine) return;
        const int64_t lex = canon_index<HALF>(geo, r, i, p);
        cx<double> v[12];
        load_as_double<PREC>(fr, i, v);
#pragma unroll
        for (int k = 0; k < 12; ++k) canon[lex * 12 + k] = make_double2(v[k].re, v[k].im);
    } else {
        // whole tiles: the last one of a field is padded in memory
        const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int first = __builtin_amdgcn_readfirstlane(i & ~63);
        if (first >= f.V) return;
        const int64_t lex = mine ? canon_index<HALF>(geo, r, i, p) : -1;
        const char *src = (const char *)fr.data + (size_t)(first >> 6) * TB;
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int k = 0; k < TB / 1024; ++k)
            __builtin_amdgcn_global_load_lds((const void *)(src + k * 1024 + lane * 16),
                                             (lds_void *)(img[w] + k * 1024), 16, 0, 0);
        if constexpr (PREC == WD_F16)
            __builtin_amdgcn_global_load_lds((const void *)(src + 3072 + lane * 4),
                                             (lds_void *)(img[w] + 3072), 4, 0, 0);
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
        FieldRef tile = fr;
        tile.data = img[w];
        export_tile<PREC>(canon, lex, tile);
    }
}

template <int PREC>
__global__ void k_zero(FieldRef f) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= f.V) return;
    cx<double> v[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = {0.0, 0.0};
    store_from_double<PREC>(rhs_view(f, blockIdx.y), i, v);
}

// x64 += xlo ; xlo = 0 for the rhs a reliable update takes (GATE_TRIGGER),
// else for every rhs not yet converged.  An rhs whose last alpha p is still
// pending (it froze between the r update and the lagged x update) adds it:
// x64 += xlo + alpha p, in float64.
template <int PL, int PP>
__global__ void __launch_bounds__(kSiteBlock) k_accum_zero(FieldRef x, FieldRef xl, FieldRef p,
                                                         Gate gate) {
    const int r = blockIdx.y;
    if (gate.mode == GATE_TRIGGER) {
        if (gate_off(gate) || !gate_rhs(gate, r)) return;
    } else if (gate.st[r].converged) {
        return;
    }
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= x.V) return;
    const FieldRef xv = rhs_view(x, r), lv = rhs_view(xl, r);
    cx<double> b[12];
    load_as_double<PL>(lv, i, b);
    if (gate.st[r].pend) {
        const double alpha = gate.st[r].alpha;
        cx<double> q[12];
        load_as_double<PP>(rhs_view(p, r), i, q);
#pragma unroll
        for (int k = 0; k < 12; ++k) b[k] = {b[k].re + alpha * q[k].re, b[k].im + alpha * q[k].im};
    }
    {
        cx<double> a[12];
        load_as_double<WD_F64>(xv, i, a);
#pragma unroll
        for (int k = 0; k < 12; ++k) b[k] = a[k] + b[k];
    }
    store_from_double<WD_F64>(xv, i, b);
#pragma unroll
    for (int k = 0; k < 12; ++k) b[k] = {0.0, 0.0};
    store_from_double<PL>(lv, i, b);
}

#define WD_DISPATCH_PREC(P, ...)                   \
    switch (P) {                                   \
        case WD_F64: { constexpr int PP = WD_F64; __VA_ARGS__; } break; \
        case WD_F32: { constexpr int PP = WD_F32; __VA_ARGS__; } break; \
        default: { constexpr int PP = WD_F16; __VA_ARGS__; } break;     \
    }

template <bool HALF>
static void import_any(const double *canon, FieldRef f, int p, const Geom &geo, hipStream_t s) {
    const dim3 gr = field_grid(f), bs(kSiteBlock);
    const double2 *c = (const double2 *)canon;
    if constexpr (HALF) {
        if (((uintptr_t)canon & 15) == 0) {
            WD_DISPATCH_PREC(f.prec, hipLaunchKernelGGL((k_import<PP, HALF, false>), gr, bs, 0, s,
                                                        c, f, p, geo));
            return;
        }
    }
    WD_DISPATCH_PREC(f.prec, hipLaunchKernelGGL((k_import<PP, HALF, true>), gr, bs, 0, s, c, f, p,
                                                geo));
}

template <bool HALF>
static void export_any(FieldRef f, double *canon, int p, const Geom &geo, hipStream_t s) {
    const dim3 gr = field_grid(f), bs(kSiteBlock);
    double2 *c = (double2 *)canon;
    if (((uintptr_t)canon & 15) == 0) {
        WD_DISPATCH_PREC(f.prec, hipLaunchKernelGGL((k_export<PP, HALF, false>), gr, bs, 0, s, f,
                                                    c, p, geo));
    } else {
        WD_DISPATCH_PREC(f.prec, hipLaunchKernelGGL((k_export<PP, HALF, true>), gr, bs, 0, s, f, c,
                                                    p, geo));
    }
}

void launch_import(const double *canon, FieldRef f, const Geom &geo, hipStream_t s) {
    import_any<false>(canon, f, 0, geo, s);
}
void launch_export(FieldRef f, double *canon, const Geom &geo, hipStream_t s) {
    export_any<false>(f, canon, 0, geo, s);
}
void launch_import_half(const double *canon, FieldRef f, int p, const Geom &geo, hipStream_t s) {
    import_any<true>(canon, f, p, geo, s);
}
void launch_export_half(FieldRef f, double *canon, int p, const Geom &geo, hipStream_t s) {
    export_any<true>(f, canon, p, geo, s);
}

void launch_zero(FieldRef f, hipStream_t s) {
    WD_DISPATCH_PREC(f.prec,
                     hipLaunchKernelGGL(k_zero<PP>, field_grid(f), dim3(kSiteBlock), 0, s, f));
}

void launch_accum_zero(FieldRef x, FieldRef xl, FieldRef p, Gate gate, hipStream_t s) {
    const dim3 gr = field_grid(x), bs(kSiteBlock);
    if (xl.prec == WD_F64)
        hipLaunchKernelGGL((k_accum_zero<WD_F64, WD_F64>), gr, bs, 0, s, x, xl, p, gate);
    else if (p.prec == WD_F32)
        hipLaunchKernelGGL((k_accum_zero<WD_F32, WD_F32>), gr, bs, 0, s, x, xl, p, gate);
    else
        hipLaunchKernelGGL((k_accum_zero<kF16XrPrec, WD_F16>), gr, bs, 0, s, x, xl, p, gate);
}

// ------------------------------------------------------------------ CG updates

// x += alpha p ; r -= alpha Ap ; |r|^2.  x, r in precision PX (F64 or F32);
// p, Ap in PP (same as PX, or F16 with PX = F32).  Arithmetic in the compute
// type of PX, the norm in float64.  A frozen rhs's workgroups return at once
// (the finaliser ignores its partials).
template <int PX, int PPP>
__global__ void __launch_bounds__(kSiteBlock) k_update_xr(FieldRef x, FieldRef r, FieldRef p,
                                                        FieldRef Ap, RedArgs red, Gate gate) {
    if (gate_off(gate)) return;
    const int rhs = blockIdx.y;
    if (!gate_rhs(gate, rhs)) return;
    using R = typename Spinor<PX>::R;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    double nrm = 0.0;
    if (i < x.V) {
        const FieldRef xf = rhs_view(x, rhs), rf = rhs_view(r, rhs);
        const R alpha = (R)gate.st[rhs].alpha;
        cx<R> xv[12], rv[12], pv[12], av[12];
        Spinor<PX>::load(xf, i, xv);
        Spinor<PX>::load(rf, i, rv);
        Spinor<PPP>::load(rhs_view(p, rhs), i, pv);
        Spinor<PPP>::load(rhs_view(Ap, rhs), i, av);
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            xv[k] = {xv[k].re + alpha * pv[k].re, xv[k].im + alpha * pv[k].im};
            rv[k] = {rv[k].re - alpha * av[k].re, rv[k].im - alpha * av[k].im};
            nrm += (double)rv[k].re * (double)rv[k].re + (double)rv[k].im * (double)rv[k].im;
        }
        Spinor<PX>::store(xf, i, xv);
        Spinor<PX>::store(rf, i, rv);
    }
    reduce_block(nrm, red.partials, (size_t)blockIdx.x * x.nrhs + rhs);
}

// p = r + beta p
template <int PX, int PPP>
__global__ void k_update_p(FieldRef p, FieldRef r, Gate gate) {
    const int rhs = blockIdx.y;
    if (!gate_rhs(gate, rhs)) return;
    using R = typename Spinor<PX>::R;
    using RP = typename Spinor<PPP>::R;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= p.V) return;
    const FieldRef pf = rhs_view(p, rhs);
    const R beta = (R)gate.st[rhs].beta;
    cx<R> rv[12];
    cx<RP> q[12];
    Spinor<PX>::load(rhs_view(r, rhs), i, rv);
    Spinor<PPP>::load(pf, i, q);
#pragma unroll
    for (int k = 0; k < 12; ++k)
        q[k] = {(RP)(rv[k].re + beta * (R)q[k].re), (RP)(rv[k].im + beta * (R)q[k].im)};
    Spinor<PPP>::store(pf, i, q);
}

// After a reliable update: r_lo = r64 rounded to its format, p = r_lo + beta p
// (at the first update p = r_lo), with r_lo as stored.
template <int PX, int PPP>
__global__ void k_restart(FieldRef r64, FieldRef rlo, FieldRef p, Gate gate) {
    const int rhs = blockIdx.y;
    if (!gate_rhs(gate, rhs)) return;
    const RhsState &st = gate.st[rhs];
    using R = typename Spinor<PX>::R;
    using RP = typename Spinor<PPP>::R;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= p.V) return;
    const FieldRef pf = rhs_view(p, rhs), rf = rhs_view(rlo, rhs);
    cx<double> d[12];
    Spinor<WD_F64>::load(rhs_view(r64, rhs), i, d);
    store_from_double<PX>(rf, i, d);
    cx<R> rv[12];
    if constexpr (PX == WD_F16) {
        Spinor<PX>::load(rf, i, rv);
    } else {
#pragma unroll
        for (int k = 0; k < 12; ++k) rv[k] = {(R)d[k].re, (R)d[k].im};
    }
    cx<RP> o[12];
    if (st.updates == 1) {
#pragma unroll
        for (int k = 0; k < 12; ++k) o[k] = {(RP)rv[k].re, (RP)rv[k].im};
    } else {
        const R beta = (R)st.beta;
        Spinor<PPP>::load(pf, i, o);
#pragma unroll
        for (int k = 0; k < 12; ++k)
            o[k] = {(RP)(rv[k].re + beta * (R)o[k].re), (RP)(rv[k].im + beta * (R)o[k].im)};
    }
    Spinor<PPP>::store(pf, i, o);
}

// non-temporal loads and stores in k_update_xp: each field streams through
// once per iteration (48^3 x 96: -5% float64, -8% in the binary16 mode)
#ifndef WD_NT_XP
#define WD_NT_XP 1
#endif

// x += alpha p ; p = r + beta p: the x update of the iteration whose r
// update a stencil did, merged with the p update (p read once).  Same
// arithmetic as k_update_xr's x update and k_update_p.
// DEFER: the reduction of |r|^2 that gives beta is finished here (Cons); the
// fields are loaded before it is waited for.
template <int PX, int PPP, bool DEFER>
__global__ void __launch_bounds__(kSiteBlock) k_update_xp(FieldRef x, FieldRef p, FieldRef r,
                                                          Gate gate, Cons rr, SolveCtl ctl) {
    const int rhs = blockIdx.y;
    using R = typename Spinor<PX>::R;
    using RP = typename Spinor<PPP>::R;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const FieldRef xf = rhs_view(x, rhs), pf = rhs_view(p, rhs), rf = rhs_view(r, rhs);
    Deferred d{};
    if constexpr (DEFER) d = defer_load(rr, ctl.nrhs, rhs);
    if constexpr (DEFER) {
        const RhsState &f = rr.from[rhs];  // not written by this kernel
        if (!f.active) {
            // failed at the first reduction: the iterate's state learns it here
            if (f.failed && blockIdx.x == 0 && threadIdx.x == 0) copy_state(rr.next[rhs], f);
            return;
        }
    } else {
        if (!gate_rhs(gate, rhs)) return;
    }
    cx<RP> q[12];
    cx<R> v[12], w[DEFER ? 12 : 1];
    R alpha, beta;
    if constexpr (DEFER) {
        if (i < p.V) {
            Spinor<PPP>::template load<WD_NT_XP>(pf, i, q);
            Spinor<PX>::template load<WD_NT_XP>(xf, i, v);
            Spinor<PX>::template load<WD_NT_XP>(rf, i, w);
        }
        const RhsState &s = rr.from[rhs];
        const double total = uniform(defer_sum(rr, d));
        if (blockIdx.x == 0) defer_write(rr, ctl, RED_RR, rhs, total);
        if (!rr_goes_on(s, ctl, total) || i >= p.V) return;
        alpha = (R)s.alpha;
        beta = (R)(total / s.rr);
    } else {
        if (i >= p.V) return;
        alpha = (R)gate.st[rhs].alpha;
        beta = (R)gate.st[rhs].beta;
        Spinor<PPP>::template load<WD_NT_XP>(pf, i, q);
        Spinor<PX>::template load<WD_NT_XP>(xf, i, v);
    }
#pragma unroll
    for (int k = 0; k < 12; ++k)
        v[k] = {v[k].re + alpha * (R)q[k].re, v[k].im + alpha * (R)q[k].im};
    Spinor<PX>::template store<WD_NT_XP>(xf, i, v);
    if constexpr (DEFER) {
#pragma unroll
        for (int k = 0; k < 12; ++k) v[k] = w[k];
    } else {
        Spinor<PX>::template load<WD_NT_XP>(rf, i, v);
    }
    cx<RP> o[12];
#pragma unroll
    for (int k = 0; k < 12; ++k)
        o[k] = {(RP)(v[k].re + beta * (R)q[k].re), (RP)(v[k].im + beta * (R)q[k].im)};
    Spinor<PPP>::template store<WD_NT_XP>(pf, i, o);
}

template <bool DEFER>
static void update_xp_impl(FieldRef x, FieldRef p, FieldRef r, Gate gate, const Cons &rr,
                           const SolveCtl &ctl, hipStream_t s) {
    const dim3 gr = field_grid(p), bs(kSiteBlock);
    if (x.prec == WD_F64)
        hipLaunchKernelGGL((k_update_xp<WD_F64, WD_F64, DEFER>), gr, bs, 0, s, x, p, r, gate, rr, ctl);
    else if (p.prec == WD_F32)
        hipLaunchKernelGGL((k_update_xp<WD_F32, WD_F32, DEFER>), gr, bs, 0, s, x, p, r, gate, rr, ctl);
    else
        hipLaunchKernelGGL((k_update_xp<kF16XrPrec, WD_F16, DEFER>), gr, bs, 0, s, x, p, r, gate, rr, ctl);
}

void launch_update_xp(FieldRef x, FieldRef p, FieldRef r, Gate gate, const Cons &rr,
                      const SolveCtl &ctl, hipStream_t s) {
    if (rr.nb)
        update_xp_impl<true>(x, p, r, gate, rr, ctl, s);
    else
        update_xp_impl<false>(x, p, r, gate, rr, ctl, s);
}

void launch_update_xr(FieldRef x, FieldRef r, FieldRef p, FieldRef Ap, const RedArgs &red,
                      Gate gate, hipStream_t s) {
    const dim3 gr = field_grid(x), bs(kSiteBlock);
    if (x.prec == WD_F64)
        hipLaunchKernelGGL((k_update_xr<WD_F64, WD_F64>), gr, bs, 0, s, x, r, p, Ap, red, gate);
    else if (p.prec == WD_F32)
        hipLaunchKernelGGL((k_update_xr<WD_F32, WD_F32>), gr, bs, 0, s, x, r, p, Ap, red, gate);
    else
        hipLaunchKernelGGL((k_update_xr<kF16XrPrec, WD_F16>), gr, bs, 0, s, x, r, p, Ap, red, gate);
    launch_finalize(red, gr.x, s);
}

void launch_update_p(FieldRef p, FieldRef r, Gate gate, hipStream_t s) {
    const dim3 gr = field_grid(p), bs(kSiteBlock);
    if (r.prec == WD_F64)
        hipLaunchKernelGGL((k_update_p<WD_F64, WD_F64>), gr, bs, 0, s, p, r, gate);
    else if (p.prec == WD_F32)
        hipLaunchKernelGGL((k_update_p<WD_F32, WD_F32>), gr, bs, 0, s, p, r, gate);
    else
        hipLaunchKernelGGL((k_update_p<kF16XrPrec, WD_F16>), gr, bs, 0, s, p, r, gate);
}

void launch_restart(FieldRef r64, FieldRef rlo, FieldRef p, Gate gate, hipStream_t s) {
    const dim3 gr = field_grid(p), bs(kSiteBlock);
    if (rlo.prec == WD_F64)
        hipLaunchKernelGGL((k_restart<WD_F64, WD_F64>), gr, bs, 0, s, r64, rlo, p, gate);
    else if (p.prec == WD_F32)
        hipLaunchKernelGGL((k_restart<WD_F32, WD_F32>), gr, bs, 0, s, r64, rlo, p, gate);
    else
        hipLaunchKernelGGL((k_restart<kF16XrPrec, WD_F16>), gr, bs, 0, s, r64, rlo, p, gate);
}

// ------------------------------------------------------------------ residual / norms

// r = b - Ax (Ax absent: r = b), float64; reduce |r|^2.  A gated-off rhs
// writes no partial (the finaliser ignores it).
__global__ void k_residual(FieldRef r, FieldRef b, FieldRef Ax, RedArgs red, Gate gate) {
    if (gate_off(gate)) return;
    const int rhs = blockIdx.y;
    if (!gate_rhs(gate, rhs)) return;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    double nrm = 0.0;
    if (i < r.V) {
        cx<double> bv[12];
        Spinor<WD_F64>::load(rhs_view(b, rhs), i, bv);
        if (Ax.data) {
            cx<double> av[12];
            Spinor<WD_F64>::load(rhs_view(Ax, rhs), i, av);
#pragma unroll
            for (int k = 0; k < 12; ++k) bv[k] = bv[k] - av[k];
        }
#pragma unroll
        for (int k = 0; k < 12; ++k) nrm += bv[k].re * bv[k].re + bv[k].im * bv[k].im;
        Spinor<WD_F64>::store(rhs_view(r, rhs), i, bv);
    }
    reduce_block(nrm, red.partials, (size_t)blockIdx.x * r.nrhs + rhs);
}

template <int PREC>
__global__ void k_norm(FieldRef f, RedArgs red) {
    const int rhs = blockIdx.y;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    double nrm = 0.0;
    if (i < f.V) {
        cx<double> v[12];
        load_as_double<PREC>(rhs_view(f, rhs), i, v);
#pragma unroll
        for (int k = 0; k < 12; ++k) nrm += v[k].re * v[k].re + v[k].im * v[k].im;
    }
    reduce_block(nrm, red.partials, (size_t)blockIdx.x * f.nrhs + rhs);
}

void launch_residual(FieldRef r, FieldRef b, FieldRef Ax, const RedArgs &red, Gate gate,
                     hipStream_t s) {
    const dim3 gr = field_grid(r);
    hipLaunchKernelGGL(k_residual, gr, dim3(kSiteBlock), 0, s, r, b, Ax, red, gate);
    launch_finalize(red, gr.x, s);
}

void launch_norm(FieldRef f, const RedArgs &red, hipStream_t s) {
    const dim3 gr = field_grid(f);
    WD_DISPATCH_PREC(f.prec, hipLaunchKernelGGL(k_norm<PP>, gr, dim3(kSiteBlock), 0, s, f, red));
    launch_finalize(red, gr.x, s);
}

__global__ void k_init_state(RhsState *st, RhsState *st2, int nrhs) {
    if ((int)threadIdx.x < nrhs) st[threadIdx.x] = st2[threadIdx.x] = RhsState{};
}

void launch_init_state(RhsState *st, RhsState *st2, int nrhs, hipStream_t s) {
    hipLaunchKernelGGL(k_init_state, dim3(1), dim3(64), 0, s, st, st2, nrhs);
}

}  // namespace wd
