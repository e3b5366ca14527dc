// Stencils on even-odd half fields: the off-diagonal blocks D_eo, D_oe of Eq. (1)
// (nearest neighbours have opposite parity) that the Schur complement M = 1 -
// D_eo D_oe is applied with.
#include "march.hpp"

namespace wd {

// canonical index of the first site (even x) of pair h
__device__ __forceinline__ int pair_lex(const Geom &g, int h) {
    int x, y, z, t;
    coords_of(g, 2 * h, x, y, z, t);
    return lex_of(g, x, y, z, t);
}

// Even-odd hopping term on half fields (one lane per site of one rhs):
//   out_p = cs * c_p - k * H_{p,1-p} in_{1-p}
// with H the hop sum of Eq. (1) (projectors exchanged for DAG).  Entry h of a
// half field is site site_of_half(h, p); the neighbours, of the other
// parity, sit at their internal index >> 1.  Forward links come from the
// parity-p half array gp, backward links U_mu(x - mu) from gq.  The hops are
// summed in the order of the full stencil.
// XR: the CG update r -= alpha out_p in place of storing out (the reduction
// is then |r|^2; with HASC and RED).  LF: the link form.
// COUT: the output (p = 0) goes to a canonical float64 field (out.data, out.V
// sites of the half) with zero at the odd sites.
template <int PREC, bool DAG, bool RED, bool HASC, int GROUP, bool XR = false, int LF = PREC,
          bool COUT = false>
__global__ void __launch_bounds__(256) k_hop_half(Geom g, const void *__restrict__ gp,
                                                  const void *__restrict__ gq, int p, FieldRef in,
                                                  FieldRef c, FieldRef out, double k_d,
                                                  double cs_d, RedArgs red, Gate gate,
                                                  XrArgs xr) {
    using R = typename Spinor<PREC>::R;
    if (gate_off(gate)) return;  // grid-uniform
    const int nrhs = in.nrhs;
    const int lb = logical_block();
    const int sb = lb / nrhs;
    const int rhs = lb - sb * nrhs;
    if (!gate_rhs(gate, rhs)) {  // workgroup-uniform
        if (XR && sb == 0) defer_skip(xr.alpha, rhs);
        return;
    }
    // the reduction that gives alpha, if it is left to this kernel
    Deferred dfr{};
    double rr = 0.0;
    if constexpr (XR) {
        dfr = defer_load(xr.alpha, nrhs, rhs);
        rr = gate.st[rhs].rr;
    }
    const FieldRef fin = rhs_view(in, rhs);
    const int h = sb * blockDim.x + threadIdx.x;
    __shared__ __align__(16) char stage[COUT ? kSiteBlock / 64 * Spinor<PREC>::kTileBytes : 16];
    const FieldRef tile = lds_view(
        fin, stage + (COUT ? (threadIdx.x >> 6) * Spinor<PREC>::kTileBytes : 0));
    int64_t pair = -1;
    int second = 0;
    double nrm = 0.0;
    cx<R> o[12];
    if (h < out.V) {
        const int i = site_of_half(g, h, p);
        const Nbrs nb = neighbours(g, i);
        const bool neg_tp = g.antiperiodic && nb.cross_tp;
        const bool neg_tm = g.antiperiodic && nb.cross_tm;
        cx<R> acc[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = {R(0), R(0)};
        constexpr int SF = DAG ? +1 : -1;
        constexpr int SB = -SF;
#define WD_HOP_FENCE(k) \
    if ((k) % GROUP == 0) __builtin_amdgcn_sched_barrier(0)
        hop<0, SF, false, PREC, LF>(gp, fin, nb.xp >> 1, h, false, acc);
        WD_HOP_FENCE(1);
        hop<0, SB, true, PREC, LF>(gq, fin, nb.xm >> 1, nb.xm >> 1, false, acc);
        WD_HOP_FENCE(2);
        hop<1, SF, false, PREC, LF>(gp, fin, nb.yp >> 1, h, false, acc);
        WD_HOP_FENCE(3);
        hop<1, SB, true, PREC, LF>(gq, fin, nb.ym >> 1, nb.ym >> 1, false, acc);
        WD_HOP_FENCE(4);
        hop<2, SF, false, PREC, LF>(gp, fin, nb.zp >> 1, h, false, acc);
        WD_HOP_FENCE(5);
        hop<2, SB, true, PREC, LF>(gq, fin, nb.zm >> 1, nb.zm >> 1, false, acc);
        WD_HOP_FENCE(6);
        hop<3, SF, false, PREC, LF>(gp, fin, nb.tp >> 1, h, neg_tp, acc);
        WD_HOP_FENCE(7);
        hop<3, SB, true, PREC, LF>(gq, fin, nb.tm >> 1, nb.tm >> 1, neg_tm, acc);
        WD_HOP_FENCE(8);
#undef WD_HOP_FENCE
        if constexpr (HASC) {
            Spinor<PREC>::load(rhs_view(c, rhs), h, o);
            const R cs = (R)cs_d;
#pragma unroll
            for (int k = 0; k < 12; ++k) o[k] = scale(cs, o[k]);
        } else {
#pragma unroll
            for (int k = 0; k < 12; ++k) o[k] = {R(0), R(0)};
        }
        const R kk = (R)k_d;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            o[k] = o[k] - scale(kk, acc[k]);
            if (RED && !XR)
                nrm += (double)o[k].re * (double)o[k].re + (double)o[k].im * (double)o[k].im;
        }
        if constexpr (COUT) {
            pair = (int64_t)rhs * g.V + pair_lex(g, h);
            second = i & 1;
            Spinor<PREC>::store(tile, (int)(threadIdx.x & 63), o);
        } else if constexpr (!XR) {
            Spinor<PREC>::store(rhs_view(out, rhs), h, o);
        }
    }
    if constexpr (COUT) export_tile_pairs<PREC>((double2 *)out.data, pair, second, tile);
    if constexpr (XR) {
        R alpha;
        if (xr.alpha.nb) {
            const double tt = uniform(defer_sum(xr.alpha, dfr));
            if (sb == 0) defer_write(xr.alpha, xr.ctl, RED_ALPHA, rhs, tt);
            if (!alpha_goes_on(tt)) return;
            alpha = (R)(rr / tt);
        } else {
            alpha = (R)gate.st[rhs].alpha;
        }
        if (h < out.V) nrm = xr_site<PREC>(xr, rhs, h, alpha, o);
    }
    if (RED) reduce_block(nrm, red.partials, (size_t)sb * nrhs + rhs);
}

// The half-field stencil in the time-marching form (lattices whose brick
// slices hold a multiple of 64 sites of each parity).  The parity-p half of
// a brick slice is bvol / 2 consecutive entries of a half field, and so is
// the parity-(1-p) half, pair by pair: output entry hs + l and input entry
// hs + l sit on the same site pair.  One workgroup per (chunk, column, part,
// rhs) marches t as the full stencil does, with two LDS images of its part
// of the input half slice:
//  - x/y/z neighbours (input entries nbr >> 1) from the current image when
//    they fall in the part, else from memory;
//  - the forward t neighbour of output lane l is input entry l of the next
//    half slice (same x, y, z; the other parity), from the new image;
//  - the backward t hop of slice t+1 is input entry l of slice t with its own
//    U_t (parity 1 - p links), carried in registers.
// Hops are summed in the order of k_hop_half.  Forward links come from gp at
// the output entry, backward ones from gq at the neighbour's entry.
// RAG: parts as in k_dslash_tm where a half slice is no whole number of tiles.
// COUT: as in k_hop_half.
template <int PREC, bool DAG, bool RED, bool HASC, int GROUP, bool XR, int LF, bool RAG,
          bool COUT = false>
__global__ void __launch_bounds__(kTmMaxBlock) k_hop_half_tm(Geom g, const void *__restrict__ gp,
                                                     const void *__restrict__ gq, int p,
                                                     FieldRef in, FieldRef c, FieldRef out,
                                                     double k_d, double cs_d, RedArgs red,
                                                     Gate gate, int tchunk, int ncols, int w,
                                                     XrArgs xr) {
    using R = typename Spinor<PREC>::R;
    extern __shared__ __align__(16) char lds[];
    // wave sums of the step, double-buffered by its parity: wave 0 reads them
    // after the barrier that ends the step, while others are in the next one
    __shared__ double wsum[2][kTmMaxBlock / 64];
    if (gate_off(gate)) return;  // grid-uniform
    const int nrhs = in.nrhs;
    const int hvol = g.bvol >> 1;  // entries of one parity per brick slice
    const int nsub = RAG ? (hvol + w - 1) / w : hvol / w;
    const int lb = logical_block();
    const int cb = lb / nrhs;
    const int rhs = lb - cb * nrhs;
    if (!gate_rhs(gate, rhs)) {  // workgroup-uniform
        if (XR && cb == 0) defer_skip(xr.alpha, rhs);
        return;
    }
    Deferred dfr{};  // (see k_dslash_tm)
    double rr = 0.0;
    if constexpr (XR) {
        dfr = defer_load(xr.alpha, nrhs, rhs);
        rr = gate.st[rhs].rr;
    }
    const FieldRef fin = rhs_view(in, rhs);
    const int cc = cb / nsub;
    const int hp = cb - cc * nsub;
    const int chunk = cc / ncols;
    const int col = cc - chunk * ncols;
    const int Lt = g.L[3];
    const int tid = (int)threadIdx.x;
    // entries of this workgroup's part; lanes past it repeat its last (see
    // k_dslash_tm)
    const int wvol = RAG && hvol - hp * w < w ? hvol - hp * w : w;
    const bool mine = !RAG || tid < wvol;
    const PartLane pl = RAG ? part_lane(tid, wvol) : PartLane{tid, tid};
    const int l = pl.l;
    const int t0 = chunk * tchunk;
    const int t1 = t0 + tchunk < Lt ? t0 + tchunk : Lt;
    // first entry of this workgroup's part of half slice t: hbase + t * hvol
    const int hbase = col * Lt * hvol + hp * w;
    char *img0 = lds;
    char *img1 = lds + slice_bytes<PREC>((int)blockDim.x);
    constexpr int SF = DAG ? +1 : -1;
    constexpr int SB = -SF;
    const R kappa = (R)k_d;

    // prologue: input half slice t0 into image 0, and the backward t hop of
    // slice t0 from input entry l of slice t0 - 1
    auto copy = [&](int t, char *img) {
        if constexpr (RAG)
            slice_copy_ragged<PREC>(fin, hbase + t * hvol + l, img);
        else
            slice_copy<PREC>(fin, (hbase + t * hvol) >> 6, img);
    };
    copy(t0, img0);
    cx<R> cw0[3], cw1[3];
    {
        const int ip = hbase + (t0 == 0 ? Lt - 1 : t0 - 1) * hvol + l;
        cx<R> v[12];
        Spinor<PREC>::load(fin, ip, v);
        cx<R> h0[3], h1[3];
        project<3, SB>(v, h0, h1);
        const R sg = (g.antiperiodic && t0 == 0) ? R(-1) : R(1);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            h0[k] = scale(sg, h0[k]);
            h1[k] = scale(sg, h1[k]);
        }
        cx<R> u[9];
        Link<LF>::load(gq, 3, ip, u);
        su3_mul<true>(u, h0, cw0);
        su3_mul<true>(u, h1, cw1);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    R alpha = R(0);
    if constexpr (XR) {
        if (xr.alpha.nb) {
            const double tt = uniform(defer_sum(xr.alpha, dfr));
            if (cb == 0) defer_write(xr.alpha, xr.ctl, RED_ALPHA, rhs, tt);
            if (!alpha_goes_on(tt)) return;
            alpha = (R)(rr / tt);
        } else {
            alpha = (R)gate.st[rhs].alpha;
        }
    }
    for (int t = t0; t < t1; ++t) {
        const bool odd = (t - t0) & 1;
        const FieldRef cur = lds_view(fin, odd ? img1 : img0);
        const FieldRef nxt = lds_view(fin, odd ? img0 : img1);
        const int tn = t + 1 < Lt ? t + 1 : 0;
        copy(tn, (char *)nxt.data);
        const int hs = hbase + t * hvol;
        const int H = hs + l;  // output entry
        // (not with 18-real float64 links: registers would spill)
        constexpr bool XPRE = XR && ((WD_XR_PREFETCH >> PREC) & 1) && LF != WD_F64;
        cx<R> rpre[XPRE ? 12 : 1];
        if constexpr (XPRE)
            Spinor<xr_prec_of(PREC)>::template load<WD_NT_RLOAD>(
                rhs_view(xr.r, rhs), H, rpre);
        const Nbrs nb = neighbours(g, site_of_half(g, H, p));
        cx<R> acc[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = {R(0), R(0)};
#define WD_HOP_FENCE(k) \
    if ((k) % GROUP == 0) __builtin_amdgcn_sched_barrier(0)
        hop_s<0, SF, false, PREC, LF>(gp, fin, cur, hs, wvol, nb.xp >> 1, H, acc);
        WD_HOP_FENCE(1);
        hop_s<0, SB, true, PREC, LF>(gq, fin, cur, hs, wvol, nb.xm >> 1, nb.xm >> 1, acc);
        WD_HOP_FENCE(2);
        hop_s<1, SF, false, PREC, LF>(gp, fin, cur, hs, wvol, nb.yp >> 1, H, acc);
        WD_HOP_FENCE(3);
        hop_s<1, SB, true, PREC, LF>(gq, fin, cur, hs, wvol, nb.ym >> 1, nb.ym >> 1, acc);
        WD_HOP_FENCE(4);
        hop_s<2, SF, false, PREC, LF>(gp, fin, cur, hs, wvol, nb.zp >> 1, H, acc);
        WD_HOP_FENCE(5);
        hop_s<2, SB, true, PREC, LF>(gq, fin, cur, hs, wvol, nb.zm >> 1, nb.zm >> 1, acc);
        WD_HOP_FENCE(6);
#undef WD_HOP_FENCE
        cx<R> ut[9], ub[9];
        Link<LF>::template load<WD_NT_LINK || WD_NT_LINK_T>(gp, 3, H, ut);
        Link<LF>::template load<WD_NT_LINK || WD_NT_LINK_T>(gq, 3, H, ub);
        // this wave's copy of the next half slice has landed (see k_dslash_tm)
        copy_landed<PREC>();
        {
            cx<R> nx[12];
            Spinor<PREC>::load(nxt, pl.place, nx);
            hop_p<3, SF, false>(nx, ut, g.antiperiodic && t == Lt - 1, acc);
        }
        accumulate<3, SB>(cw0, cw1, acc);
        // carry for slice t + 1: input entry l of this slice with its U_t
        {
            cx<R> v[12];
            Spinor<PREC>::load(cur, l, v);
            cx<R> h0[3], h1[3];
            project<3, SB>(v, h0, h1);
            su3_mul<true>(ub, h0, cw0);
            su3_mul<true>(ub, h1, cw1);
        }
        cx<R> o[12];
        if constexpr (HASC) {
            Spinor<PREC>::load(rhs_view(c, rhs), H, o);
            const R cs = (R)cs_d;
#pragma unroll
            for (int k = 0; k < 12; ++k) o[k] = scale(cs, o[k]);
        } else {
#pragma unroll
            for (int k = 0; k < 12; ++k) o[k] = {R(0), R(0)};
        }
        double nrm = 0.0;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            o[k] = o[k] - scale(kappa, acc[k]);
            if (RED && !XR)
                nrm += (double)o[k].re * (double)o[k].re + (double)o[k].im * (double)o[k].im;
        }
        if constexpr (RAG && XR) pin(o);
        if constexpr (XPRE)
            nrm = xr_site_r<PREC>(xr, rhs, H, alpha, o, rpre, mine);
        else if constexpr (XR)
            nrm = xr_site<PREC>(xr, rhs, H, alpha, o, mine);
        else if constexpr (!COUT)
            Spinor<PREC>::template store<WD_NT_OUT>(rhs_view(out, rhs), H, o);
        if (RED) {
            if (!mine) nrm = 0.0;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) nrm += __shfl_xor(nrm, off, 64);
            if ((tid & 63) == 0) wsum[odd][tid >> 6] = nrm;
        }
        __syncthreads();  // the current image is free for the next copy
        if constexpr (COUT) {
            FieldRef tile = cur;
            tile.data = (char *)cur.data +
                        __builtin_amdgcn_readfirstlane(tid >> 6) * Spinor<PREC>::kTileBytes;
            Spinor<PREC>::store(tile, tid & 63, o);
            export_tile_pairs<PREC>((double2 *)out.data,
                                    mine ? (int64_t)rhs * g.V + pair_lex(g, H) : -1,
                                    site_of_half(g, H, p) & 1, tile);
        }
        if (RED && tid == 0) {
            double sum = 0.0;
            for (int v = 0; v < (int)(blockDim.x >> 6); ++v) sum += wsum[odd][v];
            red.partials[(((size_t)col * Lt + t) * nsub + hp) * nrhs + rhs] = sum;
        }
    }
}

// WD_EO_SITE=1 keeps the half-field stencil one lane per site (tuning and
// tests; read at every launch)
static bool eo_site_forced() {
    const char *e = getenv("WD_EO_SITE");
    return e && atoi(e) != 0;
}

// The marching form pays where link and spinor bytes bound the launch: at
// 48^3 x 96 float64 half launches take 1.29-1.49 ms against 1.65-1.77 one
// lane per site, float32 -2%, while binary16 (bound by its arithmetic) is
// 3-8% slower marching and stays one lane per site.  Over half slices that are
// no whole tiles float32 does not gain (30^3 x 60, the two launches of the
// operator: 114 + 133 us marching, 117 + 127 one lane per site).  Float64 does from
// 12 time slices: with fewer, chunks that read two slices more and a last round of
// few workgroups cost more than one lane per site does; and not between 32768 and
// 200000 sites, which one round of one-lane workgroups holds.  48 iterations, one
// lane per site against marching: 30^3 x 8 7.9 and 9.4 ms, x 12 12.8 and 12.0, x 20 22.8
// and 18.6, x 60 61.6 and 56.8; 26^3 x 10 7.2 and 8.8, 26^4 18.9 and 16.1; 18^4 4.7 and
// 5.3, 14^3 x 28 4.3 and 4.7; 10^3 x 20 3.4 and 3.0, 6^3 x 20 3.3 and 2.7.  (Not a rule
// on the number of rhs: the sums of a batch are those of its single solves.)
template <int PREC>
static March eo_march(const Geom &g, int nrhs, bool red, int64_t partials_cap) {
    March m{};
    if (PREC == WD_F16 || eo_site_forced()) return m;
    m = march_of<PREC>(g, g.bvol / 2, nrhs);
    if (m.p.ragged && (PREC == WD_F32 || g.L[3] < 12 || (g.V >= 32768 && g.V < 200000)))
        m.ok = false;
    if (red && m.ok) m.ok = (int64_t)tm_partials(g, m.p) * nrhs <= partials_cap;
    return m;
}

// one half-field launch, marching where the geometry allows, with its
// finaliser
template <int PREC, bool DAG, bool RED, bool HASC, bool XR, int LF>
static void launch_eo(const Geom &g, const void *gp, const void *gq, int p, FieldRef in,
                      FieldRef c, FieldRef out, double k, double cs, const RedArgs &r,
                      Gate gate, const XrArgs &xr, hipStream_t s) {
    constexpr int G = HopGroup<PREC>::value;
    int nb;
    const March m = eo_march<PREC>(g, in.nrhs, RED, r.partials_cap);
    if (m.ok) {
        if constexpr (PREC != WD_F16) {
            auto go = [&](auto kern) {
                allow_lds(kern, m.lds);
                hipLaunchKernelGGL(kern, m.grid, m.bs, m.lds, s, g, gp, gq, p, in, c, out, k, cs,
                                   r, gate, m.tch, m.ncols, m.p.w, xr);
            };
            if constexpr (PREC == WD_F64) {
                if (m.p.ragged)
                    go(k_hop_half_tm<PREC, DAG, RED, HASC, G, XR, LF, true>);
                else
                    go(k_hop_half_tm<PREC, DAG, RED, HASC, G, XR, LF, false>);
            } else {
                go(k_hop_half_tm<PREC, DAG, RED, HASC, G, XR, LF, false>);
            }
        }
        nb = tm_partials(g, m.p);
    } else {
        nb = site_blocks(out.V);
        hipLaunchKernelGGL((k_hop_half<PREC, DAG, RED, HASC, G, XR, LF>), dim3(nb * in.nrhs),
                           dim3(kSiteBlock), 0, s, g, gp, gq, p, in, c, out, k, cs, r, gate, xr);
    }
    if (RED) launch_finalize(r, nb, s);
}

void hop_half_partials(const Geom &g, int prec, int nrhs, int *nb, int *threads) {
    const int64_t cap = reduce_partials_cap(g, nrhs);
    const March m = prec == WD_F64   ? eo_march<WD_F64>(g, nrhs, true, cap)
                    : prec == WD_F32 ? eo_march<WD_F32>(g, nrhs, true, cap)
                                     : eo_march<WD_F16>(g, nrhs, true, cap);
    *nb = m.ok ? tm_partials(g, m.p) : site_blocks(g.V / 2);
    *threads = m.ok ? m.p.threads : kSiteBlock;
}

template <int PREC, int LF = PREC>
static void launch_hop_half_prec(const Geom &g, const void *gp, const void *gq, int p, double k,
                                 double cs, int dagger, FieldRef in, FieldRef c, FieldRef out,
                                 const RedArgs *red, Gate gate, hipStream_t s) {
    RedArgs r{};
    if (red) r = *red;
    const XrArgs nx{};
    const bool hc = c.data != nullptr;
    const int sel = (dagger ? 4 : 0) | (red ? 2 : 0) | (hc ? 1 : 0);
    switch (sel) {
        case 0: launch_eo<PREC, false, false, false, false, LF>(g, gp, gq, p, in, c, out, k, cs, r, gate, nx, s); break;
        case 1: launch_eo<PREC, false, false, true, false, LF>(g, gp, gq, p, in, c, out, k, cs, r, gate, nx, s); break;
        case 2: launch_eo<PREC, false, true, false, false, LF>(g, gp, gq, p, in, c, out, k, cs, r, gate, nx, s); break;
        case 3: launch_eo<PREC, false, true, true, false, LF>(g, gp, gq, p, in, c, out, k, cs, r, gate, nx, s); break;
        case 4: launch_eo<PREC, true, false, false, false, LF>(g, gp, gq, p, in, c, out, k, cs, r, gate, nx, s); break;
        case 5: launch_eo<PREC, true, false, true, false, LF>(g, gp, gq, p, in, c, out, k, cs, r, gate, nx, s); break;
        case 6: launch_eo<PREC, true, true, false, false, LF>(g, gp, gq, p, in, c, out, k, cs, r, gate, nx, s); break;
        default: launch_eo<PREC, true, true, true, false, LF>(g, gp, gq, p, in, c, out, k, cs, r, gate, nx, s); break;
    }
}

// the even half of an operator's output, canonical, with zero odd sites
template <int PREC, bool DAG, int LF>
static void launch_eo_canon(const Geom &g, const void *gp, const void *gq, FieldRef in,
                            FieldRef c, FieldRef out, double k, double cs, hipStream_t s) {
    constexpr int G = HopGroup<PREC>::value;
    const Gate none{nullptr, 0, GATE_ACTIVE};
    const March m = eo_march<PREC>(g, in.nrhs, false, 0);
    if constexpr (PREC != WD_F16) {
        if (m.ok) {
            auto go = [&](auto kern) {
                allow_lds(kern, m.lds);
                hipLaunchKernelGGL(kern, m.grid, m.bs, m.lds, s, g, gp, gq, 0, in, c, out, k, cs,
                                   RedArgs{}, none, m.tch, m.ncols, m.p.w, XrArgs{});
            };
            if constexpr (PREC == WD_F64) {
                if (m.p.ragged) {
                    go(k_hop_half_tm<PREC, DAG, false, true, G, false, LF, true, true>);
                    return;
                }
            }
            go(k_hop_half_tm<PREC, DAG, false, true, G, false, LF, false, true>);
            return;
        }
    }
    hipLaunchKernelGGL((k_hop_half<PREC, DAG, false, true, G, false, LF, true>),
                       dim3(site_blocks(out.V) * in.nrhs), dim3(kSiteBlock), 0, s, g, gp, gq, 0,
                       in, c, out, k, cs, RedArgs{}, none, XrArgs{});
}

void launch_hop_half_canon(const Geom &g, const void *gp, const void *gq, double k, double cs,
                           int dagger, FieldRef in, FieldRef c, double *out, hipStream_t s,
                           bool r12) {
    FieldRef o = c;  // the half's sites
    o.data = out;
    auto go = [&](auto prec, auto lf) {
        constexpr int P = decltype(prec)::value, F = decltype(lf)::value;
        if (dagger)
            launch_eo_canon<P, true, F>(g, gp, gq, in, c, o, k, cs, s);
        else
            launch_eo_canon<P, false, F>(g, gp, gq, in, c, o, k, cs, s);
    };
    if (in.prec == WD_F32)
        go(Int<WD_F32>{}, Int<WD_F32>{});
    else if (in.prec == WD_F16 && g.f16_links8)
        go(Int<WD_F16>{}, Int<kLinkF16R8>{});
    else if (in.prec == WD_F16)
        go(Int<WD_F16>{}, Int<WD_F16>{});
    else if (r12)
        go(Int<WD_F64>{}, Int<kLinkF64R12>{});
    else
        go(Int<WD_F64>{}, Int<WD_F64>{});
}

template <int PREC, int LF = PREC>
static void launch_hop_half_xr_prec(const Geom &g, const void *gp, const void *gq, int p,
                                    double k, double cs, int dagger, FieldRef in, FieldRef c,
                                    const XrArgs &xr, const RedArgs &red, Gate gate,
                                    hipStream_t s) {
    // out only sizes the launch (xr.r is a half field like it)
    if (dagger)
        launch_eo<PREC, true, true, true, true, LF>(g, gp, gq, p, in, c, xr.r, k, cs, red, gate, xr, s);
    else
        launch_eo<PREC, false, true, true, true, LF>(g, gp, gq, p, in, c, xr.r, k, cs, red, gate, xr, s);
}

void launch_hop_half_xr(const Geom &g, const void *gp, const void *gq, int p, double k, double cs,
                        int dagger, FieldRef in, FieldRef c, const XrArgs &xr,
                        const RedArgs &red, Gate gate, hipStream_t s, bool r12) {
    switch (in.prec) {
        case WD_F64:
            if (r12)
                launch_hop_half_xr_prec<WD_F64, kLinkF64R12>(g, gp, gq, p, k, cs, dagger, in, c,
                                                              xr, red, gate, s);
            else
                launch_hop_half_xr_prec<WD_F64>(g, gp, gq, p, k, cs, dagger, in, c, xr, red, gate,
                                                s);
            break;
        case WD_F32:
            launch_hop_half_xr_prec<WD_F32>(g, gp, gq, p, k, cs, dagger, in, c, xr, red, gate, s);
            break;
        default:
            if (g.f16_links8)
                launch_hop_half_xr_prec<WD_F16, kLinkF16R8>(g, gp, gq, p, k, cs, dagger, in, c,
                                                             xr, red, gate, s);
            else
                launch_hop_half_xr_prec<WD_F16>(g, gp, gq, p, k, cs, dagger, in, c, xr, red, gate,
                                                s);
            break;
    }
}

void launch_hop_half(const Geom &g, const void *gp, const void *gq, int p, double k, double cs,
                     int dagger, FieldRef in, FieldRef c, FieldRef out, const RedArgs *red,
                     Gate gate, hipStream_t s, bool r12) {
    switch (in.prec) {
        case WD_F64:
            if (r12)
                launch_hop_half_prec<WD_F64, kLinkF64R12>(g, gp, gq, p, k, cs, dagger, in, c, out,
                                                          red, gate, s);
            else
                launch_hop_half_prec<WD_F64>(g, gp, gq, p, k, cs, dagger, in, c, out, red, gate, s);
            break;
        case WD_F32: launch_hop_half_prec<WD_F32>(g, gp, gq, p, k, cs, dagger, in, c, out, red, gate, s); break;
        default:
            if (g.f16_links8)
                launch_hop_half_prec<WD_F16, kLinkF16R8>(g, gp, gq, p, k, cs, dagger, in, c, out,
                                                         red, gate, s);
            else
                launch_hop_half_prec<WD_F16>(g, gp, gq, p, k, cs, dagger, in, c, out, red, gate,
                                             s);
            break;
    }
}

}  // namespace wd
