// Wilson-Dirac stencil (Eq. (1) of Sec. 2.1 with the minus sign) on gfx950.
//
// One lane per site of one right-hand side.  Each of the eight hops projects the
// neighbour spinor to a half-spinor with 1 -+ gamma_mu (two spin components
// of three colours; the projectors have rank 2, Sec. 2.1), multiplies the two
// colour vectors by U_mu(x) (forward) or U_mu(x-mu)^dag (backward), and
// rebuilds the lower two spin components from the upper two by a sign or a
// factor +-i.  The result is out(x) = in(x) - kappa * sum of the hops.
// D^dag uses the same kernel with the projector signs exchanged.
//
// Half-spinor table for (1 + s gamma_mu) psi with the Appendix A basis:
//   mu=0: h0 = psi0 + s i psi3, h1 = psi1 + s i psi2;  lower: -s i h1, -s i h0
//   mu=1: h0 = psi0 - s psi3,   h1 = psi1 + s psi2;    lower:  s h1,   -s h0
//   mu=2: h0 = psi0 + s i psi2, h1 = psi1 - s i psi3;  lower: -s i h0,  s i h1
//   mu=3: h0 = psi0 + s psi2,   h1 = psi1 + s psi3;    lower:  s h0,    s h1
// D uses s = -1 forward and s = +1 backward; D^dag the opposite.
//
// Bandwidth bound: 1320 flop per site against 960 bytes (FP64, 18-real
// links), so there is no matrix-core work here; the kernel is written for
// coalesced 16-byte loads from the structure-of-arrays planes.
#include "march.hpp"

namespace wd {

// COUT: the output goes to a canonical float64 field (out.data) instead.
template <int PREC, bool DAG, bool RED, int GROUP, int LF = PREC, bool COUT = false>
__global__ void __launch_bounds__(256) k_dslash(Geom g, const void *__restrict__ gauge, FieldRef in,
                                                FieldRef out, double kappa_d, RedArgs red,
                                                Gate gate) {
    using R = typename Spinor<PREC>::R;
    if (gate_off(gate)) return;  // grid-uniform
    // logical block = site block * nrhs + rhs: the workgroups of all rhs on
    // the same sites are neighbours in the XCD's run and share its L2 links
    const int nrhs = in.nrhs;
    const int lb = logical_block();
    const int sb = lb / nrhs;
    const int rhs = lb - sb * nrhs;
    // a gated-off rhs: the finaliser ignores its partials
    if (!gate_rhs(gate, rhs)) return;  // workgroup-uniform
    const FieldRef fin = rhs_view(in, rhs);
    const int site = sb * blockDim.x + threadIdx.x;
    __shared__ __align__(16) char stage[COUT ? kSiteBlock / 64 * Spinor<PREC>::kTileBytes : 16];
    const FieldRef tile = lds_view(
        fin, stage + (COUT ? (threadIdx.x >> 6) * Spinor<PREC>::kTileBytes : 0));
    int64_t lex = -1;
    double nrm = 0.0;
    if (site < g.V) {
        const Nbrs nb = neighbours(g, site);
        const int xp = nb.xp, xm = nb.xm, yp = nb.yp, ym = nb.ym;
        const int zp = nb.zp, zm = nb.zm, tp = nb.tp, tm = nb.tm;
        const bool neg_tp = g.antiperiodic && nb.cross_tp;
        const bool neg_tm = g.antiperiodic && nb.cross_tm;

        cx<R> acc[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = {R(0), R(0)};
        // forward projector sign: D -> s = -1, D^dag -> s = +1; backward opposite
        constexpr int SF = DAG ? +1 : -1;
        constexpr int SB = -SF;
        // A scheduling barrier after every GROUP hops bounds how many hops'
        // operands the compiler keeps in flight (registers versus
        // memory-level parallelism).
#define WD_HOP_FENCE(k) \
    if ((k) % GROUP == 0) __builtin_amdgcn_sched_barrier(0)
        hop<0, SF, false, PREC, LF>(gauge, fin, xp, site, false, acc);
        WD_HOP_FENCE(1);
        hop<0, SB, true, PREC, LF>(gauge, fin, xm, xm, false, acc);
        WD_HOP_FENCE(2);
        hop<1, SF, false, PREC, LF>(gauge, fin, yp, site, false, acc);
        WD_HOP_FENCE(3);
        hop<1, SB, true, PREC, LF>(gauge, fin, ym, ym, false, acc);
        WD_HOP_FENCE(4);
        hop<2, SF, false, PREC, LF>(gauge, fin, zp, site, false, acc);
        WD_HOP_FENCE(5);
        hop<2, SB, true, PREC, LF>(gauge, fin, zm, zm, false, acc);
        WD_HOP_FENCE(6);
        hop<3, SF, false, PREC, LF>(gauge, fin, tp, site, neg_tp, acc);
        WD_HOP_FENCE(7);
        hop<3, SB, true, PREC, LF>(gauge, fin, tm, tm, neg_tm, acc);
        WD_HOP_FENCE(8);
#undef WD_HOP_FENCE

        cx<R> c[12];
        Spinor<PREC>::load(fin, site, c);
        const R kappa = (R)kappa_d;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            c[k] = c[k] - scale(kappa, acc[k]);
            if (RED) nrm += (double)c[k].re * (double)c[k].re + (double)c[k].im * (double)c[k].im;
        }
        if constexpr (COUT) {
            int x, y, z, t;
            coords_of(g, site, x, y, z, t);
            lex = (int64_t)rhs * g.V + lex_of(g, x, y, z, t);
            Spinor<PREC>::store(tile, (int)(threadIdx.x & 63), c);
        } else {
            Spinor<PREC>::store(rhs_view(out, rhs), site, c);
        }
    }
    if constexpr (COUT) export_tile<PREC>((double2 *)out.data, lex, tile);
    if (RED) reduce_block(nrm, red.partials, (size_t)sb * nrhs + rhs);
}

// Time-marching stencil.  One workgroup per brick column, chunk of time
// slices, part of the brick slice (all of it, or one of several contiguous
// runs of whole tiles) and rhs, one lane per site.  The workgroup steps through its
// slices together with two LDS images of its part:
//  - at the start of step t the next slice t+1 is copied from memory into
//    the spare image, while the x/y/z hops of slice t read their neighbours
//    from the current image (inside the part) or from memory (across a
//    brick face or into another part);
//  - the forward t hop reads psi(t+1) from the new image, which is the
//    current one of the next step, so every site of the column is read from
//    memory once;
//  - the backward t hop U_t(x, t-1)^dag (1 -+ gamma_t) psi(x, t-1) is carried
//    from the previous step in registers.
// The hops are summed in the order of the one-lane-per-site kernel.
// Logical blocks are ordered chunk, column, part, rhs (rhs fastest), so each
// XCD's contiguous run covers one band of time slices of many neighbouring
// columns, and the workgroups of all rhs of a column part run side by side
// and read its links from L2 after the first.
// The fused reduction writes one partial per (column, slice, part, rhs), so
// its summation order does not depend on the chunk length or on nrhs.
// HALO: the lattice is one t-slab of a larger one; the t hops across its
// ends read staged faces (see Halo) in place of the wrapped slices: only the
// sources of the prologue's spinor and link, of the last step's slice copy,
// and the boundary sign change.
// XR: the CG update that consumes q = A p is done where q is formed, so q is
// never stored: r -= alpha q, and the reduction is |r|^2 (see XrArgs).  out
// is unused.
// LF: the link form (PREC's own, or F64-12 for float64).
// COUT: the output goes to a canonical float64 field (out.data) instead.
// RAG: the brick slice is no whole number of tiles; parts of w sites that
// start anywhere, the last one shorter (see PartShape; without HALO).  Such
// lattices took one lane per site before: 30^3 x 60 float64 520 -> 387 us,
// float32 187 -> 148, binary16 95 -> 82, float64 CG iteration (with the fused
// r update, which only this form has) 1584 -> 1105 us; 18^3 x 36 float64 69 ->
// 46 us, CG iteration 212 -> 148.  (Their float64 links have 18 reals: links12.
// With 12 the stencil at 30^3 x 60 takes 320 us, the iteration 1000.)
template <int PREC, bool DAG, bool RED, int GROUP, bool HALO = false, bool XR = false,
          int LF = PREC, bool COUT = false, bool RAG = false>
__global__ void __launch_bounds__(kTmMaxBlock) k_dslash_tm(Geom g, const void *__restrict__ gauge,
                                                   FieldRef in, FieldRef out, double kappa_d,
                                                   RedArgs red, Gate gate, int tchunk,
                                                   int ncols, int w, Halo halo, XrArgs xr) {
    using R = typename Spinor<PREC>::R;
    extern __shared__ __align__(16) char lds[];
    // wave sums of the step, double-buffered by its parity: wave 0 reads them
    // after the barrier that ends the step, while others are in the next one
    __shared__ double wsum[2][kTmMaxBlock / 64];
    if (gate_off(gate)) return;  // grid-uniform
    const int nrhs = in.nrhs;
    const int nsub = RAG ? (g.bvol + w - 1) / w : g.bvol / w;
    const int lb = logical_block();
    const int cb = lb / nrhs;
    const int rhs = lb - cb * nrhs;
    // a gated-off rhs: the finaliser ignores its partials
    if (!gate_rhs(gate, rhs)) {  // workgroup-uniform
        if (XR && cb == 0) defer_skip(xr.alpha, rhs);
        return;
    }
    // the reduction that gives alpha, if it is left to this kernel
    Deferred dfr{};
    double rr = 0.0;
    if constexpr (XR) {
        dfr = defer_load(xr.alpha, nrhs, rhs);
        rr = gate.st[rhs].rr;
    }
    const FieldRef fin = rhs_view(in, rhs), fout = rhs_view(out, rhs);
    const int cc = cb / nsub;
    const int h = cb - cc * nsub;
    const int lchunk = cc / ncols;
    const int col = cc - lchunk * ncols;
    const int chunk = HALO ? halo.cfirst + lchunk * halo.cstep : lchunk;
    const int Lt = g.L[3], bvol = g.bvol;
    const int tid = (int)threadIdx.x;
    // sites of this workgroup's part of a slice; lanes past it repeat its last,
    // with its result (what is not a plain store of it asks `mine`)
    const int wvol = RAG && bvol - h * w < w ? bvol - h * w : w;
    const bool mine = !RAG || tid < wvol;
    const PartLane pl = RAG ? part_lane(tid, wvol) : PartLane{tid, tid};
    const int l = pl.l;
    const int t0 = chunk * tchunk;
    const int t1 = t0 + tchunk < Lt ? t0 + tchunk : Lt;
    // first site of this workgroup's part of slice t: cbase + t * bvol
    const int cbase = col * Lt * bvol + h * w;
    char *img0 = lds;
    char *img1 = lds + slice_bytes<PREC>((int)blockDim.x);
    constexpr int SF = DAG ? +1 : -1;
    constexpr int SB = -SF;
    const R kappa = (R)kappa_d;

    // halo: this workgroup's part of a face (first face site, staged views)
    const int fbase = col * bvol + h * w;
    FieldRef hprev = fin, hnext = fin;
    if (HALO) {
        hprev.data = (void *)halo.prev;
        hnext.data = (void *)halo.next;
        const int vf = g.V / Lt;
        hprev.V = hnext.V = vf;
        hprev.stride = hnext.stride = rhs_stride(vf);
        hprev = rhs_view(hprev, rhs);
        hnext = rhs_view(hnext, rhs);
    }
    const bool prev_from_halo = HALO && t0 == 0;

    // prologue: slice t0 into image 0, and the backward t hop from t0 - 1
    if constexpr (RAG)
        slice_copy_ragged<PREC>(fin, cbase + t0 * bvol + l, img0);
    else
        slice_copy<PREC>(fin, (cbase + t0 * bvol) >> 6, img0);
    cx<R> cw0[3], cw1[3];
    {
        const int tprev = t0 == 0 ? Lt - 1 : t0 - 1;
        const int ip = cbase + tprev * bvol + l;
        cx<R> p[12];
        Spinor<PREC>::load(prev_from_halo ? hprev : fin, prev_from_halo ? fbase + l : ip, p);
        cx<R> h0[3], h1[3];
        project<3, SB>(p, h0, h1);
        const R sg = (g.antiperiodic && t0 == 0 && (!HALO || halo.first)) ? R(-1) : R(1);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            h0[c] = scale(sg, h0[c]);
            h1[c] = scale(sg, h1[c]);
        }
        cx<R> u[9];
        if constexpr (HALO && LF == PREC) {
            Link<PREC>::load(prev_from_halo ? halo.links : gauge, 3,
                             prev_from_halo ? fbase + l : ip, u);
        } else if constexpr (HALO) {
            // the entering links are float64 with 18 reals
            if (prev_from_halo)
                Link<PREC>::load(halo.links, 3, fbase + l, u);
            else
                Link<LF>::load(gauge, 3, ip, u);
        } else {
            Link<LF>::load(gauge, 3, ip, u);
        }
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
        // the slice after the slab's last one is the staged next face
        const bool next_from_halo = HALO && t + 1 == Lt;
        if constexpr (RAG)
            slice_copy_ragged<PREC>(fin, cbase + tn * bvol + l, (char *)nxt.data);
        else
            slice_copy<PREC>(next_from_halo ? hnext : fin,
                             next_from_halo ? fbase >> 6 : (cbase + tn * bvol) >> 6,
                             (char *)nxt.data);
        const int sbase = cbase + t * bvol;
        const int i = sbase + l;
        constexpr bool XPRE = XR && ((WD_XR_PREFETCH >> PREC) & 1);
        cx<R> rpre[XPRE ? 12 : 1];
        if constexpr (XPRE)
            Spinor<xr_prec_of(PREC)>::template load<WD_NT_RLOAD>(
                rhs_view(xr.r, rhs), i, rpre);
        const Nbrs nb = neighbours(g, i);
        cx<R> acc[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) acc[k] = {R(0), R(0)};
#define WD_HOP_FENCE(k) \
    if ((k) % GROUP == 0) __builtin_amdgcn_sched_barrier(0)
        hop_s<0, SF, false, PREC, LF>(gauge, fin, cur, sbase, wvol, nb.xp, i, acc);
        WD_HOP_FENCE(1);
        hop_s<0, SB, true, PREC, LF>(gauge, fin, cur, sbase, wvol, nb.xm, nb.xm, acc);
        WD_HOP_FENCE(2);
        hop_s<1, SF, false, PREC, LF>(gauge, fin, cur, sbase, wvol, nb.yp, i, acc);
        WD_HOP_FENCE(3);
        hop_s<1, SB, true, PREC, LF>(gauge, fin, cur, sbase, wvol, nb.ym, nb.ym, acc);
        WD_HOP_FENCE(4);
        hop_s<2, SF, false, PREC, LF>(gauge, fin, cur, sbase, wvol, nb.zp, i, acc);
        WD_HOP_FENCE(5);
        hop_s<2, SB, true, PREC, LF>(gauge, fin, cur, sbase, wvol, nb.zm, nb.zm, acc);
        WD_HOP_FENCE(6);
#undef WD_HOP_FENCE
        // binary16 with 12-real links: the t hops on packed halves too
        constexpr bool H2 = PREC == WD_F16 && LF == WD_F16 && WD_F16_DOT2;
        cx<R> ut[H2 ? 1 : 9];
        h2_t ut2[H2 ? 9 : 1];
        if constexpr (H2)
            Link<WD_F16>::template load_h2<WD_NT_LINK || WD_NT_LINK_T>(gauge, 3, i, ut2);
        else
            Link<LF>::template load<WD_NT_LINK || WD_NT_LINK_T>(gauge, 3, i, ut);
        // this wave's copy of the next slice has landed in LDS: the forward t
        // hop reads it at the lane's own place (the other waves' tiles are read
        // after the barrier that ends the step)
        copy_landed<PREC>();
        const bool neg_tp = g.antiperiodic && t == Lt - 1 && (!HALO || halo.last);
        cx<R> c[12];
        if constexpr (H2) {
            {
                h2_t q[12];
                float sc;
                Spinor<WD_F16>::load_raw(nxt, pl.place, q, sc);
                h2_t h0[3], h1[3];
                project_h2<3, SF>(q, h0, h1);
                cx<float> w0[3], w1[3];
                su3_mul_h2<false>(ut2, h0, w0);
                su3_mul_h2<false>(ut2, h1, w1);
                accumulate_s<3, SF>(neg_tp ? -sc : sc, w0, w1, acc);
            }
            accumulate<3, SB>(cw0, cw1, acc);
            h2_t q[12];
            float sc;
            Spinor<WD_F16>::load_raw(cur, l, q, sc);
#pragma unroll
            for (int k = 0; k < 12; ++k) c[k] = {sc * (float)q[k].x, sc * (float)q[k].y};
            // carry for slice t + 1, scaled here as the float carry is
            h2_t h0[3], h1[3];
            project_h2<3, SB>(q, h0, h1);
            su3_mul_h2<true>(ut2, h0, cw0);
            su3_mul_h2<true>(ut2, h1, cw1);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                cw0[k] = scale(sc, cw0[k]);
                cw1[k] = scale(sc, cw1[k]);
            }
        } else {
            {
                cx<R> nx[12];
                Spinor<PREC>::load(nxt, pl.place, nx);
                hop_p<3, SF, false>(nx, ut, neg_tp, acc);
            }
            accumulate<3, SB>(cw0, cw1, acc);
            Spinor<PREC>::load(cur, l, c);
            // carry for slice t + 1 (never crosses the boundary inside a chunk)
            cx<R> h0[3], h1[3];
            project<3, SB>(c, h0, h1);
            su3_mul<true>(ut, h0, cw0);
            su3_mul<true>(ut, h1, cw1);
        }
        double nrm = 0.0;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            c[k] = c[k] - scale(kappa, acc[k]);
            if (RED && !XR)
                nrm += (double)c[k].re * (double)c[k].re + (double)c[k].im * (double)c[k].im;
        }
        if constexpr (RAG && XR) pin(c);
        if constexpr (XPRE)
            nrm = xr_site_r<PREC>(xr, rhs, i, alpha, c, rpre, mine);
        else if constexpr (XR)
            nrm = xr_site<PREC>(xr, rhs, i, alpha, c, mine);
        else if constexpr (!COUT)
            Spinor<PREC>::template store<WD_NT_OUT>(fout, i, c);
        if (RED) {
            if (!mine) nrm = 0.0;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) nrm += __shfl_xor(nrm, off, 64);
            if ((tid & 63) == 0) wsum[odd][tid >> 6] = nrm;
        }
        __syncthreads();  // the current image is free for the next copy
        if constexpr (COUT) {
            // out through this wave's tile of the image
            int x, y, z, tt;
            coords_of(g, i, x, y, z, tt);
            FieldRef tile = cur;
            tile.data = (char *)cur.data +
                        __builtin_amdgcn_readfirstlane(tid >> 6) * Spinor<PREC>::kTileBytes;
            Spinor<PREC>::store(tile, tid & 63, c);
            export_tile<PREC>((double2 *)out.data,
                              mine ? (int64_t)rhs * g.V + lex_of(g, x, y, z, tt) : -1, tile);
        }
        if (RED && tid == 0) {
            double s = 0.0;
            for (int v = 0; v < (int)(blockDim.x >> 6); ++v) s += wsum[odd][v];
            red.partials[(((size_t)col * Lt + t) * nsub + h) * nrhs + rhs] = s;
        }
    }
}

static const Halo kNoHalo{nullptr, nullptr, nullptr, 0, 0, 0, 0, 1};

template <int PREC, bool DAG, bool RED, bool XR, int LF, bool COUT = false>
static void launch_tm(const March &m, const Geom &g, const void *gauge, FieldRef in, FieldRef out,
                      double kappa, const RedArgs &r, Gate gate, const XrArgs &xr,
                      hipStream_t s) {
    constexpr int G = HopGroup<PREC>::value;
    auto go = [&](auto k) {
        allow_lds(k, m.lds);
        hipLaunchKernelGGL(k, m.grid, m.bs, m.lds, s, g, gauge, in, out, kappa, r, gate, m.tch,
                           m.ncols, m.p.w, kNoHalo, xr);
    };
    if (m.p.ragged)
        go(k_dslash_tm<PREC, DAG, RED, G, false, XR, LF, COUT, true>);
    else
        go(k_dslash_tm<PREC, DAG, RED, G, false, XR, LF, COUT, false>);
}

template <int PREC, int LF = PREC>
static void launch_prec(const Geom &g, const void *gauge, double kappa, int dagger, FieldRef in,
                        FieldRef out, const RedArgs *red, Gate gate, hipStream_t s,
                        const void *g12) {
    RedArgs r{};
    if (red) r = *red;
    // the marching stencil writes one partial per part of a slice: use it
    // only when the caller's partial buffer holds them (it always does when
    // sized by reduce_partials_cap)
    March m = march_of<PREC>(g, g.bvol, in.nrhs);
    if (m.p.ragged && !red && !ragged_marches<PREC>(g, in.nrhs)) m.ok = false;
    if (m.ok && (!red || (int64_t)tm_partials(g, m.p) * in.nrhs <= red->partials_cap)) {
        auto go = [&](auto lf, const void *links) {
            constexpr int F = decltype(lf)::value;
            if (dagger && red)
                launch_tm<PREC, true, true, false, F>(m, g, links, in, out, kappa, r, gate, {}, s);
            else if (dagger)
                launch_tm<PREC, true, false, false, F>(m, g, links, in, out, kappa, r, gate, {}, s);
            else if (red)
                launch_tm<PREC, false, true, false, F>(m, g, links, in, out, kappa, r, gate, {}, s);
            else
                launch_tm<PREC, false, false, false, F>(m, g, links, in, out, kappa, r, gate, {}, s);
        };
        if constexpr (PREC == WD_F64) {
            if (g12)
                go(Int<kLinkF64R12>{}, g12);
            else
                go(Int<WD_F64>{}, gauge);
        } else {
            go(Int<LF>{}, gauge);
        }
        if (red) launch_finalize(r, tm_partials(g, m.p), s);
        return;
    }
    const int nb = site_blocks(g.V);
    const dim3 grid(nb * in.nrhs), bs(kSiteBlock);
    constexpr int G = HopGroup<PREC>::value;
    if (dagger) {
        if (red)
            hipLaunchKernelGGL((k_dslash<PREC, true, true, G, LF>), grid, bs, 0, s, g, gauge, in, out, kappa, r, gate);
        else
            hipLaunchKernelGGL((k_dslash<PREC, true, false, G, LF>), grid, bs, 0, s, g, gauge, in, out, kappa, r, gate);
    } else {
        if (red)
            hipLaunchKernelGGL((k_dslash<PREC, false, true, G, LF>), grid, bs, 0, s, g, gauge, in, out, kappa, r, gate);
        else
            hipLaunchKernelGGL((k_dslash<PREC, false, false, G, LF>), grid, bs, 0, s, g, gauge, in, out, kappa, r, gate);
    }
    if (red) launch_finalize(r, nb, s);
}

void launch_dslash(const Geom &g, const void *gauge, double kappa, int dagger, FieldRef in,
                   FieldRef out, const RedArgs *red, Gate gate, hipStream_t s, const void *g12) {
    switch (in.prec) {
        case WD_F64: launch_prec<WD_F64>(g, gauge, kappa, dagger, in, out, red, gate, s, g12); break;
        case WD_F32: launch_prec<WD_F32>(g, gauge, kappa, dagger, in, out, red, gate, s, nullptr); break;
        default:
            if (g.f16_links8)
                launch_prec<WD_F16, kLinkF16R8>(g, gauge, kappa, dagger, in, out, red, gate, s,
                                                nullptr);
            else
                launch_prec<WD_F16>(g, gauge, kappa, dagger, in, out, red, gate, s, nullptr);
            break;
    }
}

// the plain stencil with a canonical float64 output (float32, binary16)
template <int PREC, bool DAG, int LF>
static void launch_canon_out(const Geom &g, const void *gauge, double kappa, FieldRef in,
                             FieldRef out, hipStream_t s) {
    constexpr int G = HopGroup<PREC>::value;
    const Gate none{nullptr, 0, GATE_ACTIVE};
    // The marching binary16 stencil scales its carried t hop before it is
    // summed, one lane per site while it is: the last binary16 bits differ.
    // On slices that are no whole tiles a plain application keeps the form it
    // always had (18^3 x 36, 2 rhs: 70.9 against 70.2 us); a solve's stencils
    // march.
    March m = march_of<PREC>(g, g.bvol, in.nrhs);
    if (m.p.ragged && !ragged_marches<PREC>(g, in.nrhs)) m.ok = false;
    if (m.ok) {
        launch_tm<PREC, DAG, false, false, LF, true>(m, g, gauge, in, out, kappa, RedArgs{}, none,
                                                     {}, s);
        return;
    }
    hipLaunchKernelGGL((k_dslash<PREC, DAG, false, G, LF, true>),
                       dim3(site_blocks(g.V) * in.nrhs), dim3(kSiteBlock), 0, s, g, gauge, in, out,
                       kappa, RedArgs{}, none);
}

void launch_dslash_canon(const Geom &g, const void *gauge, double kappa, int dagger, FieldRef in,
                         double *out, hipStream_t s) {
    FieldRef o{};
    o.data = out;
    if (in.prec == WD_F32) {
        if (dagger)
            launch_canon_out<WD_F32, true, WD_F32>(g, gauge, kappa, in, o, s);
        else
            launch_canon_out<WD_F32, false, WD_F32>(g, gauge, kappa, in, o, s);
    } else if (g.f16_links8) {
        if (dagger)
            launch_canon_out<WD_F16, true, kLinkF16R8>(g, gauge, kappa, in, o, s);
        else
            launch_canon_out<WD_F16, false, kLinkF16R8>(g, gauge, kappa, in, o, s);
    } else {
        if (dagger)
            launch_canon_out<WD_F16, true, WD_F16>(g, gauge, kappa, in, o, s);
        else
            launch_canon_out<WD_F16, false, WD_F16>(g, gauge, kappa, in, o, s);
    }
}

template <int PREC>
static bool xr_ok(const Geom &g, int nrhs, int partials_cap) {
    const March m = march_of<PREC>(g, g.bvol, nrhs);
    return m.ok && (int64_t)tm_partials(g, m.p) * nrhs <= partials_cap;
}

bool dslash_xr_supported(const Geom &g, int prec, int nrhs, int partials_cap) {
    switch (prec) {
        case WD_F64: return xr_ok<WD_F64>(g, nrhs, partials_cap);
        case WD_F32: return xr_ok<WD_F32>(g, nrhs, partials_cap);
        default: return xr_ok<WD_F16>(g, nrhs, partials_cap);
    }
}

void dslash_partials(const Geom &g, int prec, int nrhs, int *nb, int *threads) {
    const March m = prec == WD_F64   ? march_of<WD_F64>(g, g.bvol, nrhs)
                    : prec == WD_F32 ? march_of<WD_F32>(g, g.bvol, nrhs)
                                     : march_of<WD_F16>(g, g.bvol, nrhs);
    *nb = m.ok ? tm_partials(g, m.p) : site_blocks(g.V);
    *threads = m.ok ? m.p.threads : kSiteBlock;
}

template <int PREC, int LF = PREC>
static bool xr_prec(const Geom &g, const void *gauge, double kappa, int dagger, FieldRef in,
                    const XrArgs &xr, const RedArgs &red, Gate gate, hipStream_t s) {
    if (!xr_ok<PREC>(g, in.nrhs, red.partials_cap)) return false;
    const March m = march_of<PREC>(g, g.bvol, in.nrhs);
    if (dagger)
        launch_tm<PREC, true, true, true, LF>(m, g, gauge, in, FieldRef{}, kappa, red, gate, xr, s);
    else
        launch_tm<PREC, false, true, true, LF>(m, g, gauge, in, FieldRef{}, kappa, red, gate, xr, s);
    launch_finalize(red, tm_partials(g, m.p), s);
    return true;
}

bool launch_dslash_xr(const Geom &g, const void *gauge, double kappa, int dagger, FieldRef in,
                      const XrArgs &xr, const RedArgs &red, Gate gate, hipStream_t s,
                      const void *g12) {
    switch (in.prec) {
        case WD_F64:
            if (g12)
                return xr_prec<WD_F64, kLinkF64R12>(g, g12, kappa, dagger, in, xr, red, gate, s);
            return xr_prec<WD_F64>(g, gauge, kappa, dagger, in, xr, red, gate, s);
        case WD_F32: return xr_prec<WD_F32>(g, gauge, kappa, dagger, in, xr, red, gate, s);
        default:
            if (g.f16_links8)
                return xr_prec<WD_F16, kLinkF16R8>(g, gauge, kappa, dagger, in, xr, red, gate, s);
            return xr_prec<WD_F16>(g, gauge, kappa, dagger, in, xr, red, gate, s);
    }
}

// ------------------------------------------------------------------ halo exchange

// Faces of a t-slab for its neighbours (float64, wire format): one lane per
// face site and rhs.  to_prev: (1 + SF gamma_t) psi(x, 0), the projection
// the previous slab's forward t hop applies; to_next: (1 + SB gamma_t)
// psi(x, Lt-1) for the next slab's backward t hop (which multiplies it by
// U_t(x, Lt-1)^dag, a link the next slab holds as its entering links).
template <bool DAG>
__global__ void __launch_bounds__(256) k_halo_pack(Geom g, FieldRef in, double2 *__restrict__ to_prev,
                                                   double2 *__restrict__ to_next) {
    constexpr int SF = DAG ? +1 : -1;
    constexpr int SB = -SF;
    const int Lt = g.L[3];
    const int vf = g.V / Lt;
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= vf) return;
    const int rhs = blockIdx.y;
    const FieldRef fin = rhs_view(in, rhs);
    const int col = f / g.bvol, loc = f - col * g.bvol;
    const int i0 = col * Lt * g.bvol + loc;  // slice 0
    const int il = i0 + (Lt - 1) * g.bvol;   // slice Lt - 1
    const size_t fofs = (size_t)rhs * 6 * vf;
    cx<double> p[12], h0[3], h1[3];
    Spinor<WD_F64>::load(fin, i0, p);
    project<3, SF>(p, h0, h1);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        to_prev[fofs + (size_t)c * vf + f] = make_double2(h0[c].re, h0[c].im);
        to_prev[fofs + (size_t)(3 + c) * vf + f] = make_double2(h1[c].re, h1[c].im);
    }
    Spinor<WD_F64>::load(fin, il, p);
    project<3, SB>(p, h0, h1);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        to_next[fofs + (size_t)c * vf + f] = make_double2(h0[c].re, h0[c].im);
        to_next[fofs + (size_t)(3 + c) * vf + f] = make_double2(h1[c].re, h1[c].im);
    }
}

void launch_halo_pack(const Geom &g, int dagger, FieldRef in, double *to_prev, double *to_next,
                      hipStream_t s) {
    const dim3 grid(blocks_for(g.V / g.L[3], 256), in.nrhs), bs(256);
    if (dagger)
        hipLaunchKernelGGL(k_halo_pack<true>, grid, bs, 0, s, g, in, (double2 *)to_prev,
                           (double2 *)to_next);
    else
        hipLaunchKernelGGL(k_halo_pack<false>, grid, bs, 0, s, g, in, (double2 *)to_prev,
                           (double2 *)to_next);
}

// wire-format face -> spinor tiles: spins 0, 1 = the half-spinor, spins 2, 3
// zero (the t projectors then return the half-spinor exactly)
__global__ void __launch_bounds__(256) k_halo_stage(const double2 *__restrict__ wire, FieldRef st,
                                                    int vf) {
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= vf) return;
    const int rhs = blockIdx.y;
    const size_t fofs = (size_t)rhs * 6 * vf;
    cx<double> v[12];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const double2 d = wire[fofs + (size_t)k * vf + f];
        v[k] = {d.x, d.y};
        v[6 + k] = {0.0, 0.0};
    }
    Spinor<WD_F64>::store(rhs_view(st, rhs), f, v);
}

void launch_halo_stage(const Geom &g, const double *wire, FieldRef staged, hipStream_t s) {
    const int vf = g.V / g.L[3];
    hipLaunchKernelGGL(k_halo_stage, dim3(blocks_for(vf, 256), staged.nrhs), dim3(256), 0, s,
                       (const double2 *)wire, staged, vf);
}

// canonical U_t(x, -1) over the (x, y, z) of a face -> gauge tiles over face
// sites (mu = 3 planes; the others are not read)
__global__ void __launch_bounds__(256) k_halo_links(Geom g, const double2 *__restrict__ canon,
                                                    void *__restrict__ links) {
    const int vf = g.V / g.L[3];
    const int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= vf) return;
    const int col = f / g.bvol, loc = f - col * g.bvol;
    int x, y, z, t;
    coords_of(g, col * g.L[3] * g.bvol + loc, x, y, z, t);
    const double2 *src = canon + (size_t)(x + g.L[0] * (y + g.L[1] * z)) * 9;
    cx<double> u[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) u[k] = {src[k].x, src[k].y};
    Link<WD_F64>::store(links, 3, f, u);
}

void launch_halo_links(const Geom &g, const double *canon, void *links, hipStream_t s) {
    const int vf = g.V / g.L[3];
    hipLaunchKernelGGL(k_halo_links, dim3(blocks_for(vf, 256)), dim3(256), 0, s, g,
                       (const double2 *)canon, links);
}

// (slabs whose bricks are no whole tiles are refused)
bool halo_supported(const Geom &g) {
    return tm_eligible(g) && 2 * slice_bytes<WD_F64>(tm_wvol(g, WD_F64)) + 64 <= max_lds_per_block();
}

template <int LF>
static void launch_halo_lf(const Geom &g, const void *gauge, double kappa, int dagger,
                           FieldRef in, FieldRef out, const Halo &region, hipStream_t s) {
    const PartShape p = tm_part(g, WD_F64);
    const int ncols = g.V / (g.L[3] * g.bvol);
    const size_t lds = 2 * slice_bytes<WD_F64>(p.threads);
    int tch = tm_chunk(g, in.nrhs * p.nsub);
    // (a slab in two launches keeps short chunks: the longer the ends' chunks,
    // the less is left to run while the faces travel)
    if (region.region == 0 && env_chunk() <= 0)
        tch = balanced_chunk(g.L[3], (int64_t)ncols * p.nsub * in.nrhs,
                             wgs_at_once(WD_F64, p.threads, lds), tch,
                             chunk_gain(WD_F64, in.nrhs));
    // chunks of this launch: all; the interior ones (neither slice 0 nor
    // Lt - 1: no staged face is read); or the one or two holding the ends
    const int nch = (g.L[3] + tch - 1) / tch;
    Halo halo = region;
    int count = nch;
    halo.cfirst = 0;
    halo.cstep = 1;
    if (region.region == 1) {
        count = nch - 2;
        halo.cfirst = 1;
    } else if (region.region == 2) {
        count = nch < 2 ? nch : 2;
        halo.cstep = nch - 1 > 0 ? nch - 1 : 1;
    }
    if (count <= 0) return;
    const dim3 grid(ncols * count * p.nsub * in.nrhs), bs(p.threads);
    constexpr int G = HopGroup<WD_F64>::value;
    const Gate none{nullptr, 0, GATE_ACTIVE};
    auto go = [&](auto k) {
        allow_lds(k, lds);
        hipLaunchKernelGGL(k, grid, bs, lds, s, g, gauge, in, out, kappa, RedArgs{}, none, tch,
                           ncols, p.w, halo, XrArgs{});
    };
    if (dagger)
        go(k_dslash_tm<WD_F64, true, false, G, true, false, LF>);
    else
        go(k_dslash_tm<WD_F64, false, false, G, true, false, LF>);
}

void launch_dslash_halo(const Geom &g, const void *gauge, double kappa, int dagger, FieldRef in,
                        FieldRef out, const Halo &halo, hipStream_t s, const void *g12) {
    if (g12)
        launch_halo_lf<kLinkF64R12>(g, g12, kappa, dagger, in, out, halo, s);
    else
        launch_halo_lf<WD_F64>(g, gauge, kappa, dagger, in, out, halo, s);
}

}  // namespace wd
