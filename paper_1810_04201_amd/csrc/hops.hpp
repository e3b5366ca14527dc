// Spin projection, link multiplication and reconstruction of one hop, shared by
// the stencils on the internal layout (dslash.hip) and on the canonical one
// (apply.hip).
#pragma once

#include "device.hpp"

#ifndef WD_XCD_REMAP
#define WD_XCD_REMAP 1
#endif

namespace wd {

// a compile-time integer as an argument
template <int N>
struct Int {
    static constexpr int value = N;
};

template <int MU, int S, typename R>
__device__ __forceinline__ void project(const cx<R> p[12], cx<R> h0[3], cx<R> h1[3]) {
    // p[3*spin + colour]
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const cx<R> a0 = p[c], a1 = p[3 + c], a2 = p[6 + c], a3 = p[9 + c];
        if (MU == 0) {
            h0[c] = S > 0 ? a0 + times_i(a3) : a0 - times_i(a3);
            h1[c] = S > 0 ? a1 + times_i(a2) : a1 - times_i(a2);
        } else if (MU == 1) {
            h0[c] = S > 0 ? a0 - a3 : a0 + a3;
            h1[c] = S > 0 ? a1 + a2 : a1 - a2;
        } else if (MU == 2) {
            h0[c] = S > 0 ? a0 + times_i(a2) : a0 - times_i(a2);
            h1[c] = S > 0 ? a1 - times_i(a3) : a1 + times_i(a3);
        } else {
            h0[c] = S > 0 ? a0 + a2 : a0 - a2;
            h1[c] = S > 0 ? a1 + a3 : a1 - a3;
        }
    }
}

template <int MU, int S, typename R>
__device__ __forceinline__ void accumulate(const cx<R> w0[3], const cx<R> w1[3], cx<R> acc[12]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        acc[c] = acc[c] + w0[c];
        acc[3 + c] = acc[3 + c] + w1[c];
        if (MU == 0) {
            // lower: -s i w1, -s i w0
            acc[6 + c] = S > 0 ? acc[6 + c] - times_i(w1[c]) : acc[6 + c] + times_i(w1[c]);
            acc[9 + c] = S > 0 ? acc[9 + c] - times_i(w0[c]) : acc[9 + c] + times_i(w0[c]);
        } else if (MU == 1) {
            // lower: s w1, -s w0
            acc[6 + c] = S > 0 ? acc[6 + c] + w1[c] : acc[6 + c] - w1[c];
            acc[9 + c] = S > 0 ? acc[9 + c] - w0[c] : acc[9 + c] + w0[c];
        } else if (MU == 2) {
            // lower: -s i w0, s i w1
            acc[6 + c] = S > 0 ? acc[6 + c] - times_i(w0[c]) : acc[6 + c] + times_i(w0[c]);
            acc[9 + c] = S > 0 ? acc[9 + c] + times_i(w1[c]) : acc[9 + c] - times_i(w1[c]);
        } else {
            // lower: s w0, s w1
            acc[6 + c] = S > 0 ? acc[6 + c] + w0[c] : acc[6 + c] - w0[c];
            acc[9 + c] = S > 0 ? acc[9 + c] + w1[c] : acc[9 + c] - w1[c];
        }
    }
}

// w = U h  or  w = U^dag h
template <bool ADJ, typename R>
__device__ __forceinline__ void su3_mul(const cx<R> u[9], const cx<R> h[3], cx<R> w[3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        cx<R> s = {R(0), R(0)};
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            if (ADJ)
                s = cfmac(u[3 * b + a], h[b], s);  // conj(U[b][a]) h[b]
            else
                s = cfma(u[3 * a + b], h[b], s);   // U[a][b] h[b]
        }
        w[a] = s;
    }
}

// Workgroups are dealt round-robin to the 8 XCDs (each with its own L2).
// With WD_XCD_REMAP each XCD instead walks one contiguous run of logical
// blocks, so that neighbours within a few thousand sites share an L2.
__device__ __forceinline__ int logical_block() {
#if WD_XCD_REMAP
    const int nb = gridDim.x, b = blockIdx.x;
    const int x = b & 7, i = b >> 3;
    const int q = nb >> 3, r = nb & 7;
    return x * q + (x < r ? x : r) + i;
#else
    return blockIdx.x;
#endif
}

// one hop with the neighbour spinor and the link already in registers
template <int MU, int S, bool BWD, typename R>
__device__ __forceinline__ void hop_p(const cx<R> p[12], const cx<R> u[9], bool negate,
                                      cx<R> acc[12]) {
    cx<R> h0[3], h1[3];
    project<MU, S>(p, h0, h1);
    const R sg = negate ? R(-1) : R(1);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        h0[c] = scale(sg, h0[c]);
        h1[c] = scale(sg, h1[c]);
    }
    cx<R> w0[3], w1[3];
    su3_mul<BWD>(u, h0, w0);
    su3_mul<BWD>(u, h1, w1);
    accumulate<MU, S>(w0, w1, acc);
}

// Orders this wave's LDS accesses around an exchange between its lanes (the
// hardware keeps a wave's LDS accesses in order; the compiler must too).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ------------------------------------------------------------------ canonical spinors

constexpr int kSiteBytes = 192;  // a canonical spinor: 24 float64

// The 64 sites of a wave's LDS tile (field format PREC, entry = lane) to the
// canonical field f: what exporting them from a field gives.  The lanes read
// the tile one 16-byte element of the output after the other, so that every
// store instruction writes consecutive memory.  24^3 x 48, 12 rhs in float32,
// with the import before it: 1.18 ms, where three passes take 1.49 and stores
// element by element per lane, 192 bytes apart, 1.52.
// site: the canonical index of the lane's own site in f, -1 for none.
template <int PREC>
__device__ __forceinline__ void export_tile(double2 *f, int64_t site, const FieldRef &tile) {
    int lane = (int)(threadIdx.x & 63);
    // opaque, so that nothing built from it is kept in registers between the
    // steps of a marching kernel
    asm volatile("" : "+v"(lane));
    wave_lds_sync();
    const int lo = (int)(uint32_t)site, hi = (int)(site >> 32);
#pragma unroll
    for (int j = 0; j < 12; ++j) {
        const int e = j * 64 + lane, src = e / 12, k = e - src * 12;
        const int64_t st = ((int64_t)__shfl(hi, src, 64) << 32) | (uint32_t)__shfl(lo, src, 64);
        d2_t o;
        if constexpr (PREC == WD_F16) {
            const float sc = *Spinor<WD_F16>::scale_ptr(tile, src);
            const h2_t q = *(const h2_t *)(tile_elem(tile.data, Spinor<WD_F16>::kTileBytes, src,
                                                     k >> 2) + (k & 3) * 4);
            o = d2_t{(double)(sc * (float)q.x), (double)(sc * (float)q.y)};
        } else if constexpr (PREC == WD_F32) {
            const float *q = (const float *)(tile_elem(tile.data, Spinor<WD_F32>::kTileBytes, src,
                                                       k >> 1) + (k & 1) * 8);
            o = d2_t{(double)q[0], (double)q[1]};
        } else {
            o = *(const d2_t *)tile_elem(tile.data, Spinor<WD_F64>::kTileBytes, src, k);
        }
        if (st >= 0) *(d2_t *)((char *)f + st * kSiteBytes + k * 16) = o;
    }
    wave_lds_sync();
}

// The same for 64 entries of an even half field: each result to its even site,
// zero to the odd site beside it in x (the two are 384 consecutive bytes).  The
// Schur operator is three launches with it instead of six: 30^3 x 60 float32 461
// -> 345 us, 48^3 x 96 float64 4.58 -> 3.48 ms.
// site: the canonical index of the pair's first site (even x) in f, -1 for none;
// odd: 1 where the even-parity site is the second.  PREC float64 too.
template <int PREC>
__device__ __forceinline__ void export_tile_pairs(double2 *f, int64_t site, int odd,
                                                  const FieldRef &tile) {
    int lane = (int)(threadIdx.x & 63);
    asm volatile("" : "+v"(lane));  // (see export_tile)
    wave_lds_sync();
    const int lo = (int)(uint32_t)site, hi = (int)(site >> 32);
#pragma unroll
    for (int j = 0; j < 24; ++j) {
        const int e = j * 64 + lane, src = e / 24, k2 = e - src * 24;
        const int second = k2 >= 12, k = second ? k2 - 12 : k2;
        const int64_t st = ((int64_t)__shfl(hi, src, 64) << 32) | (uint32_t)__shfl(lo, src, 64);
        const bool value = __shfl(odd, src, 64) == second;
        d2_t o;
        if constexpr (PREC == WD_F16) {
            const float sc = *Spinor<WD_F16>::scale_ptr(tile, src);
            const h2_t q = *(const h2_t *)(tile_elem(tile.data, Spinor<WD_F16>::kTileBytes, src,
                                                     k >> 2) + (k & 3) * 4);
            o = d2_t{(double)(sc * (float)q.x), (double)(sc * (float)q.y)};
        } else if constexpr (PREC == WD_F32) {
            const float *q = (const float *)(tile_elem(tile.data, Spinor<WD_F32>::kTileBytes, src,
                                                       k >> 1) + (k & 1) * 8);
            o = d2_t{(double)q[0], (double)q[1]};
        } else {
            o = *(const d2_t *)tile_elem(tile.data, Spinor<WD_F64>::kTileBytes, src, k);
        }
        if (!value) o = d2_t{0.0, 0.0};
        if (st >= 0) *(d2_t *)((char *)f + st * kSiteBytes + k2 * 16) = o;
    }
    wave_lds_sync();
}

}  // namespace wd
