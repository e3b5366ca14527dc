// Launch shape of the stencil on canonical spinors (apply.hip).
#pragma once

#include "wd_internal.hpp"

namespace wd {

constexpr int kApplySiteBlock = 64;
// sites per marching workgroup, at most: two workgroups of 192, with two 39
// KiB images each, share a CU.  384 (one workgroup per CU) measured 2.01
// against 2.04 ms at 48^3 x 96 but 371 against 339 us at 30^3 x 60 (12-real
// links), whose bricks fill parts of 192 better.
constexpr int kApplyPart = 192;

// The marching form, else one lane per site.  The line: 12^3 x 24 (41472
// sites) 12.2 us one lane per site against 12.9 marching, 16^3 x 32 (131072)
// 36.5 against 30.5.  A brick slice of less than half a wave leaves the
// marching form's lanes idle.
inline bool apply_march(const Geom &g, int nrhs) {
    return g.bvol >= 32 && (int64_t)g.V * nrhs >= 65536;
}

// a workgroup's two slice images: tiles of 64 sites, 208 bytes apart
constexpr int kImgTile = 64 * 208;
inline size_t apply_lds(int threads) { return 2 * (size_t)(threads / 64) * kImgTile; }

// launch shape of the marching form
struct ApplyShape {
    int w, nsub;  // sites per part of a brick slice, parts
    int ncols, tchunk, nchunks;
};

inline ApplyShape apply_shape(const Geom &g, int nrhs) {
    ApplyShape a{};
    const int Lt = g.L[3];
    a.ncols = g.V / (Lt * g.bvol);
    a.nsub = (g.bvol + kApplyPart - 1) / kApplyPart;
    a.w = (g.bvol + a.nsub - 1) / a.nsub;
    static const int env = [] {
        const char *e = getenv("WD_TCHUNK");
        return e ? atoi(e) : 0;
    }();
    a.tchunk = tm_chunk_len(g, nrhs * a.nsub, env);
    if (env <= 0) {
        const int threads = (a.w + 63) / 64 * 64;
        a.tchunk = balanced_chunk(Lt, (int64_t)a.ncols * a.nsub * nrhs,
                                  wgs_at_once(WD_F64, threads, apply_lds(threads)), a.tchunk,
                                  chunk_gain(WD_F64, nrhs));
    }
    a.nchunks = (Lt + a.tchunk - 1) / a.tchunk;
    return a;
}

}  // namespace wd
