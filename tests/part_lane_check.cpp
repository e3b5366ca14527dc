// Host check of what a lane of a marching workgroup reads before the barrier
// that ends a step: its own entry, from a place of the LDS image that its own
// wave has filled; for every slice size, with last parts that leave whole waves
// of their workgroup without a site.  Exit code 0 on success.
#include <cstdio>
#include <vector>

#include "apply.hpp"

// parts of w of n entries, by `threads` lanes each: the number of whole idle
// waves, -1 if a lane's place is not its own wave's or does not hold its entry
static int idle_waves(int n, int w, int threads) {
    int idle = 0;
    for (int h = 0; h * w < n; ++h) {
        const int m = n - h * w < w ? n - h * w : w;  // as the kernels cut them
        // the copy: lane tid brings the entry it works on to place tid
        std::vector<int> img(threads);
        for (int tid = 0; tid < threads; ++tid) img[tid] = wd::part_lane(tid, m).l;
        for (int tid = 0; tid < threads; ++tid) {
            const wd::PartLane p = wd::part_lane(tid, m);
            if (p.l != (tid < m ? tid : m - 1)) return -1;
            if (p.place < 0 || p.place >= threads || p.place / 64 != tid / 64) return -1;
            if (img[p.place] != p.l) return -1;
            if (tid % 64 == 0 && tid >= m) ++idle;
        }
    }
    return idle;
}

int main() {
    int fails = 0, found[4] = {0, 0, 0, 0};
    for (int n = 1; n <= 4200; ++n) {
        for (int prec = 0; prec < 3; ++prec) {
            const wd::PartShape p = wd::part_shape(n, prec);
            const int k = idle_waves(n, p.w, p.threads);
            if (k < 0) ++fails;
            found[prec] += k > 0;
        }
        wd::Geom g{};
        g.bvol = n;
        g.L[3] = 2;
        g.V = 2 * n;
        const wd::ApplyShape a = wd::apply_shape(g, 1);
        const int k = idle_waves(n, a.w, (a.w + 63) / 64 * 64);
        if (k < 0) ++fails;
        found[3] += k > 0;
    }
    for (int k : found)
        if (!k) ++fails;
    // the lattices of the GPU tests leave a wave idle: (brick, or the default
    // one), full slice or half, precision
    struct Case { int L[4], t[3], half, prec; };
    const Case cs[] = {{{34, 34, 4, 4}, {0, 0, 0}, 0, WD_F32},
                       {{386, 2, 2, 4}, {386, 1, 1}, 0, WD_F64},
                       {{514, 2, 2, 12}, {514, 1, 1}, 1, WD_F64}};
    for (const Case &c : cs) {
        wd::Geom g{};
        g.V = 1;
        for (int k = 0; k < 4; ++k) g.V *= g.L[k] = c.L[k];
        if (c.t[0])
            g.bvol = c.t[0] * c.t[1] * c.t[2];
        else
            wd::choose_bricks(g);
        const int n = c.half ? g.bvol / 2 : g.bvol;
        const wd::PartShape p = wd::geom_part(g, n, c.prec);
        const int k = idle_waves(n, p.w, p.threads);
        printf("%dx%dx%dx%d: slice %d, parts of %d in %d lanes, %d idle waves\n", c.L[0], c.L[1],
               c.L[2], c.L[3], n, p.w, p.threads, k);
        if (k < 1) ++fails;
    }
    printf(fails ? "FAIL %d\n" : "OK\n", fails);
    return fails ? 1 : 0;
}
