// Host check of the marching stencils' parts where a brick slice is no whole
// number of tiles: every site of a slice once, workgroups within the launch
// limits, room for every partial sum, and the default bricks of such lattices.
// Exit code 0 on success.
#include <cstdio>
#include <vector>

#include "runtime.hpp"

int main() {
    int fails = 0;
    for (int n = 1; n <= 2100; ++n)
        for (int prec = 0; prec < 3; ++prec) {
            const wd::PartShape p = wd::part_shape(n, prec);
            if (p.ragged != (n % 64 != 0)) ++fails;
            if (p.threads % 64 || p.threads < p.w || p.threads - p.w >= 64 ||
                p.threads > wd::kTmMaxBlock)
                ++fails;
            std::vector<int> seen(n, 0);
            for (int h = 0; h < p.nsub; ++h) {
                const int m = n - h * p.w < p.w ? n - h * p.w : p.w;  // as the kernels cut them
                if (m < 1) ++fails;
                for (int l = 0; l < p.threads; ++l) {
                    const int s = h * p.w + (l < m ? l : m - 1);
                    if (s < 0 || s >= n) ++fails;
                    else if (l < m) seen[s]++;
                }
            }
            for (int s = 0; s < n; ++s)
                if (seen[s] != 1) ++fails;
        }
    const int dims[][4] = {{6, 10, 14, 4}, {10, 10, 10, 10}, {18, 18, 18, 36}, {30, 30, 30, 60},
                           {22, 22, 22, 8}, {2, 4, 2, 6}, {2, 2, 2, 2}, {26, 14, 10, 16},
                           {34, 38, 46, 6}, {1000, 2, 6, 4}, {14, 6, 6, 6}, {40, 38, 30, 82}};
    for (const auto &d : dims) {
        wd::Geom g{};
        g.V = 1;
        for (int k = 0; k < 4; ++k) g.V *= g.L[k] = d[k];
        wd::choose_bricks(g);
        if (g.L[0] % g.tx || g.L[1] % g.ty || g.L[2] % g.tz || g.bvol != g.tx * g.ty * g.tz ||
            (g.tx & 1))
            ++fails;
        printf("%dx%dx%dx%d: %dx%dx%d\n", d[0], d[1], d[2], d[3], g.tx, g.ty, g.tz);
        for (int prec = 0; prec < 3; ++prec)
            for (int nrhs = 1; nrhs <= 12; ++nrhs) {
                const long long cap = wd::reduce_partials_cap(g, nrhs);
                if (wd::marches(g.bvol) &&
                    (long long)wd::tm_partials(g, wd::tm_part(g, prec)) * nrhs > cap)
                    ++fails;
                if (wd::marches(g.bvol / 2) &&
                    (long long)wd::tm_partials(g, wd::eo_part(g, prec)) * nrhs > cap)
                    ++fails;
            }
    }
    // chunk lengths: in range; c0 itself where one round holds everything; never
    // one that the count behind the choice ranks behind c0 (whole rounds only)
    for (int Lt = 2; Lt <= 96; Lt += 2)
        for (long long parts = 1; parts <= 6000; parts = parts * 3 / 2 + 1)
            for (int at : {256, 512, 768, 1024, 1536})
                for (int c0 : {1, 2, 5, Lt}) {
                    if (c0 > Lt) continue;
                    const int c = wd::balanced_chunk(Lt, parts, at, c0, 1.0 / 32);
                    if (c < 1 || c > Lt) ++fails;
                    if (wd::balanced_chunk(Lt, parts, at, c0, 1.0) != c0) ++fails;
                    // the least count over all lengths
                    int best = c0;
                    auto cost = [&](int k) {
                        const long long wgs = parts * ((Lt + k - 1) / k);
                        const double last = (double)(wgs % at) / at;
                        return ((double)(wgs / at) + (last > 0 ? 0.35 + 0.65 * last : 0.0)) *
                               (k + 0.5);
                    };
                    for (int k = 1; k <= Lt; ++k)
                        if (cost(k) < cost(best)) best = k;
                    if (c != (cost(best) < (1.0 - 1.0 / 32) * cost(c0) ? best : c0)) ++fails;
                    const long long r0 = (parts * ((Lt + c0 - 1) / c0) + at - 1) / at;
                    const long long r = (parts * ((Lt + c - 1) / c) + at - 1) / at;
                    if (c > c0 && r >= r0) ++fails;
                }
    printf(fails ? "FAIL %d\n" : "OK\n", fails);
    return fails ? 1 : 0;
}
