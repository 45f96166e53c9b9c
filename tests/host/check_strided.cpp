// Host check of the one-pass strided kernels' index arithmetic: over every
// workgroup, unit and lane, the pairs that the two phases attend are the merged
// strided set (Sec. 4.3), each exactly once, from the queries' side and from the
// keys'; every row is owned by one class unit; no index leaves the sequence.
#include <cstdio>
#include <vector>

#include "sa_strided.h"

static int fail(const char* what, int n, int l) {
    std::printf("fail: %s n=%d l=%d\n", what, n, l);
    return 1;
}

int main() {
    long long checked = 0;
    for (int n : {16, 48, 112, 128, 256, 272, 304, 528})
        for (int l : {1, 2, 7, 8, 12, 15, 16, 17, 31, 32, 33, 40, 64, 100, 111, 255, 256, 300, 600}) {
            sa::AttnArgs a{};
            a.n = n;
            a.l = l;
            a.batch = 1;
            a.heads = 3;
            a.ss = 64;
            std::vector<int> by_query((size_t)n * n, 0), by_key((size_t)n * n, 0), owned(3 * n, 0);
            const uint32_t groups = (uint32_t)((sa::strided_tiles(a) + 7) / 8 * 8);
            for (uint32_t L = 0; L < groups; ++L) {
                sa::STile t;
                if (!sa::strided_tile(a, L, &t)) continue;
                if (t.b != 0 || t.h < 0 || t.h > 2) return fail("head", n, l);
                for (int cls = 0; cls < 2; ++cls)
                    for (int u = 0; u < 16; ++u)
                        for (int r = 0; r < 16; ++r)
                            for (int keys = 0; keys < 2; ++keys) {
                                const sa::Walk w = keys ? sa::key_walk(a, t, cls, u, r) : sa::query_walk(a, t, cls, u, r);
                                if (!w.on) continue;
                                const int step = cls ? l : 1, start = cls ? t.r0 + u : 0;  // row of index x: start + x step
                                if (w.at != (int64_t)start * a.ss || w.stride != (int64_t)step * a.ss || w.stat != start ||
                                    w.stat_stride != step)
                                    return fail("rows", n, l);
                                if (w.own > w.own_last || start + w.own_last * step >= n || w.own < 0)
                                    return fail("own rows", n, l);
                                // rows past the last, and in the band those of the next step, are not this unit's
                                const bool mine = w.own + r <= w.own_last && (cls || t.r0 + r < l);
                                const int row = start + (w.own + r) * step;
                                if (cls && mine && !keys) ++owned[t.h * n + row];
                                for (int c = 0; c < (w.count + 31) / 32; ++c) {
                                    const int first = w.first + 32 * c;
                                    if (first < 0 || first > w.last || start + w.last * step >= n)
                                        return fail("chunk", n, l);
                                    const bool full = 32 * c >= w.full_lo && 32 * c + 31 <= w.full_hi;
                                    for (int x = 0; x < 32; ++x) {
                                        const bool on = 32 * c + x >= w.lo && 32 * c + x <= w.hi;
                                        if (full && mine && !on) return fail("full", n, l);
                                        if (!on || !mine || t.h != 1) continue;
                                        if (first + x > w.last) return fail("attended past the last", n, l);
                                        const int other = start + (first + x) * step;
                                        ++(keys ? by_key[(size_t)other * n + row] : by_query[(size_t)row * n + other]);
                                        ++checked;
                                    }
                                }
                                // a walk's chunks reach every attended index
                                if (mine && w.hi >= w.lo && w.hi >= (w.count + 31) / 32 * 32) return fail("reach", n, l);
                            }
            }
            for (int x : owned)
                if (x != 1) return fail("owned", n, l);
            for (int i = 0; i < n; ++i)
                for (int j = 0; j < n; ++j) {
                    const int want = j <= i && (i - j <= l || (i - j) % l == 0) ? 1 : 0;
                    if (by_query[(size_t)i * n + j] != want) return fail("queries", n, l);
                    if (by_key[(size_t)i * n + j] != want) return fail("keys", n, l);
                }
        }
    // a launch holds fewer than 2^32 threads: shares of eight workgroups of up to 1,024
    for (int tiles = (1 << 22) - 16; tiles <= (1 << 22) + 16; ++tiles) {
        sa::AttnArgs a{};
        a.n = 256;
        a.l = 16;
        a.batch = 1;
        a.heads = tiles;
        if (sa::strided_tiles(a) != tiles) return fail("tiles", a.n, a.l);
        const int64_t threads = ((int64_t)tiles + 7) / 8 * 8 * 1024;
        if (sa::strided_grid_fits(a) != (threads < ((int64_t)1 << 32))) return fail("grid", tiles, a.l);
    }
    std::printf("ok %lld pairs\n", checked);
    return 0;
}
