// Host check of the dispatch rules on the fixed pattern's walks: the estimate of their
// block steps and longest walks against a count of the present blocks, and the rules on
// sharing a walk among four waves and on two query blocks per workgroup at shapes
// measured on both sides of their lines.
#include <cstdio>

#include "sa_internal.h"

static sa::AttnArgs call(int mode, int n, int l, int c, int B, int d, int batch, int heads) {
    sa::AttnArgs a{};
    a.pattern = sa::FIXED;
    a.mode = mode;
    a.n = n;
    a.l = l;
    a.c = c;
    a.block = B;
    a.nq = n / B;
    a.d = d;
    a.batch = batch;
    a.heads = heads;
    return a;
}

static bool near(double x, double y, double tol) { return x - y <= tol * y + 2.0 && y - x <= tol * y + 2.0; }

int main() {
    int checked = 0;
    // sizes that the blocks divide: the estimate is off by the ends of the ranges alone;
    // l-blocks that straddle blocks add up to a block at each end
    for (int mode : {sa::MODE_A1, sa::MODE_A2, sa::MODE_MERGED, sa::MODE_INTERLEAVED})
        for (int B : {16, 32, 64})
            for (int n : {1024, 2048, 4160})
                for (int l : {64, 96, 128, 300, 512, 1024, 2048, 5000})
                    for (int c : {8, 32, 64}) {
                        const int heads = 4, nq = n / B;
                        const sa::AttnArgs a = call(mode, n - n % B, l, c, B, 64, 1, heads);
                        double steps = 0, row = 0, column = 0;
                        for (int h = 0; h < (mode == sa::MODE_INTERLEAVED ? 2 : 1); ++h) {
                            sa::Pattern p;
                            p.pattern = sa::FIXED;
                            p.part = sa::part_of_head(mode, h);
                            p.l = l;
                            p.c = c;
                            p.w = l - c;
                            for (int x = 0; x < nq; ++x) {
                                int in_row = 0, in_column = 0;
                                for (int y = 0; y < nq; ++y) {
                                    if (y <= x) in_row += sa::block_present(p, (int64_t)x * B, (int64_t)x * B + B - 1,
                                                                            (int64_t)y * B, (int64_t)y * B + B - 1);
                                    if (y >= x) in_column += sa::block_present(p, (int64_t)y * B, (int64_t)y * B + B - 1,
                                                                               (int64_t)x * B, (int64_t)x * B + B - 1);
                                }
                                steps += (double)in_row * heads / (mode == sa::MODE_INTERLEAVED ? 2 : 1);
                                row = in_row > row ? in_row : row;
                                column = in_column > column ? in_column : column;
                            }
                        }
                        const sa::WalkEstimate w = sa::walk_estimate(a);
                        const bool whole = l % B == 0 && c % B == 0 && n % l == 0;
                        const double tol = whole ? 0.3 : 1.0;
                        if (!near(w.steps / (heads * nq), steps / (heads * nq), tol) || !near(w.longest_row, row, tol) ||
                            !near(w.longest_column, column, tol)) {
                            std::printf("fail: mode %d n %d l %d c %d B %d: steps %g of %g, row %g of %g, column %g of %g\n",
                                        mode, n, l, c, B, w.steps, steps, w.longest_row, row, w.longest_column, column);
                            return 1;
                        }
                        ++checked;
                    }
    struct Side {
        int mode, n, l, c, B, d, batch, heads;
        bool rows, columns;
    };
    for (const Side& s : {
             // few walks: shared
             Side{sa::MODE_INTERLEAVED, 3072, 128, 32, 32, 128, 4, 2, false, true},
             Side{sa::MODE_MERGED, 3072, 128, 32, 32, 128, 1, 4, true, true},
             Side{sa::MODE_MERGED, 4096, 1024, 32, 16, 64, 1, 4, true, true},
             Side{sa::MODE_MERGED, 12288, 128, 32, 16, 64, 1, 4, false, true},
             // long walks inside the l-blocks, or one l-block, and many heads: they fill the chip by themselves
             Side{sa::MODE_MERGED, 2048, 4096, 32, 32, 64, 1, 64, false, false},
             Side{sa::MODE_MERGED, 2048, 4096, 32, 16, 128, 1, 64, false, false},
             Side{sa::MODE_MERGED, 2048, 4096, 32, 32, 128, 1, 16, false, false},
             Side{sa::MODE_MERGED, 4096, 1024, 32, 32, 128, 1, 16, false, false},
             Side{sa::MODE_MERGED, 2048, 512, 32, 32, 64, 1, 64, false, false},
             Side{sa::MODE_A2, 2048, 4096, 32, 32, 64, 4, 4, false, false},  // nothing attended
             Side{sa::MODE_MERGED, 1024, 256, 32, 16, 128, 1, 64, false, false},
             Side{sa::MODE_MERGED, 12288, 128, 32, 32, 64, 1, 16, false, false},
         }) {
        const sa::AttnArgs a = call(s.mode, s.n, s.l, s.c, s.B, s.d, s.batch, s.heads);
        if (sa::walk_phases(a, false) != s.rows || sa::walk_phases(a, true) != s.columns) {
            std::printf("fail: phases mode %d n %d l %d c %d B %d d %d %d x %d: rows %d columns %d\n", s.mode, s.n, s.l, s.c,
                        s.B, s.d, s.batch, s.heads, sa::walk_phases(a, false), sa::walk_phases(a, true));
            return 1;
        }
        ++checked;
    }
    // two query blocks per workgroup: many workgroups of long walks
    struct Wide {
        int mode, n, l, c, batch, heads;
        bool on;
    };
    for (const Wide& s : {
             Wide{sa::MODE_MERGED, 65536, 256, 32, 1, 8, true}, Wide{sa::MODE_MERGED, 12288, 128, 32, 2, 8, true},
             Wide{sa::MODE_MERGED, 4096, 128, 40, 4, 8, true}, Wide{sa::MODE_INTERLEAVED, 12288, 256, 32, 2, 8, true},
             Wide{sa::MODE_A2, 12288, 512, 32, 2, 8, true}, Wide{sa::MODE_A1, 16384, 4096, 32, 4, 8, true},
             Wide{sa::MODE_MERGED, 8192, 2048, 32, 4, 8, true}, Wide{sa::MODE_MERGED, 12224, 2944, 16, 2, 8, false},
             Wide{sa::MODE_A1, 12288, 2048, 32, 2, 8, false}, Wide{sa::MODE_A1, 12288, 128, 32, 2, 8, false}, Wide{sa::MODE_A1, 12288, 1024, 32, 2, 8, false},
             Wide{sa::MODE_MERGED, 2048, 128, 32, 8, 8, false}, Wide{sa::MODE_MERGED, 4096, 512, 32, 4, 8, false},
             Wide{sa::MODE_INTERLEAVED, 12288, 512, 32, 2, 8, false}, Wide{sa::MODE_INTERLEAVED, 12288, 2048, 32, 2, 8, false},
             Wide{sa::MODE_A2, 12288, 2048, 32, 2, 8, false}, Wide{sa::MODE_A2, 2048, 256, 32, 8, 8, false},
         }) {
        const sa::AttnArgs a = call(s.mode, s.n, s.l, s.c, 64, 64, s.batch, s.heads);
        if (sa::wide_rows(a) != s.on) {
            std::printf("fail: wide mode %d n %d l %d c %d %d x %d\n", s.mode, s.n, s.l, s.c, s.batch, s.heads);
            return 1;
        }
        ++checked;
    }
    std::printf("ok %d shapes\n", checked);
    return 0;
}
