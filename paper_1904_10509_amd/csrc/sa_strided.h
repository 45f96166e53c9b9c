// Index arithmetic of the one-pass strided kernels (sa_strided.hip), host and
// device: the rows of each workgroup's units and the rows that they meet.
#pragma once

#include "sa_internal.h"

namespace sa {

__host__ __device__ inline int min32(int a, int b) { return a < b ? a : b; }
__host__ __device__ inline int max32(int a, int b) { return a > b ? a : b; }

// Tiles of 16 steps x 16 classes over a call.
inline int64_t strided_tiles(const AttnArgs& a) {
    const int64_t M = (a.n - 1) / a.l + 1;
    return ((M + 15) / 16) * ((a.l - 1) / 16 + 1) * a.batch * a.heads;
}

// Workgroups of a launch: the tiles are dealt to the eight XCDs in equal shares (see
// strided_tile).  The largest has 1,024 threads, and a launch holds fewer than 2^32.
inline int64_t strided_groups(const AttnArgs& a) { return (strided_tiles(a) + 7) / 8 * 8; }
inline bool strided_grid_fits(const AttnArgs& a) { return strided_groups(a) * 1024 < ((int64_t)1 << 32); }

// The 16 x 16 tile of a workgroup.
struct STile {
    int b, h, m0, r0;
};
__host__ __device__ inline bool strided_tile(const AttnArgs& a, uint32_t group, STile* t) {
    const uint32_t M = (uint32_t)((a.n - 1) / a.l + 1), mt = (M + 15) / 16, rt = (uint32_t)((a.l - 1) / 16 + 1);
    const uint32_t total = mt * rt * (uint32_t)(a.batch * a.heads), share = (total + 7) / 8;
    // workgroup L runs on XCD L mod 8, which takes `share` consecutive tiles
    const uint32_t s = group / 8, id = (group % 8) * share + s;
    if (s >= share || id >= total) return false;
    const uint32_t bh = id / (mt * rt), rest = id - bh * (mt * rt), mi = rest / rt;
    t->b = (int)(bh / (uint32_t)a.heads);
    t->h = (int)(bh % (uint32_t)a.heads);
    t->m0 = 16 * (int)(mt - 1 - mi);  // longest classes first
    t->r0 = 16 * (int)(rest - mi * rt);
    return true;
}

// The rows of a unit and the rows of the other side that they meet.
struct Walk {
    bool on;               // the unit holds a row
    int64_t at, stride;    // element of index 0 and distance of neighbouring indices
    int own, own_last;     // first own index, last existing index
    int64_t stat, stat_stride;  // LSE / row statistics: of index 0, distance
    int first, count;      // other side: first index and how many
    int last;              // last existing index of the other side
    int lo, hi;            // attended by this lane's row: first + lo .. first + hi
    int full_lo, full_hi;  // attended by every row of the unit (as offsets from first)
};

// Rows of a unit as queries: band keys i - l .. i, class keys m' <= m - 2.
__host__ __device__ inline Walk query_walk(const AttnArgs& a, const STile& t, bool cls, int u, int r) {
    Walk w;
    if (!cls) {
        const int64_t i0l = (int64_t)(t.m0 + u) * a.l + t.r0;
        w.on = i0l < a.n;
        const int i0 = w.on ? (int)i0l : 0;
        w.at = 0;
        w.stride = a.ss;
        w.stat = 0;
        w.stat_stride = 1;
        w.own = i0;
        w.own_last = w.last = a.n - 1;
        w.first = max32(0, i0 - a.l);
        w.count = min32(i0 + 15, a.n - 1) - w.first + 1;
        w.lo = i0 + r - a.l - w.first;
        w.hi = i0 + r - w.first;
        w.full_lo = i0 + 15 - a.l - w.first;
        w.full_hi = i0 - w.first;
    } else {
        const int c = t.r0 + u;
        w.on = c < a.l && c < a.n;
        const int rows = w.on ? (a.n - 1 - c) / a.l + 1 : 1;
        w.on = w.on && t.m0 < rows;
        w.at = (int64_t)c * a.ss;
        w.stride = (int64_t)a.l * a.ss;
        w.stat = c;
        w.stat_stride = a.l;
        w.own = t.m0;
        w.own_last = w.last = rows - 1;
        w.first = 0;
        w.count = max32(0, min32(t.m0 + 15, rows - 1) - 1);
        w.lo = 0;
        w.hi = t.m0 + r - 2;
        w.full_lo = 0;
        w.full_hi = t.m0 - 2;
    }
    return w;
}

// Rows of a unit as keys: band queries j .. j + l, class queries m' >= m + 2.
// Queries past the sequence's (class's) last row are not attended.
__host__ __device__ inline Walk key_walk(const AttnArgs& a, const STile& t, bool cls, int u, int r) {
    Walk w = query_walk(a, t, cls, u, r);
    const int key = w.own + r;
    if (!cls) {
        w.first = w.own;
        w.count = (int)min64((int64_t)a.n - 1, (int64_t)w.own + 15 + a.l) - w.first + 1;
        w.lo = r;
        w.hi = (int)min64((int64_t)w.last, (int64_t)key + a.l) - w.first;
        w.full_lo = 15;
        w.full_hi = (int)min64((int64_t)w.last, (int64_t)w.own + a.l) - w.first;
    } else {
        w.first = w.own + 2;
        w.count = max32(0, w.last - w.first + 1);
        w.lo = r;
        w.hi = w.last - w.first;
        w.full_lo = 15;
        w.full_hi = w.hi;
    }
    return w;
}

}  // namespace sa
