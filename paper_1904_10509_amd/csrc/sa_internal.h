// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "sa_mask.h"
#include "sa_pattern.h"

namespace sa {

constexpr float kLog2eHost = 1.4426950408889634f;

// Present blocks of one layout, counted on the host with the O(1) test.
int64_t layout_count_host(const Pattern& p, int64_t n, int64_t B);

hipError_t layout_launch(int64_t n, int32_t block, int32_t pattern, int32_t mode, int32_t sub, int64_t l,
                         int64_t c, int n_layouts, int32_t* row_ptr, int32_t* col_idx,
                         uint8_t* kind, int32_t* col_ptr, int32_t* row_idx, uint8_t* kind_t,
                         hipStream_t stream);

// Calls f(pattern, mode) with both as compile-time constants
// (std::integral_constant), so that kernels are specialised per pattern and
// head mode.
template <typename F>
inline hipError_t with_pattern_mode(int pattern, int mode, F&& f) {
    using S = std::integral_constant<int, STRIDED>;
    using X = std::integral_constant<int, FIXED>;
    using M0 = std::integral_constant<int, MODE_A1>;
    using M1 = std::integral_constant<int, MODE_A2>;
    using M2 = std::integral_constant<int, MODE_MERGED>;
    using M3 = std::integral_constant<int, MODE_INTERLEAVED>;
    if (pattern == STRIDED) {
        switch (mode) {
        case MODE_A1: return f(S{}, M0{});
        case MODE_A2: return f(S{}, M1{});
        case MODE_MERGED: return f(S{}, M2{});
        default: return f(S{}, M3{});
        }
    }
    switch (mode) {
    case MODE_A1: return f(X{}, M0{});
    case MODE_A2: return f(X{}, M1{});
    case MODE_MERGED: return f(X{}, M2{});
    default: return f(X{}, M3{});
    }
}

// Orders in which the dK / dV kernel takes its work.
enum { CLAIM_QUEUES = 0, CLAIM_ROUND_ROBIN = 1, CLAIM_SERPENTINE = 2, CLAIM_XCD_SERPENTINE = 3 };

// Which blocks a kernel walks:
//   WALK_LAYOUT  the present blocks of the layout;
//   WALK_BAND    the blocks of the strided band A1 = {i - l .. i}, without a
//                layout: ceil(l / B) blocks before the diagonal one in a row,
//                after it in a column;
//   WALK_DENSE   every block kb <= qb, without a layout (dense causal).
enum { WALK_LAYOUT = 0, WALK_BAND = 1, WALK_DENSE = 2 };

// What a kernel does with its result:
//   EPI_STORE  writes it;
//   EPI_MERGE  (forward) combines it, by log-sum-exp, with the O and LSE
//              already in the outputs (a softmax over a disjoint part of
//              each row's set);
//   EPI_ADD    (dQ, dK, dV) adds it to the gradient already in the output.
enum { EPI_STORE = 0, EPI_MERGE = 1, EPI_ADD = 2 };

// Everything a kernel needs to know about one call.
struct AttnArgs {
    int32_t pattern, mode;
    int32_t l, c;          // validated to fit in 32 bits
    int32_t n, nq, block;  // n < 2^31
    int32_t batch, heads, d;
    int64_t sb, sh, ss;    // element strides: batch, head, sequence
    float scale;           // softmax scale (> 0)
    float scale_log2;      // scale * log2(e)
    uint64_t period_bits;  // bits at multiples of l below 64 (strided masks)
    uint64_t sum_lo, sum_hi;  // summary positions below 128 (fixed masks, l <= 64, subblock 0)
    int32_t sub;           // fixed: 0 = one summary window for all heads, else floor(l / c) subblocks
    int32_t claim_mode;    // dK / dV work order, one of CLAIM_* (set by the backward launcher)
    int32_t pairs;         // dK / dV: summary halves walked in pairs (set by the backward launcher)
    int32_t row_stats;     // dQ: compute the row statistics itself, in place of the pre kernel (set by the launcher)
    int64_t sched_first;   // dQ with row_stats: the first workgroup that builds the dK / dV schedule (set by the launcher)
    DivL dl;               // division by l
    int32_t walk;          // WALK_*
    int32_t qshift;        // masks see query i as i - qshift (a causal limit j <= i - qshift)
    int32_t epilogue;      // EPI_*
    int64_t lse_sb, lse_sh, lse_ss;  // element strides of LSE and the row statistics (batch, head, row)
    int64_t off, lse_off;  // first element of the tensors and of LSE / the row statistics (a subset of the heads)
    int64_t ws_rows;       // rows of the whole call: the size of each row statistic in the workspace
    int32_t seq;           // residue classes: positions of the whole sequence (class h of l has
                           // ceil((seq - h) / l) of them, the rest of its last block is padding); else 0
    const int32_t* row_ptr;
    const int32_t* col_idx;
    const int32_t* col_ptr;
    const int32_t* row_idx;
};

// Blocks before (row) or after (column) the diagonal one in the strided band.
__host__ __device__ inline int band_blocks(const AttnArgs& a) { return (a.l - 1) / a.block + 1; }
constexpr int kLongBand = 8;  // from here on a band's walks count as long

// Block steps of the fixed pattern's walks, from its sizes alone: every step of a call,
// and the longest walk of a row block and of a key block.  (Per (batch, head) nq walks;
// those of far blocks, which hold summary keys, reach half the sequence on average,
// those inside an l-block half of it.)
struct WalkEstimate {
    double far, local;  // blocks of the last row: with summary keys, and of its own l-block
    double steps, longest_row, longest_column;
};
inline WalkEstimate walk_estimate(const AttnArgs& a) {
    const int32_t a2_heads = a.mode == MODE_INTERLEAVED ? a.heads / 2 : a.mode == MODE_A1 ? 0 : a.heads;
    const int32_t a1_heads = a.mode == MODE_MERGED ? a.heads : a.heads - a2_heads;
    const double nq = a.nq;
    auto least = [&](double x) { return x < nq ? x : nq; };
    const double far = a2_heads == 0 || a.n <= a.l - a.c
                           ? 0.0
                           : least((double)((a.n - 1) / a.l + 1) * ((a.c - 1) / a.block + 1));
    const double local = a1_heads == 0 ? 0.0 : least((a.l - 1) / a.block + 1);
    const double column = far > 0.0 ? nq - (a.l - a.c) / a.block : 0.0;
    WalkEstimate w;
    w.far = far;
    w.local = local;
    w.steps = 0.5 * nq * a.batch * (a2_heads * far + a1_heads * (local + 1.0));
    w.longest_row = a.mode == MODE_MERGED ? far + local : far > local ? far : local;
    w.longest_column = column > local ? column : local;
    return w;
}

// Whether a workgroup of the forward or the dQ kernel takes two query blocks (four
// waves of 32 rows): where both walk the same blocks but for the diagonal's, i.e.
// the strided band, and in the fixed pattern l-blocks of whole pairs.  A staged
// tile then serves 128 rows, and in the forward each K / V operand read from LDS
// feeds 32 rows instead of 16, at three waves per SIMD instead of four (with one
// query block per workgroup the ring's LDS allowed 2.5, and 32 rows were slower).
// Fixed n = 65,536, 8 heads: forward 0.712 -> 0.643 ms, dQ 0.736 -> 0.702; n =
// 12,288, 16 heads: forward 110 -> 104 us; dense limit, n = 12,288, 16 heads:
// forward 375 -> 343 us, backward 1,070 -> 1,020.  Half as many workgroups of twice
// the length: kWideGroups of them keep the chip full to the end (strided band, 1,024:
// 190 against 189 us; 480, n = 4,096: 20.6 against 25.4), and a short walk is over before
// the wider reads pay (strided, l = 128, 3 blocks: 25.5 against 29.2 us).  In the fixed
// pattern rows differ in length, and the line depends on how many steps an average row
// walks: far ones (summary halves in pairs count once) and those of its own l-block.
// Forward, us, one block | two, c = 32 unless given:
//   kWideGroups, 16 far steps: n = 4,096, l = 128, c = 40, 32 heads 74 | 64; fewer: c = 32, 8 far
//     39 | 42, c = 64, l = 256, 8 far 40 | 43, l = 512 31 | 35;
//   half as many again (n = 12,288, 16 heads): merged, 6 far: l = 128, 24 131 | 119, l = 512, 6
//     62 | 61 (dQ 79 | 75), n = 12,224, l = 2,944, 2.5 116 | 128; A2 alone, 3: l = 1,024 26 | 25,
//     l = 2,048, 1.5 19 | 20; alternating heads, 8: l = 256, 12 59 | 54, l = 512, 6 37 | 41, l =
//     2,048, 1.5 83 | 98;
//   twice as many: long walks inside the l-blocks as well, which leave few workgroups to the
//     end; A1 alone, 12 steps: n = 16,384, 32 heads, l = 2,048 223 | 213, l = 1,024 112 | 118,
//     l = 128 47 | 51 (with fewer: n = 12,288, 16 heads, l = 2,048 93 | 100, l = 128 21 | 23, dQ
//     34 | 37); merged, 10: n = 8,192, 32 heads, l = 2,048, 18.5 128 | 119, l = 512, 8.5 66 | 65.
constexpr int64_t kWideGroups = 1024;
inline bool wide_rows(const AttnArgs& a) {
    const int64_t groups = (int64_t)a.batch * a.heads * ((a.nq + 1) / 2);
    if (a.pattern == STRIDED) return a.walk == WALK_BAND && band_blocks(a) >= kLongBand && groups >= kWideGroups;
    if (a.walk != WALK_LAYOUT || a.l % 128 != 0 || groups < kWideGroups) return false;
    const WalkEstimate w = walk_estimate(a);
    const bool pairs = a.c == 32 && a.block == 64;
    const double far = (pairs ? 0.25 : 0.5) * w.far, local = 0.5 * (w.local + 1.0);
    if (far >= 16.0) return true;
    if (groups < kWideGroups + kWideGroups / 2) return false;
    const bool many = groups >= 2 * kWideGroups;
    switch (a.mode) {
    case MODE_A1: return many && local >= 12.0;
    case MODE_A2: return far >= 3.0;
    case MODE_MERGED: return far >= 6.0 || (many && far + local >= 10.0);
    default: return far >= 8.0;
    }
}

// Whether four waves share each row's (dQ) or each key group's (dK / dV) walk, in the
// fixed pattern with B < 64.  A workgroup of one or two waves walks a row or column
// alone, and the longest (a summary column: every block below it) sets the time while
// all walks together do not fill the chip.  Four phases make it a quarter as long, but
// their rings leave a compute unit one to four workgroups, whose waves wait for each
// other at every step: with the chip full they take up to 2.4 times as long.  So the
// line is on the work per compute unit in units of the longest walk: all block steps,
// and kWalkSteps more for each walk (its own rows, the sum of the phases), over 256 times
// the longest walk's steps.  dQ's line lies further out.  Measured on either side of
// the lines (work: us without | with phases; l = 128 or as given, c = 32, merged):
//   d = 128, B = 32, one workgroup per compute unit: dQ n = 3,072, 4 heads 2.1: 27 | 26; l =
//     512, n = 2,048, 8 heads 3.5: 21 | 24; dK / dV l = 1,024, n = 4,096, 8 heads 1.8: 84 | 64;
//     A2 alone, l = 256, n = 1,024, 16 heads 2.1: 28 | 35; l = 2 n, 16 heads 3.5: 60 | 85;
//     two heads of l = n = 11,520, 1.8, dK / dV: 622 | 798 both; of c = l, n = 15,360, 2.3, dQ:
//     867 | 1,097;
//   d = 64, B = 32, two: dQ n = 3,072, 8 heads 4.1: 20 | 22; dK / dV l = 512, n = 8,192, 8 heads
//     1.3: 132 | 106; n = 3,072, 16 heads 2.5: 54 | 53; l = 256, n = 1,024, 16 heads 2.4: 18 |
//     19; l = 2 n, 64 heads 14: 98 | 186;
//   d = 64, B = 16, four: dQ n = 3,072, 8 heads 5.6: 23 | 20; l = 512, n = 2,048, 16 heads 8.9:
//     19 | 20; dK / dV n = 12,288, 8 heads 3.9: 300 | 210, 16 heads 7.8: 334 | 416;
//   d = 32, B = 32, four: dK / dV l = 1,024, n = 4,096, 16 heads 3.5: 51 | 36; n = 12,288, 16
//     heads 4.7: 175 | 192.
// Walks of a few steps gain less than the sum of the phases costs (l = 128, n = 608, one
// head of 128: 19.5 | 22).
constexpr double kWalkSteps = 24.0, kMinPhaseSteps = 8.0;
inline bool walk_phases(const AttnArgs& a, bool columns) {
    if (a.pattern != FIXED || a.mode == MODE_A1) return false;
    const WalkEstimate w = walk_estimate(a);
    const double work = (w.steps + kWalkSteps * a.nq * a.heads * a.batch) / 256.0;
    const int row = a.d * a.block;  // elements of a ring stage: phases' workgroups per compute unit
    const double line = columns ? (row > 2048 ? 1.6 : row > 1024 ? 2.3 : 3.8) : (row > 2048 ? 2.2 : row > 1024 ? 4.0 : 6.6);
    const double longest = columns ? w.longest_column : w.longest_row;
    return longest >= kMinPhaseSteps && work <= line * longest;
}

// The (head, query block, batch) of a row-view workgroup, on the grid
// (heads, nq, batch).  The dispatcher hands consecutive workgroups to the 8
// XCDs in turn, so workgroup L (x fastest) runs on XCD L mod 8.  A walk of
// every block (the residue classes, each a short dense problem read at a
// stride of l rows) gives the nq workgroups of one (batch, head) consecutive
// places s = L / 8 on one XCD: its keys then stay in that XCD's L2 while all
// its query blocks walk them, instead of leaving it between the query-block
// generations of the plain order.  Needs batch x heads a multiple of 8;
// otherwise, and for other walks, query blocks (pairs of them, for a grid of half
// as many) from the longest rows down, every (batch, head) of one before the next:
// with the batch outermost its last element's long rows started late (dense
// limit, n = 12,288, 2 x 8 heads: forward 400 -> 375 us, backward 1,145 -> 1,070).
// A band of few blocks keeps the batch outermost: its rows are equal, and
// neighbouring ones share their keys in L2 (n = 12,288, l = 128: backward 2 to 4%).
struct GridItem {
    int h, qb, b;
};
__device__ inline GridItem row_grid_item(const AttnArgs& a) {
    const uint64_t L = blockIdx.x + (uint64_t)gridDim.x * (blockIdx.y + (uint64_t)gridDim.y * blockIdx.z);
    if (a.walk == WALK_DENSE && ((int64_t)a.batch * a.heads) % 8 == 0) {
        const uint64_t s = L / 8;
        const uint64_t u = (s / (uint64_t)a.nq) * 8 + L % 8;  // (batch, head) unit
        return {(int)(u % (uint64_t)a.heads), a.nq - 1 - (int)(s % (uint64_t)a.nq), (int)(u / (uint64_t)a.heads)};
    }
    if (a.walk == WALK_BAND && band_blocks(a) < kLongBand)
        return {(int)blockIdx.x, (int)(gridDim.y - 1 - blockIdx.y), (int)blockIdx.z};
    const uint64_t units = (uint64_t)a.batch * a.heads, y = L / units, u = L - y * units;
    return {(int)(u % (uint64_t)a.heads), (int)(gridDim.y - 1 - y), (int)(u / (uint64_t)a.heads)};
}

// First element of (batch b, head h) in the tensors.
__host__ __device__ inline int64_t head_base(const AttnArgs& a, int b, int h) {
    return a.off + (int64_t)b * a.sb + (int64_t)h * a.sh;
}

// Index of row i of (batch b, head h) in LSE and the backward's row statistics.
__host__ __device__ inline int64_t stat_index(const AttnArgs& a, int b, int h, int64_t i) {
    return a.lse_off + (int64_t)b * a.lse_sb + (int64_t)h * a.lse_sh + i * a.lse_ss;
}

// Rows of head h: in a residue-class view (whose heads are the l classes)
// class h's positions, else n.  Padding rows beyond them are read as the last
// row, masked where they are queries of a column, and never written.
__host__ __device__ inline int head_rows(const AttnArgs& a, int h) {
    return a.seq > 0 ? (a.seq - 1 - h) / a.heads + 1 : a.n;
}


// Layout that head h reads.
__host__ __device__ inline int head_layout(const AttnArgs& a, int h) { return layout_of_head(a.mode, a.sub, h); }

// First summary position of subblock s inside an l-block (fixed pattern).
__host__ __device__ inline int32_t window_start(const AttnArgs& a, int s) {
    return (int32_t)summary_start(a.l, a.c, s);
}

// Mask parameters of one part and summary subblock s.  With distinct
// subblocks and l <= 64 the 128-position summary words are built here (a few
// scalar steps per workgroup); otherwise they come with the call.
__device__ inline MaskParams mask_params(const AttnArgs& a, int pattern, int part, int s) {
    MaskParams mp{pattern, part, a.l, a.c, a.period_bits, a.sum_lo, a.sum_hi, window_start(a, s)};
    if (pattern == FIXED && s != 0 && a.l <= 64) summary_words(a.l, a.c, mp.w, &mp.sum_lo, &mp.sum_hi);
    return mp;
}
__device__ inline MaskParams head_mask_params(const AttnArgs& a, int pattern, int mode, int h) {
    return mask_params(a, pattern, part_of_head(mode, h), subblock_of_head(a.sub, h));
}

// Forward.  q, k, v, o use the strides in `a`; lse is [batch, heads, n].
hipError_t fwd_launch(const AttnArgs& a, int dtype, const void* q, const void* k, const void* v,
                      void* o, float* lse, hipStream_t stream);
hipError_t fwd_f32(const AttnArgs& a, const void* q, const void* k, const void* v, void* o, float* lse,
                   hipStream_t stream);

// Strided merged heads in one pass (bf16; sa_strided.hip).
hipError_t strided_fwd(const AttnArgs& a, const void* q, const void* k, const void* v, void* o, float* lse,
                       hipStream_t stream);
hipError_t strided_bwd(const AttnArgs& a, const void* q, const void* k, const void* v, const void* o, const void* dout,
                       const float* lse, void* dq, void* dk, void* dv, void* workspace, hipStream_t stream, int parts);

// Backward workspace: D and the base-2 LSE per row [b, h, n] (fp32), then
// the work queues and the column order of the dK / dV kernel.
// Whether the row-view kernels (forward, dQ) carry a second step body for
// fully attended blocks: always in the fixed pattern and for walks of the band
// or of every block (l / B - 1 of a band row's l / B + 1 blocks are full, and
// all but the diagonal of a dense row); over a strided layout when those
// blocks (l / B - 1 per row) outnumber the diagonal-only blocks of a middle
// row (about n / 2l), i.e. 2 l^2 > n B, as in the dense limit l >= n.
// Otherwise the second copy of the code costs more than it saves.
template <int PAT, typename F>
inline hipError_t with_full_body(const AttnArgs& a, F&& f) {
    if constexpr (PAT == FIXED) {
        return f(std::true_type{});
    } else {
        if (a.walk != WALK_LAYOUT || 2.0 * (double)a.l * (double)a.l > (double)a.n * (double)a.block)
            return f(std::true_type{});
        return f(std::false_type{});
    }
}

size_t decode_workspace_bytes(int pattern, int mode, int32_t sub, int32_t pos, int32_t l, int32_t c,
                              int64_t batch, int64_t heads, int d);
hipError_t decode_launch(int pattern, int mode, int32_t sub, int32_t pos, int32_t l, int32_t c, int batch, int heads,
                         int d, int dtype, const void* q, const int64_t* q_strides, const void* k, const void* v,
                         const int64_t* kv_strides, float scale, void* o, float* lse, void* workspace,
                         hipStream_t stream);

size_t bwd_workspace_bytes(int64_t batch, int64_t heads, int64_t n, int64_t nq, int n_layouts);

// Launches of a backward call: the row statistics (pre), dQ, and dK / dV.
enum { BWD_PRE = 1, BWD_DQ = 2, BWD_DKDV = 4, BWD_ALL = 7 };

// Backward; `parts` selects its launches.
hipError_t bwd_launch(const AttnArgs& a, int dtype, const void* q, const void* k, const void* v,
                      const void* o, const void* dout, const float* lse, void* dq, void* dk,
                      void* dv, void* workspace, hipStream_t stream, int parts = BWD_ALL);

}  // namespace sa
