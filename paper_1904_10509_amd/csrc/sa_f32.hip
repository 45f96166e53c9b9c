// fp32 forward and backward on the matrix cores (v_mfma_f32_16x16x4_f32:
// fp32 products and sums, the precision of the VALU).
//
// A workgroup of eight waves takes one group of 16 query rows (forward, dQ) or
// 16 key columns (dK, dV) of one (batch, head).  Its waves share out the
// 16 x 16 tiles of that strip that hold an attended pair: consecutive waves take
// consecutive 16-wide groups of a block, rotating from block to block (in the
// fixed pattern the live groups of every far block are the same ones).  Each
// wave keeps its own partial result, and the partials are combined in wave
// order through LDS at the end, so results are the same on every run.
//
// What bounds it: one instruction does 2,048 FLOP in 32 cycles, so a 16 x 16
// tile costs 1,024 (forward) to 2,048 (dK, dV) cycles at d = 64 and the strips
// have to be spread thinly to fill 1,024 SIMDs: at n = 2,048 with four heads
// there are 512 strips, and the strip of a summary column has 128 tiles.  One
// wave per strip leaves half the SIMDs idle and the longest strip alone takes
// over 100 us; eight waves bring it to 16 tiles.  Operands come straight from
// global memory in 16-byte loads (each tile's rows are read by one wave only, so
// LDS staging would add a pass), the next tile's ahead of this one's products.
// Measured (forward + backward): strided n = 256, one head of 32: 736 -> 23 us;
// fixed n = 2,048, l = 128, c = 32, four heads of 64: 7,213 -> 157 us, both against
// one thread per row or column on the VALU, with smaller errors (8.0e-7 -> 4.2e-7 of
// the largest gradient's norm).  Exponentials are expf: __expf, whose error grows
// with its argument (weights of e^-24 off by 8e-7 against 2e-7), saves 4%.
//
// Operand layout (lane = 16 g + r).  A 16x16x4 product takes A[r][g] and B[g][r],
// one fp32 each, and returns D[4g + t][r].  The contraction index may run over
// any permutation used by both operands:
//   over d: lane (g, r) holds row r, elements 16 s + 4 g .. + 3 (a 16-byte load);
//     step (s, t) contracts the four elements 16 s + 4 g + t;
//   over the tile's rows: step t contracts rows 4 g + t, so the D results of the
//     first product are the B operands of the second, and its A operand, the
//     transpose of a row-major tile, is element d of row 4 g + t.  The 16-wide
//     d blocks are interleaved (d = 16 V hb + V i + x for result row i, block V hb
//     + x), so that a lane's elements of a row are V neighbours: one load.
#include "sa_bwd_kernels.h"

namespace sa {

namespace {

constexpr int kF32Waves = 8;
constexpr int kF32Threads = 64 * kF32Waves;
constexpr int64_t kF32MaxGrid = 1 << 22;  // workgroups in x; longer sequences take several strips each

__device__ inline f32x4 mfma_f32(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int D>
struct F32 {
    static constexpr int KS = D / 16;            // 16-byte chunks of a lane along d
    static constexpr int V = D >= 64 ? 4 : 2;    // neighbours in d per transposed load
    static constexpr int HB = D / (16 * V);      // transposed loads per row
    static constexpr int DB = D / 16;            // 16-wide d blocks of a result
    static constexpr int RS = D + 4;             // row stride of the LDS partials (floats)
    static constexpr bool PREFETCH = D <= 64;    // registers for the next tile's rows beside this one's
    typedef float vec __attribute__((ext_vector_type(V)));
};

// Rows of a 16-row tile as operands of the products over d.
template <int D>
struct RowOp {
    f32x4 x[F32<D>::KS];
    __device__ void load(const float* tile, int64_t ss, int g, int r) {
        const float* p = tile + (int64_t)r * ss + 4 * g;
#pragma unroll
        for (int s = 0; s < F32<D>::KS; ++s) x[s] = *reinterpret_cast<const f32x4*>(p + 16 * s);
    }
};

// A . B^T over d: two accumulation chains, so that a product does not wait for the one before it.
template <int D>
__device__ inline f32x4 dot_tile(const RowOp<D>& a, const RowOp<D>& b) {
    f32x4 c0 = zero4(), c1 = zero4();
#pragma unroll
    for (int s = 0; s < F32<D>::KS; ++s) {
        c0 = mfma_f32(a.x[s][0], b.x[s][0], c0);
        c1 = mfma_f32(a.x[s][1], b.x[s][1], c1);
        c0 = mfma_f32(a.x[s][2], b.x[s][2], c0);
        c1 = mfma_f32(a.x[s][3], b.x[s][3], c1);
    }
    return c0 + c1;
}

// The transposed operand of a 16-row tile: rows 4 g + t, this lane's d.
template <int D>
struct ColOp {
    typename F32<D>::vec x[4][F32<D>::HB];
    __device__ void load(const float* tile, int64_t ss, int g, int r) {
        constexpr int V = F32<D>::V;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int hb = 0; hb < F32<D>::HB; ++hb)
                x[t][hb] = *reinterpret_cast<const typename F32<D>::vec*>(tile + (int64_t)(4 * g + t) * ss +
                                                                          16 * V * hb + V * r);
    }
    // acc[d][r] += sum over the tile's rows of x[row][d] b[row][r]
    __device__ void accumulate(f32x4 b, f32x4* acc) const {
        constexpr int V = F32<D>::V;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int hb = 0; hb < F32<D>::HB; ++hb)
#pragma unroll
                for (int e = 0; e < V; ++e) acc[V * hb + e] = mfma_f32(x[t][hb][e], b[t], acc[V * hb + e]);
    }
};

// Infinities and NaN.  A pair that is not attended has b = 0 in the sums above, but 0
// x infinity and 0 x NaN are NaN.  The walks take no notice (a test in every partly
// attended tile cost registers, and with them a workgroup per compute unit); a wave
// whose sums come out non-finite walks its tiles a second time, with each row's
// products kept by the columns that attend it alone, so that such an element
// reaches what attends it and nothing else.
// acc[d][r] += sum over the tile's rows of tile[row][d] b[row][r] where (row, r) is
// attended (mask: bit t, this lane's pair 4 g + t).
template <int D>
__device__ inline void accumulate_attended(const float* tile, int64_t ss, f32x4 b, uint32_t mask, f32x4* acc, int g,
                                           int r) {
    constexpr int V = F32<D>::V, HB = F32<D>::HB;
#pragma unroll 1
    for (int t = 0; t < 4; ++t) {
        typename F32<D>::vec x[HB];
#pragma unroll
        for (int hb = 0; hb < HB; ++hb)
            x[hb] = *reinterpret_cast<const typename F32<D>::vec*>(tile + (int64_t)(4 * g + t) * ss + 16 * V * hb + V * r);
        const float bt = t == 0 ? b[0] : t == 1 ? b[1] : t == 2 ? b[2] : b[3];
#pragma unroll 1
        for (int row = 0; row < 4; ++row) {  // rows 4 row + t, one at a time
            const bool on = (__shfl(mask, 16 * row + r) >> t) & 1u;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int hb = 0; hb < HB; ++hb)
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const f32x4 sum = mfma_f32(g == row ? x[hb][e] : 0.f, g == row ? bt : 0.f, acc[V * hb + e]);
                    if (on) acc[V * hb + e] = sum;
                    __builtin_amdgcn_sched_barrier(0);  // one sum in flight: registers
                }
        }
    }
}

// x, as a value the compiler knows nothing about.  The second walk is to need no more
// registers than the first: what it computes from opaque lane numbers stays inside it.
__device__ inline int opaque(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// dot_tile of rows in memory, with no operand kept.
template <int D>
__device__ inline f32x4 dot_rows(const float* a, const float* b, int64_t ss, int g, int r) {
    f32x4 c = zero4();
    a += (int64_t)r * ss + 4 * g;
    b += (int64_t)r * ss + 4 * g;
#pragma unroll 1
    for (int s = 0; s < F32<D>::KS; ++s) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(a + 16 * s), y = *reinterpret_cast<const f32x4*>(b + 16 * s);
#pragma unroll
        for (int t = 0; t < 4; ++t) c = mfma_f32(x[t], y[t], c);
    }
    return c;
}

// Whether an element of a wave's sums is an infinity or a NaN (by its bits: the
// build lets comparisons assume that there is none).
template <int D>
__device__ inline bool non_finite(const f32x4* acc) {
    uint32_t top = 0;
#pragma unroll
    for (int db = 0; db < F32<D>::DB; ++db)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint32_t v = __float_as_uint(acc[db][t]) & 0x7FFFFFFFu;
            top = v > top ? v : top;
        }
    return __builtin_amdgcn_ballot_w64(top >= 0x7F800000u) != 0ull;
}

// A wave's partial result [16 rows][D] to LDS, rows at stride RS.
template <int D>
__device__ inline void store_partial(float* dst, const f32x4* acc, int g, int r) {
    constexpr int V = F32<D>::V;
#pragma unroll
    for (int hb = 0; hb < F32<D>::HB; ++hb) {
        float* p = dst + r * F32<D>::RS + 16 * V * hb + 4 * V * g;
        if constexpr (V == 4) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                *reinterpret_cast<f32x4*>(p + 4 * t) =
                    f32x4{acc[4 * hb][t], acc[4 * hb + 1][t], acc[4 * hb + 2][t], acc[4 * hb + 3][t]};
        } else {
            *reinterpret_cast<f32x4*>(p) = f32x4{acc[0][0], acc[1][0], acc[0][1], acc[1][1]};
            *reinterpret_cast<f32x4*>(p + 4) = f32x4{acc[0][2], acc[1][2], acc[0][3], acc[1][3]};
        }
    }
}

// A live 16 x 16 tile of a strip: the first position of its other side, and
// which of this lane's four pairs (4 g + t) are attended.
struct Tile {
    int first;  // -1: none left
    uint32_t mask;
};

// This wave's tiles of a strip of 16 query rows (row_lane x, first row i0 as the
// masks see it) or 16 key columns.  A wave visits every (8 / groups per block)-th
// entry and one 16-wide group of it.
struct TileWalk {
    MaskParams mp;
    DivL dl;
    const int32_t* idx;
    bool dense;
    int e, e1, step, block, group, groups;

    __device__ void init(const AttnArgs& a, const MaskParams& m, const int32_t* index, int first, int last, int w) {
        mp = m;
        dl = a.dl;
        idx = index;
        dense = a.walk != WALK_LAYOUT;
        block = a.block;
        groups = block / 16;
        step = kF32Waves / groups;
        e = first + w / groups;
        e1 = last;
        group = w % groups;
    }
    // The next visited (block, group), as its first position; -1 at the end.
    __device__ int visit() {
        if (e >= e1) return -1;
        const int blk = dense ? e : __builtin_amdgcn_readfirstlane(idx[e]);
        const int first = blk * block + 16 * group;
        e += step;
        group = group + 1 == groups ? 0 : group + 1;
        return first;
    }
    __device__ Tile rows(const RowLane& x, int i0, int g) {
        for (;;) {
            const int j0 = visit();
            if (j0 < 0) return {-1, 0u};
            if (block_full32(mp.pattern, mp.part, dl, mp.c, mp.w, i0, i0 + 15, j0, j0 + 15)) return {j0, 15u};
            const int j0_mod = mod_l(dl, j0);
            const uint64_t sum = mp.pattern == FIXED ? summary_bits(mp, j0_mod) : 0ull;
            uint32_t bits;
            if (mp.pattern == FIXED && far_block(FIXED, dl, i0, j0, 16))
                bits = mp.part == PART_A1 ? 0u : (uint32_t)sum;  // every row attends the summary keys alone
            else
                bits = (uint32_t)row_mask(mp, x, j0, j0_mod, sum);
            bits &= 0xFFFFu;
            if (__builtin_amdgcn_ballot_w64(bits != 0u) != 0ull) return {j0, (bits >> (4 * g)) & 15u};
        }
    }
    __device__ Tile cols(const ColLane& y, int j0, int qshift, bool any_summary, int g) {
        for (;;) {
            const int q0 = visit();
            if (q0 < 0) return {-1, 0u};
            const int i0 = q0 - qshift;  // first query as the masks see it
            if (block_full32(mp.pattern, mp.part, dl, mp.c, mp.w, i0, i0 + 15, j0, j0 + 15)) return {q0, 15u};
            uint32_t bits;
            if (mp.pattern == FIXED && far_block(FIXED, dl, i0, j0, 16)) {
                // summary keys alone, attended by every later query (the entries ascend)
                if (mp.part == PART_A1 || !any_summary) {
                    e = e1;
                    return {-1, 0u};
                }
                bits = y.summary ? 0xFFFFu : 0u;
            } else {
                bits = (uint32_t)col_mask(mp, y, i0, mod_l(dl, i0)) & 0xFFFFu;
            }
            if (__builtin_amdgcn_ballot_w64(bits != 0u) != 0ull) return {q0, (bits >> (4 * g)) & 15u};
        }
    }
};

// Runs body(tile, rows of operand A, rows of operand B) over a wave's tiles,
// the operands loaded one tile ahead where they fit the registers.
template <int D, bool TWO, typename Next, typename F>
__device__ inline void for_tiles(Next&& next, const float* pa, const float* pb, int64_t ss, int g, int r, F&& body) {
    Tile cur = next();
    if constexpr (F32<D>::PREFETCH) {
        RowOp<D> a, b;
        if (cur.first >= 0) {
            a.load(pa + (int64_t)cur.first * ss, ss, g, r);
            if constexpr (TWO) b.load(pb + (int64_t)cur.first * ss, ss, g, r);
        }
        while (cur.first >= 0) {
            const Tile nxt = next();
            RowOp<D> an, bn;
            if (nxt.first >= 0) {
                an.load(pa + (int64_t)nxt.first * ss, ss, g, r);
                if constexpr (TWO) bn.load(pb + (int64_t)nxt.first * ss, ss, g, r);
            }
            body(cur, a, b);
            a = an;
            if constexpr (TWO) b = bn;
            cur = nxt;
        }
    } else {
        while (cur.first >= 0) {
            RowOp<D> a, b;
            a.load(pa + (int64_t)cur.first * ss, ss, g, r);
            if constexpr (TWO) b.load(pb + (int64_t)cur.first * ss, ss, g, r);
            body(cur, a, b);
            cur = next();
        }
    }
}

// One tile of the online softmax: scores s to weights, the running state rescaled.
template <int D>
__device__ inline f32x4 softmax_step(const Tile& t, f32x4 s, float scale, float& m_run, float& l_run, f32x4* acc) {
    float mloc = -INFINITY;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        s[x] = (t.mask >> x) & 1u ? s[x] * scale : -INFINITY;
        mloc = fmaxf(mloc, s[x]);
    }
    const float m_new = fmaxf(m_run, max_over_g(mloc));
    // rows with nothing attended so far keep m = -inf; 0 as reference gives p = 0
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = expf(m_run - m_ref);
    float psum = 0.f;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        s[x] = expf(s[x] - m_ref);
        psum += s[x];
    }
    l_run = fmaf(l_run, alpha, psum);
    m_run = m_new;
#pragma unroll
    for (int db = 0; db < F32<D>::DB; ++db) acc[db] *= alpha;
    return s;
}

// Entries of row block qb and column block kb a walk visits (see WALK_*).
__device__ inline void row_entries(const AttnArgs& a, const int32_t* row_ptr, int lay, int qb, int* e0, int* e1) {
    *e0 = a.walk == WALK_BAND ? max(0, qb - band_blocks(a)) : 0;
    *e1 = qb + 1;
    if (a.walk != WALK_LAYOUT) return;
    const int64_t rp = (int64_t)lay * (a.nq + 1) + qb;
    *e0 = __builtin_amdgcn_readfirstlane(row_ptr[rp]);
    *e1 = __builtin_amdgcn_readfirstlane(row_ptr[rp + 1]);
}
__device__ inline void col_entries(const AttnArgs& a, const int32_t* col_ptr, int lay, int kb, int* e0, int* e1) {
    *e0 = kb;
    *e1 = a.walk == WALK_BAND ? min(a.nq, kb + band_blocks(a) + 1) : a.nq;
    if (a.walk != WALK_LAYOUT) return;
    const int64_t cp = (int64_t)lay * (a.nq + 1) + kb;
    *e0 = __builtin_amdgcn_readfirstlane(col_ptr[cp]);
    *e1 = __builtin_amdgcn_readfirstlane(col_ptr[cp + 1]);
}

// Forward.  grid: (16-row groups, heads, batch), longest rows first.
template <int D>
__global__ void __launch_bounds__(kF32Threads) __attribute__((amdgpu_waves_per_eu(4)))
fwd_f32_kernel(AttnArgs a, const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
               const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
               float* __restrict__ o, float* __restrict__ lse) {
    using C = F32<D>;
    __shared__ __attribute__((aligned(16))) float sO[kF32Waves][16 * C::RS];
    __shared__ float sM[kF32Waves][16], sL[kF32Waves][16];
    const int h = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = tid % 64, g = lane / 16, r = lane % 16;
    const int w = __builtin_amdgcn_readfirstlane(tid / 64);
    const MaskParams mp = head_mask_params(a, a.pattern, a.mode, h);
    const int64_t base = head_base(a, b, h);
    for (int rg = a.n / 16 - 1 - (int)blockIdx.x; rg >= 0; rg -= (int)gridDim.x) {
        const int row0 = 16 * rg, i0 = row0 - a.qshift;
        const RowLane rl = row_lane(i0 + r, a.dl);
        RowOp<D> qf;
        qf.load(q + base + (int64_t)row0 * a.ss, a.ss, g, r);
        f32x4 acc[C::DB];
#pragma unroll
        for (int db = 0; db < C::DB; ++db) acc[db] = zero4();
        float m_run = -INFINITY, l_run = 0.f;
        int e0, e1;
        row_entries(a, row_ptr, head_layout(a, h), row0 / a.block, &e0, &e1);
        TileWalk walk;
        walk.init(a, mp, col_idx, e0, e1, w);
        for_tiles<D, false>([&] { return walk.rows(rl, i0, g); }, k + base, nullptr, a.ss, g, r,
                            [&](const Tile& t, const RowOp<D>& kf, const RowOp<D>&) {
            ColOp<D> vt;
            vt.load(v + base + (int64_t)t.first * a.ss, a.ss, g, r);
            // key t.first + 4 g + t, query row0 + r
            vt.accumulate(softmax_step<D>(t, dot_tile<D>(kf, qf), a.scale, m_run, l_run, acc), acc);
        });
        if (non_finite<D>(acc)) {
#pragma unroll
            for (int db = 0; db < C::DB; ++db) acc[db] = zero4();
            m_run = -INFINITY;
            l_run = 0.f;
            walk.init(a, mp, col_idx, e0, e1, w);
            for (Tile t = walk.rows(rl, i0, g); t.first >= 0; t = walk.rows(rl, i0, g)) {
                const int gg = opaque(g), rr = opaque(r);
                const int64_t at = base + (int64_t)t.first * a.ss;
                const f32x4 s = dot_rows<D>(k + at, q + base + (int64_t)row0 * a.ss, a.ss, gg, rr);
                accumulate_attended<D>(v + at, a.ss, softmax_step<D>(t, s, a.scale, m_run, l_run, acc), t.mask, acc, gg, rr);
            }
        }
        // combine the waves' states, in wave order
        l_run = sum_over_g(l_run);
        store_partial<D>(sO[w], acc, g, r);
        if (g == 0) {
            sM[w][r] = m_run;
            sL[w][r] = l_run;
        }
        __syncthreads();
        const int row = tid / 32;
        constexpr int N = D / 32;  // elements per thread
        const int col = (tid % 32) * N;
        float mx = -INFINITY;
#pragma unroll
        for (int x = 0; x < kF32Waves; ++x) mx = fmaxf(mx, sM[x][row]);
        float l_tot = 0.f, out[N];
#pragma unroll
        for (int c = 0; c < N; ++c) out[c] = 0.f;
#pragma unroll
        for (int x = 0; x < kF32Waves; ++x) {
            const float wt = sM[x][row] == -INFINITY ? 0.f : expf(sM[x][row] - mx);
            l_tot = fmaf(wt, sL[x][row], l_tot);
#pragma unroll
            for (int c = 0; c < N; ++c) out[c] = fmaf(wt, sO[x][row * C::RS + col + c], out[c]);
        }
        float* orow = o + base + (int64_t)(row0 + row) * a.ss + col;
        float* lrow = lse + stat_index(a, b, h, row0 + row);
        float w1 = 0.f, w2 = 1.f, z = l_tot, res = l_tot > 0.f ? mx + logf(l_tot) : -INFINITY;
        if (a.epilogue == EPI_MERGE) {
            // combine with the O and LSE of the disjoint part already there
            const float lse1 = *lrow;
            const float top = fmaxf(lse1, res);
            w1 = lse1 == -INFINITY ? 0.f : expf(lse1 - top);
            w2 = l_tot > 0.f ? expf(mx - top) : 0.f;
            z = w1 + w2 * l_tot;
            res = z > 0.f ? top + logf(z) : -INFINITY;
        }
        const float inv = z > 0.f ? 1.f / z : 0.f;
#pragma unroll
        for (int c = 0; c < N; ++c)
            orow[c] = a.epilogue == EPI_MERGE ? (w1 * orow[c] + w2 * out[c]) * inv : out[c] * inv;
        __syncthreads();  // LSE read by all its row's threads; the partials are free again
        if (tid % 32 == 0) *lrow = res;
    }
}

// Score gradients of a tile in the dQ kernel's view, zero where a pair is not attended.
__device__ inline f32x4 score_grad(const Tile& t, f32x4 s, f32x4 dp, float scale, float L, float nd) {
    f32x4 ds;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const float p = expf(fmaf(s[x], scale, -L));
        ds[x] = (t.mask >> x) & 1u ? p * (dp[x] + nd) : 0.f;
    }
    return ds;
}

// Sums the waves' partials [16][D] in LDS into this thread's D / 32 elements.
template <int D>
__device__ inline void sum_partials(const float (*s)[16 * F32<D>::RS], int row, int col, float* out) {
#pragma unroll
    for (int c = 0; c < D / 32; ++c) out[c] = 0.f;
#pragma unroll
    for (int x = 0; x < kF32Waves; ++x)
#pragma unroll
        for (int c = 0; c < D / 32; ++c) out[c] += s[x][row * F32<D>::RS + col + c];
}

// dQ.  With a.row_stats it also forms -D_i = -dO_i . O_i of its rows and writes
// it for the dK / dV kernel.  grid as the forward's.
template <int D>
__global__ void __launch_bounds__(kF32Threads) __attribute__((amdgpu_waves_per_eu(2)))
bwd_dq_f32_kernel(AttnArgs a, const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                  const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                  const float* __restrict__ o, const float* __restrict__ dout, const float* __restrict__ lse,
                  float* __restrict__ ndelta, float* __restrict__ dq) {
    using C = F32<D>;
    __shared__ __attribute__((aligned(16))) float sAcc[kF32Waves][16 * C::RS];
    const int h = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = tid % 64, g = lane / 16, r = lane % 16;
    const int w = __builtin_amdgcn_readfirstlane(tid / 64);
    const MaskParams mp = head_mask_params(a, a.pattern, a.mode, h);
    const int64_t base = head_base(a, b, h);
    for (int rg = a.n / 16 - 1 - (int)blockIdx.x; rg >= 0; rg -= (int)gridDim.x) {
        const int row0 = 16 * rg, i0 = row0 - a.qshift;
        const RowLane rl = row_lane(i0 + r, a.dl);
        RowOp<D> qf, of;
        qf.load(q + base + (int64_t)row0 * a.ss, a.ss, g, r);
        of.load(dout + base + (int64_t)row0 * a.ss, a.ss, g, r);
        const int64_t si = stat_index(a, b, h, row0 + r);
        const float L = lse[si];
        float nd;
        if (a.row_stats) {
            RowOp<D> oo;
            oo.load(o + base + (int64_t)row0 * a.ss, a.ss, g, r);
            float part = 0.f;
#pragma unroll
            for (int s = 0; s < C::KS; ++s)
#pragma unroll
                for (int t = 0; t < 4; ++t) part = fmaf(oo.x[s][t], of.x[s][t], part);
            nd = -sum_over_g(part);
            if (w == 0 && g == 0) ndelta[si] = nd;
        } else {
            nd = ndelta[si];
        }
        f32x4 acc[C::DB];
#pragma unroll
        for (int db = 0; db < C::DB; ++db) acc[db] = zero4();
        int e0, e1;
        row_entries(a, row_ptr, head_layout(a, h), row0 / a.block, &e0, &e1);
        TileWalk walk;
        walk.init(a, mp, col_idx, e0, e1, w);
        for_tiles<D, true>([&] { return walk.rows(rl, i0, g); }, k + base, v + base, a.ss, g, r,
                           [&](const Tile& t, const RowOp<D>& kf, const RowOp<D>& vf) {
            ColOp<D> kt;
            kt.load(k + base + (int64_t)t.first * a.ss, a.ss, g, r);
            const f32x4 s = dot_tile<D>(kf, qf), dp = dot_tile<D>(vf, of);
            kt.accumulate(score_grad(t, s, dp, a.scale, L, nd), acc);
        });
        if (non_finite<D>(acc)) {
#pragma unroll
            for (int db = 0; db < C::DB; ++db) acc[db] = zero4();
            walk.init(a, mp, col_idx, e0, e1, w);
            const int64_t own = base + (int64_t)row0 * a.ss;
            for (Tile t = walk.rows(rl, i0, g); t.first >= 0; t = walk.rows(rl, i0, g)) {
                const int gg = opaque(g), rr = opaque(r);
                const int64_t at = base + (int64_t)t.first * a.ss;
                const f32x4 s = dot_rows<D>(k + at, q + own, a.ss, gg, rr);
                const f32x4 dp = dot_rows<D>(v + at, dout + own, a.ss, gg, rr);
                accumulate_attended<D>(k + at, a.ss, score_grad(t, s, dp, a.scale, L, nd), t.mask, acc, gg, rr);
            }
        }
        store_partial<D>(sAcc[w], acc, g, r);
        __syncthreads();
        const int row = tid / 32, col = (tid % 32) * (D / 32);
        float out[D / 32];
        sum_partials<D>(sAcc, row, col, out);
        float* drow = dq + base + (int64_t)(row0 + row) * a.ss + col;
#pragma unroll
        for (int c = 0; c < D / 32; ++c) drow[c] = (a.epilogue == EPI_ADD ? drow[c] : 0.f) + out[c] * a.scale;
        __syncthreads();
    }
}

// Weights and score gradients of a tile in the dK / dV kernel's view, zero where a
// pair is not attended.
__device__ inline void weights(const Tile& t, f32x4 s, f32x4 dp, float scale, const float* L, const float* nd, f32x4* p,
                               f32x4* ds) {
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const bool on = (t.mask >> x) & 1u;
        (*p)[x] = on ? expf(fmaf(s[x], scale, -L[x])) : 0.f;
        (*ds)[x] = on ? (*p)[x] * (dp[x] + nd[x]) : 0.f;
    }
}

// dK and dV.  grid: (16-key groups, heads, batch), longest columns first.
template <int D>
__global__ void __launch_bounds__(kF32Threads) __attribute__((amdgpu_waves_per_eu(2)))
bwd_dkdv_f32_kernel(AttnArgs a, const int32_t* __restrict__ col_ptr, const int32_t* __restrict__ row_idx,
                    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                    const float* __restrict__ dout, const float* __restrict__ lse, const float* __restrict__ ndelta,
                    float* __restrict__ dk, float* __restrict__ dv) {
    using C = F32<D>;
    __shared__ __attribute__((aligned(16))) float sAcc[kF32Waves][16 * C::RS];
    const int h = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x, lane = tid % 64, g = lane / 16, r = lane % 16;
    const int w = __builtin_amdgcn_readfirstlane(tid / 64);
    const MaskParams mp = head_mask_params(a, a.pattern, a.mode, h);
    const int64_t base = head_base(a, b, h);
    for (int kg = (int)blockIdx.x; kg < a.n / 16; kg += (int)gridDim.x) {
        const int j0 = 16 * kg;
        const ColLane cl = col_lane(j0 + r, a.dl, a.c, mp.w);
        const bool any_summary = __builtin_amdgcn_ballot_w64(cl.summary) != 0ull;
        RowOp<D> kf, vf;
        kf.load(k + base + (int64_t)j0 * a.ss, a.ss, g, r);
        vf.load(v + base + (int64_t)j0 * a.ss, a.ss, g, r);
        f32x4 dkacc[C::DB], dvacc[C::DB];
#pragma unroll
        for (int db = 0; db < C::DB; ++db) dkacc[db] = dvacc[db] = zero4();
        int e0, e1;
        col_entries(a, col_ptr, head_layout(a, h), j0 / a.block, &e0, &e1);
        auto load_stats = [&](const Tile& t, int g, float* L, float* nd) {
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int64_t si = stat_index(a, b, h, t.first + 4 * g + x);
                L[x] = lse[si];
                nd[x] = ndelta[si];
            }
        };
        TileWalk walk;
        walk.init(a, mp, row_idx, e0, e1, w);
        for_tiles<D, true>([&] { return walk.cols(cl, j0, a.qshift, any_summary, g); }, q + base, dout + base, a.ss, g, r,
                           [&](const Tile& t, const RowOp<D>& qf, const RowOp<D>& of) {
            float L[4], nd[4];  // queries t.first + 4 g + x
            load_stats(t, g, L, nd);
            ColOp<D> ot, qt;
            ot.load(dout + base + (int64_t)t.first * a.ss, a.ss, g, r);
            const f32x4 s = dot_tile<D>(qf, kf), dp = dot_tile<D>(of, vf);
            qt.load(q + base + (int64_t)t.first * a.ss, a.ss, g, r);
            f32x4 p, ds;
            weights(t, s, dp, a.scale, L, nd, &p, &ds);
            ot.accumulate(p, dvacc);
            qt.accumulate(ds, dkacc);
        });
        if (non_finite<D>(dkacc) || non_finite<D>(dvacc)) {
#pragma unroll
            for (int db = 0; db < C::DB; ++db) dkacc[db] = dvacc[db] = zero4();
            walk.init(a, mp, row_idx, e0, e1, w);
            const int64_t own = base + (int64_t)j0 * a.ss;
            for (Tile t = walk.cols(cl, j0, a.qshift, any_summary, g); t.first >= 0;
                 t = walk.cols(cl, j0, a.qshift, any_summary, g)) {
                const int gg = opaque(g), rr = opaque(r);
                const int64_t at = base + (int64_t)t.first * a.ss;
                float L[4], nd[4];
                load_stats(t, gg, L, nd);
                f32x4 p, ds;
                weights(t, dot_rows<D>(q + at, k + own, a.ss, gg, rr), dot_rows<D>(dout + at, v + own, a.ss, gg, rr), a.scale,
                        L, nd, &p, &ds);
                accumulate_attended<D>(dout + at, a.ss, p, t.mask, dvacc, gg, rr);
                accumulate_attended<D>(q + at, a.ss, ds, t.mask, dkacc, gg, rr);
            }
        }
        const int row = tid / 32, col = (tid % 32) * (D / 32);
        const int64_t at = base + (int64_t)(j0 + row) * a.ss + col;
        const bool add = a.epilogue == EPI_ADD;
        float out[D / 32];
        store_partial<D>(sAcc[w], dvacc, g, r);
        __syncthreads();
        sum_partials<D>(sAcc, row, col, out);
#pragma unroll
        for (int c = 0; c < D / 32; ++c) dv[at + c] = (add ? dv[at + c] : 0.f) + out[c];
        __syncthreads();
        store_partial<D>(sAcc[w], dkacc, g, r);
        __syncthreads();
        sum_partials<D>(sAcc, row, col, out);
#pragma unroll
        for (int c = 0; c < D / 32; ++c) dk[at + c] = (add ? dk[at + c] : 0.f) + out[c] * a.scale;
        __syncthreads();
    }
}

dim3 strip_grid(const AttnArgs& a) {
    const int64_t strips = a.n / 16;
    return dim3((unsigned)(strips < kF32MaxGrid ? strips : kF32MaxGrid), (unsigned)a.heads, (unsigned)a.batch);
}

template <int D>
hipError_t launch_fwd(const AttnArgs& a, const void* q, const void* k, const void* v, void* o, float* lse,
                      hipStream_t stream) {
    hipLaunchKernelGGL((fwd_f32_kernel<D>), strip_grid(a), dim3(kF32Threads), 0, stream, a, a.row_ptr, a.col_idx,
                       (const float*)q, (const float*)k, (const float*)v, (float*)o, lse);
    return hipGetLastError();
}

template <int D>
hipError_t launch_bwd(const AttnArgs& a, const void* q, const void* k, const void* v, const void* o, const void* dout,
                      const float* lse, void* dq, void* dk, void* dv, const BwdWorkspace& ws, hipStream_t stream,
                      int parts) {
    AttnArgs aq = a;
    // the statistics always go with dQ (no call has them alone in fp32); its grid covers every row
    aq.row_stats = (parts & BWD_PRE) != 0;
    if (parts & BWD_DQ)
        hipLaunchKernelGGL((bwd_dq_f32_kernel<D>), strip_grid(a), dim3(kF32Threads), 0, stream, aq, a.row_ptr,
                           a.col_idx, (const float*)q, (const float*)k, (const float*)v, (const float*)o,
                           (const float*)dout, lse, ws.ndelta, (float*)dq);
    if (parts & BWD_DKDV)
        hipLaunchKernelGGL((bwd_dkdv_f32_kernel<D>), strip_grid(a), dim3(kF32Threads), 0, stream, a, a.col_ptr,
                           a.row_idx, (const float*)q, (const float*)k, (const float*)v, (const float*)dout, lse,
                           ws.ndelta, (float*)dk, (float*)dv);
    return hipGetLastError();
}

}  // namespace

hipError_t fwd_f32(const AttnArgs& a, const void* q, const void* k, const void* v, void* o, float* lse,
                   hipStream_t stream) {
    switch (a.d) {
    case 32: return launch_fwd<32>(a, q, k, v, o, lse, stream);
    case 64: return launch_fwd<64>(a, q, k, v, o, lse, stream);
    default: return launch_fwd<128>(a, q, k, v, o, lse, stream);
    }
}

hipError_t bwd_f32(const AttnArgs& a, const void* q, const void* k, const void* v, const void* o, const void* dout,
                   const float* lse, void* dq, void* dk, void* dv, const BwdWorkspace& ws, hipStream_t stream,
                   int parts) {
    switch (a.d) {
    case 32: return launch_bwd<32>(a, q, k, v, o, dout, lse, dq, dk, dv, ws, stream, parts);
    case 64: return launch_bwd<64>(a, q, k, v, o, dout, lse, dq, dk, dv, ws, stream, parts);
    default: return launch_bwd<128>(a, q, k, v, o, dout, lse, dq, dk, dv, ws, stream, parts);
    }
}

}  // namespace sa
