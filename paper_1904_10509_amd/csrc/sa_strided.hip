// Strided merged heads (A1 u A2, bf16) in one pass: the band A1 = {i - l .. i} and
// the rest of A2 by residue classes (Sec. 5.5) in the same kernel.
//
// Write position i as m l + r (class r, step m).  The band of a row is a run of
// neighbouring rows, so its products want query tiles of neighbouring r; A2 \ A1
// = {m' <= m - 2 of the same class} wants query tiles of neighbouring m.  A
// workgroup therefore takes the 256 rows of 16 steps x 16 classes and works in
// two phases of 16 units each, shared out over its waves:
//   band:   unit u is the 16 rows of step m0 + u, r = r0 .. r0 + 15;
//   class:  unit u is the 16 rows of class r0 + u, m = m0 .. m0 + 15.
// Between the phases the units' fp32 state (O, running maximum and sum; dQ; dK and dV) changes owner
// through LDS, so every output is summed in fp32 and written once, where
// separate band and class kernels write, read back and rewrite it in bf16 and
// read every tensor twice.
//
// A wave walks its unit's other side in chunks of 32 rows (of neighbouring rows
// in the band, l rows apart in a class), alone, and there is no barrier inside a
// phase.  In the class phase no two units share rows.  In the band phase they do
// (units l rows apart; neighbouring tiles), and each reads its own: where the band
// kernel's tiles of 64 rows serve a longer band, that is what the one-pass form loses.  A chunk goes to the wave's own part of LDS by direct loads,
// whole rows at a time (as row operands straight into registers, 16 rows' 16
// bytes per 16 lanes, the same rows took 52 cycles per KiB and CU: forward at n =
// 12,288, l = 128 93 us).  Both its forms, by rows and transposed, are read into
// registers at once, and the next chunk's loads are issued into the same place
// before the exponentials.
//
// Workgroups of neighbouring r of one head and step range share their band rows
// and those of one head their class rows, so each XCD takes a consecutive range
// of them.
#include "sa_bwd_kernels.h"
#include "sa_finite.h"
#include "sa_strided.h"

namespace sa {

namespace {

// W waves per workgroup, 16 / W units each: eight where two workgroups then share
// a compute unit (forward and dQ up to d = 64: one's exchange beside the other's
// products, 49.9 -> 48.0 and 59.5 -> 55.6 us at n = 12,288, l = 128; at d = 128 one
// workgroup's LDS and registers fill it), sixteen for dK / dV up to d = 64, whose
// accumulators of two units would spill.
template <int D, int W>
struct SCfg {
    static constexpr int NW = W;
    static constexpr int NT = 64 * NW;
    static constexpr int UNITS = 16 / NW;
    static constexpr int WAVES_PER_EU = D == 128 ? 2 : 4;
    static constexpr int KS = D / 32;
    static constexpr int DB = D / 16;
    static constexpr int TILE = 32 * D;  // elements of a staged chunk
    // Exchange of a unit's rows: element d of (unit u, row t) at u XA + t XB + d.
    // Both strides are odd multiples of 4 words (of 64 banks): writing a unit's rows
    // and reading one row of every unit are free of bank conflicts.
    static constexpr int XB = D + 4;
    static constexpr int XA = 16 * XB + 4;
};

// 16 rows as row operands (a unit's own rows), clamped to last.
template <int D>
__device__ inline void load_unit(bf16x8* x, const uint16_t* p, int64_t stride, int first, int last, int g, int r) {
    const uint16_t* row = p + (int64_t)min(first + r, last) * stride + 8 * g;
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) x[ks] = ld_bf16x8(row + 32 * ks);
}

// This lane's pairs of chunk c: bit 16 kb + t after the shift.
__device__ inline uint32_t chunk_mask(const Walk& w, int c, int g) {
    return (uint32_t)(bit_range(w.lo - 32 * c, w.hi - 32 * c) & 0xFFFFFFFFull) >> (4 * g);
}

// Zero where a pair is not attended.
__device__ inline void mask_pairs(f32x4* x, uint64_t bits) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) x[kb][e] = select_or_zero(bit_lane_mask(bits, 16 * kb + e), x[kb][e]);
}

// Runs body(full, chunk index, next) over a unit's chunks, rows of pa in the LDS
// tile ta and rows of pb in tb; full (wave-uniform): every pair of the chunk is
// attended.  The body calls next() once it has read the tiles: the next chunk's
// rows are loaded in their place.
template <int D, typename F>
__device__ inline void for_chunks(const Walk& w, const uint16_t* pa, const uint16_t* pb, const uint16_t* ta,
                                  const uint16_t* tb, int lane, F&& body) {
    const int chunks = w.on ? (w.count + 31) / 32 : 0;
    if (chunks <= 0) return;
    TileLoader<D, 32, 1> ld;
    ld.init(w.stride, 0, lane);
    const uint32_t da = lds_addr(ta), db = lds_addr(tb);
    auto load = [&](int c) {
        const int64_t at = (int64_t)(w.first + 32 * c) * w.stride;
        const int rows = w.last - (w.first + 32 * c) + 1;  // rows past the last are filled with it
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the tiles have been read
        if (rows >= 32) {
            ld.issue(pa + at, da);
            ld.issue(pb + at, db);
        } else {
            ld.issue_rows(pa + at, da, w.stride, rows, lane);
            ld.issue_rows(pb + at, db, w.stride, rows, lane);
        }
    };
    load(0);
    for (int c = 0; c < chunks; ++c) {
        wait_loads_upto<0>();
        asm volatile("" ::: "memory");  // reads of the tiles stay after the wait
        body(32 * c >= w.full_lo && 32 * c + 31 <= w.full_hi, c, [&] {
            if (c + 1 < chunks) load(c + 1);
        });
    }
}

// Hands the units' accumulators (lane (g, r): row r, elements 16 db + 4 g + t) from
// the band's rows to the classes' rows.  Uses all of LDS: barriers on both sides.
template <int D, int W>
__device__ inline void exchange_rows(float* x, f32x4 (*acc)[SCfg<D, W>::DB], int w, int g, int r) {
    using C = SCfg<D, W>;
    __syncthreads();
#pragma unroll
    for (int uu = 0; uu < C::UNITS; ++uu)
#pragma unroll
        for (int db = 0; db < C::DB; ++db)
            *reinterpret_cast<f32x4*>(x + (w + W * uu) * C::XA + r * C::XB + 16 * db + 4 * g) = acc[uu][db];
    __syncthreads();
#pragma unroll
    for (int uu = 0; uu < C::UNITS; ++uu)
#pragma unroll
        for (int db = 0; db < C::DB; ++db)
            acc[uu][db] = *reinterpret_cast<const f32x4*>(x + r * C::XA + (w + W * uu) * C::XB + 16 * db + 4 * g);
    __syncthreads();
}

template <int D, int W, bool STATS>
struct SShared {
    static constexpr int kWave = 2 * SCfg<D, W>::TILE * 2 + (STATS ? 256 : 0);  // bytes of a wave's tiles
    static constexpr int kStage = W * kWave;
    static constexpr int kExchange = 16 * SCfg<D, W>::XA * 4;
    static constexpr int kBytes = kStage > kExchange ? kStage : kExchange;
};

template <int D, int W>
__global__ void __launch_bounds__((SCfg<D, W>::NT)) __attribute__((amdgpu_waves_per_eu(SCfg<D, W>::WAVES_PER_EU)))
strided_fwd_kernel(AttnArgs a, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                   const uint16_t* __restrict__ v, uint16_t* __restrict__ o, float* __restrict__ lse) {
    using C = SCfg<D, W>;
    __shared__ __attribute__((aligned(16))) unsigned char smem[SShared<D, W, false>::kBytes];
    __shared__ float sM[16][17], sL[16][17];  // [unit][row]
    __shared__ uint32_t sBad;
    STile t;
    if (!strided_tile(a, blockIdx.x, &t)) return;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid / 64);
    const int64_t base = head_base(a, t.b, t.h);
    const uint16_t* tK = reinterpret_cast<const uint16_t*>(smem + w * SShared<D, W, false>::kWave);
    const uint16_t* tV = tK + C::TILE;
    const float c2 = a.scale_log2;

    f32x4 acc[SCfg<D, W>::UNITS][C::DB];
    float m_run[SCfg<D, W>::UNITS], l_run[SCfg<D, W>::UNITS];
    if (tid == 0) sBad = 0;
    auto run = [&](auto again) {
    constexpr bool kAgain = decltype(again)::value;
    const int lane = kAgain ? opaque(tid % 64) : tid % 64, g = lane / 16, r = lane % 16;
    TileReader<D> rd;
    rd.init(g, r);
    auto unit = [&](bool cls, int uu) {
        const Walk wk = query_walk(a, t, cls, w + C::NW * uu, r);
        if (!wk.on) return;
        bf16x8 qf[C::KS];
        load_unit<D>(qf, q + base + wk.at, wk.stride, wk.own, wk.own_last, g, r);
        for_chunks<D>(wk, k + base + wk.at, v + base + wk.at, tK, tV, lane, [&](bool full, int c, auto next) {
            f32x4 s[2];  // key 16 kb + 4 g + x, query r
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                s[kb] = zero4();
#pragma unroll
                for (int ks = 0; ks < C::KS; ++ks) s[kb] = mfma_16x16x32(rd.row(tK, 16 * kb, ks), qf[ks], s[kb]);
            }
            bf16x8 vt[C::DB];
#pragma unroll
            for (int db = 0; db < C::DB; ++db) vt[db] = rd.tr(tV, 0, 16, db);
            next();
            if (!full) {
                const uint64_t bits = chunk_mask(wk, c, g);
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        s[kb][x] = select_or_neg_inf(bit_lane_mask(bits, 16 * kb + x), s[kb][x]);
            }
            float mloc = -INFINITY;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                mloc = fmaxf(fmaxf(mloc, s[kb][0]), s[kb][1]);
                mloc = fmaxf(fmaxf(mloc, s[kb][2]), s[kb][3]);
            }
            const float m_new = fmaxf(m_run[uu], max_over_g(mloc));
            // rows with nothing attended so far keep m = -inf; 0 as reference gives p = 0
            const float m_ref = m_new == -INFINITY ? 0.f : m_new;
            const float neg = -m_ref * c2;
            float psum = 0.f;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    s[kb][x] = exp2_fast(fmaf(s[kb][x], c2, neg));
                    psum += s[kb][x];
                }
            const bf16x8 pf = pack_bf16x8(s[0], s[1]);
            const float alpha = exp2_fast((m_run[uu] - m_ref) * c2);
            l_run[uu] = fmaf(l_run[uu], alpha, psum);
            m_run[uu] = m_new;
            if constexpr (kAgain) {
#pragma unroll
                for (int db = 0; db < C::DB; ++db) acc[uu][db] *= alpha;
                accumulate_attended<C::DB>(vt, pf, full ? 0 : wk.lo - 32 * c, full ? 31 : wk.hi - 32 * c, g, acc[uu]);
                return;
            }
#pragma unroll
            for (int db = 0; db < C::DB; ++db) acc[uu][db] = mfma_16x16x32(vt[db], pf, acc[uu][db] * alpha);
        });
    };
#pragma unroll
    for (int uu = 0; uu < SCfg<D, W>::UNITS; ++uu) {
#pragma unroll
        for (int db = 0; db < C::DB; ++db) acc[uu][db] = zero4();
        m_run[uu] = -INFINITY;
        l_run[uu] = 0.f;
        unit(false, uu);
        l_run[uu] = sum_over_g(l_run[uu]);
        if (g == 0) {
            sM[w + C::NW * uu][r] = m_run[uu];
            sL[w + C::NW * uu][r] = l_run[uu];
        }
    }
    exchange_rows<D, W>(reinterpret_cast<float*>(smem), acc, w, g, r);
#pragma unroll
    for (int uu = 0; uu < SCfg<D, W>::UNITS; ++uu) {
        const int u = w + C::NW * uu;
        m_run[uu] = sM[r][u];
        l_run[uu] = g == 0 ? sL[r][u] : 0.f;  // one lane of the row carries the sum
        unit(true, uu);
        const float l_tot = sum_over_g(l_run[uu]);
        const Walk wk = query_walk(a, t, true, u, r);
        if (!wk.on || wk.own + r > wk.own_last) continue;
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        uint16_t* orow = o + base + wk.at + (int64_t)(wk.own + r) * wk.stride;
#pragma unroll
        for (int db = 0; db < C::DB; ++db)
            *reinterpret_cast<uint2*>(orow + db * 16 + 4 * g) = pack_bf16x4_bits(acc[uu][db] * inv);
        if (g == 0)
            lse[stat_index(a, t.b, t.h, wk.stat + (int64_t)(wk.own + r) * wk.stat_stride)] =
                l_tot > 0.f ? m_run[uu] * a.scale + __logf(l_tot) : -INFINITY;
    }
    };
    run(std::false_type{});
    if (non_finite<C::UNITS * C::DB>(&acc[0][0])) sBad = 1;
    __syncthreads();
    if (sBad) run(std::true_type{});
}

// dQ.  With a.row_stats it also forms its rows' -D_i = -dO_i . O_i and -LSE_i
// log2 e and writes them for the dK / dV kernel.
template <int D, int W>
__global__ void __launch_bounds__((SCfg<D, W>::NT)) __attribute__((amdgpu_waves_per_eu(SCfg<D, W>::WAVES_PER_EU)))
strided_dq_kernel(AttnArgs a, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                  const uint16_t* __restrict__ v, const uint16_t* __restrict__ dout, const uint16_t* __restrict__ o,
                  const float* __restrict__ lse, float* __restrict__ nlse2, float* __restrict__ ndelta,
                  uint16_t* __restrict__ dq) {
    using C = SCfg<D, W>;
    __shared__ __attribute__((aligned(16))) unsigned char smem[SShared<D, W, false>::kBytes];
    __shared__ float sD[16][17], sN[16][17];  // -D and -LSE log2 e, [unit][row]
    __shared__ uint32_t sBad;
    STile t;
    if (!strided_tile(a, blockIdx.x, &t)) return;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid / 64);
    const int64_t base = head_base(a, t.b, t.h);
    const uint16_t* tK = reinterpret_cast<const uint16_t*>(smem + w * SShared<D, W, false>::kWave);
    const uint16_t* tV = tK + C::TILE;
    const float c2 = a.scale_log2;

    f32x4 acc[SCfg<D, W>::UNITS][C::DB];
    if (tid == 0) sBad = 0;
    auto run = [&](auto again) {
    constexpr bool kAgain = decltype(again)::value;
    const int lane = kAgain ? opaque(tid % 64) : tid % 64, g = lane / 16, r = lane % 16;
    TileReader<D> rd;
    rd.init(g, r);
    auto unit = [&](bool cls, int uu) {
        const int u = w + C::NW * uu;
        const Walk wk = query_walk(a, t, cls, u, r);
        if (!wk.on) return;
        bf16x8 qf[C::KS], of[C::KS];
        load_unit<D>(qf, q + base + wk.at, wk.stride, wk.own, wk.own_last, g, r);
        load_unit<D>(of, dout + base + wk.at, wk.stride, wk.own, wk.own_last, g, r);
        float nd, nl2;
        if (cls) {
            nd = sD[r][u];
            nl2 = sN[r][u];
        } else {
            const int i = min(wk.own + r, wk.own_last);
            const int64_t si = stat_index(a, t.b, t.h, i);
            if (a.row_stats) {
                bf16x8 oo[C::KS];
                load_unit<D>(oo, o + base, wk.stride, wk.own, wk.own_last, g, r);
                float part = 0.f;
#pragma unroll
                for (int ks = 0; ks < C::KS; ++ks) part += dot_bf16x8(of[ks], oo[ks]);
                nd = -sum_over_g(part);
                nl2 = -lse[si] * kLog2e;
                // (rows past the class range belong to the next step's unit)
                if (g == 0 && t.r0 + r < a.l && wk.own + r <= wk.own_last) {
                    ndelta[si] = nd;
                    nlse2[si] = nl2;
                }
            } else {
                nd = ndelta[si];
                nl2 = nlse2[si];
            }
            if (g == 0) {
                sD[u][r] = nd;
                sN[u][r] = nl2;
            }
        }
        for_chunks<D>(wk, k + base + wk.at, v + base + wk.at, tK, tV, lane, [&](bool full, int c, auto next) {
            f32x4 s[2], dp[2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                s[kb] = zero4();
                dp[kb] = f32x4{nd, nd, nd, nd};
#pragma unroll
                for (int ks = 0; ks < C::KS; ++ks) {
                    s[kb] = mfma_16x16x32(rd.row(tK, 16 * kb, ks), qf[ks], s[kb]);
                    dp[kb] = mfma_16x16x32(rd.row(tV, 16 * kb, ks), of[ks], dp[kb]);
                }
            }
            bf16x8 kt[C::DB];
#pragma unroll
            for (int db = 0; db < C::DB; ++db) kt[db] = rd.tr(tK, 0, 16, db);
            next();
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int x = 0; x < 4; ++x) s[kb][x] = exp2_fast(fmaf(s[kb][x], c2, nl2));
            if (!full) mask_pairs(s, chunk_mask(wk, c, g));
            s[0] *= dp[0];
            s[1] *= dp[1];
            if constexpr (kAgain) {
                if (!full) mask_pairs(s, chunk_mask(wk, c, g));
                accumulate_attended<C::DB>(kt, pack_bf16x8(s[0], s[1]), full ? 0 : wk.lo - 32 * c,
                                           full ? 31 : wk.hi - 32 * c, g, acc[uu]);
                return;
            }
            const bf16x8 dsf = pack_bf16x8(s[0], s[1]);
#pragma unroll
            for (int db = 0; db < C::DB; ++db) acc[uu][db] = mfma_16x16x32(kt[db], dsf, acc[uu][db]);
        });
    };
#pragma unroll
    for (int uu = 0; uu < SCfg<D, W>::UNITS; ++uu) {
#pragma unroll
        for (int db = 0; db < C::DB; ++db) acc[uu][db] = zero4();
        unit(false, uu);
    }
    exchange_rows<D, W>(reinterpret_cast<float*>(smem), acc, w, g, r);
#pragma unroll
    for (int uu = 0; uu < SCfg<D, W>::UNITS; ++uu) {
        unit(true, uu);
        const Walk wk = query_walk(a, t, true, w + C::NW * uu, r);
        if (!wk.on || wk.own + r > wk.own_last) continue;
        uint16_t* drow = dq + base + wk.at + (int64_t)(wk.own + r) * wk.stride;
#pragma unroll
        for (int db = 0; db < C::DB; ++db)
            *reinterpret_cast<uint2*>(drow + db * 16 + 4 * g) = pack_bf16x4_bits(acc[uu][db] * a.scale);
    }
    };
    run(std::false_type{});
    if (non_finite<C::UNITS * C::DB>(&acc[0][0])) sBad = 1;
    __syncthreads();
    if (sBad) run(std::true_type{});
}

template <int D, int W>
__global__ void __launch_bounds__((SCfg<D, W>::NT)) __attribute__((amdgpu_waves_per_eu(SCfg<D, W>::WAVES_PER_EU)))
strided_dkdv_kernel(AttnArgs a, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                    const uint16_t* __restrict__ v, const uint16_t* __restrict__ dout,
                    const float* __restrict__ nlse2, const float* __restrict__ ndelta, uint16_t* __restrict__ dk,
                    uint16_t* __restrict__ dv) {
    using C = SCfg<D, W>;
    __shared__ __attribute__((aligned(16))) unsigned char smem[SShared<D, W, true>::kBytes];
    __shared__ uint32_t sBad[2];
    STile t;
    if (!strided_tile(a, blockIdx.x, &t)) return;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid / 64);
    const int64_t base = head_base(a, t.b, t.h);
    const uint16_t* tQ = reinterpret_cast<const uint16_t*>(smem + w * SShared<D, W, true>::kWave);
    const uint16_t* tO = tQ + C::TILE;
    float* tS = reinterpret_cast<float*>(smem + w * SShared<D, W, true>::kWave + 4 * C::TILE);  // a chunk's -LSE log2 e, then -D
    const float c2 = a.scale_log2;

    // At d = 128 dV and dK take a round each (S formed twice): accumulators of
    // both do not fit the registers.
    if (tid < 2) sBad[tid] = 0;
    auto round = [&](auto which) {
    constexpr bool kV = decltype(which)::value != 2, kK = decltype(which)::value != 1;
    f32x4 dvacc[SCfg<D, W>::UNITS][C::DB], dkacc[SCfg<D, W>::UNITS][C::DB];
    auto run = [&](auto again) {
    constexpr bool kAgain = decltype(again)::value;
    const int lane = kAgain ? opaque(tid % 64) : tid % 64, g = lane / 16, r = lane % 16;
    TileReader<D> rd;
    rd.init(g, r);
    auto unit = [&](bool cls, int uu) {
        const Walk wk = key_walk(a, t, cls, w + C::NW * uu, r);
        if (!wk.on || wk.count <= 0) return;
        bf16x8 kf[C::KS], vf[C::KS];
        load_unit<D>(kf, k + base + wk.at, wk.stride, wk.own, wk.own_last, g, r);
        load_unit<D>(vf, v + base + wk.at, wk.stride, wk.own, wk.own_last, g, r);
        // lanes 0 .. 31 fetch -LSE log2 e of a chunk's queries, the others -D
        const float* stats = (lane < 32 ? nlse2 : ndelta) + stat_index(a, t.b, t.h, wk.stat);
        auto stat = [&](int c) {
            return stats[(int64_t)min(wk.first + 32 * c + lane % 32, wk.last) * wk.stat_stride];
        };
        float st = stat(0);
        for_chunks<D>(wk, q + base + wk.at, dout + base + wk.at, tQ, tO, lane, [&](bool full, int c, auto next) {
            tS[lane] = st;
            asm volatile("" ::: "memory");  // (LDS operations of a wave complete in order)
            f32x4 p[2], ds[2];  // query 16 kb + 4 g + x, key r
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                p[kb] = zero4();
                if constexpr (kK) ds[kb] = *reinterpret_cast<const f32x4*>(tS + 32 + 16 * kb + 4 * g);
#pragma unroll
                for (int ks = 0; ks < C::KS; ++ks) {
                    p[kb] = mfma_16x16x32(rd.row(tQ, 16 * kb, ks), kf[ks], p[kb]);
                    if constexpr (kK) ds[kb] = mfma_16x16x32(rd.row(tO, 16 * kb, ks), vf[ks], ds[kb]);
                }
            }
            f32x4 nl[2];
            nl[0] = *reinterpret_cast<const f32x4*>(tS + 4 * g);
            nl[1] = *reinterpret_cast<const f32x4*>(tS + 16 + 4 * g);
            bf16x8 ot[C::DB], qt[C::DB];
            auto read = [&](bool o, bool q) {
#pragma unroll
                for (int db = 0; db < C::DB; ++db) {
                    if (o) ot[db] = rd.tr(tO, 0, 16, db);
                    if (q) qt[db] = rd.tr(tQ, 0, 16, db);
                }
            };
            if constexpr (!kAgain) {
                read(kV, kK);
                next();
            }
            st = stat(c + 1);  // (clamped to the last row past the end)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int x = 0; x < 4; ++x) p[kb][x] = exp2_fast(fmaf(p[kb][x], c2, nl[kb][x]));
            if (!full) mask_pairs(p, chunk_mask(wk, c, g));
            if constexpr (kK) {
                ds[0] *= p[0];
                ds[1] *= p[1];
            }
            if constexpr (kAgain) {
                const int lo = full ? 0 : wk.lo - 32 * c, hi = full ? 31 : wk.hi - 32 * c;
                if constexpr (kV) {
                    read(true, false);
                    accumulate_attended<C::DB>(ot, pack_bf16x8(p[0], p[1]), lo, hi, g, dvacc[uu]);
                }
                if constexpr (kK) {
                    read(false, true);
                    if (!full) mask_pairs(ds, chunk_mask(wk, c, g));
                    accumulate_attended<C::DB>(qt, pack_bf16x8(ds[0], ds[1]), lo, hi, g, dkacc[uu]);
                }
                next();
                return;
            }
            if constexpr (kV) {
                const bf16x8 pb = pack_bf16x8(p[0], p[1]);
#pragma unroll
                for (int db = 0; db < C::DB; ++db)
                    dvacc[uu][db] = mfma_16x16x32(ot[db], pb, dvacc[uu][db]);
            }
            if constexpr (kK) {
                const bf16x8 sb = pack_bf16x8(ds[0], ds[1]);
#pragma unroll
                for (int db = 0; db < C::DB; ++db)
                    dkacc[uu][db] = mfma_16x16x32(qt[db], sb, dkacc[uu][db]);
            }
        });
    };
#pragma unroll
    for (int uu = 0; uu < SCfg<D, W>::UNITS; ++uu) {
#pragma unroll
        for (int db = 0; db < C::DB; ++db) dvacc[uu][db] = dkacc[uu][db] = zero4();
        unit(false, uu);
    }
    if constexpr (kV) exchange_rows<D, W>(reinterpret_cast<float*>(smem), dvacc, w, g, r);
    if constexpr (kK) exchange_rows<D, W>(reinterpret_cast<float*>(smem), dkacc, w, g, r);
#pragma unroll
    for (int uu = 0; uu < SCfg<D, W>::UNITS; ++uu) {
        unit(true, uu);
        const Walk wk = key_walk(a, t, true, w + C::NW * uu, r);
        if (!wk.on || wk.own + r > wk.own_last) continue;
        const int64_t at = base + wk.at + (int64_t)(wk.own + r) * wk.stride;
#pragma unroll
        for (int db = 0; db < C::DB; ++db) {
            if constexpr (kV)
                *reinterpret_cast<uint2*>(dv + at + db * 16 + 4 * g) = pack_bf16x4_bits(dvacc[uu][db]);
            if constexpr (kK)
                *reinterpret_cast<uint2*>(dk + at + db * 16 + 4 * g) = pack_bf16x4_bits(dkacc[uu][db] * a.scale);
        }
    }
    };
    run(std::false_type{});
    uint32_t* const bad = &sBad[kV ? 0 : 1];
    if ((kV && non_finite<C::UNITS * C::DB>(&dvacc[0][0])) || (kK && non_finite<C::UNITS * C::DB>(&dkacc[0][0]))) *bad = 1;
    __syncthreads();
    if (*bad) run(std::true_type{});
    };
    if constexpr (D == 128) {
        round(std::integral_constant<int, 1>{});
        round(std::integral_constant<int, 2>{});
    } else {
        round(std::integral_constant<int, 3>{});
    }
}

template <int D>
hipError_t launch_fwd(const AttnArgs& a, const void* q, const void* k, const void* v, void* o, float* lse,
                      hipStream_t stream) {
    hipLaunchKernelGGL((strided_fwd_kernel<D, 8>), dim3((unsigned)strided_groups(a)), dim3(512), 0, stream, a,
                       (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (uint16_t*)o, lse);
    return hipGetLastError();
}

template <int D>
hipError_t launch_bwd(const AttnArgs& a, const void* q, const void* k, const void* v, const void* o, const void* dout,
                      const float* lse, void* dq, void* dk, void* dv, const BwdWorkspace& ws, hipStream_t stream,
                      int parts) {
    AttnArgs aq = a;
    aq.row_stats = (parts & BWD_PRE) && (parts & BWD_DQ);  // the dQ grid covers every row
    const int64_t rows = (int64_t)a.batch * a.heads * a.n;
    if ((parts & BWD_PRE) && !aq.row_stats)
        hipLaunchKernelGGL((bwd_pre_kernel<D>), dim3((unsigned)((rows + kPreRows - 1) / kPreRows)), dim3(256),
                           0, stream, a, (const uint16_t*)o, (const uint16_t*)dout, lse, ws.ndelta, ws.nlse2,
                           (unsigned long long*)nullptr, (int32_t*)nullptr, (int32_t*)nullptr);
    if (parts & BWD_DQ)
        hipLaunchKernelGGL((strided_dq_kernel<D, 8>), dim3((unsigned)strided_groups(a)), dim3(512), 0, stream, aq,
                           (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)dout,
                           (const uint16_t*)o, lse, ws.nlse2, ws.ndelta, (uint16_t*)dq);
    constexpr int W = D == 128 ? 8 : 16;
    if (parts & BWD_DKDV)
        hipLaunchKernelGGL((strided_dkdv_kernel<D, W>), dim3((unsigned)strided_groups(a)), dim3(64 * W), 0, stream, a,
                           (const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)dout, ws.nlse2,
                           ws.ndelta, (uint16_t*)dk, (uint16_t*)dv);
    return hipGetLastError();
}

}  // namespace

hipError_t strided_fwd(const AttnArgs& a, const void* q, const void* k, const void* v, void* o, float* lse,
                       hipStream_t stream) {
    switch (a.d) {
    case 32: return launch_fwd<32>(a, q, k, v, o, lse, stream);
    case 64: return launch_fwd<64>(a, q, k, v, o, lse, stream);
    default: return launch_fwd<128>(a, q, k, v, o, lse, stream);
    }
}

hipError_t strided_bwd(const AttnArgs& a, const void* q, const void* k, const void* v, const void* o, const void* dout,
                       const float* lse, void* dq, void* dk, void* dv, void* workspace, hipStream_t stream, int parts) {
    const BwdWorkspace ws = bwd_workspace(workspace, a.ws_rows, 1);
    switch (a.d) {
    case 32: return launch_bwd<32>(a, q, k, v, o, dout, lse, dq, dk, dv, ws, stream, parts);
    case 64: return launch_bwd<64>(a, q, k, v, o, dout, lse, dq, dk, dv, ws, stream, parts);
    default: return launch_bwd<128>(a, q, k, v, o, dout, lse, dq, dk, dv, ws, stream, parts);
    }
}

}  // namespace sa
