// Infinities and NaN in the bf16 residue-class and one-pass kernels.
//
// A pair that is not attended enters the products with weight 0, but 0 x infinity and
// 0 x NaN are NaN, and the neighbours of an attended row in a chunk of a class are l
// positions apart: an infinite or NaN element would reach rows up to 63 l positions
// away.  The kernels take no notice on their way (a test per chunk would cost
// registers); sums that come out non-finite are formed a second time with every row's
// product kept by the rows that attend it alone, so that such an element reaches what
// attends it and nothing else.  The one-pass kernels run a second time; a wave of the
// class kernels forms its 16 rows or keys again by itself, straight from global
// memory.  The test of the sums costs (n = 12,288, 16 heads of 64, backward, us): l =
// 128 131.4 -> 133.7, l = 111 152.5 -> 154.2, A2 alone 62.6 -> 64.1.
#pragma once

#include "sa_internal.h"
#include "sa_mfma.h"

namespace sa {

// x, as a value the compiler knows nothing about: what a second run computes from it
// stays inside it and holds no registers in the first.
__device__ inline int opaque(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Whether an element of this lane's sums is an infinity or a NaN (by its bits: the
// build lets comparisons assume that there is none).
template <int N>
__device__ inline bool non_finite(const f32x4* acc) {
    uint32_t top = 0;
#pragma unroll
    for (int x = 0; x < N; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            const uint32_t v = __float_as_uint(acc[x][y]) & 0x7FFFFFFFu;
            top = v > top ? v : top;
        }
    return top >= 0x7F800000u;
}

// acc += the products of chunk rows 0 .. 31 (operands a, b, see pack_bf16x8) with this
// lane's row, which attends the rows lo .. hi of the chunk.
template <int DB>
__device__ inline void accumulate_attended(const bf16x8* a, bf16x8 b, int lo, int hi, int g, f32x4* acc) {
    const u32x4 bw = __builtin_bit_cast(u32x4, b);
#pragma unroll 1
    for (int x = 0; x < 32; ++x) {  // one row at a time
        const int e = (x >> 4) * 4 + (x & 3);
        u32x4 keep;
#pragma unroll
        for (int y = 0; y < 4; ++y)
            keep[y] = g == ((x >> 2) & 3) && y == (e >> 1) ? ((e & 1) ? 0xFFFF0000u : 0xFFFFu) : 0u;
        const bf16x8 bx = __builtin_bit_cast(bf16x8, bw & keep);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const bf16x8 ax = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, a[db]) & keep);
            const f32x4 sum = mfma_16x16x32(ax, bx, acc[db]);
            if (x >= lo && x <= hi) acc[db] = sum;
            __builtin_amdgcn_sched_barrier(0);  // one sum in flight: registers
        }
    }
}

// Rows of one class in global memory: row m at p + m ss, rows past the last read as it.
struct ClassRows {
    int64_t ss;
    int last, g, r;

    // x . y over d: rows a + 16 kb + 4 g + t of x against row b + r of y, in s[kb][t].
    template <int D>
    __device__ void dot(const uint16_t* x, int a, const uint16_t* y, int b, f32x4* s) const {
        const uint16_t* py = y + (int64_t)min(b + r, last) * ss + 8 * g;
        for (int kb = 0; kb < 2; ++kb) {
            const uint16_t* px = x + (int64_t)min(a + 16 * kb + r, last) * ss + 8 * g;
#pragma unroll 1
            for (int ks = 0; ks < D / 32; ++ks)
                s[kb] = mfma_16x16x32(ld_bf16x8(px + 32 * ks), ld_bf16x8(py + 32 * ks), s[kb]);
        }
    }
    // The transposed operand of rows a .. a + 31: column col of rows a + 4 g + t and a + 16 + 4 g + t.
    __device__ bf16x8 column(const uint16_t* x, int a, int col) const {
        u32x4 w = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int row = min(a + 16 * (e / 4) + 4 * g + e % 4, last);
            w[e / 2] |= (uint32_t)x[(int64_t)row * ss + col] << (16 * (e & 1));
        }
        return __builtin_bit_cast(bf16x8, w);
    }
    // acc[col] += x^T b over the attended rows lo .. hi of the chunk at a, columns 16 db + r.
    __device__ void add(const uint16_t* x, int a, int db, bf16x8 b, int lo, int hi, f32x4* acc) const {
        const bf16x8 xt = column(x, a, 16 * db + r);
        accumulate_attended<1>(&xt, b, lo, hi, g, acc);
    }
    // Four results at row, columns 16 db + 4 g + t (added to what is there with `add`).
    __device__ void store(uint16_t* out, int row, int db, f32x4 x, bool add) const {
        if (row > last) return;
        uint2* dst = reinterpret_cast<uint2*>(out + (int64_t)row * ss + 16 * db + 4 * g);
        if (add) x += bf16x4_to_f32x4(*dst);
        *dst = pack_bf16x4_bits(x);
    }
};

__device__ inline ClassRows class_rows(const AttnArgs& a, int rows) {
    const int lane = opaque((int)threadIdx.x % 64);
    return {a.ss, rows - 1, lane / 16, lane % 16};
}

// The functions below form the results of one wave's 16 rows (keys) and write them;
// 16 columns at a time and everything else anew for each, so that they need few
// registers.  Tensors and LSE start at the class's first row.

// Forward, queries row0 + r, which attend the class's keys up to row0 + r - a.qshift.
template <int D>
__device__ inline void class_forward_again(const AttnArgs& a, int rows, int row0, const uint16_t* q, const uint16_t* k,
                                           const uint16_t* v, uint16_t* o, float* lse) {
    const ClassRows c = class_rows(a, rows);
    const int i = row0 + c.r, hi = min(i - a.qshift, c.last), end = min(row0 + 15 - a.qshift, c.last);
    float m = -INFINITY, l = 0.f, m_ref = 0.f;
    f32x4 p[2];
    auto scores = [&](int j0) {  // key j0 + 16 kb + 4 g + t
        p[0] = p[1] = zero4();
        c.dot<D>(k, j0, q, row0, p);
#pragma unroll
        for (int x = 0; x < 8; ++x)
            p[x / 4][x % 4] = j0 + 16 * (x / 4) + 4 * c.g + x % 4 <= hi ? p[x / 4][x % 4] : -INFINITY;
    };
    auto weights = [&] {
        float sum = 0.f;
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            p[x / 4][x % 4] = exp2_fast(fmaf(p[x / 4][x % 4], a.scale_log2, -m_ref * a.scale_log2));
            sum += p[x / 4][x % 4];
        }
        return sum;
    };
#pragma unroll 1
    for (int j0 = 0; j0 <= end; j0 += 32) {
        scores(j0);
        float top = -INFINITY;
#pragma unroll
        for (int x = 0; x < 8; ++x) top = fmaxf(top, p[x / 4][x % 4]);
        const float m_new = fmaxf(m, max_over_g(top));
        m_ref = m_new == -INFINITY ? 0.f : m_new;
        l = fmaf(l, exp2_fast((m - m_ref) * a.scale_log2), weights());
        m = m_new;
    }
    l = sum_over_g(l);
    // with EPI_MERGE, O and LSE of a disjoint part of the row's set are in the outputs
    const bool merge = a.epilogue == EPI_MERGE;
    float* lrow = lse + (int64_t)min(i, c.last) * a.lse_ss;
    const float lse1 = merge ? *lrow : -INFINITY, lse2 = l > 0.f ? m * a.scale + __logf(l) : -INFINITY;
    const float top = fmaxf(lse1, lse2);
    const float w1 = lse1 == -INFINITY ? 0.f : __expf(lse1 - top);
    const float w2 = l > 0.f ? __expf(m * a.scale - top) : 0.f;
    const float z = w1 + w2 * l, inv = z > 0.f ? 1.f / z : 0.f;
#pragma unroll 1
    for (int db = 0; db < D / 16; ++db) {
        f32x4 acc = zero4();
#pragma unroll 1
        for (int j0 = 0; j0 <= end; j0 += 32) {
            scores(j0);
            weights();
            c.add(v, j0, db, pack_bf16x8(p[0], p[1]), 0, hi - j0, &acc);
        }
        if (merge && i <= c.last)
            acc = acc * w2 + bf16x4_to_f32x4(*reinterpret_cast<const uint2*>(o + (int64_t)i * a.ss + 16 * db + 4 * c.g)) * w1;
        else
            acc *= w2;
        c.store(o, i, db, acc * inv, false);
    }
    if (c.g == 0 && i <= c.last) *lrow = z > 0.f ? top + __logf(z) : -INFINITY;
}

// dQ of the queries row0 + r (nl2, nd: -LSE log2 e and -D of this lane's).
template <int D>
__device__ inline void class_dq_again(const AttnArgs& a, int rows, int row0, const uint16_t* q, const uint16_t* k,
                                      const uint16_t* v, const uint16_t* dout, float nl2, float nd, uint16_t* dq) {
    const ClassRows c = class_rows(a, rows);
    const int hi = min(row0 + c.r - a.qshift, c.last);
#pragma unroll 1
    for (int db = 0; db < D / 16; ++db) {
        f32x4 acc = zero4();
#pragma unroll 1
        for (int j0 = 0; j0 <= min(row0 + 15 - a.qshift, c.last); j0 += 32) {
            f32x4 s[2] = {zero4(), zero4()}, dp[2] = {f32x4{nd, nd, nd, nd}, f32x4{nd, nd, nd, nd}};
            c.dot<D>(k, j0, q, row0, s);
            c.dot<D>(v, j0, dout, row0, dp);
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const bool on = j0 + 16 * (x / 4) + 4 * c.g + x % 4 <= hi;
                s[x / 4][x % 4] = on ? exp2_fast(fmaf(s[x / 4][x % 4], a.scale_log2, nl2)) * dp[x / 4][x % 4] : 0.f;
            }
            c.add(k, j0, db, pack_bf16x8(s[0], s[1]), 0, hi - j0, &acc);
        }
        c.store(dq, row0 + c.r, db, acc * a.scale, a.epilogue == EPI_ADD);
    }
}

// dV and dK of the keys key0 + r, attended by the queries from key0 + r + a.qshift on.
template <int D>
__device__ inline void class_dkdv_again(const AttnArgs& a, int rows, int key0, const uint16_t* q, const uint16_t* k,
                                        const uint16_t* v, const uint16_t* dout, const float* nlse2,
                                        const float* ndelta, uint16_t* dk, uint16_t* dv) {
    const ClassRows c = class_rows(a, rows);
    const int lo = key0 + c.r + a.qshift;
#pragma unroll 1
    for (int part = 0; part < D / 8; ++part) {  // dV's columns, then dK's
        const bool is_dv = part < D / 16;
        const int db = part % (D / 16);
        f32x4 acc = zero4();
#pragma unroll 1
        for (int i0 = key0 + a.qshift; i0 <= c.last; i0 += 32) {
            f32x4 p[2] = {zero4(), zero4()}, ds[2];  // query i0 + 16 kb + 4 g + t, key key0 + r
            c.dot<D>(q, i0, k, key0, p);
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const int i = i0 + 16 * (x / 4) + 4 * c.g + x % 4;
                const int64_t at = (int64_t)min(i, c.last) * a.lse_ss;
                ds[x / 4][x % 4] = ndelta[at];
                p[x / 4][x % 4] = i >= lo && i <= c.last ? exp2_fast(fmaf(p[x / 4][x % 4], a.scale_log2, nlse2[at])) : 0.f;
            }
            if (!is_dv) {
                c.dot<D>(dout, i0, v, key0, ds);
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    const int i = i0 + 16 * (x / 4) + 4 * c.g + x % 4;
                    p[x / 4][x % 4] = i >= lo && i <= c.last ? p[x / 4][x % 4] * ds[x / 4][x % 4] : 0.f;
                }
            }
            c.add(is_dv ? dout : q, i0, db, pack_bf16x8(p[0], p[1]), lo - i0, c.last - i0, &acc);
        }
        c.store(is_dv ? dv : dk, key0 + c.r, db, is_dv ? acc : acc * a.scale, a.epilogue == EPI_ADD);
    }
}

}  // namespace sa
