// C ABI (include/sparse_attn.h): argument validation, launch configuration and
// status codes.  Nothing is enqueued unless every argument is valid.
#include <math.h>

#include <mutex>

#include "sparse_attn.h"
#include "sa_internal.h"
#include "sa_mask.h"
#include "sa_strided.h"

namespace {

using sa::Pattern;

// Summary subblocks per l-block that heads can be spread over; beyond this the
// per-subblock layouts would outgrow any useful head count.
constexpr int kMaxSubblocks = 64;

struct PatternArgs {
    int64_t n;
    int32_t block, l, c;
    int32_t pattern;  // STRIDED or FIXED (SA_FIXED_PER_HEAD is FIXED with sub > 0)
    int32_t mode;
    int32_t sub;      // summary subblocks, 0 = one window for all heads
    int64_t nq;
    int n_layouts;
};

// Pattern, stride and summary width (shared by the block and decoding entry
// points): internal pattern and subblock count.
int check_pattern_code(int32_t l, int32_t c, int32_t pattern, int32_t mode, int32_t* internal, int32_t* sub) {
    if (l < 1) return SA_ERR_INVALID;
    if (pattern != SA_STRIDED && pattern != SA_FIXED && pattern != SA_FIXED_PER_HEAD) return SA_ERR_INVALID;
    if (mode < SA_MODE_A1 || mode > SA_MODE_INTERLEAVED) return SA_ERR_INVALID;
    if (pattern != SA_STRIDED && (c < 1 || c > l)) return SA_ERR_INVALID;
    if (pattern == SA_STRIDED && c != 0) return SA_ERR_INVALID;
    *internal = pattern == SA_STRIDED ? sa::STRIDED : sa::FIXED;
    *sub = 0;
    if (pattern == SA_FIXED_PER_HEAD) {
        if (l / c > kMaxSubblocks) return SA_ERR_UNSUPPORTED;
        *sub = l / c;
    }
    return SA_OK;
}

int check_pattern(int64_t n, int32_t block, int32_t l, int32_t c, int32_t pattern, int32_t mode,
                  PatternArgs* out) {
    if (block != 16 && block != 32 && block != 64) return SA_ERR_INVALID;
    if (n < 1 || n > INT32_MAX || n % block != 0) return SA_ERR_INVALID;
    int32_t internal = 0, sub = 0;
    const int st = check_pattern_code(l, c, pattern, mode, &internal, &sub);
    if (st != SA_OK) return st;
    out->n = n;
    out->block = block;
    out->l = l;
    out->c = c;
    out->pattern = internal;
    out->mode = mode;
    out->sub = sub;
    out->nq = n / block;
    out->n_layouts = sa::layout_count(mode, sub);
    return SA_OK;
}

Pattern pattern_of_layout(const PatternArgs& p, int g) {
    Pattern s;
    s.pattern = p.pattern;
    s.part = sa::part_of_layout(p.mode, g);
    s.l = p.l;
    s.c = p.c;
    s.w = sa::summary_start(p.l, p.c, sa::subblock_of_layout(p.mode, p.sub, g));
    return s;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_tensor_args(const PatternArgs& p, int32_t batch, int32_t heads, int32_t d, int32_t dtype,
                      const int64_t* strides) {
    if (batch < 1 || heads < 1) return SA_ERR_INVALID;
    if (dtype != SA_F32 && dtype != SA_BF16) return SA_ERR_INVALID;
    if (d != 32 && d != 64 && d != 128) return SA_ERR_UNSUPPORTED;
    if (!strides) return SA_ERR_INVALID;
    const int64_t unit = dtype == SA_BF16 ? 8 : 4;  // elements per 16 bytes
    for (int t = 0; t < 3; ++t)
        if (strides[t] < 0 || strides[t] % unit != 0) return SA_ERR_INVALID;
    if (strides[2] < d) return SA_ERR_INVALID;
    if ((int64_t)batch * heads > INT32_MAX / 2) return SA_ERR_INVALID;
    // the bf16 kernels stage a B x d tile with 32-bit byte offsets from its first row
    if (dtype == SA_BF16 && strides[2] * 2 * p.block >= ((int64_t)1 << 32)) return SA_ERR_UNSUPPORTED;
    return SA_OK;
}

sa::AttnArgs make_args(const PatternArgs& p, int32_t batch, int32_t heads, int32_t d,
                       const int64_t* strides, float scale, const int32_t* row_ptr,
                       const int32_t* col_idx, const int32_t* col_ptr, const int32_t* row_idx) {
    sa::AttnArgs a;
    a.pattern = p.pattern;
    a.mode = p.mode;
    a.l = p.l;
    a.c = p.c;
    a.n = (int32_t)p.n;
    a.nq = (int32_t)p.nq;
    a.block = p.block;
    a.batch = batch;
    a.heads = heads;
    a.d = d;
    a.sb = strides[0];
    a.sh = strides[1];
    a.ss = strides[2];
    a.scale = scale;
    a.scale_log2 = scale * sa::kLog2eHost;
    a.period_bits = sa::host_period_bits(p.l);
    sa::summary_words(p.l, p.c, p.l - p.c, &a.sum_lo, &a.sum_hi);
    a.sub = p.sub;
    a.claim_mode = sa::CLAIM_QUEUES;
    a.pairs = 0;
    a.row_stats = 0;
    a.sched_first = 0;
    a.dl = sa::make_divl(p.l);
    a.walk = sa::WALK_LAYOUT;
    a.qshift = 0;
    a.epilogue = sa::EPI_STORE;
    a.lse_sb = (int64_t)heads * p.n;  // LSE and row statistics: [batch, heads, n]
    a.lse_sh = p.n;
    a.lse_ss = 1;
    a.off = a.lse_off = 0;
    a.ws_rows = (int64_t)batch * heads * p.n;
    a.seq = 0;
    a.row_ptr = row_ptr;
    a.col_idx = col_idx;
    a.col_ptr = col_ptr;
    a.row_idx = row_idx;
    return a;
}

// Strided A2 by residue classes (Sec. 5.5, a stride becomes a local window once
// positions are reordered by their residue mod l).  Position i = m l + r (class
// r, step m) meets j = m' l + r of its own class only, and A2 \ A1 of the merged
// set is {m' <= m - 2}: dense causal attention inside each class, with the
// queries' causal limit moved back by `shift` = 2 steps (A2 alone: by none).
// The classes are strided views of the [b, h, n, d] tensors, so the block
// kernels walk them unchanged: batch = the (b, h) units, heads = the l classes
// (stride of one row), sequence stride l rows, every block kb <= qb present (no
// layout), LSE and row statistics in row order.  Where class blocks of cb do
// not divide every class the sequence length goes along (AttnArgs::seq), and the
// kernels pad the last block of each class.
int class_view(int64_t n, int32_t l, int32_t cb, int32_t shift, int64_t units, int64_t unit_stride, int64_t ss,
               int32_t d, int32_t dtype, float scale, sa::AttnArgs* cls) {
    if (cb != 16 && cb != 32 && cb != 64) return SA_ERR_INVALID;
    const int64_t M = ((n + l - 1) / l + cb - 1) / cb * cb;  // positions per class, padded
    if (M / cb > 65535 || units > 65535) return SA_ERR_UNSUPPORTED;  // grid dimensions
    const int64_t cls_strides[3] = {unit_stride, ss, (int64_t)l * ss};
    PatternArgs c;
    int st = check_pattern(M, cb, (int32_t)M, 0, SA_STRIDED, SA_MODE_A1, &c);
    if (st != SA_OK) return st;
    st = check_tensor_args(c, (int32_t)units, l, d, dtype, cls_strides);
    if (st != SA_OK) return st;
    *cls = make_args(c, (int32_t)units, l, d, cls_strides, scale, nullptr, nullptr, nullptr, nullptr);
    cls->walk = sa::WALK_DENSE;
    cls->qshift = shift;
    cls->seq = M * l == n ? 0 : (int32_t)n;
    cls->lse_sb = n;  // row i = m l + r of unit u sits at u n + r + m l
    cls->lse_sh = 1;
    cls->lse_ss = l;
    cls->ws_rows = units * n;
    return SA_OK;
}

// The class view of a call with the caller's class block (which must divide the
// classes).
int class_args(int64_t n, int32_t l, int32_t cb, int32_t mode, int32_t batch, int32_t heads, int32_t d,
               int32_t dtype, const int64_t* strides, float scale, sa::AttnArgs* cls) {
    if (n % l != 0) return SA_ERR_INVALID;
    if (cb != 16 && cb != 32 && cb != 64) return SA_ERR_INVALID;
    if ((n / l) % cb != 0) return SA_ERR_INVALID;
    if (batch > 1 && strides[0] != (int64_t)heads * strides[1]) return SA_ERR_UNSUPPORTED;  // (b, h) as one index
    return class_view(n, l, cb, mode == SA_MODE_MERGED ? 2 : 0, (int64_t)batch * heads, strides[1], strides[2], d,
                      dtype, scale, cls);
}

// How a bf16 strided call runs without its layout: the band A1 of the heads that
// attend it, and the residue classes of the heads that attend A2 (merged heads:
// the rest of A2, combined with the band's results; alternating heads: the band
// for the even heads, the classes for the odd ones); or merged heads in one pass.
struct StridedPlan {
    bool fused;            // merged heads in one pass (sa_strided.hip; arguments: rows)
    bool band, classes;
    bool merge;            // the classes' results join the band's
    sa::AttnArgs b, c;
    sa::AttnArgs rows;     // row view of the class heads
};

// Returns false where the block path over the layout stays: fp32; (batch, head)
// strides that do not make one index; grids out of range; and the sizes below.
//
// Precision first.  With l a multiple of B the block path takes the blocks away from
// the band, single diagonals, with fp32 probabilities and score gradients; the class
// and one-pass kernels round both to bf16 (A2 alone, n = 2,560, l = 64: error of dV
// 1.36 times the rounding of the result against 1.12, of dQ 1.61 against 1.32).  So
// with B | l only classes that fill blocks of 16 or more, merged or A2 alone, go by
// classes (n = 12,288, l = 128, 16 heads merged, backward: 135 us).  With any other l
// the block path rounds them as well.
//
// Merged heads, B | l and filled classes: band and class launches, which meet in
// bf16, or one pass.  One pass is used for the forward up to l = 128 (n = 12,288, 16
// heads, l = 128: 49 against 56 us; l = 512: 81 against 70; n = 65,536, 8 heads, l =
// 256: 190 against 160: its waves read the band's keys for 16 rows each, the band
// kernel for 64; between 128 and 256 nothing was measured), for classes of up to 256
// (l = 128, 4 heads, M = 512: 111 against 94) and from 192 workgroups (d = 128: 32 24
// against 13, 128 23.5 against 22.6, 192 30 against 35; d = 64: 32 14 against 10, 256
// 18 against 24), and never for the backward (137 against 135, l = 256 155 against
// 139).
//
// Merged heads otherwise: one pass or the block path, which steps through every block
// that holds a pair: per multiple of l two blocks of a row, or every block when l < B.
// One pass wins where those outnumber the band's blocks by kFarToBand (forward +
// backward, 16 heads of 64, 2.4 times: n = 12,288, l = 111 1,379 -> 203 us; 1.5 to 2: n
// = 1,024, l = 100 66 -> 47; 1.1: n = 4,096, l = 400 103 -> 113; 0.45: l = 600 107 ->
// 161; 8 heads, 3.6: n = 65,536, l = 1,000 2,719 -> 1,405), and where a row has enough
// of them: a short sequence's one pass is bound by the latency of its phases, whatever
// n (d = 64 about 40 us, d = 128 82), and the block path by its steps, the cheaper the
// smaller B (d = 128, 4 to 16 heads, block path | one pass: B = 64, 3.3 steps a row 55
// | 83, 5.3 74 | 82, 6.3 90 | 83; B = 32, 9 51 | 63; B = 16, 15 92 | 83; d = 64: B = 64,
// 3.3 38 | 40; B = 32, 3.5 31 | 37).
//
// A2 alone, l no multiple of B, goes by classes from kMinFarBlocks block steps a row on
// average (block path | classes, forward + backward, d = 64: n = 8,192, l = 1,000, 8.2
// steps 72 | 34 us; n = 1,024, l = 24, 6 steps 67 | 12), alternating heads, two
// launches more, from kMinFarAlternate (l = 1,000 116 | 90; n = 768, l = 50, 6.1 steps 55
// | 27: the line is on the safe side).
constexpr double kFarToBand = 1.3, kMinFarBlocks = 4.0, kMinFarAlternate = 8.0;
constexpr int32_t kFusedMinStride = 8, kFusedAlignedMaxStride = 128, kFusedAlignedMaxClass = 256;
constexpr int64_t kFusedAlignedMinTiles = 192;

bool strided_plan(const PatternArgs& p, int32_t batch, int32_t heads, int32_t d, int32_t dtype,
                  const int64_t* strides, float scale, bool backward, StridedPlan* s) {
    if (p.pattern != sa::STRIDED || dtype != SA_BF16) return false;
    const bool alternate = p.mode == SA_MODE_INTERLEAVED;
    const int64_t M = (p.n + p.l - 1) / p.l;  // positions of the longest class
    s->fused = false;
    s->merge = p.mode == SA_MODE_MERGED;
    s->band = p.mode != SA_MODE_A2;
    const int32_t class_heads = alternate ? heads / 2 : (p.mode == SA_MODE_A1 ? 0 : heads);
    s->classes = class_heads > 0 && !(s->merge && M <= 2);
    PatternArgs pb = p;
    pb.mode = SA_MODE_A1;
    pb.n_layouts = 1;
    // every second head (alternate), from the first or the second
    auto subset = [&](int32_t count, int32_t first) {
        const int64_t step = alternate ? 2 : 1;
        const int64_t st[3] = {strides[0], step * strides[1], strides[2]};
        sa::AttnArgs a = make_args(pb, batch, count, d, st, scale, nullptr, nullptr, nullptr, nullptr);
        a.walk = sa::WALK_BAND;
        a.lse_sb = (int64_t)heads * p.n;
        a.lse_sh = step * p.n;
        a.off = first * strides[1];
        a.lse_off = first * p.n;
        a.ws_rows = (int64_t)batch * heads * p.n;
        return a;
    };
    if (s->band) s->b = subset(alternate ? (heads + 1) / 2 : heads, 0);
    if (!s->classes) return true;
    const int32_t first = alternate ? 1 : 0;
    s->rows = subset(class_heads, first);
    // classes that fill blocks of 16 or more
    const bool filled = p.n % p.l == 0 && M % 16 == 0;
    if (p.l % p.block == 0 && (alternate || !filled)) return false;  // fp32 diagonals
    const double steps = p.l >= p.block ? 2.0 : (double)p.l / p.block;  // the block path's, per multiple of l
    if (s->merge) {
        const bool aligned = filled && p.l % p.block == 0;
        const double far = 0.5 * (double)(M - 2) * steps;
        const bool better = aligned ? !backward && p.l <= kFusedAlignedMaxStride && M <= kFusedAlignedMaxClass &&
                                              sa::strided_tiles(s->rows) >= kFusedAlignedMinTiles
                                    : far >= kFarToBand * (sa::band_blocks(s->rows) + 1) &&
                                          far >= (d == 128 ? 6.0 : 4.0) * (p.block == 64 ? 1.0 : p.block == 32 ? 1.6 : 2.5);
        s->fused = better && p.l >= kFusedMinStride && 64 * (int64_t)p.l * strides[2] < ((int64_t)1 << 32) &&
                   sa::strided_grid_fits(s->rows);
        if (s->fused) return true;
        if (!aligned) return false;
    } else if (p.l % p.block != 0 && 0.5 * (double)M * steps < (alternate ? kMinFarAlternate : kMinFarBlocks)) {
        return false;
    }
    if (batch > 1 && (strides[0] != (int64_t)heads * strides[1] || (alternate && heads % 2 != 0))) return false;
    const int32_t cb = M >= 256 ? 64 : (M > 16 ? 32 : 16);
    if (class_view(p.n, p.l, cb, s->merge ? 2 : 0, (int64_t)batch * class_heads, s->rows.sh, strides[2], d, dtype,
                   scale, &s->c) != SA_OK)
        return false;
    s->c.lse_sb = s->rows.lse_sh;
    s->c.off = s->rows.off;
    s->c.lse_off = s->rows.lse_off;
    s->c.ws_rows = s->rows.ws_rows;
    return true;
}

// Pattern arguments of a decoding step (no block size: S_pos is enumerated).
int check_decode_pattern(int64_t pos, int32_t l, int32_t c, int32_t pattern, int32_t mode, int32_t* internal,
                         int32_t* sub) {
    if (pos < 0 || pos > INT32_MAX) return SA_ERR_INVALID;
    return check_pattern_code(l, c, pattern, mode, internal, sub);
}
int check_decode_shape(int32_t batch, int32_t heads, int32_t d, int32_t dtype) {
    if (batch < 1 || heads < 1 || (int64_t)batch * heads > INT32_MAX / 2) return SA_ERR_INVALID;
    if (dtype != SA_F32 && dtype != SA_BF16) return SA_ERR_INVALID;
    if (d != 32 && d != 64 && d != 128) return SA_ERR_UNSUPPORTED;
    return SA_OK;
}

// Merged strided heads by transposition through the explicit entry points:
// the band over the caller's strided A1 layout, the classes in blocks of
// class_block (see class_args); tensors contiguous.
struct TransposedPlan {
    PatternArgs band;
    int64_t strides[3];
    sa::AttnArgs cls;
    size_t workspace;  // bytes: the band backward's workspace
};

int plan_transposed(int64_t n, int32_t block, int32_t l, int32_t class_block, int32_t batch, int32_t heads, int32_t d,
                    int32_t dtype, float scale, TransposedPlan* p) {
    int st = check_pattern(n, block, l, 0, SA_STRIDED, SA_MODE_A1, &p->band);
    if (st != SA_OK) return st;
    if (batch < 1 || heads < 1) return SA_ERR_INVALID;
    p->strides[0] = (int64_t)heads * n * d;
    p->strides[1] = n * d;
    p->strides[2] = d;
    st = check_tensor_args(p->band, batch, heads, d, dtype, p->strides);
    if (st != SA_OK) return st;
    st = class_args(n, l, class_block, SA_MODE_MERGED, batch, heads, d, dtype, p->strides, scale, &p->cls);
    if (st != SA_OK) return st;
    p->workspace = sa::bwd_workspace_bytes(batch, heads, n, p->band.nq, 1);
    return SA_OK;
}

// Arguments of a backward call, shared by sparse_attn_bwd and
// sparse_attn_bwd_noalloc: everything but the workspace.  Fills the kernel
// arguments and the workspace size the call needs.
int check_bwd(int64_t n, int32_t block, int32_t stride_l, int32_t summary_c, int32_t pattern, int32_t head_mode,
              const int32_t* row_ptr, const int32_t* col_idx, const uint8_t* kind, const int32_t* col_ptr,
              const int32_t* row_idx, const uint8_t* kind_t, int32_t batch, int32_t heads, int32_t d_head,
              int32_t dtype, const void* q, const void* k, const void* v, const void* o, const void* dout,
              const float* lse, const int64_t* strides, float softmax_scale, void* dq, void* dk, void* dv,
              sa::AttnArgs* a, size_t* need, bool* planned, StridedPlan* plan) {
    PatternArgs p;
    int st = check_pattern(n, block, stride_l, summary_c, pattern, head_mode, &p);
    if (st != SA_OK) return st;
    st = check_tensor_args(p, batch, heads, d_head, dtype, strides);
    if (st != SA_OK) return st;
    if (!row_ptr || !col_idx || !kind || !col_ptr || !row_idx || !kind_t) return SA_ERR_INVALID;
    if (!q || !k || !v || !o || !dout || !lse || !dq || !dk || !dv) return SA_ERR_INVALID;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(dout) ||
        !aligned16(dq) || !aligned16(dk) || !aligned16(dv))
        return SA_ERR_INVALID;
    if (!isfinite(softmax_scale) || !(softmax_scale > 0.f)) return SA_ERR_INVALID;
    *need = sa::bwd_workspace_bytes(batch, heads, n, p.nq, p.n_layouts);
    *a = make_args(p, batch, heads, d_head, strides, softmax_scale, row_ptr, col_idx, col_ptr, row_idx);
    *planned = strided_plan(p, batch, heads, d_head, dtype, strides, softmax_scale, true, plan);
    return SA_OK;
}

// The launches of a validated backward call.  By a strided plan: the band's
// stages first (its row statistics go with its dQ), the row statistics of heads
// without a band, then the classes' dQ and dK / dV, last and together (short
// classes run them as one launch).
// `parts`: the stages to launch (sa::BWD_*), in their order.
hipError_t launch_bwd(const sa::AttnArgs& a, bool planned, StridedPlan& plan, int dtype, const void* q, const void* k,
                      const void* v, const void* o, const void* dout, const float* lse, void* dq, void* dk, void* dv,
                      void* ws, hipStream_t s, int parts = sa::BWD_ALL) {
    if (!planned) return sa::bwd_launch(a, dtype, q, k, v, o, dout, lse, dq, dk, dv, ws, s, parts);
    if (plan.fused) return sa::strided_bwd(plan.rows, q, k, v, o, dout, lse, dq, dk, dv, ws, s, parts);
    hipError_t e = hipSuccess;
    if (plan.band) e = sa::bwd_launch(plan.b, dtype, q, k, v, o, dout, lse, dq, dk, dv, ws, s, parts);
    if (!plan.classes) return e;
    if (e == hipSuccess && !plan.merge && (parts & sa::BWD_PRE))
        e = sa::bwd_launch(plan.rows, dtype, q, k, v, o, dout, lse, dq, dk, dv, ws, s, sa::BWD_PRE);
    const int classes = parts & (sa::BWD_DQ | sa::BWD_DKDV);
    if (plan.merge) plan.c.epilogue = sa::EPI_ADD;
    if (e == hipSuccess && classes)
        e = sa::bwd_launch(plan.c, dtype, q, k, v, o, dout, lse, dq, dk, dv, ws, s, classes);
    return e;
}

}  // namespace

// ---------------------------------------------------------------------------
// Scratch of sparse_attn_bwd_noalloc: a fixed device array in place of the
// caller's workspace, one copy per device, held until the process ends.  In
// host code `scratch` names a host-side stand-in, not device memory, so its
// device address is looked up once per device (with that device current)
// and only that address is ever passed on.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices];  // device address of `scratch` per device, guarded by g_scratch_mutex

// Device address of the scratch array on the device of `stream`, which must
// be the current device.
int scratch_address(hipStream_t stream, void** out) {
    int dev = -1, stream_dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return SA_ERR_HIP;
    if (hipStreamGetDevice(stream, &stream_dev) != hipSuccess) return SA_ERR_HIP;
    if (stream_dev != dev) return SA_ERR_INVALID;
    if (dev < 0 || dev >= kMaxDevices) return SA_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return SA_ERR_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return SA_OK;
}

}  // namespace

extern "C" {

int sparse_attn_layout_size(int64_t n, int32_t block, int32_t stride_l, int32_t summary_c,
                            int32_t pattern, int32_t head_mode, int32_t* n_layouts,
                            int64_t* nnz) {
    PatternArgs p;
    int st = check_pattern(n, block, stride_l, summary_c, pattern, head_mode, &p);
    if (st != SA_OK) return st;
    if (!n_layouts || !nnz) return SA_ERR_INVALID;
    int64_t counts[1 + kMaxSubblocks] = {0};
    int64_t total = 0;
    for (int g = 0; g < p.n_layouts; ++g) {
        counts[g] = sa::layout_count_host(pattern_of_layout(p, g), n, block);
        total += counts[g];
    }
    if (total > INT32_MAX) return SA_ERR_UNSUPPORTED;  // int32 layout indices
    *n_layouts = p.n_layouts;
    const int entries = p.n_layouts > 2 ? p.n_layouts : 2;
    for (int g = 0; g < entries; ++g) nnz[g] = counts[g];
    return SA_OK;
}

int sparse_attn_layout_count(int32_t stride_l, int32_t summary_c, int32_t pattern, int32_t head_mode,
                             int32_t* n_layouts) {
    int32_t internal = 0, sub = 0;
    const int st = check_pattern_code(stride_l, summary_c, pattern, head_mode, &internal, &sub);
    if (st != SA_OK) return st;
    if (!n_layouts) return SA_ERR_INVALID;
    *n_layouts = sa::layout_count(head_mode, sub);
    return SA_OK;
}

int sparse_attn_layout(int64_t n, int32_t block, int32_t stride_l, int32_t summary_c,
                       int32_t pattern, int32_t head_mode, int32_t* row_ptr, int32_t* col_idx,
                       uint8_t* kind, int32_t* col_ptr, int32_t* row_idx, uint8_t* kind_t,
                       int64_t capacity, void* stream) {
    PatternArgs p;
    int st = check_pattern(n, block, stride_l, summary_c, pattern, head_mode, &p);
    if (st != SA_OK) return st;
    if (!row_ptr || !col_idx || !kind || !col_ptr || !row_idx || !kind_t) return SA_ERR_INVALID;
    int64_t total = 0;
    for (int g = 0; g < p.n_layouts; ++g) total += sa::layout_count_host(pattern_of_layout(p, g), n, block);
    if (total > INT32_MAX) return SA_ERR_UNSUPPORTED;
    if (capacity < total) return SA_ERR_BUFFER_TOO_SMALL;
    hipError_t e = sa::layout_launch(n, block, p.pattern, head_mode, p.sub, stride_l, summary_c, p.n_layouts,
                                     row_ptr, col_idx, kind, col_ptr, row_idx, kind_t,
                                     static_cast<hipStream_t>(stream));
    return e == hipSuccess ? SA_OK : SA_ERR_HIP;
}

int sparse_attn_fwd(int64_t n, int32_t block, int32_t stride_l, int32_t summary_c,
                    int32_t pattern, int32_t head_mode, const int32_t* row_ptr,
                    const int32_t* col_idx, const uint8_t* kind, int32_t batch, int32_t heads,
                    int32_t d_head, int32_t dtype, const void* q, const void* k, const void* v,
                    const int64_t* strides, float softmax_scale, void* o, float* lse,
                    void* stream) {
    PatternArgs p;
    int st = check_pattern(n, block, stride_l, summary_c, pattern, head_mode, &p);
    if (st != SA_OK) return st;
    st = check_tensor_args(p, batch, heads, d_head, dtype, strides);
    if (st != SA_OK) return st;
    if (!row_ptr || !col_idx || !kind || !q || !k || !v || !o || !lse) return SA_ERR_INVALID;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o)) return SA_ERR_INVALID;
    if (!isfinite(softmax_scale) || !(softmax_scale > 0.f)) return SA_ERR_INVALID;
    sa::AttnArgs a = make_args(p, batch, heads, d_head, strides, softmax_scale, row_ptr, col_idx, nullptr, nullptr);
    const hipStream_t s = static_cast<hipStream_t>(stream);
    StridedPlan plan;
    if (strided_plan(p, batch, heads, d_head, dtype, strides, softmax_scale, false, &plan)) {
        hipError_t e = hipSuccess;
        if (plan.fused) {
            e = sa::strided_fwd(plan.rows, q, k, v, o, lse, s);
            return e == hipSuccess ? SA_OK : SA_ERR_HIP;
        }
        if (plan.band) e = sa::fwd_launch(plan.b, dtype, q, k, v, o, lse, s);
        if (plan.merge) plan.c.epilogue = sa::EPI_MERGE;  // the classes join the band
        if (e == hipSuccess && plan.classes) e = sa::fwd_launch(plan.c, dtype, q, k, v, o, lse, s);
        return e == hipSuccess ? SA_OK : SA_ERR_HIP;
    }
    hipError_t e = sa::fwd_launch(a, dtype, q, k, v, o, lse, s);
    return e == hipSuccess ? SA_OK : SA_ERR_HIP;
}

int sparse_attn_bwd_workspace_size(int64_t n, int32_t block, int32_t stride_l,
                                   int32_t summary_c, int32_t pattern, int32_t head_mode,
                                   int32_t batch, int32_t heads, int32_t d_head, int32_t dtype,
                                   size_t* bytes) {
    PatternArgs p;
    int st = check_pattern(n, block, stride_l, summary_c, pattern, head_mode, &p);
    if (st != SA_OK) return st;
    if (batch < 1 || heads < 1 || (dtype != SA_F32 && dtype != SA_BF16) || !bytes) return SA_ERR_INVALID;
    if (d_head != 32 && d_head != 64 && d_head != 128) return SA_ERR_UNSUPPORTED;
    *bytes = sa::bwd_workspace_bytes(batch, heads, n, p.nq, p.n_layouts);
    return SA_OK;
}

int sparse_attn_bwd(int64_t n, int32_t block, int32_t stride_l, int32_t summary_c,
                    int32_t pattern, int32_t head_mode, const int32_t* row_ptr,
                    const int32_t* col_idx, const uint8_t* kind, const int32_t* col_ptr,
                    const int32_t* row_idx, const uint8_t* kind_t, int32_t batch,
                    int32_t heads, int32_t d_head, int32_t dtype, const void* q, const void* k,
                    const void* v, const void* o, const void* dout, const float* lse,
                    const int64_t* strides, float softmax_scale, void* dq, void* dk, void* dv,
                    void* workspace, size_t workspace_bytes, void* stream) {
    sa::AttnArgs a;
    StridedPlan plan;
    size_t need = 0;
    bool planned = false;
    const int st = check_bwd(n, block, stride_l, summary_c, pattern, head_mode, row_ptr, col_idx, kind, col_ptr,
                             row_idx, kind_t, batch, heads, d_head, dtype, q, k, v, o, dout, lse, strides,
                             softmax_scale, dq, dk, dv, &a, &need, &planned, &plan);
    if (st != SA_OK) return st;
    if (workspace_bytes < need) return SA_ERR_BUFFER_TOO_SMALL;
    if (need > 0 && (!workspace || !aligned16(workspace))) return SA_ERR_INVALID;
    hipError_t e = launch_bwd(a, planned, plan, dtype, q, k, v, o, dout, lse, dq, dk, dv, workspace,
                              static_cast<hipStream_t>(stream));
    return e == hipSuccess ? SA_OK : SA_ERR_HIP;
}

int sparse_attn_bwd_stage(int64_t n, int32_t block, int32_t stride_l, int32_t summary_c, int32_t pattern,
                          int32_t head_mode, const int32_t* row_ptr, const int32_t* col_idx, const uint8_t* kind,
                          const int32_t* col_ptr, const int32_t* row_idx, const uint8_t* kind_t, int32_t batch,
                          int32_t heads, int32_t d_head, int32_t dtype, const void* q, const void* k, const void* v,
                          const void* o, const void* dout, const float* lse, const int64_t* strides,
                          float softmax_scale, void* dq, void* dk, void* dv, void* workspace, size_t workspace_bytes,
                          int32_t stages, void* stream) {
    if (stages < 1 || stages > SA_BWD_ALL_STAGES) return SA_ERR_INVALID;
    sa::AttnArgs a;
    StridedPlan plan;
    size_t need = 0;
    bool planned = false;
    const int st = check_bwd(n, block, stride_l, summary_c, pattern, head_mode, row_ptr, col_idx, kind, col_ptr,
                             row_idx, kind_t, batch, heads, d_head, dtype, q, k, v, o, dout, lse, strides,
                             softmax_scale, dq, dk, dv, &a, &need, &planned, &plan);
    if (st != SA_OK) return st;
    if (workspace_bytes < need) return SA_ERR_BUFFER_TOO_SMALL;
    if (need > 0 && (!workspace || !aligned16(workspace))) return SA_ERR_INVALID;
    // the fp32 path has no separate stages
    const int parts = dtype == SA_BF16 ? stages : sa::BWD_ALL;
    if (dtype != SA_BF16 && stages != SA_BWD_ALL_STAGES) return SA_ERR_UNSUPPORTED;
    hipError_t e = launch_bwd(a, planned, plan, dtype, q, k, v, o, dout, lse, dq, dk, dv, workspace,
                              static_cast<hipStream_t>(stream), parts);
    return e == hipSuccess ? SA_OK : SA_ERR_HIP;
}

int sparse_attn_bwd_noalloc_max_workspace(size_t* bytes) {
    if (!bytes) return SA_ERR_INVALID;
    *bytes = kScratchBytes;
    return SA_OK;
}

int sparse_attn_bwd_noalloc(int64_t n, int32_t block, int32_t stride_l, int32_t summary_c, int32_t pattern,
                            int32_t head_mode, const int32_t* row_ptr, const int32_t* col_idx, const uint8_t* kind,
                            const int32_t* col_ptr, const int32_t* row_idx, const uint8_t* kind_t, int32_t batch,
                            int32_t heads, int32_t d_head, int32_t dtype, const void* q, const void* k, const void* v,
                            const void* o, const void* dout, const float* lse, const int64_t* strides,
                            float softmax_scale, void* dq, void* dk, void* dv, void* stream) {
    sa::AttnArgs a;
    StridedPlan plan;
    size_t need = 0;
    bool planned = false;
    int st = check_bwd(n, block, stride_l, summary_c, pattern, head_mode, row_ptr, col_idx, kind, col_ptr, row_idx,
                       kind_t, batch, heads, d_head, dtype, q, k, v, o, dout, lse, strides, softmax_scale, dq, dk,
                       dv, &a, &need, &planned, &plan);
    if (st != SA_OK) return st;
    if (need > kScratchBytes) return SA_ERR_BUFFER_TOO_SMALL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    void* ws = nullptr;
    st = scratch_address(s, &ws);
    if (st != SA_OK) return st;
    // the workspace's contents on entry are ignored: the pre kernel writes the
    // row statistics and empties the work counters before anything reads them
    hipError_t e = launch_bwd(a, planned, plan, dtype, q, k, v, o, dout, lse, dq, dk, dv, ws, s);
    return e == hipSuccess ? SA_OK : SA_ERR_HIP;
}


int sparse_attn_decode_workspace_size(int64_t pos, int32_t stride_l, int32_t summary_c, int32_t pattern,
                                      int32_t head_mode, int32_t batch, int32_t heads, int32_t d_head,
                                      int32_t dtype, size_t* bytes) {
    int32_t internal = 0, sub = 0;
    int st = check_decode_pattern(pos, stride_l, summary_c, pattern, head_mode, &internal, &sub);
    if (st != SA_OK) return st;
    st = check_decode_shape(batch, heads, d_head, dtype);
    if (st != SA_OK) return st;
    if (!bytes) return SA_ERR_INVALID;
    *bytes = sa::decode_workspace_bytes(internal, head_mode, sub, (int32_t)pos, stride_l, summary_c, batch, heads,
                                        d_head);
    return SA_OK;
}

int sparse_attn_decode(int64_t pos, int32_t stride_l, int32_t summary_c, int32_t pattern, int32_t head_mode,
                       int32_t batch, int32_t heads, int32_t d_head, int32_t dtype, const void* q,
                       const int64_t* q_strides, const void* k_cache, const void* v_cache,
                       const int64_t* kv_strides, float softmax_scale, void* o, float* lse, void* workspace,
                       size_t workspace_bytes, void* stream) {
    int32_t internal = 0, sub = 0;
    int st = check_decode_pattern(pos, stride_l, summary_c, pattern, head_mode, &internal, &sub);
    if (st != SA_OK) return st;
    st = check_decode_shape(batch, heads, d_head, dtype);
    if (st != SA_OK) return st;
    if (!q || !q_strides || !k_cache || !v_cache || !kv_strides || !o || !lse) return SA_ERR_INVALID;
    if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(o)) return SA_ERR_INVALID;
    const int64_t unit = dtype == SA_BF16 ? 8 : 4;  // elements per 16 bytes
    for (int t = 0; t < 2; ++t)
        if (q_strides[t] < 0 || q_strides[t] % unit != 0) return SA_ERR_INVALID;
    for (int t = 0; t < 3; ++t)
        if (kv_strides[t] < 0 || kv_strides[t] % unit != 0) return SA_ERR_INVALID;
    if (kv_strides[2] < d_head) return SA_ERR_INVALID;
    if (!isfinite(softmax_scale) || !(softmax_scale > 0.f)) return SA_ERR_INVALID;
    const size_t need = sa::decode_workspace_bytes(internal, head_mode, sub, (int32_t)pos, stride_l, summary_c, batch,
                                                   heads, d_head);
    if (workspace_bytes < need) return SA_ERR_BUFFER_TOO_SMALL;
    if (!workspace || !aligned16(workspace)) return SA_ERR_INVALID;
    hipError_t e = sa::decode_launch(internal, head_mode, sub, (int32_t)pos, stride_l, summary_c, batch, heads, d_head,
                                     dtype, q, q_strides, k_cache, v_cache, kv_strides, softmax_scale, o, lse,
                                     workspace, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? SA_OK : SA_ERR_HIP;
}

int sparse_attn_transposed_workspace_size(int64_t n, int32_t block, int32_t stride_l, int32_t class_block,
                                          int32_t batch, int32_t heads, int32_t d_head, int32_t dtype, size_t* bytes) {
    TransposedPlan p;
    const int st = plan_transposed(n, block, stride_l, class_block, batch, heads, d_head, dtype, 1.f, &p);
    if (st != SA_OK) return st;
    if (!bytes) return SA_ERR_INVALID;
    *bytes = p.workspace;
    return SA_OK;
}

int sparse_attn_fwd_transposed(int64_t n, int32_t block, int32_t stride_l, int32_t class_block,
                               const int32_t* row_ptr, const int32_t* col_idx, const uint8_t* kind, int32_t batch,
                               int32_t heads, int32_t d_head, int32_t dtype, const void* q, const void* k,
                               const void* v, float softmax_scale, void* o, float* lse, void* workspace,
                               size_t workspace_bytes, void* stream) {
    if (!isfinite(softmax_scale) || !(softmax_scale > 0.f)) return SA_ERR_INVALID;
    TransposedPlan p;
    const int st = plan_transposed(n, block, stride_l, class_block, batch, heads, d_head, dtype, softmax_scale, &p);
    if (st != SA_OK) return st;
    if (!row_ptr || !col_idx || !kind || !q || !k || !v || !o || !lse) return SA_ERR_INVALID;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o)) return SA_ERR_INVALID;
    if (workspace_bytes < p.workspace) return SA_ERR_BUFFER_TOO_SMALL;
    if (p.workspace > 0 && (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0)) return SA_ERR_INVALID;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    // the band (strided A1 layout), then the classes merged into it
    const sa::AttnArgs band = make_args(p.band, batch, heads, d_head, p.strides, softmax_scale, row_ptr, col_idx,
                                        nullptr, nullptr);
    sa::AttnArgs cls = p.cls;
    cls.epilogue = sa::EPI_MERGE;
    hipError_t e = sa::fwd_launch(band, dtype, q, k, v, o, lse, s);
    if (e == hipSuccess) e = sa::fwd_launch(cls, dtype, q, k, v, o, lse, s);
    return e == hipSuccess ? SA_OK : SA_ERR_HIP;
}

int sparse_attn_bwd_transposed(int64_t n, int32_t block, int32_t stride_l, int32_t class_block,
                               const int32_t* row_ptr, const int32_t* col_idx, const uint8_t* kind,
                               const int32_t* col_ptr, const int32_t* row_idx, const uint8_t* kind_t, int32_t batch,
                               int32_t heads, int32_t d_head, int32_t dtype, const void* q, const void* k,
                               const void* v, const void* o, const void* dout, const float* lse, float softmax_scale,
                               void* dq, void* dk, void* dv, void* workspace, size_t workspace_bytes, void* stream) {
    if (!isfinite(softmax_scale) || !(softmax_scale > 0.f)) return SA_ERR_INVALID;
    TransposedPlan p;
    const int st = plan_transposed(n, block, stride_l, class_block, batch, heads, d_head, dtype, softmax_scale, &p);
    if (st != SA_OK) return st;
    if (!row_ptr || !col_idx || !kind || !col_ptr || !row_idx || !kind_t) return SA_ERR_INVALID;
    if (!q || !k || !v || !o || !dout || !lse || !dq || !dk || !dv) return SA_ERR_INVALID;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(dout) || !aligned16(dq) ||
        !aligned16(dk) || !aligned16(dv))
        return SA_ERR_INVALID;
    if (workspace_bytes < p.workspace) return SA_ERR_BUFFER_TOO_SMALL;
    if (p.workspace > 0 && (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0)) return SA_ERR_INVALID;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    // the band's backward given the merged O and LSE, then the classes' dQ and
    // dK / dV added to it
    const sa::AttnArgs band = make_args(p.band, batch, heads, d_head, p.strides, softmax_scale, row_ptr, col_idx,
                                        col_ptr, row_idx);
    sa::AttnArgs cls = p.cls;
    cls.epilogue = sa::EPI_ADD;
    hipError_t e = sa::bwd_launch(band, dtype, q, k, v, o, dout, lse, dq, dk, dv, workspace, s);
    if (e == hipSuccess)
        e = sa::bwd_launch(cls, dtype, q, k, v, o, dout, lse, dq, dk, dv, workspace, s, sa::BWD_DQ | sa::BWD_DKDV);
    return e == hipSuccess ? SA_OK : SA_ERR_HIP;
}

const char* sparse_attn_status_string(int status) {
    switch (status) {
    case SA_OK: return "success";
    case SA_ERR_INVALID: return "invalid argument";
    case SA_ERR_UNSUPPORTED: return "unsupported configuration";
    case SA_ERR_BUFFER_TOO_SMALL: return "buffer too small";
    case SA_ERR_HIP: return "HIP runtime error";
    default: return "unknown status";
    }
}

}  // extern "C"
