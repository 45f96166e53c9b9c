// Backward entry of the library (Sec. 5.4, recomputation): workspace size and
// dispatch to the bf16 kernels of each head size (sa_bwd_kernels.h,
// sa_bwd_bf16_d*.hip) and the fp32 kernels (sa_f32.hip).
#include "sa_bwd_kernels.h"

namespace sa {

size_t bwd_workspace_bytes(int64_t batch, int64_t heads, int64_t n, int64_t nq, int n_layouts) {
    return (size_t)bwd_workspace_size(batch * heads * n, nq, n_layouts);
}

hipError_t bwd_launch(const AttnArgs& a, int dtype, const void* q, const void* k, const void* v,
                      const void* o, const void* dout, const float* lse, void* dq, void* dk,
                      void* dv, void* workspace, hipStream_t stream, int parts) {
    const BwdWorkspace ws = bwd_workspace(workspace, a.ws_rows, layout_count(a.mode, a.sub));
    if (dtype == 1) {
        switch (a.d) {
        case 32: return bwd_bf16_d32(a, q, k, v, o, dout, lse, dq, dk, dv, ws, stream, parts);
        case 64: return bwd_bf16_d64(a, q, k, v, o, dout, lse, dq, dk, dv, ws, stream, parts);
        default: return bwd_bf16_d128(a, q, k, v, o, dout, lse, dq, dk, dv, ws, stream, parts);
        }
    }
    return bwd_f32(a, q, k, v, o, dout, lse, dq, dk, dv, ws, stream, parts);
}

}  // namespace sa
