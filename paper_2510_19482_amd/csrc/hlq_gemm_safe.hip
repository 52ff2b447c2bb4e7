// Fallback of the tiled matrix-core GEMM for weights it cannot represent.  That kernel rebuilds
// W^ = sum_j s_j b_j + z (Eq. 3) in fp16 registers with pre-scaled scales (s_j * 2^7), which is only
// finite for |s_j| < 512; any finite fp16 scale is a valid HLQ parameter, though.  The tiled kernel
// therefore looks at every scale and zero it loads and raises a flag in the workspace if one lies
// outside its range; behind it comes this kernel (or, where K is split, the kernel that adds the partial sums, with the
// same function in it: one launch less), leaves at once if the flag
// is down (the normal case: one scalar load per workgroup), and otherwise computes the whole
// product again the plain way -- W^ element by element in fp32 from the plane bits, fp32
// accumulation -- and overwrites Y.  Slow, exact to fp32 rounding, valid for every finite fp16
// parameter.  The last workgroup to finish lowers the flag again.
#include "hlq_gemm_safe.h"

namespace {

__global__ void __launch_bounds__(64)
hlq_gemm_safe_kernel(const HlqSafeProbs pr, const int M, const int out_f32, int *flag, int *done)
{
    // an ordinary load: the flag was written by the launch before this one, and a kernel boundary makes that visible
    if (*(const int *)flag == 0) return;
    hlq_safe_recompute(pr, M, out_f32, flag, done, blockIdx.x, gridDim.x);
}

} // namespace

// Launches the fallback behind a tiled-kernel launch over the same problems.  `ws` is the call's workspace.
hlq_status hlq_launch_gemm_safe(int count, const HlqGemvItem *items, int64_t M, hlq_out_dtype out, void *ws, hipStream_t st)
{
    HlqSafeProbs pr;
    const hlq_status s = hlq_safe_problems(count, items, M, pr);
    if (s != HLQ_OK) return s;
    // few workgroups: in the normal case all of them only look at the flag and leave, and that costs per workgroup
    const unsigned grid = (unsigned)(pr.items_total < HLQ_SAFE_WAVES ? pr.items_total : HLQ_SAFE_WAVES);
    hlq_gemm_safe_kernel<<<grid, 64, 0, st>>>(pr, (int)M, out == HLQ_OUT_F32, hlq_ws_range_flag(ws), hlq_ws_range_flag(ws) + 1);
    return HLQ_OK;
}
