// Fallback of the tiled matrix-core GEMM (and of the short-M one where it cuts K across workgroups) for weights it cannot represent.  That kernel rebuilds
// W^ = sum_j s_j b_j + z (Eq. 3) in fp16 registers with pre-scaled scales (s_j * 2^7), which is only
// finite for |s_j| < 512; any finite fp16 scale is a valid HLQ parameter, though.  The tiled kernel
// therefore looks at every scale and zero it loads and raises a flag in the workspace if one lies
// outside its range; behind it comes this kernel (or, where K is split, the kernel that adds the partial sums, with the
// same function in it: one launch less), leaves at once if the flag
// is down (the normal case: one scalar load per workgroup), and otherwise computes the whole
// product again the plain way -- W^ element by element in fp32 from the plane bits, fp32
// accumulation -- and overwrites Y.  Slow, exact to fp32 rounding, valid for every finite fp16
// parameter.  The last workgroup to finish lowers the flag again.
#include "hlq_gemm_reduce.h"
#include "hlq_gemm_safe.h"

namespace {

__global__ void __launch_bounds__(64)
hlq_gemm_safe_kernel(const HlqSafeProbs pr, const int M, const int out_f32, int *flag, int *done)
{
    // an ordinary load: the flag was written by the launch before this one, and a kernel boundary makes that visible
    if (*(const int *)flag == 0) return;
    hlq_safe_recompute(pr, M, out_f32, flag, done, blockIdx.x, gridDim.x);
}

// Adds the partial sums of the problems of a launch whose K was split, four outputs per lane (N is a multiple of 8), or,
// if the kernel before it met parameters outside its range, computes the call again: one launch behind the tiled kernel instead
// of two.  A dependent launch costs 1.7 us even when it only looks at the flag; the sums are latency-bound themselves
// (one 4-byte load per lane and slice and a 64-bit division per output before).
typedef int int4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));

// index of the problem that owns block `blk`: the table is ascending, unused entries INT_MAX
__device__ __forceinline__ int reduce_problem_of(const int4v &bb_lo, const int4v &bb_hi, int blk)
{
    return blk >= bb_hi.w ? 7 : blk >= bb_hi.z ? 6 : blk >= bb_hi.y ? 5 : blk >= bb_hi.x ? 4
         : blk >= bb_lo.w ? 3 : blk >= bb_lo.z ? 2 : blk >= bb_lo.y ? 1 : 0;
}

__device__ __forceinline__ void store_out(void *y, size_t idx, float v, int out_f32)
{
    if (out_f32) ((float *)y)[idx] = v;
    else ((_Float16 *)y)[idx] = (_Float16)v;   // round-to-nearest-even
}

__global__ void __launch_bounds__(HLQ_REDUCE_LANES)
hlq_gemm_mfma_group_reduce_kernel(const int4v bb_lo, const int4v bb_hi, const int M, const int out_f32, int *flag,
                                  const HlqReduceProbs probs, const HlqSafeProbs again)
{
    const int redo = *(const int *)flag;   // written by the launch before this one
    const int blk = (int)blockIdx.x;
    const HlqReduceProb P = probs.p[reduce_problem_of(bb_lo, bb_hi, blk)];
    const size_t i = ((size_t)(blk - P.blk_begin) * HLQ_REDUCE_LANES + threadIdx.x) * 4;
    const size_t total = (size_t)M * P.N;
    if (redo == 0) {
        if (i >= total) return;
        float4v a = {0.f, 0.f, 0.f, 0.f};
        const float *src = P.part + i;
        int s = 0;
        for (; s + 4 <= P.nslices; s += 4) {   // four slices in flight, added in slice order
            const float4v v0 = *(const float4v *)(src + (size_t)(s + 0) * total), v1 = *(const float4v *)(src + (size_t)(s + 1) * total);
            const float4v v2 = *(const float4v *)(src + (size_t)(s + 2) * total), v3 = *(const float4v *)(src + (size_t)(s + 3) * total);
            a = (((a + v0) + v1) + v2) + v3;
        }
        for (; s < P.nslices; ++s) a += *(const float4v *)(src + (size_t)s * total);
        const size_t m = total <= 0xffffffffu ? (unsigned)i / (unsigned)P.N : i / (unsigned)P.N;
        const size_t at = m * P.ldy + (i - m * P.N);
        typedef _Float16 half4v __attribute__((ext_vector_type(4)));
        if (P.wide && out_f32) {
            *(float4v *)((float *)P.Y + at) = a;
        } else if (P.wide) {
            *(half4v *)((_Float16 *)P.Y + at) = (half4v){(_Float16)a.x, (_Float16)a.y, (_Float16)a.z, (_Float16)a.w};
        } else {
            store_out(P.Y, at + 0, a.x, out_f32);
            store_out(P.Y, at + 1, a.y, out_f32);
            store_out(P.Y, at + 2, a.z, out_f32);
            store_out(P.Y, at + 3, a.w, out_f32);
        }
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    hlq_safe_recompute(again, M, out_f32, flag, flag + 1, (long)blk * (HLQ_REDUCE_LANES / 64) + wave, (long)gridDim.x * (HLQ_REDUCE_LANES / 64));
}

// Workgroups of that launch: those of the sums, and enough that the call is computed again by as many wavefronts as behind
// a tiled launch without split K (a group may split nothing but a narrow problem).  The surplus ones look at the flag and leave.
unsigned reduce_blocks(long sums, const HlqSafeProbs &again)
{
    const long redo = (again.items_total + HLQ_REDUCE_LANES / 64 - 1) / (HLQ_REDUCE_LANES / 64), most = HLQ_SAFE_WAVES / (HLQ_REDUCE_LANES / 64);
    const long want = redo < most ? redo : most;
    return (unsigned)(sums > want ? sums : want);
}

} // namespace

hlq_status hlq_launch_gemm_reduce(HlqReduce &red, int count, const HlqGemvItem *items, void *ws, hipStream_t st)
{
    static_assert(HLQ_MAX_BATCH == 8, "the kernel takes the first blocks of eight problems");
    for (int i = red.count; i < HLQ_MAX_BATCH; ++i) {
        red.probs.p[i] = red.probs.p[0];
        red.begin[i] = 0x7fffffff;
    }
    const int *b = red.begin;
    HlqSafeProbs again;
    const hlq_status s = hlq_safe_problems(count, items, red.M, again);
    if (s != HLQ_OK) return s;
    hlq_gemm_mfma_group_reduce_kernel<<<reduce_blocks(red.blocks, again), HLQ_REDUCE_LANES, 0, st>>>((int4v){b[0], b[1], b[2], b[3]}, (int4v){b[4], b[5], b[6], b[7]},
                                                                                     (int)red.M, red.out_f32, hlq_ws_range_flag(ws), red.probs, again);
    return hlq_hip_status(hipGetLastError());
}

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
