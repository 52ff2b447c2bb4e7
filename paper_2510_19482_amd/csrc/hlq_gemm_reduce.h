// The launch behind a matrix-core GEMM whose K was cut into slices: adds the slices' partial sums (hlq_gemm_safe.hip).
#pragma once

#include "hlq_internal.h"

struct HlqReduceProb {
    const float *part;   // [nslices][M][N]
    void *Y;
    long ldy;
    int N, nslices, blk_begin;
    int wide;   // Y's rows are aligned to four elements: one store per lane
};
struct HlqReduceProbs {
    HlqReduceProb p[HLQ_MAX_BATCH];
};
constexpr int HLQ_REDUCE_LANES = 256, HLQ_REDUCE_OUT = 4 * HLQ_REDUCE_LANES;   // outputs per block

// host: the problems with partial sums of a call, in the order in which they are added
struct HlqReduce {
    HlqReduceProbs probs;
    int begin[HLQ_MAX_BATCH], count = 0, out_f32;
    int64_t M;
    long blocks = 0;

    HlqReduce(int64_t M_, int f32) : out_f32(f32), M(M_) {}
    bool add(const float *part, void *Y, long ldy, int N, int nslices)
    {
        HlqReduceProb &r = probs.p[count];
        r.part = part;
        r.Y = Y;
        r.ldy = ldy;
        r.N = N;
        r.nslices = nslices;
        r.blk_begin = begin[count] = (int)blocks;
        r.wide = (((uintptr_t)Y | ((uintptr_t)ldy * (out_f32 ? 4u : 2u))) & (out_f32 ? 15u : 7u)) == 0;
        ++count;
        blocks += (long)(((size_t)M * N + HLQ_REDUCE_OUT - 1) / HLQ_REDUCE_OUT);
        return blocks <= 0x7fffffffL / (HLQ_REDUCE_LANES / 64);
    }
};
// items: all problems of the call, which are computed again if the flag is up
hlq_status hlq_launch_gemm_reduce(HlqReduce &red, int count, const HlqGemvItem *items, void *ws, hipStream_t st);
