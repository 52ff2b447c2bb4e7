// The fp32 recomputation behind the matrix-core GEMMs that rebuild weights in fp16 (hlq_gemm_safe.hip says when and why), as
// device functions: the launch behind the tiled kernel, or behind K slices of either, runs it if the flag was raised; a workgroup of
// the short-M kernel that has all of K runs it for its own tile.
#pragma once

#include "hlq_internal.h"

constexpr int SAFE_ROWS = 8;   // activation rows per work item
#define HLQ_SAFE_WAVES 512      // wavefronts of a launch that does nothing else: each of them costs the normal case a look at the flag

__device__ __forceinline__ float half_bits_to_float(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }

// One work item: SAFE_ROWS rows from m0 on of one column tile, by one wavefront.
__device__ __forceinline__ void hlq_safe_item(const HlqSafeProb &P, const int tile, const int m0, const int M, const int out_f32)
{
    const int lane = threadIdx.x & 63;
    const int tw = hlq_tile_width(tile, P.N);
    const bool col_ok = lane < tw;
    const int lane_c = col_ok ? lane : tw - 1;
    const char *tile_base = P.packed + (size_t)tile * HLQ_TILE_N * P.col_bytes;
    const int q = P.q, G = P.G;
    float acc[SAFE_ROWS];
#pragma unroll
    for (int r = 0; r < SAFE_ROWS; ++r) acc[r] = 0.f;
    for (int c = 0; c < P.nchunks; ++c) {
        const char *rec = tile_base + hlq_rec_in_tile(tw, c, q, G);
        // scales of the chunk's quant segments; a 256-wide group keeps them in the record of its even chunk
        const int cm = G > 128 ? (c & ~1) : c;
        const uint16_t *mp = (const uint16_t *)(tile_base + hlq_rec_in_tile(tw, cm, q, G) + (size_t)tw * q * 16);
        float s[4] = {0.f, 0.f, 0.f, 0.f}, z = 0.f;
        // word by word (32 k), all indices known at compile time: nothing of this is in scratch memory, which the launch
        // that also adds the partial sums would have to set aside in every call
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = j < q ? ((const uint32_t *)rec)[(j * tw + lane_c) * 4 + d] : 0u;
            if (d == 0 || G == 32 || (G == 64 && d == 2)) {   // a quant group begins
                const int sg = G >= 128 ? 0 : 32 * d / G;
#pragma unroll
                for (int j = 0; j < 4; ++j) s[j] = j < q ? half_bits_to_float(mp[(sg * (q + 1) + j) * tw + lane_c]) : 0.f;
                z = half_bits_to_float(mp[(sg * (q + 1) + q) * tw + lane_c]);
            }
            for (int b = 0; b < 32; ++b) {
                const int bit = hlq_bit_pos(b);
                float wv = z;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if ((w[j] >> bit) & 1u) wv += s[j];
                const size_t k = (size_t)c * 128 + 32 * d + b;
#pragma unroll
                for (int r = 0; r < SAFE_ROWS; ++r) {
                    const int m = min(m0 + r, M - 1);   // rows past M repeat the last one and are dropped
                    acc[r] += half_bits_to_float(P.X[(size_t)m * P.ldx + k]) * wv;
                }
            }
        }
    }
    if (col_ok) {
        const size_t n = (size_t)tile * HLQ_TILE_N + lane;
#pragma unroll
        for (int r = 0; r < SAFE_ROWS; ++r) {
            if (m0 + r >= M) break;
            if (out_f32) ((float *)P.Y)[(size_t)(m0 + r) * P.ldy + n] = acc[r];
            else ((_Float16 *)P.Y)[(size_t)(m0 + r) * P.ldy + n] = (_Float16)acc[r];
        }
    }
}

// Wavefront `wave` of `waves` (all of the launch, every one of which comes here) computes its share of the items; the last
// one to finish lowers the flag for the next call.
__device__ __forceinline__ void hlq_safe_recompute(const HlqSafeProbs &pr, const int M, const int out_f32, int *flag, int *done,
                                                   const long wave, const long waves)
{
    const int lane = threadIdx.x & 63;
    for (long item = wave; item < pr.items_total; item += waves) {
        int pi = 0;
        while (pi + 1 < pr.count && item >= pr.p[pi + 1].item_begin) ++pi;
        const HlqSafeProb &P = pr.p[pi];
        const long local = item - P.item_begin;
        hlq_safe_item(P, (int)(local % P.ntiles), (int)(local / P.ntiles) * SAFE_ROWS, M, out_f32);
    }
    if (lane == 0) {
        const int old = __hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (old == (int)waves - 1) {
            __hip_atomic_store(done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(flag, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// host: the problems of a call
static inline hlq_status hlq_safe_problems(int count, const HlqGemvItem *items, int64_t M, HlqSafeProbs &pr)
{
    if (count < 1 || count > HLQ_MAX_BATCH || M < 1 || M > 0x7fffffff) return HLQ_ERR_UNSUPPORTED;
    long total = 0;
    for (int i = 0; i < count; ++i) {
        HlqSafeProb &p = pr.p[i];
        p.packed = (const char *)items[i].packed;
        p.col_bytes = items[i].dm.col_bytes;
        p.X = items[i].x;
        p.ldx = items[i].ldx;
        p.Y = items[i].y;
        p.ldy = items[i].ldy;
        p.N = items[i].dm.N;
        p.ntiles = items[i].dm.ntiles;
        p.nchunks = items[i].dm.nchunks;
        p.q = items[i].dm.q;
        p.G = items[i].dm.G;
        p.item_begin = total;
        total += (long)items[i].dm.ntiles * (long)((M + SAFE_ROWS - 1) / SAFE_ROWS);
    }
    for (int i = count; i < HLQ_MAX_BATCH; ++i) pr.p[i] = pr.p[0];
    pr.count = count;
    pr.items_total = total;
    return HLQ_OK;
}
