// Pieces shared by the matrix-core kernels: rebuilding fp16 weights from bit-plane words.
#pragma once

#include "hlq_internal.h"

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));

// vmcnt(0) with the other counters left alone (expcnt 7, lgkmcnt 15)
constexpr int HLQ_WAIT_VM0 = (7 << 4) | (15 << 8);

// 16 bytes per lane from global memory straight into LDS at lds_base + 16 * lane.  Issued as inline
// assembly so that the compiler's wait-count bookkeeping does not tie later LDS reads (of the other
// buffer) to it; completion is awaited explicitly (vmcnt) before the barrier that publishes the tile.
__device__ __forceinline__ void dma_16B_per_lane(const void *gptr, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gptr), "s"(lds_base) : "memory", "m0");
}

// In a plane word, bits p and p+16 are the adjacent weights k0 = 2p, 2p+1 of the word's 32-k block.
// (w << t) & 0x20002000 isolates pair p at bit 13 of both 16-bit halves: as packed fp16 that is
// (2^-7 b[2p], 2^-7 b[2p+1]); with 0x40004000 (bit 14) it is (2 b, 2 b).  Position (13 or 14) and
// left shift that bring pair p there; pair 15 is reached with a right shift by one (shift = -1).
__host__ __device__ constexpr int hlq_pair_pos(int p) { return p == 15 ? 14 : (p == 0 ? 14 : (p % 2 == 1 ? 13 : 14)); }
__host__ __device__ constexpr int hlq_pair_shift(int p) { return p == 15 ? -1 : hlq_pair_pos(p) - p; }

// Rebuilding weights: the words of Q planes and the parameters of a quant segment -> packed fp16 pairs
// (W^[2p], W^[2p + 1]), p = 0..15 (Eq. 3).
//
// Two and three planes: a segment has four or eight different weights.  They are made once per segment (sums in
// fp32, rounded to fp16 once), their low and high bytes in a register (pair) each, and v_perm_b32 looks four weights up at a
// time: a selector word holds the codes of plane bits p, p + 8, p + 16, p + 24 in its bytes, two look-ups give
// their low and high bytes, and two more byte permutations make pairs p and p + 8 of them (bits p and p + 16 are adjacent k).
// The selectors of two planes come from words with their bits interleaved, even and odd plane bits apart: 18
// instructions a word.  A word takes 50 instructions at q = 2 and 66 at q = 3; a mask and a packed FMA per plane and pair
// (one plane, and the fourth of four: 106 a word instead of 160) take 80 and 120.
// The rounding is one instead of one per plane: relative error 2.4e-4 -> 1.9e-4 at q = 2, 3, 3.1e-4 -> 2.6e-4 at q = 4.
// us a call by FMA -> by look-up: 8B layer M = 512 q = 2 / 3 / 4 243 / 279 / 303 -> 239 / 250 / 281, M = 2048 q = 2 832 -> 809,
// q = 3 with G = 64 1006 -> 891; 4096 x 14336, q = 3, G = 64, M = 24 21.4 -> 19.8.
template <int Q>
struct HlqRebuild {
    static constexpr int TABLE = Q == 1 ? 0 : Q < 4 ? Q : 3;   // planes looked up; the others by FMA
    uint32_t lo[2], hi[2];      // bytes of the 2^TABLE weights
    half2v z2, s13, s14;        // one plane: its start value; the scale of the plane added by FMA, see hlq_pair_pos
    uint32_t even, odd;         // planes 0 and 1 of the word, bits interleaved: code of bit 2k (2k + 1) at bit 2k
    uint32_t w2, wf;            // the third plane's word, the word of the plane added by FMA

    // mt: fp16 bit patterns of s_0 .. s_{Q-1}, z (16- or 32-bit containers).  Requires |s| < 512 (hlq_gemm_safe.hip has the rest).
    template <typename T>
    __device__ __forceinline__ void segment(const T (&mt)[Q + 1])
    {
        auto param = [&](int r) { return __builtin_bit_cast(_Float16, (uint16_t)mt[r]); };
        if constexpr (TABLE > 0) {
            float v[8];
            v[0] = (float)param(Q);
#pragma unroll
            for (int j = 0; j < TABLE; ++j)
#pragma unroll
                for (int c = 0; c < (1 << j); ++c) v[(1 << j) + c] = v[c] + (float)param(j);
#pragma unroll
            for (int i = 0; i < (1 << TABLE) / 4; ++i) {
                const uint32_t a = pack(v[4 * i], v[4 * i + 1]), b = pack(v[4 * i + 2], v[4 * i + 3]);
                lo[i] = __builtin_amdgcn_perm(b, a, 0x06040200u);
                hi[i] = __builtin_amdgcn_perm(b, a, 0x07050301u);
            }
        } else {
            const _Float16 z = param(Q);
            z2 = (half2v){z, z};
        }
        if constexpr (Q == 1 || Q == 4) {   // s * 2^7 for pairs read at bit 13, s / 2 for pairs read at bit 14
            const _Float16 s = param(Q - 1), a = s * (_Float16)128.0f, b = s * (_Float16)0.5f;
            s13 = (half2v){a, a};
            s14 = (half2v){b, b};
        }
    }
    __device__ __forceinline__ void word(const uint32_t (&w)[Q][4], int d)
    {
        if constexpr (TABLE > 0) {
            even = (w[0][d] & 0x55555555u) | ((w[1][d] << 1) & 0xaaaaaaaau);
            odd = ((w[0][d] >> 1) & 0x55555555u) | (w[1][d] & 0xaaaaaaaau);
            if constexpr (TABLE > 2) w2 = w[2][d];
        }
        if constexpr (Q == 1 || Q == 4) wf = w[Q - 1][d];
    }
    // pairs p and p + 8 (p < 8) of the word
    __device__ __forceinline__ void pairs(int p, uint32_t &first, uint32_t &second) const
    {
        if constexpr (TABLE > 0) {
            uint32_t s = ((p & 1 ? odd : even) >> (p & 6)) & 0x03030303u;
            if constexpr (TABLE > 2) s |= (p < 2 ? w2 << (2 - p) : w2 >> (p - 2)) & 0x04040404u;
            const uint32_t l = __builtin_amdgcn_perm(lo[TABLE > 2 ? 1 : 0], lo[0], s), h = __builtin_amdgcn_perm(hi[TABLE > 2 ? 1 : 0], hi[0], s);
            first = __builtin_amdgcn_perm(h, l, 0x06020400u);
            second = __builtin_amdgcn_perm(h, l, 0x07030501u);
        } else {
            first = second = __builtin_bit_cast(uint32_t, z2);
        }
        if constexpr (Q == 1 || Q == 4) {
            first = add_plane(first, p);
            second = add_plane(second, p + 8);
        }
    }

private:
    static __device__ __forceinline__ uint32_t pack(float a, float b)
    {
        return __builtin_bit_cast(uint32_t, (half2v){(_Float16)a, (_Float16)b});   // nearest even
    }
    __device__ __forceinline__ uint32_t add_plane(uint32_t o, int p) const
    {
        const uint32_t sh = hlq_pair_shift(p) < 0 ? (wf >> 1) : (wf << (hlq_pair_shift(p) < 0 ? 0 : hlq_pair_shift(p)));
        const uint32_t m = sh & (hlq_pair_pos(p) == 13 ? 0x20002000u : 0x40004000u);
        const half2v r = __builtin_bit_cast(half2v, m) * (hlq_pair_pos(p) == 13 ? s13 : s14) + __builtin_bit_cast(half2v, o);
        return __builtin_bit_cast(uint32_t, r);
    }
};
