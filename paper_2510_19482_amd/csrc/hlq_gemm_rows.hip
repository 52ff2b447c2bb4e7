// hlq_lut_gemm for a handful of rows (small-batch decode, 3 <= M <= 16, quant groups of 128 or 256):
// the bit-serial product of Sec. 2 "Bit-Serial LUT-Based GEMM" / App. B with the per-plane dot products
// on the MX matrix cores, as in hlq_gemv_mx.hip, arranged for many activation rows:
//
//   Y[m,n] = sum_groups ( sum_j s_j[g,n] * <b_j[.,n], X[m,.]>_g  +  z[g,n] * sum_g(X[m,.]) )
//
// Planes become fp4 codes by AND masks.  An activation is a sum of four bf6 (e3m2) terms: 32 activations of a row (the
// k block that shares a scale in the matrix core) are brought below 16 by a power of two, the largest to [8, 16), each term is
// the remainder so far rounded to the nearest code, and the next remainder is multiplied by 16.  A term holds three
// significant bits and the sign of what it leaves; what four of them leave is at most 2^-20 of the block's largest, and
// nothing for an activation of more than 2^-9 of it (both as weighted by the plane codes, see below).  The terms' powers of two are the matrix core's own block scales (E8M0,
// a byte per lane and term), so nothing is undone at the end.
// Why bf6: with no operand wider than six bits the instruction takes 16 clocks and not 32, and it adds the products of a
// block exactly down to 2^-24 of the largest (measured), where bf8 x fp4 drops what is below 2^-13 of the largest of eight
// neighbours.  Four such terms are half the time of four exact bf8 terms and closer to the exact product: relative error of fp32 results,
// 4096 x 4096, q = 4, M = 16: 3.0e-6 -> 3.0e-7, with 1 % of the channels times 20 1.2e-5 -> 2.5e-6.
// Three terms are short of it where outliers share a block with the rest (2.5e-4 of a row's largest result, 1 % of K = 1024
// times 20), and so are four beside a massive activation, in the columns whose weights are zero there: one channel in 32 a
// thousand times the rest, relative error 5e-4 (bf8 terms: the fp32 sums' own).  Blocks in which all activations of an
// expansion register are 2^-8 or less of the largest, as weighted, are wide: their chunk has a second record with four terms of
// what the first four leave, scaled by itself (down to 2^-36 of the block's largest; 3e-7), and the main kernel goes
// through such chunks once more at its end.  In the others what is left of an activation is at most 2^-11 of the largest of its
// register.  With 1 % of the channels times 20 one block in 80000 is wide.  The test and the look at the flags cost 0.1 to 0.5 us
// a call (8B layer, q = 4, M = 16 41.9 -> 42.2, 4096 x 14336 18.7 -> 19.1).
//
// The terms lie along the ACCUMULATION: operand o holds terms [o TPO, (o + 1) TPO) of 16 / TPO activation
// rows, the NT = 4 / TPO matrix-core instructions of an item (plane j, block of 16 columns) chain
// through their accumulator, and what comes out is the finished dot product of every row -- one scale
// multiplication per (row, column, plane).  NT = 2 carries up to 8 rows, NT = 4 up to 16.  NT = 1 is the other
// end: all four terms of up to 4 rows in one operand, one matrix-core instruction per item, the four terms of a
// result in the four 16-lane groups, added by two cross-lane adds at the very end.
//
// Two kernels.  hlq_rows_split_kernel runs once per call and cuts every activation into its terms, in the form in which
// the matrix core wants them: a lane of it makes 32 activations of a row, with the packed conversions, and writes the six
// registers of every term and the scales of one lane of the main kernel.  Blocks carry their own scales, so there is
// no pass over the row before.  It is 4.2 us of a call of 4 rows, 5.5 of 8, 7.4 of 16 (8B layer), the hand-over between the
// launches included.  Made inside the main kernel instead, by all wavefronts of a workgroup for its run of chunks, the
// operands cost as much: nothing is requested while they are made (M = 4 31.7 us against 31.6, M = 16 53 against 43).
// hlq_gemm_rows_kernel has no activation work at all: a lane loads its operands straight into registers, one chunk ahead.
//
// Work split of the main kernel.  A workgroup of W wavefronts owns W / kw adjacent column tiles and one
// K slice; the kw wavefronts of a tile take consecutive runs of chunks and add their results through LDS
// at the end (as in hlq_gemv_mx.hip); nothing is shared before that, so there is no barrier in the chunk
// loop.  K slices of different workgroups meet in the workspace (partial sums, one arrival counter per
// tile, the last arriver adds in slice order).
//
// What bounds it, 8B layer at q = 4 in one launch (126 MB, 18 us at 6.9 TB/s): the pre-pass and the start of the main kernel, then
// the wait for weights requested two chunks ahead by 1.7 wavefronts per SIMD; at M = 16 68 matrix-core instructions (1088
// clocks) beside 290 vector instructions (1160) a chunk and wavefront.  Four bf8 terms -> four bf6 terms, us a call:
// q = 4  M = 4 32.8 -> 31.9, M = 8 39.1 -> 34.5, M = 16 56.5 -> 42.7;  q = 2  M = 8 28.9 -> 24.7, M = 16 44.2 -> 29.5.
#include "hlq_gemv_common.h"

#include <type_traits>

namespace {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half32_t __attribute__((ext_vector_type(32)));
typedef unsigned int uint6v __attribute__((ext_vector_type(6)));
typedef int int8v __attribute__((ext_vector_type(8)));
typedef unsigned int uint2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint16_t __attribute__((may_alias)) u16_alias;
typedef uint32_t __attribute__((may_alias)) u32_alias;

constexpr int rows_meta_stride(int Q) { return ((Q + 1) * 2 + 7) & ~7; }
// LDS per wavefront: scales [64][stride] | results [16][64] fp32 for the sum over the tile's kw runs
constexpr int rows_wave_lds(int Q) { return 64 * rows_meta_stride(Q) + 16 * 64 * 4; }
constexpr int rows_lds_bytes(int Q, int W) { return W * rows_wave_lds(Q); }
// The activations of a chunk in the workspace, NT operands of 16 rows: what lane (row, k block) of the main kernel holds,
// 6 NT words of codes and one of scales (byte o: operand o), four words at a time as [word / 4][lane][4]; a single
// word left over as [lane]
constexpr int rows_words(int NT) { return 6 * NT + 1; }
constexpr int rows_quads(int NT) { return rows_words(NT) % 4 == 1 ? rows_words(NT) / 4 : (rows_words(NT) + 3) / 4; }
constexpr int rows_chunk_bytes(int NT) { return rows_quads(NT) * 1024 + (rows_words(NT) % 4 == 1 ? 256 : 0); }
// operands, and activation rows they carry
constexpr int rows_operands(int rows) { return rows <= 4 ? 1 : rows <= 8 ? 2 : 4; }
constexpr int rows_carried(int NT) { return 4 * NT; }

// A block is wide if all activations of an expansion register (that are not all zero) are this many binary places below the
// largest, as weighted.
constexpr int ROWS_WIDE = 8;

// the workspace of a problem: records of all chunks, records of what they leave (of the chunks that have it), a flag for each
// chunk that has
__device__ __forceinline__ int *rows_flags(const GemvProb &P, int nt) { return (int *)(P.xt + (size_t)P.nchunks * 2 * rows_chunk_bytes(nt)); }
// plane codes are worth 1/2, 1, 2, 2 by expansion register: the activations' weights 1/2, 1/4, 1/8, 1/8 make every product a quarter
__device__ __forceinline__ constexpr int rows_weight(int rr) { return rr < 3 ? rr + 1 : 3; }
__device__ __forceinline__ float power_of_two(int e) { return __builtin_bit_cast(float, (uint32_t)(127 + e) << 23); }

// Workgroup = one wavefront = 16 / RPO chunks of all rows; problem blockIdx.y.  A lane takes 32 consecutive k of one row.
// Position 8 rr + 4 hh + n of a k block holds its activation 8 n + 2 rr + hh: weight k0 = 2 p + hh is plane bit p = 4 n + rr,
// which the plane expansion puts into nibble n + 4 hh of register rr.  The 4 of rows_weight goes into the scale.
template <int NT>
__global__ void __launch_bounds__(64) hlq_rows_split_kernel(const GemvProbs probs)
{
    constexpr int RPO = rows_carried(NT), TPO = 4 / NT, QUADS = rows_quads(NT);
    const GemvProb &P = probs.p[blockIdx.y];
    const int lane = (int)threadIdx.x, m = lane % RPO, g = lane / RPO % 4, ch = (int)blockIdx.x * (16 / RPO) + lane / (4 * RPO);
    if (!P.xt_own || ch >= P.nchunks) return;
    const bool have = m < P.M;
    const uint4 *src = (const uint4 *)(P.x + (size_t)min(m, P.M - 1) * P.ldx + (size_t)ch * 128 + 32 * g);
    uint32_t x[4][4];   // [n][rr]: activations 8 n + 2 rr, + 1
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const uint4 v = src[n];
        x[n][0] = v.x; x[n][1] = v.y; x[n][2] = v.z; x[n][3] = v.w;
    }
    // biased exponent ew of the largest weighted magnitude: all of them are below 2^(ew - 14), brought below 16
    int ew = -2, eall = 0, own[4];
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
        ushort2_t mx = {0, 0};
#pragma unroll
        for (int n = 0; n < 4; ++n) mx = __builtin_elementwise_max(mx, __builtin_bit_cast(ushort2_t, x[n][rr] & 0x7fff7fffu));
        const int largest = max((int)mx.x, (int)mx.y), e = largest >> 10;
        own[rr] = largest ? max(e, 1) - rows_weight(rr) : 99;
        ew = max(ew, max(e, 1) - rows_weight(rr));
        eall = max(eall, e);
    }
    const bool real = have && eall < 31;   // a row that the call has, and neither an infinity nor a NaN in the block
    const uint64_t wide = __ballot(real && ew - min(min(own[0], own[1]), min(own[2], own[3])) > ROWS_WIDE);
    const int s = 18 - ew;
    half32_t v;
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
        const int sr = s - rows_weight(rr), k1 = sr / 2, k2 = sr - k1;   // two factors: 2^sr need not be an fp16 number
        const _Float16 f1 = __builtin_bit_cast(_Float16, (uint16_t)((15 + k1) << 10)), f2 = __builtin_bit_cast(_Float16, (uint16_t)((15 + k2) << 10));
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int n = 0; n < 4; n += 2) {
                const half2_t p = __builtin_bit_cast(half2_t, __builtin_amdgcn_perm(x[n + 1][rr], x[n][rr], hh ? 0x07060302u : 0x05040100u)) * (half2_t){f1, f1} * (half2_t){f2, f2};
                v[8 * rr + 4 * hh + n] = p.x;
                v[8 * rr + 4 * hh + n + 1] = p.y;
            }
    }
    // a row the call does not have: zeros.  An infinity or a NaN: no such codes, but such a scale, and the row's results are NaN
    uint6v term[4];
    auto cut = [&](bool some) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            term[t] = __builtin_amdgcn_cvt_scalef32_pk32_bf6_f16(v, 1.0f);
            if (t < 3) v = (v - __builtin_amdgcn_cvt_scalef32_pk32_f16_bf6(term[t], 1.0f)) * (_Float16)16.0f;   // exact
            if (!some) term[t] = (uint6v){0u, 0u, 0u, 0u, 0u, 0u};
        }
    };
    // lane `row` of k block g: its words; `scale`: the scale byte of term 0
    auto emit = [&](char *dst, uint32_t scale, uint32_t per_term) {
#pragma unroll
        for (int h = 0; h < TPO; ++h) {   // operand rows h RPO + m
            const int row = h * RPO + m;
            uint32_t w[4 * QUADS + 1] = {};
#pragma unroll
            for (int o = 0; o < NT; ++o) {
                const int t = o * TPO + h;
#pragma unroll
                for (int i = 0; i < 6; ++i) w[6 * o + i] = term[t][i];
                w[6 * NT] |= (scale - per_term * t) << 8 * o;
            }
#pragma unroll
            for (int i = 0; i < QUADS; ++i) ((uint4 *)dst)[64 * i + 16 * g + row] = make_uint4(w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]);
            if (rows_words(NT) % 4 == 1) ((uint32_t *)(dst + 1024 * QUADS))[16 * g + row] = w[4 * QUADS];
        }
    };
    cut(have);
    char *const record = P.xt + (size_t)ch * rows_chunk_bytes(NT);
    emit(record, real ? (uint32_t)(127 + 2 - s) : have ? 255u : 127u, real ? 4u : 0u);
    if (lane % (4 * RPO) == 0) rows_flags(P, NT)[ch] = (wide >> lane & (~0ull >> (64 - 4 * RPO))) != 0;
    if (__builtin_expect(wide == 0, 1)) return;

    // What the four terms leave, in four more.  It is no more than the activation's own bits, so exact in fp32 and, brought
    // to where the block's largest remainder lies in [8, 16), in fp16 down to 2^-28 of that.
    float left[32], most = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const half32_t held = __builtin_amdgcn_cvt_scalef32_pk32_f16_bf6(term[t], 1.0f);
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const int rr = i >> 3, hh = i >> 2 & 1, n = i & 3;
            if (t == 0) left[i] = (float)__builtin_bit_cast(_Float16, (uint16_t)(x[n][rr] >> (16 * hh))) * power_of_two(s - rows_weight(rr));
            left[i] -= (float)held[i] * (1.0f / (float)(1 << 4 * t));
            if (t == 3) most = fmaxf(most, fabsf(left[i]));
        }
    }
    const bool some = real && most > 0.f;
    const int up = some ? 3 + 127 - (int)(__builtin_bit_cast(uint32_t, most) >> 23) : 0;
    const float factor = power_of_two(up);
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = (_Float16)(left[i] * factor);
    cut(some);
    emit(record + (size_t)P.nchunks * rows_chunk_bytes(NT), some ? (uint32_t)(127 + 2 - s - up) : 127u, some ? 4u : 0u);
}

template <int Q>
struct RowsRegs {
    uint32_t w[Q][4];      // plane j: the four words (32 k each) of column `lane`
    uint16_t mt[Q + 1];    // scales and zero of column `lane` for the chunk's quant group
};

template <int Q, int G, int NT>
__global__ void __launch_bounds__(512)
hlq_gemm_rows_kernel(const int4v bb_lo, const int4v bb_hi, const int out_f32_flag, const GemvProbs probs)
{
    static_assert(G >= 128, "one quant segment per chunk");
    static_assert(NT == 1 || NT == 2 || NT == 4, "one operand, or two or four chained ones");
    constexpr int MSTR = rows_meta_stride(Q);
    using Regs = RowsRegs<Q>;
    const int W = (int)(blockDim.x >> 6);
    extern __shared__ __attribute__((aligned(256))) char lds[];

    const GemvProb P = probs.p[gemv_problem_of(bb_lo, bb_hi, (int)blockIdx.x)];
    int tg, slice;
    gemv_split_block(P, (int)blockIdx.x - P.blk_begin, tg, slice);

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int KW = P.kw, KSH = P.kw_shift, part = wave & (KW - 1);   // W and KW are powers of two
    const int tile = tg * (W >> KSH) + (wave >> KSH);
    const bool tile_ok = tile < P.ntiles;             // a surplus wavefront gets an empty run
    const int tile_c = tile_ok ? tile : P.ntiles - 1;
    const int M = P.M;
    // this wavefront's run of chunks: the workgroup's K slice is cut into KW near-equal parts
    const int sbeg = min(slice * P.cps, P.nchunks - 1);
    const int send = min(sbeg + P.cps, P.nchunks);
    const int len = send - sbeg;
    const int cbeg = sbeg + ((len * part) >> KSH);
    const int cend = tile_ok ? sbeg + ((len * (part + 1)) >> KSH) : cbeg;

    const int tw = hlq_tile_width(tile_c, P.N);
    const char *tile_base = P.packed + (size_t)tile_c * HLQ_TILE_N * P.col_bytes;
    const int c = lane & 15, g = lane >> 4;
    const uint32_t moff = (uint32_t)(lane < tw ? lane : tw - 1) * 2u;   // clamped column: loads stay in bounds
    const uint32_t woff = moff * 8u;
    char *meta = lds + wave * rows_wave_lds(Q);           // this wavefront's scales [64][MSTR]
    float *red = (float *)(meta + 64 * MSTR);             // and results [16][64] for the sum over the tile's KW runs

    // ---- weights: range-checked loads through a descriptor over [tile start, end of the run's last record) ----
    const uint32_t run_end = tile_ok ? hlq_rec_in_tile(tw, cend, Q, G) : 0u;
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc((void *)tile_base, 0, (int)run_end, 0x00020000);
    auto load_plane = [&](int ch, Regs &R, int j) {
        const uint32_t vo = woff + hlq_rec_in_tile(tw, ch, Q, G);
        const int4v v = __builtin_bit_cast(int4v, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, (int)vo, j * tw * 16, 2));
        R.w[j][0] = v.x; R.w[j][1] = v.y; R.w[j][2] = v.z; R.w[j][3] = v.w;
    };
    auto load_meta = [&](int ch, Regs &R) {
        const int cm = G > 128 ? (ch & ~1) : ch;      // a 256-wide group keeps its scales in its first (even) chunk
        const uint32_t vo = moff + hlq_rec_in_tile(tw, cm, Q, G);
#pragma unroll
        for (int r = 0; r <= Q; ++r) R.mt[r] = __builtin_amdgcn_raw_buffer_load_b16(wrsrc, (int)vo, tw * Q * 16 + r * tw * 2, 0);
    };

    // first loads: the weights of the first two chunks
    Regs R[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int j = 0; j < Q; ++j) load_plane(cbeg + i, R[i], j);
        load_meta(cbeg + i, R[i]);
    }

    // ---- activation operands: made by hlq_rows_split_kernel, this lane's words of every chunk
    struct Ops {
        int8v A[NT];   // of which the instruction reads six registers
        int scale;     // byte o: operand o
    };
    auto load_record = [&](const char *src, Ops &o) {
        int w[4 * rows_quads(NT) + 1];
#pragma unroll
        for (int i = 0; i < rows_quads(NT); ++i) {
            const int4v v = ((const int4v *)src)[64 * i + lane];
            w[4 * i] = v.x; w[4 * i + 1] = v.y; w[4 * i + 2] = v.z; w[4 * i + 3] = v.w;
        }
        if (rows_words(NT) % 4 == 1) w[4 * rows_quads(NT)] = ((const int *)(src + 1024 * rows_quads(NT)))[lane];
#pragma unroll
        for (int t = 0; t < NT; ++t) o.A[t] = (int8v){w[6 * t], w[6 * t + 1], w[6 * t + 2], w[6 * t + 3], w[6 * t + 4], w[6 * t + 5], 0, 0};
        o.scale = w[6 * NT];
    };
    auto load_ops = [&](int ch, Ops &o) {
        const int chx = max(min(ch, cend - 1), sbeg);   // stays inside K also past the end of the run
        load_record(P.xt + (size_t)chx * rows_chunk_bytes(NT), o);
    };
    // scales: lane <-> column to LDS, read back per column block (this lane's column 16 cb + c)
    struct Sc {
        uint32_t m[4][MSTR / 4];
    };
    auto stage_scales = [&](const Regs &Rn, Sc &s) {
#pragma unroll
        for (int r = 0; r <= Q; ++r) ((u16_alias *)(meta + lane * MSTR))[r] = Rn.mt[r];
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int i = 0; i < MSTR / 4; ++i) s.m[cb][i] = ((const u32_alias *)(meta + (16 * cb + c) * MSTR))[i];
    };
    auto scale_of = [](const uint32_t (&m)[MSTR / 4], int i) -> float {
        const half2_t h = __builtin_bit_cast(half2_t, m[i >> 1]);
        return (float)((i & 1) ? h.y : h.x);
    };
    auto expand = [](uint32_t w) -> int8v {   // plane word -> 32 fp4 codes (bit 4p+r -> nibble p of register r)
        return (int8v){(int)(w & 0x11111111u), (int)(w & 0x22222222u), (int)(w & 0x44444444u),
                       (int)((w >> 1) & 0x44444444u), 0, 0, 0, 0};
    };
    const float4v zero4 = {0.f, 0.f, 0.f, 0.f};
    // one matrix-core instruction: operand t of the activations (bf6) and a plane operand (fp4, scale 1)
    auto mfma = [&](auto tc, const Ops &o, const int8v &B, const float4v &d) -> float4v {
        constexpr int t = decltype(tc)::value;
        return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(o.A[t], B, d, 3, 4, t, o.scale, 0, 0x7f7f7f7f);
    };
    // acc[sl][cb]: output (operand row 4 g + sl, column 16 cb + c) -- for NT = 2 still split by term half
    float acc[4][4];
#pragma unroll
    for (int sl = 0; sl < 4; ++sl)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) acc[sl][cb] = 0.f;

    auto transpose = [&](const Regs &R, uint32_t (&wt)[Q][4]) {   // 4 x 4 over (16-lane group, word)
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const uint2v s01 = __builtin_amdgcn_permlane16_swap(R.w[j][0], R.w[j][1], false, false);
            const uint2v s23 = __builtin_amdgcn_permlane16_swap(R.w[j][2], R.w[j][3], false, false);
            const uint2v t02 = __builtin_amdgcn_permlane32_swap(s01.x, s23.x, false, false);
            const uint2v t13 = __builtin_amdgcn_permlane32_swap(s01.y, s23.y, false, false);
            wt[j][0] = t02.x; wt[j][2] = t02.y; wt[j][1] = t13.x; wt[j][3] = t13.y;
        }
    };
    auto apply = [&](const Sc &s, const float4v &d, int cb, int which) {
        const float sc = scale_of(s.m[cb], which);
#pragma unroll
        for (int sl = 0; sl < 4; ++sl) acc[sl][cb] += sc * d[sl];
    };
    const int8v ones = {0x11111111, 0x22222222, 0x44444444, 0x44444444, 0, 0, 0, 0};
    // One chunk: the items (plane j, column block cb) as a software pipeline -- matrix-core chain of item n |
    // expansion of the word of item n + 1, scales applied to the result of item n - 1.  R's planes are reloaded
    // (chunk two ahead) right after their last item; past the end of the slice the range check answers with zeros.
    auto step = [&](Regs &R, const Ops &o, const Sc &s, int ch_reload) {
        constexpr int NI = 4 * Q;
        float4v xs = zero4;   // the chunk's activation sums per row, for the zero points
        unrolled<NT>([&](auto t) { xs = mfma(t, o, ones, xs); });
        uint32_t wt[Q][4];
        transpose(R, wt);
        load_meta(ch_reload, R);             // its scales were staged one chunk ahead
        // Items go through the matrix core two at a time: the chains of a pair are independent, so the second
        // instruction of one never waits for the first of the same chain, and the vector work of the stage (expansion
        // of the next pair's words, scales on the previous pair's results) is dealt out between the matrix-core
        // instructions instead of queueing behind them.
        constexpr int NP = NI / 2;
        int8v B0 = expand(wt[0][0]), B1 = expand(wt[0][1]);
        float4v pA = zero4, pB = zero4;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int pr = 0; pr < NP; ++pr) {
            const int n0 = 2 * pr, n1 = 2 * pr + 1;
            float4v dA = zero4, dB = zero4;
            unrolled<NT>([&](auto t) {
                dA = mfma(t, o, B0, dA);
                dB = mfma(t, o, B1, dB);
            });
            int8v nB0 = B0, nB1 = B1;
            if (pr + 1 < NP) {
                nB0 = expand(wt[(n0 + 2) / 4][(n0 + 2) % 4]);
                nB1 = expand(wt[(n1 + 2) / 4][(n1 + 2) % 4]);
            }
            if (n1 % 4 == 3) load_plane(ch_reload, R, n1 / 4);   // the plane's last item is in this pair
            if (pr >= 1) {
                apply(s, pA, (n0 - 2) % 4, (n0 - 2) / 4);
                apply(s, pB, (n1 - 2) % 4, (n1 - 2) / 4);
            }
            // 2 NT matrix-core instructions, each followed by its share of the stage's vector instructions
#pragma unroll
            for (int i = 0; i < 2 * NT; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, NT == 1 ? 9 : NT == 2 ? 6 : 3, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            pA = dA; pB = dB; B0 = nB0; B1 = nB1;
        }
        apply(s, pA, (NI - 2) % 4, (NI - 2) / 4);
        apply(s, pB, (NI - 1) % 4, (NI - 1) / 4);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) apply(s, xs, cb, Q);
    };

    // ---- chunk loop: no barrier; weights two chunks ahead, activation operands and staged scales one chunk ahead -----
    // which of the run's chunks have a second record: lane l looks at chunk base + l.  Requested ahead of the first operands and
    // made use of in the loop, in name: what is waited for the operands has it arrive, and nothing waits for it behind the loop
    // (4096 x 14336, q = 4, M = 16: 0.9 us)
    auto flag = [&](int base) -> int { return rows_flags(P, NT)[min(base + lane, P.nchunks - 1)]; };
    int first_flags = flag(cbeg);
    Ops oA, oB;
    load_ops(cbeg, oA);
    Sc sc0, sc1;
    stage_scales(R[0], sc0);
    for (int ch = cbeg; ch < cend; ch += 2) {   // two chunks per trip: register sets are named at compile time
        load_ops(ch + 1, oB);
        stage_scales(R[1], sc1);
        step(R[0], oA, sc0, ch + 2);
        asm volatile("" : "+v"(first_flags));
        if (ch + 1 < cend) {
            load_ops(ch + 2, oA);
            stage_scales(R[0], sc0);
            step(R[1], oB, sc1, ch + 3);
        }
    }

    // ---- what the four terms of wide blocks leave: the same products with the second record of the chunks that have one.  Rare, so
    // nothing is arranged for speed.
    auto remainder = [&](int ch) {
        Regs Rw;
#pragma unroll
        for (int j = 0; j < Q; ++j) load_plane(ch, Rw, j);
        load_meta(ch, Rw);
        Ops o;
        load_record(P.xt + (size_t)(P.nchunks + ch) * rows_chunk_bytes(NT), o);
        Sc s;
        stage_scales(Rw, s);
        uint32_t wt[Q][4];
        transpose(Rw, wt);
        auto chain = [&](const int8v &B) {
            float4v d = zero4;
            unrolled<NT>([&](auto t) { d = mfma(t, o, B, d); });
            return d;
        };
#pragma unroll
        for (int j = 0; j <= Q; ++j)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) apply(s, chain(j < Q ? expand(wt[j < Q ? j : 0][cb]) : ones), cb, j);
    };
    uint64_t wide = __ballot(first_flags != 0 && cbeg + lane < cend);
    for (int base = cbeg; base < cend; base += 64) {
        if (base > cbeg) wide = __ballot(flag(base) != 0 && base + lane < cend);
        for (; wide != 0; wide &= wide - 1) remainder(base + __builtin_ctzll(wide));
    }

    // ---- add the terms that lie in different lanes and the tile's KW runs, store --------------------
    float y[4][4];
#pragma unroll
    for (int sl = 0; sl < 4; ++sl) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            float v = acc[sl][cb];
            if (NT == 1) v += __shfl_xor(v, 16);   // one term per 16-lane group
            if (NT <= 2) v += __shfl_xor(v, 32);   // NT = 2: lanes 32..63 hold terms 1, 3 of the same rows
            y[sl][cb] = v;
        }
    }
    if (KW > 1) {
#pragma unroll
        for (int sl = 0; sl < 4; ++sl)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) red[(sl * 4 + cb) * 64 + lane] = y[sl][cb];
        __syncthreads();
        if (part == 0) {
            constexpr int RSTR = rows_wave_lds(Q) / 4;   // floats between wavefronts' blocks
#pragma unroll
            for (int sl = 0; sl < 4; ++sl)
#pragma unroll
                for (int cb = 0; cb < 4; ++cb)
                    for (int w2 = 1; w2 < KW; ++w2) y[sl][cb] += red[w2 * RSTR + (sl * 4 + cb) * 64 + lane];
        }
    }
    if (!tile_ok || part != 0) return;
    if ((NT == 2 && g >= 2) || (NT == 1 && g >= 1)) return;
    const int row0 = (NT == 1 ? 0 : NT == 2 ? 4 * (g & 1) : 4 * g);
    const size_t n0 = (size_t)tile * HLQ_TILE_N;
    const size_t ldy = (size_t)P.ldy;
    const int out_f32 = out_f32_flag;

    if (P.nslices == 1) {
#pragma unroll
        for (int sl = 0; sl < 4; ++sl)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
                if (row0 + sl < M && 16 * cb + c < tw) store_out(P.y, (size_t)(row0 + sl) * ldy + n0 + 16 * cb + c, y[sl][cb], out_f32);
        return;
    }
    // ---- split-K across workgroups: write-through partials [slice][row][N], arrival counter per tile, the last
    // workgroup to arrive adds in slice order
    const size_t MN = (size_t)M * P.N;
#pragma unroll
    for (int sl = 0; sl < 4; ++sl)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
            if (row0 + sl < M && 16 * cb + c < tw)
                __hip_atomic_store(&P.part[(size_t)slice * MN + (size_t)(row0 + sl) * P.N + n0 + 16 * cb + c], y[sl][cb],
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // every lane that stored has its writes acknowledged once the whole wavefront is past the wait above
    int old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(&P.cnt[tile], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    old = __builtin_amdgcn_readfirstlane(old);
    if (old != P.nslices - 1) return;
    // all sixteen outputs of a lane, of four slices, are read before any is added (64 loads in flight); the sums
    // still run in slice order
    {
        float a[4][4];
        const float *src[4][4];
        bool on[4][4];
#pragma unroll
        for (int sl = 0; sl < 4; ++sl)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                a[sl][cb] = 0.f;
                on[sl][cb] = row0 + sl < M && 16 * cb + c < tw;
                // lanes without an output re-read a valid one (row 0 of this tile's first column) and drop it
                src[sl][cb] = &P.part[on[sl][cb] ? (size_t)(row0 + sl) * P.N + n0 + 16 * cb + c : n0];
            }
        for (int s2 = 0; s2 < P.nslices; s2 += 4) {   // four slices per trip; slices past the last re-read it and add zero
            float v[4][4][4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int sl = 0; sl < 4; ++sl)
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb)
                        v[k][sl][cb] = __hip_atomic_load(src[sl][cb] + (size_t)min(s2 + k, P.nslices - 1) * MN, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int sl = 0; sl < 4; ++sl)
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb) a[sl][cb] += s2 + k < P.nslices ? v[k][sl][cb] : 0.f;
        }
#pragma unroll
        for (int sl = 0; sl < 4; ++sl)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
                if (on[sl][cb]) store_out(P.y, (size_t)(row0 + sl) * ldy + n0 + 16 * cb + c, a[sl][cb], out_f32);
    }
    if (lane == 0) __hip_atomic_store(&P.cnt[tile], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int Q, int G>
void launch_qg(const GemvBatch &b, unsigned nblocks, int W, int rows, hipStream_t st)
{
    const dim3 blk(64 * W);
    const GemvKernelArgs a = gemv_kernel_args(b);
    unsigned chunks = 1;
    for (int i = 0; i < b.count; ++i) chunks = (unsigned)b.p[i].nchunks > chunks ? (unsigned)b.p[i].nchunks : chunks;
    if constexpr (G >= 128) {
        auto launch = [&](auto nt) {
            constexpr int NT = decltype(nt)::value, per_wave = 16 / rows_carried(NT);
            hlq_rows_split_kernel<NT><<<dim3((chunks + per_wave - 1) / per_wave, b.count), 64, 0, st>>>(a.probs);
            hlq_gemm_rows_kernel<Q, G, NT><<<nblocks, blk, (size_t)rows_lds_bytes(Q, W), st>>>(a.lo, a.hi, a.out_f32, a.probs);
        };
        switch (rows_operands(rows)) {
        case 1: launch(std::integral_constant<int, 1>{}); break;
        case 2: launch(std::integral_constant<int, 2>{}); break;
        default: launch(std::integral_constant<int, 4>{}); break;
        }
    }
}

template <int Q>
hlq_status launch_q(int G, const GemvBatch &b, unsigned nblocks, int W, int rows, hipStream_t st)
{
    switch (G) {
    case 128: launch_qg<Q, 128>(b, nblocks, W, rows, st); return HLQ_OK;
    case 256: launch_qg<Q, 256>(b, nblocks, W, rows, st); return HLQ_OK;
    }
    return HLQ_ERR_UNSUPPORTED;
}

} // namespace

size_t hlq_gemm_rows_xt_bytes(const HlqDims &dm, int64_t M)
{
    if (M < 1 || M > hlq_gemm_rows_max(dm.G)) return 0;
    const size_t flags = ((size_t)dm.nchunks * sizeof(int) + 255) & ~(size_t)255;
    return (size_t)dm.nchunks * 2 * rows_chunk_bytes(rows_operands((int)M)) + flags + 256;   // kept 256-byte aligned
}

// rows this kernel carries for group size G (0: no instantiation)
int hlq_gemm_rows_max(int G) { return G >= 128 ? 16 : 0; }

hlq_status hlq_launch_gemm_rows(const GemvBatch &b, unsigned nblocks, int W, int rows, int q, int G, hipStream_t st)
{
    if ((W != 2 && W != 4 && W != 8) || rows < 1 || rows > hlq_gemm_rows_max(G)) return HLQ_ERR_UNSUPPORTED;
    switch (q) {
    case 1: return launch_q<1>(G, b, nblocks, W, rows, st);
    case 2: return launch_q<2>(G, b, nblocks, W, rows, st);
    case 3: return launch_q<3>(G, b, nblocks, W, rows, st);
    case 4: return launch_q<4>(G, b, nblocks, W, rows, st);
    }
    return HLQ_ERR_UNSUPPORTED;
}
