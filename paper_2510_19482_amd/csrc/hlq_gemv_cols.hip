// hlq_lut_gemv / hlq_lut_gemv_batch, matrix-core formulation for one activation row, and for two to four (Sec. 2, paragraph
// "Bit-Serial LUT-Based GEMM", and App. B; weights in the format of Eq. 3):
//
//   y[n] = sum_groups ( sum_j s_j[g,n] * <b_j[.,n], x>_g  +  z[g,n] * sum_g(x) )
//
// with the bit-plane dot products <b_j, x> on v_mfma_f32_16x16x128_f8f6f4, planes as fp4 codes and activations as an exact
// sum of four bf8 terms, as hlq_gemv_mx.hip describes them (that kernel serves the launches that the rules in hlq_gemv.hip leave to it).  What is different
// here is what a wavefront owns: 16 columns x a window of 4 chunks (512 k) instead of 64 columns x 1 chunk.
//
//   - Lane c + 16 g loads the 16 bytes of column c in chunk g of the window, so its four words are, as loaded, the plane
//     operands of four matrix-core instructions: instruction i multiplies word i of every lane, lane group g being the
//     matrix core's k block g.  No lane swaps.
//   - The 16 rows of the activation operand are (chunk g, term t): row 4 g + t holds term t of the activations of chunk g
//     in k block g and zeros elsewhere.  The result of lane (c, g) is then column c's four terms for chunk g: the lane
//     that loaded the chunk's scales for that column.  No trip of the scales through LDS, and the four instructions of a
//     quant group of 128 k chain through their accumulator: one scale multiplication per plane and group.
//   - A wavefront keeps its window and walks over columns: the activations are split into terms once per window, the four
//     operands (32 registers) and the groups' activation sums (for the zero points) stay in registers.  Scales are
//     fetched as 16-byte pieces of rows, one or two loads a step instead of one per plane and group, and spread through
//     LDS.
//
// What bounds it: on small launches the fixed trip (arguments, first load, a step, the sum over the wavefronts, store), on
// long ones the stream of weights.  A step (as many weights as a chunk of 64 columns) is 63 vector instructions and 8
// matrix-core ones at q = 2, G = 128, against 75 and 9 of the 64-column form, and a quarter of the width: 4096 x 4096
// is 256 workgroups of eight wavefronts with one trip to memory each, where 64-column tiles made 64 workgroups with two.
// Measured per launch (graph replay, weights from HBM, q = 2, G = 128; 64-column kernel -> this one): 4096 x 1024 4.95 ->
// 3.17 us, 4096 x 4096 5.42 -> 3.53 (q = 4: 7.86 -> 4.15; q = 4, G = 64: 8.85 -> 4.43), 4096 x 6144 5.6 -> 4.3, 14336 x 4096
// 7.95 -> 6.5, 8192 x 8192 7.8 -> 6.1, 8B layer as one launch 13.8 -> 13.1 (65 MB: 4.9 TB/s), 70B layer 42.1 -> 40.9.
// Tried: two register sets (loads two steps ahead) 0.1-0.4 us slower on small launches and up to 10 % on long ones (100 instead
// of 90 registers); 2-byte scale loads 0.2 us slower (q = 4, G = 64: 0.1 per load); the four column blocks of a tile in
// four wavefronts at a time instead of one after the other: no gain on long launches; 80 registers (six wavefronts on a
// SIMD): spills, 10-20 % slower.
//
// Two and four rows (the launches of hlq_gemm_few_wins): every row has four operands of its own, which share the expanded
// plane words.  They are bf6 terms as in hlq_gemm_rows.hip -- 24 registers a row and not 32, 16 clocks an instruction and not
// 32 -- with the matrix core's own scale per word, so the window's largest magnitude is not needed; made of the same
// eight activations per lane, through the packed conversions (at one row their latency, 72 clocks a conversion, is longer than
// what bf8 terms take).  Relative error of fp32 results at 4096 x 4096, q = 4, 4 rows, 1 % outliers: 1.6e-5 -> 4e-6.  What four
// terms leave in wide words (as in hlq_gemm_rows.hip) is added in a second pass of the wavefront over its windows that have one;
// whether one has costs four instructions a row (a count of the small activations instead: 0.3 to 0.6 us of 5 to 9).
//
// Work split.  A workgroup of W wavefronts owns adjacent column blocks and one K slice; the windows of the slice are
// dealt out to the wavefronts, whose results meet in LDS.  K slices of different workgroups meet in the workspace: two
// in an exchange per column, more as in the other GEMV kernels (partial sums, an arrival counter per workgroup column, the
// last one adds in slice order).  Column blocks of one 64-column tile share the cache lines of its scales: neighbouring
// workgroups run on one XCD (they go to the eight XCDs in turn, so the block order is dealt out to match).
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
// the activation codes are written as 64-bit words and read back as 128-bit ones
typedef unsigned int uint2a __attribute__((ext_vector_type(2), may_alias));
typedef uint16_t __attribute__((may_alias)) u16_alias;
typedef uint32_t __attribute__((may_alias)) u32_alias;
typedef int int4a __attribute__((ext_vector_type(4), may_alias));

// NR: activation rows carried (1, 2 or 4)
template <int NR>
struct ColsProbs {
    std::conditional_t<NR == 1, ColsProb, ColsRowsProb> p[HLQ_MAX_BATCH];
};

template <int CTRL, int ROWMASK = 0xf>
__device__ __forceinline__ uint32_t max_dpp(uint32_t v)
{
    const uint32_t moved = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWMASK, 0xf, false);
    return max(v, moved);
}

template <int Q, int G>
struct ColsRegs {
    static constexpr int SEG = G < 128 ? 128 / G : 1;
    uint32_t w[Q][4];          // plane j: the four words (32 k each) of column c in chunk g
    // scales and zeros of the 16 columns, rows of 32 bytes: half a row (16 bytes, 8 columns) per lane, so that a step asks for
    // them in one to three loads instead of one 2-byte load per plane and group; they are spread through LDS
    static constexpr int ROWS = SEG * (Q + 1);           // rows per chunk
    static constexpr int NM = (8 * ROWS + 63) / 64;      // loads
    int4v mt[NM];
};

// LDS per wavefront: activation codes [term][chunk][word][32], the terms 16 bytes apart from a multiple of the bank
// count -- the same bytes hold a step's scales while no operands are being made -- then 128 zero bytes
// (two and four rows: [row][term][chunk][word][24 bytes], and behind the zeros the scales [row][chunk][word])
constexpr uint32_t COLS_WIDE = 8;   // see ROWS_WIDE in hlq_gemm_rows.hip
constexpr int COLS_TERM = 4 * 128 + 16, COLS_CODES = 96;
template <int Q, int G, int NR>
constexpr int cols_zero_at()
{
    constexpr int codes = NR == 1 ? 4 * COLS_TERM : NR * 16 * COLS_CODES, scales = 1024 * ColsRegs<Q, G>::NM;
    return codes > scales ? codes : scales;
}
template <int Q, int G, int NR>
constexpr int cols_wave_lds() { return cols_zero_at<Q, G, NR>() + 128 + 64; }

// wavefronts per workgroup: sixteen, i.e. at most 128 registers; q = 4 with groups of 32 would spill at that, and so would
// the operands of two and four rows
constexpr int cols_max_waves(int q, int G, int NR) { return NR > 1 || (q == 4 && G == 32) ? 8 : 16; }

// ONE: no wavefront of the launch has more than one step (nothing is loaded ahead)
template <int Q, int G, bool ONE, int NR>
__global__ void __launch_bounds__(64 * cols_max_waves(Q, G, NR))
hlq_gemv_cols_kernel(const int4v bb_lo, const int4v bb_hi, const int out_f32, const ColsProbs<NR> probs)
{
    using Regs = ColsRegs<Q, G>;
    constexpr int WAVE_LDS = cols_wave_lds<Q, G, NR>(), ZERO_AT = cols_zero_at<Q, G, NR>();
    constexpr int SEG = Regs::SEG, CHAIN = 4 / SEG;   // words (matrix-core instructions) per quant group of a chunk
    extern __shared__ __attribute__((aligned(256))) char lds[];

    auto P = probs.p[gemv_problem_of(bb_lo, bb_hi, (int)blockIdx.x)];
    asm volatile("" : "+s"(P.slice_magic), "+s"(P.cb_rem));   // with the others, in one burst: not loaded where first used
    const int local = (int)blockIdx.x - P.blk_begin;
    int tg = P.nslices > 1 ? (int)__umulhi((unsigned)local, P.slice_magic) : local;
    const int slice = local - tg * P.nslices;
    {   // neighbours share a tile's cache lines: each XCD (workgroups go to the eight in turn) takes consecutive ones
        const int xcd = tg & 7, each = P.ntg >> 3;
        tg = xcd * each + min(xcd, P.ntg & 7) + (tg >> 3);
    }
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c = lane & 15, g = lane >> 4;

    // KW wavefronts share a column block and deal the slice's windows out among themselves (the first ones take one more);
    // the W / KW streams of a workgroup take consecutive shares of its column blocks
    const int KSH = P.kw_shift, KW = 1 << KSH, W = KW << P.st_shift, part = wave & (KW - 1), stream = wave >> KSH;
    const int sbeg = min(slice * P.cps, P.nchunks - 1);
    const int send = min(sbeg + P.cps, P.nchunks);          // windows end at the slice's end at the latest
    const bool tail = slice == P.nslices - 1;
    const int wbase = tail ? P.wbase_l : P.wbase, wrem = tail ? P.wrem_l : P.wrem;
    const int wbeg = part * wbase + min(part, wrem), wend = wbeg + wbase + (part < wrem ? 1 : 0);
    // column blocks of this workgroup (dealt out like the windows), and of this wavefront's stream
    const int cb0 = tg * P.cb_base + min(tg, P.cb_rem), ncb = P.cb_base + (tg < P.cb_rem ? 1 : 0), cb1 = cb0 + ncb;
    const int spc = (ncb + (1 << P.st_shift) - 1) >> P.st_shift;
    const int s0 = min(cb0 + stream * spc, cb1), s1 = min(s0 + spc, cb1);
    const int steps = (wend - wbeg) * (s1 - s0);
    const int full_cbs = (P.N & 63) ? P.N >> 6 << 2 : 0x7fffffff;   // column blocks in tiles of full width

    char *xt = lds + wave * WAVE_LDS;
    float *red = (float *)(lds + W * WAVE_LDS);             // [column block][part][row][16]

    // ---- loads -----------------------------------------------------------------------------------------------
    // A step's loads go through descriptors that start at the window's first record, at the column block, and end with the
    // slice's last record: what lies past the slice (a window's missing chunks) comes back as zeros without touching
    // memory.  From one column block to the next only the start moves.  Plane words are read once per call:
    // non-temporal; the scales' cache lines are shared by the four column blocks of a tile and keep the default policy.
    auto rec = [&](int w, int ch) { return hlq_rec_in_tile(w, ch, Q, G); };
    // bytes per column from the start of a window to its chunk i (with 256-wide groups windows start at an even chunk)
    auto rel = [](uint32_t i) -> uint32_t {
        return G <= 128 ? __umul24(i, 16 * Q + SEG * (Q + 1) * 2) : __umul24(i, 16 * Q) + __umul24((i + 1) >> 1, (Q + 1) * 2);
    };
    int l_win = wbeg, l_cb = s0;         // what is loaded next
    const char *l_plane, *l_meta;
    int l_size;
    uint32_t vo, vm[Regs::NM];           // lane offsets: its chunk's record and its column; its halves of rows of scales
    int o_plane;                         // byte stride of planes
    auto locate = [&]() {
        const int tile = l_cb >> 2, sub = l_cb & 3, cw = sbeg + 4 * l_win;
        const int tw = hlq_tile_width(tile, P.N);
        const uint32_t r0 = rec(tw, cw);
        const char *first = P.packed + (size_t)tile * P.tile_bytes + r0;
        l_plane = first + sub * 256;
        l_meta = first + sub * 32;
        l_size = (int)(rec(tw, send) - r0);
        // a narrow last tile: columns past its width re-read its last ones and are dropped at the end
        vo = __umul24((uint32_t)tw, rel(g)) + (uint32_t)min(c, tw - 1 - 16 * sub) * 16u;
        const int half = min(8 * (lane & 1), tw - 8 - 16 * sub);
#pragma unroll
        for (int i = 0; i < Regs::NM; ++i) {
            const uint32_t row = 32 * i + (lane >> 1), ch = row / Regs::ROWS, in = row - ch * Regs::ROWS;
            // with 256-wide groups the scales sit in the group's first (even) chunk
            const uint32_t at = __umul24((uint32_t)tw, rel(G > 128 ? ch & ~1u : ch) + 16 * Q + 2 * in) + (uint32_t)half * 2u;
            vm[i] = ch < 4 ? at : 0x7fff0000u;   // no such row: past every range
        }
        o_plane = tw * 16;
    };
    auto advance = [&]() {
        if (++l_cb == s1) {
            l_cb = s0;
            if (++l_win < wend) locate();
            else l_size = 0;   // nothing left: what is asked for now comes back as zeros
        } else if (l_cb >= full_cbs) {   // the narrow last tile
            locate();
        } else {
            const bool same = (l_cb & 3) != 0;
            l_plane += same ? 256 : (size_t)P.tile_bytes - 768;
            l_meta += same ? 32 : (size_t)P.tile_bytes - 96;
        }
    };
    auto load_plane = [&](Regs &R, int j) {
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)l_plane, 0, l_size, 0x00020000);
        const int4v v = __builtin_bit_cast(int4v, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)vo, j * o_plane, 2));   // aux 2: non-temporal
        R.w[j][0] = v.x; R.w[j][1] = v.y; R.w[j][2] = v.z; R.w[j][3] = v.w;
    };
    auto load_meta = [&](Regs &R) {
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)l_meta, 0, l_size, 0x00020000);
#pragma unroll
        for (int i = 0; i < Regs::NM; ++i) R.mt[i] = __builtin_bit_cast(int4v, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)vm[i], 0, 0));
    };
    // activations of a window: lane (chunk g, word i, register r) takes the pairs 32 i + 2 r + 8 m, m = 0..3, which are
    // the eight codes of expansion register r (weight k0 = 8 (n & 3) + 2 r + (n >> 2) is nibble n)
    const int xi = (lane >> 2) & 3, xr = lane & 3;
    uint32_t xw[NR][4];
    auto load_x = [&](int win) {
        const int cw = sbeg + 4 * win;
#pragma unroll
        for (int row = 0; row < NR; ++row) {
            const uint16_t *x = P.x + (size_t)cw * 128;
            if constexpr (NR > 1) x += (size_t)min(row, P.M - 1) * P.ldx;   // (a row more than the call has: dropped at the end)
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)x, 0, (send - cw) * 256, 0x00020000);
#pragma unroll
            for (int m = 0; m < 4; ++m) xw[row][m] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, g * 256 + xi * 64 + xr * 4 + 16 * m, 0, 0);
        }
    };

        Regs R;
    l_size = 0;
    if (steps > 0) {
        load_x(wbeg);      // first out, so first back: the operands are made while the weights arrive
        locate();
        load_meta(R);
#pragma unroll
        for (int j = 0; j < Q; ++j) load_plane(R, j);
        if (!ONE) advance();
    }

    // ---- the window's operands ---------------------------------------------------------------------------------
    // row (lane & 15) = 4 sg + t of the activation operand; its codes sit in k block sg, i.e. in 16-k run g & 1 of the lane
    // groups g with g >> 1 == sg & 1, first half (k below 64) for sg < 2
    const int a_sg = (lane & 15) >> 2, a_t = lane & 3;
    const bool a_on = (g >> 1) == (a_sg & 1);
    const char *a_zero = xt + ZERO_AT, *a_data = xt + a_t * COLS_TERM + a_sg * 128 + 16 * (g & 1);
    const char *a_lo = a_on && a_sg < 2 ? a_data : a_zero, *a_hi = a_on && a_sg >= 2 ? a_data : a_zero;
    if (lane < 8) ((int4a *)(xt + ZERO_AT))[lane] = (int4a){0, 0, 0, 0};
    auto expand = [](uint32_t w) -> int8v {   // plane word -> 32 fp4 codes (bit 4p+r -> nibble p of register r)
        return (int8v){(int)(w & 0x11111111u), (int)(w & 0x22222222u), (int)(w & 0x44444444u),
                       (int)((w >> 1) & 0x44444444u), 0, 0, 0, 0};
    };
    const float4v zero4 = {0.f, 0.f, 0.f, 0.f};
    int8v A[NR][4];       // several rows: six registers of each are used
    int ascale[NR];       // several rows: byte i: the scale of word i
    float xs[NR][SEG], yscale = 0.f;
    // one matrix-core instruction: word i of the activations of a row and a plane operand
    auto mfma = [&](auto ic, int row, const int8v &B, const float4v &d) -> float4v {
        constexpr int i = decltype(ic)::value;
        if constexpr (NR == 1) return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A[0][i], B, d, 1, 4, 0, 0, 0, 0);
        else return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A[row][i], B, d, 3, 4, i, ascale[row], 0, 0x7f7f7f7f);
    };
    auto sum_groups = [&]() {
        const int8v ones = {0x11111111, 0x22222222, 0x44444444, 0x44444444, 0, 0, 0, 0};
#pragma unroll
        for (int row = 0; row < NR; ++row)
            unrolled<SEG>([&](auto sg) {   // activation sums of the quant groups, for the zero points
                float4v d = zero4;
                unrolled<CHAIN>([&](auto i) { d = mfma(std::integral_constant<int, decltype(sg)::value * CHAIN + decltype(i)::value>{}, row, ones, d); });
                xs[row][sg] = (d[0] + d[1]) + (d[2] + d[3]);
            });
    };
    // Several rows: the terms of the many-rows kernel (hlq_gemm_rows.hip), four bf6 codes per activation with one power of two
    // per 32 activations, i.e. per word; a lane makes the eight codes of one expansion register for every row.  LEFT: the same
    // terms of what these four leave.  Returns whether a word is wide
    // (as there): a lane that has activations has only such as are 2^-8 of the word's largest, as weighted.
    auto make_rows = [&](auto left_c) -> bool {
        constexpr bool LEFT = decltype(left_c)::value;
        int mine = lane;
        if constexpr (Q == 4 && G == 32 && NR == 4) asm volatile("" : "+v"(mine));   // what follows from it is made again: no registers are left to keep it in
        const int g = mine >> 4, xi = (mine >> 2) & 3, xr = mine & 3, a_sg = (mine & 15) >> 2, a_t = mine & 3;
        // row (lane & 15) = 4 sg + t holds the codes of chunk sg, which are k block sg: in lane group g == sg
        const char *r_data = g == a_sg ? xt + (a_t * 4 + a_sg) * COLS_CODES : xt + ZERO_AT;
        half32_t v;
        const int weight = xr < 3 ? xr + 1 : 3;
        char *scales = xt + ZERO_AT + 128;
        int s[NR];
        bool odd_row[NR], wide = false;   // an infinity or a NaN
        auto pair = [&](int row, int n) -> half2_t {   // codes 2 n, 2 n + 1: the even activations of the dwords, then the odd ones
            return __builtin_bit_cast(half2_t, __builtin_amdgcn_perm(xw[row][2 * (n & 1) + 1], xw[row][2 * (n & 1)], n < 2 ? 0x05040100u : 0x07060302u));
        };
#pragma unroll
        for (int row = 0; row < NR; ++row) {
            uint32_t mx = 0;
#pragma unroll
            for (int m = 0; m < 4; ++m)
                mx = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, mx), __builtin_bit_cast(ushort2_t, xw[row][m] & 0x7fff7fffu)));
            const uint32_t e = max(mx & 0xffffu, mx >> 16) >> 10;
            // biased exponent of the word's largest weighted magnitude, plus four; an infinity or a NaN beyond all of them
            const uint32_t own = max(e, 1u) - (uint32_t)weight + 4u;
            uint32_t ew = own + (e == 31u ? 256u : 0u);
            ew = max_dpp<0xB1>(ew);          // quad_perm [1,0,3,2]
            ew = max_dpp<0x4E>(ew);          // quad_perm [2,3,0,1]
            odd_row[row] = ew >= 256u;
            wide = wide || (mx != 0u && ew - own - (COLS_WIDE + 1u) < 64u);
            s[row] = 18 + 4 - (int)(ew & 0xffu);
            const int sr = s[row] - weight, k1 = sr / 2, k2 = sr - k1;
            const _Float16 f1 = __builtin_bit_cast(_Float16, (uint16_t)((15 + k1) << 10)), f2 = __builtin_bit_cast(_Float16, (uint16_t)((15 + k2) << 10));
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                const half2_t p = pair(row, n) * (half2_t){f1, f1} * (half2_t){f2, f2};
                v[8 * row + 2 * n] = p.x;
                v[8 * row + 2 * n + 1] = p.y;
                if constexpr (NR == 2) {   // the conversions take 32
                    v[16 + 8 * row + 2 * n] = (_Float16)0.0f;
                    v[16 + 8 * row + 2 * n + 1] = (_Float16)0.0f;
                }
            }
        }
        if constexpr (LEFT) {
            // at most the activation's own bits, so exact in fp32, and in fp16 down to 2^-28 of the largest
            float rest[8 * NR];
#pragma unroll
            for (int row = 0; row < NR; ++row)
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    const half2_t p = pair(row, n);
                    const float f = __builtin_bit_cast(float, (uint32_t)(127 + s[row] - weight) << 23);
                    rest[8 * row + 2 * n] = (float)p.x * f;
                    rest[8 * row + 2 * n + 1] = (float)p.y * f;
                }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const half32_t held = __builtin_amdgcn_cvt_scalef32_pk32_f16_bf6(__builtin_amdgcn_cvt_scalef32_pk32_bf6_f16(v, 1.0f), 1.0f);
                if (t < 3) v = (v - held) * (_Float16)16.0f;
#pragma unroll
                for (int i = 0; i < 8 * NR; ++i) rest[i] -= (float)held[i] * (1.0f / (float)(1 << 4 * t));
            }
#pragma unroll
            for (int row = 0; row < NR; ++row) {
                float most = 0.f;
#pragma unroll
                for (int i = 0; i < 8; ++i) most = fmaxf(most, fabsf(rest[8 * row + i]));
                uint32_t b = __builtin_bit_cast(uint32_t, most);
                b = max_dpp<0xB1>(b);
                b = max_dpp<0x4E>(b);
                const bool some = b != 0u && !odd_row[row];
                const int up = some ? 3 + 127 - (int)(b >> 23) : 0;
                const float f = __builtin_bit_cast(float, (uint32_t)(127 + up) << 23);
#pragma unroll
                for (int i = 0; i < 8; ++i) v[8 * row + i] = some ? (_Float16)(rest[8 * row + i] * f) : (_Float16)0.0f;
                s[row] = some ? s[row] + up : 2;
                odd_row[row] = false;
            }
        }
        if (xr == 0) {
#pragma unroll
            for (int row = 0; row < NR; ++row) ((uint8_t *)scales)[(row * 4 + g) * 4 + xi] = (uint8_t)(odd_row[row] ? 255 : 127 + 2 - s[row]);
        }
        // 48 bits a row and term at byte 6 xr of the word's 24: a 32-bit and a 16-bit store, in this order or the other
        const bool odd = xr & 1;
        char *dst = xt + g * COLS_CODES + xi * 24 + 6 * xr;
        char *dst32 = dst + (odd ? 2 : 0), *dst16 = dst + (odd ? 0 : 4);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint6v c = __builtin_amdgcn_cvt_scalef32_pk32_bf6_f16(v, 1.0f);
            if (t < 3) v = (v - __builtin_amdgcn_cvt_scalef32_pk32_f16_bf6(c, 1.0f)) * (_Float16)16.0f;   // exact
#pragma unroll
            for (int row = 0; row < NR; ++row) {
                const uint32_t w0 = c[3 * row / 2], w1 = c[3 * row / 2 + 1];
                const uint32_t low = row & 1 ? __builtin_amdgcn_alignbit(w1, w0, 16) : w0, high = row & 1 ? w1 >> 16 : w1 & 0xffffu;
                const int at = (row * 4 + t) * 4 * COLS_CODES;
                *(u32_alias *)(dst32 + at) = __builtin_amdgcn_alignbit(high, low, odd ? 16 : 0);
                *(u16_alias *)(dst16 + at) = (uint16_t)(odd ? low : high);
            }
        }
#pragma unroll
        for (int row = 0; row < NR; ++row) {
            int4a q[6];
#pragma unroll
            for (int n = 0; n < 6; ++n) q[n] = *(const int4a *)(r_data + (g == a_sg ? row * 16 * COLS_CODES : 0) + 16 * n);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
                for (int k = 0; k < 6; ++k) A[row][i][k] = q[(6 * i + k) / 4][(6 * i + k) % 4];
                A[row][i][6] = A[row][i][7] = 0;
            }
            // term t is 4 t binary places further down (a NaN scale stays one in term 0); where there are no codes any scale will do
            ascale[row] = g == a_sg ? (int)(((const u32_alias *)scales)[row * 4 + a_sg] - 0x04040404u * a_t) : 0x7f7f7f7f;
        }
        sum_groups();
        return __any(wide);
    };
    auto make_operands = [&]() {
        // largest magnitude of the window -> power-of-two scale (biased fp16 exponent e: |x| < 2^(e-14), scaled by 2^(29-e)
        // below 2^15).  Plane codes are worth 1/2, 1, 2, 2 by register: weights 1/2, 1/4, 1/8, 1/8 make every product
        // bit x activation / 4.  The factor (at most 2^29) is applied as two fp16 multiplications.
        uint32_t mx = 0;
#pragma unroll
        for (int m = 0; m < 4; ++m)
            mx = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, mx), __builtin_bit_cast(ushort2_t, xw[0][m] & 0x7fff7fffu)));
        mx = max(mx & 0xffffu, mx >> 16);
        mx = max_dpp<0xB1>(mx);          // quad_perm [1,0,3,2]
        mx = max_dpp<0x4E>(mx);          // quad_perm [2,3,0,1]
        mx = max_dpp<0x124>(mx);         // row_ror:4
        mx = max_dpp<0x128>(mx);         // row_ror:8: every lane holds its row's maximum
        mx = max_dpp<0x142, 0xa>(mx);    // row_bcast15: rows 1, 3 take rows 0, 2 in
        mx = max_dpp<0x143, 0xc>(mx);    // row_bcast31: row 3 takes row 1 in
        const int e = (int)((uint32_t)__builtin_amdgcn_readlane((int)mx, 63) >> 10);
        const int k1 = (29 - e) / 2, k2 = (29 - e) - k1 - (xr == 0 ? 1 : xr == 1 ? 2 : 3);   // -4 <= k2 <= 14
        const _Float16 f1 = __builtin_bit_cast(_Float16, (uint16_t)((15 + k1) << 10));
        const _Float16 f2 = __builtin_bit_cast(_Float16, (uint16_t)((15 + k2) << 10));
        yscale = __builtin_bit_cast(float, (uint32_t)(127 + 2 - 29 + e) << 23);   // 4 * 2^(e-29)
        half2_t p[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) p[m] = (__builtin_bit_cast(half2_t, xw[0][m]) * (half2_t){f1, f1}) * (half2_t){f2, f2};   // exact
        char *dst = xt + g * 128 + xi * 32 + xr * 8;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            // cut to three significant bits: the high byte of an fp16 is a bf8 code; the remainder is exact, and four
            // terms hold all eleven bits
            uint32_t u[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                u[m] = __builtin_bit_cast(uint32_t, p[m]) & 0xff00ff00u;
                p[m] = p[m] - __builtin_bit_cast(half2_t, u[m]);
            }
            const uint32_t a01 = __builtin_amdgcn_perm(u[1], u[0], 0x07030501u), a23 = __builtin_amdgcn_perm(u[3], u[2], 0x07030501u);
            const uint32_t first = __builtin_amdgcn_perm(a23, a01, 0x05040100u), second = __builtin_amdgcn_perm(a23, a01, 0x07060302u);
            *(uint2a *)(dst + t * COLS_TERM) = (uint2a){first, second};
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int4a lo = *(const int4a *)(a_lo + 32 * i), hi = *(const int4a *)(a_hi + 32 * i);
            A[0][i] = (int8v){lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        }
        sum_groups();
    };

    // ---- steps ---------------------------------------------------------------------------------------------------
    auto scale = [](uint16_t h) -> float { return (float)__builtin_bit_cast(_Float16, h); };
    int win = wbeg, cb = s0;
    bool any_wide = false;   // several rows
    // AHEAD: the next step's loads are requested on the way
    auto step = [&](auto ahead_c, bool more) {
        constexpr bool AHEAD = decltype(ahead_c)::value;
        if (cb == s0 && !more) {
            if constexpr (NR == 1) make_operands();
            else any_wide = make_rows(std::false_type{}) || any_wide;
            if (win + 1 < wend) load_x(win + 1);
        }
        __builtin_amdgcn_sched_barrier(0);   // the operands are made before anything waits for the weights
        float y[NR];
#pragma unroll
        for (int row = 0; row < NR; ++row) y[row] = 0.f;
        uint16_t mt[SEG][Q + 1];
#pragma unroll
        for (int i = 0; i < Regs::NM; ++i) ((int4a *)xt)[64 * i + lane] = R.mt[i];
        if (AHEAD) load_meta(R);
#pragma unroll
        for (int sg = 0; sg < SEG; ++sg) {
#pragma unroll
            for (int r = 0; r <= Q; ++r) mt[sg][r] = ((const u16_alias *)xt)[(g * Regs::ROWS + sg * (Q + 1) + r) * 16 + c];
#pragma unroll
            for (int row = 0; row < NR; ++row) y[row] += scale(mt[sg][Q]) * xs[row][sg];
        }
        constexpr int NI = 4 * Q;   // item n: plane n / 4, word n % 4
        int8v B = expand(R.w[0][0]);
        float4v d[2][NR];
        __builtin_amdgcn_sched_barrier(0);
        auto apply = [&](int done) {
            const float sc = scale(mt[done % SEG][done / SEG]);
#pragma unroll
            for (int row = 0; row < NR; ++row) {
                const float4v &f = d[done & 1][row];
                y[row] += sc * ((f[0] + f[1]) + (f[2] + f[3]));
            }
        };
        unrolled<NI>([&](auto nc) {
            constexpr int n = decltype(nc)::value, chain = n / CHAIN;   // (plane, segment)
#pragma unroll
            for (int row = 0; row < NR; ++row) d[chain & 1][row] = mfma(std::integral_constant<int, n % 4>{}, row, B, n % CHAIN ? d[chain & 1][row] : zero4);
            if constexpr (NR == 1) __builtin_amdgcn_sched_barrier(0);
            if (n + 1 < NI) {
                uint32_t &w = R.w[(n + 1) / 4][(n + 1) % 4];
                asm volatile("" : "+v"(w));   // expanded here and not earlier, where it would hold four more registers
                B = expand(w);
            }
            if (AHEAD && n % 4 == 2) load_plane(R, n / 4);   // the plane's last word has been expanded: the next step's
            if (n >= CHAIN && n % CHAIN == (CHAIN > 1 ? 1 : 0)) apply(chain - 1);
            __builtin_amdgcn_sched_barrier(0);
        });
        apply(NI / CHAIN - 1);
        // the window's four chunks (lane groups)
        auto fold = [](const uint2v &v) -> float {
            const uint32_t own = v.x, other = v.y;
            return __builtin_bit_cast(float, own) + __builtin_bit_cast(float, other);
        };
#pragma unroll
        for (int row = 0; row < NR; ++row) {
            const uint32_t y1 = __builtin_bit_cast(uint32_t, y[row]);
            y[row] = fold(__builtin_amdgcn_permlane32_swap(y1, y1, false, false));
            const uint32_t y2 = __builtin_bit_cast(uint32_t, y[row]);
            y[row] = fold(__builtin_amdgcn_permlane16_swap(y2, y2, false, false));
        }
        if constexpr (NR == 1) {
            y[0] *= yscale;
            float *slot = red + ((cb - cb0) * KW + part) * 16 + c;
            if (lane < 16) {
                if (win > wbeg) y[0] += *slot;
                *slot = y[0];
            }
        } else {   // lane group g stores row g
            float v = g & 1 ? y[1] : y[0];
            if constexpr (NR == 4) v = g & 2 ? (g & 1 ? y[3] : y[2]) : v;
            float *slot = red + (((cb - cb0) * KW + part) * NR + (g & (NR - 1))) * 16 + c;
            if (g < NR) {
                if (win > wbeg || more) v += *slot;
                *slot = v;
            }
        }
        if (AHEAD) advance();
        if (++cb == s1) {
            cb = s0;
            ++win;
        }
    };
    if (steps > 0) {
        for (int s = 0; s < (ONE ? 1 : steps); ++s) step(std::integral_constant<bool, !ONE>{}, false);
        // once more through the windows with wide words, with what the terms leave of them
        if constexpr (NR > 1) {
            if (__builtin_expect(any_wide, 0))
                for (int w = wbeg; w < wend; ++w) {
                    load_x(w);
                    if (!make_rows(std::true_type{})) continue;
                    win = w;
                    for (cb = s0; win == w;) {
                        l_win = w;
                        l_cb = cb;
                        locate();
                        load_meta(R);
#pragma unroll
                        for (int j = 0; j < Q; ++j) load_plane(R, j);
                        step(std::false_type{}, true);
                    }
                }
        }
    } else if (wend == wbeg) {   // no window: nothing to add
        for (int i = lane; i < (s1 - s0) * 16 * NR; i += 64) red[((s0 - cb0 + i / (16 * NR)) * KW + part) * 16 * NR + i % (16 * NR)] = 0.f;
    }
    __syncthreads();

    // ---- add the wavefronts' windows, store ---------------------------------------------------------------------
    const int cols = min(16 * (cb1 - cb0), P.N - 16 * cb0);
    // sum of the wavefronts' windows: column i of the workgroup's, one of the rows
    auto total = [&](int i, int row) -> float {
        float v = 0.f;
        for (int w2 = 0; w2 < KW; ++w2) v += red[(((i >> 4) * KW + w2) * NR + row) * 16 + (i & 15)];
        return v;
    };
    if constexpr (NR > 1) {
        if (P.nslices == 1) {
            for (int row = 0; row < P.M; ++row)
                for (int i = tid; i < cols; i += 64 * W) store_out(P.y, (size_t)row * P.ldy + (size_t)16 * cb0 + i, total(i, row), out_f32);
            return;
        }
        // as for one row below, with a row of partial sums for every row
        if (wave != 0) return;
        const size_t n = (size_t)16 * cb0 + lane;
        if (lane < cols)
            for (int row = 0; row < P.M; ++row)
                __hip_atomic_store(&P.part[((size_t)slice * P.M + row) * P.N + n], total(lane, row), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        int old = 0;
        if (lane == 0) old = __hip_atomic_fetch_add(&P.cnt[tg], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        old = __builtin_amdgcn_readfirstlane(old);
        if (old != P.nslices - 1) return;
        if (lane < cols)
            for (int row = 0; row < P.M; ++row) {
                float a = 0.f;
                for (int sl = 0; sl < P.nslices; ++sl)
                    a += __hip_atomic_load(&P.part[((size_t)sl * P.M + row) * P.N + n], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                store_out(P.y, (size_t)row * P.ldy + n, a, out_f32);
            }
        if (lane == 0) __hip_atomic_store(&P.cnt[tg], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    } else {
    if (P.nslices == 1) {
        for (int i = tid; i < cols; i += 64 * W) store_out(P.y, (size_t)16 * cb0 + i, total(i, 0), out_f32);
        return;
    }
    // K in two slices: every column has a 64-bit slot that is zero between launches.  Each side swaps its sum in, marked in
    // the upper half; who gets a marked value back has both, adds them (in either order the same) and clears the slot.  One
    // trip to device memory, where partial sums and a counter take three.
    if (P.pairs) {
        for (int i = tid; i < cols; i += 64 * W) {
            const float v = total(i, 0);
            unsigned long long *slot = (unsigned long long *)P.cnt + 16 * cb0 + i;
            const unsigned long long mine = 1ull << 32 | __builtin_bit_cast(uint32_t, v);
            const unsigned long long met = __hip_atomic_exchange(slot, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (met >> 32) {
                store_out(P.y, (size_t)16 * cb0 + i, v + __builtin_bit_cast(float, (uint32_t)met), out_f32);
                __hip_atomic_store(slot, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        return;
    }
    // more slices (at most four column blocks a workgroup, so one wavefront does it): write-through partial sums, one
    // arrival counter per workgroup column, the last workgroup to arrive adds in slice order
    if (wave != 0) return;
    const bool col_ok = lane < cols;
    const size_t n = (size_t)16 * cb0 + lane;
    if (col_ok) {
        __hip_atomic_store(&P.part[(size_t)slice * P.N + n], total(lane, 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(&P.cnt[tg], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    old = __builtin_amdgcn_readfirstlane(old);
    if (old != P.nslices - 1) return;
    if (col_ok) {
        const float *src = &P.part[n];
        float a = 0.f;
        int sl = 0;
        for (; sl + 4 <= P.nslices; sl += 4) {
            const float v0 = __hip_atomic_load(src + (size_t)(sl + 0) * P.N, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const float v1 = __hip_atomic_load(src + (size_t)(sl + 1) * P.N, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const float v2 = __hip_atomic_load(src + (size_t)(sl + 2) * P.N, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const float v3 = __hip_atomic_load(src + (size_t)(sl + 3) * P.N, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            a = (((a + v0) + v1) + v2) + v3;
        }
        for (; sl < P.nslices; ++sl) a += __hip_atomic_load(src + (size_t)sl * P.N, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        store_out(P.y, n, a, out_f32);
    }
    if (lane == 0) __hip_atomic_store(&P.cnt[tg], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <int Q, int G, int NR>
void launch_rows(const GemvBatch &b, unsigned nblocks, int W, bool one, int slots, hipStream_t st)
{
    const size_t lds = (size_t)W * cols_wave_lds<Q, G, NR>() + (size_t)slots * 64 * NR;
    const int4v lo = {b.blk_begin[0], b.blk_begin[1], b.blk_begin[2], b.blk_begin[3]};
    const int4v hi = {b.blk_begin[4], b.blk_begin[5], b.blk_begin[6], b.blk_begin[7]};
    ColsProbs<NR> probs;
    for (int i = 0; i < HLQ_MAX_BATCH; ++i) {
        (ColsProb &)probs.p[i] = b.cp[i];
        if constexpr (NR > 1) {
            probs.p[i].M = b.p[i].M;
            probs.p[i].ldx = b.p[i].ldx;
            probs.p[i].ldy = b.p[i].ldy;
        }
    }
    if (one) hlq_gemv_cols_kernel<Q, G, true, NR><<<nblocks, 64 * W, lds, st>>>(lo, hi, b.out_f32, probs);
    else hlq_gemv_cols_kernel<Q, G, false, NR><<<nblocks, 64 * W, lds, st>>>(lo, hi, b.out_f32, probs);
}

template <int Q, int G>
void launch_qg(const GemvBatch &b, unsigned nblocks, int W, int rows, bool one, int slots, hipStream_t st)
{
    if (rows == 1) launch_rows<Q, G, 1>(b, nblocks, W, one, slots, st);
    else if (rows == 2) launch_rows<Q, G, 2>(b, nblocks, W, one, slots, st);
    else launch_rows<Q, G, 4>(b, nblocks, W, one, slots, st);
}

template <int Q>
hlq_status launch_q(int G, const GemvBatch &b, unsigned nblocks, int W, int rows, bool one, int slots, hipStream_t st)
{
    switch (G) {
    case 32: launch_qg<Q, 32>(b, nblocks, W, rows, one, slots, st); return HLQ_OK;
    case 64: launch_qg<Q, 64>(b, nblocks, W, rows, one, slots, st); return HLQ_OK;
    case 128: launch_qg<Q, 128>(b, nblocks, W, rows, one, slots, st); return HLQ_OK;
    case 256: launch_qg<Q, 256>(b, nblocks, W, rows, one, slots, st); return HLQ_OK;
    }
    return HLQ_ERR_UNSUPPORTED;
}

} // namespace

int hlq_gemv_cols_max_waves(int q, int G, int rows) { return cols_max_waves(q, G, rows); }

hlq_status hlq_launch_gemv_cols(const GemvBatch &b, unsigned nblocks, int W, int rows, int q, int G, hipStream_t st)
{
    if (rows < 1 || rows > HLQ_COLS_ROWS || W < 1 || W > cols_max_waves(q, G, rows)) return HLQ_ERR_UNSUPPORTED;
    bool one = true;
    int slots = 1;   // (column block, part) pairs a workgroup keeps results of
    for (int i = 0; i < b.count; ++i) {
        const ColsProb &p = b.cp[i];
        const int ncb = p.cb_base + (p.cb_rem > 0), streams = 1 << p.st_shift;
        slots = (ncb << p.kw_shift) > slots ? ncb << p.kw_shift : slots;
        one = one && ncb <= streams && p.wbase + (p.wrem > 0) <= 1 && p.wbase_l + (p.wrem_l > 0) <= 1;
    }
    if (slots > HLQ_COLS_MAX_SLOTS) return HLQ_ERR_UNSUPPORTED;
    switch (q) {
    case 1: return launch_q<1>(G, b, nblocks, W, rows, one, slots, st);
    case 2: return launch_q<2>(G, b, nblocks, W, rows, one, slots, st);
    case 3: return launch_q<3>(G, b, nblocks, W, rows, one, slots, st);
    case 4: return launch_q<4>(G, b, nblocks, W, rows, one, slots, st);
    }
    return HLQ_ERR_UNSUPPORTED;
}
