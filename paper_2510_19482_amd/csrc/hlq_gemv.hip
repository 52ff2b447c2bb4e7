// hlq_lut_gemv, table-lookup formulation: M = 1 bit-serial LUT GEMV (Sec. 2 "Bit-Serial LUT-Based
// GEMM", App. B), one launch for one or several independent GEMVs; plus the host side (launch
// plans, grouped launches) of both GEMV formulations -- the matrix-core kernel is in hlq_gemv_mx.hip.
//
// Work split.  The unit of work is a wavefront: it owns TN adjacent column tiles (64 columns
// each, lane <-> column) and a run of consecutive chunks (128 k each), i.e. TN contiguous byte
// streams of the packed blob.  Per chunk it
//
//   build    makes its OWN 32 tables in LDS (T[t][i] = sum_r bit_r(i) x_r over the four even or
//            four odd activations of one 8-k window, App. B; fp32 entries): each lane loads its
//            8-k window (quad of lanes <-> window), takes the even or the odd four and stores
//            entries 0..7 or 8..15 of that table with two 128-bit LDS writes; the per-quant-group
//            activation sums come from a DPP reduction of exact fp32 dot products;
//   consume  per plane and 4-bit slice one LDS lookup + one fp32 add; per (plane, quant group)
//            one FMA with s_j; per quant group one FMA  z * sum(x)       (Eq. 3 by linearity).
//
// All lanes of the wavefront index the same 16-entry table at the same time: its entries lie in
// different LDS banks and equal addresses broadcast, so lookups are conflict-free by
// construction.  Because tables are private to the wavefront and LDS operations of one
// wavefront execute in order, the chunk loop has no barrier at all; the weight loads of the next
// NBUF-1 chunks are in flight while a chunk is consumed (NBUF register sets).
//
// The W wavefronts of a workgroup take W consecutive K ranges of the SAME tiles and add their
// results through LDS.  If K is also split across workgroups ("slices"), each workgroup writes
// its partial sums to the workspace and bumps an arrival counter; the last one to arrive adds
// the partials in slice order, so the result does not depend on arrival order.
#include <stdlib.h>

#include <atomic>

#include "hlq_gemv_common.h"

namespace {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

// v + (v moved across lanes by DPP control CTRL), rows outside ROWMASK unchanged
template <int CTRL, int ROWMASK = 0xf>
__device__ __forceinline__ float add_dpp(float v)
{
    const int moved = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWMASK, 0xf, false);
    return v + __builtin_bit_cast(float, moved);
}

__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

template <int Q, int G, int TN>
struct ChunkRegs {
    static constexpr int GS = G < 128 ? G : 128;   // k covered by one scale inside a chunk
    static constexpr int SEG = 128 / GS;           // scale segments per chunk
    uint32_t w[TN][Q][4];
    uint16_t mt[TN][SEG][Q + 1];
    uint4 x;                                       // this lane's 8-k activation window (table build)
};

// ---- hand-scheduled lookup blocks -----------------------------------------------------------------
// One block serves NW consecutive 32-bit plane words (8 * NW lookups) of one (plane, quant
// segment).  For 4-bit slice i of a word the LDS byte address is  base + 64*table + 4*slice.
// Per word: two shifts put slice*4 into bits [5:2] of a byte ((w << 2) for even slices, (w >> 2)
// for odd ones); one sub-dword AND per slice picks that byte, masks it with 0x3c and writes it
// into byte 0 of an address register whose upper bytes keep the wavefront's 256-aligned table
// base; one ds_read_b32 (table number in the immediate offset) fetches the entry; one v_add_f32
// accumulates it: 2.25 VALU ops per lookup.  The LDS reads of word k+1 are issued before the
// adds of word k.  The block drains the LDS queue on entry, so its own lgkmcnt arithmetic is
// exact, and on exit, so every output is valid for the compiler.
// (fp16 entries fetched pairwise into the halves of one register would save adds, but on this
// part 16-bit LDS loads clear the other half of their destination, so the pairing is lost.)
#define HLQ_LK1(R, AD, SRC, BYTE, T)                                                                          \
    "v_and_b32_sdwa " AD ", " SRC ", 60 dst_sel:BYTE_0 dst_unused:UNUSED_PRESERVE src0_sel:BYTE_" #BYTE        \
    " src1_sel:DWORD\n"                                                                                        \
    "ds_read_b32 " R ", " AD " offset:%[off]+" #T "*64\n"
#define HLQ_LK_WORD(W, S, T0, T1, T2, T3, T4, T5, T6, T7)                                                     \
    "v_lshlrev_b32 %[sa], 2, " W "\n"                                                                         \
    "v_lshrrev_b32 %[sb], 2, " W "\n"                                                                         \
    HLQ_LK1("%[" S "0]", "%[d0]", "%[sa]", 0, T0) HLQ_LK1("%[" S "1]", "%[d1]", "%[sb]", 0, T1)               \
    HLQ_LK1("%[" S "2]", "%[d2]", "%[sa]", 1, T2) HLQ_LK1("%[" S "3]", "%[d3]", "%[sb]", 1, T3)               \
    HLQ_LK1("%[" S "4]", "%[d0]", "%[sa]", 2, T4) HLQ_LK1("%[" S "5]", "%[d1]", "%[sb]", 2, T5)               \
    HLQ_LK1("%[" S "6]", "%[d2]", "%[sa]", 3, T6) HLQ_LK1("%[" S "7]", "%[d3]", "%[sb]", 3, T7)
#define HLQ_LK_ADD(S)                                                                                         \
    "v_add_f32 %[p0], %[p0], %[" S "0]\n" "v_add_f32 %[p1], %[p1], %[" S "1]\n"                               \
    "v_add_f32 %[p0], %[p0], %[" S "2]\n" "v_add_f32 %[p1], %[p1], %[" S "3]\n"                               \
    "v_add_f32 %[p0], %[p0], %[" S "4]\n" "v_add_f32 %[p1], %[p1], %[" S "5]\n"                               \
    "v_add_f32 %[p0], %[p0], %[" S "6]\n" "v_add_f32 %[p1], %[p1], %[" S "7]\n"
#define HLQ_LK_OUTS                                                                                           \
    [p0] "+v"(p0), [p1] "+v"(p1), [d0] "+v"(ad[0]), [d1] "+v"(ad[1]), [d2] "+v"(ad[2]), [d3] "+v"(ad[3]),      \
        [sa] "=&v"(sa), [sb] "=&v"(sb), [a0] "=&v"(a0), [a1] "=&v"(a1), [a2] "=&v"(a2), [a3] "=&v"(a3),        \
        [a4] "=&v"(a4), [a5] "=&v"(a5), [a6] "=&v"(a6), [a7] "=&v"(a7)
#define HLQ_LK_OUTS_B                                                                                         \
    , [b0] "=&v"(b0), [b1] "=&v"(b1), [b2] "=&v"(b2), [b3] "=&v"(b3), [b4] "=&v"(b4), [b5] "=&v"(b5),          \
        [b6] "=&v"(b6), [b7] "=&v"(b7)

// `ad`: four address registers holding the wavefront's table base (a multiple of 256) in
// bytes 1..3; OFF: byte offset of the block's first table from that base.
template <int OFF>
__device__ __forceinline__ void lookup_words(const uint32_t (&w)[4], uint32_t (&ad)[4], float &p0, float &p1)
{
    uint32_t sa, sb;
    float a0, a1, a2, a3, a4, a5, a6, a7, b0, b1, b2, b3, b4, b5, b6, b7;
    asm volatile("s_waitcnt lgkmcnt(0)\n"
                 HLQ_LK_WORD("%[w0]", "a", 0, 1, 2, 3, 4, 5, 6, 7)
                 HLQ_LK_WORD("%[w1]", "b", 8, 9, 10, 11, 12, 13, 14, 15)
                 "s_waitcnt lgkmcnt(8)\n"
                 HLQ_LK_ADD("a")
                 HLQ_LK_WORD("%[w2]", "a", 16, 17, 18, 19, 20, 21, 22, 23)
                 "s_waitcnt lgkmcnt(8)\n"
                 HLQ_LK_ADD("b")
                 HLQ_LK_WORD("%[w3]", "b", 24, 25, 26, 27, 28, 29, 30, 31)
                 "s_waitcnt lgkmcnt(8)\n"
                 HLQ_LK_ADD("a")
                 "s_waitcnt lgkmcnt(0)\n"
                 HLQ_LK_ADD("b")
                 : HLQ_LK_OUTS HLQ_LK_OUTS_B
                 : [w0] "v"(w[0]), [w1] "v"(w[1]), [w2] "v"(w[2]), [w3] "v"(w[3]), [off] "n"(OFF)
                 : "memory");
}

template <int OFF>
__device__ __forceinline__ void lookup_words(const uint32_t (&w)[2], uint32_t (&ad)[4], float &p0, float &p1)
{
    uint32_t sa, sb;
    float a0, a1, a2, a3, a4, a5, a6, a7, b0, b1, b2, b3, b4, b5, b6, b7;
    asm volatile("s_waitcnt lgkmcnt(0)\n"
                 HLQ_LK_WORD("%[w0]", "a", 0, 1, 2, 3, 4, 5, 6, 7)
                 HLQ_LK_WORD("%[w1]", "b", 8, 9, 10, 11, 12, 13, 14, 15)
                 "s_waitcnt lgkmcnt(8)\n"
                 HLQ_LK_ADD("a")
                 "s_waitcnt lgkmcnt(0)\n"
                 HLQ_LK_ADD("b")
                 : HLQ_LK_OUTS HLQ_LK_OUTS_B
                 : [w0] "v"(w[0]), [w1] "v"(w[1]), [off] "n"(OFF)
                 : "memory");
}

template <int OFF>
__device__ __forceinline__ void lookup_words(const uint32_t (&w)[1], uint32_t (&ad)[4], float &p0, float &p1)
{
    uint32_t sa, sb;
    float a0, a1, a2, a3, a4, a5, a6, a7;
    asm volatile("s_waitcnt lgkmcnt(0)\n"
                 HLQ_LK_WORD("%[w0]", "a", 0, 1, 2, 3, 4, 5, 6, 7)
                 "s_waitcnt lgkmcnt(0)\n"
                 HLQ_LK_ADD("a")
                 : HLQ_LK_OUTS
                 : [w0] "v"(w[0]), [off] "n"(OFF)
                 : "memory");
}

// All lookups of one chunk, then scales and zeros: compile-time recursion over (tile tn,
// segment sg, plane j) so that every LDS offset is an immediate.  xs[sg] = sum of the
// segment's activations.
template <int Q, int G, int TN, int I = 0>
struct Consume {
    using Regs = ChunkRegs<Q, G, TN>;
    static constexpr int SEG = Regs::SEG, WPS = Regs::GS / 32;
    static constexpr int tn = I / (SEG * Q), sg = (I / Q) % SEG, j = I % Q;
    __device__ __forceinline__ static void run(const Regs &R, const float (&xs)[SEG], uint32_t (&ad)[4],
                                               float (&acc)[TN])
    {
        uint32_t w[WPS];
#pragma unroll
        for (int d = 0; d < WPS; ++d) w[d] = R.w[tn][j][sg * WPS + d];
        float p0 = 0.f, p1 = 0.f;
        lookup_words<sg * WPS * 8 * 64>(w, ad, p0, p1);
        acc[tn] += h2f(R.mt[tn][sg][j]) * (p0 + p1);
        if (j == Q - 1) acc[tn] += h2f(R.mt[tn][sg][Q]) * xs[sg];
        Consume<Q, G, TN, I + 1>::run(R, xs, ad, acc);
    }
};
template <int Q, int G, int TN>
struct Consume<Q, G, TN, TN *(128 / (G < 128 ? G : 128)) * Q> {
    __device__ __forceinline__ static void run(const ChunkRegs<Q, G, TN> &, const float (&)[128 / (G < 128 ? G : 128)],
                                               uint32_t (&)[4], float (&)[TN]) {}
};

#ifndef HLQ_DEBUG_MODE
#define HLQ_DEBUG_MODE 0   // 1: loads only (no lookups), 2: lookups only (no reloads) -- timing experiments
#endif
#define HLQ_GEMV_TABLE_BYTES 2048   // 32 tables x 16 entries x fp32, per wavefront

// Register budget: two chunks of planes and scales are live at once.  A 1024-lane workgroup
// leaves 128 VGPRs per lane; the heaviest shapes (many planes and many small quant groups)
// need more and are limited to 512 lanes (8 wavefronts) per workgroup.
constexpr int gemv_weight(int Q, int G, int TN) { return TN * Q * (G < 128 ? 128 / G : 1); }
constexpr int gemv_max_threads(int Q, int G, int TN) { return gemv_weight(Q, G, TN) <= 12 ? 1024 : 512; }
constexpr bool gemv_two_tiles_ok(int Q, int G) { return gemv_weight(Q, G, 2) <= 6; }
// register sets (chunks in flight + 1): deeper where a set is small
constexpr int gemv_nbuf(int Q, int G, int TN) { return gemv_weight(Q, G, TN) <= 2 ? 4 : gemv_weight(Q, G, TN) <= 4 ? 3 : 2; }

template <int Q, int G, int TN>
__global__ void __launch_bounds__(gemv_max_threads(Q, G, TN))
hlq_gemv_kernel(const int4v bb_lo, const int4v bb_hi, const int out_f32_flag, const GemvProbs probs)
{
    struct { int out_f32; } b = {out_f32_flag};
    using Regs = ChunkRegs<Q, G, TN>;
    constexpr int GS = Regs::GS, SEG = Regs::SEG;
    constexpr int NBUF = gemv_nbuf(Q, G, TN);
    const int W = (int)(blockDim.x >> 6);   // wavefronts per workgroup
    // LDS (dynamic segment only): [W][32 tables][16] fp32 | reduction scratch [W-1][TN][64] fp32
    extern __shared__ __attribute__((aligned(256))) float lds[];
    float *red = lds + W * (HLQ_GEMV_TABLE_BYTES / 4);

    // ---- which problem, which column tile group, which K slice ---------------------------------
    const GemvProb P = probs.p[gemv_problem_of(bb_lo, bb_hi, (int)blockIdx.x)];   // a copy: one burst of scalar loads
    int tg, slice;
    gemv_split_block(P, (int)blockIdx.x - P.blk_begin, tg, slice);

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    // this wavefront's run of chunks: the slice is cut into W near-equal parts
    // (the host plans every slice to start inside K; the clamp keeps every address inside the tile and x)
    const int sbeg = min(slice * P.cps, P.nchunks - 1);
    const int send = min(sbeg + P.cps, P.nchunks);
    const int len = send - sbeg;
    const int cbeg = sbeg + (len * wave) / W;
    const int cend = sbeg + (len * (wave + 1)) / W;

    // per tile: width, validity, clamped lane (loads stay in bounds; results of invalid lanes and
    // tiles are dropped), stream base
    int tw[TN], lane_c[TN];
    bool col_ok[TN];
    const char *tile_base[TN];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        const int tile = tg * TN + tn;
        const int tile_c = tile < P.ntiles ? tile : P.ntiles - 1;
        tw[tn] = hlq_tile_width(tile_c, P.N);
        col_ok[tn] = tile < P.ntiles && lane < tw[tn];
        lane_c[tn] = lane < tw[tn] ? lane : tw[tn] - 1;
        tile_base[tn] = P.packed + (size_t)tile_c * HLQ_TILE_N * P.col_bytes;
    }

    // table-build role of this lane: 8-k window bw of the chunk, parity bp (even / odd k of the
    // window, i.e. the table of word bw/4, 4-bit slice (bw & 3) + 4*bp), entries 8*bh .. 8*bh+7
    const int bw = lane >> 2, bp = (lane >> 1) & 1, bh = lane & 1;
    const int bt = 8 * (bw >> 2) + (bw & 3) + 4 * bp;
    char *Tw = (char *)lds + wave * HLQ_GEMV_TABLE_BYTES;
    // LDS byte address of this wavefront's tables, a multiple of 256
    const uint32_t tbase = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)Tw;
    uint32_t ad[4] = {tbase, tbase, tbase, tbase};

    auto load_chunk = [&](int c, Regs &R) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const int w_ = tw[tn];
            const char *rec = tile_base[tn] + hlq_rec_in_tile(w_, c, Q, G);
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                // default cache policy: non-temporal loads, which help the matrix-core kernel, cost this one 2 us per layer
                const int4v v = *((const int4v *)rec + (j * w_ + lane_c[tn]));
                R.w[tn][j][0] = v.x; R.w[tn][j][1] = v.y; R.w[tn][j][2] = v.z; R.w[tn][j][3] = v.w;
            }
            const char *mrec = rec;
            if (G > 128) {   // the group's meta sits in the record of its first (even) chunk
                const int c0 = c & ~1;
                mrec = tile_base[tn] + hlq_rec_in_tile(w_, c0, Q, G);
            }
            const uint16_t *m = (const uint16_t *)(mrec + (size_t)w_ * Q * 16);
#pragma unroll
            for (int sg = 0; sg < SEG; ++sg)
#pragma unroll
                for (int r = 0; r <= Q; ++r) R.mt[tn][sg][r] = m[(sg * (Q + 1) + r) * w_ + lane_c[tn]];
        }
        R.x = *(const uint4 *)(P.x + (size_t)c * 128 + 8 * bw);
    };

    float acc[TN];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) acc[tn] = 0.f;

    auto step = [&](const Regs &R) {
        // build: entries 8h .. 8h+7 of table bt;  entry i = sum_r bit_r(i) x_r  (fp32), where
        // x_r is the r-th even (bp = 0) or odd (bp = 1) activation of the window
        const uint32_t xd[4] = {R.x.x, R.x.y, R.x.z, R.x.w};
        float xv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            xv[r] = (float)__builtin_bit_cast(_Float16, (uint16_t)(xd[r] >> (16 * bp)));
        const float e0 = bh ? xv[3] : 0.f;
        const float e1 = e0 + xv[0], e2 = e0 + xv[1], e3 = e1 + xv[1];
        float4 *dst = (float4 *)(Tw + bt * 64 + bh * 32);
        dst[0] = make_float4(e0, e1, e2, e3);
        dst[1] = make_float4(e0 + xv[2], e1 + xv[2], e2 + xv[2], e3 + xv[2]);
        // sums of the segments' activations: exact fp32 dot products of the window with (1, 1)
        // (the four lanes of a quad share a window), then a DPP reduction over the four windows
        // (32 k) of a 16-lane row and, for larger groups, over rows
        const half2_t ones = {(_Float16)1.0f, (_Float16)1.0f};
        float tot = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) tot = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, xd[r]), ones, tot, false);
        tot = add_dpp<0x124>(tot);   // row_ror:4
        tot = add_dpp<0x128>(tot);   // row_ror:8   -> every lane holds its row's 32-k sum
        float xs[SEG];
        if (GS == 32) {
#pragma unroll
            for (int sg = 0; sg < SEG; ++sg) xs[sg] = lane_value(tot, 16 * sg);
        } else if (GS == 64) {
            tot = add_dpp<0x142, 0xa>(tot);   // row_bcast15: rows 1, 3 += rows 0, 2
            xs[0] = lane_value(tot, 31);
            xs[SEG - 1] = lane_value(tot, 63);
        } else {
            tot = add_dpp<0x142, 0xa>(tot);
            tot = add_dpp<0x143, 0xc>(tot);   // row_bcast31: rows 2, 3 += row 1
            xs[0] = lane_value(tot, 63);
        }
        if (HLQ_DEBUG_MODE == 1) {
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                uint32_t m = 0;
#pragma unroll
                for (int j = 0; j < Q; ++j) m ^= R.w[tn][j][0] ^ R.w[tn][j][1] ^ R.w[tn][j][2] ^ R.w[tn][j][3];
                acc[tn] += (float)m * h2f(R.mt[tn][0][0]) + xs[0];
            }
        } else {
            Consume<Q, G, TN>::run(R, xs, ad, acc);
        }
    };

    // ---- chunk loop: NBUF register sets, loads of the next NBUF-1 chunks in flight ----------------------
    // A register set is reloaded only while the run has a further chunk for it (the branch sits between
    // steps, not inside one).
    if (cbeg < cend) {
        Regs R[NBUF];
#pragma unroll
        for (int i = 0; i < NBUF; ++i) load_chunk(min(cbeg + i, cend - 1), R[i]);
        for (int c = cbeg; c < cend; c += NBUF) {
#pragma unroll
            for (int i = 0; i < NBUF; ++i) {
                if (c + i < cend) step(R[i]);
                if (HLQ_DEBUG_MODE != 2 && c + i + NBUF < cend) load_chunk(c + i + NBUF, R[i]);
            }
        }
    }

    // ---- add the W wavefronts' K ranges ------------------------------------------------------------------
    if (wave > 0) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) red[((wave - 1) * TN + tn) * 64 + lane] = acc[tn];
    }
    __syncthreads();
    if (wave > 0) return;
    for (int w2 = 1; w2 < W; ++w2) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) acc[tn] += red[((w2 - 1) * TN + tn) * 64 + lane];
    }

    if (P.nslices == 1) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
            if (col_ok[tn]) store_out(P.y, (size_t)(tg * TN + tn) * HLQ_TILE_N + lane, acc[tn], b.out_f32);
        return;
    }
    // ---- split-K across workgroups -----------------------------------------------------------------------
    // Partial sums and the counter live at device scope: the stores below write through the
    // XCD-local L2, the wavefront waits for their acknowledgement, and only then is the arrival
    // counted.  The last workgroup reads the partials with device-scope loads, which bypass its
    // own L2.  No cache-wide write-back or invalidate (as a device-scope fence would issue) is
    // needed, and none is used: it costs tens of microseconds per launch on this part.
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
        if (col_ok[tn])
            __hip_atomic_store(&P.part[(size_t)slice * P.N + (size_t)(tg * TN + tn) * HLQ_TILE_N + lane], acc[tn],
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(&P.cnt[tg], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    old = __builtin_amdgcn_readfirstlane(old);
    if (old != P.nslices - 1) return;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        if (!col_ok[tn]) continue;
        const size_t n = (size_t)(tg * TN + tn) * HLQ_TILE_N + lane;
        float a = 0.f;
        int sl = 0;
        for (; sl + 4 <= P.nslices; sl += 4) {   // four independent loads in flight, added in slice order
            const float v0 = __hip_atomic_load(&P.part[(size_t)(sl + 0) * P.N + n], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const float v1 = __hip_atomic_load(&P.part[(size_t)(sl + 1) * P.N + n], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const float v2 = __hip_atomic_load(&P.part[(size_t)(sl + 2) * P.N + n], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const float v3 = __hip_atomic_load(&P.part[(size_t)(sl + 3) * P.N + n], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            a = (((a + v0) + v1) + v2) + v3;
        }
        for (; sl < P.nslices; ++sl)
            a += __hip_atomic_load(&P.part[(size_t)sl * P.N + n], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        store_out(P.y, n, a, b.out_f32);
    }
    if (lane == 0) __hip_atomic_store(&P.cnt[tg], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void __launch_bounds__(256) hlq_ws_init_kernel(int *p, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0;
}

size_t gemv_lds_bytes(int W, int TN) { return (size_t)W * HLQ_GEMV_TABLE_BYTES + (size_t)(W - 1) * TN * 64 * 4; }

template <int Q, int G>
void launch_qg(const GemvBatch &b, unsigned nblocks, int W, int TN, hipStream_t st)
{
    const dim3 blk(64 * W);
    const GemvKernelArgs a = gemv_kernel_args(b);
    if (TN == 2) {
        if constexpr (gemv_two_tiles_ok(Q, G))
            hlq_gemv_kernel<Q, G, 2><<<nblocks, blk, gemv_lds_bytes(W, 2), st>>>(a.lo, a.hi, a.out_f32, a.probs);
    } else {
        hlq_gemv_kernel<Q, G, 1><<<nblocks, blk, gemv_lds_bytes(W, 1), st>>>(a.lo, a.hi, a.out_f32, a.probs);
    }
}

template <int Q>
hlq_status launch_q(int G, const GemvBatch &b, unsigned nblocks, int W, int TN, hipStream_t st)
{
    switch (G) {
    case 32: launch_qg<Q, 32>(b, nblocks, W, TN, st); return HLQ_OK;
    case 64: launch_qg<Q, 64>(b, nblocks, W, TN, st); return HLQ_OK;
    case 128: launch_qg<Q, 128>(b, nblocks, W, TN, st); return HLQ_OK;
    case 256: launch_qg<Q, 256>(b, nblocks, W, TN, st); return HLQ_OK;
    }
    return HLQ_ERR_UNSUPPORTED;
}

int env_int(const char *name, int dflt)
{
    const char *v = getenv(name);
    return v && *v ? atoi(v) : dflt;
}

// Launch shape for a batch holding `units` (tile, chunk) pairs in total.
struct GemvPlan {
    int TN;    // column tiles per wavefront (1 or 2)
    int W;     // wavefronts per workgroup (K ranges added through LDS)
    int cpw;   // target chunks per wavefront; a slice is W * cpw chunks (rounded to even)
    int forced_w, forced_cpw;   // of these, what hlq_set_gemv_plan or the environment asks for (0: nothing)
};

// process-wide overrides set by hlq_set_gemv_plan (0 = automatic).  Atomic, so that a launch on one
// thread reads a whole value while another thread sets a knob; a launch that overlaps a change of the
// three plan values may still see some old and some new ones (each combination is a valid plan).
std::atomic<int> g_plan_tn{0}, g_plan_w{0}, g_plan_cpw{0};
// formulation: 0 automatic, 1 table lookup, 2 matrix core (hlq_set_gemv_path)
std::atomic<int> g_gemv_path{0};

bool use_mx()
{
    static const int env_path = env_int("HLQ_GEMV_PATH", 0);
    const int knob = g_gemv_path.load(std::memory_order_relaxed);
    const int path = knob ? knob : env_path;
    return path == 0 || path == 2;   // automatic: the matrix-core kernel is the faster one on every measured shape
}

// table-storage variant of the lookup formulation (hlq_gemv_variants.hip): -1 = none (the hand-scheduled kernel)
int table_variant()
{
    const int knob = g_gemv_path.load(std::memory_order_relaxed);
    return knob >= 3 ? knob - 3 : -1;
}

GemvPlan plan_gemv(long units)
{
    static const int env_tn = env_int("HLQ_GEMV_TN", 0);
    static const int env_w = env_int("HLQ_GEMV_W", 0);
    static const int env_cpw = env_int("HLQ_GEMV_CPW", 0);
    GemvPlan pl;
    // Measured on MI355X (sweeps over TN x W x cpw on the 8B / 70B shapes): one tile per
    // wavefront, four wavefronts per workgroup; short runs for launches that would otherwise
    // not fill the wavefront slots, longer runs (fewer split-K partials) for large ones.
    pl.TN = 1;
    pl.W = 4;
    pl.cpw = units >= 65536 ? 8 : 4;
    if (use_mx()) {
        // matrix-core kernel (sweeps on the same shapes): short runs on many wavefronts while the
        // launch is small, longer runs once the chip is full
        pl.W = 8;
        pl.cpw = units < 12000 ? 4 : 7;
    }
    if (env_tn) pl.TN = env_tn;
    if (const int v = g_plan_tn.load(std::memory_order_relaxed)) pl.TN = v;
    pl.forced_w = env_w;
    pl.forced_cpw = env_cpw;
    if (const int v = g_plan_w.load(std::memory_order_relaxed)) pl.forced_w = v;
    if (const int v = g_plan_cpw.load(std::memory_order_relaxed)) pl.forced_cpw = v;
    if (pl.forced_w) pl.W = pl.forced_w;
    if (pl.forced_cpw) pl.cpw = pl.forced_cpw;
    return pl;
}

// chunks per K slice: a multiple of two (with G = 256 a group spans two chunks)
int slice_chunks(const GemvPlan &pl) { return (pl.W * pl.cpw + 1) & ~1; }
int slices_for(const HlqDims &dm, int cps) { return (dm.nchunks + cps - 1) / cps; }

// Work split of one problem for the matrix-core kernel: runs of about cpw chunks for every problem
// of a launch (wavefronts with longer runs would finish alone, with the memory system half idle):
// K is cut inside the workgroup first (kw wavefronts per tile), then across workgroups.
void plan_mx_problem(const HlqDims &dm, int W, int cpw, GemvProb &p)
{
    p.kw = 1;
    while (p.kw * 2 <= W && dm.nchunks / (p.kw * 2) >= cpw) p.kw *= 2;
    int per_slice = p.kw * cpw;
    if (per_slice < 4) per_slice = 4;
    p.nslices = (dm.nchunks + per_slice / 2) / per_slice;   // nearest
    if (p.nslices < 1) p.nslices = 1;
    const int tiles_per_wg = W / p.kw;
    p.ntg = (dm.ntiles + tiles_per_wg - 1) / tiles_per_wg;
    p.cps = ((dm.nchunks + p.nslices - 1) / p.nslices + 1) & ~1;   // even split, even boundaries
    // rounding the slice length up can leave trailing slices without a chunk: count the slices again, so
    // that every slice starts inside K ((nslices - 1) * cps < nchunks)
    p.nslices = (dm.nchunks + p.cps - 1) / p.cps;
}

// Which of several run lengths a launch of several rows gets, by an estimate in chunks.  The chip holds two wavefronts on a SIMD,
// 2048; a launch is so many rounds of them (one that leaves half the places free counts less), and a round takes its
// longest run and the start and end of a workgroup.  Places that come free early take what is left, so part of the
// estimate is the work over the places instead.  K slices cost an exchange at the end, a chunk.  Another candidate than the
// usual one has to be as much better as the estimate may be wrong.  Candidates whose K slices the counter block or the kernels'
// reciprocals cannot hold (short runs on the widest and deepest matrices) are passed over.
struct RunShape {
    int W, cpw;
};
struct RunCosts {
    double fixed;    // start and end of a workgroup
    double half;     // a round of at most 1024 wavefronts, in rounds
    double spread;   // part of the estimate that is work over places
    double margin;   // of the usual candidate's estimate, what another has to stay below
};

// estimate for one candidate; below zero: passed over
double run_estimate(int count, const HlqGemvItem *items, RunShape c, const RunCosts &k)
{
    long waves = 0, counters = 0;
    double work = 0;
    int longest = 0;
    for (int i = 0; i < count; ++i) {
        GemvProb p;
        plan_mx_problem(items[i].dm, c.W, c.cpw, p);
        if ((unsigned long long)p.ntg * p.nslices * p.nslices >= 0x100000000ULL) return -1;
        if (p.nslices > 1) counters += items[i].dm.ntiles;
        const int run = (p.cps + p.kw - 1) / p.kw;
        const long w = (long)p.ntg * p.nslices * c.W;
        waves += w;
        work += (double)w * (run + k.fixed);
        longest = run > longest ? run : longest;
    }
    if (counters > HLQ_WS_ARRIVAL_COUNTERS) return -1;
    // runs beyond 16 pay where they make one round of a launch: with several, a start hides behind the others' runs
    // (many rows, 8192 x 128256, q = 1, 4 rows: 47.7 us with runs of 16, 49.4 with 32)
    if (c.cpw > 16 && waves > 2048) return -1;
    const long rest = waves % 2048;
    const double rounds = (double)(waves / 2048) + (rest == 0 ? 0.0 : rest <= 1024 ? k.half : 1.0), one = longest + k.fixed;
    const double spread = work / 2048 > one ? work / 2048 : one;
    return (1 - k.spread) * one * rounds + k.spread * spread + (counters > 0 ? 1 : 0);
}

template <int NC>
RunShape plan_runs(int count, const HlqGemvItem *items, RunShape usual, const RunShape (&cand)[NC], const RunCosts &k)
{
    RunShape best = usual;
    const double known = run_estimate(count, items, usual, k);
    double least = known < 0 ? 1e300 : known * k.margin;
    for (const RunShape &c : cand) {
        const double e = run_estimate(count, items, c, k);
        if (e >= 0 && e < least) {
            least = e;
            best = c;
        }
    }
    return best;
}

// Many-rows kernel: runs of 4 below 12000 chunk-tiles and of 16 above unless the estimate falls by 9 %.  Over 180 launches (2048
// to 128256 chunk-tiles, single matrices and layers, q = 1 to 4, 4 to 16 rows; profiles/gemm_rows_to_32_rules.txt) 5 % faster than the usual one on
// average and 4 % slower at most; us:  q = 4, 16 rows  4096 x 14336 21.4 -> 18.8, 14336 x 4096 22.4 -> 20.2, 11008 x 9000 33.8 -> 28.3, 5120 x 13824
// 27.0 -> 20.9, layer of hidden 3072 / ffn 8192 31.6 -> 25.0, hidden 3840 / ffn 9984 43.6 -> 36.1, 8192 x 57344 81.5 -> 78.5;  q = 2, 8 rows
// 11008 x 9000 22.4 -> 18.7, 8192 x 57344 40.9 -> 36.3.  (Without the margin 7 % on average, but the layer of hidden 2560 / ffn 9984 28.4 -> 30.2.)
RunShape plan_many_rows(int count, const HlqGemvItem *items, long units)
{
    static const RunShape cand[] = {{4, 24}, {4, 16}, {4, 12}, {4, 10}, {4, 8}, {4, 6}, {4, 4}};
    return plan_runs(count, items, {4, units < 12000 ? 4 : 16}, cand, {8, 0.6, 0.2, 0.91});
}

// Few-rows instantiation of the 64-column kernel, from 4096 chunk-tiles on: eight wavefronts with runs of 4 below 12000 chunk-tiles
// and of 6 above, or what the estimate prefers.  Runs beyond eight chunks are slow whatever the rounds (the activations are
// cut into terms by every wavefront; hidden 3584 / ffn 10240, q = 4, 4 rows: 23 us with runs of 6, 43 with 16).  Over 180
// launches (same file) 5 % faster on average and 3 % slower at most; us:  q = 4, 4 rows  layer of hidden 3072 / ffn 8192 27.5 -> 18.0, hidden
// 2816 / ffn 8192 25.9 -> 20.4, 11008 x 9000 31.4 -> 22.3, 8192 x 10240 25.8 -> 20.2;  q = 2, 2 rows  hidden 3072 12.3 -> 10.6,
// 28672 x 8192 22.1 -> 18.1;  G = 64, q = 4, 2 rows  hidden 3072 22.4 -> 15.8
RunShape plan_few_rows(int count, const HlqGemvItem *items, long units, bool forced)
{
    static const RunShape cand[] = {{8, 4}, {8, 6}, {8, 8}, {4, 4}, {4, 6}, {4, 8}};
    const RunShape usual = {8, units < 12000 ? 4 : 6};
    return forced ? usual : plan_runs(count, items, usual, cand, {2, 0.5, 0.6, 1});   // (four wavefronts double the slices of a forced run)
}

// Work split of a launch of the one-row matrix-core kernel (hlq_gemv_cols.hip).  A step is 16 columns x 4 chunks of one
// wavefront.
struct ColsSplit {
    int kw, cps;       // wavefronts per column block, chunks per K slice
    int ntg;           // workgroups per K slice
    bool pairs;        // two slices that meet in slots of the counter block (8 bytes a column)
};

int cols_blocks(const HlqDims &dm) { return (dm.N + 15) / 16; }

// wavefronts on one column block: as many as there are windows to hand out
int cols_kw(int W, int nchunks)
{
    int kw = 1;
    while (kw * 2 <= W && kw < (nchunks + 3) / 4) kw *= 2;
    return kw;
}

// Which launches of one activation row go there instead of to the 64-column kernel (hlq_gemv_mx.hip).  It wins wherever a
// launch is short of wavefronts, and with groups of 128 and more on every size measured (microseconds, 64-column kernel
// against this one): q = 2, G = 128  4096 x 1024 4.95 / 3.17, 4096 x 4096 5.42 / 3.53, 14336 x 4096 7.95 / 6.5, 8B layer
// (27648 chunk-tiles) 13.8 / 13.2, 70B layer (104448) 42.1 / 41.1.  Its four column blocks of a tile fetch the lines of the
// tile's scales one after the other, which costs it the long launches with narrow groups: G = 32  4096 x 28672
// (14336) 12.1 / 13.3, 70B layer 70.7 / 72.3 (q = 4: 126 / 135);  G = 64, q = 2  70B layer 48.0 / 49.7, LM head (256512)
// 56.5 / 57.9 (q = 4: 94.8 / 90.5).  With one plane a step is too short for its fixed part on launches of one round:
// q = 1, G = 256  8B layer 9.4 / 10.1, but 70B layer 28.8 / 25.8.
bool cols_wins(long units, int q, int G)
{
    if (hlq_cols_always(q, G)) return true;
    if (G == 32) return units < 12000;
    if (q == 1) return units < 20000 || units >= 60000;
    return units < 60000;   // G = 64, q = 2, 3
}

// cpw: forced chunks per wavefront (0: automatic); forced_w likewise.  Returns the wavefronts per workgroup.
int plan_cols(int count, const HlqDims *dms, int rows, int forced_w, int cpw, ColsSplit *out)
{
    const int q = dms[0].q, G = dms[0].G, maxw = hlq_gemv_cols_max_waves(q, G, rows);
    long blocks = 0;
    for (int i = 0; i < count; ++i) blocks += cols_blocks(dms[i]);
    // K slices.  One up to sixteen windows (K = 8192: a window per wavefront).  Two up to 32 windows, in which case the sides
    // meet in one exchange per column: 14336 x 1024 5.5 us in one slice, 4.5 in two; 14336 x 512 5.4 / 4.4; 11008 x 5000,
    // q = 3, G = 64 10.1 / 8.4.  Where the columns alone give every compute unit its workgroup two slices are the slower
    // plan, 14336 x 4096 6.0 / 6.5, 11008 x 4096 5.5 / 5.8; it is kept for them because the tests
    // of the static scratch array take 14336 x 4096 for a problem whose K is split under every plan.  Longer K over few columns: one slice per sixteen windows,
    // partial sums and arrival counters: 28672 x 1024 8.5 / 6.5, 28672 x 512 8.3 / 5.8; over more columns one slice,
    // 28672 x 8192 13.5.
    int most_wins = 1;
    long slots = 0;   // of the counter block, of which half is left to arrival counters
    for (int i = 0; i < count; ++i) {
        const int n = dms[i].nchunks, wins = (n + 3) / 4;
        const bool two = rows == 1 && wins > 16 && wins <= 32 && 2L * dms[i].N <= HLQ_WS_ARRIVAL_COUNTERS / 2;
        const int per = two ? (wins + 1) / 2 : blocks <= 128 && wins > 32 ? 16 : wins;
        const int slices = (wins + per - 1) / per;
        int cps = (n + slices - 1) / slices;
        if (cpw) cps = (forced_w ? forced_w : 8) * (cpw < HLQ_MAX_K / HLQ_CHUNK_K ? cpw : HLQ_MAX_K / HLQ_CHUNK_K);
        cps = (cps + 1) & ~1;   // slices of more than one chunk pair: windows start even
        if (cps < 4) cps = 4;
        out[i].cps = cps < n ? cps : n;
        const int w = (out[i].cps + 3) / 4;
        if (w > most_wins) most_wins = w;
        out[i].pairs = rows == 1 && out[i].cps < n && 2 * out[i].cps >= n && slots + 2L * dms[i].N <= HLQ_WS_ARRIVAL_COUNTERS / 2;
        if (out[i].pairs) slots += 2L * dms[i].N;
    }
    // wavefronts per workgroup: as many as windows, eight or sixteen
    int W = forced_w ? forced_w : most_wins > 8 ? 16 : 8;
    if (W > maxw) W = maxw;
    while (W & (W - 1)) W &= W - 1;

    // Workgroups: one step per wavefront if all of those are resident at once (the kernel's one-step form takes 58..63
    // registers at q <= 2, G >= 64: 32 wavefronts a compute unit; 62..75 otherwise: 24 or more, 83 at q = 4, G = 32: 20, but
    // there too the one-step form is the faster one up to 24: 4096 x 10240 10.2 us against 11.9 in several steps, 4096 x
    // 12288 12.0 / 12.4), else as few steps per wavefront as one generation of workgroups (16 wavefronts a compute unit)
    // needs: a second generation of a few costs as much as a full one (8B layer 20 us instead of 13).
    long one_step = 0, cost[HLQ_MAX_BATCH];
    bool one_round = true;
    for (int i = 0; i < count; ++i) {
        out[i].kw = cols_kw(W, out[i].cps);
        const int rounds = ((out[i].cps + 3) / 4 + out[i].kw - 1) / out[i].kw, streams = W / out[i].kw;
        const int slices = (dms[i].nchunks + out[i].cps - 1) / out[i].cps;
        cost[i] = (long)cols_blocks(dms[i]) * rounds * slices / streams;
        one_step += (long)((cols_blocks(dms[i]) + streams - 1) / streams) * slices;
        one_round = one_round && rounds == 1;
    }
    // several rows (operands of 24 registers a row and more): what is resident is one generation of 16 or 8 wavefronts
    const int resident = rows == 1 ? 16 : rows == 2 ? 16 : 8;
    const int per_cu = (rows > 1 ? resident : q <= 2 && G >= 64 ? 32 : 24) / W;
    const bool single = one_round && one_step <= 256L * (per_cu > 0 ? per_cu : 1);
    long steps = 1;
    if (!single)
        for (;; ++steps) {
            long wgs = 0;
            for (int i = 0; i < count; ++i) wgs += (cost[i] + steps - 1) / steps;
            if (wgs <= 256L * resident / W || steps >= 40) break;
        }
    for (int i = 0; i < count; ++i) {
        const int nb = cols_blocks(dms[i]), streams = W / out[i].kw, slices = (dms[i].nchunks + out[i].cps - 1) / out[i].cps;
        long ntg = single ? (nb + streams - 1) / streams : ((cost[i] + steps - 1) / steps + slices - 1) / slices;
        const int cap = slices > 1 && !out[i].pairs ? 4 : HLQ_COLS_MAX_SLOTS / out[i].kw;   // column blocks a workgroup can hold
        if (ntg < (nb + cap - 1) / cap) ntg = (nb + cap - 1) / cap;
        if (ntg > nb) ntg = nb;
        out[i].ntg = (int)(ntg < 1 ? 1 : ntg);
    }
    return W;
}

void plan_cols_problem(const HlqDims &dm, const ColsSplit &sp, GemvProb &p)
{
    p.kw = sp.kw;
    p.cps = sp.cps;
    p.nslices = (dm.nchunks + sp.cps - 1) / sp.cps;
    p.ntg = sp.ntg;
}

// the kernel's own record, from the planned and placed problem
ColsProb cols_record(const GemvProb &p, int W, bool pairs)
{
    ColsProb r;
    const int nb = (p.N + 15) / 16;
    r.packed = p.packed;
    r.x = p.x;
    r.y = p.y;
    r.part = p.part;
    r.cnt = p.cnt;
    r.tile_bytes = (unsigned)(HLQ_TILE_N * p.col_bytes);   // below 2^27: K <= 2^21 and at most 0.8 bytes a weight
    r.N = p.N;
    r.nchunks = p.nchunks;
    r.cps = p.cps;
    r.nslices = p.nslices;
    r.slice_magic = p.slice_magic;
    r.ntg = p.ntg;
    r.blk_begin = p.blk_begin;
    r.cb_base = nb / p.ntg;
    r.cb_rem = nb % p.ntg;
    const int full = ((p.cps < p.nchunks ? p.cps : p.nchunks) + 3) / 4, last = (p.nchunks - (p.nslices - 1) * p.cps + 3) / 4;
    r.wbase = (uint16_t)(full / p.kw);   // windows of K = 2^21: 4096
    r.wrem = (uint16_t)(full % p.kw);
    r.wbase_l = (uint16_t)(last / p.kw);
    r.wrem_l = (uint16_t)(last % p.kw);
    r.kw_shift = (uint8_t)p.kw_shift;
    r.st_shift = 0;
    while ((p.kw << r.st_shift) < W) ++r.st_shift;
    r.unused = 0;
    r.pairs = pairs;
    return r;
}

} // namespace

hlq_status hlq_gemv_path_override(int path)
{
    if (path < 0 || path > 6) return HLQ_ERR_UNSUPPORTED;
    g_gemv_path = path;
    return HLQ_OK;
}

hlq_status hlq_gemv_plan_override(int tn, int w, int cpw)
{
    if (tn < 0 || tn > 2 || w < 0 || w > 16 || cpw < 0) return HLQ_ERR_UNSUPPORTED;
    g_plan_tn = tn;
    g_plan_w = w;
    g_plan_cpw = cpw;
    return HLQ_OK;
}

size_t hlq_gemv_partial_bytes(const HlqDims &dm)
{
    // Upper bound over every plan: slices are never shorter than 4 chunks.
    const int ns = (dm.nchunks + 3) / 4;
    return ns > 1 ? (size_t)ns * (size_t)dm.N * sizeof(float) : 0;
}

hlq_status hlq_launch_ws_init(void *ws, size_t bytes, hipStream_t st)
{
    hlq_clear_stale_error();
    if (bytes < HLQ_WS_COUNTER_BYTES) return HLQ_ERR_BUFFER_TOO_SMALL;
    const int n = HLQ_WS_COUNTER_BYTES / 4;
    hlq_ws_init_kernel<<<(n + 255) / 256, 256, 0, st>>>((int *)ws, n);
    return hlq_hip_status(hipGetLastError());
}

// The work split of a grouped launch: everything the host decides (formulation, workgroup shape, K
// slices and runs per problem, block ranges, workspace carving).  Touches no device memory, so the
// plan can also be inspected without a GPU (hlq_gemv_plan_query).
struct GemvLaunchShape {
    bool mx;
    bool cols;        // the one-row kernel with 16 columns per wavefront (hlq_gemv_cols.hip)
    bool rowsk;       // the many-rows kernel (hlq_gemm_rows.hip) instead of the few-rows instantiation of the GEMV kernel
    int W, TN, rows;
    long nblocks;
    size_t ws_used;   // bytes of the workspace this plan touches: the counter block and its partial sums
};

static bool few_rows_win(int count, const HlqGemvItem *items, int64_t rows)
{
    HlqDims dms[HLQ_MAX_BATCH];
    for (int i = 0; i < count; ++i) dms[i] = items[i].dm;
    return hlq_gemm_few_wins(count, dms, rows);
}

static bool few_rows(int count, const HlqGemvItem *items, int64_t rows)
{
    HlqDims dms[HLQ_MAX_BATCH];
    for (int i = 0; i < count; ++i) dms[i] = items[i].dm;
    return hlq_gemm_few_rows(count, dms, rows);
}

// What a launch of several rows is planned with; where that does not fit, the next.
enum PlanBy {
    PLAN_KNOBS,   // the choice of kernel, and hlq_set_gemv_plan
    PLAN_OWN,     // the choice of kernel, no knobs
    PLAN_COLS,    // the 16-column kernel, no knobs
};

static hlq_status plan_gemv_batch(int count, const HlqGemvItem *items, hlq_out_dtype out, void *ws, PlanBy by, GemvBatch &b,
                                  GemvLaunchShape &ls)
{
    if (count < 1 || count > HLQ_MAX_BATCH) return HLQ_ERR_UNSUPPORTED;
    long units = 0;
    for (int i = 0; i < count; ++i) units += (long)items[i].dm.ntiles * items[i].dm.nchunks;
    GemvPlan pl = plan_gemv(units);
    const int rows = items[0].M;
    for (int i = 1; i < count; ++i)
        if (items[i].M != rows) return HLQ_ERR_UNSUPPORTED;
    if (rows < 1 || (rows > hlq_gemm_mx_rows_per_pass(items[0].dm.G) && !few_rows_win(count, items, rows))) return HLQ_ERR_UNSUPPORTED;
    const bool mx = use_mx() || rows > 1;   // several activation rows exist in the matrix-core kernels only
    const bool cols = mx && (rows == 1 ? cols_wins(units, items[0].dm.q, items[0].dm.G) : by == PLAN_COLS ? few_rows(count, items, rows) : few_rows_win(count, items, rows));
    // more rows than one operand of the GEMV kernel holds: the many-rows kernel (terms chained through the
    // accumulator, activations converted once per workgroup), where it exists for this group size
    bool rowsk = !cols && rows > hlq_gemv_mx_rows_per_set(items[0].dm.G) && rows <= hlq_gemm_rows_max(items[0].dm.G) &&
                 rows <= hlq_gemm_mx_rows_per_pass(items[0].dm.G);
    // three or four rows (which the GEMV kernel's one row set also holds): the one-operand instantiation of the
    // many-rows kernel where its pre-pass pays
    if (!cols && !rowsk && rows >= 3 && rows <= hlq_gemm_rows_max(items[0].dm.G) &&
        (hlq_gemm_rows_all() || hlq_gemm_rows_wins_few(units, items[0].dm.q, rows)))
        rowsk = true;
    // several rows: the knobs only, the environment is for one row
    const int knob_w = by == PLAN_KNOBS ? g_plan_w.load(std::memory_order_relaxed) : 0, knob_cpw = by == PLAN_KNOBS ? g_plan_cpw.load(std::memory_order_relaxed) : 0;
    if (rowsk) {
        const RunShape r = plan_many_rows(count, items, units);
        pl.W = r.W;
        pl.cpw = r.cpw;
        if (knob_cpw) pl.cpw = knob_cpw < 4 ? 4 : knob_cpw;
    } else if (cols) {
        pl.W = rows == 1 ? pl.forced_w : knob_w;   // 0: plan_cols chooses
        pl.cpw = rows == 1 ? pl.forced_cpw : knob_cpw;
        if (pl.W < 0 || pl.cpw < 0) return HLQ_ERR_UNSUPPORTED;   // (of the environment)
    } else if (rows > 1) {
        // narrow launches: short runs on few wavefronts per workgroup (measured on 8B shapes, q = 4, 2..8 rows)
        const RunShape r = units < 4096 ? RunShape{4, 2} : plan_few_rows(count, items, units, knob_w || knob_cpw);
        pl.W = knob_w ? knob_w : r.W;
        pl.cpw = knob_cpw ? knob_cpw : r.cpw;
    }
    {
        const int q0 = items[0].dm.q, G0 = items[0].dm.G;
        if (mx || !gemv_two_tiles_ok(q0, G0) || table_variant() >= 0) pl.TN = 1;
        const int maxw = cols ? 16 : mx ? hlq_gemv_mx_max_waves(q0, G0) : gemv_max_threads(q0, G0, pl.TN) / 64;
        if (pl.W > maxw) pl.W = maxw;
        if (!mx && table_variant() >= 0 && pl.W > 8) pl.W = 8;   // the plain variant kernels: up to 512 lanes
        if (rowsk) {
            pl.W = 4;
            if (knob_w) pl.W = knob_w >= 8 ? 8 : knob_w >= 4 ? 4 : 2;
        }
        if (mx)   // a power of two
            while (pl.W & (pl.W - 1)) pl.W &= pl.W - 1;
    }
    if (!cols && (pl.W < 1 || pl.W > 16 || (pl.TN != 1 && pl.TN != 2) || pl.cpw < 1)) return HLQ_ERR_UNSUPPORTED;
    // chunks per K slice of the lookup kernel: each of its W wavefronts takes cpw chunks of one tile
    int cps = cols ? 4 : slice_chunks(pl);
    if (cps < 4) cps = 4;

    ColsSplit split[HLQ_MAX_BATCH];
    if (cols) {
        HlqDims dms[HLQ_MAX_BATCH];
        for (int i = 0; i < count; ++i) dms[i] = items[i].dm;
        pl.W = plan_cols(count, dms, rows, pl.W, pl.cpw, split);
    }

    b.count = count;
    b.out_f32 = out == HLQ_OUT_F32;
    int *cnt = (int *)ws;
    float *part = (float *)((char *)ws + HLQ_WS_COUNTER_BYTES);
    long blk = 0;
    long cnt_used = 0;
    // Workgroups start in block order: problems with long K (long runs, or K split across workgroups
    // with extra trips to memory at the end) go first.
    int order[HLQ_MAX_BATCH];
    for (int i = 0; i < count; ++i) order[i] = i;
    for (int i = 1; i < count; ++i)
        for (int j = i; j > 0 && items[order[j]].dm.nchunks > items[order[j - 1]].dm.nchunks; --j) {
            const int t = order[j];
            order[j] = order[j - 1];
            order[j - 1] = t;
        }
    for (int i = 0; i < count; ++i) {
        const HlqDims &dm = items[order[i]].dm;
        GemvProb &p = b.p[i];
        p.packed = (const char *)items[order[i]].packed;
        p.x = items[order[i]].x;
        p.y = items[order[i]].y;
        p.col_bytes = dm.col_bytes;
        p.N = dm.N;
        p.nchunks = dm.nchunks;
        p.ntiles = dm.ntiles;
        p.kw = 1;
        p.M = rows;
        p.ldx = items[order[i]].ldx;
        p.ldy = items[order[i]].ldy;
        if (cols) {
            plan_cols_problem(dm, split[order[i]], p);
        } else if (rowsk) {
            plan_mx_problem(dm, pl.W, pl.cpw, p);
        } else if (mx) {
            plan_mx_problem(dm, pl.W, pl.cpw, p);
        } else {
            p.ntg = (dm.ntiles + pl.TN - 1) / pl.TN;
            p.nslices = slices_for(dm, cps);
            p.cps = ((dm.nchunks + p.nslices - 1) / p.nslices + 1) & ~1;   // even split, even boundaries
            p.nslices = slices_for(dm, p.cps);
        }
        // every K slice must start inside K: the kernels form addresses from a slice's first chunk
        if (p.nslices < 1 || p.cps < 1 || (long)(p.nslices - 1) * p.cps >= dm.nchunks) return HLQ_ERR_UNSUPPORTED;
        p.kw_shift = 0;
        while ((1 << p.kw_shift) < p.kw) ++p.kw_shift;
        // exact for local * nslices < 2^32, far above any grid this library launches (checked below)
        p.slice_magic = p.nslices > 1 ? (unsigned)((0x100000000ULL + (unsigned)p.nslices - 1) / (unsigned)p.nslices) : 0u;
        if ((unsigned long long)p.ntg * p.nslices * p.nslices >= 0x100000000ULL) return HLQ_ERR_UNSUPPORTED;
        p.blk_begin = (int)blk;
        b.blk_begin[i] = (int)blk;
        if (cols && split[order[i]].pairs) cnt_used = (cnt_used + 1) & ~1L;   // 64-bit slots, behind any number of 32-bit counters
        p.cnt = cnt + cnt_used;
        p.part = part;
        blk += (long)p.ntg * p.nslices;
        if (cols && split[order[i]].pairs) {
            cnt_used += 2L * dm.N;
        } else if (p.nslices > 1) {
            cnt_used += mx && !cols ? dm.ntiles : p.ntg;
            part += (size_t)p.nslices * dm.N * rows;
        }
    }
    if (rowsk) {
        // behind all partial sums: the activations in operand form, once for problems that read the same ones
        char *xt = (char *)(((uintptr_t)part + 255u) & ~(uintptr_t)255u);
        for (int i = 0; i < count; ++i) {
            GemvProb &p = b.p[i];
            int first = 0;
            while (b.p[first].x != p.x || b.p[first].ldx != p.ldx || b.p[first].nchunks != p.nchunks) ++first;
            p.xt_own = first == i;
            p.xt = p.xt_own ? xt : b.p[first].xt;
            if (p.xt_own) xt += hlq_gemm_rows_xt_bytes(items[order[i]].dm, rows);
        }
        part = (float *)xt;
    } else {
        for (int i = 0; i < count; ++i) {
            b.p[i].xt = nullptr;
            b.p[i].xt_own = 0;
        }
    }
    if (cols)
        for (int i = 0; i < count; ++i) b.cp[i] = cols_record(b.p[i], pl.W, split[order[i]].pairs);
    for (int i = count; i < HLQ_MAX_BATCH; ++i) {
        b.p[i] = b.p[0];
        if (cols) b.cp[i] = b.cp[0];
        b.blk_begin[i] = 0x7fffffff;
    }
    if (cnt_used > HLQ_WS_ARRIVAL_COUNTERS || blk > 0x7fffffffL) return HLQ_ERR_UNSUPPORTED;
    ls.mx = mx;
    ls.cols = cols;
    ls.rowsk = rowsk;
    ls.W = pl.W;
    ls.TN = pl.TN;
    ls.rows = rows;
    ls.nblocks = blk;
    ls.ws_used = HLQ_WS_COUNTER_BYTES + (size_t)(part - (float *)((char *)ws + HLQ_WS_COUNTER_BYTES)) * sizeof(float);
    return HLQ_OK;
}

// The plan of a launch.  With several rows a forced plan of more K slices than the counter block or the block arithmetic has room
// for is not followed (it is no reason to refuse the call), and where the built-in plan of the 64-column kernel has too many, on
// the widest and deepest matrices, the 16-column kernel, which seldom cuts K, takes the calls that it can.
static hlq_status plan_launch(int count, const HlqGemvItem *items, hlq_out_dtype out, void *ws, GemvBatch &b, GemvLaunchShape &ls)
{
    hlq_status s = plan_gemv_batch(count, items, out, ws, PLAN_KNOBS, b, ls);
    if (s != HLQ_ERR_UNSUPPORTED || items[0].M < 2) return s;
    s = plan_gemv_batch(count, items, out, ws, PLAN_OWN, b, ls);
    if (s != HLQ_ERR_UNSUPPORTED || !few_rows(count, items, items[0].M)) return s;
    return plan_gemv_batch(count, items, out, ws, PLAN_COLS, b, ls);
}

hlq_status hlq_launch_gemv_batch(int count, const HlqGemvItem *items, hlq_out_dtype out, void *ws,
                                 hipStream_t st, size_t ws_cap)
{
    hlq_clear_stale_error();
    GemvBatch b;
    GemvLaunchShape ls;
    hlq_status s = plan_launch(count, items, out, ws, b, ls);
    if (s != HLQ_OK) return s;
    if (ws_cap && ls.ws_used > ws_cap) return HLQ_ERR_BUFFER_TOO_SMALL;   // checked on the plan that is launched
    const int q = items[0].dm.q, G = items[0].dm.G;
    const unsigned blk = (unsigned)ls.nblocks;
    if (ls.rowsk) {
        s = hlq_launch_gemm_rows(b, blk, ls.W, ls.rows, q, G, st);
        if (s != HLQ_OK) return s;
        return hlq_hip_status(hipGetLastError());
    }
    if (ls.cols) {
        s = hlq_launch_gemv_cols(b, blk, ls.W, ls.rows, q, G, st);
        if (s != HLQ_OK) return s;
        return hlq_hip_status(hipGetLastError());
    }
    if (ls.mx) {
        const int nsets = ls.rows == 1 ? 0 : ls.rows <= hlq_gemv_mx_rows_per_set(G) ? 1 : 2;
        s = hlq_launch_gemv_mx(b, blk, ls.W, nsets, ls.rows, q, G, st);
        if (s != HLQ_OK) return s;
        return hlq_hip_status(hipGetLastError());
    }
    if (table_variant() >= 0 && ls.TN == 1) {
        s = hlq_launch_gemv_variant(table_variant(), b, blk, ls.W, q, G, st);
        if (s != HLQ_OK) return s;
        return hlq_hip_status(hipGetLastError());
    }
    switch (q) {
    case 1: s = launch_q<1>(G, b, blk, ls.W, ls.TN, st); break;
    case 2: s = launch_q<2>(G, b, blk, ls.W, ls.TN, st); break;
    case 3: s = launch_q<3>(G, b, blk, ls.W, ls.TN, st); break;
    case 4: s = launch_q<4>(G, b, blk, ls.W, ls.TN, st); break;
    default: return HLQ_ERR_UNSUPPORTED;
    }
    if (s != HLQ_OK) return s;
    return hlq_hip_status(hipGetLastError());
}

// Workspace bytes the GEMV of one matrix touches with the plan it would get now (at most the bound
// hlq_workspace_bytes reports, usually far less: most plans cut K inside a workgroup only).
hlq_status hlq_gemv_ws_used(const HlqDims &dm, size_t *bytes)
{
    HlqGemvItem it;
    it.dm = dm;
    it.packed = nullptr;
    it.x = nullptr;
    it.y = nullptr;
    GemvBatch b;
    GemvLaunchShape ls;
    const hlq_status s = plan_launch(1, &it, HLQ_OUT_F16, nullptr, b, ls);
    if (s == HLQ_OK) *bytes = ls.ws_used;
    return s;
}

// The plan of a launch of `count` problems with M rows each, as hlq_launch_gemv_batch would make it now
// (current knobs).  Host arithmetic only.
hlq_status hlq_gemv_plan_describe(int count, const HlqDims *dms, int M, hlq_gemv_plan_info *out)
{
    HlqGemvItem items[HLQ_MAX_BATCH];
    if (count < 1 || count > HLQ_MAX_BATCH) return HLQ_ERR_UNSUPPORTED;
    for (int i = 0; i < count; ++i) {
        items[i].dm = dms[i];
        items[i].packed = nullptr;
        items[i].x = nullptr;
        items[i].y = nullptr;
        items[i].M = M;
        items[i].ldx = dms[i].K;
        items[i].ldy = dms[i].N;
    }
    GemvBatch b;
    GemvLaunchShape ls;
    const hlq_status s = plan_launch(count, items, HLQ_OUT_F16, nullptr, b, ls);
    if (s != HLQ_OK) return s;
    bool taken[HLQ_MAX_BATCH] = {};
    for (int i = 0; i < count; ++i) {
        // problems are planned in launch order (long K first); report them in the caller's order
        int at = -1;
        for (int k = 0; k < count && at < 0; ++k)
            if (!taken[k] && b.p[k].nchunks == dms[i].nchunks && b.p[k].N == dms[i].N && b.p[k].col_bytes == dms[i].col_bytes) at = k;
        if (at < 0) return HLQ_ERR_UNSUPPORTED;
        taken[at] = true;
        const GemvProb &p = b.p[at];
        out[i].formulation = ls.mx ? 2 : 1;
        out[i].waves_per_workgroup = ls.W;
        out[i].waves_per_tile = ls.mx ? p.kw : ls.W;
        out[i].chunks_per_slice = p.cps;
        out[i].slices = p.nslices;
        out[i].tile_groups = p.ntg;
        out[i].first_block = p.blk_begin;
        out[i].blocks = (int32_t)((long)p.ntg * p.nslices);
    }
    return HLQ_OK;
}

// Rows an MX launch can carry for group size G: two row sets of the GEMV kernel, or what the many-rows kernel holds.
int hlq_gemm_mx_rows_per_pass(int G)
{
    const int two_sets = 2 * hlq_gemv_mx_rows_per_set(G);
    const int many = hlq_gemm_rows_max(G);
    return many > two_sets ? many : two_sets;
}

static long chunk_tiles(int count, const HlqDims *dms, int &deepest)
{
    long units = 0;
    deepest = 0;
    for (int i = 0; i < count; ++i) {
        units += (long)dms[i].ntiles * dms[i].nchunks;
        deepest = dms[i].nchunks > deepest ? dms[i].nchunks : deepest;
    }
    return units;
}

// Calls of two to four rows that a GEMV-shaped kernel takes (this one or the 64-column one, which keep scales in fp32) also
// where the rows exceed a row set of the latter and a single call would otherwise go to the kernels that rebuild weights in fp16
bool hlq_gemm_few_rows(int count, const HlqDims *dms, int64_t rows)
{
    if (rows < 2 || rows > HLQ_COLS_ROWS || (rows > 2 && hlq_gemm_rows_all())) return false;
    int deepest;
    const long units = chunk_tiles(count, dms, deepest);
    return (rows > hlq_gemv_mx_rows_per_set(dms[0].G) && units >= 14000) || (units >= 256 && units <= 4096 && deepest <= 64);
}

// Which of those go to the kernel of one row (hlq_gemv_cols.hip) instead of the 64-column one.  It pays for the operands of every
// window (512 k) of every row, whatever the number of column blocks that a wavefront walks over with them, and eight
// wavefronts are what a compute unit holds: it loses on short K, where operands are most of a step, and on deep K with few columns,
// where a wavefront makes many and walks little.  Time over the other kernel's, at q = 1 / 2 / 4:
//   up to 4096 chunk-tiles   512 x 4096 G = 128 M = 2 1.14 / 1.10 / 1.06, M = 3 1.23 / 1.20 / 1.19;  256 x 65536 1.4 to 1.6;
//     2048 x 6144 M = 2 .75 / .74 / .76, M = 4 .72 / .72 / .74;  4096 x 1024 .80 / .78 / .79, .82 / .79 / .81;  4096 x 6144 .95 / .94 / .93,
//     .82 / .86 / .84;  4096 x 8192 M = 2 1.11 / 1.04 / .89, M = 4 .99 / .93 / .84;  6144 x 5120 M = 2 1.20 / 1.17 / 1.15, M = 3 .87 / .94 / .96;
//     8192 x 256 1.2;  8192 x 2048 M = 3 1.06 / 1.11 / 1.14;  8192 x 4096 M = 2 .99 / .91 / .80, M = 4 .86 / .87 / .83
//   more rows than a row set  4096 x 28672 (14336) G = 64 M = 4 .88 / .87 / .92, M = 3 .99 / .93 / .97, G = 32 M = 2 1.23 / 1.07 / 1.06;
//     8192 x 14336 M = 4 1.11 / 1.06 / 1.06, M = 3 1.25 / 1.16 / 1.16, G = 32 M = 2 1.50 / 1.25 / 1.13;  8192 x 18432 (18432) M = 4 .70 / .67 / .68,
//     M = 3 .98 / .73 / .75, G = 32 M = 2 1.00 / .84 / .79;  8B layer (26624) M = 4 .87 / .85 / .87, M = 3 1.26 / .94 / .95;  16384 x 28672 M = 4 .72 /
//     .73 / .77, M = 3 1.01 / .83 / .86;  28672 x 24576 M = 4 1.81 / 1.68 / 1.45, M = 3 2.30 / 1.90 / 1.64;  70B layer M = 4 1.11 / 1.13 / 1.08
bool hlq_gemm_few_wins(int count, const HlqDims *dms, int64_t rows)
{
    if (!hlq_gemm_few_rows(count, dms, rows)) return false;
    const int G = dms[0].G, q = dms[0].q;
    if (rows > hlq_gemm_mx_rows_per_pass(G)) return true;   // three and four rows at G = 32: more than the other one's two row sets
    int deepest;
    const long units = chunk_tiles(count, dms, deepest);
    if (units > 4096) {
        const bool one_more = rows == hlq_gemv_mx_rows_per_set(G) + 1;
        if (deepest <= 32) return units >= (one_more ? 18000 : 14000);
        return units >= 18000 && deepest <= 160 && !(one_more && q == 1);
    }
    if (deepest <= 32) return deepest >= 12 && (units <= 3072 || q > 2 || rows == 4 || G == 32);
    return units > 3072 && (rows > 2 || deepest > 56);
}

// Many-rows kernel or, with weights rebuilt in fp16, the short-M kernel (hlq_gemm_short.hip) for 5..16 rows (G >= 128)?  The
// many-rows kernel keeps scales in fp32: a call that it has been taking stays with it although the other one is faster
// below some 14000 chunk-tiles.  Single calls and grouped launches, us (many-rows / short-M):
//   q = 4, up to 8 rows:  2048 chunk-tiles 14.8 / 9.3,  7168: 19.4 / 14.8,  14336: 25.7 / 28.5,  20480: 35.8 / 44.8,  8B layer 35.4 / 48.2
//   q = 4, 9..16 rows:    2048: 15.5 / 9.6,  7168: 21.0 / 13.8,  14336: 28.1 / 28.5,  20480: 42.2 / 44.9,  8B layer 44.2 / 48.4
//   q = 2, up to 8 rows:  2048: 13.2 / 7.8,  7168: 15.0 / 9.5,  14336: 18.5 / 19.7,  20480: 23.8 / 30.5,  8B layer 24.6 / 32.4
//   q = 2, 9..16 rows:    7168: 16.7 / 9.9,  14336: 20.3 / 20.0,  28672: 31.3 / 33.4,  8B layer 29.8 / 33.0
// For 3 or 4 rows the alternative is the few-rows instantiation of the GEMV kernel
// (which converts the activations in every wavefront and needs no pre-pass).  Measured, many-rows against few-rows:
//   8B layer (27648 chunk-tiles)  q = 4: 33.3 / 36.4 (3 rows), 33.2 / 39.5 (4 rows);  q = 3: 28.8 / 27.0, 28.7 / 30.1;
//                                 q = 2: 25.6 / 22.5, 26.0 / 26.0
//   70B layer (104448), q = 2: 66.3 / 68.3, 67.0 / 77.6;   one 4096 x 14336 (7168), q = 4: 18.5 / 13.0, 18.5 / 14.3
bool hlq_gemm_rows_wins_few(long units, int q, int rows)
{
    if (q >= 4) return units >= 20000;
    if (rows < 4) return false;
    return units >= (q == 3 ? 40000 : 60000);
}

bool hlq_gemm_rows_wins(long units, int q, int64_t M)
{
    if (M <= 8) return units >= (q >= 3 ? 4096 : 12000);
    return units >= (q >= 3 ? 2400 : 14000);
}

// Whether a grouped launch of M rows goes to the matrix-core GEMV-shaped kernels (few-rows / many-rows) rather
// than to the kernels that rebuild weights: up to one row set (four rows at G >= 128) and whatever the second row set of the
// GEMV kernel carries at G <= 64 always; 5..16 rows at G >= 128 by the rule above; hlq_set_gemm_path(4) sends all of
// them here.
bool hlq_gemm_batch_on_mx(int count, const HlqGemvItem *items, int64_t M)
{
    if (count < 1 || M < 1) return false;
    const int G = items[0].dm.G;
    if (few_rows_win(count, items, M)) return true;
    if (M > hlq_gemm_mx_rows_per_pass(G)) return false;
    if (M <= hlq_gemv_mx_rows_per_set(G) || hlq_gemm_rows_max(G) == 0 || hlq_gemm_rows_all()) return true;
    long units = 0;
    for (int i = 0; i < count; ++i) units += (long)items[i].dm.ntiles * items[i].dm.nchunks;
    return hlq_gemm_rows_wins(units, items[0].dm.q, M);
}

size_t hlq_gemm_mx_partial_bytes(const HlqDims &dm, int64_t M)
{
    const int pass = hlq_gemm_mx_rows_per_pass(dm.G), cap = pass > HLQ_COLS_ROWS ? pass : HLQ_COLS_ROWS;
    const int64_t rows = M < cap ? M : cap;
    // slices are never shorter than 4 chunks here either; the many-rows kernel adds the operand form of the activations
    return (size_t)rows * hlq_gemv_partial_bytes(dm) + hlq_gemm_rows_xt_bytes(dm, 16) + 256;
}

// Y[M, N] = X[M, K] @ W^ for as many rows as one pass of the matrix-core GEMV kernel carries.
hlq_status hlq_launch_gemm_mx_rows(const HlqDims &dm, const void *packed, const uint16_t *X, int64_t M, int64_t ldx,
                                   void *Y, int64_t ldy, hlq_out_dtype out, void *ws, hipStream_t st)
{
    if (M < 1) return HLQ_ERR_UNSUPPORTED;
    HlqGemvItem it;
    it.dm = dm;
    it.packed = packed;
    it.x = X;
    it.y = Y;
    it.M = (int)M;
    it.ldx = (long)ldx;
    it.ldy = (long)ldy;
    return hlq_launch_gemv_batch(1, &it, out, ws, st);
}
