// hlq_lut_gemm for up to 32 rows (those the many-rows kernel does not take, where hlq_gemm_short_wins finds it faster than the
// tiled kernel): the formulation of the tiled kernel (hlq_gemm_mfma.hip) -- W^ = sum_j s_j b_j + z (Eq. 3) rebuilt in fp16 registers,
// v_mfma_f32_32x32x16_f16 -- with K cut inside the workgroup instead of across workgroups.
//
// Work split.  A workgroup of eight wavefronts owns one tile of 64 columns and one K slice (all of K if there are enough
// tiles); wavefront p takes part p of the slice's chunks, and the parts' results meet in LDS.  The tiled kernel gives a
// workgroup 256 columns and needs eight K slices to fill the chip with 4096 x 14336: 11 MB of partial sums written and
// read back, and a second launch for them.
//
// A step is a chunk: lane = column as in the tiled kernel, the same exchange of register halves between lanes 0..31 and
// 32..63, two matrix-core instructions (columns 0..31, 32..63) per A fragment.  X is the wavefront's own: its chunk of all
// rows goes through registers, a step ahead, to its part of LDS (16-byte units, unit u of row r at u ^ (r & 7)), so
// wavefronts wait for nobody before the end.  (Two wavefronts with 32 columns each and two chunks a step need no lane
// exchange but share X and a barrier every step, after which all eight want the vector unit at once and wait for memory
// at once: 8B layer at q = 4, M = 32 61.0 us against 53.9; 4096 x 14336, q = 3, G = 64, M = 24 the same.)
//
// Parameters outside the range of the rebuild (hlq_gemm_safe.hip): without K slices the workgroup itself computes its
// tile again in fp32; with them it raises the flag for the launch that adds the slices.
//
// What bounds it: the vector unit (rebuilding: 66 instructions per word at q = 3, four words and 16 matrix-core
// instructions a step) once a step's loads are hidden, and the trips to memory at both ends.  465 vector instructions a step at
// q = 3, G = 64, which two wavefronts on a SIMD issue at five clocks each: 2.2 us for each 1024 k of 4096 x 14336 and M = 24, and
// 6.7 us for the launch, its start and end.  Tiled kernel -> this one, us a call: 4096 x 14336, q = 3, G = 64, M = 24 19.8 -> 14.3;
// 4096 x 4096, q = 4, G = 64, M = 12 12.1 -> 9.8, q = 2, G = 128, M = 16 10.3 -> 8.2; 4096 x 1024, q = 2, M = 16 8.6 -> 7.4;
// 14336 x 4096, q = 3, M = 24 22 -> 17.3; 8B layer q = 4, G = 64, M = 16 62 -> 54, M = 32, G = 128 62 -> 54.
#include "hlq_gemm_safe.h"
#include "hlq_gemm_reduce.h"
#include "hlq_mfma_common.h"

#include <type_traits>

namespace {

typedef int int4v __attribute__((ext_vector_type(4)));
typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
typedef unsigned uint4a __attribute__((ext_vector_type(4), may_alias));
typedef _Float16 half8a __attribute__((ext_vector_type(8), may_alias));

constexpr int SHORT_WAVES = 8;

struct ShortProb {
    const char *packed;
    size_t col_bytes;
    const uint16_t *X;
    long ldx;
    void *Y;
    long ldy;
    float *part;          // [nslices][M][N] partial sums (nslices > 1)
    int N, ntiles, nchunks, cps, nslices, blk_begin;
    unsigned ns_magic;    // ceil(2^32 / nslices): local / nslices = umulhi(local, ns_magic)
};
struct ShortProbs {
    ShortProb p[HLQ_MAX_BATCH];
};

// LDS, for calls of up to MR rows (16 or 32): X of a wavefront's chunk; the wavefronts' results take its place at the end
constexpr int short_x_bytes(int MR) { return MR * 256; }
static_assert(short_x_bytes(1) == 64 * 4, "a row of 128 fp16 takes what a row of 64 fp32 results does");

__device__ __forceinline__ int short_problem_of(const int4v &bb_lo, const int4v &bb_hi, int blk)
{
    return blk >= bb_hi.w ? 7 : blk >= bb_hi.z ? 6 : blk >= bb_hi.y ? 5 : blk >= bb_hi.x ? 4
         : blk >= bb_lo.w ? 3 : blk >= bb_lo.z ? 2 : blk >= bb_lo.y ? 1 : 0;
}

template <int Q, int G, int MR>
__global__ void __launch_bounds__(64 * SHORT_WAVES)
hlq_gemm_short_kernel(const int4v bb_lo, const int4v bb_hi, const int M, const int out_f32, int *range_flag, const ShortProbs probs)
{
    constexpr int GS = G < 128 ? G : 128, SEG = 128 / GS;
    __shared__ __attribute__((aligned(256))) char lds[SHORT_WAVES * short_x_bytes(MR)];
    const int blk = (int)blockIdx.x;
    const ShortProb P = probs.p[short_problem_of(bb_lo, bb_hi, blk)];
    const int local = blk - P.blk_begin;
    const int tile = P.nslices > 1 ? (int)__umulhi((unsigned)local, P.ns_magic) : local;
    const int slice = local - tile * P.nslices;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int tw = hlq_tile_width(tile, P.N);
    const char *tile_base = P.packed + (size_t)tile * HLQ_TILE_N * P.col_bytes;

    // this wavefront's chunks [c0, c0 + steps) of the slice
    const int sbeg = slice * P.cps, len = min(P.cps, P.nchunks - sbeg);
    const int c0 = sbeg + len * wave / SHORT_WAVES, steps = sbeg + len * (wave + 1) / SHORT_WAVES - c0;

    // ---- loads.  No branch around one (what is waited for would no longer be known): weights through a descriptor that ends
    // with this wavefront's chunks, X of the last chunk again.  Columns past the tile's width re-read its last ones and are
    // dropped at the end.
    struct Regs {
        uint32_t w[Q][4];
        uint32_t mt[SEG][Q + 1];   // parameters of two columns, this lane's at bit `mshift` (a 16-bit load would be extended
                                   // right behind itself, i.e. waited for)
    };
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc((void *)tile_base, 0, (int)hlq_rec_in_tile(tw, c0 + steps, Q, G), 0x00020000);
    const uint32_t col = (uint32_t)min(lane, tw - 1), mshift = 16 * (col & 1);
    auto load_w = [&](int s, Regs &R) {
        const int ch = c0 + s;
        const uint32_t vo = col * 16u + hlq_rec_in_tile(tw, ch, Q, G);
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const int4v v = __builtin_bit_cast(int4v, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, (int)vo, j * tw * 16, 2));
            R.w[j][0] = v.x; R.w[j][1] = v.y; R.w[j][2] = v.z; R.w[j][3] = v.w;
        }
        // with 256-wide groups the parameters sit in the group's first (even) chunk
        const uint32_t mo = (col & ~1u) * 2u + hlq_rec_in_tile(tw, G > 128 ? ch & ~1 : ch, Q, G);
#pragma unroll
        for (int sg = 0; sg < SEG; ++sg)
#pragma unroll
            for (int r = 0; r <= Q; ++r)
                R.mt[sg][r] = __builtin_amdgcn_raw_buffer_load_b32(wrsrc, (int)mo, tw * Q * 16 + (sg * (Q + 1) + r) * tw * 2, 0);
    };
    // X: four rows an instruction (16 lanes a row); rows past M repeat the last
    constexpr int NX = MR / 4;
    uint4 xv[NX];
    const uint16_t *xsrc[NX];
#pragma unroll
    for (int i = 0; i < NX; ++i) xsrc[i] = P.X + (size_t)min(4 * i + (lane >> 4), M - 1) * P.ldx + 8 * (lane & 15);
    auto load_x = [&](int s) {
        const int at = min(c0 + s, P.nchunks - 1) * 128;
#pragma unroll
        for (int i = 0; i < NX; ++i) xv[i] = *(const uint4 *)(xsrc[i] + at);
    };
    char *const mine = lds + wave * short_x_bytes(MR);
    char *const xdst[2] = {mine + (lane >> 4) * 256 + (((lane & 15) ^ (lane >> 4)) << 4), mine + (lane >> 4) * 256 + (((lane & 15) ^ (4 + (lane >> 4))) << 4)};
    auto put_x = [&]() {
#pragma unroll
        for (int i = 0; i < NX; ++i) *(uint4a *)(xdst[i & 1] + i * 1024) = (uint4a){xv[i].x, xv[i].y, xv[i].z, xv[i].w};
    };

    Regs RA, RB;
    load_x(0);
    load_w(0, RA);
    __builtin_amdgcn_sched_barrier(0);
    put_x();
    load_x(1);
    load_w(1, RB);
    __builtin_amdgcn_sched_barrier(0);

    float16v acc[2];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[cb][r] = 0.f;
    ushort2v meta_max = {0, 0};

    // A fragments: lane l reads unit 4 d + 2 ks + (l >> 5) of row l & 31 (or its like among the MR: results dropped)
    const char *xrow[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) xrow[k] = mine + (lane & (MR - 1)) * 256 + ((((2 * k) | (lane >> 5)) ^ (lane & 7)) << 4);
    auto compute = [&](const Regs &R) {
#pragma unroll
        for (int sg = 0; sg < SEG; ++sg)
#pragma unroll
            for (int r = 0; r <= Q; ++r) meta_max = __builtin_elementwise_max(meta_max, __builtin_bit_cast(ushort2v, R.mt[sg][r] & 0x7fff7fffu));
        half8v a[8];   // k-steps of 16
#pragma unroll
        for (int n = 0; n < 8; ++n) a[n] = *(const half8a *)(xrow[n & 3] + (n >> 2) * 128);
        HlqRebuild<Q> rb;
        uint32_t wp[2][16];
        auto segment = [&](int sg) {
            uint32_t m[Q + 1];
#pragma unroll
            for (int r = 0; r <= Q; ++r) m[r] = R.mt[sg][r] >> mshift;
            rb.segment(m);
        };
        segment(0);
        rb.word(R.w, 0);
#pragma unroll
        for (int p = 0; p < 8; ++p) rb.pairs(p, wp[0][p], wp[0][p + 8]);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            if (d < 3) {
                if ((d + 1) * 32 % GS == 0) segment((d + 1) * 32 / GS);
                rb.word(R.w, d + 1);
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                // after the exchange lo holds columns 0..31 of the tile (k-slots 0..7 in lanes 0..31), hi columns 32..63
                uint4v lo, hi;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const uint2v r = __builtin_amdgcn_permlane32_swap(wp[d & 1][ks * 8 + v], wp[d & 1][ks * 8 + 4 + v], false, false);
                    lo[v] = r.x;
                    hi[v] = r.y;
                }
                __builtin_amdgcn_sched_barrier(0);
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[2 * d + ks], __builtin_bit_cast(half8v, lo), acc[0], 0, 0, 0);
                if (d < 3) {
#pragma unroll
                    for (int p = 4 * ks; p < 4 * ks + 2; ++p) rb.pairs(p, wp[(d + 1) & 1][p], wp[(d + 1) & 1][p + 8]);
                }
                __builtin_amdgcn_sched_barrier(0);
                acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[2 * d + ks], __builtin_bit_cast(half8v, hi), acc[1], 0, 0, 0);
                if (d < 3) {
#pragma unroll
                    for (int p = 4 * ks + 2; p < 4 * ks + 4; ++p) rb.pairs(p, wp[(d + 1) & 1][p], wp[(d + 1) & 1][p + 8]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // ---- steps: a step's X is in LDS when it begins, the next one's in registers, the weights of two steps ahead requested
    // as it ends
    auto step = [&](int s, Regs &R) {
        compute(R);
        __builtin_amdgcn_sched_barrier(0);
        put_x();
        load_x(s + 2);
        load_w(s + 2, R);
        __builtin_amdgcn_sched_barrier(0);
    };
    int s = 0;
    for (; s + 2 <= steps; s += 2) {
        step(s, RA);
        step(s + 1, RB);
    }
    if (s < steps) compute(RA);

    // ---- parameters out of range (also: not finite) ----------------------------------------------------------------------
    const bool out_of_range = __syncthreads_or(max(meta_max.x, meta_max.y) >= 0x6000);
    if (out_of_range) {
        if (P.nslices == 1) {
            HlqSafeProb sp;
            sp.packed = P.packed;
            sp.col_bytes = P.col_bytes;
            sp.X = P.X;
            sp.ldx = P.ldx;
            sp.Y = P.Y;
            sp.ldy = P.ldy;
            sp.N = P.N;
            sp.nchunks = P.nchunks;
            sp.q = Q;
            sp.G = G;
            for (int m0 = wave * SAFE_ROWS; m0 < M; m0 += SHORT_WAVES * SAFE_ROWS) hlq_safe_item(sp, tile, m0, M, out_f32);
            return;
        }
        if (tid == 0) __hip_atomic_store(range_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    // ---- add the parts, store.  Result register r of lane l is row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32; in LDS
    // [wavefront][register][column of the tile], lanes 32..63 behind lanes 0..31's registers
    float *red = (float *)lds;
    constexpr int regs = MR / 2;   // the others belong to rows past MR
#pragma unroll
    for (int r = 0; r < regs; ++r)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) red[((wave * 2 + (lane >> 5)) * regs + r) * 64 + 32 * cb + (lane & 31)] = acc[cb][r];
    __syncthreads();
    const int n = tid & 63;
    if (n >= tw) return;
    for (int m = tid >> 6; m < M; m += SHORT_WAVES) {
        const float *src = red + ((((m >> 2) & 1) * regs + 4 * (m >> 3) + (m & 3)) * 64 + n);
        float v = 0.f;
#pragma unroll
        for (int p = 0; p < SHORT_WAVES; ++p) v += src[p * 2 * regs * 64];
        const size_t at = (size_t)tile * HLQ_TILE_N + n;
        if (P.nslices > 1) P.part[((size_t)slice * M + m) * (size_t)P.N + at] = v;
        else if (out_f32) ((float *)P.Y)[(size_t)m * P.ldy + at] = v;
        else ((_Float16 *)P.Y)[(size_t)m * P.ldy + at] = (_Float16)v;
    }
}

// K slices: as many as give the launch one workgroup per place, of a chunk for each wavefront or more (but for the last: slices
// are even numbers of chunks, what is left may be less)
struct ShortPlan {
    int cps[HLQ_MAX_BATCH], nslices[HLQ_MAX_BATCH];
};
ShortPlan plan_short(int count, const HlqDims *dms, int64_t M)
{
    ShortPlan p;
    long units = 0;   // tile-chunks
    for (int i = 0; i < count; ++i) units += (long)dms[i].ntiles * dms[i].nchunks;
    long target = (units + 255) / 256;   // chunks of a workgroup
    if (target < SHORT_WAVES) target = SHORT_WAVES;
    for (int i = 0; i < count; ++i) {
        int ns = (int)(dms[i].nchunks / target);
        if (ns < 1) ns = 1;
        const int cps = (dms[i].nchunks + ns - 1) / ns;
        p.cps[i] = (cps + 1) & ~1;
        p.nslices[i] = (dms[i].nchunks + p.cps[i] - 1) / p.cps[i];
    }
    return p;
}

template <int Q>
hlq_status launch_short_q(int G, unsigned nblocks, const int4v &lo, const int4v &hi, int M, int out_f32, int *flag,
                          const ShortProbs &pr, hipStream_t st)
{
    auto launch = [&](auto g) {
        constexpr int GG = decltype(g)::value;
        if (M <= 16) hlq_gemm_short_kernel<Q, GG, 16><<<nblocks, 64 * SHORT_WAVES, 0, st>>>(lo, hi, M, out_f32, flag, pr);
        else hlq_gemm_short_kernel<Q, GG, 32><<<nblocks, 64 * SHORT_WAVES, 0, st>>>(lo, hi, M, out_f32, flag, pr);
    };
    switch (G) {
    case 32: launch(std::integral_constant<int, 32>{}); return HLQ_OK;
    case 64: launch(std::integral_constant<int, 64>{}); return HLQ_OK;
    case 128: launch(std::integral_constant<int, 128>{}); return HLQ_OK;
    case 256: launch(std::integral_constant<int, 256>{}); return HLQ_OK;
    }
    return HLQ_ERR_UNSUPPORTED;
}

} // namespace

size_t hlq_gemm_short_partial_bytes(int count, const HlqDims *dms, int64_t M)
{
    if (M < 1 || M > HLQ_SHORT_ROWS) return 0;
    const ShortPlan p = plan_short(count, dms, M);
    size_t b = 0;
    for (int i = 0; i < count; ++i)
        if (p.nslices[i] > 1) b += (size_t)p.nslices[i] * (size_t)M * (size_t)dms[i].N * sizeof(float);
    return b;
}

// One round of workgroups (256): always (0.44 to 1.05 of the tiled kernel's time).  More of them pay start and end of a workgroup per
// round, whatever the depth, where the tiled kernel has a quarter as many with four times the columns; which of the two
// is the longer time is estimated.  us, tiled / this one, M = 32, G = 64: 256 x 127976 q = 1 9.2 / 34.9,
// 1024 x 63976 12.3 / 19.3, 4096 x 63976 q = 2 44.6 / 47.9, q = 4 (M = 16) 61.4 / 56.9;  1024 x 19176 q = 2 12.2 / 10.6;  3072 x 28776 q = 2 21.5 / 19.8;
// 6144 x 38376 q = 1 31.2 / 38.3.  Over the calls the estimate was fitted to, 1 % from the better of the two on average, 23 % at most (this kernel
// always: 23 % and 4.5 times; profiles/gemm_rows_to_32_rules.txt).  From 80000 chunk-tiles on the tiled kernel: 86016 q = 2, M = 16 99.8 / 98.8, 128256 q = 2, M = 24 141 / 158.
bool hlq_gemm_short_wins(int count, const HlqDims *dms, int64_t M)
{
    if (M < 1 || M > HLQ_SHORT_ROWS) return false;
    const ShortPlan p = plan_short(count, dms, M);
    const double round = M > 16 ? 2.5 : 2.0, step = M > 16 ? 1.0 + 0.5 * dms[0].q : 0.8 + 0.47 * dms[0].q;   // us: a workgroup, and a chunk of each of its wavefronts
    long units = 0, blocks = 0;
    double work = 0, longest = 0, shortest = 1e30;
    bool sliced = false;
    for (int i = 0; i < count; ++i) {
        units += (long)dms[i].ntiles * dms[i].nchunks;
        const long n = (long)dms[i].ntiles * p.nslices[i];
        const int chunks = p.cps[i] < dms[i].nchunks ? p.cps[i] : dms[i].nchunks;
        const double t = round + step * ((chunks + SHORT_WAVES - 1) / SHORT_WAVES);
        blocks += n;
        work += (double)n * t;
        longest = t > longest ? t : longest;
        shortest = t < shortest ? t : shortest;
        sliced = sliced || p.nslices[i] > 1;
    }
    if (units >= 80000) return false;
    if (blocks <= 256) return true;
    double t = count == 1 ? (double)((blocks + 255) / 256) * longest : work / 256 + 0.5 * shortest;
    t = 1.3 + (t > longest ? t : longest) + (sliced ? 2.9 : 0.0);
    return hlq_gemm_mfma_estimate(count, dms, M) >= (dms[0].q == 1 ? 1.03 : 0.93) * t;   // (the estimates are good to 9 %)
}

hlq_status hlq_launch_gemm_short(int count, const HlqGemvItem *items, int64_t M, hlq_out_dtype out, void *ws, hipStream_t st)
{
    static_assert(HLQ_MAX_BATCH == 8, "the kernel takes the first blocks of eight problems");
    hlq_clear_stale_error();
    if (count < 1 || count > HLQ_MAX_BATCH || M < 1 || M > HLQ_SHORT_ROWS) return HLQ_ERR_UNSUPPORTED;
    // workgroups start in block order: long-K problems first
    int order[HLQ_MAX_BATCH];
    for (int i = 0; i < count; ++i) order[i] = i;
    for (int i = 1; i < count; ++i)
        for (int j = i; j > 0 && items[order[j]].dm.nchunks > items[order[j - 1]].dm.nchunks; --j) {
            const int t = order[j];
            order[j] = order[j - 1];
            order[j - 1] = t;
        }
    HlqDims dms[HLQ_MAX_BATCH];
    for (int i = 0; i < count; ++i) dms[i] = items[order[i]].dm;
    const ShortPlan plan = plan_short(count, dms, M);
    const int out_f32 = out == HLQ_OUT_F32;
    ShortProbs pr;
    HlqReduce red(M, out_f32);
    int begin[HLQ_MAX_BATCH];
    long blk = 0;
    float *part = (float *)((char *)ws + HLQ_WS_COUNTER_BYTES);
    for (int i = 0; i < count; ++i) {
        const HlqGemvItem &it = items[order[i]];
        if (it.dm.q != items[0].dm.q || it.dm.G != items[0].dm.G) return HLQ_ERR_UNSUPPORTED;
        ShortProb &p = pr.p[i];
        p.packed = (const char *)it.packed;
        p.col_bytes = it.dm.col_bytes;
        p.X = it.x;
        p.ldx = it.ldx;
        p.Y = it.y;
        p.ldy = it.ldy;
        p.part = part;
        p.N = it.dm.N;
        p.ntiles = it.dm.ntiles;
        p.nchunks = it.dm.nchunks;
        p.cps = plan.cps[i];
        p.nslices = plan.nslices[i];
        p.ns_magic = p.nslices > 1 ? (unsigned)((0x100000000ULL + (unsigned)p.nslices - 1) / (unsigned)p.nslices) : 0u;
        const unsigned long long blocks = (unsigned long long)p.ntiles * p.nslices;
        if (blocks * p.nslices >= 0x100000000ULL) return HLQ_ERR_UNSUPPORTED;   // the reciprocal is exact below
        p.blk_begin = begin[i] = (int)blk;
        blk += (long)blocks;
        if (blk > 0x7fffffffL / 64) return HLQ_ERR_UNSUPPORTED;
        if (p.nslices > 1) {
            if (!red.add(part, it.y, it.ldy, it.dm.N, p.nslices)) return HLQ_ERR_UNSUPPORTED;
            part += (size_t)p.nslices * (size_t)M * (size_t)it.dm.N;
        }
    }
    for (int i = count; i < HLQ_MAX_BATCH; ++i) {
        pr.p[i] = pr.p[0];
        begin[i] = 0x7fffffff;
    }
    const int4v lo = {begin[0], begin[1], begin[2], begin[3]}, hi = {begin[4], begin[5], begin[6], begin[7]};
    hlq_status s;
    switch (items[0].dm.q) {
    case 1: s = launch_short_q<1>(items[0].dm.G, (unsigned)blk, lo, hi, (int)M, out_f32, hlq_ws_range_flag(ws), pr, st); break;
    case 2: s = launch_short_q<2>(items[0].dm.G, (unsigned)blk, lo, hi, (int)M, out_f32, hlq_ws_range_flag(ws), pr, st); break;
    case 3: s = launch_short_q<3>(items[0].dm.G, (unsigned)blk, lo, hi, (int)M, out_f32, hlq_ws_range_flag(ws), pr, st); break;
    case 4: s = launch_short_q<4>(items[0].dm.G, (unsigned)blk, lo, hi, (int)M, out_f32, hlq_ws_range_flag(ws), pr, st); break;
    default: return HLQ_ERR_UNSUPPORTED;
    }
    if (s != HLQ_OK) return s;
    if (red.count > 0) return hlq_launch_gemm_reduce(red, count, items, ws, st);
    return hlq_hip_status(hipGetLastError());
}
