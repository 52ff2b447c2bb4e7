// hlq_pack / hlq_unpack: the offline bit-plane decomposition (App. B) and weight
// re-arrangement (App. D, Weight-Rearrange) for the CDNA4 layout described in
// hlq_internal.h.  Integer work only; pack and unpack are exact inverses.
#include "hlq_internal.h"

namespace {

typedef unsigned int uint2v __attribute__((ext_vector_type(2)));

// One wavefront per record (tile, chunk): lane 16 d + c collects word d (32 k) of the columns 4 c .. 4 c + 3, so a row of
// codes is read as one 4-byte word per lane (codes4: the rows are 4-byte aligned; else byte by byte) and 32 loads of a
// lane are in flight at once.  The bits of a plane are gathered for the four columns together -- byte i of (row >> j) &
// 0x01010101 is column i's bit -- eight rows to a byte, and four byte permutes make the columns' words of that.  A 4 x 4
// transpose over (lane group, column) then gives every lane the 16 bytes of one column: 1 KiB stores.
// Bound by the latency of one pass over the codes; the earlier form, one thread per (chunk, column) with 128 byte loads
// in a row and a second launch for the scales, had a quarter of the wavefronts.  4096 x 14336, G = 64: q = 4 41.5 -> 25.8 us,
// q = 1 36.9 -> 18.9 us a call.
template <bool WIDE>
__global__ void __launch_bounds__(256)
hlq_pack_kernel(const uint8_t *__restrict__ codes, const uint16_t *__restrict__ scales,
                const uint16_t *__restrict__ zeros, char *__restrict__ packed, int N, int ntiles, size_t col_bytes,
                int ngroups, int q, int G)
{
    const int tile = blockIdx.x * 4 + (threadIdx.x >> 6), c = blockIdx.y, lane = threadIdx.x & 63;
    if (tile >= ntiles) return;
    const int tw = hlq_tile_width(tile, N), n0 = tile * HLQ_TILE_N;
    const int cq = lane & 15, d = lane >> 4;
    char *rec = packed + hlq_rec_off(col_bytes, tile, tw, c, q, G);
    // lanes past the tile's width (a multiple of 8) read its last columns again and store nothing
    const int col = 4 * cq < tw ? 4 * cq : tw - 4;
    const uint8_t *src = codes + (size_t)(c * HLQ_CHUNK_K + 32 * d) * N + n0 + col;
    uint32_t x[32];
#pragma unroll
    for (int b = 0; b < 32; ++b) {
        const uint8_t *row = src + (size_t)b * N;
        if constexpr (WIDE) x[b] = *(const uint32_t *)row;
        else x[b] = (uint32_t)row[0] | (uint32_t)row[1] << 8 | (uint32_t)row[2] << 16 | (uint32_t)row[3] << 24;
    }
    // scales and zeros of the groups that start in this chunk: lane <-> column
    if (lane < tw) {
        const int g0 = hlq_groups_before(c, G), g1 = hlq_groups_before(c + 1, G);
        uint16_t *meta = (uint16_t *)(rec + (size_t)tw * q * 16) + lane;
        for (int g = g0; g < g1; ++g) {
            for (int r = 0; r < q; ++r) meta[((g - g0) * (q + 1) + r) * tw] = scales[((size_t)r * ngroups + g) * N + n0 + lane];
            meta[((g - g0) * (q + 1) + q) * tw] = zeros[(size_t)g * N + n0 + lane];
        }
    }
    for (int j = 0; j < q; ++j) {
        // byte b8 of a word: bits 8 b8 .. 8 b8 + 7, i.e. the even (b8 < 2) or odd k of half a block (hlq_bit_pos)
        uint32_t by[4];
#pragma unroll
        for (int b8 = 0; b8 < 4; ++b8) {
            by[b8] = 0u;
#pragma unroll
            for (int s = 0; s < 8; ++s) by[b8] |= ((x[16 * (b8 & 1) + 2 * s + (b8 >> 1)] >> j) & 0x01010101u) << s;
        }
        // word of column i = bytes i of by[0..3]
        const uint32_t p01lo = __builtin_amdgcn_perm(by[1], by[0], 0x05010400u), p01hi = __builtin_amdgcn_perm(by[1], by[0], 0x07030602u);
        const uint32_t p23lo = __builtin_amdgcn_perm(by[3], by[2], 0x05010400u), p23hi = __builtin_amdgcn_perm(by[3], by[2], 0x07030602u);
        const uint32_t w0 = __builtin_amdgcn_perm(p23lo, p01lo, 0x05040100u), w1 = __builtin_amdgcn_perm(p23lo, p01lo, 0x07060302u);
        const uint32_t w2 = __builtin_amdgcn_perm(p23hi, p01hi, 0x05040100u), w3 = __builtin_amdgcn_perm(p23hi, p01hi, 0x07060302u);
        const uint2v s01 = __builtin_amdgcn_permlane16_swap(w0, w1, false, false);
        const uint2v s23 = __builtin_amdgcn_permlane16_swap(w2, w3, false, false);
        const uint2v t02 = __builtin_amdgcn_permlane32_swap(s01.x, s23.x, false, false);
        const uint2v t13 = __builtin_amdgcn_permlane32_swap(s01.y, s23.y, false, false);
        // lane 16 d + c now holds words 0..3 of column 4 c + d
        if (4 * cq < tw) ((uint4 *)rec)[j * tw + 4 * cq + d] = make_uint4(t02.x, t13.x, t02.y, t13.y);
    }
}

__global__ void __launch_bounds__(256)
hlq_unpack_bits_kernel(const char *__restrict__ packed, uint8_t *__restrict__ codes, int N,
                       size_t col_bytes, int q, int G)
{
    const int n = blockIdx.x * 256 + threadIdx.x;
    const int c = blockIdx.y;
    if (n >= N) return;
    uint32_t w[4][4];
    const int tile = n / HLQ_TILE_N, lane = n % HLQ_TILE_N, tw = hlq_tile_width(tile, N);
    const uint4 *rec = (const uint4 *)(packed + hlq_rec_off(col_bytes, tile, tw, c, q, G));
    for (int j = 0; j < 4; ++j) {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (j < q) v = rec[j * tw + lane];
        w[j][0] = v.x; w[j][1] = v.y; w[j][2] = v.z; w[j][3] = v.w;
    }
    uint8_t *dst = codes + (size_t)c * HLQ_CHUNK_K * N + n;
    for (int d = 0; d < 4; ++d) {
        for (int b = 0; b < 32; ++b) {
            uint32_t code = 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) code |= ((w[j][d] >> hlq_bit_pos(b)) & 1u) << j;
            dst[(size_t)(32 * d + b) * N] = (uint8_t)code;
        }
    }
}

// Address of the fp16 slot (group g, row r, column n) inside the record of the chunk in which
// group g starts.
__device__ __forceinline__ size_t meta_slot(size_t col_bytes, int N, int q, int G, int g, int r, int n)
{
    const int tile = n / HLQ_TILE_N, lane = n % HLQ_TILE_N, tw = hlq_tile_width(tile, N);
    const int c = (int)(((long)g * G) / HLQ_CHUNK_K);
    const int s = g - hlq_groups_before(c, G);
    return hlq_rec_off(col_bytes, tile, tw, c, q, G) + (size_t)tw * q * 16 +
           ((size_t)(s * (q + 1) + r) * tw + lane) * 2;
}

// scales / zeros <- record meta
__global__ void __launch_bounds__(256)
hlq_unpack_meta_kernel(const char *__restrict__ packed, uint16_t *__restrict__ scales,
                       uint16_t *__restrict__ zeros, int N, size_t col_bytes, int ngroups, int q, int G)
{
    const int n = blockIdx.x * 256 + threadIdx.x;
    const int g = blockIdx.y;
    if (n >= N) return;
    if (scales)
        for (int r = 0; r < q; ++r)
            scales[((size_t)r * ngroups + g) * N + n] =
                *(const uint16_t *)(packed + meta_slot(col_bytes, N, q, G, g, r, n));
    if (zeros) zeros[(size_t)g * N + n] = *(const uint16_t *)(packed + meta_slot(col_bytes, N, q, G, g, q, n));
}

} // namespace

hlq_status hlq_launch_pack(const HlqDims &dm, const uint8_t *codes, const uint16_t *scales,
                           const uint16_t *zeros, void *packed, hipStream_t st)
{
    hlq_clear_stale_error();
    const dim3 grid((unsigned)((dm.ntiles + 3) / 4), (unsigned)dm.nchunks);
    if (((uintptr_t)codes & 3u) == 0)   // N is a multiple of 8: every row is aligned if the first is
        hlq_pack_kernel<true><<<grid, 256, 0, st>>>(codes, scales, zeros, (char *)packed, dm.N, dm.ntiles, dm.col_bytes, dm.ngroups, dm.q, dm.G);
    else
        hlq_pack_kernel<false><<<grid, 256, 0, st>>>(codes, scales, zeros, (char *)packed, dm.N, dm.ntiles, dm.col_bytes, dm.ngroups, dm.q, dm.G);
    return hlq_hip_status(hipGetLastError());
}

hlq_status hlq_launch_unpack(const HlqDims &dm, const void *packed, uint8_t *codes,
                             uint16_t *scales, uint16_t *zeros, hipStream_t st)
{
    hlq_clear_stale_error();
    const unsigned ntiles = (unsigned)((dm.N + 255) / 256);
    if (codes)
        hlq_unpack_bits_kernel<<<dim3(ntiles, dm.nchunks), 256, 0, st>>>((const char *)packed, codes, dm.N, dm.col_bytes,
                                                                         dm.q, dm.G);
    if (scales || zeros)
        hlq_unpack_meta_kernel<<<dim3(ntiles, dm.ngroups), 256, 0, st>>>((const char *)packed, scales, zeros, dm.N,
                                                                         dm.col_bytes, dm.ngroups, dm.q, dm.G);
    return hlq_hip_status(hipGetLastError());
}
