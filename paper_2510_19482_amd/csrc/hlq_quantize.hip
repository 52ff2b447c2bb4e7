// hlq_quantize: Alg. 1 (Sec. 4.1, "Alternating Optimization for Hierarchical Linear Quantization"; its two steps are
// defined in Sec. 4.2 under "Bit-Pattern Selection" and "Linear Reconstruction") --
// produces the codes, per-plane scales and zero points that hlq_pack consumes.
//
//   per group of G consecutive k of a column:  Delta = (max - min) / (2^q - 1),
//   s = [Delta, 2 Delta, ...], z = min;  then T_max times
//     bit-pattern selection   code = argmin_c | (w - z) - sum_j s_j bit_j(c) |      (Bit-Pattern Selection)
//     linear reconstruction   (s, z) = least squares of w ~ sum_j s_j b_j + z        (Linear Reconstruction, LSE)
//
// Groups are independent (App. C), so the unit of work is one lane = one (group, column), or two or four neighbouring lanes
// that take consecutive parts of the group: as many as a launch needs to have a wavefront on every SIMD, and at
// least two for groups of 256, whose weights would not fit one lane's registers.  The lanes of a group add their counts and sums
// and make the same thresholds and parameters.  A lane
// reads its weights once, into registers (G / L fp32 values; lanes of a wavefront hold adjacent
// columns, so each load is a coalesced read of a row of W (of L rows) and all are in
// flight together), and every later step works from there: W is read from HBM exactly once and the
// kernel is bound by vector instruction issue.  Within
// a pass a weight's code is chosen and immediately folded into the sums the least-squares step
// needs -- the integer Gram matrix of [1 b_0 .. b_{q-1}] and the fp64 right-hand side -- so nothing
// per weight is stored until the last iteration writes the codes.  All arithmetic is fp64: the
// step is offline, and decisions (the argmin) then agree with an fp64 reference except at exact
// ties.
//
// Rank-deficient systems (a plane constant over the group, equal or complementary planes, all
// weights equal): columns are taken in the order 1, b_0, b_1, ...; a column that depends linearly on
// the earlier ones keeps its previous parameter, whose contribution moves to the right-hand side.
// Dependence among the columns is a property of the SET of codes present in the group, so it is
// decided exactly on the small integer Gram matrix of the distinct rows [1 bits(c)] (entries <= 16):
// fraction-free elimination in column order, in which a zero pivot (the Gram determinant of the
// independent columns so far plus this one) marks a dependent column, which is then skipped.
// Every loop below has compile-time bounds and indices, so all of this lives in registers (and the tables of the search in
// LDS); none of it in scratch memory.
#include "hlq_internal.h"
#include <type_traits>

#pragma clang fp contract(off)

namespace {

// ascending odd-even merge sort of NC keys (a power of two), all comparisons at compile-time positions
template <int NC>
__device__ __forceinline__ void sort_keys(uint32_t (&key)[NC])
{
#pragma unroll
    for (int p = 1; p < NC; p *= 2)
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int j = k % p; j + k < NC; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (i + j + k < NC && (i + j) / (2 * p) == (i + j + k) / (2 * p)) {
                        const uint32_t a = key[i + j], b = key[i + j + k];
                        key[i + j] = min(a, b);
                        key[i + j + k] = max(a, b);
                    }
}

// wavefronts on a SIMD that the registers have to leave room for (a lane keeps G weights; launches with several lanes a group
// have four at most)
constexpr int quantize_waves(int q, int G, int L)
{
    return G == 32 ? (q == 1 ? (L > 1 ? 6 : 7) : q == 2 ? 5 : q == 3 ? 4 : 3) : G == 128 ? (q == 1 ? 3 : 2) : q <= 2 ? 4 : 3;
}

// Bit-pattern selection.  The codes are the argmin over 2^q candidate distances, computed in fp64, first minimum in
// code order; scanning them costs 4 x 2^q vector instructions per weight and round.  With the candidate values sorted,
// only the two neighbours of a weight compete, and which of them wins is monotone in the weight, so there is an exact
// fp32 number T at which the choice changes: the smallest fp32 weight for which the upper neighbour wins.  The 2^q - 1
// thresholds are made once per group and round, and a weight's code is then a binary search: q fp32 comparisons.
// What makes T exact (tests compare every code with the scan's):
//   - sorted neighbours at least 2^-40 S apart, S the scale of the group's numbers: all fp64 roundings together stay
//     below 2^-50 S, so only neighbours compete and the choice between them is monotone;
//   - with m the midpoint in fp64 (error below 2^-48 S) and t its rounding to fp32: where |t - m| > 2^-45 S the sign of
//     t - m decides for t, and the next fp32 number on the other side is on the other side of m as well; otherwise
//     the two distances of t and of that neighbour are compared as the scan compares them;
//   - where both of them fall on one side (a midpoint at or near zero: every group with min = -max, i.e. 0.9 % of the groups
//     and 43 % of the wavefronts for N(0, s) weights in bf16) T is found by bisection over the fp32 numbers.
// A group whose weights are all equal (padded or pruned columns) has equal candidates in every round; it takes code 0.
// A lane that meets none of this (candidates that coincide up to rounding: groups of few distinct values) sends its
// wavefront through the scan for that round, and for the ones after it.
// The first two levels of the search have their thresholds in registers, the others read them from a lane-private LDS
// column, in ascending order (the number of thresholds passed so far is the address); a second column holds, per sorted
// position, a word with byte j = 0x3f where the code has bit j: moved to the top of the high half of a double it is 2^-15,
// the factor with which the weight enters plane j's sum (the sums are kept times 2^-15: every product and rounding is the
// one without the factor).  Codes are counted in a third.
// Per weight and round 11 vector instructions at q = 2 and 25 at q = 4, instead of 27 and about 110 for a scan with counts.
// 4096 x 4096, ten rounds, q = 1 / 2 / 3 / 4, us, all rounds by scan -> search, by the weights' distribution:
//   G = 128  fp32 normals         77 / 146 / 266 / 491 -> 50 / 89 / 129 / 181
//            rounded to bf16      77 / 146 / 266 / 491 -> 52 / 91 / 131 / 182
//            a zero column in 64  77 / 146 / 267 / 490 -> 51 / 90 / 131 / 184
//            -1, 0, 1 times 0.03  77 / 146 / 266 / 488 -> 52 / 132 / 220 / 383 (scan from the second or third round on)
//   G = 32   fp32 normals         73 / 142 / 270 / 491 -> 50 / 106 / 163 / 272;  -1, 0, 1: 67 / 142 / 268 / 481 -> 58 / 149 / 233 / 435
//   G = 256                      166 / 686 / 829 / 949 -> 49 / 87 / 124 / 175 (by one lane a group, from the L2 every round, 127 / 155 / 201 / 255)
template <int Q, int G, int L>
__global__ void __launch_bounds__(256, quantize_waves(Q, G / L, L))
hlq_quantize_kernel(const float *__restrict__ W, int K, int N, int t_max, int scan_first, uint8_t *__restrict__ codes,
                    uint16_t *__restrict__ scales, uint16_t *__restrict__ zeros, float *__restrict__ group_err)
{
    constexpr int GL = G / L;   // weights of a lane
    constexpr int NC = 1 << Q, P = Q + 1, QUARTER = NC > 2 ? NC / 4 : 1;
    // few candidates: everything in registers.  At q = 2 the tables in LDS are 5 % faster on large matrices (G = 128 97 us
    // against 100), but with groups of 32 a small launch waits for them in every round (512 x 512: 25.6 us against 23.1)
    constexpr bool SMALL = Q == 1 || (Q == 2 && G == 32);
    __shared__ uint32_t lds[SMALL ? 1 : 4 * 3 * NC * 64];
    const unsigned n = (blockIdx.x * 256 + threadIdx.x) / L, part = threadIdx.x % L;   // column, and part of its group
    const int gi = (int)blockIdx.y;
    if (n >= (unsigned)N) return;
    const int ngroups = K / G;
    // the group's rows (at most 2^30 bytes: N <= 2^20) through descriptors: row i is a scalar offset and the lane's column a
    // vector one that never changes, where 64-bit addresses would take two vector registers per access in flight
    const __amdgpu_buffer_rsrc_t w_rows = __builtin_amdgcn_make_buffer_rsrc((void *)(W + (size_t)gi * G * N), 0, G * N * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t c_rows = __builtin_amdgcn_make_buffer_rsrc(codes + (size_t)gi * G * N, 0, G * N, 0x00020000);
    const int first_row = (int)(part * GL) * N;
    auto load_row = [&](int offset) -> float { return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(w_rows, (int)(n * 4) + first_row * 4, offset, 0)); };
    // as many rows as dst takes from row i on; the offset is a running sum (one scalar instruction a row)
    auto load_rows = [&](auto &dst, int i, int stride) {
        int offset = i * stride * 4;
#pragma unroll
        for (int u = 0; u < (int)(sizeof(dst) / sizeof(dst[0])); ++u) {
            dst[u] = load_row(offset);
            offset += stride * 4;
        }
    };
    // this lane's columns, one word every 64: thresholds in order | plane words by sorted position | counts.  The
    // second and third also hold the candidate values (fp64, by code) while the thresholds are made.
    uint32_t *const tree = lds + (SMALL ? 0 : (threadIdx.x >> 6) * (3 * NC * 64) + (threadIdx.x & 63));
    uint32_t *const plane = tree + NC * 64;
    uint32_t *const count = plane + NC * 64;

    float wv[GL];
    float lof, hif;   // Alg. 1 steps 2-3 (min / max are exact in fp32)
    double rw = 0.0;  // sum of the weights
    load_rows(wv, 0, N);
    lof = hif = wv[0];
    float least = fabsf(wv[0]);
#pragma unroll
    for (int i = 1; i < GL; ++i) {
        lof = wv[i] < lof ? wv[i] : lof;
        hif = wv[i] > hif ? wv[i] : hif;
        least = fminf(least, fabsf(wv[i]));
    }
    // the lanes of a group are neighbours: l apart is a permutation of four
    auto across = [](uint32_t v, auto l) -> uint32_t { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(l)::value == 1 ? 0xB1 : 0x4E, 0xf, 0xf, false); };
    auto add_parts = [&](double v) -> double {
        unrolled<(L == 4 ? 2 : L == 2 ? 1 : 0)>([&](auto k) {
            const std::integral_constant<int, 1 + decltype(k)::value> l;
            const uint64_t b = __builtin_bit_cast(uint64_t, v);
            v += __builtin_bit_cast(double, (uint64_t)across((uint32_t)(b >> 32), l) << 32 | across((uint32_t)b, l));
        });
        return v;
    };
    if constexpr (L > 1) {
        unrolled<(L == 4 ? 2 : 1)>([&](auto k) {
            const std::integral_constant<int, 1 + decltype(k)::value> l;
            const float lo2 = __builtin_bit_cast(float, across(__builtin_bit_cast(uint32_t, lof), l)), hi2 = __builtin_bit_cast(float, across(__builtin_bit_cast(uint32_t, hif), l));
            lof = lo2 < lof ? lo2 : lof;
            hif = hi2 > hif ? hi2 : hif;
            least = fminf(least, __builtin_bit_cast(float, across(__builtin_bit_cast(uint32_t, least), l)));
        });
    }
    const float largest = fmaxf(fabsf(lof), fabsf(hif));
    // The number of lanes of a group depends on the size of the launch; its results do not, since its sums are exact in fp64 and
    // so the same in any order.  fp32 weights down to 2^-21 of the largest are so as they are.  Where some (not zero) are
    // smaller, all are rounded to multiples of 2^-52 of a power of two that no sum of magnitudes exceeds: a change, by less
    // than fp64 sums are rounded by, in weights below 2^-21 of the largest.  (One number in ten million of a normal distribution.)
    double unit = 0.0;   // adding and subtracting it rounds
    auto in_units = [&](float w) -> float { return (float)(((double)w + unit) - unit); };
    if constexpr (G > 32) {
        if (__builtin_expect(__any(least < largest * 0x1p-21f), 0)) {
            least = __builtin_inff();
#pragma unroll
            for (int i = 0; i < GL; ++i) least = wv[i] != 0.f ? fminf(least, fabsf(wv[i])) : least;
            if constexpr (L > 1) unrolled<(L == 4 ? 2 : 1)>([&](auto k) { least = fminf(least, __builtin_bit_cast(float, across(__builtin_bit_cast(uint32_t, least), std::integral_constant<int, 1 + decltype(k)::value>{}))); });
            constexpr int LOG_G = G == 64 ? 6 : G == 128 ? 7 : 8;
            const int above = (int)(__builtin_bit_cast(uint32_t, largest) >> 23) - 126 + LOG_G;
            if (least < largest * 0x1p-21f && largest < __builtin_inff()) unit = __builtin_bit_cast(double, (uint64_t)(1023 + above) << 52 | 1ull << 51);
            if (__any(unit != 0.0)) {
#pragma unroll
                for (int i = 0; i < GL; ++i) {
                    asm volatile("" : "+v"(wv[i]));
                    wv[i] = in_units(wv[i]);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < GL; ++i) rw += (double)wv[i];
    rw = add_parts(rw);
    auto weight = [&](int i) -> float {
        // opaque to the optimiser, so the fp64 copies are made per use instead of being kept
        // for the whole kernel (which would double the registers held)
        asm volatile("" : "+v"(wv[i]));
        return wv[i];
    };
    const double lo = (double)lof, hi = (double)hif;
    const double delta = (hi - lo) / (double)(NC - 1);
    const bool constant = lof == hif && rw - rw == 0.0;   // all weights equal (and no NaN among them)
    double theta[P];   // theta[0] = z, theta[1 + j] = s_j
    theta[0] = lo;
#pragma unroll
    for (int j = 0; j < Q; ++j) theta[1 + j] = delta * (double)(1 << j);

    // Rounds in a row that needed the scan: a wavefront stays with it after STAY of them (data of few distinct values needs
    // it in every round: without this -1, 0, 1 at q = 2, G = 32 takes 226 us and not 149).  At q = 4 a single one can
    // be a coincidence, candidates closer than the keys' 19 bits tell apart.
    constexpr int STAY = Q == 4 ? 2 : 1;
    int scans = scan_first ? STAY : 0;
    // one iteration of Alg. 1; the last one also stores the codes (a separate instantiation: a test per weight costs more)
    auto iteration = [&](auto last_c) {
        constexpr bool last = decltype(last_c)::value;
        int stride = N;   // of rows; an opaque copy: the multiples of N that the first loads took are not kept for later
        asm volatile("" : "+s"(stride));
        const double z = theta[0];
        double S = (double)largest + fabs(z);
#pragma unroll
        for (int j = 0; j < Q; ++j) S += fabs(theta[1 + j]);
        // a group whose weights are all equal has equal candidates in every round and takes code 0: its thresholds are NaN
        const double gap_min = constant ? -1.0 : S * 0x1p-40, band = fmax(S * 0x1p-45, 0x1p-149);
        const double zt = constant ? (double)__builtin_inff() : z;

        uint32_t key[NC];
        float top[3];   // the thresholds at the quarters (q = 1: the only one); the others are in LDS
        // through readfirstlane, here and below: the optimiser takes the choice for a scalar one (otherwise it keeps the
        // registers of both ways at once) and makes no copy of the round for each value
        scans = __builtin_amdgcn_readfirstlane(scans);
        int chosen = scans >= STAY;
        if (chosen == 0) {
            // candidate values V_c = sum_j s_j bit_j(c)   (step 7), sorted by the leading bits of their fp32 rounding with
            // the code in the last q bits (an order that is not the fp64 one shows as a gap below gap_min)
            double sorted[SMALL ? NC : 1];   // SMALL: sorted as they are, with their codes as keys
            unrolled<NC>([&](auto cc) {
                constexpr int c = decltype(cc)::value;
                double v = 0.0;
#pragma unroll
                for (int j = 0; j < Q; ++j) v += theta[1 + j] * (double)((c >> j) & 1);
                if constexpr (SMALL) {
                    sorted[c] = v;
                    key[c] = (uint32_t)c;
                } else {
                    const uint64_t b = __builtin_bit_cast(uint64_t, v);
                    plane[(2 * c) * 64] = (uint32_t)b;
                    plane[(2 * c + 1) * 64] = (uint32_t)(b >> 32);
                    const uint32_t u = __builtin_bit_cast(uint32_t, (float)v);
                    key[c] = ((u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u)) & ~(uint32_t)(NC - 1)) | (uint32_t)c;
                }
            });
            if constexpr (SMALL) {
                auto order = [&](int a, int b) {
                    const bool swap = sorted[b] < sorted[a];
                    const double va = sorted[a], vb = sorted[b];
                    const uint32_t ca = key[a], cb = key[b];
                    sorted[a] = swap ? vb : va;
                    sorted[b] = swap ? va : vb;
                    key[a] = swap ? cb : ca;
                    key[b] = swap ? ca : cb;
                };
                if constexpr (NC == 2) {
                    order(0, 1);
                } else {
                    order(0, 1);
                    order(2, 3);
                    order(0, 2);
                    order(1, 3);
                    order(1, 2);
                }
            } else {
                sort_keys<NC>(key);
            }
            auto value_of = [&](uint32_t at) -> double { return __builtin_bit_cast(double, ((uint64_t)plane[at + 64] << 32) | plane[at]); };
            auto value_at = [&](int i) -> double {   // of sorted position i
                if constexpr (SMALL) return sorted[i];
                else return value_of((key[i] & (NC - 1)) * 128);
            };
            // The threshold between two neighbours (candidate values below and above; tie: the upper one's code is the smaller)
            // whose midpoint is so close to zero that fp32 numbers are denser there than the distances are exact.  Whether
            // the upper one wins, as the scan decides it, is still monotone in the weight, so the smallest fp32 number for
            // which it does is found by bisection.  The decision changes at multiples of half an fp64 unit of the numbers
            // involved: the midpoint plus small multiples of 2^-57 S are tried first, then the fp32 numbers beside the two
            // that remain, and what is still open after that is halved to the end.  open: the lane has such a threshold.
            auto bisect = [&](double below, double above, bool tie, bool open) -> float {
                auto upper_wins = [&](float w) {
                    const double what = (double)w - z;
                    const double da = fabs(what - below), db = fabs(what - above);
                    return db < da || (db == da && tie);
                };
                auto to_key = [](float f) -> int32_t {   // fp32 numbers in ascending order
                    const int32_t b = __builtin_bit_cast(int32_t, f);
                    return b ^ (b >> 31 & 0x7fffffff);
                };
                auto at_key = [](int32_t k) -> float { return __builtin_bit_cast(float, k ^ (k >> 31 & 0x7fffffff)); };
                const double mid = (double)(float)(0.5 * (below + above) + z);
                const double unit = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, S) & 0x7ff0000000000000u) * 0x1p-57;
                auto multiple = [&](int k) -> float { return (float)(mid + (double)k * unit); };
                int kl = -256, kh = 256;
                const bool inside = !upper_wins(multiple(kl)) && upper_wins(multiple(kh));
#pragma unroll 1
                for (int s = 0; s < 9; ++s) {
                    const int k = (kl + kh) >> 1;
                    const bool up = upper_wins(multiple(k));
                    kl = up ? kl : k;
                    kh = up ? k : kh;
                }
                // (no such multiple: all numbers up to S, beyond which no weight lies)
                int32_t below_k = to_key(inside ? multiple(kl) : -(float)S), above_k = to_key(inside ? multiple(kh) : (float)S);
                above_k = above_k == 0 ? -1 : above_k;   // both zeros are the same weight
                const bool first = upper_wins(at_key(below_k + 1)), second = upper_wins(at_key(above_k - 1));
                const int32_t lower = below_k + 1;
                below_k = first ? below_k : second ? lower : above_k - 1;
                above_k = first ? lower : second ? above_k - 1 : above_k;
#pragma unroll 1
                for (int s = 0; s < 32 && __any(open && (uint32_t)above_k - (uint32_t)below_k > 1u); ++s) {
                    const int32_t half = (below_k & above_k) + ((below_k ^ above_k) >> 1);
                    const bool up = upper_wins(at_key(half));
                    below_k = up ? below_k : half;
                    above_k = up ? half : above_k;
                }
                return at_key(above_k);
            };
            bool good = true;
            uint32_t hard = 0u;   // the threshold that is left to the bisection below: position, codes of the two sides
            double va = value_at(0);
            unrolled<NC - 1>([&](auto ii) {
                constexpr int i = decltype(ii)::value + 1;
                const uint32_t ca = key[i - 1] & (NC - 1), cb = key[i] & (NC - 1);
                const double vb = value_at(i);
                good = good && vb - va >= gap_min;
                const double m = 0.5 * (va + vb) + zt;
                const float t = (float)m;
                const double off = (double)t - m;
                bool upper = off > 0.0;   // the upper neighbour wins at t
                const uint32_t tb = __builtin_bit_cast(uint32_t, t);
                const uint32_t away = (int32_t)tb < 0 ? ~0u : 1u;   // one fp32 step up (away: in bits)
                const float next = __builtin_bit_cast(float, tb + away);
                const bool near = fabs(off) <= band;
                bool found = false;
                float bisected = 0.f;
                if (__any(near)) {   // in the first round mostly: the middle of the grid is an fp32 number
                    const float prev = __builtin_bit_cast(float, tb - away);
                    auto upper_wins = [&](float w) {
                        const double what = (double)w - z;
                        const double da = fabs(what - va), db = fabs(what - vb);
                        return db < da || (db == da && cb < ca);
                    };
                    const bool at_t = upper_wins(t);
                    const bool beside = upper_wins(at_t ? prev : next);
                    upper = near ? at_t : upper;
                    const bool open = near && (t == 0.f || at_t == beside);
                    if (__builtin_expect(__any(open), 0)) {
                        if constexpr (Q == 1) {
                            bisected = bisect(va, vb, cb < ca, open);
                            found = open;
                        } else {
                            good = good && !(open && hard);   // a second one
                            hard = open ? (uint32_t)i | ca << 8 | cb << 16 : hard;
                        }
                    }
                }
                float T = upper ? t : next;
                if constexpr (Q == 1) T = found ? bisected : T;
                if constexpr (i % QUARTER == 0) top[i / QUARTER - 1] = T;
                else tree[i * 64] = __builtin_bit_cast(uint32_t, T);
                va = vb;
            });
            if constexpr (Q > 1) {
                if (__builtin_expect(__any(hard != 0u), 0)) {
                    const uint32_t at = hard & 0xffu, code_below = hard >> 8 & 0xffu, code_above = hard >> 16;
                    double below, above;
                    if constexpr (SMALL) {
                        below = sorted[0];
                        above = sorted[1];
#pragma unroll
                        for (int i = 2; i < NC; ++i) {
                            below = at == (uint32_t)i ? sorted[i - 1] : below;
                            above = at == (uint32_t)i ? sorted[i] : above;
                        }
                    } else {
                        below = value_of(code_below * 128);
                        above = value_of(code_above * 128);
                    }
                    const float T = bisect(below, above, code_above < code_below, hard != 0u);
#pragma unroll
                    for (int k = 0; k < 3; ++k) top[k] = at == (uint32_t)((k + 1) * QUARTER) ? T : top[k];
                    if constexpr (NC > 4)
                        if (at) tree[at * 64] = __builtin_bit_cast(uint32_t, T);
                }
            }
            chosen = __any(!good) ? 1 : 0;
        } else {
#pragma unroll
            for (int i = 0; i < NC; ++i) key[i] = (uint32_t)i;   // (not used)
        }
        chosen = __builtin_amdgcn_readfirstlane(chosen);
        const bool scan = chosen != 0;
        scans = scan ? scans + 1 : 0;

        // per sorted position: the plane word; counts start at zero
        uint32_t words[SMALL ? NC : 1];
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const uint32_t c = key[i] & (NC - 1);
            const uint32_t ones = __umul24(c, 0x204081u) & 0x01010101u;   // bit j of the code in byte j
            if constexpr (SMALL) {
                words[i] = (ones << 6) - ones;
            } else {
                plane[i * 64] = (ones << 6) - ones;
                count[i * 64] = 0u;
            }
        }
        int cnt[NC];   // SMALL, until the pass is over: weights at or above threshold i (position i and higher)
#pragma unroll
        for (int i = 0; i < NC; ++i) cnt[i] = 0;
        double rb[Q];
#pragma unroll
        for (int j = 0; j < Q; ++j) rb[j] = 0.0;
        // folds weight i, whose plane word has been read, into the sums
        auto fold = [&](int i, float w, uint32_t word) {
            const double wd = (double)w;
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                const uint32_t hi32 = __builtin_amdgcn_perm(0u, word, ((uint32_t)j << 24) | 0x0c0c0cu);
                rb[j] = __builtin_fma(__builtin_bit_cast(double, (uint64_t)hi32 << 32), wd, rb[j]);   // exact product: same rounding as an add
            }
            if constexpr (last) {
                uint32_t c = 0;
#pragma unroll
                for (int j = 0; j < Q; ++j) c |= ((word >> (8 * j)) & 1u) << j;
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)c, c_rows, (int)n + first_row, i * stride, 0);
            }
        };
        if (__builtin_expect(!scan, 1) && SMALL) {
            // a comparison per threshold; its outcome picks the plane word and is counted
            auto take = [&](int i, float w) {
                uint32_t word = words[0];
#pragma unroll
                for (int k = 1; k < NC; ++k) {
                    const bool up = w >= top[k - 1];
                    word = up ? words[k] : word;
                    cnt[k] += up ? 1 : 0;
                }
                fold(i, w, word);
            };
#pragma unroll
            for (int i = 0; i < GL; ++i) {
                take(i, weight(i));
                if ((i & 7) == 7) __builtin_amdgcn_sched_barrier(0);
            }
        } else if (__builtin_expect(!scan, 1)) {
            if constexpr (!SMALL) {
            // Eight weights at a time, one level of the search for all of them before the next, and the sums of the
            // previous eight between the levels: an LDS read is used some thirty instructions after it was issued
            // (with the weights in registers there are two to five wavefronts on a SIMD to cover for each other).
            constexpr int B = 8;
            // LEN weights from src, the group's weights i0, i0 + 1, ..
            auto pass = [&](auto &src, auto len_c, int i0) {
                constexpr int LEN = decltype(len_c)::value;
                uint32_t word[2][B];
                uint32_t *at[B];
                // an opaque copy of the weight, made at its use: otherwise the optimiser converts every weight to fp64 once
                // and keeps both
                auto sum_up = [&](int i, uint32_t w) {
                    asm volatile("" : "+v"(src[i]));
                    fold(i0 + i, src[i], w);
                };
#pragma unroll
                for (int i = 0; i < LEN; i += B) {
                    const int par = (i / B) & 1;
                    {
                        // All comparisons of a level before what they choose: a comparison's outcome can be read two
                        // instructions later, and the compiler would wait those out eight times a level (4096 x 1024, G = 64,
                        // q = 4 80.5 -> 75.7 us, q = 3 54.5 -> 50.7).  Two planes in registers have other work to fill that with
                        // and lose the shorter encoding (4096 x 1024, G = 128 56 -> 59).
                        auto apart = [] {
                            if constexpr (Q > 2) __builtin_amdgcn_sched_barrier(0);
                        };
                        bool up[B], quarter[B];
                        float T[B];
                        uint32_t half[B];
#pragma unroll
                        for (int u = 0; u < B; ++u) up[u] = src[i + u] >= top[1];
                        apart();
#pragma unroll
                        for (int u = 0; u < B; ++u) {
                            T[u] = up[u] ? top[2] : top[0];
                            half[u] = up[u] ? NC / 2 * 64u : 0u;
                        }
                        apart();
#pragma unroll
                        for (int u = 0; u < B; ++u) quarter[u] = src[i + u] >= T[u];
                        apart();
#pragma unroll
                        for (int u = 0; u < B; ++u) at[u] = tree + half[u] + (quarter[u] ? NC / 4 * 64u : 0u);
                    }
                    constexpr int levels = Q > 2 ? Q - 1 : 1;             // LDS reads in a row
                    constexpr int per = (B + levels - 1) / levels;        // previous weights summed up behind each
#pragma unroll
                    for (int lv = 0; lv < levels; ++lv) {
                        float node[B];
                        const int step = NC >> (lv + 3);                  // positions this level decides between
#pragma unroll
                        for (int u = 0; u < B; ++u) {
                            if (lv + 1 < levels) node[u] = __builtin_bit_cast(float, at[u][step * 64]);
                            else word[par][u] = at[u][NC * 64];
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        if (i > 0) {
#pragma unroll
                            for (int u = lv * per; u < (lv + 1) * per && u < B; ++u) sum_up(i - B + u, word[par ^ 1][u]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        if (lv + 1 < levels) {
                            bool up[B];
#pragma unroll
                            for (int u = 0; u < B; ++u) up[u] = src[i + u] >= node[u];
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int u = 0; u < B; ++u) at[u] += up[u] ? step * 64u : 0u;
                        }
                    }
#pragma unroll
                    for (int u = 0; u < B; ++u) __hip_atomic_fetch_add(at[u] + 2 * NC * 64, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                }
#pragma unroll
                for (int u = 0; u < B; ++u) sum_up(LEN - B + u, word[(LEN / B - 1) & 1][u]);
            };
            pass(wv, std::integral_constant<int, GL>{}, 0);
            }
        } else {
            // the scan of all candidates
            uint32_t counted = 0u;
            double V[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                double v = 0.0;
#pragma unroll
                for (int j = 0; j < Q; ++j) v += theta[1 + j] * (double)((c >> j) & 1);
                V[c] = v;
            }
            auto take = [&](int i, float w) {
                const double what = (double)w - z;
                uint32_t best = 0;
                double bd = fabs(what - V[0]);
#pragma unroll
                for (int c = 1; c < NC; ++c) {   // first minimum wins ties
                    const double d = fabs(what - V[c]);
                    best = d < bd ? (uint32_t)c : best;
                    bd = __builtin_fmin(bd, d);
                }
                const uint32_t ones = __umul24(best, 0x204081u) & 0x01010101u;
                fold(i, w, (ones << 6) - ones);
                if constexpr (SMALL) {
                    counted += Q == 1 ? best : 1u << 8 * best;   // q = 2: four counts of at most 32
                } else {
                    __hip_atomic_fetch_add(&count[best * 64], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                }
            };
            // from the registers; at q = 4, G = 128 that would be 9000 instructions a round, and the weights come from memory,
            // requested eight ahead
            if constexpr (GL * NC <= 1024) {
#pragma unroll
                for (int i = 0; i < GL; ++i) {
                    float w;   // a copy: the register itself is the same one whichever way the round went
                    asm volatile("" : "=v"(w) : "0"(wv[i]));
                    take(i, w);
                    if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // not many weights converted ahead (registers)
                }
            } else {
                constexpr int AHEAD = 8;
                float nx[AHEAD];
                load_rows(nx, 0, stride);
#pragma unroll 1
                for (int i = 0; i < GL; i += AHEAD) {
                    float cur[AHEAD];
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u) cur[u] = nx[u];
                    if (i + AHEAD < GL) load_rows(nx, i + AHEAD, stride);
                    __builtin_amdgcn_sched_barrier(0);   // the loads go out first
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u) {
                        take(i + u, in_units(cur[u]));
                        if ((u & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // not many weights converted ahead (registers)
                    }
                }
            }
            if constexpr (SMALL) {
#pragma unroll
                for (int c = 0; c < NC; ++c) cnt[c] = Q == 1 ? (c ? (int)counted : GL - (int)counted) : (int)(counted >> 8 * c & 0xffu);
            }
        }
#pragma unroll
        for (int j = 0; j < Q; ++j) rb[j] = add_parts(rb[j] * 0x1p15);

        // counts by code, from counts by sorted position
        if constexpr (SMALL) {
            if (!scan) {
                int at[NC], by_code[NC];
                cnt[0] = GL;
#pragma unroll
                for (int i = 0; i < NC; ++i) at[i] = cnt[i] - (i + 1 < NC ? cnt[i + 1] : 0);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    by_code[c] = 0;
#pragma unroll
                    for (int i = 0; i < NC; ++i) by_code[c] += key[i] == (uint32_t)c ? at[i] : 0;
                }
#pragma unroll
                for (int c = 0; c < NC; ++c) cnt[c] = by_code[c];
            }
        } else {
#pragma unroll
            for (int i = 0; i < NC; ++i) cnt[i] = (int)count[i * 64];
            if (!scan) {
#pragma unroll
                for (int i = 0; i < NC; ++i) plane[(key[i] & (NC - 1)) * 64] = (uint32_t)cnt[i];
#pragma unroll
                for (int i = 0; i < NC; ++i) cnt[i] = (int)plane[i * 64];
            }
        }
        if constexpr (L > 1) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
                unrolled<(L == 4 ? 2 : 1)>([&](auto k) { cnt[c] += (int)across((uint32_t)cnt[c], std::integral_constant<int, 1 + decltype(k)::value>{}); });
        }
        unsigned present = 0u;
        int nb[Q], nbb[Q][Q];
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            nb[j] = 0;
#pragma unroll
            for (int k = 0; k < Q; ++k) nbb[j][k] = 0;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            present |= cnt[c] ? 1u << c : 0u;
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                if (!((c >> j) & 1)) continue;
                nb[j] += cnt[c];
#pragma unroll
                for (int k = j + 1; k < Q; ++k)
                    if ((c >> k) & 1) nbb[j][k] += cnt[c];
            }
        }

        // ---- which columns of [1 b_0 .. b_{Q-1}] are independent ---------------------------------------------
        // Fraction-free elimination on the Gram matrix of the distinct rows present.  Every
        // intermediate is a minor of that matrix: a sum over at most C(16,5) row subsets of squared
        // determinants of 0/1 matrices of order <= 5 (each <= 5), so below 2^17; products and their
        // differences stay below 2^35 and the divisions are exact, hence fp64 computes them exactly (a
        // quotient as product with the reciprocal, rounded to the nearest integer).
        bool is_act[P];
#pragma unroll
        for (int k = 0; k < P; ++k) is_act[k] = true;
        // with every code in use all columns are independent (512 x 512, q = 2, G = 32: 1 us of 24)
        if (Q == 1 || !__all(present == (1u << NC) - 1u)) {
            double gm[P][P];
#pragma unroll
            for (int a = 0; a < P; ++a)
#pragma unroll
                for (int b = a; b < P; ++b) {
                    unsigned both = 0u;   // codes whose row has a one in columns a and b
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        const int ra = a == 0 ? 1 : (c >> (a - 1)) & 1, rc = b == 0 ? 1 : (c >> (b - 1)) & 1;
                        if (ra & rc) both |= 1u << c;
                    }
                    gm[a][b] = (double)__builtin_popcount(present & both);
                }
            double prev = 1.0;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const double pv = gm[k][k];
                if (k > 0) is_act[k] = pv != 0.0;   // the column of ones always is (so A[0][0] stays G, and dividing by it is a multiplication)
                if (is_act[k]) {
                    const double inv_prev = 1.0 / prev;
#pragma unroll
                    for (int i = k + 1; i < P; ++i)
#pragma unroll
                        for (int j = i; j < P; ++j)   // symmetric
                            gm[i][j] = __builtin_rint((gm[i][j] * pv - gm[k][i] * gm[k][j]) * inv_prev);
                    prev = pv;
                }
            }
        }

        // ---- linear reconstruction: normal equations; a dependent column becomes the identity equation
        //      theta = previous value and its contribution moves to the right-hand side ----------------------
        double A[P][P], r[P];
        A[0][0] = (double)G;
        r[0] = rw;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            A[0][1 + j] = A[1 + j][0] = (double)nb[j];
            A[1 + j][1 + j] = (double)nb[j];
            r[1 + j] = rb[j];
#pragma unroll
            for (int k = j + 1; k < Q; ++k) A[1 + j][1 + k] = A[1 + k][1 + j] = (double)nbb[j][k];
        }
        bool full = true;
#pragma unroll
        for (int k = 0; k < P; ++k) full = full && is_act[k];
        if (!__all(full)) {
#pragma unroll
            for (int a = 0; a < P; ++a) {
                double v = r[a];
#pragma unroll
                for (int col = 0; col < P; ++col)
                    if (col != a && !is_act[col]) v -= A[a][col] * theta[col];
                r[a] = is_act[a] ? v : theta[a];
            }
#pragma unroll
            for (int a = 0; a < P; ++a)
#pragma unroll
                for (int b = 0; b < P; ++b)
                    if (!is_act[a] || !is_act[b]) A[a][b] = a == b ? 1.0 : 0.0;
        }
        // elimination without pivoting: the matrix is symmetric positive definite
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const double inv = 1.0 / A[k][k];
#pragma unroll
            for (int i = k + 1; i < P; ++i) {
                const double f = A[i][k] * inv;
#pragma unroll
                for (int j = k + 1; j < P; ++j) A[i][j] -= f * A[k][j];
                r[i] -= f * r[k];
            }
        }
#pragma unroll
        for (int k = P - 1; k >= 0; --k) {
            double v = r[k];
#pragma unroll
            for (int j = k + 1; j < P; ++j) v -= A[k][j] * theta[j];
            theta[k] = v / A[k][k];
        }
    };
    for (int t = 0; t + 1 < t_max; ++t) iteration(std::false_type{});
    iteration(std::true_type{});

    // ---- outputs: parameters rounded to fp16 (nearest even); error with the unrounded ones ---------------
    if (part == 0) {
        zeros[(size_t)gi * N + n] = __builtin_bit_cast(uint16_t, (_Float16)theta[0]);
#pragma unroll
        for (int j = 0; j < Q; ++j) scales[((size_t)j * ngroups + gi) * N + n] = __builtin_bit_cast(uint16_t, (_Float16)theta[1 + j]);
    }
    if (group_err) {
        // not exact: the lanes of a group one after the other, each from where the one before it stopped
        double e = 0.0;
#pragma unroll 1
        for (unsigned turn = 0; turn < (unsigned)L; ++turn) {
            const uint64_t b = __builtin_bit_cast(uint64_t, e);
            constexpr int BEFORE = L == 4 ? 0x90 : 0xA0;   // quad_perm [0,0,1,2], [0,0,2,2]
            const uint32_t lo32 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, BEFORE, 0xf, 0xf, false), hi32 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), BEFORE, 0xf, 0xf, false);
            if (turn != part) continue;
            if (turn > 0) e = __builtin_bit_cast(double, (uint64_t)hi32 << 32 | lo32);
#pragma unroll
            for (int i = 0; i < GL; ++i) {
                const int c = __builtin_amdgcn_raw_buffer_load_b8(c_rows, (int)n + first_row, i * N, 0);
                double v = theta[0];
#pragma unroll
                for (int j = 0; j < Q; ++j) v += theta[1 + j] * (double)((c >> j) & 1);
                const double dlt = (double)weight(i) - v;
                e += dlt * dlt;
            }
        }
        if (part == L - 1) group_err[(size_t)gi * N + n] = (float)e;
    }
}

template <int Q>
void launch_q(const HlqDims &dm, const float *W, int t_max, uint8_t *codes, uint16_t *scales, uint16_t *zeros,
              float *group_err, hipStream_t st)
{
    // A launch of at most one wavefront per SIMD with groups of 32 waits for its thresholds as long as for the scan, and the
    // scan takes the same time for every distribution: 512 x 512, q = 1 / 2 / 3, us, fp32 normals 11.3 / 22.7 / 38.0 by search,
    // 11.8 / 22.0 / 38.3 by scan; bf16 12.3 / 26.7 / 47 against 11.7 / 22.2 / 38; int4 steps 22 / 34 / 41 against 11.8 / 21.9 /
    // 38.  q = 4: 59 by search, 63 by scan.
    auto launch = [&](auto g, auto l) {
        constexpr int G = decltype(g)::value, L = decltype(l)::value;
        const dim3 grid((unsigned)(((long)dm.N * L + 255) / 256), (unsigned)dm.ngroups);
        const int scan_first = G == 32 && Q <= 3 && (long)grid.x * grid.y <= 256;
        hlq_quantize_kernel<Q, G, L><<<grid, 256, 0, st>>>(W, dm.K, dm.N, t_max, scan_first, codes, scales, zeros, group_err);
    };
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    using Four = std::integral_constant<int, 4>;
    // Lanes a group: a wavefront for every one of the 1024 SIMDs, if 32 weights or more stay with a lane.  Beyond that the
    // thresholds and the solution, which every lane of a group makes, cost what the shorter pass saves, except at one and two
    // planes.  us, one lane / two / four: 2048 x 1024 q = 4, G = 64 (512 wavefronts) 76 / 60, G = 128 110 / 75 / 60;  4096 x 1024 q = 4,
    // G = 64 (1024) 76 / 84, G = 128 (512) 112 / 78, G = 256 - / 112 / 80;  4096 x 4096, G = 128 (2048) q = 1 / 2 / 3 / 4 49.9 / 86.8 / 127 /
    // 177 by one lane, 47.1 / 85.6 / 134 / 200 by two.
    const long waves = ((long)dm.N + 63) / 64 * dm.ngroups;   // with one lane a group
    using G64 = std::integral_constant<int, 64>;
    using G128 = std::integral_constant<int, 128>;
    using G256 = std::integral_constant<int, 256>;
    switch (dm.G) {
    case 32: launch(std::integral_constant<int, 32>{}, One{}); break;
    case 64:
        if (waves > 512) launch(G64{}, One{});
        else launch(G64{}, Two{});
        break;
    case 128:
        if (waves > (Q <= 2 ? 2048 : 512)) launch(G128{}, One{});
        else if (waves > 256) launch(G128{}, Two{});
        else launch(G128{}, Four{});
        break;
    default:
        if (waves > 256) launch(G256{}, Two{});
        else launch(G256{}, Four{});
        break;
    }
}

} // namespace

hlq_status hlq_launch_quantize(const HlqDims &dm, const float *W, int t_max, uint8_t *codes, uint16_t *scales,
                               uint16_t *zeros, float *group_err, hipStream_t st)
{
    hlq_clear_stale_error();
    if (t_max < 1 || t_max > 1000) return HLQ_ERR_UNSUPPORTED;
    if (dm.ngroups > 65535) return HLQ_ERR_UNSUPPORTED;
    if (dm.G != 32 && dm.G != 64 && dm.G != 128 && dm.G != 256) return HLQ_ERR_UNSUPPORTED;
    switch (dm.q) {
    case 1: launch_q<1>(dm, W, t_max, codes, scales, zeros, group_err, st); break;
    case 2: launch_q<2>(dm, W, t_max, codes, scales, zeros, group_err, st); break;
    case 3: launch_q<3>(dm, W, t_max, codes, scales, zeros, group_err, st); break;
    case 4: launch_q<4>(dm, W, t_max, codes, scales, zeros, group_err, st); break;
    default: return HLQ_ERR_UNSUPPORTED;
    }
    return hlq_hip_status(hipGetLastError());
}
