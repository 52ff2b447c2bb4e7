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
// that take consecutive parts of the group.  The lanes of a group add their counts and sums and make the same thresholds and
// parameters.  A lane reads its weights once, into registers (G / L fp32 values; lanes of a wavefront hold adjacent
// columns, so each load is a coalesced read of a row of W (of L rows) and all are in
// flight together): W is read from HBM exactly once, and the kernels are bound by vector instructions and their latency.
// What a round needs of the weights is how many of them have each code, and their sums: the integer Gram matrix of
// [1 b_0 .. b_{q-1}] and the fp64 right-hand side of the least-squares step.  With up to three planes a lane sorts its weights
// once and looks those up for every threshold; with four (15 thresholds) it goes through its weights in every round.
// Nothing per weight is stored until the last round writes the codes.  All arithmetic is fp64: the
// step is offline, and decisions (the argmin) then agree with an fp64 reference except at exact ties.
//
// A round is a function of the parameters alone, so a wavefront whose parameters all stay as they are (in every bit) goes on with
// the last round: groups of 32 normal weights are there after 2 to 3 rounds on average, 64 of them together after 6 to 8
// (4096 x 4096, G = 32, when it was brought in: q = 3 138 -> 130 us, q = 4 247 -> 223; weights on a coarse grid up to a half).
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

// One comparison of a sort.  The plain instructions: fmin and fmax first pass every number that was not computed through
// another one (signalling NaNs).
__device__ __forceinline__ void order(float &a, float &b)
{
    float lower, upper;
    asm("v_min_f32 %0, %1, %2" : "=v"(lower) : "v"(a), "v"(b));
    asm("v_max_f32 %0, %1, %2" : "=v"(upper) : "v"(a), "v"(b));
    a = lower;
    b = upper;
}
__device__ __forceinline__ void order(double &a, double &b)
{
    double lower, upper;
    asm("v_min_f64 %0, %1, %2" : "=v"(lower) : "v"(a), "v"(b));
    asm("v_max_f64 %0, %1, %2" : "=v"(upper) : "v"(a), "v"(b));
    a = lower;
    b = upper;
}

// ascending odd-even merge sort (a power of two of numbers), all comparisons at compile-time positions
template <class T, int C>
__device__ __forceinline__ void sort_ascending(T (&v)[C])
{
#pragma unroll
    for (int p = 1; p < C; p *= 2)
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int j = k % p; j + k < C; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (i + j + k < C && (i + j) / (2 * p) == (i + j + k) / (2 * p)) order(v[i + j], v[i + j + k]);
}

// Candidate values V_c = sum_j s_j bit_j(c) in ascending order, with the code in the last q bits: off by 2^-48 of their size
// at most, which changes no threshold that is not within the band of those that are looked at again.
template <int Q>
__device__ __forceinline__ void candidates(const double (&theta)[Q + 1], double (&V)[1 << Q])
{
    V[0] = 0.0;
    unrolled<Q>([&](auto jj) {
        constexpr int top = 1 << decltype(jj)::value;
        V[top] = theta[1 + decltype(jj)::value];
#pragma unroll
        for (int c = 1; c < top; ++c) V[top + c] = V[c] + V[top];   // finite, as are the weights: planes without the bit add nothing
    });
#pragma unroll
    for (int c = 0; c < (1 << Q); ++c) V[c] = __builtin_bit_cast(double, (__builtin_bit_cast(uint64_t, V[c]) & ~(uint64_t)((1 << Q) - 1)) | (uint64_t)c);
    sort_ascending(V);
}

// Linear reconstruction of a group from what its codes are counted and summed up to: the weights with each code, the sums of
// the weights by plane and their sum.  Says whether the parameters changed (in any bit).
template <int Q, int G>
__device__ __forceinline__ bool reconstruct(const int (&cnt)[1 << Q], const double (&rb)[Q], double rw, double (&theta)[Q + 1])
{
    double before[Q + 1];
#pragma unroll
    for (int k = 0; k <= Q; ++k) before[k] = theta[k];
    constexpr int NC = 1 << Q, P = Q + 1;
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
    // Two codes in use that differ in one bit alone make that bit's column independent of all others: with such a pair for
    // every bit there is nothing to decide.
    bool paired = true;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        unsigned without = 0u;   // codes without the bit
#pragma unroll
        for (int c = 0; c < NC; ++c) without |= (c >> j) & 1 ? 0u : 1u << c;
        paired = paired && (present & present >> (1 << j) & without) != 0u;
    }
    if (!__all(paired)) {
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
    for (int k = 1; k < P; ++k) full = full && is_act[k];
    if (!__all(full)) {
#pragma unroll
        for (int a = 0; a < P; ++a) {
            double v = r[a];
#pragma unroll
            for (int col = 1; col < P; ++col)
                if (col != a && !is_act[col]) v -= A[a][col] * theta[col];
            r[a] = a == 0 || is_act[a] ? v : theta[a];
        }
#pragma unroll
        for (int a = 0; a < P; ++a)
#pragma unroll
            for (int b = a == 0 ? 1 : 0; b < P; ++b)
                if ((a > 0 && !is_act[a]) || (b > 0 && !is_act[b])) A[a][b] = a == b ? 1.0 : 0.0;
    }
    // elimination without pivoting: the matrix is symmetric positive definite.  A[0][0] is G, a power of two: the first
    // step's factors and products are exact, so it leaves a symmetric matrix.
    double inv[P];
    inv[0] = 1.0 / (double)G;
#pragma unroll
    for (int i = 1; i < P; ++i) {
        const double f = A[i][0] * inv[0];
#pragma unroll
        for (int j = i; j < P; ++j) A[j][i] = A[i][j] = __builtin_fma(-f, A[0][j], A[i][j]);
        r[i] -= f * r[0];
    }
#pragma unroll
    for (int k = 1; k + 1 < P; ++k) {
        inv[k] = 1.0 / A[k][k];
#pragma unroll
        for (int i = k + 1; i < P; ++i) {
            const double f = A[i][k] * inv[k];
#pragma unroll
            for (int j = k + 1; j < P; ++j) A[i][j] -= f * A[k][j];
            r[i] -= f * r[k];
        }
    }
    theta[P - 1] = r[P - 1] / A[P - 1][P - 1];
#pragma unroll
    for (int k = P - 2; k >= 0; --k) {
        double v = r[k];
#pragma unroll
        for (int j = k + 1; j < P; ++j) v -= A[k][j] * theta[j];
        // v / A[k][k], rounded once: from the rounded reciprocal by one correction of the quotient (Markstein, 1990)
        const double quotient = v * inv[k];
        theta[k] = k == 0 ? quotient : __builtin_fma(__builtin_fma(-quotient, A[k][k], v), inv[k], quotient);
    }
    bool changed = false;
#pragma unroll
    for (int k = 0; k <= Q; ++k) changed = changed || __builtin_bit_cast(uint64_t, theta[k]) != __builtin_bit_cast(uint64_t, before[k]);
    return changed;
}

// Threads of a workgroup, whose wavefronts have nothing to do with each other: one wavefront, so that its LDS is free when it
// ends; four where a wavefront reads half lines of a row (four lanes a column) and the other half should come from the same L2
// (4096 x 4096, G = 256, q = 1 47.7 -> 40.5 us; with two lanes a column 38 / 59 / 103 us by one, 43 / 60 / 129 by four wavefronts).
constexpr int quantize_threads(int l) { return l == 4 ? 256 : 64; }

// wavefronts on a SIMD that the registers leave room for
constexpr int quantize_waves(int gl) { return gl == 32 ? 3 : 2; }

// One to three planes.  The codes are the argmin over 2^q candidate distances, computed in fp64, first minimum in code order.
// With the candidate values sorted, only the two neighbours of a weight compete, and which of them wins is monotone in the
// weight, so there is an exact fp32 number T at which the choice changes: the smallest fp32 weight for which the upper
// neighbour wins.  The 2^q - 1 thresholds are made once per group and round.  The lane's weights lie in LDS in ascending order,
// with the fp64 sum of what is ahead of every block of eight (four): a search among them gives each threshold's
// rank and the sum below it, and the differences of neighbours are the counts and sums of the codes.  Sums in fp64 are exact
// here, so they are those of any other order.
// What makes T exact (tests compare every code with the scan's):
//   - sorted neighbours at least 2^-40 S apart, S the scale of the group's numbers: all fp64 roundings together stay
//     below 2^-47 S, so only neighbours compete and the choice between them is monotone;
//   - with m the midpoint in fp64 and t its rounding to fp32: where |t - m| > 2^-45 S the sign of t - m decides for t, and the
//     next fp32 number on the other side is on the other side of m as well;
//   - otherwise, where fp32 numbers are far enough apart (|t| > 2^-17 S), t is the only one in doubt, and the two distances of t
//     are compared as the scan compares them if one of the weights is t;
//   - with t next to zero they are compared for zero, the only weight that can be there (least magnitude known), and where that is
//     not so the lane's weights around the threshold are asked one after the other.
// A group whose weights are all equal (padded or pruned columns) has equal candidates in every round; it takes code 0.
// A lane that meets none of this (candidates that coincide up to rounding: groups of few distinct values) sends its
// wavefront through the scan for that round and for the rounds after it.
// Bound: vector instructions and their latency at two wavefronts per SIMD, as many as LDS takes (20 KiB for 64 weights a
// lane; blocks of four, 24 KiB and six wavefronts a compute unit, 71 us where blocks of eight take 60).  Per round and group (two lanes)
// at q = 2 some 800 instructions, where going through the weights took 2050; sorting is 1200 a lane.  4096 x 4096, ten rounds,
// us, search per weight and round -> this: G = 128 q = 1 / 2 / 3 47 / 85 / 128 -> 37 / 54 / 92;  G = 64 46 / 84 / 134 -> 35 / 53 / 91;
// G = 32 55 / 106 / 165 -> 39 / 65 / 115;  G = 256 49 / 88 / 125 -> 38 / 56 / 93;  4096 x 1024, G = 128 18 / 34 / 50 -> 16 / 21 / 36.  With four
// planes the fifteen searches cost more than they save (G = 128 190 -> 203 us).
template <int Q, int G, int L>
__global__ void __launch_bounds__(quantize_threads(L), quantize_waves(G / L))
hlq_quantize_kernel(const float *__restrict__ W, int K, int N, int t_max, uint8_t *__restrict__ codes,
                    uint16_t *__restrict__ scales, uint16_t *__restrict__ zeros, float *__restrict__ group_err)
{
    constexpr int GL = G / L;   // weights of a lane
    constexpr int NC = 1 << Q, P = Q + 1, NT = NC - 1;
    constexpr bool SMALL = Q <= 2;
    constexpr int THREADS = quantize_threads(L);
    constexpr int BLK = GL == 64 ? 8 : 4, NB = GL / BLK;
    // lane-private columns, one word every 64: weights in ascending order | sum of those ahead of each block (fp64; where the one
    // of block 0 is, which is zero, q = 3 has its counts by code for a moment, a byte each)
    constexpr int WORDS = GL + 2 * NB;
    __shared__ uint32_t lds[WORDS * THREADS];
    const unsigned n = (blockIdx.x * THREADS + threadIdx.x) / L, part = threadIdx.x % L;   // column, and part of its group
    const int gi = (int)blockIdx.y;
    if (n >= (unsigned)N) return;
    const int ngroups = K / G;
    // the group's rows (at most 2^30 bytes: N <= 2^20) through descriptors: row i is a scalar offset and the lane's column a
    // vector one that never changes, where 64-bit addresses would take two vector registers per access in flight
    const __amdgpu_buffer_rsrc_t w_rows = __builtin_amdgcn_make_buffer_rsrc((void *)(W + (size_t)gi * G * N), 0, G * N * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t c_rows = __builtin_amdgcn_make_buffer_rsrc(codes + (size_t)gi * G * N, 0, G * N, 0x00020000);
    const int first_row = (int)(part * GL) * N;
    uint32_t *const list = lds + (threadIdx.x >> 6) * (WORDS * 64) + (threadIdx.x & 63);
    uint32_t *const ahead = list + GL * 64;
    uint8_t *const counts = (uint8_t *)(lds + (threadIdx.x >> 6) * (WORDS * 64) + GL * 64) + (threadIdx.x & 63) * NC;
    auto put_f64 = [](uint32_t *at, double v) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        at[0] = (uint32_t)b;
        at[64] = (uint32_t)(b >> 32);
    };
    auto get_f64 = [](const uint32_t *at) -> double { return __builtin_bit_cast(double, ((uint64_t)at[64] << 32) | at[0]); };

    float wv[GL];
    {
        int offset = 0;   // a running sum (one scalar instruction a row)
#pragma unroll
        for (int i = 0; i < GL; ++i) {
            wv[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(w_rows, (int)(n * 4) + first_row * 4, offset, 0));
            offset += N * 4;
        }
    }
    // bits of the smallest and the largest magnitude: in ascending order for all that are not NaN, NaN above those
    uint32_t least = ~0u, most = 0u;
#pragma unroll
    for (int i = 0; i < GL; ++i) {
        const uint32_t magnitude = __builtin_bit_cast(uint32_t, wv[i]) & 0x7fffffffu;
        least = min(least, magnitude);
        most = max(most, magnitude);
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
    auto over_parts = [&](uint32_t v, auto op) -> uint32_t {
        unrolled<(L == 4 ? 2 : L == 2 ? 1 : 0)>([&](auto k) { v = op(v, across(v, std::integral_constant<int, 1 + decltype(k)::value>{})); });
        return v;
    };
    auto smaller = [](uint32_t a, uint32_t b) { return min(a, b); };
    least = over_parts(least, smaller);
    most = over_parts(most, [](uint32_t a, uint32_t b) { return max(a, b); });
    const float largest = __builtin_bit_cast(float, most);   // (NaN, if one is)
    // Sums are exact in fp64, and so the same in any order, where no weight (not zero) is below 2^-21 of the largest (2^-24 with
    // groups of 32).  Otherwise weights of larger groups are rounded to multiples of 2^-52 of a power of two that no sum of
    // magnitudes exceeds: a change, by less than fp64 sums are rounded by, in weights below 2^-21 of the largest.  (One
    // number in ten million of a normal distribution.)  With groups of 32, one lane a group, weights stay as they are
    // and a wavefront that holds such a group adds in the order of the rows; so does one with weights that are not finite.
    constexpr uint32_t INF = 0x7f800000u;
    const int infinite = __any(most >= INF);
    int in_order = infinite;
    float lof = 0.f, hif = 0.f;   // Alg. 1 steps 2-3, exact in fp32
    // where the search for the least magnitude has to leave out zeros
    constexpr float RANGE = G > 32 ? 0x1p-21f : 0x1p-24f;
    auto far_apart = [&] { return __builtin_bit_cast(float, least) < largest * RANGE && most < INF; };
    double unit = 0.0;   // adding and subtracting it rounds
    int rounded = 0;
    if (__builtin_expect(__any(far_apart()), 0)) {
        least = ~0u;
#pragma unroll
        for (int i = 0; i < GL; ++i) {
            const uint32_t magnitude = __builtin_bit_cast(uint32_t, wv[i]) & 0x7fffffffu;
            least = min(least, magnitude - 1u);
        }
        least = over_parts(least, smaller) + 1u;   // (0 - 1 is the largest)
        const bool wide = least != 0u && far_apart();
        if constexpr (G > 32) {
            constexpr int LOG_G = G == 64 ? 6 : G == 128 ? 7 : 8;
            const int above = (int)(most >> 23) - 126 + LOG_G;
            if (wide) unit = __builtin_bit_cast(double, (uint64_t)(1023 + above) << 52 | 1ull << 51);
            rounded = __any(wide);
        } else {
            in_order |= __any(wide);
        }
    }
    in_order = __builtin_amdgcn_readfirstlane(in_order);
    const bool from_list = in_order == 0 && rounded == 0;   // (where the two ends are)
    if (__builtin_expect(!from_list, 0)) {
        lof = hif = wv[0];
#pragma unroll
        for (int i = 1; i < GL; ++i) {
            lof = wv[i] < lof ? wv[i] : lof;
            hif = wv[i] > hif ? wv[i] : hif;
        }
    }
    if (__builtin_expect(rounded, 0)) {
#pragma unroll
        for (int i = 0; i < GL; ++i) {
            asm volatile("" : "+v"(wv[i]));
            wv[i] = (float)(((double)wv[i] + unit) - unit);
        }
    }
    double rl = 0.0;       // sum of the lane's weights
    float quarter[3];      // weights at the quarters of the list, the first two levels of a search
    {
        float sv[GL];
#pragma unroll
        for (int i = 0; i < GL; ++i) sv[i] = wv[i];
        if (in_order == 0) sort_ascending(sv);
        if (from_list) {
            lof = sv[0];
            hif = sv[GL - 1];
        }
#pragma unroll
        for (int i = 0; i < GL; ++i) {
            if (i % BLK == 0) put_f64(ahead + i / BLK * 128, rl);
            list[i * 64] = __builtin_bit_cast(uint32_t, sv[i]);
            rl += (double)sv[i];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) quarter[k] = sv[(k + 1) * GL / 4];
    }
    const double rw = add_parts(rl);   // of the group's
    if constexpr (L > 1) {
        unrolled<(L == 4 ? 2 : 1)>([&](auto k) {
            const std::integral_constant<int, 1 + decltype(k)::value> l;
            const float lo2 = __builtin_bit_cast(float, across(__builtin_bit_cast(uint32_t, lof), l)), hi2 = __builtin_bit_cast(float, across(__builtin_bit_cast(uint32_t, hif), l));
            lof = lo2 < lof ? lo2 : lof;
            hif = hi2 > hif ? hi2 : hif;
        });
    }
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

    // For each threshold the number of the lane's weights that are not at or above it, and their sum.
    auto search = [&](const auto &T, auto &rank, auto &sum) {
        constexpr int B = sizeof(rank) / sizeof(rank[0]);
        const uint32_t *at[B];   // in the list
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const bool right = !(quarter[1] >= T[u]);
            const float next = right ? quarter[2] : quarter[0];
            at[u] = list + (right ? GL / 2 * 64u : 0u) + (!(next >= T[u]) ? GL / 4 * 64u : 0u);
        }
#pragma unroll
        for (int step = NB / 8; step >= 1; step /= 2) {
            float head[B];
#pragma unroll
            for (int u = 0; u < B; ++u) head[u] = __builtin_bit_cast(float, at[u][step * BLK * 64]);
#pragma unroll
            for (int u = 0; u < B; ++u) at[u] += !(head[u] >= T[u]) ? step * BLK * 64u : 0u;
        }
        float v[B][BLK];
#pragma unroll
        for (int u = 0; u < B; ++u) {
#pragma unroll
            for (int e = 0; e < BLK; ++e) v[u][e] = __builtin_bit_cast(float, at[u][e * 64]);
            sum[u] = get_f64(ahead + (uint32_t)(at[u] - list) / BLK * 2);
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
            int r = (int)((at[u] - list) >> 6);
#pragma unroll
            for (int e = 0; e < BLK; ++e) {
                const bool below = !(v[u][e] >= T[u]);
                r += below ? 1 : 0;
                float part_sum = below ? v[u][e] : 0.f;
                asm("" : "+v"(part_sum));   // (one selection, not two behind the conversion)
                sum[u] += (double)part_sum;
            }
            rank[u] = r;
        }
    };

    // Runs of equal weights in the list, a bit where one starts: found when the scan first asks for them.  (In row order every weight is one.)
    using Bits = std::conditional_t<GL == 64, uint64_t, uint32_t>;
    Bits starts = ~(Bits)0;
    constexpr int MANY = (Q == 3 ? 7 : 6) * GL / 16;
    int runs_known = in_order;

    // Rounds in a row that needed the scan: a wavefront stays with it after STAY of them (data of few distinct values needs
    // it in every round).
    constexpr int STAY = 1;
    int scans = infinite ? STAY : 0;
#pragma unroll 1
    for (int t = 0; t < t_max; ++t) {
        const double z = theta[0];
        double S = (double)largest + fabs(z);
#pragma unroll
        for (int j = 0; j < Q; ++j) S += fabs(theta[1 + j]);
        // a group whose weights are all equal has equal candidates in every round and takes code 0: its thresholds are NaN
        const double gap_min = constant ? -1.0 : S * 0x1p-40, band = fmax(S * 0x1p-45, 0x1p-149);
        const double zt = constant ? (double)__builtin_inff() : z;

        uint32_t key[NC];   // codes in ascending order of their values
        float T[NT];
        uint32_t hard = 0u;   // the threshold that the list decides: position, codes of the two sides
        double below = 0.0, above = 0.0;   // and their values
        bool near[NC], any_near = false;   // midpoints within the band of an fp32 number
        auto exact_value = [&](uint32_t c) -> double {
            double v = 0.0;
#pragma unroll
            for (int j = 0; j < Q; ++j) v += (c >> j & 1u) ? theta[1 + j] : 0.0;
            return v;
        };
        auto up_from = [](float v, uint32_t &away) -> float {   // one fp32 step up (away: in bits)
            const uint32_t bits = __builtin_bit_cast(uint32_t, v);
            away = (int32_t)bits < 0 ? ~0u : 1u;
            return __builtin_bit_cast(float, bits + away);
        };
        // through readfirstlane, here and below: the optimiser takes the choice for a scalar one (otherwise it keeps the
        // registers of both ways at once) and makes no copy of the round for each value
        scans = __builtin_amdgcn_readfirstlane(scans);
        int chosen = scans >= STAY;
        if (chosen == 0) {
            double V[NC];
            candidates<Q>(theta, V);
#pragma unroll
            for (int i = 0; i < NC; ++i) key[i] = (uint32_t)__builtin_bit_cast(uint64_t, V[i]) & (NC - 1);
            bool good = true;
            // the midpoint between positions i - 1 and i, as fp32 and how far that is above it
            auto middle = [&](double va, double vb, float &mid) -> double {
                const double m = __builtin_fma(0.5, va + vb, zt);
                mid = (float)m;
                return (double)mid - m;
            };
#pragma unroll
            for (int i = 1; i < NC; ++i) {
                good = good && V[i] - V[i - 1] >= gap_min;
                float mid;
                uint32_t away;
                const double off = middle(V[i - 1], V[i], mid);
                const float next = up_from(mid, away);
                T[i - 1] = off >= -band ? mid : next;   // the upper neighbour wins at mid, or may
                near[i] = fabs(off) <= band;
                any_near = any_near || near[i];
            }
            // Near a midpoint that is not close to zero there is one fp32 number about which there is doubt; whether it is among the
            // weights shows when they have been counted.  Close to zero the decision is made here.
            if (__any(any_near)) {
                unrolled<NT>([&](auto ii) {
                    constexpr int i = decltype(ii)::value + 1;
                    const bool now = near[i] & ((in_order != 0) | (fabs((double)T[i - 1]) <= S * 0x1p-17));
                    if (!__any(now)) return;
                    const uint32_t ca = key[i - 1], cb = key[i];
                    const double va = exact_value(ca), vb = exact_value(cb);
                    float mid;
                    uint32_t away;
                    middle(va, vb, mid);
                    const float next = up_from(mid, away);
                    const float prev = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, mid) - away);
                    auto upper_wins = [&](float w) {
                        const double what = (double)w - z;
                        const double da = fabs(what - va), db = fabs(what - vb);
                        return (db < da) | ((db == da) & (cb < ca));
                    };
                    // next to zero fp32 numbers are denser than the distances are exact, but weights mostly are zero or far from it
                    const bool zero = now & (fabs((double)mid) <= band) & ((double)__builtin_bit_cast(float, least) > 4.0 * band);
                    mid = zero ? 0.f : mid;
                    const bool at_mid = upper_wins(mid);
                    const bool beside = upper_wins(at_mid ? prev : next);
                    const bool open = now & !zero & ((mid == 0.f) | (at_mid == beside));
                    T[i - 1] = now ? (at_mid ? mid : mid == 0.f ? __builtin_bit_cast(float, 1u) : next) : T[i - 1];   // (open: where the list is asked first)
                    good = good && !(open && hard);   // a second one
                    hard = open ? (uint32_t)i | ca << 8 | cb << 16 : hard;
                    below = open ? va : below;
                    above = open ? vb : above;
                });
            }
            chosen = __any(!good) ? 1 : 0;
        } else {
#pragma unroll
            for (int i = 0; i < NC; ++i) {   // (not used)
                key[i] = (uint32_t)i;
                near[i] = false;
            }
#pragma unroll
            for (int i = 0; i < NT; ++i) T[i] = 0.f;
        }
        chosen = __builtin_amdgcn_readfirstlane(chosen);
        const bool scan = chosen != 0;
        scans = scan ? scans + 1 : 0;

        int cnt[NC];      // weights by code
        double rb[Q];     // sums by plane
#pragma unroll
        for (int j = 0; j < Q; ++j) rb[j] = 0.0;
        const bool last = t == t_max - 1;
        auto store_code = [&](int i, uint32_t c) { __builtin_amdgcn_raw_buffer_store_b8((uint8_t)c, c_rows, (int)n + first_row, i * N, 0); };
        uint32_t *const places = list;   // thresholds and codes in order, when the list is not needed any more (or written again)
        // eight codes of weights i, i + 1, .. by the thresholds
        auto codes_of = [&](int i, uint32_t (&c)[8]) {
            if constexpr (SMALL) {
                // comparisons ahead of what they choose: an outcome can be read two instructions later
#pragma unroll
                for (int u = 0; u < 8; ++u) c[u] = key[0];
#pragma unroll
                for (int k = 1; k < NC; ++k) {
                    bool up[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) up[u] = weight(i + u) >= T[k - 1];
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < 8; ++u) c[u] = up[u] ? key[k] : c[u];
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                // a binary search: two levels with thresholds in registers, the others and the code from the table
                uint32_t at[8];
                float w[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    w[u] = weight(i + u);
                    const bool up = w[u] >= T[NC / 2 - 1];
                    const float Tn = up ? T[3 * NC / 4 - 1] : T[NC / 4 - 1];
                    at[u] = (up ? NC / 2 * 64u : 0u) + (w[u] >= Tn ? NC / 4 * 64u : 0u);
                }
#pragma unroll
                for (int step = NC / 8; step >= 1; step /= 2) {
                    float node[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) node[u] = __builtin_bit_cast(float, places[at[u] + step * 64]);
#pragma unroll
                    for (int u = 0; u < 8; ++u) at[u] += w[u] >= node[u] ? step * 64u : 0u;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) c[u] = places[at[u] + NC * 64];
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto make_table = [&] {
            if constexpr (!SMALL) {
#pragma unroll
                for (int i = 0; i < NC; ++i) {
                    if (i > 0) places[i * 64] = __builtin_bit_cast(uint32_t, T[i > 0 ? i - 1 : 0]);
                    places[(NC + i) * 64] = key[i];
                }
            }
        };
        if (G == 32 && __builtin_expect(!scan && in_order, 0)) {
            if constexpr (G == 32) {
                if (__any(hard != 0u)) {   // the threshold is the smallest weight for which the upper neighbour wins
                    const uint32_t at = hard & 0xffu;
                    float least_up = __builtin_inff();
#pragma unroll 1
                    for (int i = 0; i < GL; ++i) {
                        const float w = __builtin_bit_cast(float, list[i * 64]);
                        const double what = (double)w - z;
                        const double da = fabs(what - below), db = fabs(what - above);
                        const bool up = db < da || (db == da && hard >> 16 < (hard >> 8 & 0xffu));
                        least_up = up ? fminf(least_up, w) : least_up;
                    }
#pragma unroll
                    for (int i = 0; i < NT; ++i) T[i] = at == (uint32_t)(i + 1) ? least_up : T[i];
                }
                make_table();
                uint64_t counted = 0u;   // by code, eight bits each
#pragma unroll
                for (int i = 0; i < GL; i += 8) {
                    uint32_t c[8];
                    codes_of(i, c);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const double w = (double)weight(i + u);
#pragma unroll
                        for (int j = 0; j < Q; ++j) rb[j] = __builtin_fma((double)(c[u] >> j & 1u), w, rb[j]);
                        counted += 1ull << 8 * c[u];
                        if (last) store_code(i + u, c[u]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int c = 0; c < NC; ++c) cnt[c] = (int)(counted >> 8 * c & 0xffu);
                if constexpr (!SMALL) {
#pragma unroll
                    for (int i = 0; i < 2 * NC; ++i) list[i * 64] = __builtin_bit_cast(uint32_t, wv[i]);
                }
            }
        } else if (__builtin_expect(!scan, 1)) {
            int rank[NT];
            double sum[NT];
            search(T, rank, sum);
            if (__any(any_near)) {
                bool equal[NC], any_equal = false;
#pragma unroll
                for (int i = 1; i < NC; ++i) {
                    const float first = __builtin_bit_cast(float, list[min(rank[i - 1], GL - 1) * 64]);   // at or above the threshold
                    equal[i] = near[i] & (first == T[i - 1]);
                    any_equal = any_equal | equal[i];
                }
                if (__builtin_expect(__any(any_equal), 0)) {
                    unrolled<NT>([&](auto ii) {
                        constexpr int i = decltype(ii)::value + 1;
                        if (!__any(equal[i])) return;
                        const double va = exact_value(key[i - 1]), vb = exact_value(key[i]);
                        const double what = (double)T[i - 1] - z;
                        const double da = fabs(what - va), db = fabs(what - vb);
                        uint32_t away;
                        float Ts[1] = {equal[i] && !(db < da || (db == da && key[i] < key[i - 1])) ? up_from(T[i - 1], away) : T[i - 1]};
                        int rs[1];
                        double ss[1];
                        search(Ts, rs, ss);
                        T[i - 1] = Ts[0];
                        rank[i - 1] = rs[0];
                        sum[i - 1] = ss[0];
                    });
                }
            }
            if (__builtin_expect(__any(hard != 0u), 0)) {
                // Which neighbour wins is monotone in the weight: the lane's weights on the two sides of the threshold are asked, and
                // it moves past the ones that are on the wrong side (those close to zero at a midpoint of zero).
                const uint32_t at = hard & 0xffu;
                const bool tie = hard >> 16 < (hard >> 8 & 0xffu);
                auto upper_wins = [&](float w) {
                    const double what = (double)w - z;
                    const double da = fabs(what - below), db = fabs(what - above);
                    return db < da || (db == da && tie);
                };
                float Th[1] = {T[0]};
                int rh[1] = {rank[0]};
                double sh[1] = {sum[0]};
#pragma unroll
                for (int i = 1; i < NT; ++i) {
                    Th[0] = at == (uint32_t)(i + 1) ? T[i] : Th[0];
                    rh[0] = at == (uint32_t)(i + 1) ? rank[i] : rh[0];
                    sh[0] = at == (uint32_t)(i + 1) ? sum[i] : sh[0];
                }
#pragma unroll 1
                for (int s = 0; s <= GL; ++s) {   // every turn passes a value of the list, all in one direction
                    const float left = __builtin_bit_cast(float, list[max(rh[0] - 1, 0) * 64]), right = __builtin_bit_cast(float, list[min(rh[0], GL - 1) * 64]);
                    const bool down = at && rh[0] > 0 && upper_wins(left), up = at && rh[0] < GL && !upper_wins(right);
                    if (!__any(down || up)) break;
                    const uint32_t rbits = __builtin_bit_cast(uint32_t, right);
                    const float past = __builtin_bit_cast(float, rbits << 1 == 0u ? 1u : rbits + ((int32_t)rbits < 0 ? ~0u : 1u));
                    Th[0] = down ? left : up ? past : Th[0];
                    search(Th, rh, sh);
                }
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    T[i] = at == (uint32_t)(i + 1) ? Th[0] : T[i];
                    rank[i] = at == (uint32_t)(i + 1) ? rh[0] : rank[i];
                    sum[i] = at == (uint32_t)(i + 1) ? sh[0] : sum[i];
                }
            }
            // counts and sums by position in the candidates' order, then by code
            auto count_at = [&](int i) -> int { return (i < NT ? rank[i < NT ? i : 0] : GL) - (i > 0 ? rank[i > 0 ? i - 1 : 0] : 0); };
            auto sum_at = [&](int i) -> double { return (i < NT ? sum[i < NT ? i : 0] : rl) - (i > 0 ? sum[i > 0 ? i - 1 : 0] : 0.0); };
            if constexpr (SMALL) {
                uint32_t counted = 0u;   // by code, eight bits each
#pragma unroll
                for (int i = 0; i < NC; ++i) {
                    counted += (uint32_t)count_at(i) << 8 * key[i];
#pragma unroll
                    for (int j = 0; j < Q; ++j) rb[j] = __builtin_fma((double)(key[i] >> j & 1u), sum_at(i), rb[j]);   // exact, as all of these
                }
#pragma unroll
                for (int c = 0; c < NC; ++c) cnt[c] = (int)(counted >> 8 * c & 0xffu);
            } else {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the words are other lanes' there (q = 3)
#pragma unroll
                for (int i = 0; i < NC; ++i) counts[key[i]] = (uint8_t)count_at(i);
                uint32_t by_code[NC / 4];
#pragma unroll
                for (int w = 0; w < NC / 4; ++w) by_code[w] = ((const uint32_t *)counts)[w];
#pragma unroll
                for (int i = 0; i < NC; ++i) {
                    const double v = sum_at(i);
#pragma unroll
                    for (int j = 0; j < Q; ++j) rb[j] = __builtin_fma((double)(key[i] >> j & 1u), v, rb[j]);
                }
#pragma unroll
                for (int c = 0; c < NC; ++c) cnt[c] = (int)(by_code[c / 4] >> 8 * (c % 4) & 0xffu);
                // what was there again
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                put_f64(ahead, 0.0);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
        } else {
            // The scan of all candidates: one run of equal weights after the other where no lane has more than MANY, and otherwise
            // weight by weight, eight side by side (the lane that needs the scan may be one in 64, and the weights of the others all
            // different).  4096 x 4096, us, runs / weights, by the values of a column: G = 128, q = 2 10 59 / 89, 18 82 / 106, 32 121 / 125, 48
            // 155 / 134, all different 252 / 132;  q = 3 105 / 192, 133 / 209, 181 / 231, 225 / 240, 363 / 238;  1024 x 1024, G = 64 (32 weights
            // a lane) q = 2 17 / 19, 25 / 22, 35 / 26, 43 / 27, 49 / 27.
            double V[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                double v = 0.0;
#pragma unroll
                for (int j = 0; j < Q; ++j) v += theta[1 + j] * (double)((c >> j) & 1);
                V[c] = v;
            }
            auto choose = [&](float w) -> uint32_t {
                const double what = (double)w - z;
                uint32_t best = 0;
                double bd = fabs(what - V[0]);
#pragma unroll
                for (int c = 1; c < NC; ++c) {   // first minimum wins ties
                    const double d = fabs(what - V[c]);
                    best = d < bd ? (uint32_t)c : best;
                    bd = __builtin_fmin(bd, d);
                }
                return best;
            };
            if (runs_known == 0) {
                starts = 0u;
                float before = __builtin_nanf("");
#pragma unroll
                for (int i = 0; i < GL; ++i) {
                    const float v = __builtin_bit_cast(float, list[i * 64]);
                    starts |= v != before ? (Bits)1 << i : (Bits)0;
                    before = v;
                }
                runs_known = 1;
            }
            std::conditional_t<SMALL, uint32_t, uint64_t> counted = 0u;   // by code, eight bits each
            auto fold = [&](float w, uint32_t code, int number) {
                const double all = (double)number * (double)w;   // exact
#pragma unroll
                for (int j = 0; j < Q; ++j) rb[j] = __builtin_fma((double)(code >> j & 1u), all, rb[j]);
                counted += (decltype(counted))number << 8 * code;
            };
            if (__any(__popcll(starts) > MANY)) {
#pragma unroll 1
                for (int i = 0; i < GL; i += 8) {
                    float w[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) w[u] = __builtin_bit_cast(float, list[(i + u) * 64]);
#pragma unroll
                    for (int u = 0; u < 8; ++u) fold(w[u], choose(w[u]), 1);
                }
            } else {
                Bits left = starts;
#pragma unroll 1
                while (__any(left != 0u)) {
                    if (left != 0u) {
                        const int i = __builtin_ctzll(left);
                        left &= left - 1;
                        const int number = (left ? __builtin_ctzll(left) : GL) - i;
                        const float w = __builtin_bit_cast(float, list[i * 64]);
                        fold(w, choose(w), number);
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) cnt[c] = (int)(counted >> 8 * c & 0xffu);
            if (last) {
#pragma unroll
                for (int i = 0; i < GL; ++i) {
                    float w;   // a copy: the register itself is the same one whichever way the round went
                    asm volatile("" : "=v"(w) : "0"(wv[i]));
                    store_code(i, choose(w));
                    if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // not many weights converted ahead (registers)
                }
            }
        }
        // the last round stores the codes
        if (last && !scan && !(G == 32 && in_order)) {
            make_table();
#pragma unroll
            for (int i = 0; i < GL; i += 8) {
                uint32_t c[8];
                codes_of(i, c);
#pragma unroll
                for (int u = 0; u < 8; ++u) store_code(i + u, c[u]);
            }
        }
#pragma unroll
        for (int j = 0; j < Q; ++j) rb[j] = add_parts(rb[j]);
        if constexpr (L > 1) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
                unrolled<(L == 4 ? 2 : 1)>([&](auto k) { cnt[c] += (int)across((uint32_t)cnt[c], std::integral_constant<int, 1 + decltype(k)::value>{}); });
        }
        // parameters that stay as they are give the same codes and parameters in every round to come: only the last is left
        if (!__any(reconstruct<Q, G>(cnt, rb, rw, theta))) t = max(t, t_max - 2);
    }

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

// Four planes.  The same thresholds, and a binary search among them for every weight and round; midpoints next to zero by
// bisection over the fp32 numbers.
// The first two levels of the search have their thresholds in registers, the others read them from a lane-private LDS
// column, in ascending order (the number of thresholds passed so far is the address); a second column holds, per sorted
// position, a word with byte j = 0x3f where the code has bit j: moved to the top of the high half of a double it is 2^-15,
// the factor with which the weight enters plane j's sum (the sums are kept times 2^-15: every product and rounding is the
// one without the factor).  Codes are counted in a third.
// Per weight and round 25 vector instructions, instead of about 110 for a scan with counts.  The thresholds are made side by side
// and only those near an fp32 number looked at again one by one, a division is saved for all but the last unknown, and columns
// are not asked for independence where the codes show it: 4096 x 1024, G = 64 80 -> 75 us, 4096 x 4096, G = 32 / 64 / 128 / 256
// 282 / 215 / 190 / 185 -> 230 / 196 / 182 / 175.
// Groups of 64, one lane each: groups that are at rest leave their lanes to the others of their wavefront (below), 4096 x 1024 75 -> 67 us,
// 4096 x 4096 196 -> 182, bf16 weights 103 -> 79 and 237 -> 213, -1, 0, 1 130 -> 81 and 399 -> 240; two wavefronts on a SIMD instead of three for it.
template <int G, int L>
__global__ void __launch_bounds__(256, G / L == 128 || (G == 64 && L == 1) ? 2 : 3)
hlq_quantize_kernel_4(const float *__restrict__ W, int K, int N, int t_max, uint8_t *__restrict__ codes,
                    uint16_t *__restrict__ scales, uint16_t *__restrict__ zeros, float *__restrict__ group_err)
{
    constexpr int GL = G / L;   // weights of a lane
    constexpr int Q = 4, NC = 1 << Q, P = Q + 1, QUARTER = NC / 4;
    __shared__ uint32_t lds[4 * 3 * NC * 64];
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
    // this lane's columns, one word every 64: thresholds in order | plane words by sorted position | counts
    uint32_t *const tree = lds + (threadIdx.x >> 6) * (3 * NC * 64) + (threadIdx.x & 63);
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
    using Lanes = std::integral_constant<int, L>;
    auto add_parts = [&](double v, auto lanes) -> double {
        unrolled<(decltype(lanes)::value == 4 ? 2 : decltype(lanes)::value == 2 ? 1 : 0)>([&](auto k) {
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
    float largest = fmaxf(fabsf(lof), fabsf(hif));
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
    rw = add_parts(rw, Lanes{});
    auto weight = [&](int i) -> float {
        // opaque to the optimiser, so the fp64 copies are made per use instead of being kept
        // for the whole kernel (which would double the registers held)
        asm volatile("" : "+v"(wv[i]));
        return wv[i];
    };
    const double lo = (double)lof, hi = (double)hif;
    const double delta = (hi - lo) / (double)(NC - 1);
    bool constant = lof == hif && rw - rw == 0.0;   // all weights equal (and no NaN among them)
    double theta[P];   // theta[0] = z, theta[1 + j] = s_j
    theta[0] = lo;
#pragma unroll
    for (int j = 0; j < Q; ++j) theta[1 + j] = delta * (double)(1 << j);

    // Rounds in a row that needed the scan: a wavefront stays with it after STAY of them (data of few distinct values needs
    // it in every round).  Two here: the scan takes four times what a search does, and one in a row can be a coincidence.
    constexpr int STAY = 2;
    int scans = 0;
    // one iteration of Alg. 1 for groups of which `lanes` lanes have the weights src each; the last one also stores the codes (a
    // separate instantiation: a test per weight costs more).  Returns whether the lane's next round can differ.
    auto iteration = [&](auto last_c, auto &src, auto lanes) -> bool {
        constexpr bool last = decltype(last_c)::value;
        constexpr int LEN = sizeof(src) / sizeof(src[0]), PARTS = decltype(lanes)::value;
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
        float top[3];   // the thresholds at the quarters; the others are in LDS
        // through readfirstlane, here and below: the optimiser takes the choice for a scalar one (otherwise it keeps the
        // registers of both ways at once) and makes no copy of the round for each value
        scans = __builtin_amdgcn_readfirstlane(scans);
        int chosen = scans >= STAY;
        if (chosen == 0) {
            // candidate values as in the kernel above
            double V[NC];
            candidates<Q>(theta, V);
#pragma unroll
            for (int i = 0; i < NC; ++i) key[i] = (uint32_t)__builtin_bit_cast(uint64_t, V[i]) & (NC - 1);
            auto exact_value = [&](uint32_t c) -> double {
                double v = 0.0;
#pragma unroll
                for (int j = 0; j < Q; ++j) v += (c >> j & 1u) ? theta[1 + j] : 0.0;
                return v;
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
            bool good = true, near[NC], any_near = false;
            uint32_t hard = 0u;   // the threshold that is left to the bisection below: position, codes of the two sides
#pragma unroll
            for (int i = 1; i < NC; ++i) {
                good = good && V[i] - V[i - 1] >= gap_min;
                const double m = __builtin_fma(0.5, V[i - 1] + V[i], zt);
                const float t = (float)m;
                const double off = (double)t - m;
                const uint32_t tb = __builtin_bit_cast(uint32_t, t);
                const float next = __builtin_bit_cast(float, tb + ((int32_t)tb < 0 ? ~0u : 1u));   // one fp32 step up
                const float T = off > 0.0 ? t : next;   // the upper neighbour wins at t
                near[i] = fabs(off) <= band;
                any_near = any_near || near[i];
                if (i % QUARTER == 0) top[i / QUARTER - 1] = T;
                else tree[i * 64] = __builtin_bit_cast(uint32_t, T);
            }
            if (__any(any_near)) {   // in the first round mostly: the middle of the grid is an fp32 number
                unrolled<NC - 1>([&](auto ii) {
                    constexpr int i = decltype(ii)::value + 1;
                    if (!__any(near[i])) return;
                    const uint32_t ca = key[i - 1], cb = key[i];
                    const double va = exact_value(ca), vb = exact_value(cb);
                    const float t = (float)__builtin_fma(0.5, va + vb, zt);
                    const uint32_t tb = __builtin_bit_cast(uint32_t, t);
                    const uint32_t away = (int32_t)tb < 0 ? ~0u : 1u;   // one fp32 step up (away: in bits)
                    const float next = __builtin_bit_cast(float, tb + away), prev = __builtin_bit_cast(float, tb - away);
                    auto upper_wins = [&](float w) {
                        const double what = (double)w - z;
                        const double da = fabs(what - va), db = fabs(what - vb);
                        return (db < da) | ((db == da) & (cb < ca));
                    };
                    const bool at_t = upper_wins(t);
                    const bool beside = upper_wins(at_t ? prev : next);
                    const bool open = near[i] & ((t == 0.f) | (at_t == beside));
                    good = good && !(open && hard);   // a second one
                    hard = open ? (uint32_t)i | ca << 8 | cb << 16 : hard;
                    const float T = at_t ? t : next;
                    if constexpr (i % QUARTER == 0) top[i / QUARTER - 1] = near[i] ? T : top[i / QUARTER - 1];
                    else if (near[i]) tree[i * 64] = __builtin_bit_cast(uint32_t, T);
                });
            }
            if (__builtin_expect(__any(hard != 0u), 0)) {
                const uint32_t at = hard & 0xffu, code_below = hard >> 8 & 0xffu, code_above = hard >> 16;
                const double below = exact_value(code_below), above = exact_value(code_above);
                const float T = bisect(below, above, code_above < code_below, hard != 0u);
#pragma unroll
                for (int k = 0; k < 3; ++k) top[k] = at == (uint32_t)((k + 1) * QUARTER) ? T : top[k];
                if (at) tree[at * 64] = __builtin_bit_cast(uint32_t, T);
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
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const uint32_t c = key[i];
            const uint32_t ones = __umul24(c, 0x204081u) & 0x01010101u;   // bit j of the code in byte j
            plane[i * 64] = (ones << 6) - ones;
            count[i * 64] = 0u;
        }
        int cnt[NC];
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
        if (__builtin_expect(!scan, 1)) {
            // Eight weights at a time, one level of the search for all of them before the next, and the sums of the
            // previous eight between the levels: an LDS read is used some thirty instructions after it was issued
            // (with the weights in registers there are two to five wavefronts on a SIMD to cover for each other).
            constexpr int B = 8;
            {
                uint32_t word[2][B];
                uint32_t *at[B];
                // an opaque copy of the weight, made at its use: otherwise the optimiser converts every weight to fp64 once
                // and keeps both
                auto sum_up = [&](int i, uint32_t w) {
                    asm volatile("" : "+v"(src[i]));
                    fold(i, src[i], w);
                };
#pragma unroll
                for (int i = 0; i < LEN; i += B) {
                    const int par = (i / B) & 1;
                    {
                        // All comparisons of a level before what they choose: a comparison's outcome can be read two
                        // instructions later, and the compiler would wait those out eight times a level (4096 x 1024, G = 64
                        // 80.5 -> 75.7 us).
                        auto apart = [] {
                            __builtin_amdgcn_sched_barrier(0);
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
                    constexpr int levels = Q - 1;                         // LDS reads in a row
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
            }
        } else {
            // the scan of all candidates
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
                __hip_atomic_fetch_add(&count[best * 64], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            };
            // from the registers; at q = 4, G = 128 that would be 9000 instructions a round, and the weights come from memory,
            // requested eight ahead
            if constexpr (LEN * NC <= 1024) {
#pragma unroll
                for (int i = 0; i < LEN; ++i) {
                    float w;   // a copy: the register itself is the same one whichever way the round went
                    asm volatile("" : "=v"(w) : "0"(src[i]));
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
        }
#pragma unroll
        for (int j = 0; j < Q; ++j) rb[j] = add_parts(rb[j] * 0x1p15, lanes);

        // counts by code, from counts by sorted position
        {
#pragma unroll
            for (int i = 0; i < NC; ++i) cnt[i] = (int)count[i * 64];
            if (!scan) {
#pragma unroll
                for (int i = 0; i < NC; ++i) plane[key[i] * 64] = (uint32_t)cnt[i];
#pragma unroll
                for (int i = 0; i < NC; ++i) cnt[i] = (int)plane[i * 64];
            }
        }
        if constexpr (PARTS > 1) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
                unrolled<(PARTS == 4 ? 2 : 1)>([&](auto k) { cnt[c] += (int)across((uint32_t)cnt[c], std::integral_constant<int, 1 + decltype(k)::value>{}); });
        }
        return reconstruct<Q, G>(cnt, rb, rw, theta);
    };
    int left = t_max - 1;   // rounds before the last
    // Rounds for the groups of the lanes in `changing` only, with PARTS lanes and a part of the weights each, until
    // no more than `enough` of them change; returns which do (as many as before where no round is left).  At most
    // 64 / PARTS groups: one more and its numbers would be handed over in the words of another one.
    auto share_out = [&](auto parts_c, uint64_t changing, int enough) -> uint64_t {
        constexpr int PARTS = decltype(parts_c)::value, SLOTS = 64 / PARTS, LEN = GL / PARTS;
        const int lane = (int)(threadIdx.x & 63), slot = lane / PARTS, mine_of = lane % PARTS;
        const bool mine = changing >> lane & 1, used = slot < __popcll(changing);
        const int to = __popcll(changing & ((1ull << lane) - 1));
        uint32_t *const all = lds + (threadIdx.x >> 6) * (3 * NC * 64);   // of the wavefront; word i of all slots together
        auto put = [&](int word, double v, int at) {
            const uint64_t b = __builtin_bit_cast(uint64_t, v);
            all[word * SLOTS + at] = (uint32_t)b;
            all[(word + 1) * SLOTS + at] = (uint32_t)(b >> 32);
        };
        auto get = [&](int word, int at) -> double { return __builtin_bit_cast(double, (uint64_t)all[(word + 1) * SLOTS + at] << 32 | all[word * SLOTS + at]); };
        auto handed_over = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };   // (one wavefront: LDS accesses are in order)
        double own[P];
        const double own_rw = rw;
        const float own_largest = largest;
        const bool own_constant = constant;
#pragma unroll
        for (int k = 0; k < P; ++k) own[k] = theta[k];
        handed_over();
        if (mine) {
#pragma unroll
            for (int i = 0; i < GL; ++i) all[i * SLOTS + to] = __builtin_bit_cast(uint32_t, wv[i]);
        }
        handed_over();
        float few[LEN];   // (a slot without a group: equal weights)
#pragma unroll
        for (int i = 0; i < LEN; ++i) few[i] = used ? __builtin_bit_cast(float, all[(mine_of * LEN + i) * SLOTS + slot]) : 0.f;
        handed_over();
        if (mine) {
#pragma unroll
            for (int k = 0; k < P; ++k) put(2 * k, theta[k], to);
            put(2 * P, rw, to);
            all[(2 * P + 2) * SLOTS + to] = __builtin_bit_cast(uint32_t, largest);
            all[(2 * P + 3) * SLOTS + to] = constant ? 1u : 0u;
        }
        handed_over();
#pragma unroll
        for (int k = 0; k < P; ++k) theta[k] = used ? get(2 * k, slot) : 0.0;
        rw = used ? get(2 * P, slot) : 0.0;
        largest = used ? __builtin_bit_cast(float, all[(2 * P + 2) * SLOTS + slot]) : 0.f;
        constant = used ? all[(2 * P + 3) * SLOTS + slot] != 0u : true;
        handed_over();
        uint64_t still = changing;
        while (left > 0) {
            --left;
            still = __ballot(iteration(std::false_type{}, few, parts_c) && mine_of == 0);
            if (__popcll(still) <= enough) break;
        }
        handed_over();
        if (used && mine_of == 0) {
#pragma unroll
            for (int k = 0; k < P; ++k) put(2 * k, theta[k], slot);
        }
        handed_over();
#pragma unroll
        for (int k = 0; k < P; ++k) theta[k] = mine ? get(2 * k, to) : own[k];
        rw = own_rw;
        largest = own_largest;
        constant = own_constant;
        return __ballot(mine && (still >> (to * PARTS) & 1));
    };
    while (left > 0) {
        --left;
        uint64_t changing = __ballot(iteration(std::false_type{}, wv, Lanes{}));
        // A group of 64 is at rest after three or four rounds on average, the last of 64 groups after ten.  When half of them are left they
        // get two lanes each, then four.  (Their sums are exact, so the same.)
        if constexpr (L == 1 && G == 64) {
            if (__popcll(changing) <= 32 && left > 2 && __ballot(true) == ~0ull) {
                if (__popcll(changing) > 16) changing = share_out(std::integral_constant<int, 2>{}, changing, 16);
                if (changing != 0 && left > 0) changing = share_out(std::integral_constant<int, 4>{}, changing, 0);   // (rounds left: 16 or fewer change)
                break;
            }
        }
        if (changing == 0) break;
    }
    iteration(std::true_type{}, wv, Lanes{});

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
    auto launch = [&](auto g, auto l) {
        constexpr int G = decltype(g)::value, L = decltype(l)::value, THREADS = Q == 4 ? 256 : quantize_threads(L);
        const dim3 grid((unsigned)(((long)dm.N * L + THREADS - 1) / THREADS), (unsigned)dm.ngroups);
        if constexpr (Q == 4) hlq_quantize_kernel_4<G, L><<<grid, THREADS, 0, st>>>(W, dm.K, dm.N, t_max, codes, scales, zeros, group_err);
        else hlq_quantize_kernel<Q, G, L><<<grid, THREADS, 0, st>>>(W, dm.K, dm.N, t_max, codes, scales, zeros, group_err);
    };
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    using Four = std::integral_constant<int, 4>;
    // Lanes a group: a wavefront for every one of the 1024 SIMDs, if 32 weights or more stay with a lane, and 64 at most of those
    // that are sorted.  Beyond that the thresholds and the solution, which every lane of a group makes, cost what the shorter
    // pass saves.  us, one lane / two / four: 4096 x 1024, G = 64 (1024 wavefronts with one) q = 2 21.5 / 25.6, q = 3 39.5 / 46.6, q = 4
    // 75 / 80;  512 x 512 (64) 18.3 / 15.9, 34.7 / 30.3, 66 / 49;  G = 128, q = 4 512 x 512 101 / 67 / 48, 4096 x 1024 (512) 106 / 75 / 78,
    // 4096 x 4096 180 / 193 / 246.
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
        if constexpr (Q == 4) {
            if (waves > 512) {
                launch(G128{}, One{});
                break;
            }
        }
        if (waves > 256) launch(G128{}, Two{});
        else launch(G128{}, Four{});
        break;
    default:
        if constexpr (Q == 4) {
            if (waves > 256) {
                launch(G256{}, Two{});
                break;
            }
        }
        launch(G256{}, Four{});
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
