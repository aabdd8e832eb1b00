// Kept energy (sum of squares of the s0 largest magnitudes) of one block's coefficients of a
// signal, which sit in the two lanes l and l ^ 32 of a wavefront: the selection networks of the
// block-choice kernels, in fp32 and, two signals at a time, on packed fp16 magnitudes.
#pragma once

#include "device_utils.h"

namespace sbo {

// Both halves of a register pair after v_permlane32_swap(x, z):
//   first  = [x.lo, z.lo]   second = [x.hi, z.hi]   (lo/hi = lanes 0-31 / 32-63)
struct SwapPair {
    float first, second;
};
__device__ __forceinline__ SwapPair swap32(float x, float z) {
    auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x),
                                              __builtin_bit_cast(unsigned, z), false, false);
    const unsigned u0 = r[0], u1 = r[1];   // copy out first: a bit_cast applied to a vector
                                           // element expression reads element 0 for both
    return {__builtin_bit_cast(float, u0), __builtin_bit_cast(float, u1)};
}

// Sum of squares of the N largest magnitudes of the union of two sorted (descending)
// lists, one per lane of a lane pair, of which the first N <= S entries are used (the N
// largest of the union lie among the N largest of either list); valid and bitwise equal in
// both lanes.  The N largest of the union are max(a_i(lo), a_{N-1-i}(hi)); the high lane
// reverses its list so that both operands of one maximum sit in the same register, and one
// swap serves two maxima.
template <int S, int N>
__device__ __forceinline__ float pair_fold_energy(const float (&a)[S], bool hi) {
    static_assert(N >= 1 && N <= S, "fold width");
    if constexpr (N == 1) {
        SwapPair t = swap32(a[0], a[0]);
        const float m = fmaxf(t.first, t.second);
        return m * m;
    } else {
        // r_i = hi ? a_{N-1-i} : a_i as one bit-select per element (written with integer
        // masks so that it is not rewritten into a lane-dependent index into a[])
        const unsigned msk = hi ? 0xffffffffu : 0u;
        float r[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const unsigned fwd = __builtin_bit_cast(unsigned, a[i]);
            const unsigned rev = __builtin_bit_cast(unsigned, a[N - 1 - i]);
            r[i] = __builtin_bit_cast(float, (rev & msk) | (fwd & ~msk));
        }
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i + 1 < N; i += 2) {
            SwapPair t = swap32(r[i], r[i + 1]);
            const float m = fmaxf(t.first, t.second);   // low lanes: maximum i, high: i+1
            sum = fmaf(m, m, sum);
        }
        if constexpr (N % 2 == 1) {            // the middle maximum: the same in both lanes, counted once
            SwapPair t = swap32(r[N - 1], r[N - 1]);
            const float m = fmaxf(t.first, t.second);
            sum = fmaf(hi ? 0.f : m, m, sum);
        }
        SwapPair t = swap32(sum, sum);
        return t.first + t.second;
    }
}

// Energy (sum of squares) of the s0 largest magnitudes in the union of two sorted
// (descending) S-lists of magnitudes, one per lane of a lane pair.  SX = s0 when it is known
// at compile time (S/2 < SX <= S), 0 otherwise.
template <int S, int SX>
__device__ __forceinline__ float pair_list_energy(const float (&a)[S], int s0, bool hi) {
    if constexpr (SX > 0) {
        return pair_fold_energy<S, SX>(a, hi);
    } else {
        float b[S], c[S];
#pragma unroll
        for (int i = 0; i < S; ++i) b[i] = other_half(a[i]);
#pragma unroll
        for (int i = 0; i < S; ++i) c[i] = fmaxf(a[i], b[S - 1 - i]);
        bitonic_merge_desc<S>(c);
        float e = 0.f;
#pragma unroll
        for (int t = 0; t < S; ++t) e += (t < s0) ? c[t] * c[t] : 0.f;
        return e;
    }
}

// The same for the NV magnitudes x held by this lane and the NV held by its partner
// (one block's coefficients of one signal).  S = power of two >= s0, S <= 2 * NV.
template <int NV, int S, int SX>
__device__ __forceinline__ float pair_top_energy(const float (&x)[NV], int s0, bool hi) {
    constexpr int L = S < NV ? S : NV;
    float a[L];
    top_sorted<NV, L>(x, a);
    if constexpr (L == S) {
        return pair_list_energy<S, SX>(a, s0, hi);
    } else {
        static_assert(2 * L == S, "sort width exceeds the coefficients of a lane pair");
        float c[S];
#pragma unroll
        for (int i = 0; i < L; ++i) {
            c[i] = a[i];
            c[S - 1 - i] = other_half(a[i]);
        }
        bitonic_merge_desc<S>(c);
        float e = 0.f;
#pragma unroll
        for (int t = 0; t < S; ++t) e += (t < s0) ? c[t] * c[t] : 0.f;
        return e;
    }
}

// ---- packed fp16 magnitudes: two signals per register ------------------------------------------
// Non-negative fp16 numbers order as unsigned 16-bit integers, so the comparators are v_pk_max_u16
// / v_pk_min_u16: two signals per instruction, and no NaN or denormal rules to pay for.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__host__ __device__ __forceinline__ u16x2 pk_max(u16x2 a, u16x2 b) { return __builtin_elementwise_max(a, b); }
__host__ __device__ __forceinline__ void pk_cmpx_desc(u16x2& a, u16x2& b) {
    const u16x2 hi = __builtin_elementwise_max(a, b), lo = __builtin_elementwise_min(a, b);
    a = hi;
    b = lo;
}

// Sorting networks: Batcher's odd-even mergesort for L = 2, 4, 8 (1, 5, 19 comparators) and Green's
// network of 60 comparators for 16 (Knuth, TAOCP vol. 3, 5.3.4).
template <int L>
struct SortPairs {
    int n = 0;
    short a[64] = {}, b[64] = {};
    constexpr void add(int x, int y) {
        a[n] = (short)x;
        b[n] = (short)y;
        ++n;
    }
    constexpr SortPairs() {
        if (L == 16) {
            for (int d = 1; d < 16; d <<= 1)               // the 4-cube, then what it leaves open
                for (int i = 0; i < 16; ++i)
                    if ((i & d) == 0) add(i, i + d);
            constexpr short rest[28][2] = {{5, 10}, {6, 9},  {3, 12},  {13, 14}, {4, 8},  {7, 11}, {1, 2},
                                           {1, 4},  {7, 13}, {2, 8},   {11, 14}, {2, 4},  {5, 6},  {9, 10},
                                           {11, 13}, {3, 8}, {7, 12},  {6, 8},   {10, 12}, {3, 5}, {7, 9},
                                           {3, 4},  {5, 6},  {7, 8},   {9, 10},  {11, 12}, {6, 7}, {8, 9}};
            for (int c = 0; c < 28; ++c) add(rest[c][0], rest[c][1]);
            return;
        }
        for (int p = 1; p < L; p <<= 1)
            for (int k = p; k >= 1; k >>= 1)
                for (int j = k % p; j + k < L; j += 2 * k)
                    for (int i = 0; i < k && i + j + k < L; ++i)
                        if ((i + j) / (2 * p) == (i + j + k) / (2 * p)) add(i + j, i + j + k);
    }
};
template <int L>
__host__ __device__ __forceinline__ void pk_sort_desc(u16x2 (&v)[L]) {
    constexpr SortPairs<L> net;
#pragma unroll
    for (int c = 0; c < net.n; ++c) pk_cmpx_desc(v[net.a[c]], v[net.b[c]]);
}

// v[0..N) descending and then ascending -> sorted descending, N <= L (a power of two): the bitonic
// network of L entries of which the first L - N are +infinity (in front, so that the sequence
// stays bitonic); comparators with them do nothing.
template <int N, int L>
__host__ __device__ __forceinline__ void pk_bitonic_desc(u16x2 (&v)[N]) {
    constexpr int off = L - N;
#pragma unroll
    for (int half = L / 2; half >= 1; half >>= 1)
#pragma unroll
        for (int i = off; i < L; ++i)
            if ((i & half) == 0) pk_cmpx_desc(v[i - off], v[i + half - off]);
}

constexpr int pow2_at_least(int n) {
    int p = 1;
    while (p < n) p <<= 1;
    return p;
}

// run = the N largest of run and a (both sorted descending), sorted descending.
template <int N>
__host__ __device__ __forceinline__ void pk_merge_top(u16x2 (&run)[N], const u16x2 (&a)[N]) {
    u16x2 t[N];
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] = pk_max(run[i], a[N - 1 - i]);
    pk_bitonic_desc<N, pow2_at_least(N)>(t);
#pragma unroll
    for (int i = 0; i < N; ++i) run[i] = t[i];
}

// The N largest of x[0..NV), sorted descending (N <= NV; NV a power of two).  Groups of 16 by
// Green's network, of which the compiler keeps what the N largest need (100 operations for 8 of
// 16, where two sorts of 8 and their merge take 108; 80 for 6, against 94); shorter lists for N <= 2.
template <int NV, int N>
__host__ __device__ __forceinline__ void pk_top_sorted(const u16x2 (&x)[NV], u16x2 (&out)[N]) {
    constexpr int L = N <= 2 ? pow2_at_least(N) : NV < 16 ? NV : 16;
    static_assert(L <= NV, "list longer than the values");
#pragma unroll
    for (int g = 0; g < NV / L; ++g) {
        u16x2 t[L];
#pragma unroll
        for (int i = 0; i < L; ++i) t[i] = x[g * L + i];
        pk_sort_desc<L>(t);
        u16x2 a[N];
#pragma unroll
        for (int i = 0; i < N; ++i) a[i] = t[i];
        if (g == 0) {
#pragma unroll
            for (int i = 0; i < N; ++i) out[i] = a[i];
        } else {
            pk_merge_top<N>(out, a);
        }
    }
}

// Packed sorted lists (low half: signal of tile 0, high half: of tile 1), one per lane of a lane
// pair -> f(the N largest of the pair's union, packed): the low lane of the pair gets the even ones, the high lane
// the odd ones, and if N is odd both get the last one (second argument of f: it is that one).
template <int N, class F>
__device__ __forceinline__ void pk_pair_top(const u16x2 (&a)[N], bool hi, F f) {
    const unsigned msk = hi ? 0xffffffffu : 0u;
    unsigned r[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {              // the high lanes list theirs in reverse
        const unsigned fwd = __builtin_bit_cast(unsigned, a[i]), rev = __builtin_bit_cast(unsigned, a[N - 1 - i]);
        r[i] = (rev & msk) | (fwd & ~msk);
    }
#pragma unroll
    for (int i = 0; i + 1 < N; i += 2) {       // low lanes: maximum i, high lanes: maximum i + 1
        auto t = __builtin_amdgcn_permlane32_swap(r[i], r[i + 1], false, false);
        const unsigned p = t[0], q = t[1];
        f(pk_max(__builtin_bit_cast(u16x2, p), __builtin_bit_cast(u16x2, q)), false);
    }
    if constexpr (N % 2 == 1) {
        auto t = __builtin_amdgcn_permlane32_swap(r[N - 1], r[N - 1], false, false);
        const unsigned p = t[0], q = t[1];
        f(pk_max(__builtin_bit_cast(u16x2, p), __builtin_bit_cast(u16x2, q)), true);
    }
}

// Sum of squares of the N largest: lanes 0-31 receive that of their signal in tile 0, lanes 32-63
// that of their signal in tile 1.
template <int N>
__device__ __forceinline__ float pk_pair_energy(const u16x2 (&a)[N], bool hi) {
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    float s0 = 0.f, s1 = 0.f;
    pk_pair_top<N>(a, hi, [&](u16x2 v, bool both) {
        const f16x2 w = __builtin_bit_cast(f16x2, __builtin_bit_cast(unsigned, v) & (both && hi ? 0u : 0xffffffffu));
        s0 = fmaf((float)w[0], (float)w[0], s0);
        s1 = fmaf((float)w[1], (float)w[1], s1);
    });
    const SwapPair t = swap32(s0, s1);
    return t.first + t.second;
}

}  // namespace sbo
