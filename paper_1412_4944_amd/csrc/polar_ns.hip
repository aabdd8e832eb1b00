// Orthogonal polar factor Q_j = U V^T of P_j (Algorithm 1, steps 6-7) for p <= 64 by the
// Newton-Schulz iteration X <- X (3 I - X^T X) / 2 on the matrix cores, one workgroup per block.
//
// U V^T is the orthogonal polar factor of P_j, and for a matrix scaled to singular values in
// (0, sqrt(3)) the iteration converges to it quadratically; each step is two p x p x p products,
// which are dense contractions, where the Jacobi SVD is p - 1 dependent rounds of plain ALU
// work per sweep.  A block that has not converged after max_iters steps (rank-deficient or nearly
// so, zero, NaN) is handed, in the same workgroup, to the one-sided Jacobi SVD (jacobi_block.h),
// which also supplies the orthonormal completion a vanishing singular value needs.
//
// What bounds it: one workgroup on one CU per block, every step waiting for the one before, so
// the time is the number of steps times the latency of a step.  Both are kept small:
//   * Steps.  The singular values are pulled towards one by scaling X before a step: with all of
//     them in [l, 1], X sqrt(3 / (1 + l + l^2)) makes the step's polynomial map [l, 1] to the
//     smallest possible interval [l', 1].  A smaller singular value is safe (the polynomial never
//     exceeds one and is positive on (0, sqrt(3))), it only takes longer; a larger l than the guess costs steps and rounding (the
//     largest values are sent down to l' first, where an error weighs 1 / l' as much).  l starts at a guess from the spread of
//     the squared singular values, |G|_F^2 / (p mu^2) - 1 with mu = tr G / p, which the first product shows (kSpread).  The last step
//     is quintic, X (I + c1 E + c2 E^2), E = I - X^T X (ns_scale.h).  Four to seven steps where the plain iteration takes seven
//     to ten.
//   * The step.  Two wavefronts have a strip of 16 columns of X (16x16x32 MFMA tiles, four
//     consecutive rows of one column per lane and tile), half of its row tiles each; a wavefront alone on its SIMD issues
//     a vector instruction every 8 cycles, and its LDS reads, products and splits then follow one another.
//     An accumulator tile is at the same time
//     the B operand of the next product, up to an order of the contraction index that the A
//     operand shares: X^T X takes its B operand from the registers that hold X, X E takes it from
//     the registers that hold E (each with the other wavefront's half from LDS), and the A operands (the other strips'
//     columns of X, and, transposed by ds_read_b64_tr_b16 on the way out, its rows) go through LDS.  G and E are symmetric:
//     at p = 64 ten of their sixteen tiles are computed and the others read transposed.
//   * The products run at fp32 accuracy.  p < 64: every entry is the exact sum of three bf16 parts
//     (device_utils.h), six partial products with fp32 accumulation; three for E^2 in the last step, which is
//     below 1e-4 and added to E.  p = 64, where LDS moves 240 KB a step with three parts: two fp16 parts, three partial
//     products.  They leave 2^-22 of an entry.  In G that is a symmetric error, which the next step takes out; for the last
//     step the products that were left out are added.  What is left in X E is made up for by three roundings less: E is scaled by the
//     mantissa of alpha, so that the products are added to X without one, and the two steps of a contraction are summed apart.
//     |Q - Q64|_F / sqrt(p) on block matrices of training rounds (96 to 65536 signals, condition 1.3 to 700) 0.54 to 1.05 of that with three
//     parts and l = 0.16, on average 0.81 (p = 32 0.91, p = 16 0.94: the guess alone; more at kSpread); p = 32, 16 with two parts 1.3 and 1.5, in the same time.
//   * The steps' branches are those of scalars: as the sum that decides comes out of lanes, the compiler would take every one of
//     them for divergent (p = 16: 2 % of an iteration).
// Measured (p = 64, launch to launch): inside sbo_iterate (K = 16, 16384 signals) 22.4 us with a wavefront per strip, 19.5 with two; the kernel
// alone 18.4 there, 16.4 with two parts, 14.6 with the guess (seven steps -> six); on average in sbo_learn (K = 1 to 16) 17.8, 16.0, 14.7.  p = 32 8.8 -> 8.0 us, p = 16 6.8.  Of 37000 cycles
// at p = 64, K = 16 (seven steps, before the guess): the sum of the pieces 8000 (a CU takes 25 to 40 bytes a cycle of what others have just
// written), the scale of the input 2000, a step 3500, the last one's E^2 1300, output 2200.
//
// The same launch can (a) sum the per-piece partial matrices of the fused select + accumulate
// kernel on the way in, in piece order, which saves the separate reduction launch, and (b) form
// the total squared error of the coding pass in extra workgroups.
//
// X is the transpose of the stored, atom-major matrix, so a lane's four consecutive rows are
// four consecutive dims of an atom (16-byte loads and stores), and X^T X is the Gram matrix of
// P_j's columns weighted by the codes: nearly diagonal, which makes its row sums a good bound.
#include "sbo_internal.h"
#include "device_utils.h"
#include "jacobi_block.h"
#include "ns_scale.h"
#include "sq_total.h"

namespace sbo {

namespace {

struct NsArgs {
    const float* M;            // [K][p][p] finished matrices, or nullptr: sum the pieces
    const float* partial;      // [pieces][p][p] (M == nullptr)
    const int32_t* offsets;    // [K+1] (M == nullptr): the grouping the pieces were cut from
    int piece;                 // signals per piece
    const int32_t* counts;     // [K] or nullptr
    float* D;
    DictOps ops;               // the new atoms in the coding kernels' operand orders
    int32_t* fallback;         // [K] 1 = the block went to the Jacobi SVD
    int32_t* iters_out;        // [K] minus the Newton-Schulz steps, or the Jacobi sweeps
    int max_iters;
    int K;
    // total squared error (extra workgroups), or sq_out == nullptr
    const float* err;
    int64_t m;
    double* sq_part;
    int* sq_counter;
    double* sq_out;
    int nb;
    // histograms that this launch sets to zero (ChunkLists), or n_clear == 0
    int32_t* clear;
    int n_clear;
};

// sqrt(3 / (1 + l + l^2)) for a first l and then the l that the steps leave: from k = 1 on 0.064, 0.16 (k = 2), 0.37, 0.72, 0.96; from 8 on
// 0.45, 0.80, 0.98; from 14 on 0.09, 0.22, 0.49, 0.83, 0.99; one elsewhere (a chain of selects: a table would be read from memory in
// every step).
__device__ __forceinline__ float step_alpha(int k) {
    float a = 1.f;
    a = k == 1 ? 1.67603f : a;
    a = k == 2 ? 1.5907f : a;
    a = k == 3 ? 1.4081f : a;
    a = k == 4 ? 1.1601f : a;
    a = k == 5 ? 1.0206f : a;
    a = k == 14 ? 1.65287f : a;
    a = k == 15 ? 1.53661f : a;
    a = k == 16 ? 1.31621f : a;
    a = k == 17 ? 1.0889f : a;
    a = k == 18 ? 1.00613f : a;
    a = k == 8 ? 1.34738f : a;
    a = k == 9 ? 1.11f : a;
    return k == 10 ? 1.00948f : a;
}

// Where l starts, by the spread of the squared singular values: 0.45, 0.16, 0.09, 0.064.  Steps simulated in 64 bits on block matrices of
// training rounds, with 0.45 / 0.16: spread 0.13 to 0.15 4 / 5, 0.2 to 0.3 5 / 5, beyond 0.3 5.2 to 7 / 5; with 0.16 / 0.09: up to 0.7
// 5.0 / 6, 0.7 to 0.9 5.8 / 6, 0.9 to 1 6.1 / 6, 1 to 1.4 6.7 / 6.1; with 0.09 / 0.064 beyond 1.4 7.8 / 7.2.  Error against 64 bits (rms over 128
// block matrices each of 1024 to 2896 signals, s0 = 2 to 8, of that with three parts and 0.16 throughout): with the second line at 0.6
// 0.92 to 1.02, at 0.75 0.91 to 1.005, at 0.9 0.90 to 0.995, where the slowest block of a launch is one of seven steps more often (ten iterations,
// 16384 signals, K = 16 366 -> 370 us, sbo_learn 5645 -> 5710); 0.064 instead of 0.09 up to 1.15.  What the spread does not show is a
// single late value among equal ones (an atom that hardly any signal uses): with 0.45 a step more than with 0.16 (condition 100: 13 instead of 12).
// Lower l lose accuracy (0.025 beyond
// 1.4: up to 1.5 of the error), and so do 0.09 and 0.064 for p < 64, which stays with 0.16 there (1.28).
constexpr float kSpread[3] = {0.18f, 0.75f, 1.4f};
// X and E are split in two fp16 parts each (device_utils.h), times this: no singular value is above one after a step, no
// entry of E above 1.9.
template <int P>
constexpr int ns_parts() { return P == 64 ? 2 : 3; }
template <int P>
constexpr float ns_scale() { return ns_parts<P>() == 2 ? 16384.f : 1.f; }
// alpha = mantissa (in [1, 2)) times power of two, for normal numbers above zero
__device__ __forceinline__ float mantissa(float alpha) {
    return __builtin_bit_cast(float, (__builtin_bit_cast(unsigned, alpha) & 0x007fffffu) | 0x3f800000u);
}
__device__ __forceinline__ float power_of_two(float alpha) {
    return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, alpha) & 0x7f800000u);
}
// Power of two that brings entries of at most this magnitude (its bits) below kScale (three parts: 2), so that neither the parts nor the
// sums of fourth powers that show the spread leave their range; zero, so that the block goes to the Jacobi SVD, where sums of
// squares would.
template <int P>
__device__ __forceinline__ float input_scale(unsigned mx) {
    const unsigned e = mx >> 23;               // biased exponent
    if (e < 64u || e > 190u) return 0.f;
    return __builtin_bit_cast(float, (unsigned)(127 + (ns_parts<P>() == 2 ? 13 : 0) + 127 - (int)e) << 23);
}

// wavefronts per strip of 16 columns: they share out its row tiles
template <int P>
constexpr int ns_halves() {
    return P > 16 ? 2 : 1;
}
template <int P>
constexpr int ns_threads() {
    return P * 4 * ns_halves<P>();
}
// bytes of one LDS image of X or E: per strip and contraction step of 32, three parts of 64 lanes x 16 bytes
template <int P>
constexpr int ns_image_bytes() {
    return (P / 16) * ((P / 16 + 1) / 2) * ns_parts<P>() * 1024;
}
// dynamic LDS: two images (the Jacobi routine reuses this part) | red[2][8 wavefronts] | cols[6][P] floats
template <int P>
constexpr size_t ns_front_bytes() {
    const size_t rest = ns_parts<P>() == 2 ? ns_image_bytes<P>() / 2 : 0;      // what two parts leave, in the last step
    const size_t img = (size_t)2 * ns_image_bytes<P>() + rest, jac = (size_t)jacobi_lds_floats<P>() * 4;
    const size_t sq = (size_t)(ns_threads<P>() + 2) * 8;
    const size_t a = img > jac ? img : jac;
    return ((a > sq ? a : sq) + 15) / 16 * 16;
}
template <int P>
constexpr size_t ns_lds_bytes() {
    return ns_front_bytes<P>() + 16 * 4 + 6 * P * 4;
}

// Sums over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (bitwise the same in all of them).
__device__ __forceinline__ float sum_groups(float x) {
    const unsigned u = __builtin_bit_cast(unsigned, x);
    auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned a0 = r[0], a1 = r[1];
    const float y = __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1);
    const unsigned w = __builtin_bit_cast(unsigned, y);
    auto q = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    const unsigned b0 = q[0], b1 = q[1];
    return __builtin_bit_cast(float, b0) + __builtin_bit_cast(float, b1);
}
// Maximum over the 16 lanes of a row of non-negative values; a NaN wins (its bits are the largest).
__device__ __forceinline__ float row_max_nan(float x) {
    unsigned u = __builtin_bit_cast(unsigned, x);
    auto step = [&](auto f) { u = max(u, __builtin_bit_cast(unsigned, f(__builtin_bit_cast(float, u)))); };
    step([](float v) { return dpp_f<kDppXor1>(v); });
    step([](float v) { return dpp_f<kDppXor2>(v); });
    step([](float v) { return dpp_f<kDppHalfMirror>(v); });
    step([](float v) { return dpp_f<kDppRowMirror>(v); });
    return __builtin_bit_cast(float, u);
}

// Over the wavefront, in all lanes.
__device__ __forceinline__ float wave_sum(float x) { return sum_groups(group_sum<16>(x)); }
__device__ __forceinline__ float wave_max_nan(float x) {
    unsigned u = __builtin_bit_cast(unsigned, row_max_nan(x));
    auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned a0 = r[0], a1 = r[1];
    u = max(a0, a1);
    auto q = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const unsigned b0 = q[0], b1 = q[1];
    return __builtin_bit_cast(float, max(b0, b1));
}

// What all lanes agree on, as the compiler is to know it: the steps and their branches then are those of scalars.
__device__ __forceinline__ float uniform(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}
__device__ __forceinline__ bool uniform(bool x) { return __builtin_amdgcn_readfirstlane((int)x) != 0; }

// The iteration and the output, for the wavefronts that have the first (HH = 0) or the second half of a strip's row tiles
// (the branch between the two is what a choice of registers per lane costs otherwise: 48 selects a step); barriers are the
// same in both.  Returns the steps, or 0: not converged.  xr[a][r] = X[t*16 + grp*4 + r][col], t = HH*TH + a.
template <int P, int HH>
__device__ __forceinline__ int iterate(const NsArgs& g, int j, int strip, f32x4 (&xr)[P / 16 / ns_halves<P>()],
                                       unsigned char* lds_raw, float* red, float* cols) {
    constexpr int T = P / 16, S = (T + 1) / 2, HV = ns_halves<P>(), TH = T / HV, NW = T * HV, hh = HH;
    // G and E are symmetric: at p = 64 the fourth tile of a strip is the transpose of the second of another one
    constexpr bool SYM = T == 4;
    constexpr float kScale = ns_scale<P>();
    constexpr int NE = SYM && hh == 1 ? 1 : TH;          // tiles of E of this wavefront
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = lane >> 4, c16 = lane & 15, col = strip * 16 + c16;

    // The parts of a row tile, two words each: lane (grp, c16) holds rows grp*4 .. +3 of column c16.
    constexpr int NPT = ns_parts<P>();
    struct Parts {
        u32x2 p[NPT];
    };
    auto split_tile = [](f32x4 v) {
        if constexpr (NPT == 2) {
            const F16x2Pair a = split_f16x2(v.x, v.y), b = split_f16x2(v.z, v.w);
            return Parts{{u32x2{a.hi, b.hi}, u32x2{a.lo, b.lo}}};
        } else {
            const Bf16x3Pair a = split_bf16x3(v.x, v.y), b = split_bf16x3(v.z, v.w);
            return Parts{{u32x2{a.hi, b.hi}, u32x2{a.mid, b.mid}, u32x2{a.lo, b.lo}}};
        }
    };
    auto remainder = [](f32x4 v, const Parts& w) {             // what two parts leave of a tile, as fp16
        typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
        const unsigned u0 = w.p[0].x, u1 = w.p[0].y, v0 = w.p[1].x, v1 = w.p[1].y;
        const f16x2 h0 = __builtin_bit_cast(f16x2, u0), h1 = __builtin_bit_cast(f16x2, u1);
        const f16x2 l0 = __builtin_bit_cast(f16x2, v0), l1 = __builtin_bit_cast(f16x2, v1);
        return u32x2{pack_f16(v.x - (float)h0[0] - (float)l0[0], v.y - (float)h0[1] - (float)l0[1]),
                     pack_f16(v.z - (float)h1[0] - (float)l1[0], v.w - (float)h1[1] - (float)l1[1])};
    };
    // The LDS image: per (strip, step, part) 1 KiB, tile 2s in the first half, tile 2s+1 in the
    // second, 8 bytes per (grp, c16), the upper two groups with their columns exchanged by eights:
    // 32 consecutive lanes of a write, of a straight and of a transposing read each cover all banks.
    const int lane_at = (grp * 16 + (c16 ^ ((grp >> 1) * 8))) * 8;
    auto unit = [&](unsigned char* img, int st, int t, int pl) { return img + ((st * S + (t >> 1)) * NPT + pl) * 1024 + (t & 1) * 512; };
    auto rest = [&](int st, int t) { return lds_raw + 2 * ns_image_bytes<P>() + (st * S + (t >> 1)) * 1024 + (t & 1) * 512; };
    auto write_tile = [&](unsigned char* img, int t, const Parts& w) {       // of the own strip
#pragma unroll
        for (int pl = 0; pl < NPT; ++pl) *reinterpret_cast<u32x2*>(unit(img, strip, t, pl) + lane_at) = w.p[pl];
    };
    auto read_tile = [&](unsigned char* img, int st, int t, int pl) {
        return *reinterpret_cast<const u32x2*>(unit(img, st, t, pl) + lane_at);
    };
    // half of an A operand whose row m is row t*16 + m of X (contraction over columns: lane (grp, .) takes
    // columns grp*4 .. +3 of strip st).  ds_read_b64_tr_b16: of the 16 lanes of a row, lane
    // i addresses four consecutive rows (4 (i & 3) ..) of column grp*4 + (i >> 2) and receives row i
    // of the four columns.
    const int tr_at = ((c16 & 3) * 16 + ((grp * 4 + (c16 >> 2)) ^ (((c16 & 3) >> 1) * 8))) * 8;
    auto read_rows = [&](unsigned char* img, int st, int t, int pl) {
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) s16x4* lds_ptr;
        const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(unit(img, st, t, pl) + tr_at));
        return __builtin_bit_cast(u32x2, a);
    };
    // tile number i of strip st of E
    auto read_e = [&](unsigned char* img, int st, int i, int pl) {
        return SYM && i == 3 ? read_rows(img, (st + 3) & 3, 1, pl) : read_tile(img, st, i, pl);
    };
    auto mfma = [](u32x2 a0, u32x2 a1, u32x2 b0, u32x2 b1, f32x4 c) {
        const u32x4 a = {a0.x, a0.y, a1.x, a1.y}, b = {b0.x, b0.y, b1.x, b1.y};
        if constexpr (NPT == 2)
            return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
        else
            return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    };
    // the partial products, smallest first: (A part, B part)
    constexpr int NP = NPT == 2 ? 3 : 6;
    constexpr int TA[6] = {NPT == 2 ? 1 : 2, 0, NPT == 2 ? 0 : 1, 1, 0, 0};
    constexpr int TB[6] = {0, NPT == 2 ? 1 : 2, NPT == 2 ? 0 : 1, 0, 1, 0};
    constexpr int kOrder[3] = {NPT - 1, 0, 1}; // in which they first use the parts
    const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
    const u32x2 none = {0u, 0u};
    // Row tiles of G and E are kept in the order strip, strip + 1, ... (mod T); this wavefront has numbers
    // hh*TH .. of them.  Number 0 is the tile on the diagonal.
    int strip_of[T];
#pragma unroll
    for (int i = 0; i < T; ++i) strip_of[i] = (strip + i) & (T - 1);
    auto mine = [&](int a) { return (strip + hh * TH + a) & (T - 1); };
    f32x4 diag[NE];                            // what this wavefront's tiles have of I
#pragma unroll
    for (int a = 0; a < NE; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) diag[a][r] = hh == 0 && a == 0 && grp * 4 + r == c16 ? 1.f : 0.f;
    // all tiles of a strip as B operands: the own parts, and those of the other wavefront from the image
    auto whole = [&](unsigned char* img, const Parts (&own)[TH], Parts (&all)[T]) {
        if constexpr (HV == 1) {
            all[0] = own[0];
        } else {
#pragma unroll
            for (int k = 0; k < NPT; ++k)
#pragma unroll
                for (int a = 0; a < TH; ++a) {
                    all[hh * TH + a].p[kOrder[k]] = own[a].p[kOrder[k]];
                    all[(1 - hh) * TH + a].p[kOrder[k]] = read_tile(img, strip, (1 - hh) * TH + a, kOrder[k]);
                }
        }
    };
    auto whole_e = [&](unsigned char* img, const Parts (&own)[NE], Parts (&all)[T]) {
#pragma unroll
        for (int k = 0; k < NPT; ++k)
#pragma unroll
            for (int i = 0; i < T; ++i)
                all[i].p[kOrder[k]] = i >= hh * TH && i < hh * TH + NE ? own[(i - hh * TH) % NE].p[kOrder[k]] : read_e(img, strip, i, kOrder[k]);
    };
    // one value per wavefront -> the sum over the workgroup; slot: 0, 1, reused two barriers later at the earliest
    auto publish = [&](int slot, float v) {
        if (lane == 0) red[slot * 8 + wave] = v;
    };

    unsigned char* const ximg = lds_raw;
    unsigned char* const eimg = lds_raw + ns_image_bytes<P>();
    int it = 0;
    int first = 0, first_test = 1;             // the step's place in step_alpha's order; the first one that can be the last
    while (true) {
        Parts xo[TH], xq[T];
#pragma unroll
        for (int a = 0; a < TH; ++a) {
            xo[a] = split_tile(xr[a]);
            write_tile(ximg, hh * TH + a, xo[a]);
        }
        __syncthreads();

        // this wavefront's tiles of G = X^T X
        f32x4 ge[NE];
        u32x2 rows[T][NPT][TH];
        {
            u32x2 a[T][NPT][NE];                 // requested in the order in which the products use them
            whole(ximg, xo, xq);
#pragma unroll
            for (int k = 0; k < NPT; ++k)
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int i = 0; i < NE; ++i) {
                        if (hh == 0 && i == 0) continue;       // the diagonal tile: the own strip
                        a[2 * s][kOrder[k]][i] = read_tile(ximg, mine(i), 2 * s, kOrder[k]);
                        if (2 * s + 1 < T) a[2 * s + 1][kOrder[k]][i] = read_tile(ximg, mine(i), 2 * s + 1, kOrder[k]);
                    }
            // The A operands of X E: on their way during the products of G.
#pragma unroll
            for (int k = 0; k < NPT; ++k)
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int i = 0; i < TH; ++i) {
                        rows[2 * s][kOrder[k]][i] = read_rows(ximg, strip_of[2 * s], hh * TH + i, kOrder[k]);
                        if (2 * s + 1 < T)
                            rows[2 * s + 1][kOrder[k]][i] = read_rows(ximg, strip_of[2 * s + 1 < T ? 2 * s + 1 : 0], hh * TH + i, kOrder[k]);
                    }
#pragma unroll
            for (int i = 0; i < NE; ++i) ge[i] = zero4;
            f32x4 g1[NE];                      // the second step's: two shorter chains, and less is rounded
#pragma unroll
            for (int i = 0; i < NE; ++i) g1[i] = zero4;
#pragma unroll
            for (int q = 0; q < NP; ++q)
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int i = 0; i < NE; ++i) {
                        constexpr int last = T - 1;
                        const int t1 = 2 * s + 1 < T ? 2 * s + 1 : last;
                        const bool own = hh == 0 && i == 0;
                        f32x4& sum = s > 0 ? g1[i] : ge[i];
                        sum = mfma(own ? xq[2 * s].p[TA[q]] : a[2 * s][TA[q]][i],
                                   T == 1 ? none : own ? xq[t1].p[TA[q]] : a[t1][TA[q]][i], xq[2 * s].p[TB[q]],
                                   T > 1 ? xq[t1].p[TB[q]] : none, sum);
                    }
            if constexpr (S > 1) {
#pragma unroll
                for (int i = 0; i < NE; ++i) ge[i] += g1[i];
            }
        }

        float alpha = step_alpha(first + min(it, 5)) / kScale;               // xr times this is X, scaled as the step wants it
        bool last = false;
        float fr_own = 0.f;
        // Whether this can be the last step.  Not the second and the third of a spectrum that is not narrow: two scaled steps
        // leave values that were more than a tenth apart further from one than the line allows.  (NaN stays NaN.)
        const bool test = it >= first_test;
        if (it == 0) {
            // The scale of the input.  The iteration sends every singular value in (0, sqrt(3)) to
            // +1, one in (sqrt(3), sqrt(5)) to -1 (an orthogonal matrix that is NOT U V^T, and
            // which no later test can tell apart), so the scale must be a guaranteed bound: the
            // largest absolute row sum of G is at least its largest eigenvalue sigma_max^2, and
            // alpha^2 <= 2.9 / that keeps every scaled sigma^2 below 2.9.  Where the bound is tight, the
            // aim is sigma_max = 1 times the scaling for l, with the largest norm of a column of
            // G (a lower bound of its largest eigenvalue) as the estimate; a narrow spectrum (ns_scale.h) is
            // centred at one.
            float rs = 0.f, r2 = 0.f, tr = 0.f;
#pragma unroll
            for (int i = 0; i < NE; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    rs += fabsf(ge[i][r]);
                    r2 = fmaf(ge[i][r], ge[i][r], r2);
                    tr = fmaf(diag[i][r], ge[i][r], tr);
                }
            rs = sum_groups(rs);
            r2 = sum_groups(r2);
            float rsmax, r2max, sum2, mu = sum_groups(group_sum<16>(tr));
            if constexpr (NW == 1) {
                rsmax = row_max_nan(rs);
                r2max = row_max_nan(r2);
                sum2 = group_sum<16>(r2);
            } else {
                publish(0, mu);
                if (grp == 0) {
                    cols[hh * P + col] = rs;
                    cols[(3 + hh) * P + col] = r2;
                }
                if constexpr (SYM && hh == 0) {    // the second tile, by rows
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float v = ge[NE - 1][r], a = group_sum<16>(fabsf(v)), q = group_sum<16>(v * v);
                        if (c16 == r) {
                            cols[2 * P + mine(1) * 16 + grp * 4 + r] = a;
                            cols[5 * P + mine(1) * 16 + grp * 4 + r] = q;
                        }
                    }
                }
                __syncthreads();
                const int c = lane & (P - 1);      // (p < 64: every column 64 / p times)
                rsmax = cols[c] + cols[P + c];
                r2max = cols[3 * P + c] + cols[4 * P + c];
                mu = red[0];
                if constexpr (SYM) {
                    rsmax += cols[2 * P + c];
                    r2max += cols[5 * P + c];
                }
                sum2 = wave_sum(r2max) * (P / 64.f);
                rsmax = wave_max_nan(rsmax);
                r2max = wave_max_nan(r2max);
#pragma unroll
                for (int w = 1; w < NW; ++w) mu += red[w];
            }
            mu *= 1.f / P;
            // zero, infinite, NaN or overflowing input: not for this iteration
            if (!uniform(rsmax > 1e-37f && rsmax < 3e37f)) return 0;
            float b2 = 2.9f * __builtin_amdgcn_rcpf(rsmax);
            const float r = __builtin_amdgcn_rcpf(mu), spread = uniform((sum2 * r) * (r * (1.f / P))) - 1.f;
            if (spread < kNarrow<P> * kNarrow<P>) {
                b2 = fminf(b2, __builtin_amdgcn_rcpf(mu));
                first = 20;                    // as it is
            } else {
                first = spread < kSpread[0] ? 8 : spread < kSpread[1] || P < 64 ? 2 : spread < kSpread[2] ? 14 : 1;
                first_test = spread < kSpread[1] || P < 64 ? 3 : 4;
                const float a0 = step_alpha(first);
                if (r2max > 1e-37f && r2max < 3e37f) b2 = fminf(b2, a0 * a0 * (1.f / 1.04f) * __builtin_amdgcn_rsqf(r2max));
            }
            alpha = uniform(__builtin_amdgcn_sqrtf(b2));
        } else if (test) {
            float fr = 0.f;
#pragma unroll
            for (int i = NE - 1; i >= 0; --i) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float e = fmaf(-1.f / (kScale * kScale), ge[i][r], diag[i][r]);
                    fr = fmaf(e, e, fr);
                }
                if (SYM && hh == 0 && i == 1) fr *= 2.f;       // and its transpose
            }
            fr_own = sum_groups(group_sum<16>(fr));
            if constexpr (NW > 1) publish(it & 1, fr_own);
        }
        // E = I - alpha^2 G (times kScale), then X <- alpha (X + X E / 2)
        f32x4 eo[NE];
        Parts ep[NE], eq[T];
        // (times the mantissa of alpha: what the products add to X is then scaled by a power of two, without a rounding)
        auto make_e = [&]() {
            const float beta = NPT == 2 ? mantissa(alpha) : 1.f, a2 = beta * kScale * alpha * alpha;
#pragma unroll
            for (int i = 0; i < NE; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float e = (beta * kScale) * diag[i][r] - a2 * ge[i][r];
                    asm("" : "+v"(e));         // (or it is rounded to fp16 in a second such instruction, twice)
                    eo[i][r] = e;
                }
        };
        auto share_e = [&](bool image) {       // its parts, and to the image
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                ep[i] = split_tile(eo[i]);
                if (image) write_tile(eimg, hh * TH + i, ep[i]);
            }
        };
        make_e();
        share_e(HV > 1);
        if (NW > 1) __syncthreads();           // (and the last reads of X's image)
        whole_e(eimg, ep, eq);
        if (test) {                            // has this been the last but one step?
            float fr = NW > 1 ? red[(it & 1) * 8] : fr_own;
#pragma unroll
            for (int w = 1; w < NW; ++w) fr += red[(it & 1) * 8 + w];
            fr = uniform(fr);
            if (!(fr < 2.f * P)) return 0;     // NaN or diverging: leave it to the Jacobi SVD
            last = fr < kLastEps * kLastEps;   // |E|_F, a bound on the spectral norm of E
            if (!last && it >= g.max_iters) return 0;
        }
        if (last) {                            // uniform
            if constexpr (NPT == 2) {
#pragma unroll
                for (int a = 0; a < TH; ++a) *reinterpret_cast<u32x2*>(rest(strip, hh * TH + a) + lane_at) = remainder(xr[a], xo[a]);
            }
            if (HV == 1 || alpha != 1.f / kScale) {            // uniform: E without the scaling
                __syncthreads();               // (E's image has been read)
                alpha = 1.f / kScale;
                make_e();
                share_e(true);
                __syncthreads();
                whole_e(eimg, ep, eq);
            }
            // E^2 from the three largest partial products: 2^-16 of something below 1e-4
            f32x4 e2[NE];
#pragma unroll
            for (int i = 0; i < NE; ++i) e2[i] = zero4;
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int i = 0; i < NE; ++i) {
                    // E is symmetric: its rows are the strips, each with its tiles in its own order
                    const int pa = (2 * s - hh * TH - i) & (T - 1), pb = (pa + 1) & (T - 1);
                    u32x2 lo[2], hi[2];
#pragma unroll
                    for (int pl = 0; pl < 2; ++pl) {
                        lo[pl] = read_e(eimg, mine(i), pa, pl);
                        hi[pl] = T > 1 ? read_e(eimg, mine(i), pb, pl) : none;
                    }
                    const int t1 = T > 1 ? 2 * s + 1 : 0;
                    auto b = [&](int pl) { return T > 1 ? eq[t1].p[pl] : none; };
                    e2[i] = mfma(lo[1], hi[1], eq[2 * s].p[0], b(0), e2[i]);
                    e2[i] = mfma(lo[0], hi[0], eq[2 * s].p[1], b(1), e2[i]);
                    e2[i] = mfma(lo[0], hi[0], eq[2 * s].p[0], b(0), e2[i]);
                }
            __syncthreads();                   // E's image has been read
            if constexpr (NPT == 2) {
                // What the two parts have left out of G, where it decides the rounding of the result: the products of
                // what they leave of X, and on the diagonal, where they add up, those of the second parts.
                f32x4 c[NE];
#pragma unroll
                for (int i = 0; i < NE; ++i) c[i] = zero4;
                auto rest_tile = [&](int st, int t) { return *reinterpret_cast<const u32x2*>(rest(st, t) + lane_at); };
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const u32x2 x0 = read_tile(ximg, strip, 2 * s, 0), x1 = read_tile(ximg, strip, 2 * s + 1, 0);
                    const u32x2 d0 = rest_tile(strip, 2 * s), d1 = rest_tile(strip, 2 * s + 1);
#pragma unroll
                    for (int i = 0; i < NE; ++i) {
                        c[i] = mfma(read_tile(ximg, mine(i), 2 * s, 0), read_tile(ximg, mine(i), 2 * s + 1, 0), d0, d1, c[i]);
                        c[i] = mfma(rest_tile(mine(i), 2 * s), rest_tile(mine(i), 2 * s + 1), x0, x1, c[i]);
                    }
                    if (hh == 0) {
                        const u32x2 l0 = read_tile(ximg, strip, 2 * s, 1), l1 = read_tile(ximg, strip, 2 * s + 1, 1);
                        c[0] = mfma(l0, l1, l0, l1, c[0]);
                    }
                }
#pragma unroll
                for (int i = 0; i < NE; ++i) eo[i] -= (1.f / kScale) * c[i];
            }
#pragma unroll
            for (int i = 0; i < NE; ++i) eo[i] = kLastLinear * eo[i] + (kLastSquare / kScale) * e2[i];
            share_e(HV > 1);
            if (HV > 1) __syncthreads();
            whole_e(eimg, ep, eq);
        }
        // row tiles of X E
        f32x4 acc[TH], acc1[TH];
#pragma unroll
        for (int i = 0; i < TH; ++i) acc[i] = acc1[i] = zero4;
#pragma unroll
        for (int q = 0; q < NP; ++q)
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int i = 0; i < TH; ++i) {
                    const int t1 = T > 1 ? 2 * s + 1 : 0;
                    f32x4& sum = s > 0 ? acc1[i] : acc[i];
                    sum = mfma(rows[2 * s][TA[q]][i], T > 1 ? rows[t1][TA[q]][i] : none, eq[2 * s].p[TB[q]],
                               T > 1 ? eq[t1].p[TB[q]] : none, sum);
                }
#pragma unroll
        for (int i = 0; i < TH; ++i) {
            if constexpr (S > 1) acc[i] += acc1[i];
            xr[i] = (kScale * alpha) * xr[i] + (0.5f * (NPT == 2 ? power_of_two(alpha) : alpha)) * acc[i];
        }
        ++it;
        if (last) break;
    }
#pragma unroll
    for (int a = 0; a < TH; ++a) xr[a] *= 1.f / kScale;

    // D[j][k][:] = column k of X; the same values in the coding kernels' operand orders
    f32x4* Dj = reinterpret_cast<f32x4*>(g.D + (int64_t)j * P * P);
    float q2 = 0.f, r2 = 0.f;
#pragma unroll
    for (int a = 0; a < TH; ++a) {
        const int d4 = (hh * TH + a) * 4 + grp;
        Dj[col * (P / 4) + d4] = xr[a];
        if (g.ops.f32 != nullptr) store_operand_f32<P>(g.ops.f32, j * P + col, d4, xr[a]);
        if (g.ops.bf16 != nullptr) store_operand_split<P>(g.ops.bf16, j * P + col, d4, xr[a]);
        if (g.ops.f16 != nullptr) store_operand_f16x2<P>(g.ops.f16, j * P + col, d4, split_f16x2_dict(xr[a], q2, r2));
    }
    if (g.ops.f16 != nullptr) {                // uniform
        q2 = sum_groups(q2);
        r2 = sum_groups(r2);
        if constexpr (HV > 1) {                // (cols: last read in the first step)
            if (hh == 1 && grp == 0) {
                cols[col] = q2;
                cols[P + col] = r2;
            }
            __syncthreads();
            q2 += cols[col];
            r2 += cols[P + col];
        }
        q2 = row16_max(q2);
        r2 = row16_max(r2);
        if (lane == 0 && hh == 0) g.ops.dnorm[j * T + strip] = float2{sqrtf(q2), sqrtf(r2)};
    }
    return it;
}

template <int P>
__global__ __launch_bounds__(ns_threads<P>()) void polar_ns_kernel(NsArgs g) {
    constexpr int T = P / 16;                  // tiles per side = strips
    constexpr int HV = ns_halves<P>(), TH = T / HV;            // wavefronts of a strip, row tiles of each
    constexpr int NTH = ns_threads<P>();
    constexpr int TPP_FALLBACK = NTH / (P / 2);          // the Jacobi routine with this workgroup's threads
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    float* red = reinterpret_cast<float*>(lds_raw + ns_front_bytes<P>());   // [2][8]
    float* cols = red + 16;                                                 // [2 values][3][P]

    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= g.K) {              // uniform: the workgroups of the squared-error total
        const int b = (int)blockIdx.x - g.K;
        if (g.sq_out != nullptr && b < g.nb)
            sq_total_part<NTH>(g.err, g.m, b, g.nb, g.sq_part, g.sq_counter, g.sq_out,
                               reinterpret_cast<double*>(lds_raw));
        return;
    }
    const int j = blockIdx.x;
    for (int e = j * NTH + tid; e < g.n_clear; e += g.K * NTH) g.clear[e] = 0;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int strip = wave & (T - 1), hh = HV > 1 ? wave / T : 0;           // (the two of a strip on one SIMD)
    const int grp = lane >> 4, c16 = lane & 15;
    // Where P_j comes from.  Pieces: block j' has ceil(n_j' / piece) of them, in block order.
    BlockMatrixSource src = {nullptr, g.partial, 0, 1, P * P};
    bool empty;
    if (g.M != nullptr) {
        src.M = g.M + (int64_t)j * P * P;
        empty = g.counts != nullptr && g.counts[j] == 0;
    } else {
        int before = 0;                        // every wavefront for itself
        for (int jj = lane; jj < j; jj += 64) before += (g.offsets[jj + 1] - g.offsets[jj] + g.piece - 1) / g.piece;
        const int n_j = g.offsets[j + 1] - g.offsets[j];
        if (j > 0) {                           // uniform
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) before += __shfl_xor(before, o, 64);
        }
        src.pc_beg = __builtin_amdgcn_readfirstlane(before);
        src.pc_end = src.pc_beg + (n_j + g.piece - 1) / g.piece;
        empty = n_j == 0;
    }
    if (empty) {                               // uniform: block keeps its basis
        if (tid == 0) {
            g.fallback[j] = 0;
            if (g.iters_out != nullptr) g.iters_out[j] = 0;
        }
        return;
    }

    // xr[a][r] = X[t*16 + grp*4 + r][col], t = hh*TH + a, summed over the block's pieces in piece order (the order,
    // and so the bits, of accum_reduce_kernel; a finished matrix is a single piece).  A wavefront
    // reads its share of the strip's 16 atoms as whole cache lines, kInFlight pieces at a time (each round of loads is a
    // trip to memory that other CUs have just written); LDS turns the sums into its own layout.
    f32x4 xr[TH];
    {
        constexpr int kInFlight = P == 64 ? 16 : 8;
        constexpr int LD = P / 4 + 1;          // 16-byte units per atom (odd: 16 atoms cover all banks)
        static_assert(16 * LD * 16 * T <= (int)ns_front_bytes<P>(), "the strips fit in front");
        const int u0 = hh * (TH * 64) + lane;  // of the strip's T * 64 units
        const f32x4* base = reinterpret_cast<const f32x4*>(src.M != nullptr ? src.M : src.partial) + strip * (4 * P) + u0;
        f32x4 sum[TH];
#pragma unroll
        for (int t = 0; t < TH; ++t) sum[t] = base[(int64_t)src.pc_beg * (P * P / 4) + t * 64];
        for (int pc = src.pc_beg + 1; pc < src.pc_end; pc += kInFlight) {
            f32x4 v[kInFlight][TH];
#pragma unroll
            for (int k = 0; k < kInFlight; ++k)
                if (pc + k < src.pc_end) {                        // uniform
#pragma unroll
                    for (int t = 0; t < TH; ++t) v[k][t] = base[(int64_t)(pc + k) * (P * P / 4) + t * 64];
                }
#pragma unroll
            for (int k = 0; k < kInFlight; ++k)
                if (pc + k < src.pc_end) {                        // uniform
#pragma unroll
                    for (int t = 0; t < TH; ++t) sum[t] += v[k][t];
                }
        }
        unsigned mx = 0;                       // largest magnitude (a NaN wins)
#pragma unroll
        for (int t = 0; t < TH; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) mx = max(mx, __builtin_bit_cast(unsigned, fabsf(sum[t][r])));
        mx = __builtin_bit_cast(unsigned, wave_max_nan(__builtin_bit_cast(float, mx)));
        if (lane == 0) red[wave] = __builtin_bit_cast(float, mx);
        f32x4* rows = reinterpret_cast<f32x4*>(lds_raw) + strip * (16 * LD);
#pragma unroll
        for (int t = 0; t < TH; ++t) {
            const int u = u0 + t * 64;
            rows[(u / (P / 4)) * LD + u % (P / 4)] = sum[t];
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < T * HV; ++w) mx = max(mx, __builtin_bit_cast(unsigned, red[w]));
        const float scale = input_scale<P>(mx);
#pragma unroll
        for (int a = 0; a < TH; ++a) xr[a] = scale * rows[c16 * LD + (hh * TH + a) * 4 + grp];
        __syncthreads();                       // the strips become the images
    }

    int it;
    if constexpr (HV == 1) it = iterate<P, 0>(g, j, strip, xr, lds_raw, red, cols);
    else if (hh == 0) it = iterate<P, 0>(g, j, strip, xr, lds_raw, red, cols);
    else it = iterate<P, HV - 1>(g, j, strip, xr, lds_raw, red, cols);

    if (it == 0) {                             // uniform: the Jacobi SVD of this block, right here
        __syncthreads();
        if (tid == 0) g.fallback[j] = 1;
        jacobi_block<P, TPP_FALLBACK>(src, g.D + (int64_t)j * P * P, nullptr, kPolarDone, g.ops, j,
                                      g.iters_out ? g.iters_out + j : nullptr,
                                      reinterpret_cast<float*>(lds_raw));
        return;
    }
    if (tid == 0) {
        g.fallback[j] = 0;
        if (g.iters_out != nullptr) g.iters_out[j] = -it;   // negative: Newton-Schulz steps, not sweeps
    }

}

template <int P>
hipError_t launch_ns_p(const NsArgs& a, LdsRaised* raised, hipStream_t st) {
    constexpr size_t lds = ns_lds_bytes<P>();
    if (lds > 64 * 1024) {
        if (raised == nullptr) return hipErrorInvalidValue;
        if (hipError_t e = raised->ensure(reinterpret_cast<const void*>(&polar_ns_kernel<P>), lds); e != hipSuccess)
            return e;
    }
    hipLaunchKernelGGL((polar_ns_kernel<P>), dim3(a.K + (a.sq_out ? a.nb : 0)), dim3(ns_threads<P>()), lds, st, a);
    return hipGetLastError();
}

}  // namespace

// Newton-Schulz (Jacobi SVD in the same workgroup for a block that does not converge) for all K
// blocks.  fallback[j] = 1 for every block that went to the Jacobi SVD.
// M == nullptr: P_j = the sum of block j's pieces in partial (cut from offsets with `piece`
// signals per piece).  sq.out != nullptr: extra workgroups form *sq.out = sum of sq.err[0..m).
hipError_t launch_polar_ns(int p, int K, const float* M, const float* partial, const int32_t* offsets,
                           int piece, const int32_t* counts, float* D, const DictOps& ops,
                           int32_t* fallback, int32_t* iters, const SqTotalArgs& sq, LdsRaised* raised,
                           hipStream_t st, int32_t* clear, int n_clear) {
    constexpr int kMaxIters = 26;
    NsArgs a;
    a.M = M;
    a.partial = partial;
    a.offsets = offsets;
    a.piece = piece;
    a.counts = counts;
    a.D = D;
    a.ops = ops;
    a.fallback = fallback;
    a.iters_out = iters;
    a.max_iters = kMaxIters;
    a.K = K;
    a.err = sq.err;
    a.m = sq.m;
    a.sq_part = sq.part;
    a.sq_counter = sq.counter;
    a.sq_out = sq.out;
    a.clear = clear;
    a.n_clear = n_clear;
    a.nb = sq.out != nullptr ? sq.nb : 0;
    if (M == nullptr && (partial == nullptr || offsets == nullptr || piece < 1)) return hipErrorInvalidValue;
    switch (p) {
        case 16: return launch_ns_p<16>(a, raised, st);
        case 32: return launch_ns_p<32>(a, raised, st);
        case 64: return launch_ns_p<64>(a, raised, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sbo
