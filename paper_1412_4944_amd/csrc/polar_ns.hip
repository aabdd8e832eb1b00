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
//     exceeds one and is positive on (0, sqrt(3))), it only takes longer; l starts at 0.16 (block
//     matrices of this method have condition numbers of 2 to 10).  The last step is quintic, X (I + c1 E + c2 E^2),
//     E = I - X^T X (ns_scale.h).  Five steps where the plain iteration takes seven.
//   * The step.  A wavefront owns a strip of 16 columns of X (v_mfma_f32_16x16x32_bf16 tiles, four
//     consecutive rows of one column per lane and tile).  An accumulator tile is at the same time
//     the B operand of the next product, up to an order of the contraction index that the A
//     operand shares: X^T X takes its B operand from the registers that hold X, X E takes it from
//     the registers that hold E, and only the A operands (the other wavefronts' columns of X,
//     and, transposed by ds_read_b64_tr_b16 on the way out, its rows) go through LDS.
//   * The products run at fp32 accuracy: every entry is the exact sum of three bf16 parts
//     (device_utils.h), six partial products with fp32 accumulation; three for E^2 in the last step, which is
//     below 1e-4 and added to E.  (With its leading parts alone, three products for X E and the plain series, a
//     signed permutation with one late singular value came out up to 4.2e-7 off; now exactly, in the same time.)
// Measured inside sbo_iterate (launch to launch, K = 32, p = 64): 31 us with 32 x 32 tiles, both operands
// of every product through LDS and the plain iteration, 16 us as it is; p = 32: 21 -> 9 us, p = 16:
// 22 -> 7 us.  A step at p = 64 is 4800 cycles (matrix work 1650 of them), the sum of eight pieces
// 5000 (12000 with loads that touch half cache lines).
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
};

// sqrt(3 / (1 + l + l^2)) for l = 0.16 and then the l that the steps leave: 0.16, 0.375, 0.71, 0.96
__device__ constexpr float kAlpha[4] = {1.5907f, 1.4081f, 1.1601f, 1.0206f};

template <int P>
constexpr int ns_threads() {
    return P * 4;                              // a wavefront per strip of 16 columns
}
// bytes of one LDS image of X: per strip and contraction step of 32, three parts of 64 lanes x 16 bytes
template <int P>
constexpr int ns_image_bytes() {
    return (P / 16) * ((P / 16 + 1) / 2) * 3 * 1024;
}
// dynamic LDS: two images (the Jacobi routine reuses this part) | red[4 slots][4 wavefronts] floats
template <int P>
constexpr size_t ns_front_bytes() {
    const size_t img = (size_t)2 * ns_image_bytes<P>(), jac = (size_t)jacobi_lds_floats<P>() * 4;
    const size_t sq = (size_t)(ns_threads<P>() + 2) * 8;
    const size_t a = img > jac ? img : jac;
    return ((a > sq ? a : sq) + 15) / 16 * 16;
}
template <int P>
constexpr size_t ns_lds_bytes() {
    return ns_front_bytes<P>() + 16 * 4;
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

template <int P>
__global__ __launch_bounds__(ns_threads<P>()) void polar_ns_kernel(NsArgs g) {
    constexpr int T = P / 16;                  // tiles per side = strips = wavefronts
    constexpr int S = (T + 1) / 2;             // contraction steps of 32 (p = 16: half of one)
    constexpr int NTH = ns_threads<P>();
    constexpr int TPP_FALLBACK = NTH / (P / 2);          // the Jacobi routine with this workgroup's threads
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    float* red = reinterpret_cast<float*>(lds_raw + ns_front_bytes<P>());   // [4 slots][4 wavefronts]

    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= g.K) {              // uniform: the workgroups of the squared-error total
        const int b = (int)blockIdx.x - g.K;
        if (g.sq_out != nullptr && b < g.nb)
            sq_total_part<NTH>(g.err, g.m, b, g.nb, g.sq_part, g.sq_counter, g.sq_out,
                               reinterpret_cast<double*>(lds_raw));
        return;
    }
    const int j = blockIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = lane >> 4, c16 = lane & 15;
    const int col = wave * 16 + c16;           // this lane's column of X = atom
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
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) before += __shfl_xor(before, o, 64);
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

    // xr[t][r] = X[t*16 + grp*4 + r][col], summed over the block's pieces in piece order (the order,
    // and so the bits, of accum_reduce_kernel; a finished matrix is a single piece).  A wavefront
    // reads its 16 atoms as whole cache lines, kInFlight pieces at a time (each round of loads is a
    // trip to memory that other CUs have just written), and turns the sum into its own layout
    // through LDS.
    f32x4 xr[T];
    {
        constexpr int kInFlight = 8;
        constexpr int LD = P / 4 + 1;          // 16-byte units per atom (odd: 16 atoms cover all banks)
        static_assert(16 * LD * 16 * T <= (int)ns_front_bytes<P>(), "the strips fit in front");
        const f32x4* base = reinterpret_cast<const f32x4*>(src.M != nullptr ? src.M : src.partial) + wave * (4 * P) + lane;
        f32x4 sum[T];
#pragma unroll
        for (int t = 0; t < T; ++t) sum[t] = base[(int64_t)src.pc_beg * (P * P / 4) + t * 64];
        for (int pc = src.pc_beg + 1; pc < src.pc_end; pc += kInFlight) {
            f32x4 v[kInFlight][T];
#pragma unroll
            for (int k = 0; k < kInFlight; ++k)
                if (pc + k < src.pc_end) {                        // uniform
#pragma unroll
                    for (int t = 0; t < T; ++t) v[k][t] = base[(int64_t)(pc + k) * (P * P / 4) + t * 64];
                }
#pragma unroll
            for (int k = 0; k < kInFlight; ++k)
                if (pc + k < src.pc_end) {                        // uniform
#pragma unroll
                    for (int t = 0; t < T; ++t) sum[t] += v[k][t];
                }
        }
        f32x4* strip = reinterpret_cast<f32x4*>(lds_raw) + wave * (16 * LD);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int u = t * 64 + lane;
            strip[(u / (P / 4)) * LD + u % (P / 4)] = sum[t];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int t = 0; t < T; ++t) xr[t] = strip[c16 * LD + t * 4 + grp];
        __syncthreads();                       // the strips become the images
    }

    // Three bf16 parts of a strip of tiles as a B operand: lane (grp, c16) holds, for contraction step
    // s, rows grp*4 .. +3 of tiles 2s and 2s+1.
    auto split_strip = [&](const f32x4 (&v)[T], u32x4 (&out)[S][3]) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const f32x4 lo = v[2 * s];
            const f32x4 hi = 2 * s + 1 < T ? v[2 * s + 1 < T ? 2 * s + 1 : 0] : f32x4{0.f, 0.f, 0.f, 0.f};
            const Bf16x3Pair a = split_bf16x3(lo.x, lo.y), b = split_bf16x3(lo.z, lo.w);
            const Bf16x3Pair c = split_bf16x3(hi.x, hi.y), d = split_bf16x3(hi.z, hi.w);
            out[s][0] = u32x4{a.hi, b.hi, c.hi, d.hi};
            out[s][1] = u32x4{a.mid, b.mid, c.mid, d.mid};
            out[s][2] = u32x4{a.lo, b.lo, c.lo, d.lo};
        }
    };
    // The LDS image: per (strip, step, part) 1 KiB, tile 2s in the first half, tile 2s+1 in the
    // second, 8 bytes per (grp, c16), the upper two groups with their columns exchanged by eights:
    // 32 consecutive lanes of a write, of a straight and of a transposing read each cover all banks.
    const int lane_at = (grp * 16 + (c16 ^ ((grp >> 1) * 8))) * 8;
    auto unit = [&](unsigned char* img, int strip, int s, int pl) { return img + ((strip * S + s) * 3 + pl) * 1024; };
    auto write_part = [&](unsigned char* img, int s, int pl, u32x4 w) {
        unsigned char* u = unit(img, wave, s, pl) + lane_at;
        *reinterpret_cast<u32x2*>(u) = u32x2{w.x, w.y};
        if (2 * s + 1 < T) *reinterpret_cast<u32x2*>(u + 512) = u32x2{w.z, w.w};
    };
    // A operand whose row m is column m of strip `strip` (contraction over rows of X)
    auto read_cols = [&](unsigned char* img, int strip, int s, int pl) {
        const unsigned char* u = unit(img, strip, s, pl) + lane_at;
        const u32x2 a = *reinterpret_cast<const u32x2*>(u);
        u32x2 b = {0u, 0u};
        if (2 * s + 1 < T) b = *reinterpret_cast<const u32x2*>(u + 512);
        return u32x4{a.x, a.y, b.x, b.y};
    };
    // A operand whose row m is row t*16 + m of X (contraction over columns: lane (grp, .) takes
    // columns grp*4 .. +3 of strips sa and sb).  ds_read_b64_tr_b16: of the 16 lanes of a row, lane
    // i addresses four consecutive rows (4 (i & 3) ..) of column grp*4 + (i >> 2) and receives row i
    // of the four columns.
    const int tr_at = ((c16 & 3) * 16 + ((grp * 4 + (c16 >> 2)) ^ (((c16 & 3) >> 1) * 8))) * 8;
    auto read_rows = [&](unsigned char* img, int t, int sa, int sb, int pl) {
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) s16x4* lds_ptr;
        const int at = (t & 1) * 512 + tr_at;
        const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(unit(img, sa, t >> 1, pl) + at));
        s16x4 b = {0, 0, 0, 0};
        if (T > 1) b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(unit(img, sb, t >> 1, pl) + at));
        const u32x2 ua = __builtin_bit_cast(u32x2, a), ub = __builtin_bit_cast(u32x2, b);
        return u32x4{ua.x, ua.y, ub.x, ub.y};
    };
    auto mfma = [](u32x4 a, u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
    };
    // the six partial products, smallest first: (A part, B part)
    constexpr int TA[6] = {2, 0, 1, 1, 0, 0};
    constexpr int TB[6] = {0, 2, 1, 0, 1, 0};
    const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
    // Row tiles of G (and E) are kept in the order wave, wave + 1, ... (mod T): tile 0 is the one on
    // the diagonal, and its operand is in this wavefront's registers.
    int strip_of[T];
#pragma unroll
    for (int i = 0; i < T; ++i) strip_of[i] = (wave + i) & (T - 1);
    f32x4 diag;                                // the diagonal tile of I
#pragma unroll
    for (int r = 0; r < 4; ++r) diag[r] = grp * 4 + r == c16 ? 1.f : 0.f;
    // The A operands of X E, requested in the order in which the products use them, all of them
    // before the first product (the compiler would otherwise keep only a few in flight, and with
    // one wavefront per SIMD nothing else covers the wait).
    auto load_rows = [&](unsigned char* img, u32x4 (&a)[S][3][T]) {
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const int pl = k == 0 ? 2 : k - 1;
                    a[s][pl][t] = read_rows(img, t, strip_of[2 * s], strip_of[T > 1 ? 2 * s + 1 : 0], pl);
                }
        __builtin_amdgcn_sched_barrier(0);
    };
    // acc[t] = X E for row tile t from the parts of E
    auto times = [&](const u32x4 (&a)[S][3][T], const u32x4 (&eq)[S][3], f32x4 (&acc)[T]) {
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = zero4;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int t = 0; t < T; ++t) acc[t] = mfma(a[s][TA[q]][t], eq[s][TB[q]], acc[t]);
    };
    // one value per wavefront -> the sum (maximum) over the workgroup; slot: 0 .. 3, a slot is
    // reused two barriers later at the earliest
    auto publish = [&](int slot, float v) {
        if (lane == 0) red[slot * 4 + wave] = v;
    };

    unsigned char* img = lds_raw;              // the image of the current X; the other one is free
    unsigned char* other = lds_raw + ns_image_bytes<P>();
    u32x4 xq[S][3];
    int it = 0;
    bool converged = false, narrow = false;
    while (true) {
        split_strip(xr, xq);
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) write_part(img, s, pl, xq[s][pl]);
        __syncthreads();

        // this wavefront's columns of G = X^T X; the diagonal tile needs no operand from LDS and
        // covers the wait for the others
        f32x4 ge[T];
        {
            u32x4 a[S][3][T];
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int i = 1; i < T; ++i) {
                        const int pl = k == 0 ? 2 : k - 1;     // in the order in which the products use them
                        a[s][pl][i] = read_cols(img, strip_of[i], s, pl);
                    }
            __builtin_amdgcn_sched_barrier(0);
            f32x4 g0[S];
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int s = 0; s < S; ++s) g0[s] = mfma(xq[s][TA[q]], xq[s][TB[q]], q == 0 ? zero4 : g0[s]);
#pragma unroll
            for (int i = 1; i < T; ++i) ge[i] = zero4;
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int q = 0; q < 6; ++q)
#pragma unroll
                    for (int i = 1; i < T; ++i) ge[i] = mfma(a[s][TA[q]][i], xq[s][TB[q]], ge[i]);
            ge[0] = S > 1 ? g0[0] + g0[S - 1] : g0[0];
        }

        float alpha = it < 4 && !narrow ? kAlpha[it] : 1.f;            // X is scaled by this before the step
        bool last = false;
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
            for (int r = 0; r < 4; ++r) tr = fmaf(diag[r], ge[0][r], tr);
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    rs += fabsf(ge[i][r]);
                    r2 = fmaf(ge[i][r], ge[i][r], r2);
                }
            publish(0, row_max_nan(sum_groups(rs)));
            r2 = sum_groups(r2);
            publish(1, row_max_nan(r2));
            publish(2, group_sum<16>(r2));
            publish(3, sum_groups(group_sum<16>(tr)));
            __syncthreads();
            float rsmax = red[0], r2max = red[4], sum2 = red[8], mu = red[12];
#pragma unroll
            for (int w = 1; w < T; ++w) {      // as bits: a NaN wins
                rsmax = __builtin_bit_cast(float, max(__builtin_bit_cast(unsigned, rsmax), __builtin_bit_cast(unsigned, red[w])));
                r2max = __builtin_bit_cast(float, max(__builtin_bit_cast(unsigned, r2max), __builtin_bit_cast(unsigned, red[4 + w])));
                sum2 += red[8 + w];
                mu += red[12 + w];
            }
            mu *= 1.f / P;
            // zero, infinite, NaN or overflowing input: not for this iteration
            if (!(rsmax > 1e-37f && rsmax < 3e37f)) break;
            float b2 = 2.9f * __builtin_amdgcn_rcpf(rsmax);
            narrow = narrow_spectrum<P>(sum2, mu);
            if (narrow)
                b2 = fminf(b2, __builtin_amdgcn_rcpf(mu));
            else if (r2max > 1e-37f && r2max < 3e37f)
                b2 = fminf(b2, kAlpha[0] * kAlpha[0] / 1.04f * __builtin_amdgcn_rsqf(r2max));
            alpha = __builtin_amdgcn_sqrtf(b2);
        } else {
            float fr = 0.f;
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float e = i == 0 ? diag[r] - ge[i][r] : ge[i][r];
                    fr = fmaf(e, e, fr);
                }
            publish(2 + (it & 1), sum_groups(group_sum<16>(fr)));
        }
        // E = I - alpha^2 G, then X <- alpha (X + X E / 2)
        auto make_e = [&](float a2) {
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) ge[i][r] = i == 0 ? diag[r] - a2 * ge[i][r] : -a2 * ge[i][r];
        };
        u32x4 rows[S][3][T], eq[S][3];
        load_rows(img, rows);
        f32x4 g0[T];
#pragma unroll
        for (int i = 0; i < T; ++i) g0[i] = ge[i];
        make_e(alpha * alpha);
        split_strip(ge, eq);
        if (it > 0) {                          // has this been the last but one step?  (the split hides the wait)
            __syncthreads();
            float fr = red[(2 + (it & 1)) * 4];
#pragma unroll
            for (int w = 1; w < T; ++w) fr += red[(2 + (it & 1)) * 4 + w];
            if (!(fr < 2.f * P)) break;        // NaN or diverging: leave it to the Jacobi SVD
            last = fr < kLastEps * kLastEps;   // |E|_F, a bound on the spectral norm of E
            if (!last && it >= g.max_iters) break;
        }
        f32x4 acc[T];
        if (last) {                            // uniform
            alpha = 1.f;
#pragma unroll
            for (int i = 0; i < T; ++i) ge[i] = g0[i];
            make_e(1.f);
            // E^2 from the three largest partial products: 2^-16 of something below 1e-4
            split_strip(ge, eq);
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int pl = 0; pl < 2; ++pl) write_part(other, s, pl, eq[s][pl]);
            __syncthreads();
            f32x4 e2[T];
#pragma unroll
            for (int i = 0; i < T; ++i) e2[i] = zero4;
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int i = 0; i < T; ++i) {
                    // E is symmetric: its rows are the strips, each with its tiles in its own order
                    const int pa = (strip_of[2 * s] - strip_of[i]) & (T - 1), pb = (pa + 1) & (T - 1);
                    u32x4 a[2];
#pragma unroll
                    for (int pl = 0; pl < 2; ++pl) {
                        const u32x2 lo = *reinterpret_cast<const u32x2*>(unit(other, strip_of[i], pa >> 1, pl) + (pa & 1) * 512 + lane_at);
                        u32x2 hi = {0u, 0u};
                        if (T > 1)
                            hi = *reinterpret_cast<const u32x2*>(unit(other, strip_of[i], pb >> 1, pl) + (pb & 1) * 512 + lane_at);
                        a[pl] = u32x4{lo.x, lo.y, hi.x, hi.y};
                    }
                    e2[i] = mfma(a[1], eq[s][0], e2[i]);
                    e2[i] = mfma(a[0], eq[s][1], e2[i]);
                    e2[i] = mfma(a[0], eq[s][0], e2[i]);
                }
#pragma unroll
            for (int i = 0; i < T; ++i) ge[i] = kLastLinear * ge[i] + kLastSquare * e2[i];
            split_strip(ge, eq);
        }
        times(rows, eq, acc);
#pragma unroll
        for (int t = 0; t < T; ++t) xr[t] = alpha * xr[t] + (0.5f * alpha) * acc[t];
        ++it;
        if (last) {
            converged = true;
            break;
        }
        unsigned char* const done = img;       // (its last readers are behind the barrier after the next writes)
        img = other;
        other = done;
    }

    if (!converged) {                          // uniform: the Jacobi SVD of this block, right here
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

    // D[j][k][:] = column k of X; the same values in the coding kernels' operand orders
    f32x4* Dj = reinterpret_cast<f32x4*>(g.D + (int64_t)j * P * P);
    float q2 = 0.f, r2 = 0.f;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int d4 = t * 4 + grp;
        Dj[col * (P / 4) + d4] = xr[t];
        if (g.ops.f32 != nullptr) store_operand_f32<P>(g.ops.f32, j * P + col, d4, xr[t]);
        if (g.ops.bf16 != nullptr) store_operand_split<P>(g.ops.bf16, j * P + col, d4, xr[t]);
        if (g.ops.f16 != nullptr) store_operand_f16x2<P>(g.ops.f16, j * P + col, d4, split_f16x2_dict(xr[t], q2, r2));
    }
    if (g.ops.f16 != nullptr) {                // a wavefront holds 16 atoms
        q2 = row16_max(sum_groups(q2));
        r2 = row16_max(sum_groups(r2));
        if (lane == 0) g.ops.dnorm[j * T + wave] = float2{sqrtf(q2), sqrtf(r2)};
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
                           hipStream_t st) {
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
