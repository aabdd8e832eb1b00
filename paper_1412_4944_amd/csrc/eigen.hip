// Eigenvectors of symmetric positive semidefinite p x p matrices (the Gram matrix of a signal set; eq. (5): the left
// singular vectors of the set are its eigenvectors): Householder reduction to a tridiagonal matrix, bisection and
// twisted factorisations for that, and back.
//
// The one-sided Jacobi method that did this takes eight to ten sweeps of p - 1 dependent rounds over p x p
// matrices A and V (p = 64: 500 rounds of 900 cycles; p = 256: 2500 in teams that hand columns on); here p - 2 dependent steps
// over A, of which each is a matrix-vector product and a rank-two update, leave a tridiagonal matrix whose
// eigenvectors are independent of one another:
//   1. tridiag_kernel (one workgroup per matrix, fp32): the matrix in registers as MFMA accumulator tiles (p = 64: a tile
//      for each of four wavefronts, p = 256: four for each of sixteen), the rank-two update v w^T + w v^T one
//      v_mfma_f32_32x32x2_f32 per tile; a column is a lane's registers, so A x needs x broadcast (DPP row_newbcast) and
//      almost no reduction.  A x does not wait for the reflector (A v = A x - alpha A e), and the next x not for
//      the accumulators (it is row k + 1 less v w^T + w v^T): one barrier a step, p = 256 two.
//   2. eig_vectors_kernel (one workgroup per eigenvector).  Eigenvalue k by bisection in 256 points at a time (Sturm
//      counts; five rounds end at 2^-39 of the largest), eigenvector of the tridiagonal matrix from a twisted factorisation at
//      the index where the residual is smallest, p - 2 reflectors back; all in fp64, and beta = 2 / v^T v of the v
//      that is stored, so that the rounding of 1 does not touch orthogonality.
//   3. refine_kernel, twice (one workgroup per eigenvector, fp64).  1 rounds at 2^-24 of the largest eigenvalue, which is
//      a lot for eigenvalues that are small: a first-order correction from the matrix itself takes an error E to E^2.
//      Without it, sets whose amplitudes fall over the coordinates lost what fp32 still holds of them: Q G Q^T off its
//      diagonal by up to 1e-4 of sqrt(lambda_i lambda_j) (p = 256, three decades), where the Jacobi kernels leave 2e-6.
//   4. A matrix for which this is not good enough (eigenvalues closer than 1e-8 of the largest, as the zeros of a
//      set with fewer than p signals; a residual above 2e-11; a correction above 0.1, or above 1e-3 the second time; not
//      finite) goes to the Jacobi kernels, which compute all of its eigenvectors.
// Measured (sbo_init_base, 2048 signals; in brackets without 3): p = 16 46 us (37), p = 32 64 (52), p = 64 95 (84), p = 256
// 493 (455); by Jacobi p = 64 0.2 ms, p = 256 1.8.  Launches inside sbo_learn: p = 64 46, 23, 5, 5 (+ 5 for the one that finds
// nothing left to do), p = 256 320, 91, 21, 19 (+ 7).  Against eigenvectors in fp64 of the set, amplitudes equal or falling
// over one to four decades, along the coordinates or across them, p = 16 to 256: the error of the vectors 0.02 to 0.8 of
// that of the Jacobi kernels wherever 3 is not skipped (equal: 3 to 5e-6 against 2e-5 to 2.5e-4; two decades along the
// coordinates 2e-8 to 3e-6 against 3e-7 to 3e-5, without 3 1e-6 to 2e-4), Q G Q^T off its diagonal by at most 2e-7 of
// sqrt(lambda_i lambda_j) there, Q Q^T - I 2e-8 to 7e-7 (Jacobi 3e-7 to 5e-6), eigenvalues 2e-7 of the largest.  To the Jacobi
// kernels go: four decades from p = 32 on, and three across the coordinates at p = 256, where the Gram matrix in fp32 no
// longer determines the last directions.
//
// What bounds it: the steps of 1 depend on one another (p = 64: 1700 cycles, of which A x 420, sums over the lanes and
// scalars 500; p = 256: 3000, of which A x on the vector ALU 1300 and one wavefront's scalars 700); 2: a chain of p fused
// multiply-adds in fp64 per count, 80 cycles a link, five times over, and p - 2 reflectors of 220 to 330 cycles each; 3: launches,
// and at p = 256 the 1.3 MB that every workgroup reads from L2.
#include "sbo_internal.h"
#include "device_utils.h"

namespace sbo {

namespace {

// Per matrix, in the order of the kernels: reflectors v (gone once the first eigenvectors are there), tridiagonal matrix,
// eigenvectors z (one set per step of the refinement), A z and eigenvalues.
struct EigScratch {
    unsigned char* base;       // [matrix]{ z0[p][p] | z1[p][p], v[p][p] | A z[p][p] | (d_i, e_{i-1}^2)[p] | e[p] | beta[p] | lambda[2][p] }
    int32_t* flag;             // [matrix] left to the Jacobi SVD by kernel 1, 2, .. (0: by none)
    template <int P>
    __device__ __forceinline__ double* z(int b, int set) const {
        return reinterpret_cast<double*>(base + b * bytes<P>()) + (size_t)set * P * P;
    }
    template <int P>
    __device__ __forceinline__ float* v(int b) const { return reinterpret_cast<float*>(z<P>(b, 1)); }
    template <int P>
    __device__ __forceinline__ double* az(int b) const { return z<P>(b, 2); }
    template <int P>
    __device__ __forceinline__ double* de(int b) const { return z<P>(b, 3); }
    template <int P>
    __device__ __forceinline__ double* e(int b) const { return de<P>(b) + 2 * P; }
    template <int P>
    __device__ __forceinline__ double* beta(int b) const { return de<P>(b) + 3 * P; }
    template <int P>
    __device__ __forceinline__ double* lambda(int b, int set) const { return de<P>(b) + (4 + set) * P; }
    template <int P>
    __host__ __device__ static constexpr size_t bytes() {
        return (3 * (size_t)P * P + 6 * (size_t)P) * sizeof(double);
    }
};

template <int CTRL>
__device__ __forceinline__ double dpp_d(double x) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
// The two halves of f(x of the own row pair, x of the other): 16 lanes apart, then 32.
template <class F>
__device__ __forceinline__ double swap16(double x, F f) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    auto lo = __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)u, false, false);
    auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
    const unsigned l0 = lo[0], l1 = lo[1], h0 = hi[0], h1 = hi[1];
    return f(__builtin_bit_cast(double, (unsigned long long)h0 << 32 | l0), __builtin_bit_cast(double, (unsigned long long)h1 << 32 | l1));
}
template <class F>
__device__ __forceinline__ double swap32d(double x, F f) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    auto lo = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)u, false, false);
    auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
    const unsigned l0 = lo[0], l1 = lo[1], h0 = hi[0], h1 = hi[1];
    return f(__builtin_bit_cast(double, (unsigned long long)h0 << 32 | l0), __builtin_bit_cast(double, (unsigned long long)h1 << 32 | l1));
}
// Over aligned groups of G = 16, 32 or 64 lanes, in all of them.
template <int G, class F>
__device__ __forceinline__ double lanes_reduce(double x, F f) {
    x = f(x, dpp_d<kDppXor1>(x));
    x = f(x, dpp_d<kDppXor2>(x));
    x = f(x, dpp_d<kDppHalfMirror>(x));
    x = f(x, dpp_d<kDppRowMirror>(x));
    if constexpr (G >= 32) x = swap16(x, f);
    if constexpr (G >= 64) x = swap32d(x, f);
    return x;
}
template <int G>
__device__ __forceinline__ double lanes_sum(double x) {
    return lanes_reduce<G>(x, [](double a, double b) { return a + b; });
}
template <int G>
__device__ __forceinline__ double lanes_max(double x) {
    return lanes_reduce<G>(x, [](double a, double b) { return fmax(a, b); });
}
__device__ __forceinline__ float read_lane(float x, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
}
// Sum over aligned groups of 32 or 64 lanes, in all of them.
template <int G>
__device__ __forceinline__ float lanes_sum_f(float x) {
    x = group_sum<16>(x);
    const unsigned u = __builtin_bit_cast(unsigned, x);
    auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned a0 = r[0], a1 = r[1];
    x = __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1);
    if constexpr (G == 64) {
        const unsigned w = __builtin_bit_cast(unsigned, x);
        auto q = __builtin_amdgcn_permlane32_swap(w, w, false, false);
        const unsigned b0 = q[0], b1 = q[1];
        x = __builtin_bit_cast(float, b0) + __builtin_bit_cast(float, b1);
    }
    return x;
}
__device__ __forceinline__ double recip(double x) {            // a few ulp
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}
// Largest magnitude over the workgroup (a NaN wins); red: a word per wavefront.
template <int WAVES>
__device__ __forceinline__ float wg_max(float mx, unsigned* red) {
    unsigned u = __builtin_bit_cast(unsigned, mx);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) u = max(u, (unsigned)__shfl_xor((int)u, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = u;
    __syncthreads();
    u = red[0];
    for (int w = 1; w < WAVES; ++w) u = max(u, red[w]);
    return __builtin_bit_cast(float, u);
}


// A barrier for what is in LDS: nobody waits for the stores of the reflectors to memory.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The flag of matrix b and 1 / its scale (a power of two: exact), from the largest magnitude of a thread's entries; false: it
// is zero or not finite.
template <int P, int WAVES>
__device__ __forceinline__ bool tridiag_scale(const EigScratch& s, int b, float mx, unsigned* red, float& inv) {
    mx = wg_max<WAVES>(mx, red);
    const bool good = mx > 1e-30f && mx < 1e37f;
    const int ex = good ? (int)(__builtin_bit_cast(unsigned, mx) >> 23) - 127 : 0;
    inv = __builtin_bit_cast(float, (unsigned)(127 - ex) << 23);
    if (threadIdx.x == 0) s.flag[b] = !good;
    return good;
}

template <int R>
__device__ __forceinline__ float row_bcast(float x) {          // lane R of every 16, to all of them
    return dpp_f<0x150 + R>(x);
}
// y[..] += the terms of a tile, acc[r] times the x of its row, which lane r of every 16 holds
__device__ __forceinline__ void tile_times(const f32x16& acc, float x, float (&y)[4]) {
#define SBO_TERM(R) y[R & 3] = fmaf(row_bcast<R>(x), acc[R], y[R & 3]);
    SBO_TERM(0) SBO_TERM(1) SBO_TERM(2) SBO_TERM(3) SBO_TERM(4) SBO_TERM(5) SBO_TERM(6) SBO_TERM(7)
    SBO_TERM(8) SBO_TERM(9) SBO_TERM(10) SBO_TERM(11) SBO_TERM(12) SBO_TERM(13) SBO_TERM(14) SBO_TERM(15)
#undef SBO_TERM
}
__device__ __forceinline__ float halves_sum(float x) {         // of lanes l and l ^ 32, in both
    const unsigned u = __builtin_bit_cast(unsigned, x);
    auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const unsigned a0 = r[0], a1 = r[1];
    return __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1);
}
// What a step knows of its reflector before A x is there: S = |x|^2, x1 the first entry.  beta is that of the v that the
// update uses, in fp64: one that is off by the rounding of S would scale the matrix a little in every step (p = 256
// 2048 signals: eigenvalues 1.8e-7 of the largest off instead of 5e-8).
struct Reflect {
    float alpha, v1, beta;                     // v = x but for its first entry v1 = x1 - alpha; beta = 2 / v^T v
    double e;                                  // entry k + 1 of H x = x - beta v (v^T x)
    __device__ __forceinline__ Reflect(double S, float x1) : alpha(x1), v1(0.f), beta(0.f), e(x1) {
        if (S > 1e-30) {                       // uniform
            v1 = x1 + copysignf(__builtin_amdgcn_sqrtf((float)S), x1);
            alpha = x1 - v1;
            const double tail = fma(-(double)x1, (double)x1, S), b = 2.0 * recip(fma((double)v1, (double)v1, tail));
            e = x1 - b * v1 * fma((double)v1, (double)x1, tail);
            beta = (float)b;
        }
    }
    // w = beta A v - half v
    __device__ __forceinline__ float half(float xAx, float y1, float a11) const {
        return 0.5f * beta * beta * (xAx - 2.f * alpha * y1 + alpha * alpha * a11);
    }
};
// The end of both kernels: the last entries, and beta = 2 / v^T v of every reflector.
template <int P, int WAVES>
__device__ __forceinline__ void tridiag_end(const EigScratch& s, int b, float d1, float e1, float d2) {
    double *de = s.de<P>(b), *e = s.e<P>(b), *beta = s.beta<P>(b);
    float* V = s.v<P>(b);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int E = P > 64 ? P / 64 : 1;
    if (tid == 0) {
        de[1] = 0.0;
        de[2 * (P - 2)] = d1;
        de[2 * (P - 1)] = d2;
        de[2 * (P - 1) + 1] = (double)e1 * e1;
        e[P - 2] = e1;
        e[P - 1] = 0.0;
        beta[P - 2] = beta[P - 1] = 0.0;
    }
    for (int t = tid; t < 2 * P; t += 64 * WAVES) V[(P - 2) * P + t] = 0.f;
    __syncthreads();                           // the reflectors are in memory
    for (int k = wave; k < P - 2; k += WAVES) {
        double v2 = 0.0;
#pragma unroll
        for (int t = 0; t < E; ++t) {
            const double v = E * lane + t < P ? (double)V[k * P + E * lane + t] : 0.0;
            v2 = fma(v, v, v2);
        }
        v2 = lanes_sum<64>(v2);
        if (lane == 0) beta[k] = v2 > 0.0 ? 2.0 / v2 : 0.0;
    }
}

// 1. p <= 64 (p = 16: in a tile of 32): wavefront w holds tile (w / T, w % T): register r of lane (h, n) is row
// (r / 4) * 8 + h * 4 + r % 4, column n of it.  Vectors: entry `li` per lane, in every wavefront.
template <int P>
constexpr int tri_waves() { return P == 64 ? 4 : 1; }
template <int P>
__global__ __launch_bounds__(64 * tri_waves<P>()) void tridiag_kernel(const float* __restrict__ G, EigScratch s) {
    constexpr int W = tri_waves<P>(), T = W == 4 ? 2 : 1, N = 32 * T;
    __shared__ float edge[2][N], part[2][T][N];
    __shared__ unsigned red[W];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, n = lane & 31, I = wave / T, J = wave % T, li = T == 2 ? lane : n;
    const float* A = G + (int64_t)b * P * P;
    double *de = s.de<P>(b), *e = s.e<P>(b);
    float* V = s.v<P>(b);

    f32x16 acc;
    float mx = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = I * 32 + (r >> 2) * 8 + h * 4 + (r & 3), col = J * 32 + n;
        acc[r] = row < P && col < P ? A[row * P + col] : 0.f;
        mx = __builtin_bit_cast(float, max(__builtin_bit_cast(unsigned, mx), __builtin_bit_cast(unsigned, fabsf(acc[r]))));
    }
    float inv;
    if (!tridiag_scale<P, W>(s, b, mx, red, inv)) return;      // uniform
    acc *= inv;
    // row j of the matrix, which is symmetric -> out: one register
    auto publish = [&](int j, float* out) {
        if (j >> 5 == I) {                     // uniform
            const float v = acc[(j & 3) + ((j & 31) >> 3) * 4];
            if (h == ((j >> 2) & 1)) out[J * 32 + n] = v;
        }
    };
    publish(0, edge[0]);
    publish(1, edge[1]);
    lds_barrier();
    const int row16 = I * 32 + ((lane & 15) >> 2) * 8 + h * 4 + (lane & 3);    // what row_bcast hands out
    // row k, which the step before has made from row k of the matrix before; row k + 1 comes from the accumulators
    // by way of LDS, half a step later
    float row = edge[0][li];
    lds_barrier();                             // (edge[0] is row 2 next)

#pragma unroll 1
    for (int k = 0; k < P - 2; ++k) {
        const float x = li > k ? row : 0.f;
        const float xb = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(4 * (T == 2 ? row16 : row16 & 31), __builtin_bit_cast(int, x)));
        float y4[4] = {0.f, 0.f, 0.f, 0.f};
        tile_times(acc, xb, y4);
        const float ysum = halves_sum((y4[0] + y4[1]) + (y4[2] + y4[3]));
        if (h == 0) part[k & 1][I][J * 32 + n] = ysum;
        const Reflect r(lanes_sum<N>((double)x * x), read_lane(x, k + 1));
        lds_barrier();
        const float c = edge[(k + 1) & 1][li];
        float y = part[k & 1][0][li];
        if constexpr (T == 2) y += part[k & 1][1][li];
        y = li > k ? y : 0.f;
        const float half = r.half(lanes_sum_f<N>(x * y), read_lane(y, k + 1), read_lane(c, k + 1));
        const float v = r.beta == 0.f ? 0.f : li == k + 1 ? r.v1 : x;
        const float w = li > k ? r.beta * (y - r.alpha * c) - half * v : 0.f;
        // operands: (v, w) of the tile's rows against (-w, -v) of its columns, in the two halves of the lanes
        float a, bo;
        if constexpr (T == 2) {
            const unsigned uv = __builtin_bit_cast(unsigned, v), uw = __builtin_bit_cast(unsigned, w);
            auto vw = __builtin_amdgcn_permlane32_swap(uv, uw, false, false), wv = __builtin_amdgcn_permlane32_swap(uw, uv, false, false);
            const unsigned v0 = vw[0], v1 = vw[1], w0 = wv[0], w1 = wv[1];
            a = __builtin_bit_cast(float, I ? v1 : v0);
            bo = __builtin_bit_cast(float, J ? w1 : w0);
        } else {
            a = h ? w : v;
            bo = h ? v : w;
        }
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, -bo, acc, 0, 0, 0);
        if (wave == 0) {
            if (lane < P) V[k * P + lane] = v;
            if (lane == k) de[2 * k] = row;
            if (lane == 0) {
                e[k] = r.e;
                de[2 * (k + 1) + 1] = r.e * r.e;
            }
        }
        row = fmaf(-read_lane(v, k + 1), w, fmaf(-read_lane(w, k + 1), v, c));
        publish(k + 2, edge[k & 1]);
    }
    lds_barrier();
    tridiag_end<P, W>(s, b, read_lane(row, P - 2), read_lane(row, P - 1), edge[(P - 1) & 1][P - 1]);
}

// 1. p = 256: wavefront w holds the tiles of columns (w & 7) * 32 and rows w / 8, + 2, + 4, + 6 (of 32).  The first one, whose
// columns are done soonest, makes the reflector and w, and the next x.
__global__ __launch_bounds__(1024) void tridiag_wide_kernel(const float* __restrict__ G, EigScratch s) {
    constexpr int P = 256;
    __shared__ __attribute__((aligned(16))) float xs[P], edge[2][P], part[2][P], vw[2][P];
    __shared__ unsigned red[16];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, n = lane & 31, I0 = wave >> 3, J = I0 ? (wave & 7) ^ 2 : wave & 7;    // (a strip on two SIMDs)
    const float* A = G + (int64_t)b * P * P;
    double *de = s.de<P>(b), *e = s.e<P>(b);
    float* V = s.v<P>(b);

    f32x16 acc[4];
    float mx = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            acc[i][r] = A[((2 * i + I0) * 32 + (r >> 2) * 8 + h * 4 + (r & 3)) * P + J * 32 + n];
            mx = __builtin_bit_cast(float, max(__builtin_bit_cast(unsigned, mx), __builtin_bit_cast(unsigned, fabsf(acc[i][r]))));
        }
    float inv;
    if (!tridiag_scale<P, 16>(s, b, mx, red, inv)) return;     // uniform
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] *= inv;
    // row j of the matrix, which is symmetric -> out: a register of eight of the wavefronts
    auto publish = [&](int j, float* out) {
        if (((j >> 5) & 1) == I0) {            // uniform
            const int r = (j & 3) + ((j & 31) >> 3) * 4;
            float v = acc[0][r];
#pragma unroll
            for (int i = 1; i < 4; ++i)
                if (j >> 6 == i) v = acc[i][r];
            if (h == ((j >> 2) & 1)) out[J * 32 + n] = v;
        }
    };
    publish(0, xs);
    publish(1, edge[1]);
    lds_barrier();
    const int row16 = ((lane & 15) >> 2) * 8 + h * 4 + (lane & 3);             // of a tile: what row_bcast hands out
    f32x4 row = {0.f, 0.f, 0.f, 0.f};          // of the first wavefront: row k, four entries a lane
    if (wave == 0) row = *reinterpret_cast<const f32x4*>(xs + 4 * lane);

#pragma unroll 1
    for (int k = 0; k < P - 2; ++k) {
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        Reflect ref(0.0, 0.f);
        if (wave == 0) {                       // the reflector
            double S = 0.0;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                v[t] = 4 * lane + t > k ? row[t] : 0.f;
                S = fma((double)v[t], (double)v[t], S);
            }
            ref = Reflect(lanes_sum<64>(S), xs[k + 1]);
        }
        if (J * 32 + 31 > k) {                 // uniform: columns that are left
            float y[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r0 = (2 * i + I0) * 32;
                if (r0 + 31 > k) tile_times(acc[i], r0 + row16 > k ? xs[r0 + row16] : 0.f, y);         // uniform
            }
            const float sum = halves_sum((y[0] + y[1]) + (y[2] + y[3]));
            if (h == 0) part[I0][J * 32 + n] = sum;
        }
        lds_barrier();
        if (wave == 0) {                       // w, and x of the next step
            const f32x4 c = *reinterpret_cast<const f32x4*>(edge[(k + 1) & 1] + 4 * lane);
            const f32x4 ys = *reinterpret_cast<const f32x4*>(part[0] + 4 * lane) + *reinterpret_cast<const f32x4*>(part[1] + 4 * lane);
            const float y1 = part[0][k + 1] + part[1][k + 1], a11 = edge[(k + 1) & 1][k + 1];
            float y[4], xAx = 0.f;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                y[t] = 4 * lane + t > k ? ys[t] : 0.f;
                xAx = fmaf(v[t], y[t], xAx);
            }
            const float half = ref.half(lanes_sum_f<64>(xAx), y1, a11);
            const float v1 = ref.v1, w1 = ref.beta * (y1 - ref.alpha * a11) - half * v1;
            f32x4 w, next;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int at = 4 * lane + t;
                v[t] = ref.beta == 0.f ? 0.f : at == k + 1 ? v1 : v[t];
                w[t] = at > k ? ref.beta * (y[t] - ref.alpha * c[t]) - half * v[t] : 0.f;
                next[t] = fmaf(-v1, w[t], fmaf(-w1, v[t], c[t]));
            }
            *reinterpret_cast<f32x4*>(vw[0] + 4 * lane) = v;
            *reinterpret_cast<f32x4*>(vw[1] + 4 * lane) = w;
            *reinterpret_cast<f32x4*>(xs + 4 * lane) = next;
            if (lane == k >> 2) de[2 * k] = row[k & 3];
            row = next;
        }
        lds_barrier();
        if (J * 32 + 31 > k) {                 // uniform
            // (v, w) of a tile's rows against (-w, -v) of its columns, in the two halves of the lanes
            const float bo = -vw[h ^ 1][J * 32 + n];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r0 = (2 * i + I0) * 32;
                if (r0 + 31 > k) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(vw[h][r0 + n], bo, acc[i], 0, 0, 0);
            }
            publish(k + 2, edge[k & 1]);
        }
        if (wave == 0) {
            *reinterpret_cast<f32x4*>(V + k * P + 4 * lane) = v;
            if (lane == 0) {
                e[k] = ref.e;
                de[2 * (k + 1) + 1] = ref.e * ref.e;
            }
        }
    }
    lds_barrier();
    tridiag_end<P, 16>(s, b, xs[P - 2], xs[P - 1], edge[1][P - 1]);
}

// Number of eigenvalues below x: sign changes of the leading minors of T - x.  de: uniform (scalar loads, eight entries
// ahead of their use).
template <int P>
__device__ __forceinline__ int sturm_count(const double* __restrict__ de, double x) {
    constexpr int A = 8;
    double cur[2 * A], next[2 * A];
#pragma unroll
    for (int t = 0; t < 2 * A; ++t) cur[t] = de[t];
    double p0 = 0.0, p1 = 1.0;
    int n = 0;
#pragma unroll 1
    for (int i = 0; i < P; i += A) {
        const double* src = de + 2 * (i + A < P ? i + A : 0);
#pragma unroll
        for (int t = 0; t < 2 * A; ++t) next[t] = src[t];
        __builtin_amdgcn_sched_barrier(0);     // (their latency is what the loop would wait for)
#pragma unroll
        for (int t = 0; t < A; ++t) {
            const double p = fma(cur[2 * t] - x, p1, -(cur[2 * t + 1] * p0));
            n += (int)((unsigned)((__builtin_bit_cast(unsigned long long, p) ^ __builtin_bit_cast(unsigned long long, p1)) >> 32) >> 31);
            p0 = p1;
            p1 = p;
        }
        // eight factors of at most 2^9 and at least 2^-80 each stay inside the range; the common exponent goes
        const unsigned ex = (unsigned)(__builtin_bit_cast(unsigned long long, fmax(fabs(p0), fabs(p1))) >> 52);
        const double sc = __builtin_bit_cast(double, (unsigned long long)(2046u - min(ex, 2045u)) << 52);
        p0 *= sc;
        p1 *= sc;
#pragma unroll
        for (int t = 0; t < 2 * A; ++t) cur[t] = next[t];
    }
    return n;
}

// y = A^T x by a workgroup of NTH threads, x and y in LDS; part: NTH doubles.  Every workgroup begins at a row of its
// own, or all of them want the same lines of L2 at a time (p = 256: 24 us a refine_kernel, 19).
template <int P, int NTH, class T>
__device__ __forceinline__ void transposed_times(const T* __restrict__ A, const double* x, double* part, double* y) {
    constexpr int R = P * P / NTH;             // rows of a group of P threads (a power of two)
    const int tid = threadIdx.x, t = tid % P, r0 = tid / P * R, off = blockIdx.x;
    double sum = 0.0;
#pragma unroll 16
    for (int i = 0; i < R; ++i) {
        const int row = r0 + ((i + off) & (R - 1));
        sum = fma((double)A[row * P + t], x[row], sum);
    }
    part[tid] = sum;
    __syncthreads();
    if (tid < P) {
        for (int g = 1; g < NTH / P; ++g) sum += part[g * P + tid];
        y[tid] = sum;
    }
    __syncthreads();
}
// x, y = A x -> z, az, and the Rayleigh quotient; x, y in LDS, tid < 64 at least.
template <int P>
__device__ __forceinline__ void keep_vector(const double* x, const double* y, double* z, double* az, double* lambda) {
    const int tid = threadIdx.x;
    if (tid < P) {
        z[tid] = x[tid];
        az[tid] = y[tid];
    }
    if (tid < 64) {
        double xy = 0.0, xx = 0.0;
        for (int t = tid; t < P; t += 64) {
            xy = fma(x[t], y[t], xy);
            xx = fma(x[t], x[t], xx);
        }
        xy = lanes_sum<64>(xy);
        xx = lanes_sum<64>(xx);
        if (tid == 0) *lambda = xy / xx;
    }
}

// 2. Eigenvector blockIdx.x (by descending eigenvalue) of matrix blockIdx.y.
template <int P>
__global__ __launch_bounds__(256) void eig_vectors_kernel(const float* __restrict__ G, EigScratch s) {
    constexpr int E = P > 64 ? P / 64 : 1;     // entries of a lane in the last part
    constexpr double kGap = 1e-8, kResidual = 2e-11;           // (at most sqrt(p) times what the bisection leaves, 1e-12)
    __shared__ double dl[P], el[P], Q[2][P], redd[4];
    __shared__ int redi[8];
    const int b = blockIdx.y, k = blockIdx.x, idx = P - 1 - k, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (s.flag[b] == 1) return;                // uniform: not finite (nobody below reads the flag)
    const double* __restrict__ de = s.de<P>(b);
    // Gershgorin's bound of all eigenvalues
    double bound = 0.0;
    if (tid < P) {
        const double d = de[2 * tid], e1 = s.e<P>(b)[tid], e0 = tid > 0 ? s.e<P>(b)[tid - 1] : 0.0;
        dl[tid] = d;
        el[tid] = e1;
        bound = fabs(d) + fabs(e0) + fabs(e1);
    }
    bound = lanes_max<64>(bound);
    if (lane == 0) redd[wave] = bound;
    __syncthreads();
    bound = fmax(fmax(redd[0], redd[1]), fmax(redd[2], redd[3]));

    double lo = -bound * 1.0001, hi = bound * 1.0001;
    bool alone = true;
    constexpr int kRounds = 5;                 // (to 1e-12 of the bound: 1e-4 of a neighbour at most, which the refinement takes out)
    for (int it = 0; it < kRounds; ++it) {
        const bool last = it == kRounds - 1;   // two of its points ask whether another eigenvalue is near
        const int points = last ? 254 : 256;
        const double step = (hi - lo) * (1.0 / (points + 1));
        const double x = tid < points ? fma((double)(tid + 1), step, lo) : tid == 254 ? lo - kGap * bound : hi + kGap * bound;
        const int n = sturm_count<P>(de, x);
        const int above = __popcll(__ballot(tid < points && n <= idx));        // points at or below the eigenvalue
        if (last && tid >= points) alone = n == (tid == 254 ? idx : idx + 1);
        __syncthreads();
        if (lane == 0) redi[wave] = above;
        __syncthreads();
        const int at = redi[0] + redi[1] + redi[2] + redi[3];
        const double was = lo;
        if (at > 0) lo = fma((double)at, step, was);
        if (at < points) hi = fma((double)(at + 1), step, was);
    }
    const double lambda = 0.5 * (lo + hi);
    if (!alone) s.flag[b] = 2;

    // The pivots of T - lambda from the top (lane 0) and from the bottom (lane 1), as quotients of neighbouring minors:
    // a chain of one fused multiply-add per entry, where pivots themselves are one of divisions
    __shared__ double minor[2][P], first[2][P / 8], dm[P], e2[P + 1];
    if (tid < P) {
        dm[tid] = dl[tid] - lambda;
        e2[tid + 1] = el[tid] * el[tid];       // between tid and tid + 1
        if (tid == 0) e2[0] = 0.0;
    }
    __syncthreads();
    if (tid < 2) {
        double p0 = 0.0, p1 = 1.0;
        const int i0 = tid == 0 ? 0 : P - 1, dir = tid == 0 ? 1 : -1;
        double dv[8], ev[8], dn[8], en[8];
        auto load = [&](double (&d)[8], double (&e)[8], int t0) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int i = i0 + dir * (t0 + t);
                d[t] = dm[i];
                e[t] = e2[i + tid];
            }
        };
        load(dv, ev, 0);
#pragma unroll 1
        for (int t0 = 0; t0 < P; t0 += 8) {
            load(dn, en, t0 + 8 < P ? t0 + 8 : 0);
            first[tid][t0 / 8] = p1;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const double p = fma(dv[t], p1, -(ev[t] * p0));            // (zero: not finite below, left to Jacobi)
                minor[tid][t0 + t] = p;
                p0 = p1;
                p1 = p;
            }
            const unsigned ex = (unsigned)(__builtin_bit_cast(unsigned long long, fmax(fabs(p0), fabs(p1))) >> 52) & 0x7ffu;
            const double sc = __builtin_bit_cast(double, (unsigned long long)(2046u - min(ex, 2045u)) << 52);
            p0 *= sc;
            p1 *= sc;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                dv[t] = dn[t];
                ev[t] = en[t];
            }
        }
    }
    __syncthreads();
    if (tid < P) {
        const int t1 = P - 1 - tid;
        Q[0][tid] = minor[0][tid] * recip((tid & 7) == 0 ? first[0][tid / 8] : minor[0][tid - 1]);
        Q[1][tid] = minor[1][t1] * recip((t1 & 7) == 0 ? first[1][t1 / 8] : minor[1][t1 - 1]);
    }
    __syncthreads();
    // the twist: where the residual of the vector with z = 1 there is smallest
    {
        double g = 1e300;
        int r = 0;
        if (tid < P) {
            g = fabs(Q[0][tid] + Q[1][tid] - (dl[tid] - lambda));
            r = tid;
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const double og = __shfl_xor(g, o, 64);
            const int orr = __shfl_xor(r, o, 64);
            const bool take = og < g || (og == g && orr < r);
            g = take ? og : g;
            r = take ? orr : r;
        }
        if (lane == 0) {
            redd[wave] = g;
            redi[4 + wave] = r;
        }
    }
    __syncthreads();
    double gamma = redd[0];
    int r = redi[4];
    for (int w = 1; w < 4; ++w)
        if (redd[w] < gamma) {
            gamma = redd[w];
            r = redi[4 + w];
        }
    // z: products of ratios outwards from the twist, two scans
    __shared__ double zs[P], ys[P], part[256];
    if (wave == 0) {
        double z[E];
        {
            double up[E], down[E];                 // of entry t of this lane and what lies between it and the twist in the lane
#pragma unroll
            for (int t = 0; t < E; ++t) {
                const int i = E * lane + t;
                up[t] = i < r ? -el[i] * recip(Q[0][i]) : 1.0;
                down[t] = i > r && i < P ? -el[i - 1] * recip(Q[1][i]) : 1.0;
            }
#pragma unroll
            for (int t = E - 2; t >= 0; --t) up[t] *= up[t + 1];
#pragma unroll
            for (int t = 1; t < E; ++t) down[t] *= down[t - 1];
            double u = up[0], d = down[E - 1];     // of the lane; then of all lanes up to it
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const double ou = __shfl_down(u, o, 64), od = __shfl_up(d, o, 64);
                u *= lane + o < 64 ? ou : 1.0;
                d *= lane >= o ? od : 1.0;
            }
            const double ou = __shfl_down(u, 1, 64), od = __shfl_up(d, 1, 64);
#pragma unroll
            for (int t = 0; t < E; ++t)
                z[t] = E * lane + t >= P ? 0.0 : up[t] * (lane < 63 ? ou : 1.0) * down[t] * (lane > 0 ? od : 1.0);
        }
        double n2 = 0.0;
#pragma unroll
        for (int t = 0; t < E; ++t) n2 = fma(z[t], z[t], n2);
        n2 = lanes_sum<64>(n2);
        const double inv = 1.0 / sqrt(n2);
        if (!(gamma * inv <= kResidual * bound) && lane == 0) s.flag[b] = 2;       // (also where it is a NaN)
#pragma unroll
        for (int t = 0; t < E; ++t) z[t] *= inv;
        // Q row = H_0 H_1 .. z; eight reflectors requested at a time
        constexpr int A = 8;
        const float* V = s.v<P>(b);
        const double* beta = s.beta<P>(b);
        float cur[A][E], next[A][E];
        double bc[A], bn[A];
        const int at0 = E * lane < P ? E * lane : 0;
        auto load = [&](float (&v)[A][E], double (&bv)[A], int row) { // rows row .. row + A - 1
#pragma unroll
            for (int a = 0; a < A; ++a) {
                bv[a] = beta[row + a];
#pragma unroll
                for (int t = 0; t < E; ++t) v[a][t] = V[(row + a) * P + at0 + t];
            }
        };
        load(cur, bc, P - A);
#pragma unroll 1
        for (int row = P - A; row >= 0; row -= A) {
            load(next, bn, row >= A ? row - A : 0);
#pragma unroll
            for (int a = A - 1; a >= 0; --a) {
                double dot = 0.0;
#pragma unroll
                for (int t = 0; t < E; ++t) dot = fma((double)cur[a][t], z[t], dot);
                dot = lanes_sum<64>(dot) * -bc[a];
#pragma unroll
                for (int t = 0; t < E; ++t) z[t] = fma(dot, E * lane < P ? (double)cur[a][t] : 0.0, z[t]);
            }
#pragma unroll
            for (int a = 0; a < A; ++a) {
                bc[a] = bn[a];
#pragma unroll
                for (int t = 0; t < E; ++t) cur[a][t] = next[a][t];
            }
        }
#pragma unroll
        for (int t = 0; t < E; ++t)
            if (E * lane + t < P) zs[E * lane + t] = z[t];
    }
    __syncthreads();
    transposed_times<P, 256>(G + (int64_t)b * P * P, zs, part, ys);
    keep_vector<P>(zs, ys, s.z<P>(b, 0) + k * P, s.az<P>(b) + k * P, s.lambda<P>(b, 0) + k);
}

// 3. Step STEP of the refinement of eigenvector blockIdx.x of matrix blockIdx.y: from all vectors z_i of the step before,
// z_k += sum_i E_i z_i with E_i = (z_i^T A z_k - lambda_k z_i^T z_k) / (lambda_k - lambda_i), E_k = (1 - z_k^T z_k) / 2 (first order
// in the error of the z).  Step 2 writes the result.
template <int P>
constexpr int refine_threads() { return P == 256 ? 1024 : P == 64 ? 256 : 64; }
template <int P, int STEP>
__global__ __launch_bounds__(refine_threads<P>()) void refine_kernel(const float* __restrict__ G, EigScratch s, float* __restrict__ D,
                                                                     float* __restrict__ sv) {
    constexpr int NTH = refine_threads<P>(), E = P / 16;
    constexpr double kTurn = STEP == 1 ? 0.1 : 1e-3;
    __shared__ double zs[P], ys[P], turn[P], part[NTH];
    const int b = blockIdx.y, k = blockIdx.x, tid = threadIdx.x, l = tid & 15;
    // uniform: this launch writes no flag but STEP + 2
    const int left = s.flag[b];
    if (left != 0 && left != STEP + 2) return;
    const double* __restrict__ Z = s.z<P>(b, STEP - 1);
    const double* __restrict__ L = s.lambda<P>(b, STEP - 1);
    const double lambda = L[k];
    const auto at = [&](int e) { return E == 1 ? l : (e >> 1) * 32 + 2 * l + (e & 1); };   // entries of a lane of 16
    double zk[E], yk[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        zk[e] = Z[k * P + at(e)];
        yk[e] = s.az<P>(b)[k * P + at(e)];
    }
    if (tid < P) zs[tid] = Z[k * P + tid];
#pragma unroll 2
    for (int q = 0; q < P * 16 / NTH; ++q) {
        const int i = (q * (NTH / 16) + (tid >> 4) + k * 4) & (P - 1);
        double zy = 0.0, zz = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const double z = Z[i * P + at(e)];
            zy = fma(z, yk[e], zy);
            zz = fma(z, zk[e], zz);
        }
        zy = lanes_sum<16>(zy);
        zz = lanes_sum<16>(zz);
        if (l == 0) {
            const double t = i == k ? 0.5 * (1.0 - zz) : fma(-lambda, zz, zy) / (lambda - L[i]);
            if (!(fabs(t) <= kTurn)) s.flag[b] = STEP + 2;     // (also where it is a NaN)
            turn[i] = t;
        }
    }
    __syncthreads();
    transposed_times<P, NTH>(Z, turn, part, ys);
    if constexpr (STEP == 1) {
        if (tid < P) zs[tid] += ys[tid];
        __syncthreads();
        transposed_times<P, NTH>(G + (int64_t)b * P * P, zs, part, ys);
        keep_vector<P>(zs, ys, s.z<P>(b, 1) + k * P, s.az<P>(b) + k * P, s.lambda<P>(b, 1) + k);
    } else {
        // refined eigenvalues may have changed places
        const int rank = __syncthreads_count(tid < P && (L[tid] > lambda || (L[tid] == lambda && tid < k)));
        if (tid < P) D[((int64_t)b * P + rank) * P + tid] = (float)(zs[tid] + ys[tid]);
        if (tid == 0) sv[(int64_t)b * P + rank] = (float)sqrt(fmax(lambda, 0.0));
    }
}

template <int P>
hipError_t launch_eigen_p(int K, const float* M, float* D, float* sv, const EigScratch& s, hipStream_t st) {
    if constexpr (P > 64) hipLaunchKernelGGL(tridiag_wide_kernel, dim3(K), dim3(1024), 0, st, M, s);
    else hipLaunchKernelGGL((tridiag_kernel<P>), dim3(K), dim3(64 * tri_waves<P>()), 0, st, M, s);
    hipLaunchKernelGGL((eig_vectors_kernel<P>), dim3(P, K), dim3(256), 0, st, M, s);
    hipLaunchKernelGGL((refine_kernel<P, 1>), dim3(P, K), dim3(refine_threads<P>()), 0, st, M, s, D, sv);
    hipLaunchKernelGGL((refine_kernel<P, 2>), dim3(P, K), dim3(refine_threads<P>()), 0, st, M, s, D, sv);
    return hipGetLastError();
}

}  // namespace

size_t eigen_scratch_bytes(int p) {
    switch (p) {
        case 16: return EigScratch::bytes<16>();
        case 32: return EigScratch::bytes<32>();
        case 64: return EigScratch::bytes<64>();
        default: return EigScratch::bytes<256>();
    }
}

// As many matrices at a time as the scratch holds.
hipError_t launch_eigen(int p, int K, const float* M, float* D, float* sv, const Workspace& ws, hipStream_t st) {
    hipError_t e = hipSuccess;
    for (int j = 0; j < K && e == hipSuccess; j += ws.eig_room) {
        const int n = K - j < ws.eig_room ? K - j : ws.eig_room;
        const size_t at = (size_t)j * p * p;
        const EigScratch s = {ws.eig, ws.eig_left + j};
        switch (p) {
            case 16: e = launch_eigen_p<16>(n, M + at, D + at, sv + (size_t)j * p, s, st); break;
            case 32: e = launch_eigen_p<32>(n, M + at, D + at, sv + (size_t)j * p, s, st); break;
            case 64: e = launch_eigen_p<64>(n, M + at, D + at, sv + (size_t)j * p, s, st); break;
            case 256: e = launch_eigen_p<256>(n, M + at, D + at, sv + (size_t)j * p, s, st); break;
            default: return hipErrorInvalidValue;
        }
    }
    return e;
}

}  // namespace sbo
