// The Newton-Schulz iteration X <- X (3 I - X^T X) / 2: its last step, and its scaling for p = 256 (polar_wide.hip).
//
// With all singular values in [l, 1], X scaled by alpha(l) = sqrt(3 / (1 + l + l^2)) before a step makes the
// step's polynomial f(s) = alpha s (3 - (alpha s)^2) / 2 map [l, 1] to the smallest possible interval
// [l', 1], l' = f(l).  A smaller singular value is safe (f is positive and at most one on
// (0, sqrt(3))), but it grows by only 3/2 a step once alpha is 1: so l starts at a guess by the spread of the
// singular values (0.45, 0.16 or 0.064, below; block matrices of a trained dictionary have condition numbers of 2 to 10) and is lowered when a column of X shows it to be
// wrong: the smallest column norm is an upper bound of the smallest singular value, and where atoms are
// rarely used it is close to it.  From 0.5 on the values have met and it is left alone.  (Simulated on block
// matrices of first training rounds, condition 60 to 5000: 9 to 15 steps instead of 11 to 22; condition
// below 7: as without it.  p <= 64, condition 3 to 14, has fixed scalings for a first l by the spread alone
// (polar_ns.hip): a step less in some rounds was what the bookkeeping cost.)
//
// A narrow spectrum (atoms used equally often, over many signals) is the exception, for every p: alpha(0.16) would send
// singular values that are all near one down to 0.375 first, where the rounding of the step weighs 1 / 0.375 as
// much (condition 1.02: |Q - exact|_F / sqrt(p) 2.0e-7 in five steps at p = 64, 4.0e-7 in six at p = 256; with alpha = 1
// 4.5e-8 in two, 1.0e-7 in three; p = 256, condition 1.2 2.7e-7, 9.9e-8).  The
// eigenvalues of G have the mean mu = tr G / p and the mean square |G|_F^2 / p, so their spread is known after the
// first product, and the scale that centres them needs no estimate of the largest.  The line (spread below
// kNarrow mu): p <= 64 0.1, condition up to 1.2 where all singular values share in it, which one small value among
// 64 (0.125) does not meet.  p = 256 0.25 (condition 1.5; the rounding of more products weighs more), and no
// column below half the mean.
#pragma once

#include <hip/hip_runtime.h>

namespace sbo {

// The last step is X (I + c1 E + c2 E^2), E = I - X^T X, for |E|_F < 1e-2: (1 - e)^(-1/2) on [0, eps] (no step leaves a
// singular value above one, so E has no negative eigenvalue to speak of).  The third term of the series, 5/16 e^3
// (3e-7 where one singular value lags behind the others: more than fp32 rounding), is interpolated: 5/16 times
// e^3 - 3/2 eps e^2 + 9/16 eps^2 e lies between 0 and eps^3 / 16, 2e-8 off at most.  kLastLinear = 2 c1,
// kLastSquare = 2 c2.
constexpr float kLastEps = 1e-2f;
constexpr float kLastLinear = 1.f - 5.f / 8 * 9 / 16 * kLastEps * kLastEps, kLastSquare = 0.75f + 5.f / 8 * 3 / 2 * kLastEps;

template <int P>
__device__ constexpr float kNarrow = P <= 64 ? 0.1f : 0.25f;
// sum2 = |G|_F^2
template <int P>
__device__ __forceinline__ bool narrow_spectrum(float sum2, float mu) {
    return sum2 < P * (1.f + kNarrow<P> * kNarrow<P>) * (mu * mu);
}

// p = 256: the first l by the spread of the squared singular values (sum2 / (p mu^2) - 1), 0.16 between the lines.  Below the lower
// one 0.45 takes a step less (condition 1.5 to 2), and the error falls by a third; above the other one 0.064 takes up to two
// less (sets of 2048 signals, 12 atoms a signal: 8.5 -> 7 on average; Algorithm 2 to K = 4, 16384 signals 5646 -> 5587 us), with
// an error of 1.0 to 1.09.  With that line at 1.4, 8192 signals of 5 atoms took 7 steps instead of 6.
constexpr float kHighSpread = 2.5f, kHighL = 0.064f, kLowSpread = 0.18f, kLowL = 0.45f;

struct NsScale {
    float l = 0.16f;           // before the present step
    float alpha = 1.f, lower = 1.f;            // of the step before: its scaling, its l

    __device__ __forceinline__ float take(float alpha_) {
        alpha = alpha_;
        lower = l;
        l = fminf(map(l), 1.f);
        return alpha;
    }
    __device__ __forceinline__ float map(float s) const {
        const float a = alpha * s;
        return a * (1.5f - 0.5f * a * a);
    }
    __device__ __forceinline__ static float best(float s) {
        return s < 0.99f ? __builtin_amdgcn_sqrtf(3.f * __builtin_amdgcn_rcpf(1.f + s + s * s)) : 1.f;
    }
    // The first step, which also scales the input: the iteration sends every singular value in (0, sqrt(3))
    // to +1, one in (sqrt(3), sqrt(5)) to -1 (an orthogonal matrix that is NOT U V^T, and which no later
    // test can tell apart), so the scale must be a guaranteed bound: the largest absolute row sum of
    // G = X^T X is at least its largest eigenvalue sigma_max^2, and alpha^2 <= 2.9 / that keeps every
    // scaled sigma^2 below 2.9.  Where the bound is tight, the aim is sigma_max = 1 times alpha(l), with
    // the largest norm of a column of G (a lower bound of its largest eigenvalue) as the estimate.
    // row_sum: the former; col2: the square of the latter; diag: the smallest diagonal entry of G; sum2, mu: above.
    __device__ __forceinline__ float first(float row_sum, float col2, float diag, float sum2, float mu) {
        float b2 = 2.9f * __builtin_amdgcn_rcpf(row_sum);
        if (narrow_spectrum<256>(sum2, mu) && diag > 0.5f * mu) {
            l = 1.f;
            lower = 0.f;
            return __builtin_amdgcn_sqrtf(fminf(b2, __builtin_amdgcn_rcpf(mu)));
        }
        float est = row_sum * (1.f / 1.4f);    // of sigma_max^2
        if (col2 > 1e-37f && col2 < 3e37f) {
            est = 1.04f * __builtin_amdgcn_sqrtf(col2);
            const float r = diag > 0.f ? __builtin_amdgcn_sqrtf(diag * __builtin_amdgcn_rcpf(est)) : 0.f;
            const float even = 256 * (mu * mu);
            if (sum2 > (1.f + kHighSpread) * even) l = kHighL;
            else if (sum2 < (1.f + kLowSpread) * even) l = kLowL;
            l = fmaxf(fminf(l, r), 1e-3f);
            const float a = best(l);
            b2 = fminf(b2, a * a * __builtin_amdgcn_rcpf(est));
        }
        const float scale = __builtin_amdgcn_sqrtf(b2);
        // in units of X / sqrt(est)
        take(__builtin_amdgcn_sqrtf(b2 * est));
        alpha = 1.f;                           // (a column norm seen now is of the unscaled X: not used)
        lower = 0.f;
        return scale;
    }
    __device__ __forceinline__ float next() { return take(best(l)); }
    // diag: the smallest diagonal entry of X^T X before the step whose alpha was taken last
    __device__ __forceinline__ void seen(float diag) {
        const float s = __builtin_amdgcn_sqrtf(fmaxf(diag, 0.f));
        if (s < lower && s < 0.5f) l = fmaxf(map(s), 1e-3f);
    }
};

}  // namespace sbo
