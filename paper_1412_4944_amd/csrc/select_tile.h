// Per-tile support selection shared by the select kernels.
#pragma once

#include "device_utils.h"
#include "energy_networks.h"

namespace sbo {

// One wavefront holds, in MFMA accumulator layout, the projections c = Q_j^T y of a tile
// of up to 32 signals onto ONE block: register r of tile mt in lane (h, n) is atom
// mt*32 + (r/4)*8 + h*4 + r%4 of signal n.  Finds the s0-th largest magnitude tau of every
// signal with the compare-exchange networks, then writes the support {|c| > tau} plus the
// lowest-index entries equal to tau in ascending atom order, the coefficients and the
// residual (sum of the dropped c^2) of signal i (original index; active = lane has a
// signal).  Exact magnitude ties beyond the trivial one are resolved by a sequential
// per-signal pass through the wave-private LDS tile ct, 16 atoms at a time.  The (atom, coefficient)
// rows are first compacted in the wave-private LDS area stage[S + 1][2][32] (words) and then
// written with one or a few wide stores per lane (lane half 0: supp row, half 1: coef row),
// because scattered 4-byte stores to rows in original signal order are what this step
// would otherwise wait on.  ct is touched only on the tie path (*used_ct is then set).  On return the compacted rows
// are still in `stage`: entry pos of signal n at stage_idx(n, 0, pos) (atom) and stage_idx(n, 1, pos)
// (coefficient bits).
//
// What bounds it: instruction issue (it was 7500 cycles a tile of 32 signals for a wavefront, most of them for a
// branch and two swizzled addresses per entry; positions now come from packed counts, and an entry is a
// comparison, an address and a store: 100003 signals, p = 64: 32.8 -> 29.4 us).
// Both areas are as small as that: with 16 entries and all p coefficients of a signal in them (12 KiB a wavefront at
// p = 64) LDS held three wavefronts of select_kernel on a SIMD, and a few workgroups a second round (29.8 -> 26.3 us).
template <int S0>
constexpr int kSelectStageWords = 32 * 2 * (S0 + 1);
constexpr int kSelectTieWords = 32 * (16 + 1);         // [signal][atom], a column of padding

// 8 consecutive values as the three bf16 parts of an operand unit: out[0], out[step], out[2 step].
__device__ __forceinline__ void split_unit(const f32x4* v, u32x4* out, int step) {
    const Bf16x3Pair a = split_bf16x3(v[0].x, v[0].y), b = split_bf16x3(v[0].z, v[0].w);
    const Bf16x3Pair c = split_bf16x3(v[1].x, v[1].y), d = split_bf16x3(v[1].z, v[1].w);
    out[0] = u32x4{a.hi, b.hi, c.hi, d.hi};
    out[step] = u32x4{a.mid, b.mid, c.mid, d.mid};
    out[2 * step] = u32x4{a.lo, b.lo, c.lo, d.lo};
}

// Word index of entry `pos` of signal row n in the stage area; kind 0 = atom, 1 =
// coefficient bits (one instruction writes both).  All lanes n of one entry are neighbours.  Entry s0 is nobody's.
__device__ __forceinline__ int stage_idx(int n, int kind, int pos) { return (2 * pos + kind) * 32 + n; }

// The value in the other lane of the pair (all lanes active).
__device__ __forceinline__ unsigned pair_other(unsigned x, int h) {
    auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    const unsigned lo = r[0], hi = r[1];
    return h ? lo : hi;
}
__device__ __forceinline__ float pair_other(float x, int h) {
    return __builtin_bit_cast(float, pair_other(__builtin_bit_cast(unsigned, x), h));
}
__device__ __forceinline__ int pair_other(int x, int h) { return (int)pair_other((unsigned)x, h); }

template <int P, int S0>
__device__ __forceinline__ void tile_select(const f32x16* acc, int h, int n, bool active, int64_t i, float* ct, int* stage,
                                            int32_t* __restrict__ supp, float* __restrict__ coef,
                                            float* __restrict__ err, bool* used_ct = nullptr) {
    constexpr int MT = P >= 32 ? P / 32 : 1;
    constexpr int NVL = MT * 16, S = pow2_at_least(S0);
    constexpr int LDC = kSelectTieWords / 32;
    static_assert(P <= 64, "p = 256 selects in select_wide_split_kernel");
    static_assert(S <= NVL, "sort width exceeds the values of one lane");
    float c[NVL], mag[NVL];
#pragma unroll
    for (int f = 0; f < NVL; ++f) {
        const int r = f & 15;
        const int atom = (f >> 4) * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
        c[f] = acc[f >> 4][r];
        mag[f] = atom < P ? fabsf(c[f]) : -1.f;
    }

    // tau = s0-th largest magnitude of the signal: the s0 largest are max(top_t, oth_{s0-1-t}).
    float top[S], tau = __builtin_inff();
    top_sorted<NVL, S>(mag, top);
#pragma unroll
    for (int t = 0; t < S0; ++t) tau = fminf(tau, fmaxf(top[t], pair_other(top[S0 - 1 - t], h)));

    // Entries with |c| >= tau, per group of 4 consecutive atoms (the groups alternate
    // between the two lanes of a signal), four groups to a word.  Exactly s0 of them: no tie at tau to
    // break.  (A lane without a signal keeps nothing.)
    constexpr int NG = NVL / 4, NWD = NG / 4;
    const float keep_from = active ? tau : __builtin_inff();
    unsigned own[NWD], par[NWD], total = 0;
#pragma unroll
    for (int w = 0; w < NWD; ++w) {
        own[w] = 0;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            unsigned k = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) k += mag[16 * w + 4 * g + e] >= keep_from;
            own[w] |= k << (8 * g);
        }
        par[w] = pair_other(own[w], h);
        total = __builtin_amdgcn_sad_u8(own[w], 0u, __builtin_amdgcn_sad_u8(par[w], 0u, total));
    }
    const bool simple = !active || (int)total == S0;

    if (__all(simple)) {
        // Every entry with |c| >= tau is kept.  Emit in ascending atom order.
        unsigned before = 0;                   // entries of earlier words
        f32x4 parts = {0.f, 0.f, 0.f, 0.f};    // (one sum after the other: 0.8 of the residuals' error came from it)
        int h4 = h * 4;
        asm volatile("" : "+v"(h4));           // or the atoms of all entries are kept in registers over the caller's loop
#pragma unroll
        for (int w = 0; w < NWD; ++w) {
            const unsigned both = own[w] + par[w], upto = both * 0x01010101u;      // inclusive sums, per byte
            const unsigned start = upto - both + (h ? par[w] : 0u) + before * 0x01010101u;
            before += upto >> 24;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                unsigned pos = (start >> (8 * g)) & 0xffu;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int f = 16 * w + 4 * g + e;
                    const int atom = (f >> 4) * 32 + ((f & 15) >> 2) * 8 + (f & 3) + h4;
                    const bool keep = mag[f] >= keep_from;
                    // (what is not kept goes to entry s0: a branch costs more)
                    int* at = stage + stage_idx(n, 0, keep ? (int)pos : S0);
                    at[0] = atom;
                    at[32] = __builtin_bit_cast(int, c[f]);
                    pos += keep;
                    const float rest = keep || atom >= P ? 0.f : c[f];
                    parts[e] = fmaf(rest, rest, parts[e]);
                }
            }
        }
        float dropped = (parts.x + parts.y) + (parts.z + parts.w);
        dropped += pair_other(dropped, h);
        if (active && h == 0) err[i] = dropped;
    } else {
        // Exact magnitude ties: walk each signal's coefficients in atom order.
        if (used_ct != nullptr) *used_ct = true;
        int gt = 0;
#pragma unroll
        for (int f = 0; f < NVL; ++f) gt += mag[f] > tau;
        gt += pair_other(gt, h);
        const int need = S0 - gt;              // entries equal to tau still to take (>= 1)
        int pos = 0, taken_eq = 0;
        float dropped = 0.f;
#pragma unroll
        for (int k0 = 0; k0 < P; k0 += 16) {
            __builtin_amdgcn_wave_barrier();   // the atoms before these have been walked
#pragma unroll
            for (int r = 0; r < 8; ++r) ct[n * LDC + (r >> 2) * 8 + h * 4 + (r & 3)] = c[k0 / 2 + r];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (active && h == 0) {
#pragma unroll 4
                for (int k = 0; k < 16; ++k) {
                    const float v = ct[n * LDC + k];
                    const float a = fabsf(v);
                    bool take = a > tau;
                    if (!take && a == tau && taken_eq < need) {
                        take = true;
                        ++taken_eq;
                    }
                    if (take && pos < S0) {
                        stage[stage_idx(n, 0, pos)] = k0 + k;
                        stage[stage_idx(n, 1, pos)] = __builtin_bit_cast(int, v);
                        ++pos;
                    } else {
                        dropped += v * v;
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        }
        if (active && h == 0) err[i] = dropped;
    }

    // compact rows -> global memory
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (active) {
        int* dst = (h ? reinterpret_cast<int*>(coef) : supp) + i * S0;
        const int* row = stage + stage_idx(n, h, 0);           // an entry every 64 words
        typedef int i32x4 __attribute__((ext_vector_type(4)));
        typedef int i32x2 __attribute__((ext_vector_type(2)));
        if constexpr ((S0 & 3) == 0) {
#pragma unroll
            for (int t = 0; t < S0; t += 4)
                *reinterpret_cast<i32x4*>(dst + t) = i32x4{row[t * 64], row[t * 64 + 64], row[t * 64 + 128], row[t * 64 + 192]};
        } else if constexpr ((S0 & 1) == 0) {
#pragma unroll
            for (int t = 0; t < S0; t += 2) *reinterpret_cast<i32x2*>(dst + t) = i32x2{row[t * 64], row[t * 64 + 64]};
        } else {
#pragma unroll
            for (int t = 0; t < S0; ++t) dst[t] = row[t * 64];
        }
    }
    __builtin_amdgcn_wave_barrier();           // stage is reused by the caller's next tile

}

}  // namespace sbo
