// Sparse-coding stage 1, the block choice (Section 2, eq. (4); Section 3.1), screened: for every
// signal the orthobase whose s0 largest coefficients hold the most energy.
//
// What bounds the choice is not memory (Y is read once, 256 bytes a signal at p = 64, against
// 2 K p^2 flop) but the matrix cores AND the vector ALU: with full-precision coefficients, K = 32 and
// p = 64 take three fp16 products per product (82 us of matrix time for 262144 signals) and 250
// vector instructions per 32 signals and block for the selection networks (104 us), and the two
// overlap badly.  Almost all of that precision is spent on blocks that are far from winning.  So:
//
//   1. Screening.  One fp16 product per product (the leading fp16 part of the signal, scaled, times
//      the leading part of the dictionary) gives every coefficient to about 2^-11; the magnitudes
//      are rounded down to fp16.
//        p = 64, s0 >= 4: the kept energy is only bounded from above.  For any t,
//            sum of the s0 largest c^2  <=  sum over all of max(c^2, t) - (p - s0) t,
//      with equality at the s0-th largest one: two instructions per pair of magnitudes (a maximum and a dot
//      product) instead of the six or more of a selection network.  t is where the s0-th largest of p normal
//      values of the signal's energy lies: blocks that are far from the signal look like that, and where the
//      coefficients of the right one stand out the bound is nearly exact.  The magnitudes of the block that
//      is ahead stay in registers, and at the end one selection network gives its kept energy.
//        Otherwise: the networks for every block, on two signals per instruction (energy_networks.h).
//      The bound or kept energy of every (signal, block) goes to LDS, 16 bits each.
//   2. Decision.  The s0 largest magnitudes' norm of a block is off by at most
//          eps = sqrt(s0) (max |q| |y - hi(y)| + |y| max |q - hi(q)| + accumulation)
//      (Cauchy-Schwarz per coefficient; the two remainders' norms are computed, not bounded) and by
//      the rounding down of the magnitudes, less than 2^-10 of itself.  A block that is (whose bound is) further
//      than that below the kept energy of the one ahead cannot win.  A signal with one block left is
//      decided.
//   3. Resolution.  For the others, the blocks that are left are computed in the context's
//      arithmetic (SBO_ARITH_*), operand by operand and sum by sum what the kernels in
//      code_energy.hip do, and compared: the largest energy wins, the lower block on a tie.
// The chosen blocks are therefore those of the full computation, for every dictionary (nothing is
// assumed about D; the bound is just wide if its atoms are long).  Where a dictionary is known to consist of orthobases
// most blocks take less (home blocks, guessed blocks: below).
//
// Two shapes of the same work:
//   energy_screen_kernel<..., false, W, Choice>: a workgroup takes 64 W signals, a wavefront 64 of them and all
//     blocks; dictionary stages go through LDS, double-buffered.  W = 8; W = 4, two workgroups per CU, for a last
//     round that W = 8 would not fill.
//   energy_screen_kernel<..., true, 8, kFull>: a workgroup takes 64 signals, and its wavefronts share out the
//     blocks and read their dictionary rows straight from L2: more workgroups, for signal sets that
//     would not fill the chip otherwise, and for K beyond the LDS table of the other.  Up to 8192 signals several
//     workgroups share out the blocks (choice_split).
//
// Measured (MI355X, f16x2 results; "before" is the full-precision projection of every block): K = 32, p = 64,
// s0 = 8, 262144 signals 229 us before, 126 with networks for every block, 100 with bounds; K = 128, s0 = 6, 2^20
// signals 3283, 1712, 1400 us; p = 256, K = 16, 131072 signals 757 -> 288 us; K = 16, 16384 signals (the second
// shape) 28 -> 9 us.  Of the 100 us, 66 are the main loop at 45 us of matrix work (at the 1530 TFLOP/s that the
// chip sustains on such operands) and 40 of vector work, which share the power budget.
#pragma once

#include "sbo_internal.h"
#include "device_utils.h"
#include "energy_networks.h"
#include "screen_args.h"

#include <type_traits>

namespace sbo {

namespace {

constexpr int kScrWaves = 8;                   // at most
constexpr size_t kScrLdsMax = 160 * 1024;

// Maximum over the wavefront, in all lanes.
__device__ __forceinline__ float wave_max(float x) {
    x = row16_max(x);
    const unsigned u = __builtin_bit_cast(unsigned, x);
    auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned a0 = r[0], a1 = r[1];
    const float y = fmaxf(__builtin_bit_cast(float, a0), __builtin_bit_cast(float, a1));
    const SwapPair q = swap32(y, y);
    return fmaxf(q.first, q.second);
}

template <int P>
struct ScrGeom {
    static constexpr bool WIDE = P > 64;
    static constexpr int KS16 = P / 16;                     // contraction steps of 16 dims
    static constexpr int NB = WIDE ? 1 : 64 / P;            // blocks per 64-row stage (p <= 64)
    static constexpr int SPB = WIDE ? P / 32 : 1;           // stages of 32 rows per block (p = 256)
    static constexpr int MTS = WIDE ? 1 : 2;                // 32-row tiles per stage
    static constexpr int STAGE_U = MTS * KS16 * 64;         // 16-byte units of a stage (leading parts only)
    static constexpr int NV = WIDE ? 16 : P / 2;            // coefficients per lane, block and stage
};

// Which sizes screen with bounds from above (the header): where a wavefront meets enough blocks to pay for
// the selection at the end, and where that is long (p = 64, K = 32, 262144 signals: s0 = 2 176 us with bounds,
// 166 with networks; s0 = 8 181, 195; p = 32, s0 = 12 107, 102).
constexpr bool scr_bound(int P, int SX, bool shared) { return P == 64 && SX >= 4 && !shared; }

// A lane's half of signal i (-1: none), as exact_energy takes it (p = 256: it reads the signal itself).
template <int P, int ARITH>
struct ExactRow {
    static constexpr int N = P <= 64 ? P / 8 : 1;
    f32x4 v[N];
    __device__ __forceinline__ void load(const ScrArgs& g, int64_t i, int h) {
        if constexpr (P <= 64) {
            const f32x4* row = reinterpret_cast<const f32x4*>(g.Y + (i < 0 ? 0 : i) * P);
#pragma unroll
            for (int k = 0; k < N; ++k) {
                v[k] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (i >= 0) v[k] = row[ARITH == 0 ? h * N + k : (k >> 1) * 4 + h * 2 + (k & 1)];
            }
        }
    }
};

// Kept energy of signal i (-1: none; y: its row) in block j in the exact arithmetic, up to the signal's scale.
// DIRECT: the operands are made from the rows of D here (p <= 64), bit by bit what dict_parts_kernel makes of them.
template <int P, int S, int SX, int ARITH, bool DIRECT = false>
__device__ __forceinline__ float exact_energy(const ScrArgs& g, const ExactRow<P, ARITH>& y, int64_t i, int j, int lane) {
    constexpr int KS16 = P / 16, QN = P / 8;
    constexpr int NPL = ARITH == 3 ? 2 : 3;
    constexpr int NRT = P >= 32 ? P / 32 : 1;               // 32-row tiles of a block
    constexpr int NV = P <= 64 ? P / 2 : 16;
    const int h = lane >> 5;
    const int tile0 = P >= 32 ? j * NRT : j >> 1;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const float* yrow = g.Y + (i < 0 ? 0 : i) * P;
    auto part = [&](int ks, int e) {           // dims ks*16 + h*8 + 4 e .. +3
        if constexpr (P <= 64) return y.v[2 * ks + e];
        else return i >= 0 ? *reinterpret_cast<const f32x4*>(yrow + ks * 16 + h * 8 + 4 * e) : f32x4{0.f, 0.f, 0.f, 0.f};
    };

    // dims 4 d4 .. +3 of this lane's row of tile mt (DIRECT)
    auto row = [&](int mt, int d4) {
        const int r = (tile0 + mt) * 32 + (lane & 31);
        return r < g.K * P ? *reinterpret_cast<const f32x4*>(g.D + (int64_t)r * P + 4 * d4) : f32x4{0.f, 0.f, 0.f, 0.f};
    };
    if constexpr (ARITH == 0) {
        static_assert(P <= 64, "p = 256 in fp32 is not screened");
        const f32x4* D = reinterpret_cast<const f32x4*>(g.Dx) + (int64_t)tile0 * (QN * 64) + lane;
        f32x4 a[QN][NRT];                      // (all on their way at once)
#pragma unroll
        for (int q = 0; q < QN; ++q)
#pragma unroll
            for (int mt = 0; mt < NRT; ++mt) a[q][mt] = DIRECT ? row(mt, h * QN + q) : D[(mt * QN + q) * 64];
        f32x16 acc[NRT];
#pragma unroll
        for (int q = 0; q < QN; ++q) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                for (int mt = 0; mt < NRT; ++mt)
                    acc[mt] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q][mt][kk], y.v[q][kk],
                                                                   (q == 0 && kk == 0) ? zero : acc[mt], 0, 0, 0);
        }
        float x[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v)
            x[v] = fabsf(P == 16 ? ((j & 1) ? acc[0][(8 + v) & 15] : acc[0][v & 15]) : acc[(v >> 4) % NRT][v & 15]);
        return pair_top_energy<NV, S, SX>(x, g.s0, h != 0);
    } else {
        const u32x4* D = reinterpret_cast<const u32x4*>(g.Dx) + (int64_t)tile0 * (KS16 * NPL * 64) + lane;
        constexpr bool AHEAD = P <= 64;        // the dictionary rows on their way before anything else
        u32x4 a_all[AHEAD ? KS16 : 1][AHEAD ? NRT : 1][NPL];
        if constexpr (AHEAD && DIRECT) {
            f32x4 raw[KS16][NRT][2];
#pragma unroll
            for (int ks = 0; ks < KS16; ++ks)
#pragma unroll
                for (int mt = 0; mt < NRT; ++mt)
#pragma unroll
                    for (int e = 0; e < 2; ++e) raw[ks][mt][e] = row(mt, ks * 4 + h * 2 + e);
#pragma unroll
            for (int ks = 0; ks < KS16; ++ks)
#pragma unroll
                for (int mt = 0; mt < NRT; ++mt) {
                    const f32x4 v0 = raw[ks][mt][0], v1 = raw[ks][mt][1];
                    if constexpr (ARITH == 3) {
                        float q2 = 0.f, r2 = 0.f;
                        const F16x2Quad a = split_f16x2_dict(v0, q2, r2), b = split_f16x2_dict(v1, q2, r2);
                        a_all[ks][mt][0] = u32x4{a.hi.x, a.hi.y, b.hi.x, b.hi.y};
                        a_all[ks][mt][1] = u32x4{a.lo.x, a.lo.y, b.lo.x, b.lo.y};
                    } else {
                        const Bf16x3Pair a = split_bf16x3(v0.x, v0.y), b = split_bf16x3(v0.z, v0.w);
                        const Bf16x3Pair c = split_bf16x3(v1.x, v1.y), d = split_bf16x3(v1.z, v1.w);
                        a_all[ks][mt][0] = u32x4{a.hi, b.hi, c.hi, d.hi};
                        a_all[ks][mt][1] = u32x4{a.mid, b.mid, c.mid, d.mid};
                        a_all[ks][mt][NPL - 1] = u32x4{a.lo, b.lo, c.lo, d.lo};
                    }
                }
        } else if constexpr (AHEAD) {
#pragma unroll
            for (int ks = 0; ks < KS16; ++ks)
#pragma unroll
                for (int mt = 0; mt < NRT; ++mt)
#pragma unroll
                    for (int pl = 0; pl < NPL; ++pl) a_all[ks][mt][pl] = D[((mt * KS16 + ks) * NPL + pl) * 64];
        }
        float scale = 1.f;
        if constexpr (ARITH == 3) {
            float vmax = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS16; ++ks)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const f32x4 v = part(ks, e);
                    vmax = fmaxf(fmaxf(fmaxf(vmax, fabsf(v.x)), fmaxf(fabsf(v.y), fabsf(v.z))), fabsf(v.w));
                }
            vmax = fmaxf(vmax, other_half(vmax));
            scale = f16_signal_scale(vmax);
        }
        u32x4 yq[KS16][NPL];
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) {
            const f32x4 v0 = part(ks, 0), v1 = part(ks, 1);
            if constexpr (ARITH == 3) {
                const F16x2Pair a = split_f16x2(v0.x * scale, v0.y * scale), b = split_f16x2(v0.z * scale, v0.w * scale);
                const F16x2Pair c = split_f16x2(v1.x * scale, v1.y * scale), d = split_f16x2(v1.z * scale, v1.w * scale);
                yq[ks][0] = u32x4{a.hi, b.hi, c.hi, d.hi};
                yq[ks][1] = u32x4{a.lo, b.lo, c.lo, d.lo};
            } else {
                const Bf16x3Pair a = split_bf16x3(v0.x, v0.y), b = split_bf16x3(v0.z, v0.w);
                const Bf16x3Pair c = split_bf16x3(v1.x, v1.y), d = split_bf16x3(v1.z, v1.w);
                yq[ks][0] = u32x4{a.hi, b.hi, c.hi, d.hi};
                yq[ks][1] = u32x4{a.mid, b.mid, c.mid, d.mid};
                yq[ks][NPL - 1] = u32x4{a.lo, b.lo, c.lo, d.lo};
            }
        }
        // the partial products, smallest first: (A part, B part)
        constexpr bool F16 = ARITH == 3;
        constexpr int TA[6] = {F16 ? 0 : 2, F16 ? 1 : 0, F16 ? 0 : 1, 1, 0, 0};
        constexpr int TB[6] = {F16 ? 1 : 0, F16 ? 0 : 2, F16 ? 0 : 1, 0, 1, 0};
        constexpr int T1 = F16 ? 3 : 6;
        auto step = [&](const u32x4 (&a)[NPL], int ks, int t, f32x16 c) {
            if constexpr (F16)
                return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a[TA[t]]),
                                                              __builtin_bit_cast(f16x8, yq[ks][TB[t]]), c, 0, 0, 0);
            else
                return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[TA[t]]),
                                                               __builtin_bit_cast(bf16x8, yq[ks][TB[t]]), c, 0, 0, 0);
        };
        if constexpr (P <= 64) {
            f32x16 acc[NRT];
#pragma unroll
            for (int ks = 0; ks < KS16; ++ks) {
#pragma unroll
                for (int t = 0; t < T1; ++t)
#pragma unroll
                    for (int mt = 0; mt < NRT; ++mt) acc[mt] = step(a_all[ks][mt], ks, t, (ks == 0 && t == 0) ? zero : acc[mt]);
            }
            float x[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v)
                x[v] = fabsf(P == 16 ? ((j & 1) ? acc[0][(8 + v) & 15] : acc[0][v & 15]) : acc[(v >> 4) % NRT][v & 15]);
            return pair_top_energy<NV, S, SX>(x, g.s0, h != 0);
        } else {
            // the two halves of the contraction are summed separately, as the two wavefronts of
            // energy_split_wide_kernel do
            float run[S];
#pragma unroll 1
            for (int rt = 0; rt < NRT; ++rt) {
                f32x16 half[2];
#pragma unroll
                for (int ks = 0; ks < KS16; ++ks) {
                    u32x4 a[NPL];
#pragma unroll
                    for (int pl = 0; pl < NPL; ++pl) a[pl] = D[((rt * KS16 + ks) * NPL + pl) * 64];
                    constexpr int KH = KS16 / 2;
#pragma unroll
                    for (int t = 0; t < T1; ++t)
                        half[ks / KH] = step(a, ks, t, (ks % KH == 0 && t == 0) ? zero : half[ks / KH]);
                }
                float x[16], top[S];
#pragma unroll
                for (int v = 0; v < 16; ++v) x[v] = fabsf(half[0][v] + half[1][v]);
                top_sorted<16, S>(x, top);
                if (rt == 0) {
#pragma unroll
                    for (int t = 0; t < S; ++t) run[t] = top[t];
                } else {
#pragma unroll
                    for (int t = 0; t < S; ++t) run[t] = fmaxf(run[t], top[S - 1 - t]);
                    bitonic_merge_desc<S>(run);
                }
            }
            return pair_list_energy<S, SX>(run, g.s0, h != 0);
        }
    }
}

// LDS of a workgroup:
//   front       two dictionary stages (SHARED, p = 256: the signals); then the tasks of the resolution, then
//               the chunk histogram
//   E16         [K rounded up to whole stages][signals] 16 bits
//   (front and E16 together first hold the signals while they are converted)
//   thr, y2, r2 [signals] floats; key [signals] 64 bits; small change
template <int P, bool SHARED, int W>
constexpr size_t scr_front_bytes() {
    const size_t stages = SHARED ? (P > 64 ? (size_t)64 * P * 2 : 0) : (size_t)2 * ScrGeom<P>::STAGE_U * 16;
    return stages > 8192 ? stages : 8192;      // the wavefronts' results (SHARED), the tasks, the histogram
}
template <int P, bool SHARED, int W>
constexpr size_t scr_table_bytes(int K) {      // front + E16
    constexpr int NB = ScrGeom<P>::NB;
    const size_t rows = (size_t)((K + NB - 1) / NB * NB), sig = SHARED ? 64 : 64 * W;
    const size_t a = scr_front_bytes<P, SHARED, W>() + ((rows * sig * 2 + 15) & ~(size_t)15);
    const size_t signals = SHARED ? (size_t)64 * P * 2 : (size_t)W * 4096;
    return a > signals ? a : signals;
}
template <int P, bool SHARED, int W>
constexpr size_t scr_lds_bytes(int K) {
    return scr_table_bytes<P, SHARED, W>(K) + (size_t)(SHARED ? 64 : 64 * W) * 20 + (2 * W + (SHARED ? 2 : 4)) * 4;
}

// The workgroups of 64 signals take every K that the boundary accepts; p = 256: up to the line of screen_applies.
static_assert(scr_lds_bytes<16, true, kScrWaves>(1024) <= kScrLdsMax && scr_lds_bytes<32, true, kScrWaves>(1024) <= kScrLdsMax &&
                  scr_lds_bytes<64, true, kScrWaves>(1024) <= kScrLdsMax,
              "p <= 64: K up to 1024");
static_assert(scr_lds_bytes<256, true, kScrWaves>(kScreenWideMaxK) <= kScrLdsMax &&
                  scr_lds_bytes<256, true, kScrWaves>(kScreenWideMaxK + 1) > kScrLdsMax,
              "p = 256: K up to kScreenWideMaxK");

// One step of the main loop issues the matrix instructions of the NEXT rows and the selection networks
// of the present ones, NM and about NVALU instructions; spread them evenly: a matrix instruction
// occupies its pipe for 32 cycles and the vector ALU runs beside it, but only if the wavefront
// has something else to issue (measured: 16 matrix and 304 vector instructions, two wavefronts per
// SIMD, 2940 cycles interleaved; 3830 when the two wavefronts multiply and select in turns).
template <int NM, int NVALU>
__device__ __forceinline__ void interleave() {
    constexpr int kFirst = NVALU / NM;         // while the first operands come from LDS
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);                  // LDS reads
    __builtin_amdgcn_sched_group_barrier(0x002, kFirst, 0);             // vector ALU
#pragma unroll
    for (int i = 0; i < NM; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);              // matrix
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, (NVALU - kFirst) / NM, 0);
    }
}

// Home blocks (sbo_iterate from its second iteration on, where it takes more than 64 signals per workgroup): the signals are
// taken in the order of the previous grouping, so that most of the signals of a workgroup belong to one block, their home.  That block is screened first, in full.  For every other
// one, of which the update has just made an orthobase (sweeps), home_rows atoms decide: with R = the part of the signal's energy that
// they leave, and for any t,
//     kept energy  <=  R + s0 t + sum over them of (c^2 - min(c^2, t))  =  |y|^2 + s0 t - sum of min(c^2, t),
// which a block that has nothing to do with the signal does not bring near the kept energy of the home block of a signal that the
// dictionary represents well.  What comes near is resolved like all other candidates, so that the chosen blocks remain those of the
// full computation.  Where more than one signal in kHomeFew<P> is not represented well (kept energy below home_line), or a block
// is no orthobase, everything is screened in full: in the order of the signals if the last iteration says so, or by the workgroup that
// finds it.  Half of the products and of the selection (p = 64; p = 256: a quarter of the products, and no networks), with
// trained dictionaries: K = 32, s0 = 8, 262144 signals 104 -> 78 us, K = 128, s0 = 6, 2^20 signals 1380 -> 760, p = 256,
// K = 16, s0 = 12, 131072 signals 302 -> 115.  What is left: the products at the power limit (1.2 us a step of 16 matrix
// instructions and 130 vector instructions a wavefront), the load of the signals (7 us a workgroup of 512, p = 256 21: HBM), p = 256
// the home block (16 us).
template <int P>
constexpr float home_line(int s0) {            // weak signals (home_rest)
    return 1.f + kHomeT * s0 / P - home_rest(P);
}
// Which sizes have a kernel for home blocks: where signals at 20 dB are above the line (p = 64: s0 <= 9, p = 256: all).
template <int P>
constexpr bool home_applies(int s0) {
    return (P == 64 || P == 256) && home_line<P>(s0) < 0.97f;
}
// Without a grouping to start from (sbo_code, the first iteration; p = 64): the bounds of all blocks first.  That of a signal's
// own block is hardly below |y|^2, because half of its large coefficients is not among the atoms looked at, so the block of the
// largest bound is taken as its home, and only there is it screened in full, in tiles of 32 signals of one block.  That the
// dictionary consists of orthobases, dict_parts_kernel has measured: |Q Q^T - I|_F at most kOrthobase.  So it has that at most
// guess_weak(K) of a sample of kSample signals are weak: a workgroup sees it only when the bounds are made, and has then half as much
// work behind it as full screening takes.  262144 signals, K = 32, s0 = 8: full 106 us, guesses 95; with 2 of the 32 blocks random full 125,
// guesses anyway 199, as it is 129; random dictionary 139, 142.  (The bounds of the first blocks, seen by every workgroup for itself, tell
// only that no signal at all is represented: 199 and 149.)
// 100003 signals, K = 64, s0 = 5: call 125 -> 100; 10^6, K = 128, s0 = 6: choice 1220 -> 855.
constexpr float kOrthobase = 1e-4f;
constexpr int kGuessMaxS0 = 8, kGuessMinK = 20, kGuessMaxK = 160;           // (160: the lists of a workgroup fit where its stages were)

// Weak signals.  Such bounds leave them with most blocks, and a tile of one signal is as much work as one of 32: K tiles for the first
// weak signal of a workgroup (3.3 us each, a wavefront).  So all of them in a workgroup are listed and screened in all blocks, by all atoms
// (p = 64; at p = 256 a tile is a small part of the work).  262144 signals, K = 32, s0 = 8, 1 % of them noise, full / so / left to the
// resolution: sbo_code 113 / 109 / 128, six iterations 614 / 555 / 638; 100003, K = 64, 3 % 99 / 84 / 107.  Bad guesses too: 100003, K = 128,
// s0 = 8 164 / 125, left to the resolution 165.
// Where it pays: iterations, of the signals counted, which are the first 64 of every kWeakEvery-th workgroup (all of them: 4096 atomic
// additions to one address, 262144 signals 125 -> 152 us), one in kHomeFew (K = 32, 9 % noise, full 675, home blocks 653; K = 128 10 % 3870,
// 3160; p = 256, whose weak signals go to the resolution, less); of a workgroup one in kWeakFew.  Guesses, of the sample, guess_weak(K): the
// gain grows with K, choice of 262144 signals, K = 24, s0 = 6, full / guesses: 1 % noise 94 / 92, K = 32, s0 = 8 1 % 113 / 109, 2 % 117 / 114, 6 %
// 125 / 144; 100003, K = 64, s0 = 5 3 % 100 / 86, 6 % 104 / 104, 10 % 108 / 118; 10^6, K = 128, s0 = 6 6 % 1330 / 1230.
template <int P>
constexpr int kHomeFew = P > 64 ? 16 : 8;
template <int P>
constexpr int kWeakFew = P > 64 ? 16 : 4;
constexpr int kWeakEvery = 4, kSameCounts = 8;
constexpr int guess_weak(int K) { return K < 96 ? (K - 16) / 4 : 20; }

// What a workgroup screens in full: everything; the home blocks of its signals; the block of the largest bound.
enum Choice { kFull, kHome, kGuess };

template <int P, int S, int SX, int ARITH, bool SHARED, int W, Choice CHOICE>
__global__ __launch_bounds__(64 * W, 2) void energy_screen_kernel(ScrArgs g) {
    using G = ScrGeom<P>;
    constexpr bool HOME = CHOICE == kHome, GUESS = CHOICE == kGuess;
    constexpr int KS16 = G::KS16, MTS = G::MTS, NB = G::NB, SPB = G::SPB, NV = G::NV, STAGE_U = G::STAGE_U;
    constexpr bool WIDE = G::WIDE, BOUND = scr_bound(P, SX, SHARED);
    constexpr bool YLDS = SHARED && P >= 64;               // B operands from LDS (registers: 32 less at p = 64)
    constexpr int SIG = SHARED ? 64 : 64 * W;      // signals of the workgroup
    constexpr int NT = 2;                                   // 32-signal tiles of a wavefront
    const int K = g.K, m = g.m;

    extern __shared__ u32x4 lds_scr[];
    unsigned char* front = reinterpret_cast<unsigned char*>(lds_scr);
    unsigned short* E16 = reinterpret_cast<unsigned short*>(front + scr_front_bytes<P, SHARED, W>());
    unsigned* thr = reinterpret_cast<unsigned*>(front + scr_table_bytes<P, SHARED, W>(K));
    float* y2s = reinterpret_cast<float*>(thr + SIG);
    float* r2s = y2s + SIG;
    unsigned long long* key = reinterpret_cast<unsigned long long*>(r2s + SIG);
    float* wred = reinterpret_cast<float*>(key + SIG);     // [2][W], then a flag and a count
    int* any_flag = reinterpret_cast<int*>(wred + 2 * W);
    int* n_tasks = any_flag + 1;
    int* n_weak = n_tasks + 1;                 // HOME: weak signals, then blocks left in
    int* ids = reinterpret_cast<int*>(thr);    // HOME, until the decision: the signals themselves

    const int tid = threadIdx.x, NTH = blockDim.x, NW = NTH >> 6;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, n = lane & 31;
    const int64_t wg0 = (int64_t)blockIdx.x * SIG;         // first signal of the workgroup
    const int loc0 = SHARED ? 0 : wave * 64;               // first signal of the wavefront, in the workgroup

    // HOME: whether the dictionary represents the signals well enough (what the coding of the last iteration left in
    // weak, three counts in turn) and all its blocks are orthobases; the signals are then those at positions wg0 .. of perm.
    bool by_home = false, guess = false;
    int id_own = 0, home_lo = 0, home_hi = 0;  // own signal; the home blocks of the workgroup
    // GUESS: on their way, how far the blocks are from orthobases and which signals of the sample they represent
    constexpr int DEVS = GUESS ? (kGuessMaxK + 63) / 64 : 1, WORDS = kSample / 32, MASKS = GUESS ? 8 : 1;
    unsigned dev[DEVS][2];
    unsigned seen[MASKS];                      // words lane % WORDS, of the last block once more past the end
    auto sample_word = [&](int w) { return g.sample[min(w + lane, (K - 1) * WORDS + lane % WORDS)]; };
    if constexpr (GUESS) {
#pragma unroll
        for (int e = 0; e < DEVS; ++e) {
            const float2 d = g.dev[min(lane + 64 * e, K - 1)];
            dev[e][0] = __builtin_bit_cast(unsigned, d.x);
            dev[e][1] = __builtin_bit_cast(unsigned, d.y);
        }
#pragma unroll
        for (int e = 0; e < MASKS; ++e) seen[e] = sample_word(64 * e);
    }
    if constexpr (HOME) {
        by_home = g.weak[(g.turn + 2) % 3] * kHomeFew<P> <= (int)((gridDim.x + kWeakEvery - 1) / kWeakEvery) * 64;
        int lo = 0, hi = 0, other = 0;
        const int last = (int)min(wg0 + SIG, (int64_t)m) - 1;
        for (int j0 = 0; j0 < K; j0 += 64) {
            const int jj = j0 + lane;
            const int end = jj < K ? g.offsets[jj + 1] : 0x7fffffff, sw = jj < K ? g.sweeps[jj] : -1;
            lo += __popcll(__ballot(end <= (int)wg0));
            hi += __popcll(__ballot(end <= last));
            other += __popcll(__ballot(sw >= 0));
        }
        by_home = by_home && other == 0;
        home_lo = min(lo, K - 1);
        home_hi = min(hi, K - 1);
        const int64_t pos = wg0 + loc0 + lane;
        id_own = pos < m ? (by_home ? g.perm[pos] : (int)pos) : -1;
        // (kept there: the loops have no register for it, and a register spilled makes the first launch wait 0.1 ms for scratch memory)
        ids[loc0 + lane] = id_own;
    }

    // the dictionary's norms (most of the time one entry per thread; consumed below)
    const int n_norm = K * (P / 16);
    float2 norm = tid < n_norm ? g.dnorm[tid] : float2{0.f, 0.f};

    // Stages of the dictionary (!SHARED: all wavefronts read the same one); the first two are requested
    // before the signals.
    constexpr int FPT = (STAGE_U + 64 * W - 1) / (64 * W);
    const int n_stage = WIDE ? K * SPB : (K + NB - 1) / NB;
    u32x4(*Qs)[STAGE_U] = reinterpret_cast<u32x4(*)[STAGE_U]>(lds_scr);
    u32x4 pre[FPT];
    const __amdgpu_buffer_rsrc_t dict =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4*>(g.Dh), 0, n_stage * (2 * STAGE_U) * 16, 0x00027000);
    auto fetch = [&](u32x4 (&p)[FPT], int s) { // past the end: the last stage once more, not used
        s = min(s, n_stage - 1);
#pragma unroll
        for (int r = 0; r < FPT; ++r) {
            const int u = min(tid + 64 * W * r, STAGE_U - 1);
            p[r] = __builtin_amdgcn_raw_buffer_load_b128(dict, ((u >> 6) * 128 + (u & 63)) * 16, s * (2 * STAGE_U * 16), 0);
        }
    };
    auto stash = [&](const u32x4 (&p)[FPT], int buf) {
#pragma unroll
        for (int r = 0; r < FPT; ++r) Qs[buf][min(tid + 64 * W * r, STAGE_U - 1)] = p[r];
    };
    if constexpr (!SHARED) fetch(pre, HOME && by_home ? home_lo * SPB : 0);

    // The leading fp16 parts of the signals, every signal scaled by a power of two (largest magnitude
    // into [1/2, 1), p = 256: [1/4, 1/2), so that coefficients times the dictionary's 2^13 stay inside
    // fp16).  PARTS consecutive lanes share a signal, so that a load instruction reads whole cache
    // lines; GS signals at a time.  y2s / r2s: |y|^2 and |y - hi|^2 of the scaled signal; -1 in y2s: the
    // signal does not fit (infinite, or below 2^-63).
    constexpr int PARTS = P / 4 < 8 ? P / 4 : 8, GS = 64 / PARTS, L4 = P / 4 / PARTS;
    const int part = lane % PARTS, sub = lane / PARTS;
    auto load_group = [&](int first, f32x4 (&raw)[L4]) {   // first: in the workgroup
        const int64_t i = HOME ? (int64_t)__shfl(id_own, first - loc0 + sub, 64) : wg0 + first + sub;
#pragma unroll
        for (int e = 0; e < L4; ++e) {
            raw[e] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (HOME ? i >= 0 : i < m) raw[e] = *reinterpret_cast<const f32x4*>(g.Y + i * P + (e * PARTS + part) * 4);
        }
    };
    auto over_parts = [&](float x, auto f) {               // over the PARTS lanes of a signal
        x = f(x, dpp_f<kDppXor1>(x));
        x = f(x, dpp_f<kDppXor2>(x));
        if constexpr (PARTS == 8) x = f(x, dpp_f<kDppHalfMirror>(x));
        return x;
    };
    // dest: operand order of a tile of NN signals: ((ks*2 + hh)*NN + signal)*16 bytes, dims ks*16 + hh*8 ..
    auto convert_group = [&](int first, const f32x4 (&raw)[L4], unsigned char* dest, int NN, int at) {
        float vmax = 0.f;
#pragma unroll
        for (int e = 0; e < L4; ++e)
            vmax = fmaxf(fmaxf(fmaxf(vmax, fabsf(raw[e].x)), fmaxf(fabsf(raw[e].y), fabsf(raw[e].z))), fabsf(raw[e].w));
        vmax = over_parts(vmax, [](float a, float b) { return fmaxf(a, b); });
        const unsigned ex = (__builtin_bit_cast(unsigned, vmax) >> 23) & 0xffu;
        const bool fits = ex >= 64u && ex <= 240u;
        const float scale = fits ? __builtin_bit_cast(float, ((WIDE ? 252u : 253u) - ex) << 23) : 0.f;
        float y2 = 0.f, r2 = 0.f;
#pragma unroll
        for (int e = 0; e < L4; ++e) {
            typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
            const f32x4 v = raw[e] * scale;
            const unsigned p0 = pack_f16(v.x, v.y), p1 = pack_f16(v.z, v.w);
            const f16x2 h0 = __builtin_bit_cast(f16x2, p0), h1 = __builtin_bit_cast(f16x2, p1);
            const float d0 = v.x - (float)h0[0], d1 = v.y - (float)h0[1], d2 = v.z - (float)h1[0], d3 = v.w - (float)h1[1];
            y2 = fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, fmaf(v.w, v.w, y2))));
            r2 = fmaf(d0, d0, fmaf(d1, d1, fmaf(d2, d2, fmaf(d3, d3, r2))));
            const int d4 = e * PARTS + part;               // (ks, hh, half) = bits of d4
            *reinterpret_cast<u32x2*>(dest + ((d4 >> 1) * NN + at + sub) * 16 + (d4 & 1) * 8) = u32x2{p0, p1};
        }
        y2 = over_parts(y2, [](float a, float b) { return a + b; });
        r2 = over_parts(r2, [](float a, float b) { return a + b; });
        if (part == 0) {
            y2s[first + sub] = fits || vmax == 0.f ? y2 : -1.f;
            r2s[first + sub] = r2;
        }
    };
    auto wave_fence = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // B operand: dims ks*16 + h*8 .. +7 of this lane's signal in tile nt
    u32x4 yq[YLDS ? 1 : NT][YLDS ? 1 : KS16];
    if constexpr (SHARED) {
        for (int q = wave; q < 64 / GS; q += NW) {
            f32x4 raw[L4];
            load_group(q * GS, raw);
            convert_group(q * GS, raw, front + (q * GS / 32) * (32 * P * 2), 32, q * GS & 31);
        }
    } else if constexpr (!WIDE) {
        constexpr int NG = 32 / GS;                        // groups of a tile
        f32x4 raw[NT * NG][L4];
#pragma unroll
        for (int q = 0; q < NT * NG; ++q) load_group(loc0 + q * GS, raw[q]);
        unsigned char* mine = front + wave * 4096;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
            for (int q = 0; q < NG; ++q) convert_group(loc0 + (nt * NG + q) * GS, raw[nt * NG + q], mine, 32, q * GS);
            wave_fence();
#pragma unroll
            for (int ks = 0; ks < KS16; ++ks) yq[nt][ks] = *reinterpret_cast<const u32x4*>(mine + (ks * 64 + lane) * 16);
            wave_fence();
        }
    } else {
        static_assert(!WIDE || GS == 8, "eight signals of 512 bytes at a time");
        unsigned char* mine = front + wave * 4096;
        f32x4 raw[2][L4];
        load_group(loc0, raw[0]);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (q + 1 < 8) load_group(loc0 + (q + 1) * GS, raw[(q + 1) & 1]);
            convert_group(loc0 + q * GS, raw[q & 1], mine, GS, 0);
            wave_fence();
            if ((n >> 3) == (q & 3)) {
#pragma unroll
                for (int ks = 0; ks < KS16; ++ks)
                    yq[q >> 2][ks] = *reinterpret_cast<const u32x4*>(mine + ((ks * 2 + h) * GS + (n & 7)) * 16);
            }
            wave_fence();
        }
    }
    for (int e = tid + NTH; e < n_norm; e += NTH) {
        const float2 v = g.dnorm[e];
        norm.x = fmaxf(norm.x, v.x);
        norm.y = fmaxf(norm.y, v.y);
    }
    norm.x = wave_max(norm.x);
    norm.y = wave_max(norm.y);
    if (tid == 0) {
        any_flag[0] = any_flag[1] = 0;
        if constexpr (!SHARED) n_weak[0] = n_weak[1] = 0;
    }
    if (lane == 0) {
        wred[wave] = norm.x;
        wred[W + wave] = norm.y;
    }
    __syncthreads();
    // Lane (h, n) is the owner of signal (tile h, n) = loc0 + lane.  Energies are stored relative to |y|^2.
    const float y2_own = y2s[loc0 + lane];
    const float e_scale = y2_own > 0.f ? 0x1p-26f / y2_own : 0.f;
    if constexpr (SHARED && !YLDS) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int ks = 0; ks < KS16; ++ks)
                yq[nt][ks] = *reinterpret_cast<const u32x4*>(front + nt * (32 * P * 2) + (ks * 64 + lane) * 16);
    }

    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    constexpr int UT = SHARED ? (P == 64 ? 2 : 1) : MTS;   // 32-row tiles of a step
    constexpr int UB = WIDE ? 1 : UT * 32 / P;             // blocks of a step
    const int per_row = ((WIDE ? K : (K + UB - 1) / UB) + g.rows - 1) / g.rows;         // SHARED: units of a row of workgroups
    using Acc = f32x16[NT][UT];
    u16x2 run[SX];                             // p = 256: the pair's sorted top of the block so far
    // of the own signal, in stored units (BOUND: bounds from above)
    float bestE = -1.f, secondE = -1.f;
    int best = 0;
    auto offer = [&](float e, int j) {
        const bool better = e > bestE;
        secondE = fmaxf(secondE, fminf(bestE, e));
        best = better ? j : best;
        bestE = fmaxf(bestE, e);
        const auto q = __builtin_amdgcn_cvt_pknorm_u16(e, 0.f);
        E16[j * SIG + loc0 + lane] = (unsigned short)q[0];
        return better;
    };
    auto finish = [&](const u16x2 (&a)[SX], int j) { offer(pk_pair_energy<SX>(a, h != 0) * e_scale, j); };
    // BOUND.  keep: the best block's magnitudes (two of a signal per word); tau: sqrt(t), twice; slope:
    // (p - s0) t
    constexpr int NK = BOUND ? NV / 2 : 1;
    u16x2 keep[NT][NK], tau[NT];
    float slope[NT];
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    auto magnitudes = [&](const Acc& acc, int b, int nt, u16x2 (&x)[NK]) {
#pragma unroll
        for (int v = 0; v < NK; ++v) {
            const int f = b * NV + 2 * v;
            const auto p = __builtin_amdgcn_cvt_pkrtz(fabsf(acc[nt][(f >> 4) % UT][f & 15]), fabsf(acc[nt][(f >> 4) % UT][(f + 1) & 15]));
            x[v] = __builtin_bit_cast(u16x2, p);
        }
    };
    auto sorted_top = [&](const u16x2 (&x)[NT][NK], u16x2 (&a)[SX]) {          // of both signals, packed
        u16x2 t[2 * NK];
#pragma unroll
        for (int v = 0; v < NK; ++v) {
            const unsigned x0 = __builtin_bit_cast(unsigned, x[0][v]), x1 = __builtin_bit_cast(unsigned, x[1][v]);
            t[2 * v] = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(x1, x0, 0x05040100u));
            t[2 * v + 1] = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(x1, x0, 0x07060302u));
        }
        pk_top_sorted<2 * NK, SX>(t, a);
    };
    if constexpr (BOUND) {
        // two-sided normal tail of SX / P (a fit): where a block that has nothing to do with the signal has its
        // SX-th largest coefficient
        const float tail = __builtin_logf((float)P / SX), q2 = tail * (0.859f + 0.1314f * tail);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const float y2 = y2s[loc0 + nt * 32 + n];
            const _Float16 t16 = (_Float16)(8192.f * __builtin_amdgcn_sqrtf(fmaxf(y2, 0.f) * (q2 / P)));
            const float t = (float)t16;
            tau[nt] = __builtin_bit_cast(u16x2, f16x2{t16, t16});
            slope[nt] = (float)(P - SX) * 0.5f * (t * t);                  // (each lane of a pair takes half)
#pragma unroll
            for (int v = 0; v < NK; ++v) keep[nt][v] = u16x2{0, 0};
        }
    }
    // selection from acc, p <= 64: the UB blocks from j0 on; p = 256: 32 atoms of a block (first: of them all).  In full: by
    // networks also where bounds would do.
    auto select_as = [&](const Acc& acc, int j0, bool first, auto in_full) {
        if constexpr (BOUND && !decltype(in_full)::value) {
#pragma unroll
            for (int b = 0; b < UB; ++b) {
                u16x2 x[NT][NK];
                float up[NT][2];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    magnitudes(acc, b, nt, x[nt]);
                    up[nt][0] = -slope[nt];
                    up[nt][1] = 0.f;
                }
#pragma unroll
                for (int v = 0; v < NK; v += 2) {          // four sums, so that no instruction waits for the one before
                    f16x2 w[NT][2];
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) w[nt][k] = __builtin_bit_cast(f16x2, pk_max(x[nt][v + k], tau[nt]));
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) up[nt][k] = __builtin_amdgcn_fdot2(w[nt][k], w[nt][k], up[nt][k], false);
                }
                const SwapPair t = swap32(up[0][0] + up[0][1], up[1][0] + up[1][1]);
                const unsigned long long better = __ballot(offer((t.first + t.second) * e_scale, j0 + b));
                const unsigned long long lo = better & 0xffffffffull, hi = better >> 32;
                const bool b0 = __builtin_amdgcn_inverse_ballot_w64(lo | lo << 32), b1 = __builtin_amdgcn_inverse_ballot_w64(hi | hi << 32);
#pragma unroll
                for (int v = 0; v < NK; ++v) {
                    keep[0][v] = b0 ? x[0][v] : keep[0][v];
                    keep[1][v] = b1 ? x[1][v] : keep[1][v];
                }
            }
        } else {
#pragma unroll
            for (int b = 0; b < UB; ++b) {
                u16x2 x[NV], a[SX];
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int f = b * NV + v;
                    const auto p = __builtin_amdgcn_cvt_pkrtz(fabsf(acc[0][(f >> 4) % UT][f & 15]), fabsf(acc[1][(f >> 4) % UT][f & 15]));
                    x[v] = __builtin_bit_cast(u16x2, p);
                }
                pk_top_sorted<NV, SX>(x, a);
                if constexpr (!WIDE) {
                    finish(a, j0 + b);
                } else {
                    // (zeros below everything: the first list of a block is taken as it is)
                    const unsigned keep_run = first ? 0u : 0xffffffffu;
#pragma unroll
                    for (int t = 0; t < SX; ++t) run[t] = __builtin_bit_cast(u16x2, __builtin_bit_cast(unsigned, run[t]) & keep_run);
                    pk_merge_top<SX>(run, a);
                }
            }
        }
    };
    auto select = [&](const Acc& acc, int j0, bool first) { select_as(acc, j0, first, std::false_type{}); };
    auto multiply = [&](Acc& acc, u32x4 a, int ks, int mt) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            u32x4 b;
            if constexpr (YLDS) b = *reinterpret_cast<const u32x4*>(front + nt * (32 * P * 2) + (ks * 64 + lane) * 16);
            else b = yq[nt][ks];
            acc[nt][mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b),
                                                                 ks == 0 ? zero : acc[nt][mt], 0, 0, 0);
        }
    };
    // norms of the dictionary's rows, largest: whole, and of what the leading parts leave
    auto norms = [&]() {
        float2 v = {wred[0], wred[W]};
        for (int w = 1; w < NW; ++w) v = {fmaxf(v.x, wred[w]), fmaxf(v.y, wred[W + w])};
        return v;
    };
    auto stored = [](float e) { return (unsigned)(unsigned short)__builtin_amdgcn_cvt_pknorm_u16(e, 0.f)[0]; };
    const bool valid = wg0 + loc0 + lane < m;
    // The error of a coefficient, relative to |y|.
    auto coef_error = [&](float2 nrm) {
        const float rel = y2_own > 0.f ? r2s[loc0 + lane] / y2_own : 0.f;
        return (nrm.x * sqrtf(rel) + 1.001f * nrm.y + nrm.x * (P * 1.2e-7f)) * 1.001f;
    };
    // What a block has to reach, in stored energies, beside one that keeps `below`; 0: every block stays in, 0x10000: none
    // does (a zero signal).  units: of rounding.
    auto threshold = [&](float below, float2 nrm, float units) {
        unsigned t16 = 0u;
        const float eps = sqrtf((float)g.s0) * coef_error(nrm);
        const float qb = (float)stored(below);
        const float kept = sqrtf(fmaxf(qb - 0.5f, 0.f) * (1.f / 65535.f));
        const float t = (kept - 2.f * eps) * (1.f - 0x1.02p-10f);
        const float t2 = t > 0.f ? t * t * (65535.f * (1.f - 1e-5f)) - units : 0.f;
        if (y2_own > 0.f && t2 > 0.f) t16 = (unsigned)t2;
        return !valid || y2_own == 0.f ? 0x10000u : t16;
    };
    constexpr unsigned kWeakBelow = (unsigned)(65535.f * (home_line<P>(SX) < 1.f ? home_line<P>(SX) : 1.f));
    // Few enough signals whose best block has to be reached by others below the line; every wavefront, with a barrier.
    auto few_weak = [&](unsigned t16) {
        const int weak = __popcll(__ballot(t16 < kWeakBelow));
        if (lane == 0 && weak != 0) atomicAdd(n_weak, weak);
        __syncthreads();
        return *n_weak * kWeakFew<P> <= SIG;
    };
    bool halves = false;                       // HOME: only the home blocks have been screened in full
    unsigned t_home = 0u;
    constexpr int kMatrix = NT * UT * KS16;
    constexpr int kVector = UB * (BOUND ? NV * 4 + 16 : NV * 7 + 8 * SX);      // about

    Acc acc0, acc1;
    if constexpr (WIDE) {
#pragma unroll
        for (int t = 0; t < SX; ++t) run[t] = u16x2{0, 0};
    }
    if constexpr (!SHARED) {
        // while stage s is selected from the accumulators, stage s + 1 is multiplied from one buffer and
        // stage s + 2 written to the other (requested a stage earlier, it makes no difference)
        auto project = [&](Acc& acc, int buf) {
#pragma unroll
            for (int ks = 0; ks < KS16; ++ks)
#pragma unroll
                for (int mt = 0; mt < MTS; ++mt) multiply(acc, Qs[buf][(mt * KS16 + ks) * 64 + lane], ks, mt);
        };
        auto step = [&](Acc& now, Acc& next, int s) {
            fetch(pre, s + 2);
            project(next, (s + 1) & 1);
            select(now, s * NB, s % SPB == 0);
            stash(pre, s & 1);
            interleave<kMatrix, kVector>();
            if (WIDE && s % SPB == SPB - 1) finish(run, s / SPB);      // uniform
            __syncthreads();
        };
        if constexpr (HOME || GUESS) {
            const float2 nrm = norms();
            // the leading parts of a signal, scaled (as convert_group), as a B operand
            auto leading_parts = [](const ExactRow<P, 3>& y, u32x4 (&b)[KS16]) {
                float vmax = 0.f;
#pragma unroll
                for (int e = 0; e < P / 8; ++e)
                    vmax = fmaxf(fmaxf(fmaxf(vmax, fabsf(y.v[e].x)), fmaxf(fabsf(y.v[e].y), fabsf(y.v[e].z))), fabsf(y.v[e].w));
                vmax = fmaxf(vmax, other_half(vmax));
                const unsigned ex = (__builtin_bit_cast(unsigned, vmax) >> 23) & 0xffu;
                const float scale = ex >= 64u && ex <= 240u ? __builtin_bit_cast(float, (253u - ex) << 23) : 0.f;
#pragma unroll
                for (int ks = 0; ks < KS16; ++ks) {
                    const f32x4 v0 = y.v[2 * ks] * scale, v1 = y.v[2 * ks + 1] * scale;
                    b[ks] = u32x4{pack_f16(v0.x, v0.y), pack_f16(v0.z, v0.w), pack_f16(v1.x, v1.y), pack_f16(v1.z, v1.w)};
                }
            };
            if (HOME && by_home) {             // uniform
                // the home blocks, those of its own signals by every wavefront
                int lo = 0, hi = 0;
                const int first = (int)wg0 + loc0, last = min(first + 63, m - 1);
                for (int j0 = 0; j0 < K; j0 += 64) {
                    const int end = j0 + lane < K ? g.offsets[j0 + lane + 1] : 0x7fffffff;
                    lo += __popcll(__ballot(end <= first));
                    hi += __popcll(__ballot(end <= last));
                }
                const int n_home = (home_hi - home_lo + 1) * SPB;
                stash(pre, 0);
                for (int s = 0; s < n_home; ++s) {
                    const int j = home_lo + s / SPB;
                    fetch(pre, home_lo * SPB + min(s + 1, n_home - 1));
                    __syncthreads();
                    if (j >= lo && j <= hi) {  // uniform over the wavefront
                        project(acc0, s & 1);
                        select_as(acc0, j, s % SPB == 0, std::true_type{});
                        if (WIDE && s % SPB == SPB - 1) finish(run, j);
                    }
                    stash(pre, (s + 1) & 1);
                }
                t_home = threshold(bestE, nrm, 1.f);
                halves = few_weak(t_home);
            }
            if constexpr (GUESS) {
                unsigned mask = 0u;
#pragma unroll
                for (int e = 0; e < MASKS; ++e) mask |= seen[e];
                for (int w = 64 * MASKS; w < K * WORDS; w += 64 * MASKS) {     // uniform
#pragma unroll
                    for (int e = 0; e < MASKS; ++e) seen[e] = sample_word(w + 64 * e);
#pragma unroll
                    for (int e = 0; e < MASKS; ++e) mask |= seen[e];
                }
#pragma unroll
                for (int o = WORDS; o < 64; o <<= 1) mask |= (unsigned)__shfl_xor((int)mask, o, 64);
                int weak = 32 - __popc(mask);
#pragma unroll
                for (int o = 1; o < WORDS; o <<= 1) weak += __shfl_xor(weak, o, 64);
                constexpr unsigned line = __builtin_bit_cast(unsigned, kOrthobase * kOrthobase * 0.5f);       // of half of a block
                bool close = true;
#pragma unroll
                for (int e = 0; e < DEVS; ++e) close = close && max(dev[e][0], dev[e][1]) <= line;         // (bits: a NaN is above it)
                halves = guess = __ballot(!close) == 0ull && __builtin_amdgcn_readfirstlane(weak) <= guess_weak(K);
            }
            // Bounds from home_rows atoms for all: a step takes the first 32 atoms of two blocks, or (p = 256) half of the
            // atoms of one.  GUESS: without home blocks, the block of the largest bound is kept instead.
            if (halves) {                      // uniform
                u16x2 top[NT];             // sqrt(t), twice
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const _Float16 t = (_Float16)(8192.f * __builtin_amdgcn_sqrtf(fmaxf(y2s[loc0 + nt * 32 + n], 0.f) * (kHomeT / P)));
                    top[nt] = __builtin_bit_cast(u16x2, f16x2{t, t});
                }
                const float t_own = (float)(_Float16)(8192.f * __builtin_amdgcn_sqrtf(fmaxf(y2_own, 0.f) * (kHomeT / P)));
                // Orthobases to 1e-4, sums to a few 2^-24; and |a - b| <= d gives a^2 >= b^2 - 2 d b for the root of the sum, b <= |y|.
                constexpr float root = P > 64 ? 8.f : 5.657f;                        // of home_rows
                const float most = 1.0003f + (float)g.s0 * (t_own * t_own) * e_scale + 2.f * root * coef_error(nrm);
                const int n_step = WIDE ? 2 * K : (K + 1) / 2;
                auto fetch_home = [&](u32x4 (&q)[FPT], int s) {
                    s = min(s, n_step - 1);
                    if constexpr (WIDE) {
                        fetch(q, (s >> 1) * SPB + (s & 1));
                    } else {
#pragma unroll
                        for (int r = 0; r < FPT; ++r) {
                            const int u = min(tid + 64 * W * r, STAGE_U - 1), v = u & (STAGE_U / 2 - 1);
                            const int j = min(2 * s + u / (STAGE_U / 2), K - 1);
                            q[r] = __builtin_amdgcn_raw_buffer_load_b128(dict, (j * (2 * STAGE_U) + (v >> 6) * 128 + (v & 63)) * 16, 0, 0);
                        }
                    }
                };
                int n_left = 0;            // blocks that the bounds leave in, besides the best one, of the own signal (weak, p = 64: below)
                int last_block = -1;
                auto leave = [&](float sum, int j) {
                    const float e = most - sum * e_scale;
                    if constexpr (GUESS) {
                        const bool again = j == last_block;  // (the block past the end of an odd number of them)
                        last_block = j;
                        const float v = again ? -1.f : e;
                        secondE = fmaxf(secondE, fminf(bestE, v));
                        best = v > bestE ? j : best;
                        bestE = fmaxf(bestE, v);
                        E16[j * SIG + loc0 + lane] = (unsigned short)stored(e);
                        return;
                    }
                    const bool other = j != best;
                    secondE = fmaxf(secondE, other ? e : -1.f);
                    const unsigned q = stored(e);
                    E16[j * SIG + loc0 + lane] = (unsigned short)q;
                    n_left += other && q >= t_home;
                };
                float part_sum[NT] = {0.f, 0.f};
                auto bound = [&](const Acc& acc, int s, auto second_half) {
#pragma unroll
                    for (int b = 0; b < UT; ++b) {
                        float up[NT][2] = {{0.f, 0.f}, {0.f, 0.f}};
#pragma unroll
                        for (int v = 0; v < 16; v += 4) {
                            f16x2 w[NT][2];
#pragma unroll
                            for (int k = 0; k < 2; ++k)
#pragma unroll
                                for (int nt = 0; nt < NT; ++nt) {
                                    const auto x = __builtin_amdgcn_cvt_pkrtz(fabsf(acc[nt][b][v + 2 * k]), fabsf(acc[nt][b][v + 2 * k + 1]));
                                    w[nt][k] = __builtin_bit_cast(f16x2, __builtin_elementwise_min(__builtin_bit_cast(u16x2, x), top[nt]));
                                }
#pragma unroll
                            for (int k = 0; k < 2; ++k)
#pragma unroll
                                for (int nt = 0; nt < NT; ++nt) up[nt][k] = __builtin_amdgcn_fdot2(w[nt][k], w[nt][k], up[nt][k], false);
                        }
                        float sum[NT];
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) sum[nt] = up[nt][0] + up[nt][1];
                        if constexpr (WIDE && !decltype(second_half)::value) {
#pragma unroll
                            for (int nt = 0; nt < NT; ++nt) part_sum[nt] = sum[nt];
                        } else if constexpr (WIDE) {
                            const SwapPair t = swap32(part_sum[0] + sum[0], part_sum[1] + sum[1]);
                            leave(t.first + t.second, s >> 1);
                        } else {
                            const SwapPair t = swap32(sum[0], sum[1]);
                            leave(t.first + t.second, min(2 * s + b, K - 1));
                        }
                    }
                };
                auto home_step = [&](Acc& now, Acc& next, int s, auto second_half) {
                    stash(pre, s & 1);     // stage s + 2, requested a step ago (two steps ago: no better)
                    fetch_home(pre, s + 3);
                    project(next, (s + 1) & 1);
                    bound(now, s, second_half);
                    interleave<kMatrix, UT * 60>();
                    __syncthreads();
                };
                {
                    u32x4 pre0[FPT], pre1[FPT];            // (three trips at once)
                    fetch_home(pre0, 0);
                    fetch_home(pre1, 1);
                    fetch_home(pre, 2);
                    stash(pre0, 0);
                    stash(pre1, 1);
                }
                __syncthreads();
                project(acc0, 0);
                __syncthreads();
                for (int s = 0; s < n_step && halves; s += 2) {
                    home_step(acc0, acc1, s, std::false_type{});
                    if (s + 1 < n_step) home_step(acc1, acc0, s + 1, std::true_type{});         // uniform
                    if (!GUESS && (s & 14) == 14) {        // too many to be resolved one by one: all over again, in full
                        if (n_left != 0 && (WIDE || t_home >= kWeakBelow)) atomicAdd(&n_weak[1], n_left);
                        n_left = 0;
                        __syncthreads();
                        halves = n_weak[1] <= 2 * SIG;
                        __syncthreads();
                    }
                }
            }
            // p = 64: the weak signals, whom such bounds leave with most blocks, are screened in all of them: listed, in tiles of 32, two blocks
            // at a time by every wavefront (a tile of one signal is as much work as one of 32).
            auto screen_weak = [&]() {
                const bool wanted = t_home < kWeakBelow;
                unsigned short* list = reinterpret_cast<unsigned short*>(front);
                const unsigned long long mask = __ballot(wanted);
                __syncthreads();               // the stages are dead
                int at = 0;
                if (lane == 0 && mask != 0ull) at = atomicAdd(n_tasks, __popcll(mask));
                at = __builtin_amdgcn_readfirstlane(at);
                if (wanted) list[at + __popcll(mask & ((1ull << lane) - 1ull))] = (unsigned short)(loc0 + lane);
                __syncthreads();
                const int n_list = *n_tasks, n_pair = (K + 1) / 2;
                u32x4 rows[2][UT][KS16];
                auto look_up = [&](int pair) {
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const u32x4* D = g.Dh + (int64_t)min(2 * pair + k, K - 1) * UT * (KS16 * 128) + lane;
#pragma unroll
                        for (int mt = 0; mt < UT; ++mt)
#pragma unroll
                            for (int ks = 0; ks < KS16; ++ks) rows[k][mt][ks] = D[(mt * KS16 + ks) * 128];
                    }
                };
                for (int t0 = 0; t0 < n_list; t0 += 32) {          // uniform
                    const int id = t0 + n < n_list ? (int)list[t0 + n] : -1;
                    ExactRow<P, 3> y;
                    y.load(g, id < 0 ? (int64_t)-1 : HOME ? (int64_t)ids[id] : wg0 + id, h);
                    if (wave < n_pair) look_up(wave);
                    u32x4 yb[KS16];
                    leading_parts(y, yb);
                    const float to_stored = id < 0 ? 0.f : 0x1p-26f / y2s[id];
                    for (int pair = wave; pair < n_pair; pair += NW) {
#pragma unroll
                        for (int k = 0; k < 2; ++k)
#pragma unroll
                            for (int ks = 0; ks < KS16; ++ks)
#pragma unroll
                                for (int mt = 0; mt < UT; ++mt)
                                    acc0[k][mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                                        __builtin_bit_cast(f16x8, rows[k][mt][ks]), __builtin_bit_cast(f16x8, yb[ks]),
                                        ks == 0 ? zero : acc0[k][mt], 0, 0, 0);
                        u16x2 x[NV], a[SX];
#pragma unroll
                        for (int v = 0; v < NV; ++v) {
                            const auto q = __builtin_amdgcn_cvt_pkrtz(fabsf(acc0[0][v >> 4][v & 15]), fabsf(acc0[1][v >> 4][v & 15]));
                            x[v] = __builtin_bit_cast(u16x2, q);
                        }
                        look_up(min(pair + NW, n_pair - 1));
                        pk_top_sorted<NV, SX>(x, a);
                        const float e = pk_pair_energy<SX>(a, h != 0);
                        if (id >= 0) E16[min(2 * pair + h, K - 1) * SIG + id] = (unsigned short)stored(e * to_stored);
                    }
                }
                __syncthreads();
                if (tid == 0) *n_tasks = 0;
                if (mask != 0ull) {            // uniform over the wavefront
                    unsigned q0 = 0, q1 = 0;
                    int j0 = 0;
                    for (int j = 0; j < K; ++j) {
                        const unsigned q = E16[j * SIG + loc0 + lane];
                        q1 = max(q1, min(q0, q));
                        j0 = q > q0 ? j : j0;
                        q0 = max(q0, q);
                    }
                    const unsigned t16 = threshold((float)q0 * (1.f / 65535.f), nrm, 1.f);
                    if (wanted) {
                        best = j0;
                        secondE = (float)q1 * (1.f / 65535.f);
                        t_home = t16;
                    }
                }
            };
            if constexpr (GUESS) {
                // The kept energy of the signals in the blocks of their largest bounds, as far as the leading parts give it (a zero
                // signal: -1): the signals listed by block, in tiles of 32.
                auto guessed_energy = [&]() {
                    const bool wanted = y2_own > 0.f;
                    int* first = reinterpret_cast<int*>(front);                        // [K] signals of a block, then its first tile
                    unsigned short* tile_block = reinterpret_cast<unsigned short*>(first + K);         // [most]
                    const int most = K + SIG / 32;         // tiles
                    unsigned short* list = tile_block + ((most + 7) & ~7);             // [most][32]
                    __syncthreads();                       // the stages are dead
                    for (int j = tid; j < K; j += NTH) first[j] = 0;
                    for (int e = tid; e < most * 16; e += NTH) reinterpret_cast<unsigned*>(list)[e] = 0xffffffffu;
                    __syncthreads();
                    int slot = 0;
                    if (wanted) slot = atomicAdd(&first[best], 1);
                    __syncthreads();
                    if (wave == 0) {
                        int tiles = 0;
                        for (int j0 = 0; j0 < K; j0 += 64) {
                            const int j = j0 + lane, nt = j < K ? (first[j] + 31) >> 5 : 0, upto = tiles + wave_scan(nt);
                            for (int t = 0; t < nt; ++t) tile_block[upto - nt + t] = (unsigned short)j;
                            if (j < K) first[j] = upto - nt;
                            tiles = __builtin_amdgcn_readlane(upto, 63);
                        }
                        if (lane == 0) *n_tasks = tiles;
                    }
                    __syncthreads();
                    if (wanted) list[first[best] * 32 + slot] = (unsigned short)(loc0 + lane);
                    thr[loc0 + lane] = __builtin_bit_cast(unsigned, -1.f);
                    __syncthreads();
                    const int tiles = *n_tasks;
                    // two tiles at a time, so that the networks sort two signals per lane as elsewhere; the operands of the next
                    // two are on their way meanwhile
                    int id[2] = {-1, -1}, j_of[2] = {0, 0};
                    ExactRow<P, 3> y[2];
                    u32x4 rows[2][UT][KS16];
                    auto look_up = [&](int t) {
#pragma unroll
                        for (int k = 0; k < 2; ++k) {
                            id[k] = -1;
                            if (t + k < tiles) {           // uniform
                                j_of[k] = __builtin_amdgcn_readfirstlane((int)tile_block[t + k]);
                                const int at = (int)list[(t + k) * 32 + n];
                                id[k] = at == 0xffff ? -1 : at;
                            }
                            y[k].load(g, id[k] < 0 ? (int64_t)-1 : wg0 + id[k], h);
                            const u32x4* D = g.Dh + (int64_t)j_of[k] * UT * (KS16 * 128) + lane;
#pragma unroll
                            for (int mt = 0; mt < UT; ++mt)
#pragma unroll
                                for (int ks = 0; ks < KS16; ++ks) rows[k][mt][ks] = D[(mt * KS16 + ks) * 128];
                        }
                    };
                    look_up(2 * wave);
                    for (int t = 2 * wave; t < tiles; t += 2 * NW) {
                        const int id_out = h == 0 ? id[0] : id[1];
#pragma unroll
                        for (int k = 0; k < 2; ++k) {
                            u32x4 yb[KS16];
                            leading_parts(y[k], yb);
#pragma unroll
                            for (int ks = 0; ks < KS16; ++ks) {
#pragma unroll
                                for (int mt = 0; mt < UT; ++mt)
                                    acc0[k][mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                                        __builtin_bit_cast(f16x8, rows[k][mt][ks]), __builtin_bit_cast(f16x8, yb[ks]),
                                        ks == 0 ? zero : acc0[k][mt], 0, 0, 0);
                            }
                        }
                        u16x2 x[NV], a[SX];
#pragma unroll
                        for (int v = 0; v < NV; ++v) {
                            const auto q = __builtin_amdgcn_cvt_pkrtz(fabsf(acc0[0][v >> 4][v & 15]), fabsf(acc0[1][v >> 4][v & 15]));
                            x[v] = __builtin_bit_cast(u16x2, q);
                        }
                        look_up(t + 2 * NW);
                        pk_top_sorted<NV, SX>(x, a);
                        const float e = pk_pair_energy<SX>(a, h != 0);
                        if (id_out >= 0) thr[id_out] = __builtin_bit_cast(unsigned, e * 0x1p-26f / y2s[id_out]);
                    }
                    __syncthreads();
                    const float below = __builtin_bit_cast(float, thr[loc0 + lane]);
                    if (tid == 0) *n_tasks = 0;
                    __syncthreads();
                    return below;
                };
                if (halves) {                  // uniform
                    const float e = guessed_energy();
                    if (y2_own > 0.f) E16[best * SIG + loc0 + lane] = (unsigned short)stored(e);
                    t_home = threshold(e, nrm, 1.f);
                    halves = few_weak(t_home);
                }
            }
            if constexpr (!WIDE)
                if (halves && *n_weak != 0) screen_weak();         // uniform
            if ((by_home || guess) && !halves) {               // uniform
                bestE = secondE = -1.f;
                best = 0;
                fetch(pre, 0);
                __syncthreads();
            }
        }
        if (!halves) {                         // uniform
            u32x4 pre1[FPT];
            fetch(pre1, 1);
            stash(pre, 0);
            stash(pre1, 1);
            __syncthreads();
            project(acc0, 0);
            __syncthreads();
            for (int s = 0; s < n_stage; s += 2) {
                step(acc0, acc1, s);
                if (s + 1 < n_stage) step(acc1, acc0, s + 1);          // uniform
            }
        }
    } else {
        // A step = UT row tiles of the dictionary, p = 256: one of the SPB tiles of a block; wavefront w takes
        // the blocks (p < 64: tiles) w, w + NW, .. and reads their rows from L2, one step ahead.
        const int unit0 = (int)blockIdx.y * per_row;
        const int n_unit = min((WIDE ? K : (K + UB - 1) / UB) - unit0, per_row);
        const int n_mine = wave < n_unit ? ((n_unit - 1 - wave) / NW + 1) * SPB : 0;
        auto tile_of = [&](int t) {            // past the end: the last one once more, not used
            t = min(t, n_mine - 1);
            return WIDE ? (unit0 + wave + (t / SPB) * NW) * SPB + t % SPB : (unit0 + wave + t * NW) * UT;
        };
        u32x4 rows[UT][KS16];
        auto load = [&](int t) {
            const u32x4* src = g.Dh + (int64_t)tile_of(t) * (KS16 * 128) + lane;
#pragma unroll
            for (int mt = 0; mt < UT; ++mt)
#pragma unroll
                for (int ks = 0; ks < KS16; ++ks) rows[mt][ks] = src[(mt * KS16 + ks) * 128];
        };
        auto project = [&](Acc& acc) {
#pragma unroll
            for (int ks = 0; ks < KS16; ++ks)
#pragma unroll
                for (int mt = 0; mt < UT; ++mt) multiply(acc, rows[mt][ks], ks, mt);
        };
        auto step = [&](Acc& now, Acc& next, int t) {
            project(next);
            load(t + 2);
            select(now, WIDE ? 0 : (unit0 + wave + t * NW) * UB, t % SPB == 0);
            interleave<kMatrix, kVector>();
            if (WIDE && t % SPB == SPB - 1) finish(run, unit0 + wave + (t / SPB) * NW);           // uniform
        };
        if (n_mine > 0) {                      // uniform over the wavefront
            load(0);
            project(acc0);
            load(1);
            for (int t = 0; t < n_mine; t += 2) {
                step(acc0, acc1, t);
                if (t + 1 < n_mine) step(acc1, acc0, t + 1);
            }
        }
    }

    // Decision: the best block alone at or above the threshold, in stored energies, or not.  below: the kept
    // energy of block `best`; secondE: the largest bound of the others.
    float below = bestE;
    if constexpr (BOUND) {
        if (!halves) {                         // uniform
            u16x2 a[SX];
            sorted_top(keep, a);
            below = bestE >= 0.f ? pk_pair_energy<SX>(a, h != 0) * e_scale : -1.f;
        }
    }
    if constexpr (SHARED) {
        __syncthreads();                       // the signals in front are dead
        float* xb = reinterpret_cast<float*>(front);       // kept, best bound, second, block: [4][NW][64]
        xb[wave * 64 + lane] = below;
        xb[(NW + wave) * 64 + lane] = bestE;
        xb[(2 * NW + wave) * 64 + lane] = secondE;
        xb[(3 * NW + wave) * 64 + lane] = __builtin_bit_cast(float, best);
        __syncthreads();
        below = bestE = secondE = -1.f;
        for (int w = 0; w < NW; ++w) {         // bestE: the bound of the block that is ahead
            const float e = xb[w * 64 + lane], u = xb[(NW + w) * 64 + lane];
            const bool ahead = e > below;
            secondE = fmaxf(fmaxf(secondE, xb[(2 * NW + w) * 64 + lane]), ahead ? bestE : u);
            best = ahead ? __builtin_bit_cast(int, xb[(3 * NW + w) * 64 + lane]) : best;
            bestE = ahead ? u : bestE;
            below = fmaxf(below, e);
        }
        if (g.rows > 1) {                      // uniform
            // Of a column of workgroups the last one to finish goes on, with what all have found; nobody waits.  All of the exchange
            // goes past the caches of an XCD (atomics of the agent scope, both ways), and every store has been acknowledged before
            // the count: the order that a fence would give, without writing the L2 back (a release and an acquire: 1 to 3 us more).
            const int row = (int)blockIdx.y, col = (int)blockIdx.x;
            const int j_beg = min(row * per_row * UB, K), j_end = min((row + 1) * per_row * UB, K);
            unsigned* E_all = g.split_E + (size_t)col * K * 32;
            unsigned* E_own = reinterpret_cast<unsigned*>(E16);
            unsigned* x = g.split_x + (size_t)(col * g.rows) * 256;
            for (int e = j_beg * 32 + tid; e < j_end * 32; e += NTH)
                __hip_atomic_store(&E_all[e], E_own[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (wave == 0) {
                const float found[4] = {below, bestE, secondE, __builtin_bit_cast(float, best)};
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    __hip_atomic_store(&x[(row * 4 + k) * 64 + lane], __builtin_bit_cast(unsigned, found[k]), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (tid == 0) {
                const int before = __hip_atomic_fetch_add(&g.split_done[col], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (before == g.rows - 1) __hip_atomic_store(&g.split_done[col], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                *n_tasks = before;
            }
            __syncthreads();
            const bool last = *n_tasks == g.rows - 1;
            if (!last) return;                 // uniform
            __syncthreads();
            if (tid == 0) *n_tasks = 0;
            for (int e = tid; e < K * 32; e += NTH)
                if (e < j_beg * 32 || e >= j_end * 32)
                    E_own[e] = __hip_atomic_load(&E_all[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            below = bestE = secondE = -1.f;
            for (int r = 0; r < g.rows; ++r) {
                float v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    v[k] = __builtin_bit_cast(float, __hip_atomic_load(&x[(r * 4 + k) * 64 + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                const bool ahead = v[0] > below;
                secondE = fmaxf(fmaxf(secondE, v[2]), ahead ? bestE : v[1]);
                best = ahead ? __builtin_bit_cast(int, v[3]) : best;
                bestE = ahead ? v[1] : bestE;
                below = fmaxf(below, v[0]);
            }
        }
    }
    // one unit for the rounding of the table; BOUND: what the sum of a bound may lose to rounding
    constexpr float kUnits = 1.f + (!BOUND ? 0.f : 65535.f * P * 0x1p-25f * (1.f + (float)P / SX));
    const unsigned t16 = (HOME || GUESS) && halves ? t_home : threshold(below, norms(), kUnits);
    if constexpr (HOME || GUESS)
        if (tid == 0) g.short_cut[blockIdx.x] = halves;
    const bool undecided = stored(secondE) >= t16;
    if (t16 == 0x10000u) best = 0;             // a zero signal: block 0 (ties go to the lowest)
    if constexpr (home_applies<P>(SX))
        if (!SHARED && g.weak != nullptr && wave == 0 && blockIdx.x % kWeakEvery == 0) {   // uniform over the wavefront
            const int weak = __popcll(__ballot(t16 < kWeakBelow));
            if (lane == 0 && weak != 0) atomicAdd(&g.weak[g.turn % 3], weak);
            if (blockIdx.x == 0 && lane == 0) g.weak[(g.turn + 1) % 3] = 0;
        }
    if (!SHARED || wave == 0) {
        if constexpr (HOME) {
            id_own = ids[loc0 + lane];
            reinterpret_cast<int*>(r2s)[loc0 + lane] = id_own;                     // (its own signal's: used above)
        }
        thr[loc0 + lane] = undecided ? t16 : 0x10000u;
        key[loc0 + lane] = 0ull;
    }
    if (__ballot(undecided) != 0ull && lane == 0) *any_flag = 1;
    __syncthreads();

    // Resolution: the candidates of the undecided signals, block by block.
    if (*any_flag != 0) {                      // uniform
        // every row of the table becomes the list of its candidates, padded to whole tiles of 32 with 0xffff, and
        // the tiles of all rows one list of tasks
        unsigned short* tasks = reinterpret_cast<unsigned short*>(front);
        unsigned tr[SIG / 64];
#pragma unroll
        for (int r = 0; r < SIG / 64; ++r) tr[r] = thr[r * 64 + lane];
        for (int j = wave; j < K; j += NW) {
            unsigned short* row = E16 + j * SIG;
            unsigned v[SIG / 64];
#pragma unroll
            for (int r = 0; r < SIG / 64; ++r) v[r] = row[r * 64 + lane];
            int len = 0;
#pragma unroll
            for (int r = 0; r < SIG / 64; ++r) {
                const bool in = v[r] >= tr[r];
                const unsigned long long mask = __ballot(in);
                if (in) row[len + __popcll(mask & ((1ull << lane) - 1ull))] = (unsigned short)(r * 64 + lane);
                len += __popcll(mask);
            }
            if (len == 0) continue;            // uniform
            const int tiles = (len + 31) >> 5;
            if (len + lane < tiles * 32) row[len + lane] = 0xffff;
            int at = 0;
            if (lane == 0) at = atomicAdd(n_tasks, tiles);
            at = __builtin_amdgcn_readfirstlane(at);
            if (lane < tiles) tasks[at + lane] = (unsigned short)(j * (SIG / 32) + lane);
        }
        __syncthreads();
        const int n_task = *n_tasks;
        // (the signals of the next task are on their way while the present one is computed)
        int id_next = -1, j_next = 0;
        ExactRow<P, ARITH> y_next;
        auto signal = [&](int id) {
            return id < 0 ? (int64_t)-1 : HOME ? (int64_t)reinterpret_cast<const int*>(r2s)[id] : wg0 + id;
        };
        auto look_up = [&](int t) {
            id_next = -1;
            if (t < n_task) {                  // uniform
                const int task = __builtin_amdgcn_readfirstlane((int)tasks[t]);
                j_next = task / (SIG / 32);
                const int id = (int)E16[task * 32 + n];
                id_next = id == 0xffff ? -1 : id;
            }
            y_next.load(g, signal(id_next), h);
        };
        look_up(wave);
        for (int t = wave; t < n_task; t += NW) {
            const int id = id_next, j = j_next;
            const ExactRow<P, ARITH> y = y_next;
            look_up(t + NW);
            const float e = exact_energy<P, S, SX, ARITH>(g, y, signal(id), j, lane);
            // the largest energy (bits of a non-negative float), the lower block on a tie
            if (h == 0 && id >= 0)
                atomicMax(&key[id], ((unsigned long long)__builtin_bit_cast(unsigned, e) << 32) | (unsigned)(~j));
        }
        __syncthreads();
        if (undecided) best = (int)~(unsigned)key[loc0 + lane];
    }
    if (valid && (!SHARED || wave == 0)) g.blk[HOME ? (int64_t)id_own : wg0 + loc0 + lane] = best;

    // First step of the grouping (Section 3.3), folded in here: chunk_count[c][j] += number of
    // this workgroup's signals that chose block j (chunk is a multiple of SIG; the array is zero on
    // entry).  Integer atomics only: the sums do not depend on the order.
    if (HOME && by_home) {                     // uniform: of all chunks
        // Neighbours in a block's list are neighbours in the set where blocks are few: one addition for all signals of a wavefront that
        // are of the same chunk and chose the same block (an addition for each, 64 to one address: six iterations on 262144 signals, p = 64,
        // choice, K = 4 388 us, so 210; K = 16 387, 342; K = 32 493, 473; p = 256, 131072 signals, K = 8 669, 557).
        const unsigned at = (unsigned)id_own / (unsigned)g.chunk * (unsigned)K + (unsigned)best;
        unsigned long long left = __ballot(valid);
        for (int t = 0; t < kSameCounts && left != 0ull; ++t) {
            const int l = __builtin_ctzll(left);
            const unsigned long long same = __ballot(valid && at == (unsigned)__builtin_amdgcn_readlane((int)at, l));
            if (lane == l) atomicAdd(&g.chunk_count[at], __popcll(same));
            left &= ~same;
        }
        if ((left >> lane & 1ull) != 0ull) atomicAdd(&g.chunk_count[at], 1);
    } else if (g.chunk_count != nullptr) {     // uniform
        int* lh = reinterpret_cast<int*>(front);
        __syncthreads();                       // the lists are dead
        for (int j = tid; j < K; j += NTH) lh[j] = 0;
        __syncthreads();
        if (valid && (!SHARED || wave == 0)) atomicAdd(&lh[best], 1);
        __syncthreads();
        const unsigned cc = (unsigned)wg0 / (unsigned)g.chunk;
        for (int j = tid; j < K; j += NTH)
            if (lh[j] != 0) atomicAdd(&g.chunk_count[cc * (unsigned)K + j], lh[j]);
    }
}

template <int P, int S, int SX, int ARITH, bool SHARED, int W, Choice CHOICE>
hipError_t launch_w(const ScrArgs& a, int waves, LdsRaised* raised, hipStream_t st) {
    constexpr int sig = SHARED ? 64 : 64 * W;
    const size_t lds = scr_lds_bytes<P, SHARED, W>(a.K);
    if (lds > kScrLdsMax || a.chunk % sig != 0) return hipErrorInvalidValue;
    const void* fn = reinterpret_cast<const void*>(&energy_screen_kernel<P, S, SX, ARITH, SHARED, W, CHOICE>);
    if (hipError_t e = raised->ensure(fn, kScrLdsMax); e != hipSuccess || a.load_only) return e;
    hipLaunchKernelGGL((energy_screen_kernel<P, S, SX, ARITH, SHARED, W, CHOICE>), dim3((unsigned)((a.m + sig - 1) / sig), (unsigned)a.rows),
                       dim3(64 * waves), lds, st, a);
    return hipGetLastError();
}

// Small sets (choose_in_select): no screening.  What a call on a few hundred signals waits for is launches and trips to
// memory, not products, so a wavefront takes one block for 32 signals at full precision, with operands made from D itself
// (no launch for them), and leaves the energies; the select kernel compares them.  225 signals, K = 32, p = 64: operand
// orders 2.8 us + screened choice 11.2 -> 4.5, and 2 us in the select kernel.
template <int P, int S, int SX, int ARITH>
__global__ __launch_bounds__(64) void energy_direct_kernel(ScrArgs g) {
    const int lane = threadIdx.x, h = lane >> 5, i = (int)blockIdx.x * 32 + (lane & 31), j = (int)blockIdx.y;
    const int64_t id = i < g.m ? i : -1;
    ExactRow<P, ARITH> y;
    y.load(g, id, h);
    const float e = exact_energy<P, S, SX, ARITH, true>(g, y, id, j, lane);
    if (h == 0 && i < g.m) g.E[(int64_t)j * g.m + i] = e;
}

// Which shape (the rules of sbo_internal.h).
template <int P>
bool scr_by_256(const ScrArgs& a) {
    return P <= 64 && scr_lds_bytes<P, false, kScrWaves / 2>(a.K) <= kScrLdsMax / 2 && screen_by_256(a.m);
}
template <int P>
bool scr_shared(const ScrArgs& a) {
    return screen_shared(a.m, P == 64 && scr_by_256<P>(a)) || scr_lds_bytes<P, false, kScrWaves>(a.K) > kScrLdsMax;
}
template <int P, int S, int SX, int ARITH>
hipError_t launch_a(const ScrArgs& a, LdsRaised* raised, hipStream_t st) {
    if (scr_shared<P>(a)) {
        const int units = P == 64 || P > 64 ? a.K : (a.K * P + 31) / 32;
        ScrArgs b = a;
        b.rows = choice_split(P, a.K, a.m);
        if (b.rows > 1 && (int64_t)((a.m + 63) / 64) * a.K > a.split_room) return hipErrorInvalidValue;
        return launch_w<P, S, SX, ARITH, true, kScrWaves, kFull>(b, units < kScrWaves ? units : kScrWaves, raised, st);
    }
    if constexpr (P <= 64)
        if (scr_by_256<P>(a))
            return launch_w<P, S, SX, ARITH, false, kScrWaves / 2, kFull>(a, kScrWaves / 2, raised, st);
    return launch_w<P, S, SX, ARITH, false, kScrWaves, kFull>(a, kScrWaves, raised, st);
}

// With home blocks (the signals in the order of the grouping in g.perm), or guessing them.
template <int P, int SX, int ARITH, Choice CHOICE>
hipError_t launch_home_a(const ScrArgs& a, LdsRaised* raised, hipStream_t st) {
    constexpr int S = pow2_at_least(SX);
    if constexpr (P <= 64)
        if (scr_by_256<P>(a))
            return launch_w<P, S, SX, ARITH, false, kScrWaves / 2, CHOICE>(a, kScrWaves / 2, raised, st);
    return launch_w<P, S, SX, ARITH, false, kScrWaves, CHOICE>(a, kScrWaves, raised, st);
}
template <int P, Choice CHOICE>
hipError_t launch_home_p(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st) {
    switch (a.s0) {
#define SBO_CASE(N) \
    case N:         \
        if constexpr (home_applies<P>(N) && (CHOICE != kGuess || N <= kGuessMaxS0)) { \
            if (arith == SBO_ARITH_F16X2) return launch_home_a<P, N, 3, CHOICE>(a, raised, st); \
            if constexpr (P <= 64) return arith == SBO_ARITH_F32 ? launch_home_a<P, N, 0, CHOICE>(a, raised, st) : launch_home_a<P, N, 1, CHOICE>(a, raised, st); \
        } \
        break;
        SBO_CASE(1) SBO_CASE(2) SBO_CASE(3) SBO_CASE(4) SBO_CASE(5) SBO_CASE(6) SBO_CASE(7) SBO_CASE(8)
        SBO_CASE(9) SBO_CASE(10) SBO_CASE(11) SBO_CASE(12) SBO_CASE(13) SBO_CASE(14) SBO_CASE(15) SBO_CASE(16)
#undef SBO_CASE
        default: break;
    }
    return hipErrorInvalidValue;
}
// Whether launch_home_p has a kernel for these sizes: where workgroups take more than 64 signals, and there are steps to save.  p = 64, six
// iterations, full / home blocks: K = 3 262144 signals 649 / 649 us, s0 = 8, 3 % noise 676 / 704, K = 5 641 / 637, 682 / 702, K = 7 665 / 656,
// 713 / 724, K = 8 679 / 639, 711 / 710; 60001, K = 3 371 / 371, 389 / 401, K = 8 355 / 341, 378 / 375; p = 256, 131072, K = 2 2557 / 2502.
template <int P>
bool home_takes(const ScrArgs& a) {
    return home_applies<P>(a.s0) && !scr_shared<P>(a) && a.K >= (P > 64 ? 1 : 8);
}

// s0 is a compile-time constant of the kernels.  It pays where the selection networks take part of the time (width s0
// against the next power of two: p = 32, K = 32, 262144 signals s0 = 9 69 us, 16 92; p = 16, K = 32, 524288 signals 5 69, 8 91;
// p = 256, K = 16, 131072 signals 12 297, 16 314), not with bounds (p = 64, 5 to 16: 105 to 108 us).
template <int P, int SX>
hipError_t launch_s(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st) {
    constexpr int S = pow2_at_least(SX);
    if (arith == SBO_ARITH_F16X2) return launch_a<P, S, SX, 3>(a, raised, st);
    if constexpr (P <= 64) {
        if (arith == SBO_ARITH_F32) return launch_a<P, S, SX, 0>(a, raised, st);
        return launch_a<P, S, SX, 1>(a, raised, st);
    }
    return hipErrorInvalidValue;
}

template <int P>
hipError_t launch_direct_p(const ScrArgs& a, int arith, hipStream_t st) {
    const dim3 grid((unsigned)(a.m + 31) / 32, (unsigned)a.K);
    switch (a.s0) {
#define SBO_CASE(N) \
    case N:         \
        if constexpr (screen_applies(P, 1, N, SBO_ARITH_F16X2)) { \
            constexpr int S = pow2_at_least(N); \
            if (arith == SBO_ARITH_F16X2) hipLaunchKernelGGL((energy_direct_kernel<P, S, N, 3>), grid, dim3(64), 0, st, a); \
            else if (arith == SBO_ARITH_F32) hipLaunchKernelGGL((energy_direct_kernel<P, S, N, 0>), grid, dim3(64), 0, st, a); \
            else hipLaunchKernelGGL((energy_direct_kernel<P, S, N, 1>), grid, dim3(64), 0, st, a); \
            return hipGetLastError(); \
        } \
        break;
        SBO_CASE(1) SBO_CASE(2) SBO_CASE(3) SBO_CASE(4) SBO_CASE(5) SBO_CASE(6) SBO_CASE(7) SBO_CASE(8)
        SBO_CASE(9) SBO_CASE(10) SBO_CASE(11) SBO_CASE(12) SBO_CASE(13) SBO_CASE(14) SBO_CASE(15) SBO_CASE(16)
#undef SBO_CASE
        default: break;
    }
    return hipErrorInvalidValue;
}

template <int P>
hipError_t launch_p(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st) {
    switch (a.s0) {
#define SBO_CASE(N) \
    case N:         \
        if constexpr (screen_applies(P, 1, N, SBO_ARITH_F16X2)) return launch_s<P, N>(a, arith, raised, st); \
        break;
        SBO_CASE(1) SBO_CASE(2) SBO_CASE(3) SBO_CASE(4) SBO_CASE(5) SBO_CASE(6) SBO_CASE(7) SBO_CASE(8)
        SBO_CASE(9) SBO_CASE(10) SBO_CASE(11) SBO_CASE(12) SBO_CASE(13) SBO_CASE(14) SBO_CASE(15) SBO_CASE(16)
#undef SBO_CASE
        default: break;
    }
    return hipErrorInvalidValue;
}

}  // namespace

}  // namespace sbo
