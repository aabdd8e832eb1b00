// Sparse-coding stage 1: for every signal, the kept energy in every orthobase and
// the block where it is largest (Section 2, eq. (4); Section 3.1).
//
// c = Q_j^T y is a dense contraction for the matrix cores: 32 x 32 MFMA tiles with atoms
// on the M axis and signals on the N axis, so that the accumulator tile leaves every
// signal's coefficients in just two lanes (l and l^32).  The s0 largest magnitudes
// are then found in registers by compare-exchange networks, merged across the lane
// pair, squared and summed, and compared against the running best block.  The K*p x m
// projection never leaves the register file.
//
// Dictionary rows (atom k of block j = row j*p + k) are streamed through LDS in stages of
// 64 (p = 256: 32) rows, double-buffered, in the exact per-lane order the MFMA A operand
// wants, so every LDS read is one conflict-free 16-byte load per lane.  A small kernel
// first rewrites D into that order (zero-padded to whole stages), which makes the
// per-stage copy global -> registers -> LDS linear on both sides.
//
// The block choice of most calls is screened (code_screen.h); the kernels here choose it from full
// products, for what is not: p = 16 with s0 > 8, and p = 256 in two of the three arithmetics
// (SBO_OPT_CODING_ARITH).
//   energy_kernel              SBO_ARITH_F32: the fp32 matrix instruction (32x32x2);
//   energy_split_kernel        p = 16: every fp32 operand as three bf16 parts, six partial products, or as two
//                              fp16 parts (scaled), three partial products;
//   energy_split_wide_kernel   p = 256: three bf16 parts.
// Also here: the dictionary in the coding kernels' operand orders.
#include "sbo_internal.h"
#include "device_utils.h"
#include "energy_networks.h"
#include "screen_args.h"

namespace sbo {

namespace {

// Dsw[stage][(mt*QN + q)*64 + hh*32 + nn] = dims hh*P/2 + 4q .. +3 of row stage*64 + mt*32 + nn
// (rows past K*P are zero): the order in which a wavefront's lanes consume the A operand.
template <int P>
__global__ __launch_bounds__(256) void dict_swizzle_kernel(const float* __restrict__ D, int K,
                                                           f32x4* __restrict__ Dsw, CallStart start) {
    constexpr int QN = P / 8;
    constexpr int STAGE_F4 = 2 * QN * 64;
    start.clear();
    const f32x4* D4 = reinterpret_cast<const f32x4*>(D);
    const int rows = K * P;
    const int s = blockIdx.x;
    for (int f = threadIdx.x; f < STAGE_F4; f += 256) {
        const int nn = f & 31, hh = (f >> 5) & 1, mq = f >> 6;
        const int q = mq % QN, mt = mq / QN;
        const int grow = s * 64 + mt * 32 + nn;
        const int d4 = hh * QN + q;
        Dsw[(int64_t)s * STAGE_F4 + f] =
            grow < rows ? D4[(int64_t)grow * (P / 4) + d4] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

// The same dictionary in parts, 8 consecutive dims of a row per 16-byte unit and part (see
// device_utils.h): three bf16 (Dsb) and / or two fp16 (Dsh; then also dnorm, per 16 atoms the largest
// norm of an atom and of what its leading fp16 part leaves).  One launch for both orders.  Latency is all it is
// (a trip to memory each way), so a thread takes one or two units: p = 256, K = 16 13.3 us with 64 rows to
// a workgroup, 9.4 with 16.  GUESS (p = 64): also |Q Q^T - I|_F^2 of every block, and which of the sample of the signals it represents;
// K = 64 4.5 -> 5.4 us with the sample (in workgroups of its own, that read D once more, 8.2).
template <int P>
constexpr int dict_rows() {
    return P == 256 ? 16 : P == 64 ? 32 : 64;
}

// Which of 32 signals a block of 64 atoms represents (kSample): rows = the leading parts of its atoms in operand order, LDS,
// [atom / 32][ks][.][lane]; y: this lane's half of the dims of signal lane % 32.  One wavefront.
__device__ __forceinline__ unsigned represented(const u32x4 (&rows)[2][4][2][64], const f32x4 (&y)[4][2]) {
    const int lane = threadIdx.x & 63;
    float vmax = 0.f, y2 = 0.f;                // scaled to [1/2, 1) as in code_screen.h; zero, or too small for that: represented
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) vmax = fmaxf(vmax, fabsf(y[ks][e >> 2][e & 3]));
    vmax = fmaxf(vmax, other_half(vmax));
    const unsigned ex = (__builtin_bit_cast(unsigned, vmax) >> 23) & 0xffu;
    const float scale = ex >= 64u && ex <= 240u ? __builtin_bit_cast(float, (253u - ex) << 23) : 0.f;
    f32x16 acc[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) acc[mt] = f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const f32x4 v0 = y[ks][0] * scale, v1 = y[ks][1] * scale;
        const u32x4 b = {pack_f16(v0.x, v0.y), pack_f16(v0.z, v0.w), pack_f16(v1.x, v1.y), pack_f16(v1.z, v1.w)};
#pragma unroll
        for (int e = 0; e < 4; ++e) y2 = fmaf(v0[e], v0[e], fmaf(v1[e], v1[e], y2));
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
            acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, rows[mt][ks][0][lane]),
                                                             __builtin_bit_cast(f16x8, b), acc[mt], 0, 0, 0);
    }
    y2 = (y2 + other_half(y2)) * (kF16DictScale * kF16DictScale);
    const float top = y2 * (kHomeT / 64);
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < 16; ++v)
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) sum[2 * mt + (v & 1)] += fminf(acc[mt][v] * acc[mt][v], top);
    const float half = (sum[0] + sum[1]) + (sum[2] + sum[3]);
    return (unsigned)__ballot(half + other_half(half) <= y2 * home_rest(64));
}

template <int P, bool GUESS>
__global__ __launch_bounds__(256) void dict_parts_kernel(const float* __restrict__ D, int K,
                                                         u32x4* __restrict__ Dsb, u32x4* __restrict__ Dsh,
                                                         float2* __restrict__ dnorm, int* __restrict__ dodd,
                                                         float* __restrict__ dev, CallStart start,
                                                         SignalSample sample) {
    start.clear();
    constexpr int KS16 = P / 16, R = dict_rows<P>();
    __shared__ float qs[R][P / 8 + 1], rs[R][P / 8 + 1];
    // GUESS (p = 64): the rows of the whole block, [half, this one's first][ks][hi, lo][lane]
    __shared__ u32x4 both[GUESS ? 2 : 1][GUESS ? KS16 : 1][2][GUESS ? 64 : 1];
    __shared__ float off[2];
    const f32x4* D4 = reinterpret_cast<const f32x4*>(D);
    const int rows = K * P;
    const int row0 = blockIdx.x * R;
    // the sample of the signals: half of its tiles for each of the two workgroups of a block, one for each wavefront
    f32x4 y[GUESS ? 4 : 1][2];
    const int tile = (blockIdx.x & 1) * 4 + (int)(threadIdx.x >> 6);
    for (int g = threadIdx.x; g < R * (P / 8); g += 256) {         // (ks, hh, row)
        const int r = g % R, kh = g / R, ks = kh >> 1, hh = kh & 1;
        const int grow = row0 + r, lane = hh * 32 + (grow & 31);
        const int64_t mk = (int64_t)(grow >> 5) * KS16 + ks;       // 64 rows: two tiles of 32
        f32x4 v0 = {0.f, 0.f, 0.f, 0.f}, v1 = v0;
        if (grow < rows) {
            v0 = D4[(int64_t)grow * (P / 4) + ks * 4 + hh * 2];
            v1 = D4[(int64_t)grow * (P / 4) + ks * 4 + hh * 2 + 1];
        }
        f32x4 o0 = {0.f, 0.f, 0.f, 0.f}, o1 = o0;
        if constexpr (GUESS) {
            static_assert(P == 64 && R * (P / 8) == 256 && kSample == 8 * 32, "once; two workgroups of four wavefronts");
            const f32x4* other = D4 + (int64_t)(grow ^ 32) * (P / 4) + ks * 4 + hh * 2;
            o0 = other[0];
            o1 = other[1];
            // (last: loads return in order, and these come from further away)
            const int64_t i = (int64_t)(tile * 32 + (threadIdx.x & 31)) * sample.m / kSample;
            const f32x4* y4 = reinterpret_cast<const f32x4*>(sample.Y + i * P) + ((threadIdx.x >> 5) & 1) * 2;
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int e = 0; e < 2; ++e) y[k][e] = y4[k * 4 + e];
        }
        if (Dsb != nullptr) {
            const Bf16x3Pair a = split_bf16x3(v0.x, v0.y), b = split_bf16x3(v0.z, v0.w);
            const Bf16x3Pair c = split_bf16x3(v1.x, v1.y), d = split_bf16x3(v1.z, v1.w);
            u32x4* out = Dsb + mk * (3 * 64) + lane;
            out[0] = u32x4{a.hi, b.hi, c.hi, d.hi};
            out[64] = u32x4{a.mid, b.mid, c.mid, d.mid};
            out[128] = u32x4{a.lo, b.lo, c.lo, d.lo};
        }
        if (Dsh != nullptr) {
            float q2 = 0.f, r2 = 0.f;
            const F16x2Quad a = split_f16x2_dict(v0, q2, r2), b = split_f16x2_dict(v1, q2, r2);
            u32x4* out = Dsh + mk * (2 * 64) + lane;
            out[0] = u32x4{a.hi.x, a.hi.y, b.hi.x, b.hi.y};
            out[64] = u32x4{a.lo.x, a.lo.y, b.lo.x, b.lo.y};
            qs[r][kh] = q2;
            rs[r][kh] = r2;
            if constexpr (GUESS) {
                const int lane_g = hh * 32 + r;
                const F16x2Quad c = split_f16x2_dict(o0, q2, r2), d = split_f16x2_dict(o1, q2, r2);
                both[0][ks][0][lane_g] = u32x4{a.hi.x, a.hi.y, b.hi.x, b.hi.y};
                both[0][ks][1][lane_g] = u32x4{a.lo.x, a.lo.y, b.lo.x, b.lo.y};
                both[1][ks][0][lane_g] = u32x4{c.hi.x, c.hi.y, d.hi.x, d.hi.y};
                both[1][ks][1][lane_g] = u32x4{c.lo.x, c.lo.y, d.lo.x, d.lo.y};
            }
        }
    }
    if (Dsh != nullptr) {                      // uniform
        __syncthreads();
        if (threadIdx.x < R) {
            float q2 = 0.f, r2 = 0.f;
            for (int e = 0; e < P / 8; ++e) {
                q2 += qs[threadIdx.x][e];
                r2 += rs[threadIdx.x][e];
            }
            const bool odd = odd_norm2(q2);
            q2 = row16_max(q2);
            r2 = row16_max(r2);
            const int at = (row0 + (int)threadIdx.x) >> 4;
            if ((threadIdx.x & 15) == 0 && at < K * (P / 16)) dnorm[at] = float2{sqrtf(q2), sqrtf(r2)};
            if constexpr (P == 256) {          // (before the shuffle, or lanes of other sixteens)
                const unsigned long long mask = __ballot(odd);
                if ((threadIdx.x & 15) == 0 && at < K * (P / 16)) dodd[at] = (int)(mask >> (threadIdx.x & 48) & 0xffff) != 0;
            }
        }
        if constexpr (GUESS) {
            // Half of Q Q^T, products to 2^-22: this workgroup's rows with themselves by the third wavefront, with the others by
            // the last.
            const int lane = threadIdx.x & 63, half = (int)(threadIdx.x >> 6) - 2;
            if (half >= 0) {                   // uniform over the wavefront
                f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int t = 0; t < 3; ++t)
#pragma unroll
                    for (int ks = 0; ks < KS16; ++ks)
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, both[0][ks][t == 1][lane]),
                                                                     __builtin_bit_cast(f16x8, both[half][ks][t == 2][lane]), acc, 0, 0, 0);
                float sum = 0.f;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = (v & 3) + 8 * (v >> 2) + 4 * (lane >> 5);
                    const float d = acc[v] * (1.f / (kF16DictScale * kF16DictScale)) - (half == 0 && row == (lane & 31) ? 1.f : 0.f);
                    sum = fmaf(d, d, sum);
                }
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
                if (lane == 0) off[half] = sum;
            }
            const unsigned mask = represented(both, y);
            if (lane == 0) sample.mask[(blockIdx.x >> 1) * (kSample / 32) + tile] = mask;
            __syncthreads();
            if (threadIdx.x == 0) dev[blockIdx.x] = off[0] + off[1];
        }
    }
}

template <int P, int S, int NT, int SX>
__global__ __launch_bounds__(256) void energy_kernel(const float* __restrict__ Y, int m,
                                                     const f32x4* __restrict__ Dsw, int K, int s0,
                                                     int32_t* __restrict__ blk,
                                                     float* __restrict__ energy,
                                                     int32_t* __restrict__ chunk_count, int chunk,
                                                     int units_per_y) {
    constexpr int KS = P / 2;            // contraction steps (each lane half covers P/2 dims)
    constexpr int QN = P / 8;            // 16-byte groups of steps per 32-row tile
    constexpr int NB = P <= 64 ? 64 / P : 1;   // blocks per 64-row stage (p <= 64)
    constexpr int SPB = P <= 64 ? 1 : P / 64;  // 64-row stages per block (p > 64)
    constexpr int NV = P <= 64 ? P / 2 : 32;   // coefficients per lane per block and stage
    constexpr int STAGE_F4 = 2 * QN * 64;
    constexpr int FPT = STAGE_F4 / 256;  // 16-byte pieces each thread moves per stage
    static_assert(P == 16 || P == 32 || P == 64 || P == 256, "unsupported p");
    static_assert(P <= 64 || S <= 32, "sort width");

    extern __shared__ f32x4 Qs_raw[];    // [2][STAGE_F4]
    f32x4(*Qs)[STAGE_F4] = reinterpret_cast<f32x4(*)[STAGE_F4]>(Qs_raw);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int h = lane >> 5, n = lane & 31;
    const int64_t sig0 = ((int64_t)blockIdx.x * 4 + wave) * (32 * NT);

    // B operand: this lane's half of the dims of NT signals, kept for the whole kernel.
    float yb[NT][KS];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int64_t i = sig0 + nt * 32 + n;
        if (i < m) {
            const f32x4* src = reinterpret_cast<const f32x4*>(Y + i * P + h * KS);
#pragma unroll
            for (int q = 0; q < QN; ++q) {
                f32x4 v = src[q];
                yb[nt][4 * q + 0] = v.x;
                yb[nt][4 * q + 1] = v.y;
                yb[nt][4 * q + 2] = v.z;
                yb[nt][4 * q + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int t = 0; t < KS; ++t) yb[nt][t] = 0.f;
        }
    }

    // Small m: the blocks are split over blockIdx.y (units_per_y > 0: that many stages, for
    // p > 64 that many blocks, per workgroup row), so that the chip is filled; every row then
    // writes its own best (energy, block) per signal at offset blockIdx.y * m and
    // energy_merge_kernel picks the winner.
    const int n_stage = (K * P + 63) / 64;
    int s_beg = 0, s_end = n_stage;
    if (units_per_y > 0) {
        s_beg = min(n_stage, (int)blockIdx.y * units_per_y * SPB);
        s_end = min(n_stage, s_beg + units_per_y * SPB);
        blk += (int64_t)blockIdx.y * m;
        energy += (int64_t)blockIdx.y * m;
    }

    f32x4 pre[FPT];
    auto fetch = [&](int s) {
#pragma unroll
        for (int r = 0; r < FPT; ++r) pre[r] = Dsw[(int64_t)s * STAGE_F4 + tid + 256 * r];
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int r = 0; r < FPT; ++r) Qs[buf][tid + 256 * r] = pre[r];
    };

    if (s_beg < s_end) {                 // uniform
        fetch(s_beg);
        stash(0);
    }
    __syncthreads();

    int best[NT];
    float bestE[NT];
    float run[NT][S];                    // p > 64: lane's top-S magnitudes of the current block
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        best[nt] = 0;
        bestE[nt] = -1.f;
#pragma unroll
        for (int i = 0; i < S; ++i) run[nt][i] = 0.f;
    }

    for (int s = s_beg; s < s_end; ++s) {
        const int cur = (s - s_beg) & 1;
        if (s + 1 < s_end) fetch(s + 1);

        f32x16 acc[NT][2];
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                             0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < QN; ++q) {
            f32x4 a[2];
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) a[mt] = Qs[cur][(mt * QN + q) * 64 + lane];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        acc[nt][mt] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                            a[mt][kk], yb[nt][4 * q + kk], (q == 0 && kk == 0) ? zero : acc[nt][mt],
                            0, 0, 0);
        }

        if (s + 1 < s_end) stash(cur ^ 1);

        if constexpr (P <= 64) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    float x[NV];
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        const int f = b * NV + v;      // flattened (tile, register)
                        x[v] = fabsf(acc[nt][f >> 4][f & 15]);
                    }
                    const float e = pair_top_energy<NV, S, SX>(x, s0, h != 0);
                    const int j = s * NB + b;
                    if (j < K && e > bestE[nt]) {
                        bestE[nt] = e;
                        best[nt] = j;
                    }
                }
            }
        } else {
            // A block spans SPB stages: keep the lane's sorted top-S across them and
            // combine the lane pair after the block's last stage.
            const int part = s % SPB;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                float x[32], a[S];
#pragma unroll
                for (int f = 0; f < 32; ++f) x[f] = fabsf(acc[nt][f >> 4][f & 15]);
                top_sorted<32, S>(x, a);
                if (part == 0) {
#pragma unroll
                    for (int i = 0; i < S; ++i) run[nt][i] = a[i];
                } else {
#pragma unroll
                    for (int i = 0; i < S; ++i) run[nt][i] = fmaxf(run[nt][i], a[S - 1 - i]);
                    bitonic_merge_desc<S>(run[nt]);
                }
                if (part == SPB - 1) {
                    const float e = pair_list_energy<S, SX>(run[nt], s0, h != 0);
                    const int j = s / SPB;
                    if (j < K && e > bestE[nt]) {
                        bestE[nt] = e;
                        best[nt] = j;
                    }
                }
            }
        }
        __syncthreads();
    }

    if (h == 0) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int64_t i = sig0 + nt * 32 + n;
            if (i < m) {
                blk[i] = best[nt];
                energy[i] = bestE[nt];
            }
        }
    }

    // First step of the grouping (Section 3.3), folded in here: chunk_count[c][j] += number of
    // this workgroup's signals that chose block j, c = the chunk of consecutive signals the
    // workgroup lies in (chunk is a multiple of the signals per workgroup; the array is zero
    // on entry).  Integer atomics only: the sums do not depend on the order.
    if (chunk_count != nullptr) {        // uniform
        int* lh = reinterpret_cast<int*>(Qs_raw);          // the stage buffers are dead (>= 8 KiB)
        for (int j = tid; j < K; j += 256) lh[j] = 0;
        __syncthreads();
        if (h == 0) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (sig0 + nt * 32 + n < m) atomicAdd(&lh[best[nt]], 1);
        }
        __syncthreads();
        const int64_t c = ((int64_t)blockIdx.x * (4 * 32 * NT)) / chunk;
        for (int j = tid; j < K; j += 256)
            if (lh[j] != 0) atomicAdd(&chunk_count[c * K + j], lh[j]);
    }
}

// p = 16 with more than p / 2 coefficients kept, where the blocks of a signal all but tie and
// screening (code_screen.h) would leave most of them in: the same kernel with the projection on the
// bf16 or fp16 matrix cores.  F16 = false: every fp32 operand entry is the exact sum of three bf16
// parts (device_utils.h), and the six partial products that matter at fp32 accuracy are accumulated in
// fp32 by v_mfma_f32_32x32x16_bf16.  F16 = true: the signals are scaled by a power of two each (largest
// magnitude into [2^13, 2^14)), the dictionary by kF16DictScale, both split into hi + lo in fp16, and
// the three products hi*lo, lo*hi, hi*hi run on v_mfma_f32_32x32x16_f16: a per-term error of
// 3 * 2^-22 |a b| (an fp32 dot product of p terms guarantees p * 2^-24 sum |a b|).  The choice of the
// block does not see the scales (common to all blocks of a signal); the energy written out is scaled
// back.  The signals' parts stay in registers for the whole kernel (B operand); the dictionary
// arrives in parts and is staged through LDS, double-buffered, one barrier per stage of 64 rows; a
// wavefront owns 64 signals, and a workgroup is two teams of four wavefronts, one wavefront of each team
// per SIMD, half a stage apart: while team 0 multiplies stage s, team 1 runs the selection networks
// on its stage s - 1 results, then the roles swap; both read the same LDS stage.
constexpr int kSplitWgWaves = 8;

template <int P, int NPL = 3>
struct SplitGeom {
    static constexpr int MTS = 2;                        // 32-row tiles per stage
    static constexpr int NT = 2;                         // 32-signal tile columns per wavefront
    static constexpr int WAVES = kSplitWgWaves;
    static constexpr bool TEAMS = true;
    static constexpr int KS16 = P / 16;                  // contraction steps of 16 dims
    static constexpr int STAGE_ROWS = 32 * MTS;
    static constexpr int STAGE_U = MTS * KS16 * NPL * 64;   // 16-byte units per stage
    static constexpr size_t LDS = (size_t)2 * STAGE_U * 16;
};

template <int P, int S, int SX, bool F16>
__global__ __launch_bounds__(64 * kSplitWgWaves) void energy_split_kernel(
    const float* __restrict__ Y, int m, const u32x4* __restrict__ Dsb, int K, int s0,
    int32_t* __restrict__ blk, float* __restrict__ energy, int32_t* __restrict__ chunk_count, int chunk,
    int units_per_y) {
    constexpr int NPL = F16 ? 2 : 3;           // operand parts
    using G = SplitGeom<P, NPL>;
    constexpr int MTS = G::MTS, NT = G::NT, KS16 = G::KS16, STAGE_U = G::STAGE_U;
    constexpr int NTH = 64 * G::WAVES;
    constexpr int NB = 64 / P;                 // blocks per stage
    constexpr int SPB = 1;
    constexpr int NV = P / 2;                  // coefficients per lane per block and stage
    constexpr int FPT = (STAGE_U + NTH - 1) / NTH;         // 16-byte units each thread moves per stage
    constexpr bool kWhole = STAGE_U % NTH == 0;
    static_assert(P == 16 || P == 32 || P == 64, "unsupported p");

    extern __shared__ u32x4 Qb_raw[];    // [2][STAGE_U]
    u32x4(*Qs)[STAGE_U] = reinterpret_cast<u32x4(*)[STAGE_U]>(Qb_raw);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int team = G::TEAMS ? wave >> 2 : 0;           // wavefronts w and w + 4 share a SIMD
    const int h = lane >> 5, n = lane & 31;
    const int64_t sig0 = ((int64_t)blockIdx.x * G::WAVES + wave) * (32 * NT);
    // B operand: the parts of this lane's dims (ks*16 + h*8 .. +7) of NT signals.
    u32x4 yq[NT][KS16][NPL];
    int64_t sig[NT];                     // the signal of this lane in tile column nt (-1: none)
    float unscale[NT];                   // F16: 1 / (scale of the signal * scale of the dictionary)^2
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int64_t t = sig0 + nt * 32 + n;
        sig[nt] = t < m ? t : -1;
        const int64_t i = sig[nt];
        unscale[nt] = 1.f;
        f32x4 raw[KS16][2];
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) {
            raw[ks][0] = f32x4{0.f, 0.f, 0.f, 0.f};
            raw[ks][1] = raw[ks][0];
            if (i >= 0) {
                const f32x4* src = reinterpret_cast<const f32x4*>(Y + i * P + ks * 16 + h * 8);
                raw[ks][0] = src[0];
                raw[ks][1] = src[1];
            }
        }
        float scale = 1.f;
        if constexpr (F16) {
            float vmax = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS16; ++ks)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    vmax = fmaxf(fmaxf(fmaxf(vmax, fabsf(raw[ks][e].x)), fmaxf(fabsf(raw[ks][e].y), fabsf(raw[ks][e].z))),
                                 fabsf(raw[ks][e].w));
            vmax = fmaxf(vmax, other_half(vmax));
            scale = f16_signal_scale(vmax);
            const float inv = 1.f / (scale * kF16DictScale);       // a power of two: exact
            unscale[nt] = inv * inv;
        }
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) {
            const f32x4 v0 = raw[ks][0], v1 = raw[ks][1];
            if constexpr (F16) {
                const F16x2Pair a = split_f16x2(v0.x * scale, v0.y * scale), b = split_f16x2(v0.z * scale, v0.w * scale);
                const F16x2Pair c = split_f16x2(v1.x * scale, v1.y * scale), d = split_f16x2(v1.z * scale, v1.w * scale);
                yq[nt][ks][0] = u32x4{a.hi, b.hi, c.hi, d.hi};
                yq[nt][ks][1] = u32x4{a.lo, b.lo, c.lo, d.lo};
            } else {
                const Bf16x3Pair a = split_bf16x3(v0.x, v0.y), b = split_bf16x3(v0.z, v0.w);
                const Bf16x3Pair c = split_bf16x3(v1.x, v1.y), d = split_bf16x3(v1.z, v1.w);
                yq[nt][ks][0] = u32x4{a.hi, b.hi, c.hi, d.hi};
                yq[nt][ks][1] = u32x4{a.mid, b.mid, c.mid, d.mid};
                yq[nt][ks][2] = u32x4{a.lo, b.lo, c.lo, d.lo};
            }
        }
    }

    // Small m: the stages are split over blockIdx.y exactly as in energy_kernel.
    const int n_stage = (K * P + G::STAGE_ROWS - 1) / G::STAGE_ROWS;
    int s_beg = 0, s_end = n_stage;
    if (units_per_y > 0) {
        s_beg = min(n_stage, (int)blockIdx.y * units_per_y * SPB);
        s_end = min(n_stage, s_beg + units_per_y * SPB);
        blk += (int64_t)blockIdx.y * m;
        energy += (int64_t)blockIdx.y * m;
    }

    u32x4 pre[FPT];
    auto fetch = [&](int s) {
#pragma unroll
        for (int r = 0; r < FPT; ++r)
            if (kWhole || tid + NTH * r < STAGE_U) pre[r] = Dsb[(int64_t)s * STAGE_U + tid + NTH * r];
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int r = 0; r < FPT; ++r)
            if (kWhole || tid + NTH * r < STAGE_U) Qs[buf][tid + NTH * r] = pre[r];
    };

    int best[NT];
    float bestE[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        best[nt] = 0;
        bestE[nt] = -1.f;
    }

    // the partial products, smallest first: (A part, B part); the fp16 parts have three in all
    constexpr int TA[6] = {F16 ? 0 : 2, F16 ? 1 : 0, F16 ? 0 : 1, 1, 0, 0};
    constexpr int TB[6] = {F16 ? 1 : 0, F16 ? 0 : 2, F16 ? 0 : 1, 0, 1, 0};
    constexpr int T1 = F16 ? 3 : 6;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                         0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 acc[NT][MTS];

    // Projection of the wavefront's signals onto the rows staged in buffer buf:
    // NT x MTS x KS16 x 6 matrix instructions into acc.
    auto project = [&](int buf) {
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) {
            u32x4 a[MTS][NPL];
#pragma unroll
            for (int mt = 0; mt < MTS; ++mt)
#pragma unroll
                for (int pl = 0; pl < NPL; ++pl) a[mt][pl] = Qs[buf][((mt * KS16 + ks) * NPL + pl) * 64 + lane];
#pragma unroll
            for (int t = 0; t < T1; ++t)
#pragma unroll
                for (int mt = 0; mt < MTS; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        const f32x16 c_in = (ks == 0 && t == 0) ? zero : acc[nt][mt];
                        if constexpr (F16)
                            acc[nt][mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                                __builtin_bit_cast(f16x8, a[mt][TA[t]]), __builtin_bit_cast(f16x8, yq[nt][ks][TB[t]]),
                                c_in, 0, 0, 0);
                        else
                            acc[nt][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                __builtin_bit_cast(bf16x8, a[mt][TA[t]]),
                                __builtin_bit_cast(bf16x8, yq[nt][ks][TB[t]]), c_in, 0, 0, 0);
                    }
        }
    };
    // Kept energy of the wavefront's signals in the blocks of stage s (from acc) against the
    // running best.
    auto select = [&](int s) {
        {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    float x[NV];
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        const int f = b * NV + v;      // flattened (tile, register)
                        x[v] = fabsf(acc[nt][f >> 4][f & 15]);
                    }
                    const float e = pair_top_energy<NV, S, SX>(x, s0, h != 0);
                    const int j = s * NB + b;
                    if (j < K && e > bestE[nt]) {
                        bestE[nt] = e;
                        best[nt] = j;
                    }
                }
            }
        }
    };

    if (s_beg < s_end) {                 // uniform
        fetch(s_beg);
        stash(0);
    }
    __syncthreads();
    for (int s = s_beg; s < s_end; ++s) {
        const int cur = (s - s_beg) & 1;
        if (s + 1 < s_end) fetch(s + 1);
        if (team == 0) {                 // uniform over the wavefront
            project(cur);
            select(s);
        } else {
            if (s > s_beg) select(s - 1);
            project(cur);
        }
        if (s + 1 < s_end) stash(cur ^ 1);
        __syncthreads();
    }
    if (team == 1 && s_beg < s_end) select(s_end - 1);

    if (h == 0) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (sig[nt] >= 0) {
                blk[sig[nt]] = best[nt];
                energy[sig[nt]] = bestE[nt] * unscale[nt];
            }
        }
    }
    // the grouping's chunk histograms (see energy_kernel)
    if (chunk_count != nullptr) {        // uniform
        int* lh = reinterpret_cast<int*>(Qb_raw);          // the stage buffers are dead
        for (int j = tid; j < K; j += NTH) lh[j] = 0;
        __syncthreads();
        if (h == 0) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (sig[nt] >= 0) atomicAdd(&lh[best[nt]], 1);
        }
        __syncthreads();
        const int64_t c = ((int64_t)blockIdx.x * (G::WAVES * 32 * NT)) / chunk;
        for (int j = tid; j < K; j += NTH)
            if (lh[j] != 0) atomicAdd(&chunk_count[c * K + j], lh[j]);
    }
}

// p = 256 on the bf16 matrix cores (SBO_ARITH_BF16X3; the two fp16 parts are screened, code_screen.h).
// The three bf16 parts of 32 signals take 192 registers per lane, too many for two wavefronts per SIMD,
// and with one wavefront per SIMD the selection networks would run while the matrix cores idle.  So the
// CONTRACTION is halved instead: the two wavefronts of a SIMD (w and w + 4) share their 32 signals,
// each holds one half of the dims (96 registers) and multiplies the staged rows (32 atoms a stage,
// double-buffered) by its half.  For every block one of the two is the selector (even blocks: the
// wavefront with the lower dims, odd blocks: the other): its partner leaves its partial products in
// LDS, the selector adds them to its own one stage later and runs the selection networks on the sums
// while the partner already multiplies the next stage.  A block spans 8 stages, across which the
// selector keeps the lane's running sorted top-S; the two wavefronts' best blocks are compared
// at the end.
constexpr int kWideWaves = 8;

template <int P, int S, int SX>
__global__ __launch_bounds__(64 * kWideWaves) void energy_split_wide_kernel(
    const float* __restrict__ Y, int m, const u32x4* __restrict__ Dsb, int K, int s0,
    int32_t* __restrict__ blk, float* __restrict__ energy, int32_t* __restrict__ chunk_count, int chunk,
    int units_per_y) {
    constexpr int KS16 = P / 16, KH = KS16 / 2;            // contraction steps: all, per wavefront
    constexpr int SPB = P / 32;                            // stages per block
    constexpr int NPL = 3;                                 // operand parts
    constexpr int STAGE_U = KS16 * NPL * 64;               // 16-byte units per stage of 32 rows
    constexpr int NTH = 64 * kWideWaves;
    constexpr int FPT = STAGE_U / NTH;
    static_assert(P == 256 && STAGE_U % NTH == 0 && S <= 16, "shape");

    extern __shared__ u32x4 Qw_raw[];    // Qs[2][STAGE_U] | xch[2][4 SIMDs][4][64] (f32x4)
    u32x4(*Qs)[STAGE_U] = reinterpret_cast<u32x4(*)[STAGE_U]>(Qw_raw);
    f32x4* xch = reinterpret_cast<f32x4*>(Qw_raw + 2 * STAGE_U);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int simd = wave & 3, half = wave >> 2;           // wavefronts w and w + 4 share a SIMD
    const int h = lane >> 5, n = lane & 31;
    // B operand: the parts of dims (half*KH + ks)*16 + h*8 .. +7 of this lane's signal
    u32x4 yq[KH][NPL];
    const int64_t sig = ((int64_t)blockIdx.x * 4 + simd) * 32 + n;
#pragma unroll
    for (int ks = 0; ks < KH; ++ks) {
        f32x4 v0 = {0.f, 0.f, 0.f, 0.f}, v1 = v0;
        if (sig < m) {
            const f32x4* src = reinterpret_cast<const f32x4*>(Y + sig * P + (half * KH + ks) * 16 + h * 8);
            v0 = src[0];
            v1 = src[1];
        }
        const Bf16x3Pair a = split_bf16x3(v0.x, v0.y), b = split_bf16x3(v0.z, v0.w);
        const Bf16x3Pair c = split_bf16x3(v1.x, v1.y), d = split_bf16x3(v1.z, v1.w);
        yq[ks][0] = u32x4{a.hi, b.hi, c.hi, d.hi};
        yq[ks][1] = u32x4{a.mid, b.mid, c.mid, d.mid};
        yq[ks][2] = u32x4{a.lo, b.lo, c.lo, d.lo};
    }

    // Small m: the blocks are split over blockIdx.y exactly as in energy_kernel.
    const int n_stage = K * SPB;
    int s_beg = 0, s_end = n_stage;
    if (units_per_y > 0) {
        s_beg = min(n_stage, (int)blockIdx.y * units_per_y * SPB);
        s_end = min(n_stage, s_beg + units_per_y * SPB);
        blk += (int64_t)blockIdx.y * m;
        energy += (int64_t)blockIdx.y * m;
    }

    u32x4 pre[FPT];
    auto fetch = [&](int s) {
#pragma unroll
        for (int r = 0; r < FPT; ++r) pre[r] = Dsb[(int64_t)s * STAGE_U + tid + NTH * r];
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int r = 0; r < FPT; ++r) Qs[buf][tid + NTH * r] = pre[r];
    };

    int best = 0;
    float bestE = -1.f;
    float run[S];                        // selector: lane's top-S magnitudes of the current block
#pragma unroll
    for (int t = 0; t < S; ++t) run[t] = 0.f;

    // the six partial products, smallest first: (A part, B part)
    constexpr int TA[6] = {2, 0, 1, 1, 0, 0};
    constexpr int TB[6] = {0, 2, 1, 0, 1, 0};
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                         0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 acc = zero;
    auto selects = [&](int s) { return (((s / SPB) & 1) == half); };   // uniform over the wavefront

    // This wavefront's half of the products of the rows staged in buffer buf.
    auto project = [&](int buf) {
#pragma unroll
        for (int ks = 0; ks < KH; ++ks) {
            u32x4 a[NPL];
#pragma unroll
            for (int pl = 0; pl < NPL; ++pl) a[pl] = Qs[buf][((half * KH + ks) * NPL + pl) * 64 + lane];
#pragma unroll
            for (int t = 0; t < 6; ++t)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[TA[t]]),
                                                              __builtin_bit_cast(bf16x8, yq[ks][TB[t]]),
                                                              (ks == 0 && t == 0) ? zero : acc, 0, 0, 0);
        }
    };
    // Selector of stage s: own partial (still in acc) + the partner's (exchange buffer buf), then
    // the lane's running top-S and, after the block's last stage, the kept energy of the lane pair.
    auto select = [&](int s, int buf) {
        const int part = s % SPB;
        float x[16], a[S];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 o = xch[((buf * 4 + simd) * 4 + q) * 64 + lane];
            x[4 * q + 0] = fabsf(acc[4 * q + 0] + o.x);
            x[4 * q + 1] = fabsf(acc[4 * q + 1] + o.y);
            x[4 * q + 2] = fabsf(acc[4 * q + 2] + o.z);
            x[4 * q + 3] = fabsf(acc[4 * q + 3] + o.w);
        }
        top_sorted<16, S>(x, a);
        if (part == 0) {                 // uniform
#pragma unroll
            for (int t = 0; t < S; ++t) run[t] = a[t];
        } else {
#pragma unroll
            for (int t = 0; t < S; ++t) run[t] = fmaxf(run[t], a[S - 1 - t]);
            bitonic_merge_desc<S>(run);
        }
        if (part == SPB - 1) {           // uniform
            const float e = pair_list_energy<S, SX>(run, s0, h != 0);
            const int j = s / SPB;
            if (e > bestE) {
                bestE = e;
                best = j;
            }
        }
    };

    if (s_beg < s_end) {                 // uniform
        fetch(s_beg);
        stash(0);
    }
    __syncthreads();
    for (int s = s_beg; s < s_end; ++s) {
        const int cur = (s - s_beg) & 1;
        if (s + 1 < s_end) fetch(s + 1);
        if (s > s_beg && selects(s - 1)) select(s - 1, cur ^ 1);
        project(cur);
        if (!selects(s)) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                xch[((cur * 4 + simd) * 4 + q) * 64 + lane] =
                    f32x4{acc[4 * q + 0], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        }
        if (s + 1 < s_end) stash(cur ^ 1);
        __syncthreads();
    }
    if (s_beg < s_end && selects(s_end - 1)) select(s_end - 1, (s_end - 1 - s_beg) & 1);

    // the better of the two wavefronts' best blocks (equal energies: the lower block)
    __syncthreads();                     // the exchange buffers are free
    float* mrgE = reinterpret_cast<float*>(xch);           // [4][64]
    int* mrgJ = reinterpret_cast<int*>(xch) + 4 * 64;
    if (half == 1) {
        mrgE[simd * 64 + lane] = bestE;
        mrgJ[simd * 64 + lane] = best;
    }
    __syncthreads();
    if (half == 0) {
        const float e = mrgE[simd * 64 + lane];
        const int j = mrgJ[simd * 64 + lane];
        if (e > bestE || (e == bestE && j < best)) {
            bestE = e;
            best = j;
        }
        if (h == 0 && sig < m) {
            blk[sig] = best;
            energy[sig] = bestE;
        }
    }

    // the grouping's chunk histograms (see energy_kernel)
    if (chunk_count != nullptr) {        // uniform
        int* lh = reinterpret_cast<int*>(Qw_raw);          // the stage buffers are dead
        for (int j = tid; j < K; j += NTH) lh[j] = 0;
        __syncthreads();
        if (half == 0 && h == 0 && sig < m) atomicAdd(&lh[best], 1);
        __syncthreads();
        const int64_t c = ((int64_t)blockIdx.x * 128) / chunk;
        for (int j = tid; j < K; j += NTH)
            if (lh[j] != 0) atomicAdd(&chunk_count[c * K + j], lh[j]);
    }
}

// Winner over the rows of a split launch: part_E / part_j hold, per row y, the best energy
// and block of the row's share of the blocks (rows in ascending block order, so the strict
// comparison keeps the lowest block among equal energies).  Also the grouping histogram
// (see energy_kernel).
__global__ __launch_bounds__(256) void energy_merge_kernel(const float* __restrict__ part_E,
                                                           const int32_t* __restrict__ part_j,
                                                           int rows, int m, int K,
                                                           int32_t* __restrict__ blk,
                                                           float* __restrict__ energy,
                                                           int32_t* __restrict__ chunk_count,
                                                           int chunk) {
    extern __shared__ int lh[];          // [K]
    const int tid = threadIdx.x;
    const int i = blockIdx.x * 256 + tid;
    int best = 0;
    float bestE = -1.f;
    if (i < m) {
        for (int y = 0; y < rows; ++y) {
            const float e = part_E[(int64_t)y * m + i];
            if (e > bestE) {
                bestE = e;
                best = part_j[(int64_t)y * m + i];
            }
        }
        blk[i] = best;
        energy[i] = bestE;
    }
    if (chunk_count != nullptr) {        // uniform
        for (int j = tid; j < K; j += 256) lh[j] = 0;
        __syncthreads();
        if (i < m) atomicAdd(&lh[best], 1);
        __syncthreads();
        const int64_t c = ((int64_t)blockIdx.x * 256) / chunk;
        for (int j = tid; j < K; j += 256)
            if (lh[j] != 0) atomicAdd(&chunk_count[c * K + j], lh[j]);
    }
}

// The kernels of this file, for what code_screen.h does not screen: p = 16 with s0 > 8 (all arithmetics) and
// p = 256 in SBO_ARITH_F32 and SBO_ARITH_BF16X3 (as which SBO_ARITH_F16X2 with K > kScreenWideMaxK comes here).
// arith: SBO_ARITH_*.
template <int P, int S, int SX>
hipError_t launch_pse(const float* Y, int64_t m, int K, int s0, int arith, const Workspace& ws, int32_t* blk,
                      int32_t* chunk_count, hipStream_t st) {
    constexpr int NT = P <= 64 ? 2 : 1;
    constexpr int QN = P / 8;
    constexpr bool wide = P > 64;
    const bool split = arith != SBO_ARITH_F32;
    const int per_wg = split ? (wide ? 128 : kSplitWgWaves * 64) : 4 * 32 * NT;
    dim3 grid((unsigned)((m + per_wg - 1) / per_wg));
    const int chunk = group_geom(m).chunk;
    if (ws.raised == nullptr || chunk % per_wg != 0) return hipErrorInvalidValue;
    // Fewer workgroups than CUs: split the blocks over a second grid dimension.
    const int units = P <= 64 ? (K * P + 63) / 64 : K;     // stages (p <= 64) or blocks
    const int rows_wanted = (int)grid.x >= kEnergySplitBelow ? 1
                                                             : (2 * kNumCU + (int)grid.x - 1) / (int)grid.x;
    int rows = rows_wanted < units ? rows_wanted : units;
    if (rows > kEnergySplitRows) rows = kEnergySplitRows;
    const bool by_rows = rows > 1 && m <= kEnergySplitSignals;
    int units_per_y = 0;
    if (by_rows) {
        units_per_y = (units + rows - 1) / rows;
        rows = (units + units_per_y - 1) / units_per_y;
        grid.y = rows;
    }
    int32_t* out_j = by_rows ? ws.part_j : blk;
    float* out_E = by_rows ? ws.part_E : ws.energy;
    int32_t* hist = by_rows ? nullptr : chunk_count;
    if (!split) {
        constexpr size_t lds = (size_t)2 * (2 * QN * 64) * sizeof(f32x4);
        if (lds > 64 * 1024) {
            if (hipError_t e = ws.raised->ensure(reinterpret_cast<const void*>(&energy_kernel<P, S, NT, SX>), lds);
                e != hipSuccess)
                return e;
        }
        hipLaunchKernelGGL((energy_kernel<P, S, NT, SX>), grid, dim3(256), lds, st, Y, (int)m,
                           reinterpret_cast<const f32x4*>(ws.dsw), K, s0, out_j, out_E, hist, chunk, units_per_y);
    } else if constexpr (wide) {
        // two stages of 32 rows + the partial-product exchange (2 x 4 SIMDs x 4 KiB)
        constexpr size_t lds = (size_t)2 * (P / 16) * 3 * 64 * 16 + (size_t)2 * 4 * 4 * 64 * 16;
        if (hipError_t e = ws.raised->ensure(reinterpret_cast<const void*>(&energy_split_wide_kernel<P, S, SX>), lds);
            e != hipSuccess)
            return e;
        hipLaunchKernelGGL((energy_split_wide_kernel<P, S, SX>), grid, dim3(64 * kWideWaves), lds, st, Y, (int)m,
                           reinterpret_cast<const u32x4*>(ws.dsb), K, s0, out_j, out_E, hist, chunk, units_per_y);
    } else if (arith == SBO_ARITH_F16X2) {
        hipLaunchKernelGGL((energy_split_kernel<P, S, SX, true>), grid, dim3(64 * kSplitWgWaves),
                           (SplitGeom<P, 2>::LDS), st, Y, (int)m, reinterpret_cast<const u32x4*>(ws.dsh), K, s0, out_j,
                           out_E, hist, chunk, units_per_y);
    } else {
        hipLaunchKernelGGL((energy_split_kernel<P, S, SX, false>), grid, dim3(64 * kSplitWgWaves),
                           (SplitGeom<P, 3>::LDS), st, Y, (int)m, reinterpret_cast<const u32x4*>(ws.dsb), K, s0, out_j,
                           out_E, hist, chunk, units_per_y);
    }
    if (by_rows)
        hipLaunchKernelGGL(energy_merge_kernel, dim3((unsigned)((m + 255) / 256)), dim3(256),
                           (size_t)K * sizeof(int), st, ws.part_E, ws.part_j, rows, (int)m, K, blk, ws.energy,
                           chunk_count, chunk);
    return hipGetLastError();
}

// p = 256: s0 in (S/2, S] is a compile-time constant of the kernel (the lane-pair fold then needs no sort)
template <int S>
hipError_t launch_wide_s(const float* Y, int64_t m, int K, int s0, int arith, const Workspace& ws, int32_t* blk,
                         int32_t* chunk_count, hipStream_t st) {
    switch (S - s0) {
#define SBO_CASE(DELTA)                                                                          \
    case DELTA:                                                                                  \
        if constexpr (S - DELTA > S / 2 || S == 1)                                               \
            return launch_pse<256, S, S - DELTA>(Y, m, K, s0, arith, ws, blk, chunk_count, st);  \
        break;
        SBO_CASE(0) SBO_CASE(1) SBO_CASE(2) SBO_CASE(3) SBO_CASE(4) SBO_CASE(5) SBO_CASE(6) SBO_CASE(7)
#undef SBO_CASE
        default: break;
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_dict_swizzle(int p, int K, const float* D, float* dsw, const CallStart& start, hipStream_t st) {
    f32x4* out = reinterpret_cast<f32x4*>(dsw);
    const dim3 grid((K * p + 63) / 64);
    switch (p) {
        case 16: hipLaunchKernelGGL((dict_swizzle_kernel<16>), grid, dim3(256), 0, st, D, K, out, start); break;
        case 32: hipLaunchKernelGGL((dict_swizzle_kernel<32>), grid, dim3(256), 0, st, D, K, out, start); break;
        case 64: hipLaunchKernelGGL((dict_swizzle_kernel<64>), grid, dim3(256), 0, st, D, K, out, start); break;
        case 256: hipLaunchKernelGGL((dict_swizzle_kernel<256>), grid, dim3(256), 0, st, D, K, out, start); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_dict_parts(int p, int K, const float* D, unsigned* dsb, unsigned* dsh, float2* dnorm, int* dodd, float2* dev,
                             const SignalSample& sample, const CallStart& start, hipStream_t st) {
    u32x4 *b = reinterpret_cast<u32x4*>(dsb), *h = reinterpret_cast<u32x4*>(dsh);
    float* dv = reinterpret_cast<float*>(dev);
    if (dev != nullptr && (p != 64 || dsh == nullptr)) return hipErrorInvalidValue;
    const unsigned stages = (unsigned)(K * p + 63) / 64;           // (the last one is filled up with zeros)
    switch (p) {
#define SBO_CASE(N) \
    case N: hipLaunchKernelGGL((dict_parts_kernel<N, false>), dim3(stages * (64 / dict_rows<N>())), dim3(256), 0, st, D, K, b, h, dnorm, dodd, dv, start, sample); break;
        SBO_CASE(16) SBO_CASE(32) SBO_CASE(256)
#undef SBO_CASE
        case 64: {
            const auto kernel = dev != nullptr ? &dict_parts_kernel<64, true> : &dict_parts_kernel<64, false>;
            hipLaunchKernelGGL(kernel, dim3(stages * (64 / dict_rows<64>())), dim3(256), 0, st, D, K, b, h, dnorm, dodd, dv, start, sample);
            break;
        }
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

bool guess_applies(int p, int K, int s0, int64_t m, int arith) {
    ScrArgs a;
    a.m = (int)m;
    a.K = K;
    a.s0 = s0;
    return p == 64 && screen_applies(p, K, s0, arith) && guess_takes_64(a);
}

static hipError_t launch_energy_screen(int p, int K, int s0, int arith, const float* Y, int64_t m, const Workspace& ws,
                                int32_t* blk, int32_t* chunk_count, int turn, bool orthobases, hipStream_t st) {
    if (!screen_applies(p, K, s0, arith) || ws.raised == nullptr) return hipErrorInvalidValue;
    ScrArgs a;
    a.Y = Y;
    a.m = (int)m;
    a.Dh = reinterpret_cast<const u32x4*>(ws.dsh);
    a.Dx = arith == SBO_ARITH_F16X2 ? (const void*)ws.dsh : arith == SBO_ARITH_F32 ? (const void*)ws.dsw : (const void*)ws.dsb;
    a.dnorm = ws.dnorm;
    a.K = K;
    a.s0 = s0;
    a.blk = blk;
    a.chunk_count = chunk_count;
    a.chunk = group_geom(m).chunk;
    a.short_cut = ws.short_cut;
    a.split_E = ws.split_E;
    a.split_room = ws.split_room;
    a.split_x = ws.split_x;
    a.split_done = ws.split_done;
    if (turn >= 0 && (p == 64 ? home_takes_64(a) : p == 256 && home_takes_256(a))) {
        a.weak = ws.weak;
        a.turn = turn;
        if (orthobases) {
            // The first iteration loads the kernel of the next ones (2.3 ms, once in a process: a program that has made one
            // iteration has made ready for more).
            ScrArgs home = a;
            home.load_only = turn == 0;
            home.perm = ws.perm;
            home.offsets = ws.offsets;
            home.sweeps = ws.sweeps;
            hipError_t e = p == 64 ? launch_home_64(home, arith, ws.raised, st) : launch_home_256(home, arith, ws.raised, st);
            if (turn > 0 || e != hipSuccess) return e;
        }
    }
    if (turn <= 0 && p == 64 && guess_takes_64(a)) {
        a.dev = ws.dev;
        a.sample = ws.sample;
        return launch_guess_64(a, arith, ws.raised, st);
    }
    switch (p) {
        case 16: return launch_screen_16(a, arith, ws.raised, st);
        case 32: return launch_screen_32(a, arith, ws.raised, st);
        case 64: return launch_screen_64(a, arith, ws.raised, st);
        case 256: return launch_screen_256(a, arith, ws.raised, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_energy_direct(int p, int K, int s0, int arith, const float* Y, int64_t m, const float* D,
                                const Workspace& ws, hipStream_t st) {
    if (!choose_in_select(p, K, s0, m, arith)) return hipErrorInvalidValue;
    ScrArgs a = {};
    a.Y = Y;
    a.m = (int)m;
    a.K = K;
    a.s0 = s0;
    a.D = D;
    a.E = ws.part_E;
    switch (p) {
        case 16: return launch_direct_16(a, arith, st);
        case 32: return launch_direct_32(a, arith, st);
        default: return launch_direct_64(a, arith, st);
    }
}

hipError_t launch_energy(int p, int K, int s0, int arith, const float* Y, int64_t m, const Workspace& ws, int32_t* blk,
                         int32_t* chunk_count, hipStream_t st, int turn, bool orthobases) {
    if (screen_applies(p, K, s0, arith))
        return launch_energy_screen(p, K, s0, arith, Y, m, ws, blk, chunk_count, turn, orthobases, st);
    if (p == 16) return launch_pse<16, 16, 0>(Y, m, K, s0, arith, ws, blk, chunk_count, st);
    if (p != 256) return hipErrorInvalidValue;
    if (s0 <= 1) return launch_wide_s<1>(Y, m, K, s0, arith, ws, blk, chunk_count, st);
    if (s0 <= 2) return launch_wide_s<2>(Y, m, K, s0, arith, ws, blk, chunk_count, st);
    if (s0 <= 4) return launch_wide_s<4>(Y, m, K, s0, arith, ws, blk, chunk_count, st);
    if (s0 <= 8) return launch_wide_s<8>(Y, m, K, s0, arith, ws, blk, chunk_count, st);
    return launch_wide_s<16>(Y, m, K, s0, arith, ws, blk, chunk_count, st);
}

}  // namespace sbo
