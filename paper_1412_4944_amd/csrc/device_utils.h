// Small device helpers shared by the libsbo kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sbo {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// Value held by the lane 32 positions away (the other half of the wavefront).
__device__ __forceinline__ float other_half(float x) { return __shfl_xor(x, 32, 64); }
__device__ __forceinline__ int other_half(int x) { return __shfl_xor(x, 32, 64); }

// ---- DPP lane exchanges (all lanes active, in-row patterns) ---------------------------
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
constexpr int kDppXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // lane i <-> 7 - i inside each group of 8
constexpr int kDppRowMirror = 0x140;  // lane i <-> 15 - i inside each row of 16

// Sum over aligned groups of G = 4, 8 or 16 lanes; every lane of the group receives the
// bitwise identical total.
template <int G>
__device__ __forceinline__ float group_sum(float x) {
    x += dpp_f<kDppXor1>(x);
    x += dpp_f<kDppXor2>(x);
    if constexpr (G >= 8) x += dpp_f<kDppHalfMirror>(x);
    if constexpr (G == 16) x += dpp_f<kDppRowMirror>(x);
    return x;
}

// ---- fp32 as a sum of three bf16 -------------------------------------------------------
// v = hi + mid + lo exactly: each part is the bf16 nearest to what the parts before it leave
// (3 x 8 significand bits plus the signs of the remainders cover the 24 bits of fp32; the two
// subtractions are exact).  Two values at a time, packed as the matrix cores take them
// (first value in the low half of the word).  With a = a_hi + a_mid + a_lo and likewise b,
// a * b = hi*hi + (hi*mid + mid*hi) + (hi*lo + mid*mid + lo*hi) + terms below 2^-24 |a b|,
// every product of two bf16 being exact in fp32: six bf16 matrix products with fp32
// accumulation reproduce an fp32 contraction to fp32 accuracy.
struct Bf16x3Pair {
    unsigned hi, mid, lo;
};
__device__ __forceinline__ unsigned pack_bf16(float v0, float v1) {
    const bf16x2 t = {(__bf16)v0, (__bf16)v1};           // v_cvt_pk_bf16_f32: round to nearest even
    unsigned r = __builtin_bit_cast(unsigned, t);
    asm("" : "+v"(r));                                   // or v0 is converted once more for each use of its half
    return r;
}
__device__ __forceinline__ Bf16x3Pair split_bf16x3(float v0, float v1) {
    Bf16x3Pair r;
    r.hi = pack_bf16(v0, v1);
    const float a0 = v0 - __builtin_bit_cast(float, r.hi << 16);
    const float a1 = v1 - __builtin_bit_cast(float, r.hi & 0xffff0000u);
    r.mid = pack_bf16(a0, a1);
    const float b0 = a0 - __builtin_bit_cast(float, r.mid << 16);
    const float b1 = a1 - __builtin_bit_cast(float, r.mid & 0xffff0000u);
    r.lo = pack_bf16(b0, b1);
    return r;
}

// The same decomposition by truncation (8 + 8 + 8 significand bits), one value at a time: three
// words whose upper halves are bf16 numbers with hi + mid + lo = v exactly.
struct TriWord {
    unsigned hi, mid, lo;
};
__device__ __forceinline__ TriWord split_trunc(float v) {
    TriWord t;
    t.hi = __builtin_bit_cast(unsigned, v) & 0xffff0000u;
    const float r1 = v - __builtin_bit_cast(float, t.hi);
    t.mid = __builtin_bit_cast(unsigned, r1) & 0xffff0000u;
    const float r2 = r1 - __builtin_bit_cast(float, t.mid);
    t.lo = __builtin_bit_cast(unsigned, r2);             // at most 8 significant bits are left
    return t;
}

// Byte offset of bf16 element (row, col) in a transposed MFMA operand tile [row][16 signals]: rows
// of 32 bytes = two 16-byte units; the unit index is flipped on every other group of four rows so
// that the eight rows a quarter-wavefront reads at once cover all LDS banks.
__device__ __forceinline__ int tr_off(int row, int col) {
    return row * 32 + ((((col >> 3) ^ (row >> 2)) & 1) << 4) + (col & 7) * 2;
}

// ---- fp32 as a sum of two fp16 ------------------------------------------------------------
// For v scaled by a power of two so that |v| < 2^15: v = hi + lo + r with hi the fp16 nearest
// to v, lo the fp16 nearest to v - hi (exact in fp32) and |r| <= 2^-22 |v| (11 + 11 significand
// bits; lo is a normal fp16 unless |v| < 2^-3, where its absolute error 2^-25 is below 2^-39 of
// the largest entry).  a * b = hi*hi + hi*lo + lo*hi + terms below 3 * 2^-22 |a b|, every
// product of two fp16 being exact in fp32: three fp16 matrix products with fp32 accumulation
// give a contraction whose error per term, 3 * 2^-22 |a b|, is below the p * 2^-24 sum |a b|
// that an fp32 dot product of p >= 16 terms guarantees.
struct F16x2Pair {
    unsigned hi, lo;
};
__device__ __forceinline__ unsigned pack_f16(float v0, float v1) {
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    const f16x2 t = {(_Float16)v0, (_Float16)v1};        // round to nearest even
    return __builtin_bit_cast(unsigned, t);
}
// FINITE: magnitudes from 65520 on, which round to infinity, have the largest number as their first part; the second one takes the rest
// (below 32 for magnitudes below 65536).
template <bool FINITE = false>
__device__ __forceinline__ F16x2Pair split_f16x2(float v0, float v1) {
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    F16x2Pair r;
    r.hi = pack_f16(v0, v1);
    if constexpr (FINITE) {
        const f16x2 largest = {(_Float16)65504.f, (_Float16)65504.f};
        const f16x2 t = __builtin_elementwise_max(__builtin_elementwise_min(__builtin_bit_cast(f16x2, r.hi), largest), -largest);
        r.hi = __builtin_bit_cast(unsigned, t);
    }
    // v - 1 * hi with a one and a packed hi that the compiler does not see through: v_fma_mix_f32 reads the halves as they
    // are, four instructions a pair (eight: both values rounded apart, unpacked and subtracted)
    float one = 1.f;
    asm("" : "+s"(one));
    unsigned hi = r.hi;
    asm("" : "+v"(hi));
    const f16x2 h = __builtin_bit_cast(f16x2, hi);
    r.hi = hi;
    r.lo = pack_f16(fmaf(-(float)h[0], one, v0), fmaf(-(float)h[1], one, v1));
    return r;
}
// Dictionary entries (|q| <= 1 for orthonormal atoms; anything below 8 is representable) are
// scaled by this before the split.
constexpr float kF16DictScale = 8192.f;
// Power of two that brings a signal whose largest magnitude is vmax into [2^13, 2^14).  1 for a
// zero or non-finite signal and for one below 2^-63: its energies (squares of its coefficients)
// underflow in fp32 whatever the arithmetic, and all its parts then round to zero.
__device__ __forceinline__ float f16_signal_scale(float vmax) {
    const unsigned e = (__builtin_bit_cast(unsigned, vmax) >> 23) & 0xffu;      // biased exponent
    if (e < 64u || e == 0xffu) return 1.f;
    return __builtin_bit_cast(float, (unsigned)(127 + 13 + 127 - (int)e) << 23);   // 2^(13 - (e - 127))
}

// ---- the dictionary in the coding kernels' operand orders --------------------------------
// Rows = atoms of all blocks (row j*P + k = atom k of Q_j), in stages of 64 rows, each stage a
// run of 16-byte units in exactly the order the lanes of a wavefront consume the MFMA A operand
// (row = stage*64 + mt*32 + nn, lane = hh*32 + nn):
//   fp32 order : unit (mt*(P/8) + q)*64 + lane        = dims hh*P/2 + 4q .. +3 of the row
//   split order: unit ((mt*(P/16) + ks)*3 + pl)*64 + lane = the 8 bf16 of part pl (0 hi, 1 mid,
//                2 lo) of dims ks*16 + hh*8 .. +7 of the row
//   fp16 order : unit ((mt*(P/16) + ks)*2 + pl)*64 + lane = the 8 fp16 of part pl (0 hi, 1 lo) of
//                the same dims, entries scaled by kF16DictScale
// These store the four dims 4*d4 .. 4*d4+3 of row `grow`.
template <int P>
__device__ __forceinline__ void store_operand_f32(float* __restrict__ dsw, int grow, int d4, f32x4 row) {
    constexpr int QN = P / 8;
    const int st = grow >> 6, mt = (grow >> 5) & 1, nn = grow & 31;
    const int hh = d4 / QN, q = d4 % QN;
    reinterpret_cast<f32x4*>(dsw)[(int64_t)st * (2 * QN * 64) + (mt * QN + q) * 64 + hh * 32 + nn] = row;
}
template <int P>
__device__ __forceinline__ void store_operand_split(unsigned* __restrict__ dsb, int grow, int d4, f32x4 row) {
    constexpr int KS16 = P / 16;
    const int st = grow >> 6, mt = (grow >> 5) & 1, nn = grow & 31;
    const int ks = d4 >> 2, hh = (d4 >> 1) & 1, half = d4 & 1;
    const Bf16x3Pair a = split_bf16x3(row.x, row.y), b = split_bf16x3(row.z, row.w);
    u32x2* out = reinterpret_cast<u32x2*>(dsb) +
                 ((int64_t)st * (2 * KS16 * 3 * 64) + (int64_t)((mt * KS16 + ks) * 3) * 64 + hh * 32 + nn) * 2 + half;
    out[0] = u32x2{a.hi, b.hi};
    out[2 * 64] = u32x2{a.mid, b.mid};
    out[4 * 64] = u32x2{a.lo, b.lo};
}

// Four dims of a dictionary row as two fp16 parts, scaled by kF16DictScale; q2 / r2 += their squares and
// those of what the leading part leaves (both unscaled).
struct F16x2Quad {
    u32x2 hi, lo;
};
__device__ __forceinline__ F16x2Quad split_f16x2_dict(f32x4 row, float& q2, float& r2) {
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    constexpr float sc = kF16DictScale, inv = 1.f / kF16DictScale;
    const F16x2Pair a = split_f16x2<true>(row.x * sc, row.y * sc), b = split_f16x2<true>(row.z * sc, row.w * sc);
    const f16x2 ha = __builtin_bit_cast(f16x2, a.hi), hb = __builtin_bit_cast(f16x2, b.hi);
    const f32x4 rem = {row.x - (float)ha[0] * inv, row.y - (float)ha[1] * inv, row.z - (float)hb[0] * inv,
                       row.w - (float)hb[1] * inv};
    q2 += row.x * row.x + row.y * row.y + row.z * row.z + row.w * row.w;
    r2 += rem.x * rem.x + rem.y * rem.y + rem.z * rem.z + rem.w * rem.w;
    return {u32x2{a.hi, b.hi}, u32x2{a.lo, b.lo}};
}
// An atom of this squared norm is not well represented by those parts: below 1/16 its entries reach into fp16's smallest numbers (above,
// these cost 2^-34 of the norm at most), from 4 on they may leave its range.
__device__ __forceinline__ bool odd_norm2(float q2) { return !(q2 >= 1.f / 256 && q2 < 16.f); }
template <int P>
__device__ __forceinline__ void store_operand_f16x2(unsigned* __restrict__ dsh, int grow, int d4, F16x2Quad q) {
    constexpr int KS16 = P / 16;
    const int st = grow >> 6, mt = (grow >> 5) & 1, nn = grow & 31;
    const int ks = d4 >> 2, hh = (d4 >> 1) & 1, half = d4 & 1;
    u32x2* out = reinterpret_cast<u32x2*>(dsh) +
                 ((int64_t)st * (2 * KS16 * 2 * 64) + (int64_t)((mt * KS16 + ks) * 2) * 64 + hh * 32 + nn) * 2 + half;
    out[0] = q.hi;
    out[2 * 64] = q.lo;
}
// Where a kernel that writes dictionary rows also leaves them in the coding kernels' operand orders
// (nullptr: not wanted).
struct DictOps {
    float* f32 = nullptr;       // fp32 order
    unsigned* bf16 = nullptr;   // three bf16 parts
    unsigned* f16 = nullptr;    // two fp16 parts, and with them
    float2* dnorm = nullptr;    // per 16 atoms: largest norm, largest norm of what the leading fp16 part leaves
    int* dodd = nullptr;        // per 16 atoms (p = 256): one has a norm far from an orthobase's (odd_norm2)
};
// Maximum over the 16 lanes of a row, in all of them.
__device__ __forceinline__ float row16_max(float x) {
    x = fmaxf(x, dpp_f<kDppXor1>(x));
    x = fmaxf(x, dpp_f<kDppXor2>(x));
    x = fmaxf(x, dpp_f<kDppHalfMirror>(x));
    return fmaxf(x, dpp_f<kDppRowMirror>(x));
}

// Workgroup-wide exclusive scan of n <= 4 * blockDim.x integers produced by f(idx).
// out (LDS) receives n + 1 entries (out[n] = total); tmp (LDS) needs 16 ints.
// Every thread of the workgroup must call this; ends with a barrier.
template <class F>
__device__ __forceinline__ void wg_exclusive_scan4(F f, int n, int* out, int* tmp) {
    const int t = threadIdx.x;
    const int lane = t & 63, wave = t >> 6;
    const int nwaves = (blockDim.x + 63) >> 6;
    int v[4];
    int s = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        int idx = 4 * t + e;
        v[e] = idx < n ? f(idx) : 0;
        s += v[e];
    }
    int incl = s;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    if (lane == 63) tmp[wave] = incl;
    __syncthreads();
    int base = 0, total = 0;
    for (int w = 0; w < nwaves; ++w) {
        int x = tmp[w];
        if (w < wave) base += x;
        total += x;
    }
    int ex = base + incl - s;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        int idx = 4 * t + e;
        if (idx < n) out[idx] = ex;
        ex += v[e];
    }
    if (t == 0) out[n] = total;
    __syncthreads();
}

// Inclusive sums over the lanes of a wavefront (all lanes active).
__device__ __forceinline__ int wave_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);        // row_shr 1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);        // row_bcast 15, 31
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

// Piece `id` of the signal lists of all K blocks, cut into pieces of `piece` signals, block by block (block j has
// ceil(count_of(j) / piece) of them).  Every wavefront for itself, all lanes active: no LDS, no barrier (a workgroup's scan
// into LDS and a search there: 3500 cycles of the start of select_accum_kernel, 1400 like this).
struct Piece {
    int j;                     // its block, -1: there is no such piece
    int rank, count;           // its first signal, in the block's list, and how many it has
    int before;                // signals of the blocks before
};
template <class F>
__device__ __forceinline__ Piece find_piece(F count_of, int K, int piece, int id) {
    const int lane = threadIdx.x & 63;
    int pieces = 0, signals = 0;               // of the blocks before
    for (int j0 = 0; j0 < K; j0 += 256) {
        int n[4];                              // on their way at once
#pragma unroll
        for (int u = 0; u < 4; ++u) n[u] = j0 + 64 * u + lane < K ? count_of(j0 + 64 * u + lane) : 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (j0 + 64 * u >= K) break;       // uniform
            const int np = (int)((unsigned)(n[u] + piece - 1) / (unsigned)piece);
            const int upto = wave_scan(np), in_list = wave_scan(n[u]), at = id - pieces - (upto - np);
            const unsigned long long here = __ballot(at >= 0 && at < np);
            if (here != 0ull) {                // uniform
                const int l = __builtin_ctzll(here);
                const int rank = __builtin_amdgcn_readlane(at, l) * piece, all = __builtin_amdgcn_readlane(n[u], l);
                return {j0 + 64 * u + l, rank, min(piece, all - rank), signals + __builtin_amdgcn_readlane(in_list - n[u], l)};
            }
            pieces += __builtin_amdgcn_readlane(upto, 63);
            signals += __builtin_amdgcn_readlane(in_list, 63);
        }
    }
    return {-1, 0, 0, 0};
}

// A grouping that has not been carried out: the choices and their histograms per chunk of kListChunk signals (group.hip),
// from which a workgroup of NW wavefronts lists the signals of its own piece, or a wavefront those of its own tile.  A workgroup
// reads all histograms, and the choices of the chunks that its piece comes from.  Another launch sets the histograms to zero
// (a count of the workgroups that have read them costs more than all the rest: 144 of them, one after the other, 4 us).
constexpr int kListChunk = 512;                // signals of a chunk
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4_any __attribute__((ext_vector_type(4), aligned(4)));     // (the caller's choices: any alignment of an int)
struct ChunkLists {
    const int32_t* blk;
    int m, n_chunks;
    const int32_t* chunk_count;            // [n_chunks][K]
    int32_t *counts, *offsets;             // [K], [K+1]: written by leave()

    // The histograms -> table (LDS, table_ints ints); all wavefronts, ends with a barrier.
    static constexpr int table_ints(int NW, int K, int n_chunks) { return (n_chunks + NW) * K; }
    template <int NW>
    __device__ __forceinline__ void load(int K, int* table) const {
        constexpr int A = 16;                  // on their way at once
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        int* part = table + n_chunks * K;      // [NW][K] sums over every NW-th chunk
        for (int j = lane; j < K; j += 64) {
            int s = 0;
            for (int c0 = wave; c0 < n_chunks; c0 += A * NW) {
                int v[A];
#pragma unroll
                for (int u = 0; u < A; ++u) v[u] = chunk_count[min(c0 + u * NW, n_chunks - 1) * K + j];
#pragma unroll
                for (int u = 0; u < A; ++u)
                    if (c0 + u * NW < n_chunks) {          // uniform
                        table[(c0 + u * NW) * K + j] = v[u];
                        s += v[u];
                    }
            }
            part[wave * K + j] = s;
        }
        __syncthreads();
    }
    template <int NW>
    __device__ __forceinline__ int count_of(int K, const int* table, int j) const {
        int s = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += table[(n_chunks + w) * K + j];
        return s;
    }
    // What the grouping would have left, but for the lists; one wavefront.
    template <int NW>
    __device__ __forceinline__ void leave(int K, const int* table) const {
        const int lane = threadIdx.x & 63;
        int before = 0;
        for (int j0 = 0; j0 < K; j0 += 64) {
            const int j = j0 + lane, n = j < K ? count_of<NW>(K, table, j) : 0, upto = before + wave_scan(n);
            if (j < K) {
                counts[j] = n;
                offsets[j + 1] = upto;
            }
            before = __builtin_amdgcn_readlane(upto, 63);
        }
        if (lane == 0) offsets[0] = 0;
    }
    // The signals of a piece, in order -> ids[pc.count] (LDS): those of the chunks c with c % STEP == first, four of them on
    // their way at a time.  One wavefront; STEP of them share out a piece.  A piece of a rare block comes from as many chunks as it
    // has signals, so that what a chunk costs decides: a trip to memory, eight loads and eight ballots each made it 0.4 us (sbo_code,
    // 131000 signals, all but 900 of them in one of four blocks, p = 32: 31 us by a grouping launch, 61 so, 45 as it is; loads
    // of eight neighbours by words 62: the lines that an instruction touches).
    template <int STEP>
    __device__ __forceinline__ void collect(int K, const int* table, const Piece& pc, int* ids, int first) const {
        constexpr int H = kListChunk / 256, G = 4;         // a lane's four neighbours at a time
        static_assert(64 % STEP == 0, "c0 is a multiple of STEP");
        const unsigned long long every = STEP == 1 ? ~0ull : ~0ull / ((1ull << (STEP & 63)) - 1) << first;
        const int lane = threadIdx.x & 63;
        int front = 0;                         // signals of the chunks before
        for (int c0 = 0; c0 < n_chunks && front < pc.rank + pc.count; c0 += 64) {          // uniform
            const int n = c0 + lane < n_chunks ? table[(c0 + lane) * K + pc.j] : 0, upto = front + wave_scan(n);
            unsigned long long mask = __ballot(n > 0 && upto - n < pc.rank + pc.count && upto > pc.rank) & every;
            while (mask != 0ull) {             // uniform
                i32x4 key[G][H];
                int i0[G], at[G];              // at: of the next one, in the piece
#pragma unroll
                for (int q = 0; q < G; ++q) {
                    i0[q] = -1;
                    if (mask == 0ull) continue;            // uniform
                    const int l = __builtin_ctzll(mask);
                    mask &= mask - 1;
                    i0[q] = (c0 + l) * kListChunk;
                    at[q] = __builtin_amdgcn_readlane(upto - n, l) - pc.rank;
                    const int own = i0[q] + lane * 4;
                    if (i0[q] + kListChunk <= m) {         // uniform
#pragma unroll
                        for (int u = 0; u < H; ++u) key[q][u] = *reinterpret_cast<const i32x4_any*>(blk + own + u * 256);
                    } else {                               // the last chunk
#pragma unroll
                        for (int u = 0; u < H; ++u)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const int i = own + u * 256 + e, k = blk[min(i, m - 1)];
                                key[q][u][e] = i < m ? k : -1;
                            }
                    }
                }
#pragma unroll
                for (int q = 0; q < G; ++q) {
                    if (i0[q] < 0) break;                  // uniform
                    unsigned here[H], count = 0u;          // which of the lane's own; how many, 16 bits each
#pragma unroll
                    for (int u = 0; u < H; ++u) {
                        here[u] = 0u;
#pragma unroll
                        for (int e = 3; e >= 0; --e) here[u] = here[u] * 2 + (key[q][u][e] == pc.j);
                        count |= (unsigned)__popc(here[u]) << (16 * u);
                    }
                    const unsigned all = (unsigned)wave_scan((int)count), before = all - count;
                    int to = at[q] + (int)(before & 0xffffu);
#pragma unroll
                    for (int u = 0; u < H; ++u) {
                        for (; here[u] != 0u; ++to, here[u] &= here[u] - 1)
                            if ((unsigned)to < (unsigned)pc.count) ids[to] = i0[q] + u * 256 + lane * 4 + __builtin_ctz(here[u]);
                        to = at[q] + (__builtin_amdgcn_readlane((int)all, 63) & 0xffff) + (int)(before >> 16);
                    }
                }
            }
            front = __builtin_amdgcn_readlane(upto, 63);
        }
    }
};
static_assert(kListChunk == 512, "collect: two halves");

// The keys of the 64 A signals from `at` on, A per lane (-1 past the end): all loads are on their way at once, where
// a loop of one load per 64 signals waits for each (group_scatter_kernel, 512 signals per wavefront, A = 8: 1024
// signals, K = 4 6.8 -> 5.4 us, 16384, K = 16 9.2 -> 7.4, 262144, K = 32 8.3 -> 6.3, with the load before the scan;
// in a loop that is not unrolled half of that).
template <int A>
__device__ __forceinline__ void load_keys(const int32_t* __restrict__ blk, int at, int end, int (&key)[A]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < A; ++u) {
        const int i = at + u * 64 + lane;
        key[u] = i < end ? blk[i] : -1;
    }
}
// One wavefront puts the signals [beg, end), in order, into the lists of their blocks: run[j] (LDS, its own) is
// where the next signal of block j goes in perm.  Ids outside [0, K) are dropped.  key: load_keys of beg.
template <int A>
__device__ __forceinline__ void scatter_chunk(const int32_t* __restrict__ blk, int (&key)[A], int beg, int end, int K,
                                              int* run, int32_t* perm) {
    const int lane = threadIdx.x & 63;
    int nbits = 0;
    while ((1 << nbits) < K) ++nbits;
    for (int at = beg; at < end; at += 64 * A) {
        int next[A];
        load_keys(blk, at + 64 * A, end, next);
#pragma unroll
        for (int u = 0; u < A; ++u) {
            if (at + u * 64 >= end) break;     // uniform
            int b = key[u];
            const bool valid = (unsigned)b < (unsigned)K;
            if (!valid) b = 0;
            // lanes holding the same block as this lane
            unsigned long long same = __ballot(valid);
            for (int bit = 0; bit < nbits; ++bit) {
                const bool one = (b >> bit) & 1;
                const unsigned long long bal = __ballot(valid && one);
                same &= one ? bal : ~bal;
            }
            const unsigned long long below = same & ((1ull << lane) - 1ull);
            const int rank = __popcll(below);
            int base = 0;
            if (valid) {
                base = run[b];
                perm[base + rank] = at + u * 64 + lane;
            }
            __builtin_amdgcn_wave_barrier();   // every lane has read run[] before a leader updates it
            if (valid && rank == 0) run[b] = base + __popcll(same);
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int u = 0; u < A; ++u) key[u] = next[u];
    }
}

// A small set that has not been grouped: every wavefront finds the signals of its own tile among all choices, in LDS.
struct GroupInKernel {
    int32_t* blk;              // the choices; written first where E is given
    int m;
    int32_t* chunk_count;      // the choice's histograms, which nobody needs: set to zero
    const float* E = nullptr;  // [K][m] energies to choose from
    static constexpr int kMostBlocks = 256;                // K at most (launcher)

    // The block of largest energy of every signal (the lowest on a tie), or the choices as they are -> choice[m]; their numbers ->
    // count[K]; N threads.
    template <int N>
    __device__ __forceinline__ void choose(int K, int* choice, int* count) const {
        constexpr int A = 32;                  // energies on their way at a time
        const int tid = threadIdx.x;
        for (int j = tid; j < K; j += N) count[j] = 0;
        __syncthreads();
        for (int i = tid; i < m; i += N) {
            int best = 0;
            if (E != nullptr) {                // uniform
                float top = -1.f;
                for (int j0 = 0; j0 < K; j0 += A) {
                    float e[A];
#pragma unroll
                    for (int a = 0; a < A; ++a) e[a] = E[(int64_t)min(j0 + a, K - 1) * m + i];     // (the last one again: no larger)
#pragma unroll
                    for (int a = 0; a < A; ++a) {
                        best = e[a] > top ? j0 + a : best;
                        top = fmaxf(top, e[a]);
                    }
                }
                if (blockIdx.x == 0) blk[i] = best;
            } else {
                best = blk[i];
            }
            choice[i] = best;
            if ((unsigned)best < (unsigned)K) atomicAdd(&count[best], 1);  // out-of-range ids are dropped
        }
        if (blockIdx.x == 0)
            for (int e = tid; e < (m + 511) / 512 * K; e += N) chunk_count[e] = 0;
        __syncthreads();
    }
    // The signals of a piece, in order -> ids[pc.count]; a wavefront.
    __device__ __forceinline__ void list(const int* choice, const Piece& pc, int* ids) const {
        const int lane = threadIdx.x & 63;
        int at = -pc.rank;                     // of the next one, in the piece
        for (int i0 = 0; i0 < m && at < pc.count; i0 += 64) {              // uniform
            const bool mine = choice[min(i0 + lane, m - 1)] == pc.j && i0 + lane < m;
            const unsigned long long mask = __ballot(mine);
            const int to = at + __popcll(mask & ((1ull << lane) - 1ull));
            if (mine && to >= 0 && to < pc.count) ids[to] = i0 + lane;
            at += __popcll(mask);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
};

// Largest j in [0, n) with start[j] <= x, for a non-decreasing start[0..n].
__host__ __device__ __forceinline__ int upper_slot(const int* start, int n, int x) {
    int lo = 0, hi = n;  // invariant: start[lo] <= x, answer in [lo, hi)
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (start[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// ---- compare-exchange networks on register arrays (descending order) ---------------
__host__ __device__ __forceinline__ void cmpx_desc(float& a, float& b) {
    float hi = fmaxf(a, b), lo = fminf(a, b);
    a = hi;
    b = lo;
}

// v is bitonic -> sorted descending.
template <int N>
__host__ __device__ __forceinline__ void bitonic_merge_desc(float (&v)[N]) {
#pragma unroll
    for (int half = N / 2; half >= 1; half >>= 1) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if ((i & half) == 0) cmpx_desc(v[i], v[i + half]);
        }
    }
}

// Full bitonic sorting network, descending.
template <int N>
__host__ __device__ __forceinline__ void bitonic_sort_desc(float (&v)[N]) {
#pragma unroll
    for (int k = 2; k <= N; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                int l = i ^ j;
                if (l > i) {
                    if ((i & k) == 0 || k == N) cmpx_desc(v[i], v[l]);
                    else cmpx_desc(v[l], v[i]);
                }
            }
        }
    }
}

// 19-comparator sorting network for 8 keys (descending).
__host__ __device__ __forceinline__ void sort8_desc(float (&v)[8]) {
    cmpx_desc(v[0], v[2]); cmpx_desc(v[1], v[3]); cmpx_desc(v[4], v[6]); cmpx_desc(v[5], v[7]);
    cmpx_desc(v[0], v[4]); cmpx_desc(v[1], v[5]); cmpx_desc(v[2], v[6]); cmpx_desc(v[3], v[7]);
    cmpx_desc(v[0], v[1]); cmpx_desc(v[2], v[3]); cmpx_desc(v[4], v[5]); cmpx_desc(v[6], v[7]);
    cmpx_desc(v[2], v[4]); cmpx_desc(v[3], v[5]);
    cmpx_desc(v[1], v[4]); cmpx_desc(v[3], v[6]);
    cmpx_desc(v[1], v[2]); cmpx_desc(v[3], v[4]); cmpx_desc(v[5], v[6]);
}

// Median of three (one instruction on the device).
__host__ __device__ __forceinline__ float med3(float a, float b, float c) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_fmed3f(a, b, c);
#else
    return fmaxf(fminf(a, b), fminf(fmaxf(a, b), c));
#endif
}

// Insertion sort as a network of three-input operations (descending): inserting d into the
// sorted v[0..n) gives max(v0, d), med3(v[i-1], d, v[i]) for 0 < i < n, min(v[n-1], d): n + 1
// independent instructions.  3 + 4 + ... + N operations in all (33 for 8 keys, against 38 for
// the 19-comparator network; 133 against 160 for 16 keys).
template <int N>
__host__ __device__ __forceinline__ void insertion_sort_desc(float (&v)[N]) {
    if constexpr (N == 2) {
        cmpx_desc(v[0], v[1]);
    } else if constexpr (N >= 3) {
        {
            const float a = v[0], b = v[1], c = v[2];
            v[0] = fmaxf(fmaxf(a, b), c);
            v[1] = med3(a, b, c);
            v[2] = fminf(fminf(a, b), c);
        }
#pragma unroll
        for (int n = 3; n < N; ++n) {
            const float d = v[n];
            float r[N];
            r[0] = fmaxf(v[0], d);
#pragma unroll
            for (int i = 1; i < n; ++i) r[i] = med3(v[i - 1], d, v[i]);
            r[n] = fminf(v[n - 1], d);
#pragma unroll
            for (int i = 0; i <= n; ++i) v[i] = r[i];
        }
    }
}

template <int N>
__host__ __device__ __forceinline__ void sort_desc(float (&v)[N]) {
    if constexpr (N <= 16) insertion_sort_desc<N>(v);
    else bitonic_sort_desc<N>(v);
}

// The L largest of x[0..NV), sorted descending (NV and L powers of two, L <= NV).
template <int NV, int L>
__host__ __device__ __forceinline__ void top_sorted(const float (&x)[NV], float (&out)[L]) {
#pragma unroll
    for (int i = 0; i < L; ++i) out[i] = x[i];
    sort_desc<L>(out);
#pragma unroll
    for (int g = 1; g < NV / L; ++g) {
        float t[L];
#pragma unroll
        for (int i = 0; i < L; ++i) t[i] = x[g * L + i];
        sort_desc<L>(t);
#pragma unroll
        for (int i = 0; i < L; ++i) out[i] = fmaxf(out[i], t[L - 1 - i]);
        bitonic_merge_desc<L>(out);
    }
}

}  // namespace sbo
