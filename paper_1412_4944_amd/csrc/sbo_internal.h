// Internal declarations shared by the libsbo translation units (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <stdlib.h>
#include <vector>

#include "../../include/sbo.h"

namespace sbo {

struct DictOps;                // device_utils.h

constexpr int kWave = 64;

// ---- grouping geometry -----------------------------------------------------
// One wavefront owns one chunk of consecutive signals; a chunk is a multiple of
// 64 signals, sized so that there are at most ~1024 chunks.
struct GroupGeom {
    int chunk;     // signals per chunk (multiple of 512)
    int n_chunks;  // ceil(m / chunk)
};
inline GroupGeom group_geom(int64_t m) {
    int64_t c = (m + 1023) / 1024;
    c = ((c + 511) / 512) * 512;           // whole workgroups of the coding kernels (128, 256 or 512 signals)
    if (c < 512) c = 512;
    GroupGeom g;
    g.chunk = (int)c;
    g.n_chunks = (int)((m + c - 1) / c);
    return g;
}

// ---- accumulation geometry ---------------------------------------------------
// Each block's sorted signal list is cut into pieces of `piece` signals; one
// workgroup reduces one piece into a partial p x p matrix.
constexpr int kNumCU = 256;
constexpr int kMinPiece = 64, kMaxPiece = 4096;
inline int accum_piece(int64_t m, int K) {
    // One workgroup per CU for every p (8 wavefronts with 150 KiB of LDS for p <= 64, 512
    // registers per lane for p = 256), and all pieces resident in one round: pieces <= CUs where
    // K allows.  At least 64 signals: p = 256, K = 1, 2048 signals with 256 / 128 / 64: accumulation 49 / 30 / 21 us,
    // SVD update that sums the pieces 135 / 139 / 142.
    const int target = K < kNumCU / 2 ? kNumCU - K : kNumCU / 2;
    int64_t c = (m + target - 1) / target;
    c = ((c + 63) / 64) * 64;
    if (c < kMinPiece) c = kMinPiece;
    if (c > kMaxPiece) c = kMaxPiece;
    return (int)c;
}
inline int accum_max_pieces(int64_t m, int K) {
    int piece = accum_piece(m, K);
    return (int)((m + piece - 1) / piece) + K;
}
// The pieces of launch_accumulate.  p = 256 on the bf16 matrix cores, small sets: slices of 64 dims, a workgroup each, of
// pieces that are up to four times as long; a quarter of the results to write and for the SVD to add up.  A step of a
// slice takes two thirds of a whole one's time, so it does not pay for long.  sbo_update, whole / sliced (us): K = 1, 600
// signals 119 / 112, 2048 96 / 90, 8192 113 / 93, 16384 119 / 102, 32768 136 / 114, 65536 157 / 136; K = 2, 16384 115 / 103, 49152 133 / 124; K = 4,
// 4096 115 / 110, 16384 112 / 103, 32768 123 / 117, 49152 133 / 130; K = 8, 16384 115 / 110, 32768 120 / 119; K = 16, 5041 219 / 214, 16384
// 154 / 152, 24576 152 / 150, 32768 151 / 152; K = 24, 16384 256 / 255, 24576 243 / 247; K = 32, 16384 290 / 290, 32768 257 / 267.
// So the line in K is where it stops to pay, and the one in m is on the safe side: with few blocks it would pay up to three or four times
// as many signals, for which the error of the longer sums has not been measured.
struct AccumGeom {
    int piece, max_pieces, slices;
};
constexpr int kAccumSlices = 4, kAccumSliceMaxK = 16;
constexpr int64_t kAccumSliceMaxSignals = 16384;
inline AccumGeom accum_geom(int p, int64_t m, int K, bool parts) {
    if (p != 256 || !parts || K > kAccumSliceMaxK || m > kAccumSliceMaxSignals) return {accum_piece(m, K), accum_max_pieces(m, K), 1};
    const int target = kNumCU / kAccumSlices - K;      // (a piece more per block, at most: all resident in one round)
    const int64_t c = ((m + target - 1) / target + 63) / 64 * 64;
    return {(int)c, (int)((m + c - 1) / c) + K, kAccumSlices};
}

// ---- Jacobi stopping threshold ---------------------------------------------------
// A sweep in which every pair already had a cosine below this is the last one.
constexpr float kPolarDone = 1e-4f;

// ---- kernels that need more dynamic LDS than the default limit ---------------------
// Their limit is raised once per context (a context belongs to one device and its calls do
// not overlap), before the first launch; the context remembers which kernels have been done.
struct LdsRaised {
    std::vector<const void*> fns;
    hipError_t ensure(const void* fn, size_t bytes) {
        for (const void* f : fns)
            if (f == fn) return hipSuccess;
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e == hipSuccess) fns.push_back(fn);
        return e;
    }
};

// Polls of one wait between the workgroups of a p = 256 SVD team: seconds.
constexpr int kWidePolls = 1 << 22;

// ---- device workspace layout ---------------------------------------------------
struct Workspace {
    // grouping
    int32_t* chunk_count;  // [n_chunks_max][K]
    int32_t* chunk_base;   // [n_chunks_max][K]
    int32_t* counts;       // [K]
    int32_t* offsets;      // [K+1]
    int32_t* perm;         // [m_max]
    int* weak;             // [3] signals that the dictionary represents badly, per iteration in turn (code_screen.h)
    int* short_cut;        // [ceil(m_max / 256)] per workgroup of a choice with home or guessed blocks: 1 where these decided
    int* group_done;       // [1] workgroups of the scatter that have read the histograms (0 between launches)
    // coding
    float* energy;         // [m_max] kept energy in the winning block
    float* dsw;            // [ceil(K*p/64)*64][p] dictionary in MFMA operand order
    unsigned* dsb;         // the same rows as three bf16 parts (6 bytes per entry)
    unsigned* dsh;         // the same rows as two fp16 parts (4 bytes per entry)
    float2* dnorm;         // [K*p/16] per 16 atoms: largest norm, largest norm of what the leading fp16 part leaves
    int* dodd;             // [K*p/16] p = 256: per 16 atoms, whether one is not well represented by fp16 parts (odd_norm2)
    float2* dev;           // [K] p = 64: |Q Q^T - I|_F^2 of a block, in two parts (guess_applies)
    unsigned* sample;      // [K][kSample / 32] p = 64: which of a sample of the signals a block represents
    float* part_E;         // [kEnergySplitRows][<= kEnergySplitSignals] split coding: best energy per row; or
                           // the energies of a small set, [K][m] (at most kDirectMaxEnergies)
    int32_t* part_j;       // same shape: its block
    unsigned* split_E;     // choice_split: [ceil(m / 64)][K][64 signals] 16 bits, the energies of all blocks
    int split_room;        // ... ceil(m / 64) * K at most
    unsigned* split_x;     // ... [kNumCU][4][64] what a workgroup found
    int* split_done;       // ... [kNumCU / 2] workgroups of a column that have finished (0 between launches)
    // accumulation
    float* partial;        // [max_pieces][p][p]
    float* M;              // [K][p][p]
    float* wide;           // p > 64 only: exchange memory of polar_wide.hip (polar_wide_scratch_bytes)
    int* wide_sync;        // p > 64 only: its counters (0 between launches)
    // eigenvectors of Gram matrices
    unsigned char* eig;    // [eig_room] x eigen_scratch_bytes, in the memory of `partial`
    int eig_room;          // matrices at a time (>= 1)
    int32_t* eig_left;     // [K] not 0: left to the Jacobi SVD
    // worst-W selection
    int32_t* sel_hist;     // [4][256] digit histograms of the radix select
    int32_t* sel_state;    // [4][2] (key prefix, entries still to take) after each pass
    int32_t* sel_cnt;      // [ceil(m_max / kSelChunk)][2] entries above / equal to the threshold
    int32_t* sel_base;     // same shape: exclusive sums of sel_cnt over the chunks
    int32_t* sweeps;       // [K] most recent SVD stage: Jacobi sweeps, or minus the Newton-Schulz steps
    int32_t* ns_fallback;  // [K] 1 = Newton-Schulz left the block to the Jacobi kernel
    int32_t* sq_counter;   // [1] workgroups of the fused squared-error sum that have finished (0 between launches)
    bool parts_accum = false;   // p = 256: the accumulation on the bf16 matrix cores (any coding arithmetic but fp32)
    // iterate
    double* sq_partial;    // [kSqBlocks]
    size_t bytes;
    // host side: launch state of the owning context (not device memory)
    LdsRaised* raised;
    int device;                            // that was current when the context was created
    int wide_polls = kWidePolls;           // p > 64: how long the workgroups of an SVD team wait for one another
    bool wide_helpers = true;              // p > 64: false (tests) = the second workgroups of pairs leave at once
};
constexpr int kSqBlocks = 256;
constexpr int kEnergySplitBelow = 192;       // coding launches with fewer workgroups split the blocks
constexpr int kEnergySplitRows = 16;         // at most this many workgroup rows
constexpr int kEnergySplitSignals = 49152;   // and only up to this many signals (scratch size)
constexpr int kSelChunk = 2048;              // signals per workgroup in the worst-W compaction

size_t workspace_layout(int p, int K, int s0, int64_t m_max, Workspace* ws, char* base);

}  // namespace sbo

struct sbo_span {
    int stage;
    hipEvent_t beg, end;
};

struct sbo_ctx {
    int p, K, s0;                    // K = blocks in use (<= K_cap, see sbo_set_blocks)
    int K_cap;                       // blocks the workspace was sized for
    int64_t m_max;
    hipStream_t stream;
    char* ws_base;
    sbo::Workspace ws;
    int svd_method;                  // SBO_SVD_AUTO or SBO_SVD_JACOBI (sbo_set_option)
    int coding_arith;                // SBO_ARITH_* (sbo_set_option)
    sbo::LdsRaised raised;
    int timing;
    std::vector<sbo_span> spans;     // event pool; the first n_spans are in use
    size_t n_spans;
    double* host_sq = nullptr;       // sbo_learn: the squared error on its way to the host (pinned), from the first call on,
    hipEvent_t sq_here = nullptr;    // and when it has arrived
};

// ---- kernel launchers (each returns a hipError_t from the launch) ----------------
namespace sbo {

// Operand orders of the dictionary that a coding arithmetic reads (bit mask).
constexpr int kOpsF32 = 1, kOpsBf16 = 2, kOpsF16 = 4;

// Which calls choose the block by screening with leading fp16 parts and full products for the
// contenders only (code_screen.h).  More than p / 2 coefficients kept: the blocks of a signal all but
// tie, and almost all of them would be contenders.  p = 256 in the other arithmetics: the full
// products of three bf16 parts do not fit the registers beside the screening; and with more blocks than
// kScreenWideMaxK the table of 64 signals (128 bytes a block) does not fit LDS beside them.
constexpr int kScreenWideMaxK = 1013;
constexpr bool screen_applies(int p, int K, int s0, int arith) {
    return 2 * s0 <= p && (p <= 64 || (arith == SBO_ARITH_F16X2 && K <= kScreenWideMaxK));
}
// Which shape of the screening kernel (p <= 64): workgroups of 256 signals, two per CU, instead of 512 where the
// last round of the latter would be at most 0.65 full (196608 signals, p = 64, K = 32: 141 us instead of 160); on
// full rounds they are equal, but with fewer signals per list of candidates the resolution costs more (262144
// signals, near-random dictionary: 164 us instead of 142).  The line was found at p = 64, K = 32 and depends on m
// alone; measured over K (trained dictionary), it costs up to 4 % at K >= 32.  Where a workgroup has fewer stages to
// multiply, 256 signals are better on full rounds too: p = 64, K = 4 393216 signals 48.5 us, by 256 41.3; K = 16
// 524288 signals 110.7, 100.9; p = 16, K = 32 393216 signals 46.0, 38.6.
constexpr bool screen_by_256(int64_t m) {
    const int64_t round = (int64_t)kNumCU * 512, rest = m % round;
    return rest != 0 && 20 * rest < 13 * round;
}
// And whether workgroups of 64 signals are better than both: the larger ones read the dictionary once for
// all of theirs and are up to 1.4 times as fast on a full chip, but their time is that of whole rounds.
// Measured, p = 64, K = 32, workgroups of 64 / 256: 32768 signals 55 / 61 us, 49152 69 / 65, 65536 84 / 71, 131072
// 145 / 107; p = 256, K = 16, 64 / 512: 81920 signals 385 / 394 us, 98304 466 / 446, 131072 603 / 527, 150000 675 /
// 738, 196608 853 / 823.  The lines depend on m alone.  Measured over K: within 9 % of the best shape at p = 64, K >= 32,
// and p = 256, K = 4 to 64; not at p = 64, K = 16 (40960 signals 26.7 us, by 256 22.0), and p = 16 and 32, which share the
// line of p = 256, are better with 64 signals for longer where K is large (p = 32, K = 128, 98304 signals 84.3 us,
// by 64 64.6) and with 256 for sooner where it is small (p = 16, K = 32, 163840 signals 30.7, 21.9).
constexpr bool screen_shared(int64_t m, bool p64_by_256) {
    const int64_t round = (int64_t)kNumCU * 512, rounds = (m + round - 1) / round;
    return p64_by_256 ? 5 * m < 2 * round : 20 * m < 13 * rounds * round;
}

// Screening by workgroups of 64 signals that leave at least half of the chip idle: the blocks are shared out among rows of
// workgroups, kSplitAtoms or more to each, and the one that finishes last decides.  The exchange takes 2 to 3 us: calls of
// sbo_code, 5041 signals, p = 256, s0 = 12, K = 16 59.6 -> 51, K = 32 86 -> 65; p = 64, s0 = 6, K = 64 31.7 -> 30.0, K = 200 60 -> 47; 600
// signals, p = 64, K = 200 49 -> 32.  (2048 atoms or more: up to 7 % slower where there is room for more rows.)  With p < 64 the steps saved
// are shorter than that: p = 32, K = 128 29.6 -> 30.5, p = 16, K = 64 18.5 -> 23.
constexpr int kSplitMaxSignals = kNumCU / 2 * 64, kSplitMaxK = 256, kSplitAtoms = 1024;
constexpr int choice_split(int p, int K, int64_t m) {
    const int columns = m <= kSplitMaxSignals ? (int)((m + 63) / 64) : kNumCU, parts = K * p / kSplitAtoms;
    const int rows = kNumCU / columns < parts ? kNumCU / columns : parts;
    return p >= 64 && K <= kSplitMaxK && rows > 1 ? rows : 1;
}

// Which calls of sbo_code leave the choice among full-precision energies to the select kernel (energy_direct_kernel): those
// whose grouping is left to it, with few energies, since every one of its workgroups compares those of all signals.
// sbo_code, screened / direct (us): K = 64, 512 signals p = 16 16.8 / 16.4, p = 32 20.1 / 18.3, p = 64 30.8 / 23.9; K = 32, 1024
// signals 17.9 / 17.8, 19.5 / 19.4, 26.4 / 25.2; K = 64, 1024 signals 18.5 / 24.6, 22.0 / 27.0, 32.8 / 34.3; fewer energies 3 to 12
// less (K = 4, 64 signals 13.4 / 9.8, 14.7 / 10.9, 18.7 / 15.2).  K = 96 up to 225 signals would gain too (p = 64 35 / 20.7), up to
// 512 not everywhere.
constexpr int kDirectMaxK = 64;
constexpr int64_t kDirectMaxEnergies = 32768;  // K m (and no more signals than group_in_select allows)
// Which iterations leave the grouping to the select + accumulate kernel, which calls of sbo_code to the select kernel and which of
// sbo_update (after the histogram kernel) to the accumulation, whose workgroups list the signals of their own piece (ChunkLists in
// device_utils.h).  The histograms are read by every workgroup, a piece of a block comes from K times as many signals, and that of a
// rare block from as many chunks as it has signals: the gain depends on how even the blocks are.  With a grouping launch / lists (us),
// blocks taken evenly, by Zipf(1.1), by Zipf(2):
//   sbo_code     p = 64, K = 32 32000 signals 44 / 37, 45 / 40, 45 / 44, 65000 60 / 52, 59 / 55, 62 / 60, 81000 73 / 66, 71 / 68, 71 / 71, 131000
//                79 / 75, 81 / 81, 81 / 87; K = 16 65000 45 / 40, 45 / 41, 46 / 48, 131000 64 / 60, 64 / 63, 63 / 72; p = 16, K = 16 65000 27 / 23, 27 / 24,
//                27 / 28, 81000 31 / 28, 31 / 29, 30 / 33, 131000 29 / 32, 29 / 33, 29 / 37; p = 32, K = 64 65000 47 / 39
//   sbo_update   p = 64, K = 32 65000 48 / 41, 54 / 49; p = 32, K = 16 65000 29 / 25, 33 / 29, 38 / 38, 81000 31 / 28, 36 / 33, 40 / 43, 131000
//                35 / 32, 38 / 37, 41 / 48; p = 16, K = 32 81000 30 / 25, 32 / 32, 36 / 37, 98000 32 / 28, 33 / 35, 36 / 39
//   an iteration p = 64, K = 32 48000 77 / 71, 84 / 81; p = 32, K = 32 81000 51 / 47, 55 / 54, 63 / 64, 98000 57 / 54, 62 / 63, 68 / 71; p = 16,
//                K = 64 65000 45 / 39
// and where all blocks but one have 300 signals at most 5 more up to 81000, 8 to 13 at 131000: up to 160 chunks what even blocks gain is
// at least what the most uneven ones lose.  With up to 8 blocks it takes more than Zipf(2) to make one
// so rare: 256 chunks (the largest sets measured).  126800 signals, evenly, Zipf(1.1), (2), (3): K = 5 sbo_code p = 32 36 / 34, 36 / 34, 36 / 34, 36 / 37,
// sbo_update p = 16 32 / 28, 35 / 32, 39 / 36, 40 / 41, an iteration p = 32 47 / 43, 52 / 47, 54 / 51, 56 / 60; K = 8 sbo_code p = 64 56 / 52, 55 / 53,
// 56 / 54, 53 / 61, sbo_update p = 16 32 / 28, 35 / 31, 39 / 40, 40 / 47, an iteration p = 16 39 / 36, 42 / 39, 47 / 47, 49 / 55; K = 12 sbo_code p = 64
// 60 / 57, 60 / 57, 60 / 63, sbo_update p = 16 33 / 29, 34 / 31, 38 / 44.
// More entries than 9216: K = 64 100003 signals (p = 32) 68.9 / 74.5 evenly, K = 128 40000 49.4 /
// 49.8; iterations with K > 128: 4096, where it was measured (sbo_code with K = 200 loses beyond).  p = 256, sbo_code, K = 16
// 16000 signals 94 / 87, 65000 264 / 262, 100003 337 / 341.  Iterations at p = 64: as long as none takes its signals in the
// order of the grouping (home blocks: workgroups of more than 64 signals).  sbo_code of 1025 to 2048 signals would gain 4 to 7 us
// (K = 4 to 128, every p), but the time of the grouping stage there is one that callers get to read.
constexpr int64_t list_signals(int K) { return (K <= 8 ? 256 : 160) * 512; }
inline bool few_entries(int K, int64_t m) { return (int64_t)((m + 511) / 512 + 8) * K <= (K <= 128 ? 9216 : 4096); }
inline bool lists_in_round(int p, int K, int64_t m) {
    return p <= 64 && m <= list_signals(K) && (p < 64 || screen_shared(m, true)) && few_entries(K, m);
}
inline bool lists_in_select(int p, int K, int64_t m) {
    return m > 2048 && m <= (p <= 64 ? list_signals(K) : 65536) && K <= 128 && few_entries(K, m);
}
inline bool lists_in_update(int p, int K, int64_t m) { return p <= 64 && K <= 128 && m <= list_signals(K) && few_entries(K, m); }
inline bool group_in_select(int p, int K, int64_t m) { return p <= 64 && K <= 256 && m <= 1024; }
inline bool choose_in_select(int p, int K, int s0, int64_t m, int arith) {
    return group_in_select(p, K, m) && K <= kDirectMaxK && K * m <= kDirectMaxEnergies && screen_applies(p, K, s0, arith);
}

// What the first launch of a call that codes signals also does: the counts and histograms that the next ones add to are set
// to zero.
struct CallStart {
    int* weak = nullptr;           // ws.weak: its first count
    int32_t* hist = nullptr;       // ws.chunk_count: the first n_hist entries
    int n_hist = 0;
    // 256 threads (blockDim would be a trip to memory before everything else)
    __device__ __forceinline__ void clear() const {
        if (weak != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *weak = 0;
        for (int e = blockIdx.x * 256 + threadIdx.x; e < n_hist; e += gridDim.x * 256) hist[e] = 0;
    }
};
// dsw = D in the fp32 operand order of the coding kernels.
hipError_t launch_dict_swizzle(int p, int K, const float* D, float* dsw, const CallStart& start, hipStream_t st);
// A sample of the signals tells whether it is worth guessing blocks: kSample of them, evenly spaced, and per block which of them it
// represents (code_screen.h), a bit each.  The launch that writes the dictionary's operand order finds out.
constexpr int kSample = 256;
struct SignalSample {
    const float* Y = nullptr;
    int m = 0;
    unsigned* mask = nullptr;      // ws.sample
};
// dsb / dsh (either may be nullptr) = D as three bf16 / two fp16 parts per entry in operand order
// (device_utils.h); dnorm, and at p = 256 dodd, come with dsh.  dev (or nullptr; p = 64, dsh given): |Q Q^T - I|_F^2 per block, and the
// sample of the m signals of Y (m >= kSample).
hipError_t launch_dict_parts(int p, int K, const float* D, unsigned* dsb, unsigned* dsh, float2* dnorm, int* dodd, float2* dev,
                             const SignalSample& sample, const CallStart& start, hipStream_t st);
// Whether the block choice of a first pass (turn <= 0 of launch_energy) reads ws.dev and ws.sample.
bool guess_applies(int p, int K, int s0, int64_t m, int arith);
// The block of every signal, from the operand orders in ws that (p, s0, arith) reads (energy_ops in
// sbo_api.hip).
// chunk_count != nullptr: also add the per-chunk histograms of the chosen blocks into it (the
// first step of launch_group; the array must be zero on entry, launch_group leaves it so).
// turn: the iteration (0, 1, ...) of sbo_iterate on the same signals, or -1; orthobases: the blocks were updated by Newton-Schulz
// where ws.sweeps says so.  From turn 1 on the last grouping in ws tells where every signal comes from, and large sets are
// coded with home blocks (code_screen.h).  The blocks chosen are the same.
hipError_t launch_energy(int p, int K, int s0, int arith, const float* Y, int64_t m, const Workspace& ws, int32_t* blk,
                         int32_t* chunk_count, hipStream_t st, int turn = -1, bool orthobases = false);

// Small sets (choose_in_select): ws.part_E[j * m + i] = the energy of signal i in block j, for launch_select.
hipError_t launch_energy_direct(int p, int K, int s0, int arith, const float* Y, int64_t m, const float* D,
                                const Workspace& ws, hipStream_t st);

hipError_t launch_group(int K, const int32_t* blk, int64_t m, const Workspace& ws, bool have_hist,
                        hipStream_t st);
// Its first launch alone: the chunk histograms.
hipError_t launch_group_hist(int K, const int32_t* blk, int64_t m, const Workspace& ws, hipStream_t st);
// The grouping with its scratch in a static device array (no workspace, no allocation).
constexpr int kGroupStaticMaxK = 128;
constexpr int64_t kGroupStaticMaxM = (int64_t)1 << 20;
hipError_t launch_group_static(int K, const int32_t* blk, int64_t m, int32_t* counts, int32_t* offsets,
                               int32_t* perm, hipStream_t st);

// p = 256 reads Q in operand order, `ops`: ws.dsh (kOpsF16), ws.dsb (kOpsBf16) or ws.dsw (kOpsF32: the fp32 matrix
// instruction).  ops_valid: that buffer already holds this D (launch_dict_parts, launch_dict_swizzle, the SVD update);
// otherwise it is rewritten first.  kOpsF16: for entries below 8 (device_utils.h).  p <= 64 reads D itself; of `ops` it only takes
// whether it is kOpsF32.
// blk: nullptr, or the choices of signals that have not been grouped (where group_in_select says so; the histograms in
// ws.chunk_count are set to zero, as launch_group would).  The line: every workgroup reads the whole set, so it has to be
// small, and has to fit 64 KiB of LDS beside the tiles.
// choose: blk is written first, from the energies in ws.part_E (launch_energy_direct).
// by_pos (p = 256): the codes of the signal at position q of ws.perm go to row q, not to the row of the signal: where a
// signal is in several blocks (sbo_learn's initial sets).  launch_accumulate reads them likewise.
// lists: blk likewise, where lists_in_select says so; the histograms are left as they are, and nothing of what launch_group
// leaves.
hipError_t launch_select(int p, int K, int s0, const float* Y, int64_t m, const float* D,
                         const Workspace& ws, int32_t* supp, float* coef, float* err, bool ops_valid,
                         int ops, hipStream_t st, int32_t* blk = nullptr, bool choose = false, bool by_pos = false,
                         bool lists = false);

// M == nullptr: the pieces stay in ws.partial (cut as accum_geom(p, m, K, ws.parts_accum) says), for launch_polar_from_pieces.  blk (M == nullptr, where
// lists_in_update says so): as for launch_select_accum.
hipError_t launch_accumulate(int p, int K, int s0, const float* Y, int64_t m, const int32_t* supp,
                             const float* coef, const Workspace& ws, float* M, hipStream_t st, bool by_pos = false,
                            const int32_t* blk = nullptr);

// Fused select + per-piece accumulation (p <= 64); the piece results land in ws.partial
// and launch_accum_reduce sums them into M.  blk: nullptr, or the choices of signals that have not been grouped, with their
// histograms in ws.chunk_count (where lists_in_round says so; the launch after sets them to zero); ws.counts and ws.offsets are
// left as launch_group would leave them, ws.perm is not.
hipError_t launch_select_accum(int p, int K, int s0, const float* Y, int64_t m, const float* D,
                               const Workspace& ws, int32_t* supp, float* coef, float* err,
                               hipStream_t st, const int32_t* blk = nullptr);
// err, sq_out != nullptr: the same launch also forms *sq_out = sum of err[0..m).
hipError_t launch_accum_reduce(int p, int K, int64_t m, const Workspace& ws, float* M,
                               const float* err, double* sq_out, hipStream_t st);

// The SVD update Q_j = U V^T of every block with counts[j] > 0 (counts == nullptr: all).
// Newton-Schulz on the matrix cores (polar_ns.hip; p = 256: polar_wide.hip), in the same launch the
// Jacobi SVD for the blocks on which it does not converge (rank-deficient ones).
// jacobi_only != 0: the Jacobi SVD for every block (SBO_SVD_JACOBI).
// Uses ws.wide and ws.wide_sync (p = 256), ws.sweeps (per block: Jacobi sweeps, or minus the
// Newton-Schulz steps), ws.ns_fallback.
// eig_sv != nullptr switches to eigen mode: M[j] symmetric positive semidefinite, D[j] receives its
// eigenvectors as atoms by descending eigenvalue and eig_sv[j][p] the square roots of the eigenvalues
// (launch_eigen, then Jacobi for the matrices that it leaves; jacobi_only: Jacobi for all of them).
// write_ops: the operand orders (kOps*) in which the rows of every updated block are also left in
// ws (not in eigen mode).
hipError_t launch_polar(int p, int K, const float* M, const int32_t* counts, float* D,
                        const Workspace& ws, int jacobi_only, float* eig_sv, int write_ops,
                        hipStream_t st);

// Eigenvectors by tridiagonalisation (eigen.hip), as eigen mode above; ws.eig_left[j] != 0 where D[j] and sv[j] are
// not to be used.  Overwrites ws.partial.
size_t eigen_scratch_bytes(int p);
hipError_t launch_eigen(int p, int K, const float* M, float* D, float* sv, const Workspace& ws, hipStream_t st);

// Total squared error riding along in a launch (sq_total.h): out == nullptr = none.
struct SqTotalArgs {
    const float* err = nullptr;
    int64_t m = 0;
    double* part = nullptr;     // ws.sq_partial
    int* counter = nullptr;     // ws.sq_counter (zero between launches)
    double* out = nullptr;
    int nb = 0;                 // workgroups (<= kSqBlocks)
};
// Newton-Schulz for p <= 64 with the Jacobi SVD in the same workgroup for a block that does not
// converge.  M == nullptr: P_j = the sum of block j's pieces in `partial` (fused select +
// accumulate, cut from `offsets` with `piece` signals per piece).
hipError_t launch_polar_ns(int p, int K, const float* M, const float* partial, const int32_t* offsets,
                           int piece, const int32_t* counts, float* D, const DictOps& ops,
                           int32_t* fallback, int32_t* iters, const SqTotalArgs& sq, LdsRaised* raised,
                           hipStream_t st, int32_t* clear = nullptr, int n_clear = 0);
// The SVD update straight from the piece results (launch_select_accum, or launch_accumulate
// without its sum; Newton-Schulz path): what launch_accum_reduce + launch_polar do, in one launch.
// err / sq_out as for launch_accum_reduce.  clear_lists (p <= 64): also sets the histograms to zero that launch_select_accum
// has read.
hipError_t launch_polar_from_pieces(int p, int K, int64_t m, float* D, const Workspace& ws, int write_ops,
                                    const float* err, double* sq_out, hipStream_t st, bool clear_lists = false);

// p = 256 (polar_wide.hip): source and squared-error total as launch_polar_ns; newton_schulz_first ==
// false or eig_sv != nullptr: the Jacobi SVD for every block.  And the sizes of ws.wide, ws.wide_sync.
size_t polar_wide_scratch_bytes(int K);
size_t polar_wide_sync_bytes(int K);
// Streams of a GPU with live contexts of p = 256 (how many of these launches may run at a time there).
int wide_streams(int device);
// Whether the SVD of K orthobases is made by teams of pairs (SBO_SVD_AUTO).
bool wide_pairs(int K, int device);
hipError_t launch_polar_wide(int K, const float* M, const float* partial, const int32_t* offsets, int piece,
                             const int32_t* counts, float* D, const DictOps& ops, bool newton_schulz_first,
                             float* eig_sv, const Workspace& ws, const SqTotalArgs& sq, hipStream_t st);

// ids == nullptr: sum over all m signals; otherwise over the m listed ones.
hipError_t launch_sqerr(const float* err, const int32_t* ids, int64_t m, const Workspace& ws,
                        double* out, hipStream_t st);

// A signal set as one block: ws.perm = ids clamped to [0, m), ws.counts = {n}, ws.offsets = {0, n}.
hipError_t launch_single_block(const int32_t* ids, int64_t n, int64_t m, const Workspace& ws,
                               hipStream_t st);

// n_blocks signal sets of per_block signals each (ids[n_blocks][per_block]) as K = n_blocks blocks:
// ws.perm = the ids clamped to [0, m), ws.counts[j] = per_block, ws.offsets[j] = j * per_block.
hipError_t launch_equal_blocks(const int32_t* ids, int n_blocks, int64_t per_block, int64_t m,
                               const Workspace& ws, hipStream_t st);

// G[j] = sum over the signals of block j (ws.perm / ws.offsets for K blocks, n signals in all)
// of y y^T.
hipError_t launch_gram(int p, int K, const float* Y, int64_t n, const Workspace& ws, float* G,
                       hipStream_t st);

// ids[0..W) = the W signals with the largest err (ties: lower index), ascending.
hipError_t launch_worst(const float* err, int64_t m, int64_t W, const Workspace& ws, int32_t* ids,
                        hipStream_t st, bool block = false);

}  // namespace sbo
