// Batched SVD update Q_j = U V^T (Algorithm 1, steps 6-7) for p = 256: a team of 16 workgroups per
// block (32 where there are eight blocks or fewer and no second stream, wide_pairs), one launch for everything.
//
// A 256 x 256 matrix in the three bf16 parts that fp32 accuracy takes is 384 KiB: more than the LDS of
// a CU, and one CU alone would need 80 us of matrix time for a block.  So 16 workgroups share a block
// and meet at barriers in memory (2-3 us each); the alternative, a launch per product, pays 5 us per
// launch and has to launch as many steps as the worst matrix might need.
//
//   Newton-Schulz (polar_ns.hip has the iteration and its last step, ns_scale.h the scaling).  A
//   workgroup owns a strip of 16 columns of X, in registers.  Per step it multiplies G = X^T X (its 16
//   columns), then X E (its 16 columns), at fp32 accuracy; the A operands are ALL of X, by
//   columns for the first product and by rows for the second, read straight from L2 in operand order,
//   each exactly once: every workgroup leaves its strip in both orders when it has updated it, in fp32 (whoever reads it
//   makes the parts: two thirds of their bytes), and that is the only exchange, hence one barrier per step (two in the
//   first and the last).  A wavefront
//   makes two 16 x 16 tiles of both products; its loads run four contraction steps ahead and through from
//   the first product into the second.
//
//   The products: three bf16 parts of an operand, six partial products, in the first step (whose input has no scale yet) and for
//   the G of a step that may be the last one; elsewhere two fp16 parts, scaled, and three.  What these leave out of G (2^-22 of an entry)
//   is symmetric and goes with the next step; in X E it is made up for by a rounding less, E being scaled by alpha.  |Q - Q64|_F / sqrt(p)
//   0.85 to 0.95 of what it was (block matrices of training rounds, 384 to 16384 signals); splits and matrix work of a step are halved.
//   (Together with the sums in teams and the first l of ns_scale.h 0.69 to 0.78; nearly axis-aligned singular vectors, where the
//   result's own rounding is most of it, 1.06 to 1.15.)
//
//   Up to eight blocks on one stream, a team on each XCD: two workgroups to a strip, one for the upper and one for the lower half of its rows,
//   which halves the operands that each of them reads.  They need each other's half of X, which comes with the barrier, and of E:
//   a number in memory says when it is there, and half of the contraction runs meanwhile.  The second workgroups are helpers: if
//   they have not come when the first are all there and have waited a little, these go on without (meet_pairs), so that a
//   launch needs no more of the chip at a time than one with teams of 16.  Sums are made in the same order in every case:
//   the same bits.
//
//   A block on which that does not converge (rank-deficient, zero, NaN), every block under
//   SBO_SVD_JACOBI, and the eigenvectors of a Gram matrix: one-sided Jacobi with eight of the
//   workgroups.  Columns in 16 sets of 16; a workgroup rotates all pairs of two sets (one set's columns of A
//   and V in registers, half a wavefront each, the other's in LDS), then the sets move on: all
//   pairs of sets in 15 rounds, seven of them keeping one of the two sets in place.  A set is
//   handed over through memory with a version number; there is no barrier but one per sweep.
//
// What bounds it: Newton-Schulz by the 512 KiB of operands per workgroup and step from L2 (30 bytes a cycle arrive at a CU, no
// more with one team on an XCD than with two, or with more loads on their way; pairs 256 KiB): of 17000 cycles a step 6500 are the
// first product, 4000 the second, 1250 E, 2400 what is left for others and the parts in LDS, 2600 the barrier; with pairs, of 12900 4500,
// 3500, 900, 1550 and 2000; a step that may be the last one 22700 and 17600.  (With three parts in all products 25000 and 18000: 11300, 9000
// and 2300 of them the products and the barrier, with pairs 7200, 6700 and 2500.)  K = 4 114 -> 80 us, K = 16 131 -> 120 (9 steps from a finished matrix): 103 with pairs alone; 88, 124 because the compiler
// took the operands' descriptor and offsets for different ones in every lane (a loop around every load) and a flat load among
// them waited for all of them; the rest by a barrier of flags that a wavefront reads at once, by loads that pass L1 by,
// instead of a counter, polled by atomics (5000 cycles with pairs).  Eight steps of operands on their way instead of four: 91 us (registers spilled, and half of
// the wavefronts get theirs late).  With two fp16 parts in most products
// K = 4 80 -> 70, K = 16 120 -> 91 (a step 5.6 and 6.9 us).
// With the three parts in memory (768 KiB) 138 -> 131 us in the same profile,
// K = 16; K = 4 no difference.  Jacobi by the vector ALU
// of eight CUs (16 rotations of 256 + 256 rows per workgroup at a time) and 15 hand-overs a sweep.  Jacobi is called, not inlined,
// where a block may need it after Newton-Schulz, whose operands take all registers (inlined: 100 of them spilled, K = 16 147 us
// instead of 130, with three parts; so is a pair team's way on without its helpers).  Since every product has a body for three parts and one for
// two, 17 registers a lane are spilled all the same, with pairs 61 (488 and 860 bytes of scratch, 400 of them the called Jacobi's); the norm and the smallest diagonal entry of a step share a barrier (130 -> 126).
// Measured: K = 16 inside sbo_iterate 347 us (a launch per product and step, fp32 matrix instruction,
// 20 steps enqueued, plus launches for the sum of the pieces, the Jacobi SVD that has nothing to do,
// the operand order and the squared error: 46 launches, 400 us) -> 126 us and nothing else; K = 1 in a
// first training round 300 -> 125 us; eigenvectors of a Gram matrix (10 sweeps) 12.1 -> 1.8 ms.
//
// Waiting on other workgroups: a launch has at most 16 teams of 16 workgroups (helpers not counted), one per CU, and workgroups
// start in order.  A launch that does not have the chip to itself can hold at most 15 workgroups of an
// incomplete team on an XCD (32 CUs), so two launches at a time always leave room for one to complete a
// team.  With contexts of this size on more than two streams the teams lie in consecutive workgroups instead
// ("spread": at most 15 waiting ones on the whole chip per launch, barriers of the slower kind).  That is about
// speed only: other processes or kernels may still hold the CUs that a team needs, so every wait is bounded
// (WideArgs::polls), a workgroup whose wait ends gives the team up (gone), and the workgroup that leaves the team
// last, which by then waits for nobody, computes from their sources all blocks that one of the 16 did not
// finish (jacobi_alone).  The result is what it would have been, up to rounding; sbo_svd_sweeps shows such a block
// as one of the Jacobi SVD.
#include "sbo_internal.h"
#include "device_utils.h"
#include "ns_scale.h"
#include "sq_total.h"

#include <type_traits>

namespace sbo {

namespace {

constexpr int P = 256;
constexpr int kTeam = 16;                      // workgroups per block, of as many columns each,
constexpr int kPairs = 32;                     // or two for each of these strips
constexpr int kJacTeam = 8;
constexpr int kMaxTeams = 16;                  // blocks at a time
constexpr int kMaxPairTeams = 8;               // with pairs: one team on each XCD
constexpr int kHelperPolls = 64;               // for the second workgroups of the pairs, when the first are all there (60 us)
constexpr int kNT = 512;
constexpr int kWaves = kNT / 64;
constexpr int kMaxSweeps = 24;
constexpr float kTol = 1e-6f;                  // rotate while |a_i . a_j| > kTol |a_i| |a_j|

constexpr int kImage = 8 * 3 * 1024;           // a strip as an operand, LDS: [contraction step][part][64 lanes][16 bytes]
constexpr int kShared = 8 * 2 * 1024;          // and in memory, in fp32: [contraction step][half][64 lanes][16 bytes]
constexpr int kLdStrip = P + 4;

// A team's memory
constexpr size_t kColAt = 0;                                   // [2][16 strips] by columns
constexpr size_t kRowAt = kColAt + 2 * (size_t)kTeam * kShared;        // [2][16 row tiles] by rows
constexpr size_t kEAt = kRowAt + 2 * (size_t)kTeam * kShared;  // [16 strips][8][64 lanes][16 bytes] fp16 parts of E
constexpr size_t kJaAt = kEAt + (size_t)kTeam * 8 * 1024;      // [256 columns][256] A
constexpr float kEScale = 8192.f;                              // of those: 1e-2 is in the middle of fp16's range
constexpr size_t kJvAt = kJaAt + (size_t)P * P * 4;            // V
// red[2][4][kCarried][32] | sigma[256] | 1/|v|[256] | pairs: sums of each half of the columns [2 halves][2][256]
constexpr size_t kSmallAt = kJvAt + (size_t)P * P * 4;
constexpr float kXScale = 16384.f;                             // of X after the first step, and of E for its product with X
constexpr int kCarried = 5;                                    // floats of each workgroup that a barrier carries
constexpr int kRedSize = 4 * kCarried * kPairs;
constexpr int kSmallFloats = 2 * kRedSize + 2 * P + 4 * P;
constexpr size_t kELoAt = (kSmallAt + kSmallFloats * 4 + 255) / 256 * 256;     // pairs: second fp16 parts of E, as the first at kEAt,
constexpr size_t kEHalfAt = kELoAt + (size_t)kTeam * 8 * 1024;                 // and E in fp32, [16 strips][16 tiles][64 lanes][16 bytes]
constexpr size_t kTeamBytes = kEHalfAt + (size_t)kTeam * kShared;
// and its counters (ints, zero between launches), each on a cache line of its own
constexpr int kFlagsAt = 0, kFlagsJacAt = 64, kExitAt = 128, kUndoneAt = 129, kVersionAt = 160, kMeetAt = 192, kPairAt = 224, kPairInts = 16,
              kSyncInts = kPairAt + kPairs * kPairInts;
// Flag of a workgroup that has given up.
constexpr int kGone = 1 << 24;
constexpr unsigned long long kGoneMeet = 1ull << 62, kNoHelpers = 1ull << 61;

// LDS
constexpr int kEimgAt = kImage;
constexpr int kXimg16At = 2 * kImage;                          // X in fp16 parts: two of three KiB a contraction step
constexpr int kStripAt = 3 * kImage;                           // [16][kLdStrip] floats
constexpr int kSmallLds = 4 * P * 16 * 4 > kStripAt + 16 * kLdStrip * 4 ? 4 * P * 16 * 4 : kStripAt + 16 * kLdStrip * 4;
constexpr size_t kLds = kSmallLds + 6144;                      // 256 floats of reductions, 4 x 256 words, two flags, ..
constexpr int kDiagAt = 1282;                                  // .. and two words beside the reductions

struct WideArgs {
    const float* M;            // [K][p][p] finished matrices, or nullptr: sum the pieces
    const float* partial;      // [pieces][p][p] (M == nullptr)
    const int32_t* offsets;    // [K+1] (M == nullptr): the grouping the pieces were cut from
    int piece;
    const int32_t* counts;     // [K] or nullptr
    float* D;
    DictOps ops;
    float* eig_sv;             // eigen mode
    int32_t* fallback;
    int32_t* iters_out;
    int max_iters, K, teams;
    int spread;
    int polls;                 // of one wait, at most
    int helper_polls;          // for the second workgroups of the pairs (-1: they leave at once)
    unsigned char* data;       // [teams][kTeamBytes]
    int* sync;                 // [teams][kSyncInts]
    SqTotalArgs sq;
};

__host__ __device__ inline int wide_team_wgs(int teams, int spread, bool pairs) {
    return pairs ? 8 * kPairs : spread ? teams * kTeam : (teams + 7) / 8 * 128;
}

__device__ __forceinline__ float half_sum(float x) {           // over 32 lanes
    x = group_sum<16>(x);
    const unsigned u = __builtin_bit_cast(unsigned, x);
    auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned a0 = r[0], a1 = r[1];
    return __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1);
}

// Handing data from one workgroup to another: every thread waits for its own stores, then thread 0
// releases for all; the other side polls, acquires and lets its workgroup go on.
//
// near: both workgroups run on the same XCD (HW_REG_XCC_ID, compared when the team first meets), so
// its L2 is where they meet: a store that has been waited for is in it (L1 writes through), and a load of the
// agent scope passes L1 by and finds it there.  Otherwise the fences of the agent scope, which write L2 back and
// invalidate it: 3 us a barrier, 5 to 10 when all CUs do it, against 1.
constexpr int kPastL1 = 16;                    // buffer loads: the bit of the agent scope (the same time as without)
__device__ __forceinline__ void stores_done() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}
__device__ __forceinline__ int peek(int* p) {
    return __hip_atomic_load((__attribute__((address_space(1))) int*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void acquire(bool near) {
    if (near) asm volatile("" ::: "memory");
    else __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}
template <class F>
__device__ __forceinline__ bool poll(int polls, bool near, F ready) {
    for (int k = 0; k < polls; ++k) {
        if (ready()) {
            acquire(near);
            return true;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    return false;
}
__device__ __forceinline__ void raise_to(int* p, int v, bool near) {
    if (near) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// A barrier of `size` workgroups that carries kCarried floats of each of them.
// (a flat load would have to be waited for with all loads before and after it)
__device__ __forceinline__ float far_load(const float* p) {
    return __hip_atomic_load((const __attribute__((address_space(1))) float*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct Team {
    int* flags;                // [size] of each workgroup how many barriers it has come to
    float* red;                // [4][kCarried][32]
    int* ok;                   // LDS
    int size, q, polls;
    int epoch;                 // barriers so far
    bool near;

    __device__ __forceinline__ void raise(int v) const {       // one thread
        if (near) __hip_atomic_store(flags + q, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else __hip_atomic_store(flags + q, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
    // So that the others need not wait for as long.
    __device__ __forceinline__ void gone() const { raise(kGone); }             // thread 0

    // a .. e: of thread 0
    __device__ __forceinline__ bool sync(float a, float b = 0.f, float c = 0.f, float d = 0.f, float e = 0.f) {
        ++epoch;
        if (threadIdx.x == 0) {
            float* slot = red + (epoch & 3) * (kPairs * kCarried) + q;
            slot[0] = a;
            slot[kPairs] = b;
            slot[2 * kPairs] = c;
            slot[3 * kPairs] = d;
            slot[4 * kPairs] = e;
        }
        stores_done();
        if (threadIdx.x < 64) {                // a wavefront reads all flags at once (a counter: 32 additions, and as many
            if (threadIdx.x == 0) raise(epoch);            // polls, one after the other)
            const int at = (int)threadIdx.x < size ? (int)threadIdx.x : 0;
            bool here = false, gone = false;
            for (int k = 0; k < polls && !here && !gone; ++k) {
                const int v = peek(flags + at);
                here = __all(v >= epoch);
                gone = __any(v >= kGone);
                if (!here && !gone) __builtin_amdgcn_s_sleep(1);
            }
            acquire(near);
            if (threadIdx.x == 0) *ok = here && !gone;
        }
        __syncthreads();
        return *ok != 0;
    }
    // The first barrier of a launch, which finds out whether the team is near: a counter of six bits per XCD.
    // If it is, what was stored before is where the others look; if not, a barrier of the other kind follows.
    __device__ __forceinline__ bool meet(unsigned long long* count) {
        stores_done();
        if (threadIdx.x == 0) {
            int xcc;
            asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(xcc));
            const int field = 6 * (xcc < 8 ? xcc : 8);
            __hip_atomic_fetch_add(count, 1ull << field, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            unsigned long long v = 0;
            const bool here = poll(polls, true, [&]() {
                v = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return met(v) == size || v >= kGoneMeet;
            });
            if (!here) __hip_atomic_fetch_or(count, kGoneMeet, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *ok = !here || v >= kGoneMeet ? 0 : xcc < 8 && (int)(v >> field & 63) == size ? 2 : 1;
        }
        __syncthreads();
        const int how = *ok;
        near = how == 2;
        if (how == 1) return sync(0.f);        // (begins with a barrier: *ok has been read)
        return how != 0;
    }
    __device__ __forceinline__ static int met(unsigned long long v) {
        int n = 0;
        for (int f = 0; f <= 48; f += 6) n += (int)(v >> f) & 63;
        return n;
    }
    // The same for a team of pairs: 1 all are there, 0 a wait has ended, -1 without the helpers (the second half of the
    // workgroups): one of the first half saw these complete, waited helper_polls times and put kNoHelpers into the counter
    // before the last helper came.  A counter that has all of them and not that bit never gets it, so all read the same.
    // first (bits 54 ..): of the first half.
    __device__ __forceinline__ int meet_pairs(unsigned long long* count, int helper_polls) {
        stores_done();
        if (threadIdx.x == 0) {
            int xcc;
            asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(xcc));
            const int field = 6 * (xcc < 8 ? xcc : 8);
            const bool helper = q >= kTeam;
            __hip_atomic_fetch_add(count, (1ull << field) + (helper ? 0 : 1ull << 54), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            int how = -2;
            for (int k = 0, waited = 0; how == -2; ++k) {
                unsigned long long v = __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const int first = (int)(v >> 54) & 31;
                const bool without = (v & kNoHelpers) != 0;
                if (v >= kGoneMeet) {
                    how = 0;
                } else if (!without && met(v) == kPairs) {
                    how = xcc < 8 && (int)(v >> field & 63) == kPairs ? 2 : 1;
                } else if (without && (helper || first == kTeam)) {
                    how = -1;
                } else if (k >= polls && !helper && first < kTeam) {
                    __hip_atomic_fetch_or(count, kGoneMeet, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    how = 0;
                } else if (k >= polls || (!helper && first == kTeam && ++waited > helper_polls)) {
                    __hip_atomic_compare_exchange_strong(count, &v, v | kNoHelpers, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);      // (fails: look again)
                }
                if (how == -2) __builtin_amdgcn_s_sleep(1);
            }
            *ok = how;
        }
        __syncthreads();
        const int how = *ok;
        near = how == 2;
        if (how == 1) return sync(0.f) ? 1 : 0;
        if (how == -1) __syncthreads();        // *ok has been read
        return how > 0 ? 1 : how;
    }
    // value k of workgroup lane % size, from the last sync
    __device__ __forceinline__ float value(int k) const {
        return far_load(red + (epoch & 3) * (kPairs * kCarried) + k * kPairs + (threadIdx.x & (size - 1)));
    }
};

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
// Maximum over the wavefront, in all lanes.
__device__ __forceinline__ float wave_max(float x) {
    const unsigned u = __builtin_bit_cast(unsigned, row16_max(x));
    auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned a0 = r[0], a1 = r[1];
    const unsigned w = __builtin_bit_cast(unsigned, fmaxf(__builtin_bit_cast(float, a0), __builtin_bit_cast(float, a1)));
    auto q = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    const unsigned b0 = q[0], b1 = q[1];
    return fmaxf(__builtin_bit_cast(float, b0), __builtin_bit_cast(float, b1));
}
__device__ __forceinline__ float wave_max_nan(float x) {
    unsigned u = __builtin_bit_cast(unsigned, row_max_nan(x));
    auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned a0 = r[0], a1 = r[1];
    u = max(a0, a1);
    auto q = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const unsigned b0 = q[0], b1 = q[1];
    return __builtin_bit_cast(float, max(b0, b1));
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

// Where P_j comes from: a finished matrix, or the pieces [beg, end) summed in piece order.
struct Source {
    const float* base;         // of the first piece
    int n;
};
// 16-byte units tid and tid + 512 of the 16 columns of strip s (16 KiB in one run)
__device__ __forceinline__ void load_strip(const Source& src, int s, f32x4 (&v)[2]) {
    constexpr int kInFlight = 8;
    const f32x4* b = reinterpret_cast<const f32x4*>(src.base) + s * (16 * P / 4) + threadIdx.x;
    for (int pc = 0; pc < src.n; pc += kInFlight) {
        f32x4 w[kInFlight][2];
#pragma unroll
        for (int k = 0; k < kInFlight; ++k)
            if (pc + k < src.n) {              // uniform
#pragma unroll
                for (int u = 0; u < 2; ++u) w[k][u] = b[(int64_t)(pc + k) * (P * P / 4) + u * kNT];
            }
        if (pc == 0) v[0] = v[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < kInFlight; ++k)
            if (pc + k < src.n) {
#pragma unroll
                for (int u = 0; u < 2; ++u) v[u] += w[k][u];
            }
    }
}

// 16-byte unit (tid % 32) + 32 h of column tid / 32 of strip s: half h of its rows
__device__ __forceinline__ f32x4 load_half_strip(const Source& src, int s, int h) {
    constexpr int kInFlight = 16;
    const f32x4* b = reinterpret_cast<const f32x4*>(src.base) + s * (16 * P / 4) + (threadIdx.x >> 5) * (P / 4) + 32 * h +
                     (threadIdx.x & 31);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    for (int pc = 0; pc < src.n; pc += kInFlight) {
        f32x4 w[kInFlight];
#pragma unroll
        for (int k = 0; k < kInFlight; ++k)
            if (pc + k < src.n) w[k] = b[(int64_t)(pc + k) * (P * P / 4)];         // uniform
#pragma unroll
        for (int k = 0; k < kInFlight; ++k)
            if (pc + k < src.n) v += w[k];
    }
    return v;
}

// D[j] rows of strip s from LDS ([16][kLdStrip]), and the same rows in the operand orders.  dn: 256 floats of LDS.
__device__ __forceinline__ void emit_strip(const WideArgs& g, int j, int s, const float* strip, float* dn) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    f32x4* Dj = reinterpret_cast<f32x4*>(g.D + ((int64_t)j * P + s * 16) * P);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int e = tid + u * kNT;
        Dj[e] = *reinterpret_cast<const f32x4*>(strip + (e >> 6) * kLdStrip + 4 * (e & 63));
    }
    if (g.ops.f32 == nullptr && g.ops.bf16 == nullptr && g.ops.f16 == nullptr) return;     // uniform
    const int col = tid & 15, d8 = tid >> 4, grow = j * P + s * 16 + col;
    float q2 = 0.f, r2 = 0.f;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(strip + col * kLdStrip + 8 * d8 + 4 * u);
        if (g.ops.f32 != nullptr) store_operand_f32<P>(g.ops.f32, grow, 2 * d8 + u, v);
        if (g.ops.bf16 != nullptr) store_operand_split<P>(g.ops.bf16, grow, 2 * d8 + u, v);
        if (g.ops.f16 != nullptr) store_operand_f16x2<P>(g.ops.f16, grow, 2 * d8 + u, split_f16x2_dict(v, q2, r2));
    }
    if (g.ops.f16 == nullptr) return;          // uniform
    q2 = sum_groups(q2);
    r2 = sum_groups(r2);
    if (lane < 16) {
        dn[wave * 16 + lane] = q2;
        dn[128 + wave * 16 + lane] = r2;
    }
    __syncthreads();
    if (wave == 0) {
        q2 = r2 = 0.f;
        for (int w = 0; w < kWaves; ++w) {
            q2 += dn[w * 16 + (lane & 15)];
            r2 += dn[128 + w * 16 + (lane & 15)];
        }
        q2 = row16_max(q2);
        r2 = row16_max(r2);
        if (lane == 0) {
            g.ops.dnorm[j * (P / 16) + s] = float2{sqrtf(q2), sqrtf(r2)};
            g.ops.dodd[j * (P / 16) + s] = 0;  // (an orthobase)
        }
    }
    __syncthreads();
}

__device__ __forceinline__ unsigned char* uniform(unsigned char* p) {
    const unsigned long long v = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    // (of the global address space: flat accesses are counted with those of LDS)
    return (unsigned char*)(__attribute__((address_space(1))) unsigned char*)((unsigned long long)hi << 32 | lo);
}

enum class Outcome { done, left, dead, alone };        // left: to the Jacobi SVD; dead: a wait has ended; alone: without helpers

// Newton-Schulz for block j.  H = 1: strip `t.q` of the result is left in LDS at kStripAt; first != nullptr: the team has not met yet.
// H = 2, a team of pairs, which meets here: workgroups s and s + 16 have the upper and the lower half of strip s's rows, a
// wavefront one tile of both products, and write their halves of D[j].  The B operand of a product is the whole strip: the
// contraction starts with the own half, and the other one comes by memory meanwhile, X with the team's barrier, E with a
// number in `pair`.
template <int H>
__device__ __forceinline__ Outcome newton_schulz(const WideArgs& g, int j, const Source& src, Team& t,
                                                 unsigned long long* first, unsigned char* mem, unsigned char* lds,
                                                 float* red, int* pair, int& steps) {
    constexpr int NT = 2 / H;                  // tiles of a wavefront
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = lane >> 4, c16 = lane & 15;
    // (Uniform, which the compiler does not see of what has been through a call or a wait: every operand load was a loop over
    // the lanes' descriptors and offsets.)
    const int tq = __builtin_amdgcn_readfirstlane(t.q);
    mem = uniform(mem);
    const int sn = H == 1 ? tq : tq & (kTeam - 1), half = H == 1 ? 0 : tq / kTeam;         // the strip, which half
    const int t0 = H == 1 ? 2 * wave : half * 8 + wave, tp = (1 - half) * 8 + wave;        // the first tile; one of the other half
    unsigned char* ximg = lds;
    unsigned char* eimg = lds + kEimgAt;
    unsigned char* ximg16 = lds + kXimg16At;
    float* strip = reinterpret_cast<float*>(lds + kStripAt);

    constexpr int kAhead = 4;
    const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(mem, 0, (int)kTeamBytes, 0x00027000);
    // Two ways for the products: three bf16 parts, six partial products, or two fp16 parts and three (`two`).
    typedef std::true_type Two;
    typedef std::false_type Three;
    auto mfma = [](auto two, u32x4 a, u32x4 b, f32x4 c) {
        if constexpr (decltype(two)::value)
            return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
        else
            return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    };
    auto at16 = [](const unsigned char* p) { return *reinterpret_cast<const u32x4*>(p); };
    auto split = [](auto two, f32x4 lo, f32x4 hi, u32x4 (&out)[3]) {
        if constexpr (decltype(two)::value) {
            const F16x2Pair a = split_f16x2(lo.x, lo.y), b = split_f16x2(lo.z, lo.w);
            const F16x2Pair c = split_f16x2(hi.x, hi.y), d = split_f16x2(hi.z, hi.w);
            out[0] = u32x4{a.hi, b.hi, c.hi, d.hi};
            out[1] = u32x4{a.lo, b.lo, c.lo, d.lo};
            return;
        }
        const Bf16x3Pair a = split_bf16x3(lo.x, lo.y), b = split_bf16x3(lo.z, lo.w);
        const Bf16x3Pair c = split_bf16x3(hi.x, hi.y), d = split_bf16x3(hi.z, hi.w);
        out[0] = u32x4{a.hi, b.hi, c.hi, d.hi};
        out[1] = u32x4{a.mid, b.mid, c.mid, d.mid};
        out[2] = u32x4{a.lo, b.lo, c.lo, d.lo};
    };
    // The parts of the tiles t0 .. (or of one tile) in an image of the strip: contraction step of 32 = two tiles, a half unit each.
    auto put_tile = [&](auto two, unsigned char* img, int tile, f32x4 v) {
        if constexpr (decltype(two)::value) {
            const F16x2Pair a = split_f16x2(v.x, v.y), b = split_f16x2(v.z, v.w);
            u32x2* at = reinterpret_cast<u32x2*>(img + (tile >> 1) * 3 * 1024 + lane * 16 + (tile & 1) * 8);
            at[0] = u32x2{a.hi, b.hi};
            at[128] = u32x2{a.lo, b.lo};
            return;
        }
        const Bf16x3Pair a = split_bf16x3(v.x, v.y), b = split_bf16x3(v.z, v.w);
        u32x2* at = reinterpret_cast<u32x2*>(img + (tile >> 1) * 3 * 1024 + lane * 16 + (tile & 1) * 8);
        at[0] = u32x2{a.hi, b.hi};
        at[128] = u32x2{a.mid, b.mid};
        at[256] = u32x2{a.lo, b.lo};
    };
    auto put_parts = [&](auto two, unsigned char* img, const f32x4 (&v)[NT]) {
        if constexpr (H == 1) {
            u32x4 part[3];
            split(two, v[0], v[NT - 1], part);
#pragma unroll
            for (int pl = 0; pl < (decltype(two)::value ? 2 : 3); ++pl) *reinterpret_cast<u32x4*>(img + (wave * 3 + pl) * 1024 + lane * 16) = part[pl];
        } else {
            put_tile(two, img, t0, v[0]);
        }
    };
    // over the values that a barrier carried (H = 2: the two of a pair first)
    auto all_sum = [](float v) {
        if constexpr (H == 2) {
            const unsigned u = __builtin_bit_cast(unsigned, v);
            auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
            const unsigned a0 = r[0], a1 = r[1];
            v = __builtin_bit_cast(float, a0) + __builtin_bit_cast(float, a1);
        }
        return group_sum<16>(v);
    };
    auto all_max = [](float v) {
        v = row16_max(v);
        if constexpr (H == 2) {
            const unsigned u = __builtin_bit_cast(unsigned, v);
            auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
            const unsigned a0 = r[0], a1 = r[1];
            v = fmaxf(__builtin_bit_cast(float, a0), __builtin_bit_cast(float, a1));
        }
        return v;
    };
    // xr[k]: rows (t0 + k) * 16 + grp * 4 .. +3 of column sn * 16 + c16
    f32x4 xr[NT];
    {
        if constexpr (H == 1) {
            f32x4 v[2];
            load_strip(src, sn, v);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int e = tid + u * kNT;
                *reinterpret_cast<f32x4*>(strip + (e >> 6) * kLdStrip + 4 * (e & 63)) = v[u];
            }
        } else {
            const f32x4 v = load_half_strip(src, sn, half);
            *reinterpret_cast<f32x4*>(strip + (tid >> 5) * kLdStrip + 128 * half + 4 * (tid & 31)) = v;
            if (tid == 0) {                    // what workgroups without a tile on the diagonal say of it
                red[kDiagAt] = 3e38f;
                red[kDiagAt + 1] = 0.f;
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NT; ++k)
            xr[k] = *reinterpret_cast<const f32x4*>(strip + c16 * kLdStrip + (t0 + k) * 16 + grp * 4);
    }
    // Leaves the strip for the others (buffer buf), in fp32, and its parts in ximg.  Contraction step s of 32 = tiles 2s and
    // 2s + 1, its two halves: a lane holds rows grp * 4 .. of both, which is what an accumulator leaves it, and of the rows'
    // image four columns grp * 4 .. of a row, by way of LDS (the wavefront's own part of `strip`).
    auto publish = [&](int buf, bool scaled) {
        unsigned char* cols = mem + kColAt + ((size_t)buf * kTeam + sn) * kShared;
        unsigned char* rows = mem + kRowAt + (size_t)buf * kTeam * kShared;
        put_parts(Three{}, ximg, xr);
        if (scaled) put_parts(Two{}, ximg16, xr);              // (which of them the next step takes is known after the barrier)
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            *reinterpret_cast<f32x4*>(cols + (t0 + k) * 1024 + lane * 16) = xr[k];
            *reinterpret_cast<f32x4*>(strip + c16 * kLdStrip + (t0 + k) * 16 + grp * 4) = xr[k];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            const int td = t0 + k;
            const float* row = strip + td * 16 + c16;          // of columns 0, 1, ..
            *reinterpret_cast<f32x4*>(rows + (size_t)((td * 8 + (sn >> 1)) * 2 + (sn & 1)) * 1024 + lane * 16) =
                f32x4{row[(4 * grp) * kLdStrip], row[(4 * grp + 1) * kLdStrip], row[(4 * grp + 2) * kLdStrip],
                      row[(4 * grp + 3) * kLdStrip]};
        }
    };
    auto on_diagonal = [&](int k, int r) { return (t0 + k) * 16 + grp * 4 + r == sn * 16 + c16; };
    const bool diagonal = sn >= t0 && sn < t0 + NT;            // uniform: this wavefront has the tile on the diagonal
    // Smallest diagonal entry of G in this workgroup's columns (left in red[kDiagAt]: there after the next barrier).
    auto least_diag = [&](const f32x4 (&gm)[NT]) {
        if (!diagonal) return;
        float v = 3e38f;
#pragma unroll
        for (int k = 0; k < NT; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (on_diagonal(k, r)) v = gm[k][r];
        v = -wave_max(-v);
        if (lane == 0) red[kDiagAt] = v;
    };
    // E = I - a2 G, times a scale
    auto make_e = [&](const f32x4 (&gm)[NT], float a2, f32x4 (&e)[NT], float by = 1.f) {
        a2 *= by;
#pragma unroll
        for (int k = 0; k < NT; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) e[k][r] = (on_diagonal(k, r) ? by : 0.f) - a2 * gm[k][r];
    };

    // A product: contraction steps S0 .. S0 + 7, their A operands requested kAhead steps before and split here, the B operands
    // from an image in LDS one step before; sums apart, so that matrix instructions are independent.  H = 2: ask() before the last
    // step of the own half, have() before the first of the other one.
    auto product = [&](auto two, auto& a, auto& request, auto& turn, const unsigned char* img, auto first_step, f32x4 (&out)[NT],
                       auto&& ask, auto&& have) {
        constexpr int S0 = decltype(first_step)::value, NS = 4;
        constexpr bool kTwo = decltype(two)::value;
        constexpr int NPT = kTwo ? 2 : 3, NP = kTwo ? 3 : 6;
        constexpr int TA[6] = {kTwo ? 1 : 2, 0, kTwo ? 0 : 1, 1, 0, 0};        // the partial products, smallest first
        constexpr int TB[6] = {0, kTwo ? 1 : 2, kTwo ? 0 : 1, 0, 1, 0};
        f32x4 sum[NT][NS];
#pragma unroll
        for (int k = 0; k < NT; ++k)
#pragma unroll
            for (int c = 0; c < NS; ++c) sum[k][c] = zero4;
        u32x4 b[2][3];
        auto read = [&](int s) {
#pragma unroll
            for (int pl = 0; pl < NPT; ++pl) b[s & 1][pl] = at16(img + (turn(s) * 3 + pl) * 1024 + lane * 16);
        };
        read(S0);
#pragma unroll
        for (int s = S0; s < S0 + 8; ++s) {
            if (H == 2 && s == S0 + 3) ask();
            if (H == 2 && s == S0 + 4) {
                have();
                read(s);
            }
            if (s + 1 < S0 + 8 && !(H == 2 && s == S0 + 3)) read(s + 1);
            u32x4 part[NT][3];
#pragma unroll
            for (int k = 0; k < NT; ++k)
                split(two, __builtin_bit_cast(f32x4, a[s % kAhead][k][0]), __builtin_bit_cast(f32x4, a[s % kAhead][k][1]), part[k]);
#pragma unroll
            for (int q = 0; q < NP; ++q)
#pragma unroll
                for (int k = 0; k < NT; ++k) {
                    f32x4& to = sum[k][kTwo && q == 2 ? 2 + (s & 1) : q % NS];
                    to = mfma(two, part[k][TA[q]], b[s & 1][TB[q]], to);
                }
            if (s + kAhead < 16) request(s + kAhead);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int k = 0; k < NT; ++k) out[k] = (sum[k][0] + sum[k][1]) + (sum[k][2] + sum[k][3]);
    };

    publish(0, false);
    if constexpr (H == 2) {
        const int how = t.meet_pairs(first, g.helper_polls);
        if (how <= 0) return how < 0 ? Outcome::alone : Outcome::dead;
    } else {
        if (!(first != nullptr ? t.meet(first) : t.sync(0.f))) return Outcome::dead;
    }
    // H = 2, handing something to the other workgroup of the pair
    int handed = 0;
    auto hand = [&]() {
        stores_done();
        ++handed;
        if (tid == 0) raise_to(pair + t.q * kPairInts, handed, t.near);
    };
    auto taken = [&]() {                       // the same number of hands from there (uniform)
        int* flag = t.ok + 1;
        if (tid == 0)
            *flag = poll(t.polls, t.near, [&]() { return peek(pair + (t.q ^ kTeam) * kPairInts) >= handed; });
        __syncthreads();
        return *flag != 0;
    };
    float prev = 3e38f;                        // |I - X^T X|_F^2 before the step before
    NsScale scale;
    bool look = false;
    for (int it = 0;; ) {
        // A operands, contraction steps 0 .. 7 of X^T X, then 8 .. 15 = 0 .. 7 of X E.  Buffer loads: one
        // descriptor, a scalar offset per load (as pointers the addresses alone take 100 registers).  Every
        // wavefront of the team starts at another step: in step, they would all ask the same L2
        // channels at a time.
        const int buf = __builtin_amdgcn_readfirstlane(it & 1);
        const int cols = (int)kColAt + (buf * kTeam + t0) * kShared;
        const int rows = (int)kRowAt + (buf * kTeam + t0) * kShared;
        u32x4 a[kAhead][NT][2], other = {0u, 0u, 0u, 0u};
        // The steps of the tile's half first (H = 2 has the others later), in an order that is the same for both H: so are the sums.
        const int own4 = (t0 >> 3) * 4;
        auto turn = [&](int s) { return ((s & 4) ^ own4) | ((s + (t0 >> 1) + sn) & 3); };
        auto request = [&](int s) {
#pragma unroll
            for (int k = 0; k < NT; ++k)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    a[s % kAhead][k][e] = __builtin_amdgcn_raw_buffer_load_b128(
                        rsrc, lane * 16, (s < 8 ? cols : rows) + k * kShared + (turn(s) * 2 + e) * 1024, kPastL1);
        };
        // What the last barrier carried: asked for before the operands, which it would otherwise wait for (loads return in order).
        const float carried0 = look ? t.value(0) : 0.f, carried1 = look ? t.value(1) : 0.f;    // uniform
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (H == 2)                  // a tile of the strip's other half
            other = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, (int)kColAt + (buf * kTeam + sn) * kShared + tp * 1024, kPastL1);
#pragma unroll
        for (int s = 0; s < kAhead; ++s) request(s);
        __builtin_amdgcn_sched_barrier(0);
        if (look) {                            // uniform
            prev = all_sum(carried0);
            if (!(prev < 2.f * P)) return Outcome::left;
            scale.seen(-all_max(-carried1));
        }
        f32x4 gm[NT];
        auto gram = [&](auto two, unsigned char* img) {
            product(two, a, request, turn, img, std::integral_constant<int, 0>{}, gm, []() {},
                    [&]() {
                        put_tile(two, img, tp, __builtin_bit_cast(f32x4, other));
                        __syncthreads();
                    });
        };
        // Three parts where the input has no scale yet, and where this may be the last step (below): then the rounding of G is
        // that of the result.  Elsewhere what two parts leave out is a symmetric error of G, which the next step takes out.
        const bool exact = __builtin_amdgcn_readfirstlane((int)(it == 0 || prev < 4.f || it >= g.max_iters)) != 0;
        if (exact) gram(Three{}, ximg);
        else gram(Two{}, ximg16);
        if (it > 0) {                          // uniform
#pragma unroll
            for (int k = 0; k < NT; ++k) gm[k] *= 1.f / (kXScale * kXScale);
        }

        float alpha = 1.f, fr = 0.f;
        bool last = false, known = false;
        // |I - G|_F^2 of the workgroup's part of G: by one thread, after a barrier
        auto own_norm = [&]() {
            float v = 0.f;
            for (int w = 0; w < kWaves; ++w) v += red[(it & 1) * 8 + w];
            return v;
        };
        f32x4 e[NT];
        if (it == 0) {
            // row sums and squares by columns: of a tile, then of half a column, then of a column (the same order for both H)
#pragma unroll
            for (int k = 0; k < NT; ++k) {
                float rs = 0.f, r2 = 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    rs += fabsf(gm[k][r]);
                    r2 = fmaf(gm[k][r], gm[k][r], r2);
                }
                rs = sum_groups(rs);
                r2 = sum_groups(r2);
                if (lane < 16) {
                    red[(NT * wave + k) * 16 + lane] = rs;
                    red[256 + (NT * wave + k) * 16 + lane] = r2;
                }
            }
            __syncthreads();
            float rs[NT], r2[NT];
#pragma unroll
            for (int k = 0; k < NT; ++k) {
                rs[k] = r2[k] = 0.f;
                for (int w = 8 * k; w < 8 * k + 8; ++w) {
                    rs[k] += red[w * 16 + c16];
                    r2[k] += red[256 + w * 16 + c16];
                }
            }
            float tr = 0.f;
#pragma unroll
            for (int k = 0; k < NT; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (on_diagonal(k, r)) tr = gm[k][r];
            tr = sum_groups(group_sum<16>(tr));
            if (diagonal && lane == 0) red[kDiagAt + 1] = tr;
            least_diag(gm);
            float rsmax, r2max, sum2;
            __syncthreads();
            if constexpr (H == 1) {
                const float rc = rs[0] + rs[NT - 1], r2c = r2[0] + r2[NT - 1];
                if (!t.sync(row_max_nan(rc), row_max_nan(r2c), red[kDiagAt], group_sum<16>(r2c), red[kDiagAt + 1])) return Outcome::dead;
                rsmax = row_max_nan(t.value(0));
                r2max = row_max_nan(t.value(1));
                sum2 = t.value(3);
            } else {                           // added up by everybody
                float* sums = reinterpret_cast<float*>(mem + kSmallAt) + 2 * kRedSize + 2 * P;
                if (tid < 16) {
                    sums[(half * 2) * P + sn * 16 + tid] = rs[0];
                    sums[(half * 2 + 1) * P + sn * 16 + tid] = r2[0];
                }
                if (!t.sync(0.f, 0.f, red[kDiagAt], 0.f, red[kDiagAt + 1])) return Outcome::dead;
                float v[4][4];
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        v[k][c] = far_load(sums + k * P + c * 64 + lane);
                unsigned m1 = 0, m2 = 0;       // (a NaN wins: its bits are the largest)
                sum2 = 0.f;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float w = v[1][c] + v[3][c], of = __shfl(group_sum<16>(w), (lane & 3) * 16, 64);     // of strip 4 c + lane % 4
                    m1 = max(m1, __builtin_bit_cast(unsigned, v[0][c] + v[2][c]));
                    m2 = max(m2, __builtin_bit_cast(unsigned, w));
                    if ((c16 >> 2) == c) sum2 = of;
                }
                rsmax = wave_max_nan(__builtin_bit_cast(float, m1));
                r2max = wave_max_nan(__builtin_bit_cast(float, m2));
            }
            sum2 = group_sum<16>(sum2);
            // zero, infinite, NaN or overflowing input: not for this iteration
            if (!(rsmax > 1e-37f && rsmax < 3e37f)) return Outcome::left;
            alpha = scale.first(rsmax, r2max, -all_max(-t.value(2)), sum2, all_sum(t.value(4)) * (1.f / P));
        } else {
            make_e(gm, 1.f, e);
#pragma unroll
            for (int k = 0; k < NT; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r) fr = fmaf(e[k][r], e[k][r], fr);
            fr = sum_groups(group_sum<16>(fr));
            if (lane == 0) red[(it & 1) * 8 + wave] = fr;
            least_diag(gm);
            alpha = scale.next();
            // Close to the end the team meets here to learn whether this is the last step, and exchanges the
            // leading fp16 parts of E for its square (H = 2: the second ones too, for the other half of the strip).
            if (prev < 4.f || it >= g.max_iters) {           // uniform over the team
                const f32x4 lo = kEScale * e[0], hi = kEScale * e[NT - 1];
                const F16x2Pair a0 = split_f16x2(lo.x, lo.y), a1 = split_f16x2(lo.z, lo.w);
                const F16x2Pair a2 = split_f16x2(hi.x, hi.y), a3 = split_f16x2(hi.z, hi.w);
                if constexpr (H == 1) {
                    const u32x4 lead = {a0.hi, a1.hi, a2.hi, a3.hi};
                    *reinterpret_cast<u32x4*>(eimg + wave * 3 * 1024 + lane * 16) = lead;
                    *reinterpret_cast<u32x4*>(eimg + (wave * 3 + 1) * 1024 + lane * 16) = u32x4{a0.lo, a1.lo, a2.lo, a3.lo};
                    *reinterpret_cast<u32x4*>(mem + kEAt + ((size_t)sn * 8 + wave) * 1024 + lane * 16) = lead;
                } else {
                    const u32x2 lead = {a0.hi, a1.hi}, rest = {a0.lo, a1.lo};
                    const size_t at = ((size_t)sn * 8 + (t0 >> 1)) * 1024 + lane * 16 + (t0 & 1) * 8;
                    *reinterpret_cast<u32x2*>(eimg + (t0 >> 1) * 3 * 1024 + lane * 16 + (t0 & 1) * 8) = lead;
                    *reinterpret_cast<u32x2*>(eimg + ((t0 >> 1) * 3 + 1) * 1024 + lane * 16 + (t0 & 1) * 8) = rest;
                    *reinterpret_cast<u32x2*>(mem + kEAt + at) = lead;
                    *reinterpret_cast<u32x2*>(mem + kELoAt + at) = rest;
                }
                __syncthreads();
                if (!t.sync(own_norm())) return Outcome::dead;
                prev = all_sum(t.value(0));
                known = true;
                if (!(prev < 2.f * P)) return Outcome::left;   // NaN or diverging
                last = prev < kLastEps * kLastEps;
                if (!last && it >= g.max_iters) return Outcome::left;
            }
        }
        // uniform.  E^2: one operand in its leading fp16 part (off by 2^-11, of a term below 4e-5: 2e-8 at most, as
        // the polynomial), the other in two.  As three bf16 products it takes a second exchange and two more rounds
        // of loads, 3 us of 97 at K = 16, for an error that is the same in all digits measured.
        if (last) {
            alpha = 1.f;
            if constexpr (H == 2) {            // the other half
                const int at = (sn * 8 + (tp >> 1)) * 1024 + lane * 16 + (tp & 1) * 8;
                const u32x2 lead = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, at, (int)kEAt, kPastL1));
                const u32x2 rest = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, at, (int)kELoAt, kPastL1));
                *reinterpret_cast<u32x2*>(eimg + (tp >> 1) * 3 * 1024 + lane * 16 + (tp & 1) * 8) = lead;
                *reinterpret_cast<u32x2*>(eimg + ((tp >> 1) * 3 + 1) * 1024 + lane * 16 + (tp & 1) * 8) = rest;
                __syncthreads();
            }
            f32x4 e2[NT];
            const int er = (int)kEAt + t0 * 8 * 1024;
#pragma unroll
            for (int k = 0; k < NT; ++k) {
                e2[k] = zero4;
                u32x4 ea[8];
#pragma unroll
                for (int s = 0; s < 8; ++s) ea[s] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, er + (k * 8 + s) * 1024, kPastL1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < 8; ++s)
#pragma unroll
                    for (int pl = 1; pl >= 0; --pl)
                        e2[k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            __builtin_bit_cast(f16x8, ea[s]),
                            __builtin_bit_cast(f16x8, at16(eimg + (s * 3 + pl) * 1024 + lane * 16)), e2[k], 0, 0, 0);
            }
            __syncthreads();                   // eimg is rewritten
#pragma unroll
            for (int k = 0; k < NT; ++k) e[k] = kXScale * (kLastLinear * e[k] + (kLastSquare / (kEScale * kEScale)) * e2[k]);
        } else {
            // (times alpha, at least one: the products are then added to X without another rounding)
            make_e(gm, alpha * alpha, e, it == 0 ? 1.f : kXScale * alpha);
        }
        if (it == 0) put_parts(Three{}, eimg, e);
        else put_parts(Two{}, eimg, e);
        const int eh = (int)kEHalfAt + sn * kShared;
        if constexpr (H == 1) {
            __syncthreads();
        } else {
            *reinterpret_cast<f32x4*>(mem + eh + t0 * 1024 + lane * 16) = e[0];
            hand();
        }
        f32x4 acc[NT];
        bool here = true;
        auto turned = [&](auto two) {
            product(two, a, request, turn, eimg, std::integral_constant<int, 8>{}, acc,
                    [&]() {
                        here = taken();
                        other = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, eh + tp * 1024, kPastL1);
                    },
                    [&]() {
                        put_tile(two, eimg, tp, __builtin_bit_cast(f32x4, other));
                        __syncthreads();
                    });
        };
        if (it == 0) turned(Three{});
        else turned(Two{});
        if (H == 2 && !here) return Outcome::dead;
#pragma unroll
        for (int k = 0; k < NT; ++k)
            xr[k] = it == 0 ? (kXScale * alpha) * xr[k] + (0.5f * kXScale * alpha) * acc[k] : alpha * xr[k] + (0.5f / kXScale) * acc[k];
        if (last) {
            steps = it + 1;
            break;
        }
        publish((it + 1) & 1, true);
        if (!t.sync(it > 0 ? own_norm() : 0.f, red[kDiagAt])) return Outcome::dead;
        look = !known && it > 0;
        ++it;
    }
#pragma unroll
    for (int k = 0; k < NT; ++k)
        *reinterpret_cast<f32x4*>(strip + c16 * kLdStrip + (t0 + k) * 16 + grp * 4) = xr[k] * (1.f / kXScale);
    __syncthreads();
    if constexpr (H == 2) {                    // D[j] rows of the strip, as emit_strip; the norms of whole atoms by the first of the pair
        {
            const int c = tid >> 5, d4 = 32 * half + (tid & 31);
            reinterpret_cast<f32x4*>(g.D + ((int64_t)j * P + sn * 16 + c) * P)[d4] =
                *reinterpret_cast<const f32x4*>(strip + c * kLdStrip + 4 * d4);
        }
        if (g.ops.f32 == nullptr && g.ops.bf16 == nullptr && g.ops.f16 == nullptr) return Outcome::done;       // uniform
        const int c = tid & 15, d4 = 32 * half + (tid >> 4), grow = j * P + sn * 16 + c;
        const f32x4 v = *reinterpret_cast<const f32x4*>(strip + c * kLdStrip + 4 * d4);
        float q2 = 0.f, r2 = 0.f;
        if (g.ops.f32 != nullptr) store_operand_f32<P>(g.ops.f32, grow, d4, v);
        if (g.ops.bf16 != nullptr) store_operand_split<P>(g.ops.bf16, grow, d4, v);
        if (g.ops.f16 == nullptr) return Outcome::done;        // uniform
        store_operand_f16x2<P>(g.ops.f16, grow, d4, split_f16x2_dict(v, q2, r2));
        q2 = sum_groups(q2);
        r2 = sum_groups(r2);
        if (lane < 16) {
            red[wave * 16 + lane] = q2;
            red[128 + wave * 16 + lane] = r2;
        }
        __syncthreads();
        q2 = r2 = 0.f;
        for (int w = 0; w < kWaves; ++w) {
            q2 += red[w * 16 + c16];
            r2 += red[128 + w * 16 + c16];
        }
        float* sums = reinterpret_cast<float*>(mem + kSmallAt) + 2 * kRedSize + 2 * P + sn * 32;    // (last read in the first step)
        if (half == 1 && tid < 16) {
            sums[tid] = q2;
            sums[16 + tid] = r2;
        }
        hand();
        if (half == 1) return Outcome::done;
        if (!taken()) return Outcome::dead;
        q2 += far_load(sums + c16);
        r2 += far_load(sums + 16 + c16);
        q2 = row16_max(q2);
        r2 = row16_max(r2);
        if (tid == 0) {
            g.ops.dnorm[j * (P / 16) + sn] = float2{sqrtf(q2), sqrtf(r2)};
            g.ops.dodd[j * (P / 16) + sn] = 0;
        }
    }
    return Outcome::done;
}

// Columns in half a wavefront: rows 2 l32 + 64 k + {0, 1}
__device__ __forceinline__ void get_column(const float* col, float (&v)[8]) {
    const int l32 = threadIdx.x & 31;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float2 w = *reinterpret_cast<const float2*>(col + 2 * l32 + 64 * k);
        v[2 * k] = w.x;
        v[2 * k + 1] = w.y;
    }
}
__device__ __forceinline__ void put_column(float* col, const float (&v)[8]) {
    const int l32 = threadIdx.x & 31;
#pragma unroll
    for (int k = 0; k < 4; ++k) *reinterpret_cast<float2*>(col + 2 * l32 + 64 * k) = float2{v[2 * k], v[2 * k + 1]};
}
__device__ __forceinline__ float column_norm(const float (&w)[8]) {
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) s += w[k] * w[k];
    return sqrtf(half_sum(s));
}
// Rotates the columns x, y of A and u, v of V if x and y are not orthogonal enough (false: left as they are).
__device__ __forceinline__ bool rotate(float (&x)[8], float (&y)[8], float (&u)[8], float (&v)[8], int& rotated) {
    float al = 0.f, be = 0.f, ga = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        al += x[k] * x[k];
        be += y[k] * y[k];
        ga += x[k] * y[k];
    }
    al = half_sum(al);
    be = half_sum(be);
    ga = half_sum(ga);
    const float d = be - al, g2 = 2.f * ga, hh = d * d + g2 * g2, gg = ga * ga, ab = al * be;
    if (gg > (kPolarDone * kPolarDone) * ab) rotated = 1;
    if (!(gg > (kTol * kTol) * ab && hh > 1e-36f)) return false;
    // cos(2 theta) = |d| / hypot(d, 2 gamma), |theta| <= pi/4
    const float r = __builtin_amdgcn_rsqf(hh), w = 0.5f + 0.5f * (fabsf(d) * r), rc = __builtin_amdgcn_rsqf(w);
    const float cs = w * rc, sn = copysignf(0.5f * rc * r, d) * g2;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float a = x[k], b = y[k];
        x[k] = cs * a - sn * b;
        y[k] = sn * a + cs * b;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float a = u[k], b = v[k];
        u[k] = cs * a - sn * b;
        v[k] = sn * a + cs * b;
    }
    return true;
}
// Place of the eigenvector c among the 256 by descending sig (LDS), the lower index first.
__device__ __forceinline__ int rank_of(const float* sig, float s, int c) {
    float n = 0.f;
    for (int k = 0; k < 8; ++k) {
        const int o = (threadIdx.x & 31) + 32 * k;
        n += sig[o] > s || (sig[o] == s && o < c) ? 1.f : 0.f;
    }
    return min(max((int)half_sum(n), 0), P - 1);
}

// Q = U V^T of block j from A = U S and V in memory (the norms S of A's columns in LDS, 256 words at red + 256), its 32
// atoms q of 8, or all of them: alone, and where columns have vanished, which one workgroup completes.
__device__ __forceinline__ void write_factor(const WideArgs& g, int j, unsigned char* mem, unsigned char* lds, float* red,
                                             int* flag, int q, bool alone) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float* GA = reinterpret_cast<float*>(mem + kJaAt);
    float* sig = red + 256;                    // [256] words each
    int* isbad = reinterpret_cast<int*>(red + 512);
    float* vec = red + 768;
    float* coefs = red + 1024;
    float smax = 0.f;
    for (int c = 0; c < P; ++c) smax = fmaxf(smax, sig[c]);
    const float thr = smax * 1e-6f;
    if (tid == 0) *flag = 0;
    __syncthreads();
    if (tid < P) {
        isbad[tid] = !(sig[tid] > thr);
        if (isbad[tid]) *flag = 1;
    }
    __syncthreads();
    const bool bad = *flag != 0;               // uniform over the team
    if (bad && q != 0) return;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(uniform(mem), 0, (int)kTeamBytes, 0x00027000);
    if (bad) {                                 // one workgroup completes the vanished columns, all of A rewritten by itself
        for (int e = tid; e < P * P; e += kNT) {
            const float a = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, e * 4, (int)kJaAt, kPastL1));
            GA[e] = isbad[e / P] ? 0.f : a / sig[e / P];
        }
        __syncthreads();
        for (int c = 0; c < P; ++c) {
            if (!isbad[c]) continue;           // uniform
            if (tid < P) {
                float s = 0.f;
                for (int cc = 0; cc < P; ++cc) s += GA[cc * P + tid] * GA[cc * P + tid];
                vec[tid] = s;
            }
            __syncthreads();
            if (tid == 0) {
                int best = 0;
                for (int r = 1; r < P; ++r)
                    if (vec[r] < vec[best]) best = r;
                *flag = best;
            }
            __syncthreads();
            const int rs = *flag;
            float w = 0.f;
            if (tid < P) {
                float s = (tid == rs) ? 1.f : 0.f;
                for (int cc = 0; cc < P; ++cc) s -= GA[cc * P + rs] * GA[cc * P + tid];
                w = s;
                vec[tid] = s;
            }
            __syncthreads();
            if (tid < P) {
                float dsum = 0.f;
                for (int r = 0; r < P; ++r) dsum += GA[tid * P + r] * vec[r];
                coefs[tid] = dsum;
            }
            __syncthreads();
            if (tid < P) {
                for (int cc = 0; cc < P; ++cc) w -= coefs[cc] * GA[cc * P + tid];
            }
            __syncthreads();
            if (tid < P) vec[tid] = w;
            __syncthreads();
            if (tid < P) {
                float nrm = 0.f;
                for (int r = 0; r < P; ++r) nrm += vec[r] * vec[r];
                GA[c * P + tid] = w / sqrtf(nrm);
            }
            __syncthreads();
        }
    }
    // Q = U V^T, atom-major: D[j][k][r] = sum_c U[r][c] V[k][c]; 32 rows k at a time.  What the other workgroups have left is
    // read past L1, which may still hold the same memory as an earlier block of this launch left it (no barrier of a near team
    // invalidates it); 16 columns at a time through LDS, once for all wavefronts.
    if (bad) stores_done();
    if (tid < P) sig[tid] = bad ? 1.f : 1.f / sig[tid];
    __syncthreads();
    float* strip = reinterpret_cast<float*>(lds);              // [2][16][kLdStrip] (X and Y are dead)
    float* cu = reinterpret_cast<float*>(lds);                 // [16 columns][256], before that
    float* cv = cu + 16 * P;                   // [16 columns][32 rows]
    alone = alone || bad;
    for (int sl = alone ? 0 : q; sl < (alone ? kJacTeam : q + 1); ++sl) {
        const int q0 = 4 * lane, k0 = 4 * wave;
        float o[4][4] = {};
        for (int c0 = 0; c0 < P; c0 += 16) {
            u32x4 u[2], v = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int t = 0; t < 2; ++t)
                u[t] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (tid + t * kNT) * 16, (int)kJaAt + c0 * (P * 4), kPastL1);
            if (tid < 128)                     // 8 units of 16 bytes a column
                v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (tid >> 3) * (P * 4) + 128 * sl + (tid & 7) * 16,
                                                          (int)kJvAt + c0 * (P * 4), kPastL1);
            __syncthreads();                   // the columns before these, or the strip, have been read
#pragma unroll
            for (int t = 0; t < 2; ++t) reinterpret_cast<u32x4*>(cu)[tid + t * kNT] = u[t];
            if (tid < 128) reinterpret_cast<u32x4*>(cv)[tid] = v;
            __syncthreads();
            for (int c = 0; c < 16; ++c) {
                const f32x4 uu = *reinterpret_cast<const f32x4*>(cu + c * P + q0) * sig[c0 + c];
                const f32x4 vv = *reinterpret_cast<const f32x4*>(cv + c * 32 + k0);
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int b = 0; b < 4; ++b) o[a][b] += vv[a] * uu[b];
            }
        }
        __syncthreads();
#pragma unroll
        for (int a = 0; a < 4; ++a)
            *reinterpret_cast<f32x4*>(strip + (k0 + a) * kLdStrip + q0) = f32x4{o[a][0], o[a][1], o[a][2], o[a][3]};
        __syncthreads();
        emit_strip(g, j, 2 * sl, strip, red);
        emit_strip(g, j, 2 * sl + 1, strip + 16 * kLdStrip, red);
    }
}

// One-sided Jacobi for block j by the workgroups q < 8 of a team (t: their barrier); version: the
// numbers the column sets have reached, tbase what they all stand at.  Writes D.
__device__ __forceinline__ Outcome jacobi(const WideArgs& g, int j, const Source& src, Team& t, int* version, int& tbase,
                                          unsigned char* mem, unsigned char* lds, float* red, int* flag) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hw = tid >> 5, l32 = tid & 31, q = t.q;
    float* XA = reinterpret_cast<float*>(lds);  // [16 columns][256] each
    float* XV = XA + 16 * P;
    float* YA = XV + 16 * P;
    float* YV = YA + 16 * P;
    float* GA = reinterpret_cast<float*>(mem + kJaAt);         // [256 columns][256]
    float* GV = reinterpret_cast<float*>(mem + kJvAt);
    float* Gsig = reinterpret_cast<float*>(mem + kSmallAt) + 2 * kRedSize;
    float* Gvinv = Gsig + P;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(uniform(mem), 0, (int)kTeamBytes, 0x00027000);
    auto copy4 = [&](float* dst, const float* from) {          // 16 columns
#pragma unroll
        for (int u = 0; u < 2; ++u)
            reinterpret_cast<f32x4*>(dst)[tid + u * kNT] = reinterpret_cast<const f32x4*>(from)[tid + u * kNT];
    };
    // what another workgroup has left, past L1: 16 columns to LDS, or one to registers; at: bytes into the team's memory
    auto fetch4 = [&](float* dst, int at) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
            reinterpret_cast<u32x4*>(dst)[tid + u * kNT] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (tid + u * kNT) * 16, at, kPastL1);
    };
    auto fetch_column = [&](int at, float (&v)[8]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float2 w = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (hw * P + 2 * l32 + 64 * k) * 4, at, kPastL1));
            v[2 * k] = w.x;
            v[2 * k + 1] = w.y;
        }
    };

    // scale by 1 / max|entry| (the orthogonal factor does not depend on scale)
    float mx = 0.f, scale;
    {
        f32x4 v[2][2];
        load_strip(src, q, v[0]);
        load_strip(src, q + 8, v[1]);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) mx = fmaxf(mx, fabsf(v[s][u][e]));
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        if (lane == 0) red[wave] = mx;
        __syncthreads();
        for (int w = 0; w < kWaves; ++w) mx = fmaxf(mx, red[w]);
        if (!t.sync(mx)) return Outcome::dead;
        mx = row16_max(t.value(0));
        scale = mx > 0.f ? 1.f / mx : 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int e = tid + u * kNT, c = e >> 6, r = 4 * (e & 63);
            reinterpret_cast<f32x4*>(XA)[e] = v[0][u] * scale;
            reinterpret_cast<f32x4*>(YA)[e] = v[1][u] * scale;
            f32x4 ix, iy;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                ix[k] = r + k == 16 * q + c ? 1.f : 0.f;
                iy[k] = r + k == 16 * (q + 8) + c ? 1.f : 0.f;
            }
            reinterpret_cast<f32x4*>(XV)[e] = ix;
            reinterpret_cast<f32x4*>(YV)[e] = iy;
        }
    }

    int rotated = 0;
    // the two sets of a round: si stays while si is the same
    auto sets = [&](int r, int& si, int& sj) {
        if (r < 8) {
            si = q;
            sj = 8 + ((q + r) & 7);
        } else if (r < 12) {
            si = 8 * (q >> 2) + (q & 3);
            sj = 8 * (q >> 2) + 4 + ((q + r) & 3);
        } else if (r < 14) {
            si = 4 * (q >> 1) + (q & 1);
            sj = 4 * (q >> 1) + 2 + ((q + r) & 1);
        } else {
            si = 2 * q;
            sj = 2 * q + 1;
        }
    };
    auto moves = [](int r) { return r == 0 || r == 8 || r == 12 || r == 14; };     // si is new in round r

    float x[8], u[8];
    int sweeps = 0;
    for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
        rotated = 0;
        for (int r = 0; r < 15; ++r) {
            int si, sj;
            sets(r, si, sj);
            const int now = tbase + sweep * 15 + r;
            if (sweep > 0 || r > 0) {
                if (tid == 0)
                    *flag = poll(t.polls, t.near, [&]() {
                        return peek(version + sj) >= now && (!moves(r) || peek(version + si) >= now);
                    });
                __syncthreads();
                if (*flag == 0) return Outcome::dead;
                const int aj = __builtin_amdgcn_readfirstlane(sj) * (16 * P * 4), ai = __builtin_amdgcn_readfirstlane(si) * (16 * P * 4);
                fetch4(YA, (int)kJaAt + aj);
                fetch4(YV, (int)kJvAt + aj);
                if (r == 0) {
                    fetch4(XA, (int)kJaAt + ai);
                    fetch4(XV, (int)kJvAt + ai);
                } else if (moves(r)) {
                    fetch_column((int)kJaAt + ai, x);
                    fetch_column((int)kJvAt + ai, u);
                }
            }
            __syncthreads();
            if (r == 0) {                      // the pairs inside the sets, a tournament of 16
                const int pi = hw & 7;
                float* A = hw < 8 ? XA : YA;
                float* V = hw < 8 ? XV : YV;
                for (int s = 0; s < 15; ++s) {
                    const int ca = pi == 0 ? 15 : (pi + s) % 15, cb = pi == 0 ? s : (15 - pi + s) % 15;
                    const int lo = min(ca, cb), hi = max(ca, cb);
                    float y[8], v[8];
                    get_column(A + lo * P, x);
                    get_column(A + hi * P, y);
                    get_column(V + lo * P, u);
                    get_column(V + hi * P, v);
                    if (rotate(x, y, u, v, rotated)) {
                        put_column(A + lo * P, x);
                        put_column(A + hi * P, y);
                        put_column(V + lo * P, u);
                        put_column(V + hi * P, v);
                    }
                    __syncthreads();
                }
                get_column(XA + hw * P, x);
                get_column(XV + hw * P, u);
            }
            for (int s = 0; s < 16; ++s) {     // the pairs across the sets
                const int cy = (hw + s) & 15;
                float y[8], v[8];
                get_column(YA + cy * P, y);
                get_column(YV + cy * P, v);
                if (rotate(x, y, u, v, rotated)) {
                    put_column(YA + cy * P, y);
                    put_column(YV + cy * P, v);
                }
                __syncthreads();
            }
            copy4(GA + sj * 16 * P, YA);
            copy4(GV + sj * 16 * P, YV);
            const bool leaves = moves(r == 14 ? 0 : r + 1);
            if (leaves) {
                put_column(GA + (si * 16 + hw) * P, x);
                put_column(GV + (si * 16 + hw) * P, u);
            }
            stores_done();
            if (tid == 0) {
                raise_to(version + sj, now + 1, t.near);
                if (leaves) raise_to(version + si, now + 1, t.near);
            }
        }
        sweeps = sweep + 1;
        if (tid == 0) *flag = 0;
        __syncthreads();
        if (rotated) *flag = 1;
        __syncthreads();
        const float mine = *flag ? 1.f : 0.f;
        if (!t.sync(mine)) return Outcome::dead;
        if (!(row16_max(t.value(0)) > 0.f)) break;             // uniform over the team
    }
    tbase += sweeps * 15;
    if (tid == 0 && q == 0 && g.iters_out != nullptr) g.iters_out[j] = sweeps;

    // sigma = column norms; columns of V renormalised.  Sets 2q (x, u) and 2q + 1 (LDS).
    float y[8], v[8];
    get_column(YA + hw * P, y);
    get_column(YV + hw * P, v);
    const int cx = 32 * q + hw, cyy = 32 * q + 16 + hw;        // their columns
    const float sx = column_norm(x), sy = column_norm(y), ix = 1.f / column_norm(u), iy = 1.f / column_norm(v);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        u[k] *= ix;
        v[k] *= iy;
    }
    if (l32 == 0) {
        Gsig[cx] = sx;
        Gsig[cyy] = sy;
        Gvinv[cx] = ix;
        Gvinv[cyy] = iy;
    }
    const bool eig = g.eig_sv != nullptr;
    if (!eig) {                                // (A stands in memory already)
        put_column(GV + cx * P, u);
        put_column(GV + cyy * P, v);
    }
    if (!t.sync(0.f)) return Outcome::dead;
    float* sig = red + 256;
    if (tid < P) sig[tid] = far_load(Gsig + tid);
    __syncthreads();
    if (eig) {
        // atoms = eigenvectors (columns of V) by descending eigenvalue, eig_sv = square roots of the
        // eigenvalues: |A_c| / |V_c|, rescaled
        const int rx = rank_of(sig, sx, cx), ry = rank_of(sig, sy, cyy);
        if (l32 == 0) {
            g.eig_sv[(int64_t)j * P + rx] = sqrtf(sx * ix * mx);
            g.eig_sv[(int64_t)j * P + ry] = sqrtf(sy * iy * mx);
        }
        put_column(g.D + ((int64_t)j * P + rx) * P, u);
        put_column(g.D + ((int64_t)j * P + ry) * P, v);
    } else {
        write_factor(g, j, mem, lds, red, flag, q, false);
    }
    return Outcome::done;
}

// The same by one workgroup that waits for nobody, for what a team has given up: all pairs of columns in 255 rounds
// of 128, straight from memory (31 ms for a block that takes 11 sweeps).  The matrices are the team's, whose other workgroups have left.
__device__ __forceinline__ void jacobi_alone(const WideArgs& g, int j, const Source& src, unsigned char* mem,
                                             unsigned char* lds, float* red, int* flag) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hw = tid >> 5, l32 = tid & 31;
    float* GA = reinterpret_cast<float*>(mem + kJaAt);
    float* GV = reinterpret_cast<float*>(mem + kJvAt);
    float* sig = red + 256;
    float* vinv = red + 768;
    float mx = 0.f;
#pragma unroll 1
    for (int s = 0; s < kTeam; ++s) {
        f32x4 v[2];
        load_strip(src, s, v);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) mx = fmaxf(mx, fabsf(v[u][e]));
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    for (int w = 0; w < kWaves; ++w) mx = fmaxf(mx, red[w]);
    const float scale = mx > 0.f ? 1.f / mx : 0.f;
#pragma unroll 1
    for (int s = 0; s < kTeam; ++s) {
        f32x4 v[2];
        load_strip(src, s, v);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int e = s * (16 * P / 4) + tid + u * kNT, c = e >> 6, r = 4 * (e & 63);
            f32x4 one;
#pragma unroll
            for (int k = 0; k < 4; ++k) one[k] = r + k == c ? 1.f : 0.f;
            reinterpret_cast<f32x4*>(GA)[e] = v[u] * scale;
            reinterpret_cast<f32x4*>(GV)[e] = one;
        }
    }
    stores_done();
    int sweeps = 0;
    bool again = true;
    while (again && sweeps < kMaxSweeps) {
        int rotated = 0;
#pragma unroll 1
        for (int r = 0; r < P - 1; ++r) {
#pragma unroll 1
            for (int i = hw; i < P / 2; i += 2 * kWaves) {     // a tournament of 256
                const int ca = i == 0 ? P - 1 : (r + i) % (P - 1), cb = i == 0 ? r : (r + P - 1 - i) % (P - 1);
                const int lo = min(ca, cb), hi = max(ca, cb);
                float x[8], y[8], u[8], v[8];
                get_column(GA + lo * P, x);
                get_column(GA + hi * P, y);
                get_column(GV + lo * P, u);
                get_column(GV + hi * P, v);
                if (rotate(x, y, u, v, rotated)) {
                    put_column(GA + lo * P, x);
                    put_column(GA + hi * P, y);
                    put_column(GV + lo * P, u);
                    put_column(GV + hi * P, v);
                }
            }
            stores_done();
        }
        ++sweeps;
        if (tid == 0) *flag = 0;
        __syncthreads();
        if (rotated) *flag = 1;
        __syncthreads();
        again = *flag != 0;                    // uniform
        __syncthreads();
    }
    if (tid == 0) {
        g.fallback[j] = 1;
        if (g.iters_out != nullptr) g.iters_out[j] = sweeps;
    }
    for (int c = hw; c < P; c += 2 * kWaves) { // sigma = column norms; columns of V renormalised
        float x[8], u[8];
        get_column(GA + c * P, x);
        get_column(GV + c * P, u);
        const float sc = column_norm(x), ic = 1.f / column_norm(u);
#pragma unroll
        for (int k = 0; k < 8; ++k) u[k] *= ic;
        put_column(GV + c * P, u);
        if (l32 == 0) {
            sig[c] = sc;
            vinv[c] = ic;
        }
    }
    stores_done();
    if (g.eig_sv == nullptr) {
        write_factor(g, j, mem, lds, red, flag, 0, true);
        return;
    }
    for (int c = hw; c < P; c += 2 * kWaves) {
        float u[8];
        get_column(GV + c * P, u);
        const int rc = rank_of(sig, sig[c], c);
        if (l32 == 0) g.eig_sv[(int64_t)j * P + rc] = sqrtf(sig[c] * vinv[c] * mx);
        put_column(g.D + ((int64_t)j * P + rc) * P, u);
    }
}

// The same two, called: inlined beside Newton-Schulz, whose operands take all registers, they cost it 100 spilled ones.
// Everything by value (what a call could change through a pointer would live in memory from the start).
struct JacobiResult {
    Outcome how;
    int epoch;                 // of the barrier
    int tbase;
};
__device__ __attribute__((noinline)) JacobiResult jacobi_called(WideArgs g, int j, Source src, Team t, int* version, int tbase,
                                                                unsigned char* mem, unsigned char* lds, float* red, int* flag) {
    const Outcome how = jacobi(g, j, src, t, version, tbase, mem, lds, red, flag);
    return {how, t.epoch, tbase};
}
__device__ __attribute__((noinline)) void jacobi_alone_called(WideArgs g, int j, Source src, unsigned char* mem,
                                                              unsigned char* lds, float* red, int* flag) {
    jacobi_alone(g, j, src, mem, lds, red, flag);
}

// A team of pairs without its helpers: called for the same reason.
struct NewtonSchulzResult {
    Outcome how;
    int steps;
};
__device__ __attribute__((noinline)) NewtonSchulzResult newton_schulz_called(WideArgs g, int j, Source src, Team t, unsigned char* mem,
                                                                             unsigned char* lds, float* red) {
    int steps = 0;
    const Outcome how = newton_schulz<1>(g, j, src, t, nullptr, mem, lds, red, nullptr, steps);
    return {how, steps};
}

// NS: Newton-Schulz first; otherwise Jacobi for every block.  PAIRS: teams of 32, which have one block each.
template <bool NS, bool PAIRS>
__global__ __launch_bounds__(kNT) void wide_polar_kernel(WideArgs g) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    // The 16 workgroups of a team lie eight apart: workgroups go round the eight XCDs, so a team shares an L2
    // (spread: next to each other).
    const int team_wgs = wide_team_wgs(g.teams, g.spread, PAIRS);
    if ((int)blockIdx.x >= team_wgs) {         // uniform: the workgroups of the squared-error total
        const int b = (int)blockIdx.x - team_wgs;
        if (g.sq.out != nullptr && b < g.sq.nb)
            sq_total_part<kNT>(g.sq.err, g.sq.m, b, g.sq.nb, g.sq.part, g.sq.counter, g.sq.out,
                               reinterpret_cast<double*>(lds));
        return;
    }
    const int team = PAIRS ? (int)blockIdx.x % 8 : g.spread ? (int)blockIdx.x / 16 : (int)blockIdx.x / 128 * 8 + (int)blockIdx.x % 8;
    const int q = PAIRS ? (int)blockIdx.x / 8 : g.spread ? (int)blockIdx.x % 16 : (int)blockIdx.x % 128 / 8;
    constexpr int kSize = PAIRS ? kPairs : kTeam;
    if (team >= g.teams) return;               // uniform
    float* red = reinterpret_cast<float*>(lds + kSmallLds);
    int* flag = reinterpret_cast<int*>(red + 1280);
    unsigned char* mem = g.data + (size_t)team * kTeamBytes;
    int* sync = g.sync + team * kSyncInts;
    float* small = reinterpret_cast<float*>(mem + kSmallAt);
    Team all = {sync + kFlagsAt, small, flag, kSize, q, g.polls, 0, false};
    Team eight = {sync + kFlagsJacAt, small + kRedSize, flag + 1, kJacTeam, q, g.polls, 0, false};
    int tbase = 0;
    const int blocks = (g.K - 1 - team) / g.teams + 1;         // of this team
    int undone = blocks;

    unsigned long long* count = reinterpret_cast<unsigned long long*>(sync + kMeetAt);
    bool alive = NS || all.meet(count), met = !NS;
    eight.near = all.near;

    // where P_j comes from; false: no signals, the block keeps its basis
    auto source = [&](int j, Source& src) {
        if (g.M != nullptr) {
            src = {g.M + (int64_t)j * P * P, 1};
            return g.counts == nullptr || g.counts[j] != 0;
        }
        int before = 0, own = 0;           // every wavefront for itself; one trip for up to 64 blocks
        for (int jj = lane; jj <= j; jj += 64) {
            own = g.offsets[jj + 1] - g.offsets[jj];
            before += (own + g.piece - 1) / g.piece;
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) before += __shfl_xor(before, o, 64);
        const int n_j = __builtin_amdgcn_readlane(own, j & 63), pieces = (n_j + g.piece - 1) / g.piece;
        src = {g.partial + (int64_t)(__builtin_amdgcn_readfirstlane(before) - pieces) * P * P, pieces};
        return n_j != 0;
    };
    for (int j = team; alive && j < g.K; j += g.teams) {
        Source src;
        if (!source(j, src)) {                 // uniform over the team
            if (q == 0 && tid == 0) {
                g.fallback[j] = 0;
                if (g.iters_out != nullptr) g.iters_out[j] = 0;
            }
            --undone;
            continue;
        }
        Outcome how = Outcome::left;
        if constexpr (NS) {
            int steps = 0;
            if constexpr (PAIRS) {
                how = g.helper_polls < 0 && q >= kTeam ? Outcome::alone
                                                       : newton_schulz<2>(g, j, src, all, count, mem, lds, red, sync + kPairAt, steps);
                if (how == Outcome::alone) {   // uniform over the team
                    if (q >= kTeam) {          // nobody waits for this workgroup
                        --undone;
                        break;
                    }
                    all.size = kTeam;
                    const NewtonSchulzResult r = newton_schulz_called(g, j, src, all, mem, lds, red);
                    how = (Outcome)__builtin_amdgcn_readfirstlane((int)r.how);
                    steps = __builtin_amdgcn_readfirstlane(r.steps);
                }
            } else {
                how = newton_schulz<1>(g, j, src, all, met ? nullptr : count, mem, lds, red, nullptr, steps);
            }
            met = true;
            eight.near = all.near;
            if (q == 0 && tid == 0) {
                g.fallback[j] = how == Outcome::left;
                if (g.iters_out != nullptr && how == Outcome::done) g.iters_out[j] = -steps;
            }
            if (how == Outcome::done && all.size == kTeam) emit_strip(g, j, q, reinterpret_cast<const float*>(lds + kStripAt), red);
        }
        if (how == Outcome::left) {
            __syncthreads();
            how = Outcome::done;
            if (q < kJacTeam) {
                if constexpr (NS) {
                    const JacobiResult r = jacobi_called(g, j, src, eight, sync + kVersionAt, tbase, mem, lds, red, flag);
                    how = (Outcome)__builtin_amdgcn_readfirstlane((int)r.how);
                    eight.epoch = __builtin_amdgcn_readfirstlane(r.epoch);
                    tbase = __builtin_amdgcn_readfirstlane(r.tbase);
                } else
                    how = jacobi(g, j, src, eight, sync + kVersionAt, tbase, mem, lds, red, flag);
            }
        }
        alive = how != Outcome::dead;
        if (alive) {
            --undone;
        } else if (tid == 0) {
            all.gone();
            eight.gone();
        }
        __syncthreads();
    }
    // The last workgroup of the team to leave (the release and acquire of the agent scope hand it what the others
    // have written) does what there is left to do and sets the counters back.
    stores_done();
    if (tid == 0) {
        if (undone > 0) __hip_atomic_fetch_max(sync + kUndoneAt, undone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        flag[0] = __hip_atomic_fetch_add(sync + kExitAt, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == kSize - 1;
        flag[1] = flag[0] ? __hip_atomic_load(sync + kUndoneAt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    }
    __syncthreads();
    if (flag[0] == 0) return;                  // uniform
    const int rest = flag[1];
    for (int n = blocks - rest; n < blocks; ++n) {
        const int j = team + n * g.teams;
        Source src;
        __syncthreads();                       // flag and the reductions are read
        if (source(j, src)) {
            if constexpr (NS) jacobi_alone_called(g, j, src, mem, lds, red, flag);
            else jacobi_alone(g, j, src, mem, lds, red, flag);
        } else if (tid == 0) {
            g.fallback[j] = 0;
            if (g.iters_out != nullptr) g.iters_out[j] = 0;
        }
    }
    for (int e = tid; e < (PAIRS ? kSyncInts : kPairAt); e += kNT) {
        const bool in_l2 = all.near && (e < kMeetAt || e >= kPairAt) && e != kExitAt && e != kUndoneAt;
        if (in_l2 || rest > 0) {               // (rest > 0: this workgroup may have left without knowing that it is near)
            __hip_atomic_store(sync + e, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        if (!in_l2 || rest > 0) __hip_atomic_store(sync + e, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

}  // namespace

// Pairs take a whole XCD for a team, so they are for launches that have the chip to themselves: with contexts of this size on a second
// stream, a team of one launch and a team of the other one, which share an XCD otherwise, would follow one another.  Two SVDs on two
// streams, 2 to 8 blocks of a training round: 73 to 75 us together, in pairs 110 to 118.  One alone, 1 to 8 blocks: 58 to 60 us in
// pairs, 9 blocks, by teams of 16, 72.
bool wide_pairs(int K, int device) { return K <= kMaxPairTeams && wide_streams(device) < 2; }

size_t polar_wide_scratch_bytes(int K) { return (size_t)(K < kMaxTeams ? K : kMaxTeams) * kTeamBytes; }
size_t polar_wide_sync_bytes(int K) { return (size_t)(K < kMaxTeams ? K : kMaxTeams) * kSyncInts * sizeof(int); }

hipError_t launch_polar_wide(int K, const float* M, const float* partial, const int32_t* offsets, int piece,
                             const int32_t* counts, float* D, const DictOps& ops, bool newton_schulz_first,
                             float* eig_sv, const Workspace& ws, const SqTotalArgs& sq, hipStream_t st) {
    constexpr int kMaxIters = 26;
    if (ws.wide == nullptr || ws.wide_sync == nullptr || ws.raised == nullptr) return hipErrorInvalidValue;
    WideArgs a;
    a.M = M;
    a.partial = partial;
    a.offsets = offsets;
    a.piece = piece;
    a.counts = counts;
    a.D = D;
    a.ops = ops;
    a.eig_sv = eig_sv;
    a.fallback = ws.ns_fallback;
    a.iters_out = ws.sweeps;
    a.max_iters = kMaxIters;
    a.K = K;
    a.teams = K < kMaxTeams ? K : kMaxTeams;
    a.data = reinterpret_cast<unsigned char*>(ws.wide);
    a.sync = ws.wide_sync;
    a.sq = sq;
    a.spread = wide_streams(ws.device) > 2;
    a.polls = ws.wide_polls;
    a.helper_polls = ws.wide_helpers ? (a.polls < kHelperPolls ? a.polls : kHelperPolls) : -1;
    const bool pairs = newton_schulz_first && wide_pairs(K, ws.device);
    const unsigned grid = (unsigned)(wide_team_wgs(a.teams, a.spread, pairs) + (sq.out != nullptr ? sq.nb : 0));
    auto* kernel = pairs ? &wide_polar_kernel<true, true> : newton_schulz_first ? &wide_polar_kernel<true, false>
                                                                                : &wide_polar_kernel<false, false>;
    if (hipError_t e = ws.raised->ensure(reinterpret_cast<const void*>(kernel), kLds); e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kNT), kLds, st, a);
    return hipGetLastError();
}

}  // namespace sbo
