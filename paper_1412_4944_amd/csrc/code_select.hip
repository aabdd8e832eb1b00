// Sparse-coding stage 2: support, coefficients and residual of every signal in the
// block that won the energy comparison (Section 2: x = Q_j^T y hard-thresholded to the
// s0 entries of largest magnitude; Algorithm 1, steps 3-4).
//
// Signals arrive grouped by block (perm/offsets), or every workgroup lists those of its own tiles (Source).  One wavefront
// takes a tile of up to 32 signals of ONE block, so the projection is again one fp32 MFMA tile product with
// atoms on M and signals on N; every signal's p coefficients then sit in two lanes.
// The s0-th largest magnitude tau is found with the same compare-exchange networks as
// in stage 1, and the support {|c| > tau} plus the lowest-index entries equal to tau is
// written in ascending atom order.  Exact ties in magnitude beyond the trivial one are
// resolved by a sequential per-signal pass (rare).
#include <algorithm>

#include "sbo_internal.h"
#include "device_utils.h"
#include "select_tile.h"

namespace sbo {

namespace {

// How a select kernel finds the signals of its tiles: from the grouping; from all choices of a small set (group_in_select),
// GroupInKernel; from the choice's histograms (lists_in_select), ChunkLists.
enum Source { kGrouped, kSmall, kLists };

// kSmall: a small set (group_in_select) without a grouping launch: every workgroup reads all choices and every wavefront finds
// the signals of its tile among them (225 signals, K = 32, p = 64: 11.8 us with a sort of them all in LDS).
template <int P, int S0, Source SRC>
__global__ __launch_bounds__(256) void select_kernel(const float* __restrict__ Y,
                                                     const float* __restrict__ D, int K,
                                                     const int32_t* __restrict__ offsets,
                                                     const int32_t* __restrict__ perm,
                                                     int32_t* __restrict__ supp,
                                                     float* __restrict__ coef,
                                                     float* __restrict__ err, GroupInKernel g, ChunkLists lists) {
    constexpr int KS = P / 2;
    constexpr int QN = P / 8;
    constexpr int MT = P >= 32 ? P / 32 : 1;   // 32-row tiles per block
    extern __shared__ __attribute__((aligned(16))) int lds[];      // stage[4][...] | ties[4][...]
    int* stage_all = lds;
    float* ties_all = reinterpret_cast<float*>(stage_all + 4 * kSelectStageWords<S0>);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int h = lane >> 5, n = lane & 31;

    // behind the tiles: ids[4][32]; kSmall: count[K] | choice[m]; kLists: the table in the place of the tiles (and longer, maybe)
    constexpr int kTiles = 4 * (kSelectStageWords<S0> + kSelectTieWords);
    int* ids = lds + (SRC == kLists ? max(kTiles, ChunkLists::table_ints(4, K, lists.n_chunks)) : kTiles) + wave * 32;
    int *count = ids + (4 - wave) * 32, *choice = count + K;
    if constexpr (SRC == kSmall) g.choose<256>(K, choice, count);
    if constexpr (SRC == kLists) lists.load<4>(K, lds);
    const Piece pc = find_piece([&](int j) {
        if constexpr (SRC == kSmall) return count[j];
        else if constexpr (SRC == kLists) return lists.count_of<4>(K, lds, j);
        else return offsets[j + 1] - offsets[j];
    }, K, 32, (int)blockIdx.x * 4 + wave);
    if constexpr (SRC == kLists) {
        if (pc.j >= 0) lists.collect<1>(K, lds, pc, ids, 0);
        __syncthreads();                       // the table is dead
    }
    if (pc.j < 0) return;                      // no workgroup barrier below this line
    if constexpr (SRC == kSmall) g.list(choice, pc, ids);
    const int j = pc.j;
    const bool active = n < pc.count;
    const int64_t i = active ? (SRC != kGrouped ? ids[n] : perm[pc.before + pc.rank + n]) : -1;

    // B operand: this lane's half of the dims of signal i.
    float yb[KS];
    if (active) {
        const f32x4* src = reinterpret_cast<const f32x4*>(Y + i * P + h * KS);
#pragma unroll
        for (int q = 0; q < QN; ++q) {
            f32x4 v = src[q];
            yb[4 * q + 0] = v.x;
            yb[4 * q + 1] = v.y;
            yb[4 * q + 2] = v.z;
            yb[4 * q + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int t = 0; t < KS; ++t) yb[t] = 0.f;
    }

    // Projection c = Q_j^T y for the tile.
    f32x16 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mt][r] = 0.f;
        const int row = mt * 32 + n;           // atom fed by this lane into the A operand
        const f32x4* arow =
            reinterpret_cast<const f32x4*>(D + ((int64_t)j * P + (row < P ? row : 0)) * P + h * KS);
#pragma unroll
        for (int q = 0; q < QN; ++q) {
            f32x4 a = arow[q];
            if (row >= P) a = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                acc[mt] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[kk], yb[4 * q + kk], acc[mt], 0, 0, 0);
        }
    }

    tile_select<P, S0>(acc, h, n, active, i, ties_all + wave * kSelectTieWords, stage_all + wave * kSelectStageWords<S0>, supp,
                       coef, err);
}

// The same with the six bf16 products (every arithmetic but SBO_ARITH_F32), for larger sets.  A workgroup takes a piece of
// one block, whose Q_j it splits into LDS, in operand order, once; its NW wavefronts take every NW-th tile of 32 signals.
// What bounds select_kernel is not its matrix work (4100 cycles a tile) but that every lane reads its own row of Q_j:
// 64 lines an instruction, 16 instructions a tile, and few of them in flight; here a tile reads LDS and has 1500 cycles
// of matrix work, and what is left is the selection's instructions (select_tile.h).  Coefficients against 64 bits, of
// |y|: rms 2.3e-8 to 5.5e-8 (select_kernel 3.1e-8 to 8.5e-8), at most 3.1e-7 (4.6e-7).
template <int P, int S0, int NW, bool LISTS>
__global__ __launch_bounds__(64 * NW, 4) void select_split_kernel(const float* __restrict__ Y, const float* __restrict__ D,
                                                                  int K, int piece,
                                                                  const int32_t* __restrict__ offsets,
                                                                  const int32_t* __restrict__ perm,
                                                                  int32_t* __restrict__ supp, float* __restrict__ coef,
                                                                  float* __restrict__ err, ChunkLists lists) {
    constexpr int KS16 = P / 16, MT = P / 32, Q_U = MT * KS16 * 3 * 64;

    extern __shared__ __attribute__((aligned(16))) int lds_all[];  // ids[piece] (LISTS) | Qs[Q_U] | stage[NW][..] | ties[NW][..]
    int *ids = lds_all, *lds = lds_all + (LISTS ? piece : 0);  // (a multiple of 32); LISTS: the table in the place of the latter
    u32x4* Qs = reinterpret_cast<u32x4*>(lds);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, n = lane & 31;

    if constexpr (LISTS) lists.load<NW>(K, lds);
    const Piece pc = find_piece([&](int j) { return LISTS ? lists.count_of<NW>(K, lds, j) : offsets[j + 1] - offsets[j]; }, K, piece,
                                (int)blockIdx.x);
    if (pc.j < 0) return;                      // uniform over the workgroup
    if constexpr (LISTS) {
        lists.collect<NW>(K, lds, pc, ids, wave);
        __syncthreads();                       // the table is dead
    }
    const int j = pc.j, pos0 = pc.before + pc.rank, cnt = pc.count, n_tiles = (cnt + 31) >> 5;

    // Ids two tiles ahead, rows one tile ahead (lanes past the end take the last signal of the piece once more and keep
    // nothing of it).
    auto tile_id = [&](int t) -> int {
        const int at = min(t * 32 + n, cnt - 1);
        return LISTS ? ids[at] : perm[pos0 + at];
    };
    f32x4 raw[KS16][2];                        // this lane's dims ks*16 + h*8 .. +7 of its signal
    auto load_rows = [&](int sid) {
        const f32x4* src = reinterpret_cast<const f32x4*>(Y + (int64_t)sid * P + h * 8);
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) {
            raw[ks][0] = src[ks * 4];
            raw[ks][1] = src[ks * 4 + 1];
        }
    };
    int i_cur = tile_id(wave), i_next = tile_id(wave + NW);
    load_rows(i_cur);
#pragma unroll
    for (int g = wave; g < MT * KS16; g += NW) {
        const int ks = g % KS16, atom = (g / KS16) * 32 + n;
        const f32x4* src = reinterpret_cast<const f32x4*>(D + ((int64_t)j * P + atom) * P + ks * 16 + h * 8);
        const f32x4 v[2] = {src[0], src[1]};
        split_unit(v, Qs + g * 3 * 64 + lane, 64);
    }
    __syncthreads();

    int* stage = lds + Q_U * 4 + wave * kSelectStageWords<S0>;
    float* ties = reinterpret_cast<float*>(lds + Q_U * 4 + NW * kSelectStageWords<S0>) + wave * kSelectTieWords;
    for (int tile = wave; tile < n_tiles; tile += NW) {
        const int64_t i = i_cur;
        u32x4 yq[KS16][3];
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) split_unit(raw[ks], yq[ks], 1);
        i_cur = i_next;
        i_next = tile_id(tile + 2 * NW);
        load_rows(i_cur);

        constexpr int TA[6] = {2, 0, 1, 1, 0, 0}, TB[6] = {0, 2, 1, 0, 1, 0};      // smallest products first
        f32x16 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x16{};
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) {
            u32x4 a[MT][3];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) a[mt][pl] = Qs[((mt * KS16 + ks) * 3 + pl) * 64 + lane];
#pragma unroll
            for (int t = 0; t < 6; ++t)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[mt][TA[t]]),
                                                                      __builtin_bit_cast(bf16x8, yq[ks][TB[t]]),
                                                                      acc[mt], 0, 0, 0);
        }
        // An infinite entry has no three parts (infinity less itself): the coefficients of such a signal in fp32.
        const bool bad = acc[0][0] != acc[0][0];
        if (__any(bad)) {                      // uniform, rare
            const float* row = Y + i * P;
#pragma unroll 1
            for (int d = 0; d < P; ++d) {
                const float y = row[d];
#pragma unroll
                for (int f = 0; f < MT * 16; ++f) {
                    const int atom = (f >> 4) * 32 + ((f & 15) >> 2) * 8 + h * 4 + (f & 3);
                    const float c = fmaf(D[((int64_t)j * P + atom) * P + d], y, d == 0 ? 0.f : acc[f >> 4][f & 15]);
                    acc[f >> 4][f & 15] = bad ? c : acc[f >> 4][f & 15];
                }
            }
        }
        tile_select<P, S0>(acc, h, n, tile * 32 + n < cnt, i, ties, stage, supp, coef, err);
    }
}

// Variant for p > 64.  The p coefficients of a signal no longer fit the registers of a
// lane pair next to the signal itself, so the projection is produced 32 atoms at a time,
// written to a wave-private LDS tile [signal][atom] while the lane keeps a running sorted
// top-S of the magnitudes; the support is then emitted from the tile, each lane of a pair
// walking one half of the atoms in index order (which resolves magnitude ties directly).
template <int P, int S>
__global__ __launch_bounds__(256) void select_wide_kernel(const float* __restrict__ Y,
                                                          const f32x4* __restrict__ Dsw, int K, int s0,
                                                          const int32_t* __restrict__ offsets,
                                                          const int32_t* __restrict__ perm,
                                                          int32_t* __restrict__ supp,
                                                          float* __restrict__ coef,
                                                          float* __restrict__ err, int by_pos) {
    constexpr int KS = P / 2;
    constexpr int QN = P / 8;
    constexpr int MT = P / 32;
    constexpr int LDC = P + 1;
    constexpr int QCH = 8;                     // operand groups loaded ahead of their MFMAs
    static_assert(S <= 16 && QN % QCH == 0, "shape");

    extern __shared__ __attribute__((aligned(16))) int lds[];      // ctile[4][32][LDC]
    float* ctile_all = reinterpret_cast<float*>(lds);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int h = lane >> 5, n = lane & 31;

    const Piece pc = find_piece([&](int j) { return offsets[j + 1] - offsets[j]; }, K, 32, (int)blockIdx.x * 4 + wave);
    if (pc.j < 0) return;                      // no workgroup barrier below this line
    const int j = pc.j;
    const bool active = n < pc.count;
    const int64_t i = active ? perm[pc.before + pc.rank + n] : -1;

    float yb[KS];
    if (active) {
        const f32x4* src = reinterpret_cast<const f32x4*>(Y + i * P + h * KS);
#pragma unroll
        for (int q = 0; q < QN; ++q) {
            f32x4 v = src[q];
            yb[4 * q + 0] = v.x;
            yb[4 * q + 1] = v.y;
            yb[4 * q + 2] = v.z;
            yb[4 * q + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int t = 0; t < KS; ++t) yb[t] = 0.f;
    }

    float* ct = ctile_all + wave * 32 * LDC + n * LDC;     // this lane's signal row
    float run[S];
#pragma unroll
    for (int t = 0; t < S; ++t) run[t] = 0.f;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                         0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // A operand = rows of Q_j straight from L2, QCH 16-byte groups per chunk; the next chunk is
    // requested before the MFMAs of the current one (a wavefront has its SIMD to itself here,
    // so nothing else would cover the load latency).
    // Dsw is Q in the coding kernel's operand order (dict_swizzle_kernel): stage of 64 rows,
    // unit (mt2*QN + q)*64 + lane = dims h*P/2 + 4q.. of row stage*64 + mt2*32 + n, so a
    // wavefront's load is 1 KiB contiguous and the four wavefronts of a workgroup (tiles of the
    // same block, in step) ask for the same lines.
    auto load_chunk = [&](f32x4 (&a)[QCH], int mt, int q0) {
        const f32x4* src = Dsw + ((int64_t)j * (P / 64) + (mt >> 1)) * (2 * QN * 64) +
                           ((mt & 1) * QN + q0) * 64 + lane;
#pragma unroll
        for (int q = 0; q < QCH; ++q) a[q] = src[q * 64];
    };
    constexpr int NCH = QN / QCH;              // chunks per tile row of atoms
    static_assert(NCH == 4, "the operand ring below has four slots, one per chunk of a row");
    // chunk t (t = mt * NCH + cc) lives in slot cc; it is requested two chunks ahead
    f32x4 abuf[NCH][QCH];
    load_chunk(abuf[0], 0, 0);
    load_chunk(abuf[1], 0, QCH);
#pragma unroll 1
    for (int mt = 0; mt < MT; ++mt) {
        f32x16 acc = zero;
#pragma unroll
        for (int cc = 0; cc < NCH; ++cc) {
            // the last two requests of all re-read a valid row and are not used
            const int nmt = cc + 2 < NCH ? mt : min(mt + 1, MT - 1);
            load_chunk(abuf[(cc + 2) % NCH], nmt, ((cc + 2) % NCH) * QCH);
#pragma unroll
            for (int q = 0; q < QCH; ++q)
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(abuf[cc][q][kk],
                                                               yb[4 * (cc * QCH + q) + kk], acc, 0, 0, 0);
        }
        float x[16], top[S];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int atom = mt * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
            ct[atom] = acc[r];
            x[r] = fabsf(acc[r]);
        }
        top_sorted<16, S>(x, top);
        if (mt == 0) {
#pragma unroll
            for (int t = 0; t < S; ++t) run[t] = top[t];
        } else {
#pragma unroll
            for (int t = 0; t < S; ++t) run[t] = fmaxf(run[t], top[S - 1 - t]);
            bitonic_merge_desc<S>(run);
        }
    }

    // tau = s0-th largest magnitude of the signal
    float oth[S], mrg[S];
#pragma unroll
    for (int t = 0; t < S; ++t) oth[t] = other_half(run[t]);
#pragma unroll
    for (int t = 0; t < S; ++t) mrg[t] = fmaxf(run[t], oth[S - 1 - t]);
    bitonic_merge_desc<S>(mrg);
    float tau = mrg[0];
#pragma unroll
    for (int t = 1; t < S; ++t) tau = (t == s0 - 1) ? mrg[t] : tau;

    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    // lane h of a pair owns atoms [h*P/2, (h+1)*P/2) of its signal
    const float* mine = ct + h * (P / 2);
    int gt_own = 0, eq_own = 0;
#pragma unroll 16
    for (int k = 0; k < P / 2; ++k) {
        const float a = fabsf(mine[k]);
        gt_own += a > tau;
        eq_own += a == tau;
    }
    const int64_t at = by_pos ? pc.before + pc.rank + n : i;
    const int gt_oth = other_half(gt_own), eq_oth = other_half(eq_own);
    const int need = s0 - (gt_own + gt_oth);   // entries equal to tau to take, lowest index first
    const int gt_lo = h ? gt_oth : gt_own, eq_lo = h ? eq_oth : eq_own;
    const int eq_lo_taken = min(eq_lo, need);
    int pos = h ? gt_lo + eq_lo_taken : 0;
    int eq_taken = h ? eq_lo_taken : 0;
    float dropped = 0.f;
#pragma unroll 16
    for (int k = 0; k < P / 2; ++k) {
        const float v = mine[k];
        const float a = fabsf(v);
        bool take = a > tau;
        if (!take && a == tau && eq_taken < need) {
            take = true;
            ++eq_taken;
        }
        if (take) {
            if (active && pos < s0) {
                supp[at * s0 + pos] = h * (P / 2) + k;
                coef[at * s0 + pos] = v;
            }
            ++pos;
        } else {
            dropped += v * v;
        }
    }
    dropped += other_half(dropped);
    if (active && h == 0) err[at] = dropped;
}

// p = 256 on the bf16 matrix cores (see energy_split_kernel for the arithmetic): a workgroup has one tile of 32 signals of
// ONE block.  Its eight wavefronts share out the atoms (32 each; rows of Dsb, the dictionary in the split operand order of
// dict_parts_kernel, straight from L2, every row used once) and then the signals (four each, 16 lanes to a signal, 16
// consecutive atoms per lane).  The signals' parts are made once, by all, in LDS, whose place the coefficients take.
// What bounds it: nothing alone.  A tile's products take a CU 6100 cycles, its selection 5000 cycles of vector issue, and its
// rows and signals come in several trips; three workgroups on a CU (three contraction steps ahead, 80 registers) fill one another's gaps.
// With a tile per wavefront, four to a workgroup and one workgroup per CU (projection and signal in 320 registers, rows
// through LDS) a tile took 38 us however few there were, and nothing hid its selection.  Before and now: 2048 signals, K = 1
// 43.2 -> 17 us, 5041, K = 16 42.4 -> 19, 16384 46 -> 33, 32768 86 -> 55, 131072 212 -> 159 (two workgroups per CU, six steps
// ahead 172).
// F16: two fp16 parts and three partial products (device_utils.h), every signal scaled by a power of two, where the dictionary has them
// (select_arith in sbo_api.hip): half of the chain of products that the wavefronts of a tile go through, two thirds of the rows'
// bytes (a tile reads all of its block's: 384 KiB, now 256).  131072 signals, K = 16 143 -> 116 us, 5041, K = 16 17.2 -> 14.4.  The products with a second part are
// summed apart: the coefficients are off those in 64 bits by 0.9e-7 of theirs on average, by six bf16 products 2.0e-7 (rms; s0 = 2 to 12).  A caller's dictionary may have atoms of any size: a
// wavefront with one that these parts do not represent well (dodd) makes them of its rows of D, each scaled by itself.
// Workgroup ids are dealt out so that the workgroups of one XCD (ids equal modulo 8) take a contiguous run of tiles, that is,
// few blocks, whose rows then stay in that XCD's L2 (131072 signals, K = 16: 190 -> 172 us).
constexpr int kTileWaves = 8;
constexpr int kTileLd = 260;                  // floats per signal of the coefficients (16-byte units cover all banks)
// Bytes of the parts of y, of the coefficients, and of the table of `lists`, in one place (the table of few_entries takes most).
template <bool LISTS, bool F16>
constexpr size_t kTileRoom = LISTS || !F16 ? 256 / 16 * 3 * 64 * 16 : 32 * kTileLd * 4;
template <int S, bool LISTS, bool F16>
__global__ __launch_bounds__(64 * kTileWaves, 6) void select_wide_split_kernel(const float* __restrict__ Y, const float* __restrict__ D,
                                                                 const u32x4* __restrict__ Dsb, const int* __restrict__ dodd,
                                                                 int K, int s0, const int32_t* __restrict__ offsets,
                                                                 const int32_t* __restrict__ perm,
                                                                 int32_t* __restrict__ supp, float* __restrict__ coef,
                                                                 float* __restrict__ err, int by_pos, ChunkLists lists) {
    constexpr int P = 256, KS16 = P / 16, MT = P / 32, AHEAD = 3, NW = kTileWaves, L = 16;
    constexpr int NPT = F16 ? 2 : 3;           // parts
    constexpr int STAGE_U = KS16 * NPT * 64;   // 16-byte units of 32 rows
    extern __shared__ __attribute__((aligned(16))) int lds[];  // parts of y, then coefficients | stage | ids[32] (LISTS)
    u32x4* ys = reinterpret_cast<u32x4*>(lds);                 // [KS16][NPT][64]
    float* cs = reinterpret_cast<float*>(ys);                  // [32][kTileLd]
    int* stage = lds + kTileRoom<LISTS, F16> / 4;              // [32][2][16]; before that, largest magnitudes [8][32] (F16)
    int* ids = stage + 32 * 32;
    static_assert(32 * kTileLd * 4 <= kTileRoom<LISTS, F16> && STAGE_U * 16 <= kTileRoom<LISTS, F16>, "parts and coefficients fit");

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, n = lane & 31;
    const int per_xcd = gridDim.x >> 3;        // the grid is a multiple of 8 (launcher)
    const int id = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    int* table = reinterpret_cast<int*>(ys);   // LISTS: in the place of the signals
    if constexpr (LISTS) lists.load<NW>(K, table);
    const Piece pc = find_piece([&](int j) { return LISTS ? lists.count_of<NW>(K, table, j) : offsets[j + 1] - offsets[j]; }, K, 32, id);
    if (pc.j < 0) return;                      // uniform over the workgroup
    if constexpr (LISTS) {
        lists.collect<NW>(K, table, pc, ids, wave);
        __syncthreads();                       // the table is dead
    }
    const int j = pc.j, pos0 = pc.before + pc.rank, cnt = pc.count;

    // A operand: rows of this wavefront's 32 atoms, AHEAD contraction steps on their way
    const u32x4* Qj = Dsb + ((int64_t)j * MT + wave) * STAGE_U + lane;
    u32x4 a[AHEAD][NPT];
    auto fetch = [&](u32x4 (&v)[NPT], int ks) {
#pragma unroll
        for (int pl = 0; pl < NPT; ++pl) v[pl] = Qj[(ks * NPT + pl) * 64];
    };
    int odd = 0;                               // F16: of this wavefront's atoms (uniform)
    if constexpr (F16) {
        const int at = __builtin_amdgcn_readfirstlane(j) * (P / 16) + 2 * wave;
        odd = dodd[at] | dodd[at + 1];
    }
    int shift = 0;                             // F16: signal n is scaled by 2^shift, its largest magnitude then in [2^13, 2^14)
    {
        const int64_t i = n < cnt ? (LISTS ? ids[n] : perm[pos0 + n]) : -1;
        f32x4 v[KS16 / NW][2];
#pragma unroll
        for (int q = 0; q < KS16 / NW; ++q)     // steps NW q + wave: dims ks*16 + h*8 .. +7 of signal n
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                v[q][e] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (i >= 0) v[q][e] = reinterpret_cast<const f32x4*>(Y + i * P + (NW * q + wave) * 16 + h * 8)[e];
            }
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) fetch(a[t], t);
        if constexpr (F16) {
            unsigned mx = 0;
#pragma unroll
            for (int q = 0; q < KS16 / NW; ++q)
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float m = fabsf(v[q][e][c]);
                        mx = max(mx, __builtin_bit_cast(unsigned, m));
                    }
            mx = max(mx, pair_other(mx, h));
            if (h == 0) stage[wave * 32 + n] = (int)mx;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NW; ++w) mx = max(mx, (unsigned)stage[w * 32 + n]);
            const int e = (int)(mx >> 23);
            shift = e == 0xff ? 0 : 140 - max(e, 1);
#pragma unroll
            for (int q = 0; q < KS16 / NW; ++q) {
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[q][e][c] = __builtin_amdgcn_ldexpf(v[q][e][c], shift);
                const F16x2Pair x = split_f16x2(v[q][0].x, v[q][0].y), y = split_f16x2(v[q][0].z, v[q][0].w);
                const F16x2Pair z = split_f16x2(v[q][1].x, v[q][1].y), w = split_f16x2(v[q][1].z, v[q][1].w);
                u32x4* out = ys + ((NW * q + wave) * 2) * 64 + lane;
                out[0] = u32x4{x.hi, y.hi, z.hi, w.hi};
                out[64] = u32x4{x.lo, y.lo, z.lo, w.lo};
            }
        }
        if constexpr (!F16)
#pragma unroll
        for (int q = 0; q < KS16 / NW; ++q) {
            const Bf16x3Pair x = split_bf16x3(v[q][0].x, v[q][0].y), y = split_bf16x3(v[q][0].z, v[q][0].w);
            const Bf16x3Pair z = split_bf16x3(v[q][1].x, v[q][1].y), w = split_bf16x3(v[q][1].z, v[q][1].w);
            u32x4* out = ys + ((NW * q + wave) * 3) * 64 + lane;
            out[0] = u32x4{x.hi, y.hi, z.hi, w.hi};
            out[64] = u32x4{x.mid, y.mid, z.mid, w.mid};
            out[128] = u32x4{x.lo, y.lo, z.lo, w.lo};
        }
    }
    __syncthreads();
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 acc = zero;
    if constexpr (F16) {
        f32x16 rest = zero;                    // the products with a second part: apart, so that less is rounded at the size of the sum
        auto mfma = [](u32x4 x, u32x4 y, f32x16 z) {
            return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, x), __builtin_bit_cast(f16x8, y), z, 0, 0, 0);
        };
        if (odd != 0) {                        // a caller's dictionary, not an orthobase: rows from D, each scaled to its own largest magnitude
            const f32x4* row = reinterpret_cast<const f32x4*>(D + ((int64_t)__builtin_amdgcn_readfirstlane(j) * P + wave * 32 + n) * P) + h * 2;
            unsigned mx = 0;
#pragma unroll 1
            for (int ks = 0; ks < KS16; ++ks)
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float m = fabsf(row[ks * 4 + e][c]);
                        mx = max(mx, __builtin_bit_cast(unsigned, m));
                    }
            mx = max(mx, pair_other(mx, h));
            const int ex = (int)(mx >> 23);
            const int q_shift = ex == 0xff ? 0 : 140 - max(ex, 1);         // of atom n
#pragma unroll 1
            for (int ks = 0; ks < KS16; ++ks) {
                f32x4 v[2] = {row[ks * 4], row[ks * 4 + 1]};
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[e][c] = __builtin_amdgcn_ldexpf(v[e][c], q_shift);
                const F16x2Pair x = split_f16x2(v[0].x, v[0].y), y = split_f16x2(v[0].z, v[0].w);
                const F16x2Pair z = split_f16x2(v[1].x, v[1].y), w = split_f16x2(v[1].z, v[1].w);
                const u32x4 first = {x.hi, y.hi, z.hi, w.hi}, second = {x.lo, y.lo, z.lo, w.lo};
                const u32x4 hi = ys[ks * 2 * 64 + lane], lo = ys[(ks * 2 + 1) * 64 + lane];
                acc = mfma(second, hi, acc);
                acc = mfma(first, lo, acc);
                acc = mfma(first, hi, acc);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r)       // atom (r / 4) * 8 + h * 4 + r % 4
                acc[r] = __builtin_amdgcn_ldexpf(acc[r], -__shfl(q_shift, (r >> 2) * 8 + h * 4 + (r & 3), 64) - shift);
        } else {
#pragma unroll
            for (int ks = 0; ks < KS16; ++ks) {
                const u32x4 hi = ys[ks * 2 * 64 + lane], lo = ys[(ks * 2 + 1) * 64 + lane];
                rest = mfma(a[ks % AHEAD][NPT - 1], hi, rest);
                acc = mfma(a[ks % AHEAD][0], hi, acc);
                rest = mfma(a[ks % AHEAD][0], lo, rest);
                if (ks + AHEAD < KS16) fetch(a[ks % AHEAD], ks + AHEAD);
            }
            acc += rest;
            static_assert(kF16DictScale == 8192.f, "2^13");
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = __builtin_amdgcn_ldexpf(acc[r], -13 - shift);
        }
    } else {
        // the six partial products, smallest first: (A part, B part)
        constexpr int TA[6] = {2, 0, 1, 1, 0, 0};
        constexpr int TB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) {
            u32x4 b[3];
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) b[pl] = ys[(ks * 3 + pl) * 64 + lane];
#pragma unroll
            for (int t = 0; t < 6; ++t)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[ks % AHEAD][TA[t] % NPT]),
                                                              __builtin_bit_cast(bf16x8, b[TB[t]]), acc, 0, 0, 0);
            if (ks + AHEAD < KS16) fetch(a[ks % AHEAD], ks + AHEAD);
        }
    }
    __syncthreads();                           // the parts are dead
#pragma unroll
    for (int q = 0; q < 4; ++q)                // atoms wave*32 + q*8 + h*4 .. +3 of signal n
        *reinterpret_cast<f32x4*>(cs + n * kTileLd + wave * 32 + q * 8 + h * 4) = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    __syncthreads();

    // L lanes to a signal, lane `part` has the coefficients of C consecutive atoms.
    constexpr int C = P / L;
    const int sig = wave * (64 / L) + lane / L, part = lane % L;
    const bool active = sig < cnt;
    const float* row = cs + sig * kTileLd;
    float c[C], mag[C], top[S];
#pragma unroll
    for (int u = 0; u < C / 4; ++u) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(row + C * part + 4 * u);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            c[4 * u + e] = v[e];
            mag[4 * u + e] = fabsf(v[e]);
        }
    }
    top_sorted<C, S>(mag, top);
    auto merge = [&](auto other) {             // with the sorted list of another lane
        float o[S];
#pragma unroll
        for (int t = 0; t < S; ++t) o[t] = other(top[t]);
#pragma unroll
        for (int t = 0; t < S; ++t) top[t] = fmaxf(top[t], o[S - 1 - t]);
        bitonic_merge_desc<S>(top);
    };
    merge([](float x) { return dpp_f<kDppXor1>(x); });
    merge([](float x) { return dpp_f<kDppXor2>(x); });
    merge([](float x) { return dpp_f<kDppHalfMirror>(x); });
    merge([](float x) { return dpp_f<kDppRowMirror>(x); });
    float tau = top[0];
#pragma unroll
    for (int t = 1; t < S; ++t) tau = (t == s0 - 1) ? top[t] : tau;

    // entries above tau, and equal to it in ascending order until there are s0
    int gt = 0, eq = 0;
#pragma unroll
    for (int e = 0; e < C; ++e) {
        gt += fabsf(c[e]) > tau;
        eq += fabsf(c[e]) == tau;
    }
    int both = gt | eq << 16, upto = both;     // sums over the lanes up to this one
#pragma unroll
    for (int o = 1; o < L; o <<= 1) {
        const int v = __shfl_up(upto, o, L);
        if (part >= o) upto += v;
    }
    const int all = __shfl(upto, L - 1, L), before = upto - both;
    const int need = s0 - (all & 0xffff);
    int eq_rank = before >> 16, pos = (before & 0xffff) + min(eq_rank, need);
    float dropped = 0.f;
    int* mine = stage + sig * 32;
#pragma unroll
    for (int e = 0; e < C; ++e) {
        const float m = fabsf(c[e]);
        const bool tie = m == tau, keep = m > tau || (tie && eq_rank < need);
        eq_rank += tie;
        if (keep && pos < s0) {
            mine[pos] = part * C + e;
            mine[16 + pos] = __builtin_bit_cast(int, c[e]);
        }
        pos += keep;
        dropped = fmaf(keep ? 0.f : c[e], keep ? 0.f : c[e], dropped);
    }
    dropped = group_sum<L>(dropped);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (!active) return;
    const int64_t i = LISTS ? ids[sig] : by_pos ? pos0 + sig : perm[pos0 + sig];
    if (part == 0) err[i] = dropped;
    for (int e = part; e < s0; e += L) {
        supp[i * s0 + e] = mine[e];
        coef[i * s0 + e] = __builtin_bit_cast(float, mine[16 + e]);
    }
}

template <int S, bool F16>
hipError_t launch_wide_parts(const float* Y, int64_t m, const float* D, int K, int s0, const Workspace& ws, int32_t* supp, float* coef, float* err,
                             bool by_pos, const ChunkLists* lists, hipStream_t st) {
    // a multiple of 8, so that the kernel's dealing of ids over the XCDs covers every tile
    const int64_t tiles = (((m + 31) / 32 + K) + 7) & ~(int64_t)7;
    const size_t room = lists != nullptr ? kTileRoom<true, F16> : kTileRoom<false, F16>, lds = room + 32 * 33 * sizeof(int);
    const auto kernel = lists != nullptr ? &select_wide_split_kernel<S, true, F16> : &select_wide_split_kernel<S, false, F16>;
    if (lists != nullptr && (by_pos || ChunkLists::table_ints(kTileWaves, K, lists->n_chunks) * sizeof(int) > room))
        return hipErrorInvalidValue;
    if (hipError_t e = ws.raised->ensure(reinterpret_cast<const void*>(kernel), 64 * 1024); e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(64 * kTileWaves), lds, st, Y, D,
                       reinterpret_cast<const u32x4*>(F16 ? ws.dsh : ws.dsb), ws.dodd, K, s0, ws.offsets, ws.perm, supp, coef, err, (int)by_pos,
                       lists != nullptr ? *lists : ChunkLists{});
    return hipGetLastError();
}
template <int P, int S>
hipError_t launch_wide_ps(const float* Y, int64_t m, const float* D, int K, int s0,
                          const Workspace& ws, int32_t* supp, float* coef, float* err, int ops,
                          bool by_pos, const ChunkLists* lists, hipStream_t st) {
    // the kernels read ws.dsh / ws.dsb / ws.dsw, the same Q in operand order (kOpsF16: or D, see there)
    if (ops == kOpsF16) return launch_wide_parts<S, true>(Y, m, D, K, s0, ws, supp, coef, err, by_pos, lists, st);
    if (ops == kOpsBf16) return launch_wide_parts<S, false>(Y, m, D, K, s0, ws, supp, coef, err, by_pos, lists, st);
    if (lists != nullptr) return hipErrorInvalidValue;
    const int64_t max_tiles = (m + 31) / 32 + K;
    dim3 grid((unsigned)((max_tiles + 3) / 4));
    const size_t lds = 4 * 32 * (P + 1) * sizeof(float);
    if (hipError_t e = ws.raised->ensure(reinterpret_cast<const void*>(&select_wide_kernel<P, S>), lds);
        e != hipSuccess)
        return e;
    hipLaunchKernelGGL((select_wide_kernel<P, S>), grid, dim3(256), lds, st, Y,
                       reinterpret_cast<const f32x4*>(ws.dsw), K, s0, ws.offsets, ws.perm, supp, coef, err, (int)by_pos);
    return hipGetLastError();
}

template <int P>
hipError_t launch_wide_p(int s0, const float* Y, int64_t m, const float* D, int K,
                         const Workspace& ws, int32_t* supp, float* coef, float* err, int ops,
                         bool by_pos, const ChunkLists* lists, hipStream_t st) {
    if (s0 <= 1) return launch_wide_ps<P, 1>(Y, m, D, K, s0, ws, supp, coef, err, ops, by_pos, lists, st);
    if (s0 <= 2) return launch_wide_ps<P, 2>(Y, m, D, K, s0, ws, supp, coef, err, ops, by_pos, lists, st);
    if (s0 <= 4) return launch_wide_ps<P, 4>(Y, m, D, K, s0, ws, supp, coef, err, ops, by_pos, lists, st);
    if (s0 <= 8) return launch_wide_ps<P, 8>(Y, m, D, K, s0, ws, supp, coef, err, ops, by_pos, lists, st);
    return launch_wide_ps<P, 16>(Y, m, D, K, s0, ws, supp, coef, err, ops, by_pos, lists, st);
}

// From here on select_split_kernel (p = 32, 64), four wavefronts and up to 4 tiles for each: the fewest with which all
// workgroups are there at once.  Select stage by select_kernel / select_split_kernel (us): p = 64, K = 32, 12000 signals 11.0 /
// 11.2, 24576 11.4 / 11.6, 32768 14.8 / 13.9, 40960 15.5 / 14.2, 65537 19.4 / 17.5, 98304 22.9 / 20.1 (K = 4 and 128, s0 = 5 alike);
// the kernels alone 262144 48.9 / 33.5, 2^20 (K = 128) 215 / 140.  p = 32, K = 4 to 128: 24576 8.4 / 8.7, 32768 9.3 / 9.6,
// 40960 9.8 / 9.8, 65537 11.1 / 11.1, 98304 12.9 / 12.7; 300000 24.5 / 21, 10^6 64 / 53: one line for both, as its coefficients
// are the more exact ones.  p = 16 no faster at any size.  With one tile for each wavefront 262144 signals took 43 us, with
// eight of them (two workgroups on a CU) 36.6 to 43.
constexpr int64_t kSplitMinSignals = 32768;

template <int P, int S0>
hipError_t launch_ps(const float* Y, int64_t m, const float* D, int K, const Workspace& ws, int32_t* supp, float* coef,
                     float* err, int32_t* blk, bool choose, bool split, const ChunkLists* lists, hipStream_t st) {
    const int64_t max_tiles = (m + 31) / 32 + K;
    dim3 grid((unsigned)((max_tiles + 3) / 4));
    const int tiles_ints = 4 * (kSelectStageWords<S0> + kSelectTieWords);
    const int table_ints = lists != nullptr ? ChunkLists::table_ints(4, K, lists->n_chunks) : 0;
    if (table_ints * sizeof(int) > 64 * 1024) return hipErrorInvalidValue;
    if constexpr (P >= 32) if (split && m >= kSplitMinSignals) {
        constexpr int NW = 4, Q_U = P / 32 * (P / 16) * 3 * 64;
        const int64_t resident = 256 * (P == 64 ? 3 : 4) - K / 2;          // less the blocks' unfinished pieces
        const int tiles = (int)std::min<int64_t>(4, (m + 32 * NW * resident - 1) / (32 * NW * resident));
        const int piece = 32 * NW * tiles;
        const size_t lds = (std::max(4 * Q_U + tiles_ints, table_ints) + (lists != nullptr ? piece : 0)) * sizeof(int);
        const auto kernel = lists != nullptr ? &select_split_kernel<P, S0, NW, true> : &select_split_kernel<P, S0, NW, false>;
        if (hipError_t e = ws.raised->ensure(reinterpret_cast<const void*>(kernel), 160 * 1024); e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3((unsigned)((m + piece - 1) / piece + K)), dim3(64 * NW), lds, st, Y, D, K, piece, ws.offsets,
                           ws.perm, supp, coef, err, lists != nullptr ? *lists : ChunkLists{});
        return hipGetLastError();
    }
    const size_t lds = (std::max(tiles_ints, table_ints) + 4 * 32) * sizeof(int);
    if (lists != nullptr) {
        const void* fn = reinterpret_cast<const void*>(&select_kernel<P, S0, kLists>);
        if (hipError_t e = ws.raised->ensure(fn, 66 * 1024); e != hipSuccess) return e;
        hipLaunchKernelGGL((select_kernel<P, S0, kLists>), grid, dim3(256), lds, st, Y, D, K, nullptr, nullptr, supp, coef, err,
                           GroupInKernel{}, *lists);
    } else if (blk != nullptr) {
        if (K > GroupInKernel::kMostBlocks) return hipErrorInvalidValue;
        hipLaunchKernelGGL((select_kernel<P, S0, kSmall>), grid, dim3(256), lds + (K + m) * sizeof(int), st, Y, D, K, nullptr, nullptr,
                           supp, coef, err, GroupInKernel{blk, (int)m, ws.chunk_count, choose ? ws.part_E : nullptr}, ChunkLists{});
    } else {
        hipLaunchKernelGGL((select_kernel<P, S0, kGrouped>), grid, dim3(256), lds, st, Y, D, K, ws.offsets, ws.perm, supp, coef, err,
                           GroupInKernel{}, ChunkLists{});
    }
    return hipGetLastError();
}

template <int P>
hipError_t launch_p(int s0, const float* Y, int64_t m, const float* D, int K, const Workspace& ws, int32_t* supp, float* coef,
                    float* err, int32_t* blk, bool choose, bool split, const ChunkLists* lists, hipStream_t st) {
    switch (s0) {
#define SBO_CASE(N) \
    case N: return launch_ps<P, N>(Y, m, D, K, ws, supp, coef, err, blk, choose, split, lists, st);
        SBO_CASE(1) SBO_CASE(2) SBO_CASE(3) SBO_CASE(4) SBO_CASE(5) SBO_CASE(6) SBO_CASE(7) SBO_CASE(8)
        SBO_CASE(9) SBO_CASE(10) SBO_CASE(11) SBO_CASE(12) SBO_CASE(13) SBO_CASE(14) SBO_CASE(15) SBO_CASE(16)
#undef SBO_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_select(int p, int K, int s0, const float* Y, int64_t m, const float* D,
                         const Workspace& ws, int32_t* supp, float* coef, float* err, bool ops_valid,
                         int ops, hipStream_t st, int32_t* blk, bool choose, bool by_pos, bool lists) {
    const bool fits = lists ? blk != nullptr && !choose && lists_in_select(p, K, m) : blk != nullptr ? group_in_select(p, K, m) : !choose;
    if (!fits || (by_pos && p != 256)) return hipErrorInvalidValue;
    const GroupGeom g = group_geom(m);
    if (lists && g.chunk != kListChunk) return hipErrorInvalidValue;
    const ChunkLists from = {blk, (int)m, g.n_chunks, ws.chunk_count, nullptr, nullptr}, *l = lists ? &from : nullptr;
    if (p == 256 && !ops_valid) {              // the p = 256 kernels read Q in operand order
        hipError_t e = ops == kOpsF32 ? launch_dict_swizzle(p, K, D, ws.dsw, CallStart{}, st)
                                      : launch_dict_parts(p, K, D, ops == kOpsBf16 ? ws.dsb : nullptr, ops == kOpsF16 ? ws.dsh : nullptr,
                                                          ws.dnorm, ws.dodd, nullptr, SignalSample{}, CallStart{}, st);
        if (e != hipSuccess) return e;
    }
    const bool split = ops != kOpsF32;
    switch (p) {
        case 16: return launch_p<16>(s0, Y, m, D, K, ws, supp, coef, err, blk, choose, split, l, st);
        case 32: return launch_p<32>(s0, Y, m, D, K, ws, supp, coef, err, blk, choose, split, l, st);
        case 64: return launch_p<64>(s0, Y, m, D, K, ws, supp, coef, err, blk, choose, split, l, st);
        case 256: return launch_wide_p<256>(s0, Y, m, D, K, ws, supp, coef, err, ops, by_pos, l, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sbo
