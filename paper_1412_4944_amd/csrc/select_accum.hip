// Fused second half of sparse coding and block accumulation (p <= 64), used by
// sbo_iterate, sbo_train_rounds and sbo_new_base: for the signals of one block, support /
// coefficients / residual in that block (Section 2; Algorithm 1 steps 3-4) and, from the same
// tile while it is on chip, its contribution to P_j = Y_j X_j^T (Algorithm 1 step 5).  Y is
// read from HBM once for both, and the sparse codes feed the product without a trip through
// memory.
//
// A workgroup (8 wavefronts, one workgroup per CU) owns one piece of one block's grouped signal
// list.  Both contractions run on the bf16 matrix cores at fp32 accuracy: every fp32 operand
// entry is the exact sum of three bf16 parts and the six partial products above 2^-24 are
// accumulated in fp32 (device_utils.h).  Q_j is split once per workgroup into LDS in MFMA
// operand order.  Each wavefront walks tiles of 32 signals:
//   projection  c = Q_j^T y : atoms on M, signals on N, dims contracted; y is split in registers
//                             (a lane holds its own signal's dims);
//   selection   (select_tile.h) from the accumulators;
//   product     P_j += x y^T: atoms on M, dims on N, SIGNALS contracted, so both operands are
//                             needed with eight consecutive signals per lane: the split parts of
//                             y go through a wave-private LDS tile [signal][dim], from which
//                             ds_read_b64_tr_b16 takes them transposed, the s0 kept coefficients of every signal are scattered into a zeroed tile
//                             [atom][signal] and wiped again after use; 16 signals at a time.
// Accumulators stay in registers across the tiles of the piece; the wavefronts are added in
// wavefront order, the pieces of a block in piece order by the kernel that consumes them.
//
// What bounds it: instruction issue and LDS round trips of two wavefronts per SIMD, not memory (Y is
// read once).  Measured, 262144 signals, K = 32, p = 64, s0 = 8: 61 us with y transposed word by word through
// lane exchanges and the copies of the accumulators stored entry by entry, 44.6 us as it is (with the shorter
// selection of select_tile.h); 2^20 signals, K = 128: 265 -> 186 us.  Taken back: two fp16 parts, three products (40.4 and 166 us, and
// coefficients closer to 64 bits, 5.9e-8 of theirs instead of 9.0e-8): the range of fp16 asks for a scale of every atom and of every
// signal, and what one scale of P_j leaves of signals 2^-8 as strong as others is short of fp32.  The small products summed apart: 4.9e-8,
// but 49.3 us.
#include "sbo_internal.h"
#include "device_utils.h"
#include "select_tile.h"

namespace sbo {

namespace {

constexpr int kSaWaves = 8;

// LDS of a wavefront: the stage and the operand tiles (or the scratch for ties); at the end a copy of its accumulators.
template <int P, int S0>
constexpr int sa_wave_bytes() {
    constexpr int MT = P >= 32 ? P / 32 : 1, ops = 6 * (MT * 32 + 1) * 32, ct = kSelectTieWords * 4;
    constexpr int use = kSelectStageWords<S0> * 4 + (ops > ct ? ops : ct), copy = MT * MT * 4 * 64 * 16;
    return use > copy ? use : copy;
}

// GROUP: the signals have not been grouped, every workgroup lists those of its own piece (ChunkLists).
template <int P, int S0, bool GROUP>
__global__ __launch_bounds__(64 * kSaWaves) void select_accum_kernel(
    const float* __restrict__ Y, const float* __restrict__ D, int K, int piece,
    const int32_t* __restrict__ offsets, const int32_t* __restrict__ perm, int32_t* __restrict__ supp,
    float* __restrict__ coef, float* __restrict__ err, float* __restrict__ partial, ChunkLists lists) {
    constexpr int NW = kSaWaves, NTH = 64 * NW;
    constexpr int KS16 = P / 16;               // projection: steps of 16 dims
    constexpr int MT = P >= 32 ? P / 32 : 1;   // 32-wide tiles per side of P_j
    constexpr int ROWS = MT * 32;              // operand tile rows (atoms resp. dims; rows >= P are not used)
    constexpr int PP = P * P;
    constexpr int Q_U = MT * KS16 * 3 * 64;    // Q_j in split operand order, 16-byte units
    constexpr int PLANE_B = (ROWS + 1) * 32;   // bytes of one part of a transposed operand tile (+ a dummy row)
    constexpr int CT_B = kSelectTieWords * 4;           // tie-breaking scratch of tile_select
    constexpr int OPS_B = 6 * PLANE_B;         // x tile (3 parts) + y tile (3 parts)
    constexpr int REGION_B = (OPS_B > CT_B ? OPS_B : CT_B);
    constexpr int WAVE_B = sa_wave_bytes<P, S0>();
    static_assert(kSelectStageWords<S0> * 4 + REGION_B <= WAVE_B, "stage and region");
    constexpr int YU = P / 8 - 1 < 7 ? P / 8 - 1 : 7;      // of a signal's 16-byte units
    constexpr int NE = (S0 + 3) / 4;            // kept entries per lane and half tile

    // Qs[Q_U] | per wavefront: stage | region; GROUP: the table of `lists` in the place of the latter first, and
    // ids[piece] behind everything
    extern __shared__ __attribute__((aligned(16))) int lds[];
    u32x4* Qs = reinterpret_cast<u32x4*>(lds);
    unsigned char* waves_base = reinterpret_cast<unsigned char*>(Qs + Q_U);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, n = lane & 31;

    int* ids = reinterpret_cast<int*>(waves_base + (size_t)NW * WAVE_B);
    const int id = blockIdx.x;
    Piece pc;
    if constexpr (GROUP) {
        int* table = reinterpret_cast<int*>(waves_base);
        lists.load<NW>(K, table);
        if (id == 0 && wave == 0) lists.leave<NW>(K, table);
        pc = find_piece([&](int j) { return lists.count_of<NW>(K, table, j); }, K, piece, id);
        if (pc.j >= 0) lists.collect<NW>(K, table, pc, ids, wave);
        __syncthreads();
    } else {
        pc = find_piece([&](int j) { return offsets[j + 1] - offsets[j]; }, K, piece, id);
    }
    if (pc.j < 0) return;                      // uniform over the workgroup
    const int j = pc.j, pos0 = pc.before + pc.rank, cnt = pc.count;

    const int n_tiles = (cnt + 31) >> 5;
    // Signal ids are fetched two tiles ahead and the rows of Y one tile ahead: the loads of
    // the next tile are issued as soon as the current rows have been split, and land while
    // the matrix work and the selection run.  The loads are unconditional (lanes past the end
    // of the piece take its last signal once more and keep nothing of it).  Those of the first tile are on their way
    // before Q_j is split (50021 signals, K = 24, p = 32: 10.0 -> 9.4 us; 262144, p = 64: no difference).
    auto tile_id = [&](int t) -> int {
        const int at = min(t * 32 + n, cnt - 1);
        return GROUP ? ids[at] : perm[pos0 + at];
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

    // Q_j -> LDS, split: unit ((mt*KS16 + ks)*3 + part)*64 + hh*32 + nn = the 8 bf16 of that part
    // of dims ks*16 + hh*8 .. +7 of atom mt*32 + nn (atoms >= P: zeros); one unit per thread
    static_assert(MT * KS16 * 64 <= NTH, "one unit per thread");
    const int q_ks = (tid >> 6) % KS16, q_mt = (tid >> 6) / KS16, q_atom = q_mt * 32 + n;
    f32x4 q0 = {0.f, 0.f, 0.f, 0.f}, q1 = q0;
    if (q_mt < MT && q_atom < P) {
        const f32x4* D4 = reinterpret_cast<const f32x4*>(D + (int64_t)j * PP);
        q0 = D4[q_atom * (P / 4) + q_ks * 4 + h * 2];
        q1 = D4[q_atom * (P / 4) + q_ks * 4 + h * 2 + 1];
    }
    load_rows(i_cur);
    if (q_mt < MT) {
        const Bf16x3Pair a = split_bf16x3(q0.x, q0.y), b = split_bf16x3(q0.z, q0.w);
        const Bf16x3Pair c = split_bf16x3(q1.x, q1.y), d = split_bf16x3(q1.z, q1.w);
        u32x4* out = Qs + ((tid >> 6) * 3) * 64 + lane;
        out[0] = u32x4{a.hi, b.hi, c.hi, d.hi};
        out[64] = u32x4{a.mid, b.mid, c.mid, d.mid};
        out[128] = u32x4{a.lo, b.lo, c.lo, d.lo};
    }
    int* stage = reinterpret_cast<int*>(waves_base + (size_t)wave * WAVE_B);
    unsigned char* region = reinterpret_cast<unsigned char*>(stage + kSelectStageWords<S0>);
    unsigned char* xt = region;                // [3 parts][ROWS atoms][16 signals] bf16
    unsigned char* yt = region + 3 * PLANE_B;  // [3 parts][16 signals][P dims] bf16
    // the x tile starts out zero (and is left zero by every tile)
    for (int e = lane; e < 3 * PLANE_B / 16; e += 64) reinterpret_cast<u32x4*>(xt)[e] = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();

    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                         0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 accM[MT][MT];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < MT; ++b) accM[a][b] = zero;
    // the six partial products, smallest first: (A part, B part)
    constexpr int TA[6] = {2, 0, 1, 1, 0, 0};
    constexpr int TB[6] = {0, 2, 1, 0, 1, 0};

    for (int tile = wave; tile < n_tiles; tile += NW) {
        const int64_t i = i_cur;
        const bool active = tile * 32 + n < cnt;
        const int cnt_t = min(32, cnt - tile * 32);        // signals in this tile (uniform)

        // y in three bf16 parts (B operand of the projection)
        u32x4 yq[KS16][3];
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) {
            const f32x4 v0 = raw[ks][0], v1 = raw[ks][1];
            const Bf16x3Pair a = split_bf16x3(v0.x, v0.y), b = split_bf16x3(v0.z, v0.w);
            const Bf16x3Pair c = split_bf16x3(v1.x, v1.y), d = split_bf16x3(v1.z, v1.w);
            yq[ks][0] = u32x4{a.hi, b.hi, c.hi, d.hi};
            yq[ks][1] = u32x4{a.mid, b.mid, c.mid, d.mid};
            yq[ks][2] = u32x4{a.lo, b.lo, c.lo, d.lo};
        }
        i_cur = i_next;
        i_next = tile_id(tile + 2 * NW);
        load_rows(i_cur);                      // rows of the next tile

        // projection c = Q_j^T y
        f32x16 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = zero;
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

        // support, coefficients, residual; the (atom, coefficient) rows stay in `stage` for the
        // product below.
        // The tie-breaking scratch is the operand region: the x tile is zeroed again if it was used.
        bool ties = false;
        tile_select<P, S0>(acc, h, n, active, i, reinterpret_cast<float*>(region), stage, supp, coef, err, &ties);
        if (ties) {                            // uniform (rare): the scratch overwrote the zeroed x tile
            for (int e = lane; e < 3 * PLANE_B / 16; e += 64)
                reinterpret_cast<u32x4*>(xt)[e] = u32x4{0u, 0u, 0u, 0u};
        }

        // P_j += sum over the tile's signals of x y^T, 16 signals at a time
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (cnt_t <= 16 * half) break;     // uniform: no signal in this half
            const bool mine = (n >> 4) == half;
            const int sc = n & 15;             // this lane's signal inside the half
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // y parts: rows of signals as they are, 16-byte units (8 dims) of a row in an order that depends
            // on the row; they are transposed on the way out
            if (mine) {
#pragma unroll
                for (int ks = 0; ks < KS16; ++ks)
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl)
                        *reinterpret_cast<u32x4*>(yt + pl * PLANE_B + sc * (P * 2) + (((ks * 2 + h) ^ (sc & YU)) << 4)) = yq[ks][pl];
            }
            // kept coefficients -> [atom][signal]; four lanes of a signal share its entries
            // (entries that do not exist go to the dummy row instead of a branch)
            int at_[NE];
            {
                const int sx = lane & 15, row = 16 * half + sx;
#pragma unroll
                for (int t = 0; t < NE; ++t) {
                    const int pos = 4 * t + (lane >> 4);
                    const bool have = row < cnt_t && pos < S0;
                    const int atom = stage[stage_idx(row, 0, have ? pos : 0)];
                    const TriWord w = split_trunc(__builtin_bit_cast(float, stage[stage_idx(row, 1, have ? pos : 0)]));
                    at_[t] = tr_off(have ? (atom & (ROWS - 1)) : ROWS, sx);   // row ROWS: nobody reads it
                    *reinterpret_cast<unsigned short*>(xt + at_[t]) = (unsigned short)(w.hi >> 16);
                    *reinterpret_cast<unsigned short*>(xt + PLANE_B + at_[t]) = (unsigned short)(w.mid >> 16);
                    *reinterpret_cast<unsigned short*>(xt + 2 * PLANE_B + at_[t]) = (unsigned short)(w.lo >> 16);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // operands: lane (h, n) takes signals 8h .. 8h+7 of atom resp. dim t*32 + n; the dims by
            // ds_read_b64_tr_b16 (of 16 lanes, lane i addresses four dims, 4 (i & 3) .., of signal i >> 2 and
            // receives dim i of the four signals)
            u32x4 xa[MT][3], yb[MT][3];
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                int ya[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int sig = 8 * h + 4 * k + ((lane & 15) >> 2), d = (t * 32 + (lane & 16) + 4 * (lane & 3)) & (P - 1);
                    ya[k] = sig * (P * 2) + (((d >> 3) ^ (sig & YU)) << 4) + (d & 4) * 2;
                }
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) {
                    typedef short s16x4 __attribute__((ext_vector_type(4)));
                    typedef __attribute__((address_space(3))) s16x4* lds_ptr;
                    xa[t][pl] = *reinterpret_cast<const u32x4*>(xt + pl * PLANE_B + tr_off(t * 32 + n, 8 * h));
                    const s16x4 y0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(yt + pl * PLANE_B + ya[0]));
                    const s16x4 y1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(yt + pl * PLANE_B + ya[1]));
                    const u32x2 u0 = __builtin_bit_cast(u32x2, y0), u1 = __builtin_bit_cast(u32x2, y1);
                    yb[t][pl] = u32x4{u0.x, u0.y, u1.x, u1.y};
                }
            }
#pragma unroll
            for (int t = 0; t < 6; ++t)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < MT; ++nt)
                        accM[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            __builtin_bit_cast(bf16x8, xa[mt][TA[t]]), __builtin_bit_cast(bf16x8, yb[nt][TB[t]]),
                            accM[mt][nt], 0, 0, 0);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();   // the operands have been read: wipe the x entries again
#pragma unroll
            for (int t = 0; t < NE; ++t) {
                *reinterpret_cast<unsigned short*>(xt + at_[t]) = 0;
                *reinterpret_cast<unsigned short*>(xt + PLANE_B + at_[t]) = 0;
                *reinterpret_cast<unsigned short*>(xt + 2 * PLANE_B + at_[t]) = 0;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();       // stage and the region are rewritten by the next tile
    }
    __syncthreads();                           // all tiles done: their LDS becomes the exchange area

    // The wavefronts' accumulators are added in wavefront order: every wavefront stores its own copy as it
    // holds it, 16 bytes per lane (register r of tile (mt, nt) in lane (h, n) is atom mt*32 + (r/4)*8 + h*4 +
    // r%4, dimension nt*32 + n), then every thread adds the NW copies of a unit, four atoms of one
    // dimension, and writes them to the piece result.
    constexpr int UNITS = MT * MT * 4 * 64;
    static_assert((size_t)UNITS * 16 <= (size_t)WAVE_B, "a copy fits the wave's own area");
    {
        f32x4* mine = reinterpret_cast<f32x4*>(waves_base + (size_t)wave * WAVE_B) + lane;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < MT; ++nt)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    mine[((mt * MT + nt) * 4 + q) * 64] = f32x4{accM[mt][nt][4 * q], accM[mt][nt][4 * q + 1],
                                                                accM[mt][nt][4 * q + 2], accM[mt][nt][4 * q + 3]};
    }
    __syncthreads();
    float* out = partial + (int64_t)id * PP;
    for (int u = tid; u < UNITS; u += NTH) {
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w)
            sum += reinterpret_cast<const f32x4*>(waves_base + (size_t)w * WAVE_B)[u];
        const int tile = u >> 8, atom = (tile / MT) * 32 + ((u >> 6) & 3) * 8 + ((u >> 5) & 1) * 4;
        const int dim = (tile % MT) * 32 + (u & 31);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (atom + k < P && dim < P) out[(atom + k) * P + dim] = sum[k];
    }
}

template <int P, int S0>
hipError_t launch_ps(const float* Y, int64_t m, const float* D, int K, const Workspace& ws,
                     int32_t* supp, float* coef, float* err, hipStream_t st, const int32_t* blk) {
    constexpr int MT = P >= 32 ? P / 32 : 1;
    constexpr size_t wave_b = sa_wave_bytes<P, S0>();
    const int piece = accum_piece(m, K);
    const int max_pieces = accum_max_pieces(m, K);
    size_t lds = (size_t)MT * (P / 16) * 3 * 64 * sizeof(u32x4) + kSaWaves * wave_b;
    if (blk != nullptr) {
        const GroupGeom g = group_geom(m);
        lds += (size_t)piece * sizeof(int);
        if (g.chunk != kListChunk || lds > 160 * 1024 ||
            ChunkLists::table_ints(kSaWaves, K, g.n_chunks) * sizeof(int) > kSaWaves * wave_b)
            return hipErrorInvalidValue;
        if (hipError_t e = ws.raised->ensure(reinterpret_cast<const void*>(&select_accum_kernel<P, S0, true>), 160 * 1024);
            e != hipSuccess)
            return e;
        hipLaunchKernelGGL((select_accum_kernel<P, S0, true>), dim3(max_pieces), dim3(64 * kSaWaves), lds, st, Y, D, K,
                           piece, nullptr, nullptr, supp, coef, err, ws.partial,
                           ChunkLists{blk, (int)m, g.n_chunks, ws.chunk_count, ws.counts, ws.offsets});
        return hipGetLastError();
    }
    if (hipError_t e = ws.raised->ensure(reinterpret_cast<const void*>(&select_accum_kernel<P, S0, false>), 160 * 1024);
        e != hipSuccess)
        return e;
    hipLaunchKernelGGL((select_accum_kernel<P, S0, false>), dim3(max_pieces), dim3(64 * kSaWaves), lds, st, Y, D, K,
                       piece, ws.offsets, ws.perm, supp, coef, err, ws.partial, ChunkLists{});
    return hipGetLastError();
}

template <int P>
hipError_t launch_p(int s0, const float* Y, int64_t m, const float* D, int K, const Workspace& ws,
                    int32_t* supp, float* coef, float* err, hipStream_t st, const int32_t* blk) {
    switch (s0) {
#define SBO_CASE(N) \
    case N: return launch_ps<P, N>(Y, m, D, K, ws, supp, coef, err, st, blk);
        SBO_CASE(1) SBO_CASE(2) SBO_CASE(3) SBO_CASE(4) SBO_CASE(5) SBO_CASE(6) SBO_CASE(7) SBO_CASE(8)
        SBO_CASE(9) SBO_CASE(10) SBO_CASE(11) SBO_CASE(12) SBO_CASE(13) SBO_CASE(14) SBO_CASE(15) SBO_CASE(16)
#undef SBO_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

// Support/coefficients/residual of the grouped signals AND the per-piece partial P_j in
// ws.partial (summed in piece order by launch_polar_from_pieces or launch_accum_reduce).
// p <= 64 only.
hipError_t launch_select_accum(int p, int K, int s0, const float* Y, int64_t m, const float* D,
                               const Workspace& ws, int32_t* supp, float* coef, float* err,
                               hipStream_t st, const int32_t* blk) {
    if (blk != nullptr && !lists_in_round(p, K, m)) return hipErrorInvalidValue;
    switch (p) {
        case 16: return launch_p<16>(s0, Y, m, D, K, ws, supp, coef, err, st, blk);
        case 32: return launch_p<32>(s0, Y, m, D, K, ws, supp, coef, err, st, blk);
        case 64: return launch_p<64>(s0, Y, m, D, K, ws, supp, coef, err, st, blk);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sbo
