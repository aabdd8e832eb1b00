// C-ABI of libsbo: argument checks, workspace, stage sequencing and timing.
// All arithmetic is in the kernels; this file only enqueues them.
#include "sbo_internal.h"
#include "stream_count.h"

#include <cmath>
#include <new>
#include <string>

namespace sbo {

static size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

static int max_chunks() { return 1025; }

// At least what accum_piece() makes of any m <= m_max and at most K blocks.
static int64_t max_pieces_bound(int64_t m_max, int K, int p) {
    const int64_t smallest = (m_max + kMinPiece - 1) / kMinPiece;
    if (p <= 64) return smallest + K + 1;
    const int64_t most = (m_max + kMaxPiece - 1) / kMaxPiece;      // (they only grow beyond kNumCU when that many are largest)
    return (smallest < most + kNumCU ? smallest : most + kNumCU) + K + 1;
}

size_t workspace_layout(int p, int K, int s0, int64_t m_max, Workspace* ws, char* base) {
    (void)s0;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* ptr = base ? base + off : nullptr;
        off += align_up(bytes);
        return ptr;
    };
    Workspace w;
    w.chunk_count = (int32_t*)take((size_t)max_chunks() * K * 4);
    w.chunk_base = (int32_t*)take((size_t)max_chunks() * K * 4);
    w.counts = (int32_t*)take((size_t)K * 4);
    w.offsets = (int32_t*)take((size_t)(K + 1) * 4);
    w.perm = (int32_t*)take((size_t)m_max * 4);
    w.group_done = (int*)take(4);
    w.weak = (int*)take(3 * 4);
    w.short_cut = (int*)take((size_t)((m_max + 255) / 256) * 4);
    w.energy = (float*)take((size_t)m_max * 4);
    w.dsw = (float*)take((size_t)((K * p + 63) / 64) * 64 * p * 4);
    w.dsb = (unsigned*)take((size_t)((K * p + 63) / 64) * 64 * p * 6);
    w.dsh = (unsigned*)take((size_t)((K * p + 63) / 64) * 64 * p * 4);
    w.dnorm = (float2*)take((size_t)K * (p / 16) * 8);
    w.dodd = (int*)take(p == 256 ? (size_t)K * (p / 16) * 4 : 0);
    w.dev = (float2*)take(p == 64 ? (size_t)K * 8 : 0);
    w.sample = (unsigned*)take(p == 64 ? (size_t)K * (kSample / 8) : 0);
    const size_t split_m = (size_t)(m_max < kEnergySplitSignals ? m_max : kEnergySplitSignals);
    const size_t direct = m_max < kDirectMaxEnergies / K ? (size_t)K * m_max : (size_t)kDirectMaxEnergies;
    w.part_E = (float*)take((direct > kEnergySplitRows * split_m ? direct : kEnergySplitRows * split_m) * 4);
    w.part_j = (int32_t*)take((size_t)kEnergySplitRows * split_m * 4);
    // (a context for more blocks than are ever split may be used with fewer: sbo_set_blocks, sbo_learn)
    w.split_room = (int)(((m_max < kSplitMaxSignals ? m_max : kSplitMaxSignals) + 63) / 64) * (K < kSplitMaxK ? K : kSplitMaxK);
    w.split_E = (unsigned*)take((size_t)w.split_room * 128);
    w.split_x = (unsigned*)take((size_t)kNumCU * 4 * 64 * 4);
    w.split_done = (int*)take((size_t)kNumCU / 2 * 4);
    // The eigenvectors of a Gram matrix are computed when the pieces of that matrix have been summed: same memory.
    size_t partial = (size_t)max_pieces_bound(m_max, K, p) * p * p * 4;
    if (partial < eigen_scratch_bytes(p)) partial = eigen_scratch_bytes(p);
    w.partial = (float*)take(partial);
    w.eig = (unsigned char*)w.partial;
    w.eig_room = (int)(partial / eigen_scratch_bytes(p) < (size_t)K ? partial / eigen_scratch_bytes(p) : (size_t)K);
    w.M = (float*)take((size_t)K * p * p * 4);
    w.wide = (float*)take(p > 64 ? polar_wide_scratch_bytes(K) : 0);
    w.wide_sync = (int*)take(p > 64 ? polar_wide_sync_bytes(K) : 0);
    w.eig_left = (int32_t*)take((size_t)K * 4);
    const size_t sel_chunks = (size_t)((m_max + kSelChunk - 1) / kSelChunk);
    w.sel_hist = (int32_t*)take((size_t)4 * 256 * 4);
    w.sel_state = (int32_t*)take((size_t)4 * 2 * 4);
    w.sel_cnt = (int32_t*)take(sel_chunks * 2 * 4);
    w.sel_base = (int32_t*)take(sel_chunks * 2 * 4);
    w.sq_counter = (int32_t*)take(4);
    w.sweeps = (int32_t*)take((size_t)K * 4);
    w.ns_fallback = (int32_t*)take((size_t)K * 4);
    w.sq_partial = (double*)take((size_t)kSqBlocks * 8);
    w.bytes = off;
    w.raised = nullptr;
    w.device = 0;
    if (ws) *ws = w;
    return off;
}

static bool shape_ok(int p, int K, int s0, int64_t m_max) {
    if (!(p == 16 || p == 32 || p == 64 || p == 256)) return false;
    if (K < 1 || K > 1024) return false;
    if (s0 < 1 || s0 > 16 || s0 > p) return false;
    if (m_max < 1) return false;
    const int64_t lim = ((int64_t)1 << 31) / (p > s0 ? p : s0);
    if (m_max >= lim) return false;
    return true;
}

// The live contexts of p = 256.
static StreamCount g_wide;
int wide_streams(int device) { return g_wide.streams(device); }

static thread_local std::string g_hip_text = "no HIP error recorded";

static int hip_fail(hipError_t e) {
    g_hip_text = std::string("HIP error: ") + hipGetErrorString(e);
    return SBO_EHIP;
}

#define SBO_HIP(expr)                                   \
    do {                                                \
        hipError_t e_ = (expr);                         \
        if (e_ != hipSuccess) return sbo::hip_fail(e_); \
    } while (0)

// Records a begin event now and an end event at scope exit when timing is on.
struct StageTimer {
    sbo_ctx* c;
    long idx;                                  // index into c->spans, -1 = not timing
    StageTimer(sbo_ctx* ctx, int stage) : c(ctx), idx(-1) {
        if (!c->timing || (c->timing == 2 && stage != SBO_STAGE_ENERGY)) return;
        if (c->n_spans == c->spans.size()) {
            sbo_span s;
            s.stage = stage;
            if (hipEventCreate(&s.beg) != hipSuccess) return;
            if (hipEventCreate(&s.end) != hipSuccess) {
                (void)hipEventDestroy(s.beg);
                return;
            }
            c->spans.push_back(s);
        }
        idx = (long)c->n_spans++;
        c->spans[idx].stage = stage;
        (void)hipEventRecord(c->spans[idx].beg, c->stream);
    }
    ~StageTimer() {
        if (idx >= 0) (void)hipEventRecord(c->spans[idx].end, c->stream);
    }
};

static int check_call(const sbo_ctx* c, int64_t m) {
    if (!c) return SBO_EINVAL;
    if (m < 1 || m > c->m_max) return SBO_EINVAL;
    return SBO_OK;
}

static int run_group(sbo_ctx* c, const int32_t* blk, int64_t m, bool have_hist = false) {
    StageTimer t(c, SBO_STAGE_GROUP);
    SBO_HIP(launch_group(c->K, blk, m, c->ws, have_hist, c->stream));
    return SBO_OK;
}

static bool use_split(const sbo_ctx* c) { return c->coding_arith != SBO_ARITH_F32; }
// The arithmetic of the block choice.  Screening is now part of every arithmetic that allows it, so
// SBO_ARITH_BF16X3_SCREEN is SBO_ARITH_BF16X3.  At p = 256 only the screening kernel works with two fp16 parts:
// where it does not apply (K beyond its table), three bf16 parts, the finer of the two.
static int choice_arith(const sbo_ctx* c) {
    const int a = c->coding_arith == SBO_ARITH_BF16X3_SCREEN ? (int)SBO_ARITH_BF16X3 : c->coding_arith;
    return a == SBO_ARITH_F16X2 && c->p > 64 && !screen_applies(c->p, c->K, c->s0, a) ? (int)SBO_ARITH_BF16X3 : a;
}
// The operand orders that the block choice of this context reads.
static int energy_ops(const sbo_ctx* c) {
    const int a = choice_arith(c);
    const int own = a == SBO_ARITH_F32 ? kOpsF32 : a == SBO_ARITH_F16X2 ? kOpsF16 : kOpsBf16;
    return screen_applies(c->p, c->K, c->s0, a) ? own | kOpsF16 : own;
}

// ... that its select kernel reads (p <= 64: D itself), and both.
// Two fp16 parts after a choice that has them as well, and where the library has made the orthobases itself (own); a caller's
// dictionary without a choice may have entries beyond their range.
static int select_arith(const sbo_ctx* c, bool own) {
    const int a = c->coding_arith;
    return a == SBO_ARITH_F32 ? kOpsF32 : a == SBO_ARITH_F16X2 && own ? kOpsF16 : kOpsBf16;
}
static int code_arith(const sbo_ctx* c) { return select_arith(c, choice_arith(c) == SBO_ARITH_F16X2); }
static int select_ops(const sbo_ctx* c, bool own) { return c->p <= 64 ? 0 : select_arith(c, own); }
static int code_ops(const sbo_ctx* c) { return energy_ops(c) | (c->p <= 64 ? 0 : code_arith(c)); }

// D in the operand order(s) the coding kernels of this context read (tiny; outside the stages).
static int run_swizzle(sbo_ctx* c, const float* Y, int64_t m, const float* D) {
    const int ops = code_ops(c);
    const CallStart start = {c->ws.weak, c->ws.chunk_count, group_geom(m).n_chunks * c->K};
    if (ops & kOpsF32) SBO_HIP(launch_dict_swizzle(c->p, c->K, D, c->ws.dsw, start, c->stream));
    if (ops & (kOpsBf16 | kOpsF16))
        SBO_HIP(launch_dict_parts(c->p, c->K, D, ops & kOpsBf16 ? c->ws.dsb : nullptr,
                                  ops & kOpsF16 ? c->ws.dsh : nullptr, c->ws.dnorm, c->ws.dodd,
                                  guess_applies(c->p, c->K, c->s0, m, choice_arith(c)) ? c->ws.dev : nullptr,
                                  SignalSample{Y, (int)m, c->ws.sample}, start, c->stream));
    return SBO_OK;
}

static int run_energy(sbo_ctx* c, const float* Y, int64_t m, int32_t* blk, int turn = -1) {
    StageTimer t(c, SBO_STAGE_ENERGY);     // also leaves the chunk histograms of the grouping
    SBO_HIP(launch_energy(c->p, c->K, c->s0, choice_arith(c), Y, m, c->ws, blk, c->ws.chunk_count, c->stream, turn,
                          c->svd_method != SBO_SVD_JACOBI));
    return SBO_OK;
}

// turn: the iteration of sbo_iterate; from the second one on the workspace holds D in those orders already.
static int run_code(sbo_ctx* c, const float* Y, int64_t m, const float* D, int32_t* blk,
                    int32_t* supp, float* coef, float* err, int turn = -1) {
    int rc = SBO_OK;
    const bool direct = choose_in_select(c->p, c->K, c->s0, m, choice_arith(c));
    if (direct) {
        StageTimer t(c, SBO_STAGE_ENERGY);
        SBO_HIP(launch_energy_direct(c->p, c->K, c->s0, choice_arith(c), Y, m, D, c->ws, c->stream));
    } else {
        if (turn <= 0) rc = run_swizzle(c, Y, m, D);
        if (rc) return rc;
        rc = run_energy(c, Y, m, blk, turn);
        if (rc) return rc;
    }
    // The energy kernel left the chunk histograms: for the grouping, which the update of an iteration needs too, or for lists.
    const bool in_select = group_in_select(c->p, c->K, m), lists = turn < 0 && !in_select && lists_in_select(c->p, c->K, m) &&
                           (c->p <= 64 || use_split(c));
    if (!in_select && !lists) rc = run_group(c, blk, m, true);
    if (rc) return rc;
    {
        StageTimer t(c, SBO_STAGE_SELECT);         // p = 256 reads the operand order run_swizzle wrote
        SBO_HIP(launch_select(c->p, c->K, c->s0, Y, m, D, c->ws, supp, coef, err, true, code_arith(c), c->stream,
                              in_select || lists ? blk : nullptr, direct, false, lists));
    }
    return SBO_OK;
}

// The SVD update from the piece results of launch_select_accum or launch_accumulate;
// err / sq_out: also the squared-error total of the coding pass.  One launch on the default path;
// with the Jacobi SVD for every block the pieces are summed by their own launch first.
static int run_polar_pieces(sbo_ctx* c, int64_t m, float* D, int write_ops, const float* err, double* sq_out,
                            int K = -1, bool clear_lists = false) {
    if (K < 0) K = c->K;
    if (c->svd_method == SBO_SVD_JACOBI) {
        {
            StageTimer t(c, SBO_STAGE_ACCUM);
            SBO_HIP(launch_accum_reduce(c->p, K, m, c->ws, c->ws.M, err, sq_out, c->stream));
        }
        StageTimer t(c, SBO_STAGE_SVD);
        SBO_HIP(launch_polar(c->p, K, c->ws.M, c->ws.counts, D, c->ws, 1, nullptr, write_ops, c->stream));
        return SBO_OK;
    }
    StageTimer t(c, SBO_STAGE_SVD);
    SBO_HIP(launch_polar_from_pieces(c->p, K, m, D, c->ws, write_ops, err, sq_out, c->stream, clear_lists));
    return SBO_OK;
}

// Accumulate + SVD of K orthobases (-1: all) from codes, for signals already grouped in the workspace.
static int run_update_grouped(sbo_ctx* c, const float* Y, int64_t m, const int32_t* supp, const float* coef, float* D,
                              int write_ops = 0, const float* err = nullptr, double* sq_out = nullptr, int K = -1,
                              bool by_pos = false) {
    if (K < 0) K = c->K;
    {
        StageTimer t(c, SBO_STAGE_ACCUM);
        SBO_HIP(launch_accumulate(c->p, K, c->s0, Y, m, supp, coef, c->ws, nullptr, c->stream, by_pos));
    }
    return run_polar_pieces(c, m, D, write_ops, err, sq_out, K);
}

}  // namespace sbo

using namespace sbo;

extern "C" {

size_t sbo_workspace_bytes(int p, int K, int s0, int64_t m_max) {
    if (!shape_ok(p, K, s0, m_max)) return 0;
    return workspace_layout(p, K, s0, m_max, nullptr, nullptr);
}

int sbo_create(sbo_ctx** out, int p, int K, int s0, int64_t m_max, void* hip_stream) {
    if (!out || !shape_ok(p, K, s0, m_max)) return SBO_EINVAL;
    sbo_ctx* c = new (std::nothrow) sbo_ctx();
    if (!c) return SBO_ENOMEM;
    c->p = p;
    c->K = K;
    c->K_cap = K;
    c->s0 = s0;
    c->m_max = m_max;
    c->stream = (hipStream_t)hip_stream;
    c->svd_method = SBO_SVD_AUTO;
    c->coding_arith = SBO_ARITH_F16X2;
    c->timing = 0;
    c->n_spans = 0;
    const size_t bytes = workspace_layout(p, K, s0, m_max, nullptr, nullptr);
    void* base = nullptr;
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e == hipSuccess) e = hipMalloc(&base, bytes);
    if (e != hipSuccess) {
        delete c;
        if (e == hipErrorOutOfMemory) return SBO_ENOMEM;
        return hip_fail(e);
    }
    c->ws_base = (char*)base;
    workspace_layout(p, K, s0, m_max, &c->ws, c->ws_base);
    c->ws.raised = &c->raised;
    c->ws.device = device;
    c->ws.parts_accum = c->coding_arith != SBO_ARITH_F32;
    // Some pieces of the workspace carry an invariant between calls: the two finished-workgroup counters and the counters of
    // polar_wide.hip are zero whenever no call is in flight.
    e = hipMemsetAsync(c->ws.sq_counter, 0, 4, c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(c->ws.group_done, 0, 4, c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(c->ws.split_done, 0, (size_t)kNumCU / 2 * 4, c->stream);
    if (e == hipSuccess && p > 64) e = hipMemsetAsync(c->ws.wide_sync, 0, polar_wide_sync_bytes(K), c->stream);
    if (e != hipSuccess) {
        (void)hipFree(c->ws_base);
        delete c;
        return hip_fail(e);
    }
    if (p > 64) g_wide.add(device, c->stream);
    *out = c;
    return SBO_OK;
}

int sbo_destroy(sbo_ctx* c) {
    if (!c) return SBO_EINVAL;
    hipError_t e = hipStreamSynchronize(c->stream);
    if (c->p > 64) g_wide.remove(c->ws.device, c->stream);
    for (auto& s : c->spans) {
        (void)hipEventDestroy(s.beg);
        (void)hipEventDestroy(s.end);
    }
    if (c->sq_here != nullptr) (void)hipEventDestroy(c->sq_here);
    if (c->host_sq != nullptr) (void)hipHostFree(c->host_sq);
    hipError_t e2 = hipFree(c->ws_base);
    delete c;
    if (e != hipSuccess) return hip_fail(e);
    if (e2 != hipSuccess) return hip_fail(e2);
    return SBO_OK;
}

int sbo_code(sbo_ctx* c, const float* Y, int64_t m, const float* D, int32_t* blk, int32_t* supp,
             float* coef, float* err) {
    int rc = check_call(c, m);
    if (rc) return rc;
    if (!Y || !D || !blk || !supp || !coef || !err) return SBO_EINVAL;
    c->n_spans = 0;
    return run_code(c, Y, m, D, blk, supp, coef, err);
}

int sbo_group(sbo_ctx* c, const int32_t* blk, int64_t m, int32_t* counts, int32_t* offsets,
              int32_t* perm) {
    int rc = check_call(c, m);
    if (rc) return rc;
    if (!blk) return SBO_EINVAL;
    c->n_spans = 0;
    rc = run_group(c, blk, m);
    if (rc) return rc;
    if (counts)
        SBO_HIP(hipMemcpyAsync(counts, c->ws.counts, (size_t)c->K * 4, hipMemcpyDeviceToDevice,
                               c->stream));
    if (offsets)
        SBO_HIP(hipMemcpyAsync(offsets, c->ws.offsets, (size_t)(c->K + 1) * 4,
                               hipMemcpyDeviceToDevice, c->stream));
    if (perm)
        SBO_HIP(hipMemcpyAsync(perm, c->ws.perm, (size_t)m * 4, hipMemcpyDeviceToDevice, c->stream));
    return SBO_OK;
}

int sbo_group_static(const int32_t* blk, int64_t m, int K, int32_t* counts, int32_t* offsets,
                     int32_t* perm, void* hip_stream) {
    if (!blk || !counts || !offsets || !perm) return SBO_EINVAL;
    if (K < 1 || K > SBO_GROUP_STATIC_MAX_K || m < 1 || m > SBO_GROUP_STATIC_MAX_M) {
        g_hip_text = "sbo_group_static: K or m beyond the static scratch (K <= 128, m <= 1048576)";
        return SBO_ELIMIT;
    }
    static_assert(SBO_GROUP_STATIC_MAX_K == kGroupStaticMaxK && SBO_GROUP_STATIC_MAX_M == kGroupStaticMaxM,
                  "header and kernel limits differ");
    SBO_HIP(launch_group_static(K, blk, m, counts, offsets, perm, (hipStream_t)hip_stream));
    return SBO_OK;
}

int sbo_accumulate(sbo_ctx* c, const float* Y, int64_t m, const int32_t* blk, const int32_t* supp,
                   const float* coef, float* M) {
    int rc = check_call(c, m);
    if (rc) return rc;
    if (!Y || !blk || !supp || !coef || !M) return SBO_EINVAL;
    c->n_spans = 0;
    rc = run_group(c, blk, m);
    if (rc) return rc;
    StageTimer t(c, SBO_STAGE_ACCUM);
    SBO_HIP(launch_accumulate(c->p, c->K, c->s0, Y, m, supp, coef, c->ws, M, c->stream));
    return SBO_OK;
}

int sbo_polar(sbo_ctx* c, const float* M, const int32_t* counts, float* D) {
    if (!c || !M || !D) return SBO_EINVAL;
    c->n_spans = 0;
    StageTimer t(c, SBO_STAGE_SVD);
    SBO_HIP(launch_polar(c->p, c->K, M, counts, D, c->ws, c->svd_method, nullptr, 0, c->stream));
    return SBO_OK;
}

int sbo_update(sbo_ctx* c, const float* Y, int64_t m, const int32_t* blk, const int32_t* supp,
               const float* coef, float* D, int32_t* counts) {
    int rc = check_call(c, m);
    if (rc) return rc;
    if (!Y || !blk || !supp || !coef || !D) return SBO_EINVAL;
    c->n_spans = 0;
    if (lists_in_update(c->p, c->K, m) && c->svd_method != SBO_SVD_JACOBI) {
        {
            StageTimer t(c, SBO_STAGE_GROUP);
            SBO_HIP(launch_group_hist(c->K, blk, m, c->ws, c->stream));
        }
        {
            StageTimer t(c, SBO_STAGE_ACCUM);
            SBO_HIP(launch_accumulate(c->p, c->K, c->s0, Y, m, supp, coef, c->ws, nullptr, c->stream, false, blk));
        }
        rc = run_polar_pieces(c, m, D, 0, nullptr, nullptr);
    } else {
        rc = run_group(c, blk, m);
        if (rc) return rc;
        rc = run_update_grouped(c, Y, m, supp, coef, D);
    }
    if (rc) return rc;
    if (counts)
        SBO_HIP(hipMemcpyAsync(counts, c->ws.counts, (size_t)c->K * 4, hipMemcpyDeviceToDevice,
                               c->stream));
    return SBO_OK;
}

int sbo_iterate(sbo_ctx* c, const float* Y, int64_t m, float* D, int n_iter, int32_t* blk,
                int32_t* supp, float* coef, float* err, double* sqerr_per_iter) {
    int rc = check_call(c, m);
    if (rc) return rc;
    if (!Y || !D || !blk || !supp || !coef || !err || n_iter < 1) return SBO_EINVAL;
    c->n_spans = 0;
    const bool fused = c->p <= 64;             // select and accumulate share one pass over Y
    for (int it = 0; it < n_iter; ++it) {
        if (!fused) {
            rc = run_code(c, Y, m, D, blk, supp, coef, err, it);
            if (rc) return rc;
            rc = run_update_grouped(c, Y, m, supp, coef, D, code_ops(c), err,      // grouping reused
                                    sqerr_per_iter ? sqerr_per_iter + it : nullptr);
            if (rc) return rc;
            continue;
        }
        // The dictionary in the coding kernel's operand order: rewritten from D at the start
        // of the call, kept up to date by the SVD kernel afterwards.
        if (it == 0) {
            rc = run_swizzle(c, Y, m, D);
            if (rc) return rc;
        }
        rc = run_energy(c, Y, m, blk, it);
        if (rc) return rc;
        const bool lists = c->svd_method != SBO_SVD_JACOBI && lists_in_round(c->p, c->K, m);
        if (!lists) rc = run_group(c, blk, m, true);
        if (rc) return rc;
        {
            StageTimer t(c, SBO_STAGE_SELECT);  // includes the per-piece accumulation
            SBO_HIP(launch_select_accum(c->p, c->K, c->s0, Y, m, D, c->ws, supp, coef, err, c->stream,
                                        lists ? blk : nullptr));
        }
        rc = run_polar_pieces(c, m, D, energy_ops(c), err, sqerr_per_iter ? sqerr_per_iter + it : nullptr, -1, lists);
        if (rc) return rc;
    }
    return SBO_OK;
}

// own: D holds orthobases that the library has made.  sq_out: the squared-error total of the last round.
static int run_train_rounds(sbo_ctx* c, const float* Y, int64_t m, const int32_t* blk, float* D, int R,
                            int32_t* supp, float* coef, float* err, bool own = false, double* sq_out = nullptr) {
    int rc = run_group(c, blk, m);             // the assignment, hence the grouping, is fixed
    if (rc) return rc;
    for (int r = 0; r < R; ++r) {
        double* const sq = r == R - 1 ? sq_out : nullptr;
        const float* const sq_err = sq != nullptr ? err : nullptr;
        if (c->p <= 64) {
            {
                StageTimer t(c, SBO_STAGE_SELECT);
                SBO_HIP(launch_select_accum(c->p, c->K, c->s0, Y, m, D, c->ws, supp, coef, err,
                                            c->stream));
            }
            rc = run_polar_pieces(c, m, D, 0, sq_err, sq);
            if (rc) return rc;
            continue;
        } else {
            {
                StageTimer t(c, SBO_STAGE_SELECT);
                SBO_HIP(launch_select(c->p, c->K, c->s0, Y, m, D, c->ws, supp, coef, err, r > 0,
                                      select_arith(c, own), c->stream));
            }
            rc = run_update_grouped(c, Y, m, supp, coef, D, select_ops(c, own), sq_err, sq);
            if (rc) return rc;
        }
    }
    return SBO_OK;
}

int sbo_train_rounds(sbo_ctx* c, const float* Y, int64_t m, const int32_t* blk, float* D, int R,
                     int32_t* supp, float* coef, float* err) {
    int rc = check_call(c, m);
    if (rc) return rc;
    if (!Y || !blk || !D || !supp || !coef || !err || R < 1) return SBO_EINVAL;
    c->n_spans = 0;
    return run_train_rounds(c, Y, m, blk, D, R, supp, coef, err);
}

int sbo_set_blocks(sbo_ctx* c, int K) {
    if (!c || K < 1 || K > c->K_cap) return SBO_EINVAL;
    c->K = K;
    return SBO_OK;
}

int sbo_sqerr(sbo_ctx* c, const float* err, int64_t m, double* out) {
    int rc = check_call(c, m);
    if (rc) return rc;
    if (!err || !out) return SBO_EINVAL;
    SBO_HIP(launch_sqerr(err, nullptr, m, c->ws, out, c->stream));
    return SBO_OK;
}

int sbo_worst(sbo_ctx* c, const float* err, int64_t m, int64_t W, int32_t* ids) {
    int rc = check_call(c, m);
    if (rc) return rc;
    if (!err || !ids || W < 1 || W > m) return SBO_EINVAL;
    SBO_HIP(launch_worst(err, m, W, c->ws, ids, c->stream));
    return SBO_OK;
}

// Gram matrix of the set -> its eigenvectors by descending eigenvalue (ws.perm etc. hold the set; have_gram: ws.M the matrix).
static int run_init_base(sbo_ctx* c, const float* Y, int64_t n, float* Q, float* sv, bool have_gram = false) {
    if (!have_gram) SBO_HIP(launch_gram(c->p, 1, Y, n, c->ws, c->ws.M, c->stream));
    SBO_HIP(launch_polar(c->p, 1, c->ws.M, nullptr, Q, c->ws, c->svd_method == SBO_SVD_JACOBI,
                         sv ? sv : c->ws.energy, 0, c->stream));   // energy[m_max >= p] as a sink
    return SBO_OK;
}

int sbo_init_base(sbo_ctx* c, const float* Y, int64_t m, const int32_t* ids, int64_t n, float* Q,
                  float* sv) {
    int rc = check_call(c, m);
    if (rc) return rc;
    if (!Y || !ids || !Q || n < 1 || n > m) return SBO_EINVAL;
    if (c->m_max < c->p) return SBO_EINVAL;    // the workspace doubles as scratch of p floats
    c->n_spans = 0;
    SBO_HIP(launch_single_block(ids, n, m, c->ws, c->stream));
    return run_init_base(c, Y, n, Q, sv);
}

// ws.perm etc. already hold the set (launch_single_block).
static int run_new_base(sbo_ctx* c, const float* Y, int64_t n, int R, int have_q0, float* Q,
                        int32_t* supp, float* coef, float* err, double* sqerr_per_round, bool have_gram = false) {
    const bool own = !have_q0;
    if (!have_q0) {
        int rc = run_init_base(c, Y, n, Q, nullptr, have_gram);
        if (rc) return rc;
    }
    for (int r = 0; r < R; ++r) {
        if (c->p <= 64) {
            SBO_HIP(launch_select_accum(c->p, 1, c->s0, Y, n, Q, c->ws, supp, coef, err, c->stream));
        } else {
            SBO_HIP(launch_select(c->p, 1, c->s0, Y, n, Q, c->ws, supp, coef, err, r > 0, select_arith(c, own), c->stream));
        }
        if (sqerr_per_round)
            SBO_HIP(launch_sqerr(err, c->ws.perm, n, c->ws, sqerr_per_round + r, c->stream));
        int rc = c->p <= 64 ? run_polar_pieces(c, n, Q, 0, nullptr, nullptr, 1)
                            : run_update_grouped(c, Y, n, supp, coef, Q, select_ops(c, own), nullptr, nullptr, 1);
        if (rc) return rc;
    }
    return SBO_OK;
}

int sbo_new_base(sbo_ctx* c, const float* Y, int64_t m, const int32_t* ids, int64_t n, int R,
                 int have_q0, float* Q, int32_t* supp, float* coef, float* err,
                 double* sqerr_per_round) {
    int rc = check_call(c, m);
    if (rc) return rc;
    if (!Y || !ids || !Q || !supp || !coef || !err || n < 1 || n > m || R < 0) return SBO_EINVAL;
    if (c->m_max < c->p) return SBO_EINVAL;
    c->n_spans = 0;
    SBO_HIP(launch_single_block(ids, n, m, c->ws, c->stream));
    return run_new_base(c, Y, n, R, have_q0, Q, supp, coef, err, sqerr_per_round);
}

// RMSE of the codes in err (Section 4) on its way to the host: written there by the kernel that adds it up (a copy is a launch of
// its own), which is that of the last SVD update where there has been one (`added`) ...
static int prepare_sq(sbo_ctx* c) {
    if (c->host_sq == nullptr)
        SBO_HIP(hipHostMalloc(reinterpret_cast<void**>(&c->host_sq), sizeof(double), hipHostMallocDefault));
    if (c->sq_here == nullptr) SBO_HIP(hipEventCreateWithFlags(&c->sq_here, hipEventDisableTiming));
    return SBO_OK;
}
static int send_sq(sbo_ctx* c, const float* err, int64_t m, bool added) {
    if (!added) SBO_HIP(launch_sqerr(err, nullptr, m, c->ws, c->host_sq, c->stream));
    SBO_HIP(hipEventRecord(c->sq_here, c->stream));
    return SBO_OK;
}
// ... and there.
static int wait_rmse(sbo_ctx* c, int64_t m, double* out) {
    SBO_HIP(hipEventSynchronize(c->sq_here));
    *out = sqrt(*c->host_sq / ((double)c->p * (double)m));
    return SBO_OK;
}

// What a new orthobase starts from, in the workspace: the worst-W set as one block and its Gram matrix.
static int prepare_growth(sbo_ctx* c, const float* Y, const float* err, int64_t m, int64_t W) {
    SBO_HIP(launch_worst(err, m, W, c->ws, c->ws.perm, c->stream, true));
    SBO_HIP(launch_gram(c->p, 1, Y, W, c->ws, c->ws.M, c->stream));
    return SBO_OK;
}

int sbo_learn(sbo_ctx* c, const float* Y, int64_t m, float* D, const int32_t* init_ids, int K0,
              int64_t P0, int R, int64_t W, int K_max, double target_rmse, int32_t* blk,
              int32_t* supp, float* coef, float* err, int* K_final, double* rmse_hist, int* n_hist) {
    int rc = check_call(c, m);
    if (rc) return rc;
    if (!Y || !D || !init_ids || !blk || !supp || !coef || !err || !K_final || !rmse_hist || !n_hist)
        return SBO_EINVAL;
    if (K0 < 1 || K0 > K_max || K_max > c->K_cap || P0 < 1 || P0 > m || W < 1 || W > m || R < 1)
        return SBO_EINVAL;
    if (c->m_max < c->p) return SBO_EINVAL;
    // A graph can not wait for the host's decision.
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &capture) != hipSuccess) (void)hipGetLastError();
    if (capture != hipStreamCaptureStatusNone) return hip_fail(hipErrorStreamCaptureUnsupported);
    c->n_spans = 0;
    const int K_before = c->K;
    const size_t pp = (size_t)c->p * c->p;
    auto fail = [&](int code) {
        c->K = K_before;
        return code;
    };

    // Initialisation: K0 orthobases, each trained on its own signal set; then represent.
    // All K0 at once, the sets as K0 blocks of one grouping: eq. (5) for every block, then R rounds of selection,
    // accumulation and the SVD update over K0 blocks.  A signal that sits in two sets has its scratch rows of supp /
    // coef / err written twice, which nothing reads at p <= 64, where the codes do not go through memory; at p = 256
    // their rows are those of the positions in the grouping.  Sets that do not fit the workspace (p = 256: those
    // rows) are trained one after the other.
    const int64_t n_init = (int64_t)K0 * P0;
    if (n_init <= (c->p <= 64 ? c->m_max : m) && (int64_t)K0 * c->p <= c->m_max) {
        SBO_HIP(launch_equal_blocks(init_ids, K0, P0, m, c->ws, c->stream));
        SBO_HIP(launch_gram(c->p, K0, Y, n_init, c->ws, c->ws.M, c->stream));
        SBO_HIP(launch_polar(c->p, K0, c->ws.M, nullptr, D, c->ws, c->svd_method == SBO_SVD_JACOBI, c->ws.energy, 0,
                             c->stream));
        for (int r = 0; r < R; ++r) {
            if (c->p <= 64) {
                SBO_HIP(launch_select_accum(c->p, K0, c->s0, Y, n_init, D, c->ws, supp, coef, err, c->stream));
                rc = run_polar_pieces(c, n_init, D, 0, nullptr, nullptr, K0);
            } else {
                SBO_HIP(launch_select(c->p, K0, c->s0, Y, n_init, D, c->ws, supp, coef, err, r > 0, select_arith(c, true), c->stream,
                                      nullptr, false, true));
                rc = run_update_grouped(c, Y, n_init, supp, coef, D, select_ops(c, true), nullptr, nullptr, K0, true);
            }
            if (rc) return fail(rc);
        }
    } else {
        for (int j = 0; j < K0; ++j) {
            SBO_HIP(launch_single_block(init_ids + (size_t)j * P0, P0, m, c->ws, c->stream));
            rc = run_new_base(c, Y, P0, R, 0, D + j * pp, supp, coef, err, nullptr);
            if (rc) return fail(rc);
        }
    }
    int K = K0;
    c->K = K;
    rc = run_code(c, Y, m, D, blk, supp, coef, err);
    if (rc) return fail(rc);
    // The GPU goes on with the next growth step's worst-W set while the error travels to the host, which decides whether
    // there is to be one.  p = 64, m = 32768, K = 5 to 16: 6958 -> 6408 us (the host's answer, and the launches after
    // it, were waited for once per orthobase); a call that stops on the error pays some 40 us for a set it does not use.
    rc = prepare_sq(c);
    if (rc) return fail(rc);
    int n = 0;
    auto next_error = [&](bool added) {
        int e = send_sq(c, err, m, added);
        if (e == SBO_OK && K < K_max) e = prepare_growth(c, Y, err, m, W);
        return e != SBO_OK ? e : wait_rmse(c, m, &rmse_hist[n]);
    };
    rc = next_error(false);
    if (rc) return fail(rc);
    ++n;

    // Iterations: grow by one orthobase trained on the worst-W set, represent, train every
    // orthobase over its own signals, check the stopping rule.
    while (K < K_max && rmse_hist[n - 1] > target_rmse) {
        rc = run_new_base(c, Y, W, R, 0, D + K * pp, supp, coef, err, nullptr, true);
        if (rc) return fail(rc);
        ++K;
        c->K = K;
        rc = run_code(c, Y, m, D, blk, supp, coef, err);
        if (rc) return fail(rc);
        rc = run_train_rounds(c, Y, m, blk, D, R, supp, coef, err, true, c->host_sq);
        if (rc) return fail(rc);
        rc = next_error(true);
        if (rc) return fail(rc);
        ++n;
    }
    // Stopped by the error: the set prepared in vain still reads Y and err, which the caller may have back now.
    if (K < K_max)
        if (hipError_t e = hipStreamSynchronize(c->stream); e != hipSuccess) return fail(hip_fail(e));
    *K_final = K;
    *n_hist = n;
    c->K = K_before;
    return SBO_OK;
}

int sbo_svd_sweeps(sbo_ctx* c, int32_t* sweeps) {
    if (!c || !sweeps) return SBO_EINVAL;
    SBO_HIP(hipMemcpyAsync(sweeps, c->ws.sweeps, (size_t)c->K * 4, hipMemcpyDeviceToHost, c->stream));
    SBO_HIP(hipStreamSynchronize(c->stream));
    return SBO_OK;
}

// For tests, not in the header: sets the first n entries of ws.short_cut to -1 (read == nullptr), or reads them after a call: 1 where a
// workgroup decided by home or guessed blocks, 0 where it screened everything, -1 where another kernel chose.
int sbo_test_short_cuts(sbo_ctx* c, int32_t* read, int n) {
    if (!c || n < 0 || n > (int)((c->m_max + 255) / 256)) return SBO_EINVAL;
    if (read == nullptr)
        SBO_HIP(hipMemsetAsync(c->ws.short_cut, 0xff, (size_t)n * 4, c->stream));
    else
        SBO_HIP(hipMemcpyAsync(read, c->ws.short_cut, (size_t)n * 4, hipMemcpyDeviceToHost, c->stream));
    SBO_HIP(hipStreamSynchronize(c->stream));
    return SBO_OK;
}

// For tests, not in the header: p = 256, few orthobases: the SVD by teams whose second workgroups stay away (on = 0).
int sbo_test_wide_helpers(sbo_ctx* c, int on) {
    if (!c) return SBO_EINVAL;
    c->ws.wide_helpers = on != 0;
    return SBO_OK;
}

// For tests, not in the header: 1 = the next SVD of this context (p = 256) is made by teams of pairs.
int sbo_test_wide_pairs(sbo_ctx* c) { return c && c->p == 256 && wide_pairs(c->K, c->ws.device); }

int sbo_set_option(sbo_ctx* c, int option, int value) {
    if (!c) return SBO_EINVAL;
    switch (option) {
        case SBO_OPT_SVD_METHOD:
            if (value != SBO_SVD_AUTO && value != SBO_SVD_JACOBI) return SBO_EINVAL;
            c->svd_method = value;
            return SBO_OK;
        case SBO_OPT_CODING_ARITH:
            if (value != SBO_ARITH_F32 && value != SBO_ARITH_BF16X3 && value != SBO_ARITH_BF16X3_SCREEN &&
                value != SBO_ARITH_F16X2)
                return SBO_EINVAL;
            c->coding_arith = value;
            c->ws.parts_accum = value != SBO_ARITH_F32;
            return SBO_OK;
        case SBO_OPT_SVD_WAIT:
            if (value < 0) return SBO_EINVAL;
            c->ws.wide_polls = value;
            return SBO_OK;
        default: return SBO_EINVAL;
    }
}

int sbo_set_timing(sbo_ctx* c, int enable) {
    if (!c) return SBO_EINVAL;
    c->timing = enable == 2 ? 2 : (enable ? 1 : 0);
    c->n_spans = 0;
    return SBO_OK;
}

int sbo_stage_ms(sbo_ctx* c, float* ms) {
    if (!c || !ms) return SBO_EINVAL;
    for (int s = 0; s < SBO_N_STAGES; ++s) ms[s] = 0.f;
    SBO_HIP(hipStreamSynchronize(c->stream));
    for (size_t i = 0; i < c->n_spans; ++i) {
        float t = 0.f;
        SBO_HIP(hipEventElapsedTime(&t, c->spans[i].beg, c->spans[i].end));
        ms[c->spans[i].stage] += t;
    }
    return SBO_OK;
}

const char* sbo_strerror(int code) {
    switch (code) {
        case SBO_OK: return "success";
        case SBO_EINVAL: return "invalid argument or unsupported shape";
        case SBO_ENOMEM: return "out of device memory";
        case SBO_ELIMIT: return g_hip_text.c_str();
        case SBO_EHIP: return g_hip_text.c_str();
        default: return "unknown error code";
    }
}

}  // extern "C"
