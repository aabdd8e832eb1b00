// The W worst represented signals (Algorithm 2, step 3): ids of the W largest squared
// residuals, ties towards the lower signal index, listed in ascending signal order.
//
// Most-significant-digit radix select on an order-preserving 32-bit key: four histogram
// passes of 8 bits each narrow the key of the W-th largest value down to all 32 bits
// (threshold T) and the number `need` of entries equal to T that still belong to the set.
// Histograms use integer atomics only, so the result does not depend on scheduling.
// The set {key > T} plus the first `need` entries with key == T is then written in
// ascending signal order by a two-level stable compaction (counts per chunk, scan over
// chunks, scan inside a chunk).
//
// No kernel waits on another workgroup: the digit found by pass k is recomputed from the
// finished histogram of pass k by every workgroup of the next launch (and stored once for
// the launch after that).
//
// Up to kOneMax entries one workgroup does all of it in one launch, the keys in its registers (us a
// call, one launch / eight: 1000 entries 8.8 / 24.1, 5000 9.0 / 27.4, 16384 13.8 / 28.8, 32768 22.6 / 29.4; with 64 keys to a
// lane, which do not fit the registers, 65536 49 / 29).
#include "sbo_internal.h"
#include "device_utils.h"

namespace sbo {

namespace {

constexpr int kBins = 256;
constexpr int kSelThreads = 256;
constexpr int kSelPerThread = kSelChunk / kSelThreads;   // consecutive entries per thread

// ascending key order = ascending float order (negative values and -0 included)
__device__ __forceinline__ uint32_t order_key(float v) {
    const uint32_t b = __float_as_uint(v);
    return b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u);
}

// Digit of pass `q` and the state after it, from the state before it and hist[q]:
// among the keys that share `prefix` in their higher digits, the `remaining`-th largest
// has digit d where (#keys with digit > d) < remaining <= (#keys with digit >= d).
// Every thread of the workgroup (kSelThreads) must call this; result in st[0..1].
__device__ __forceinline__ void resolve_pass(const int* __restrict__ hist_q, uint32_t prefix,
                                             int remaining, int* above, int* tmp, int* st) {
    if (threadIdx.x == 0) {                    // defined even if the state handed in is not
        st[0] = 0;
        st[1] = 1;
    }
    // above[idx] = number of keys with digit > 255 - idx
    wg_exclusive_scan4([&](int idx) { return hist_q[kBins - 1 - idx]; }, kBins, above, tmp);
    const int t = threadIdx.x;
    if (t < kBins) {
        const int d = kBins - 1 - t;
        const int gt = above[t], ge = gt + hist_q[d];
        if (gt < remaining && remaining <= ge) {
            st[0] = (int)((prefix << 8) | (uint32_t)d);
            st[1] = remaining - gt;
        }
    }
    __syncthreads();
}

// State before pass `pass` (prefix of the higher digits, entries still to take inside it).
// state[q] = state after pass q, stored by workgroup 0 of the launch that resolved it.
__device__ __forceinline__ void state_before(int pass, int W, const int* __restrict__ hist,
                                             int* __restrict__ state, int* above, int* tmp,
                                             int* st, uint32_t& prefix, int& remaining) {
    prefix = 0;
    remaining = W;
    if (pass == 0) return;
    if (pass >= 2) {
        prefix = (uint32_t)state[(pass - 2) * 2];
        remaining = state[(pass - 2) * 2 + 1];
    }
    resolve_pass(hist + (pass - 1) * kBins, prefix, remaining, above, tmp, st);
    prefix = (uint32_t)st[0];
    remaining = st[1];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        state[(pass - 1) * 2] = st[0];
        state[(pass - 1) * 2 + 1] = st[1];
    }
}

__global__ __launch_bounds__(kSelThreads) void worst_clear_kernel(int* __restrict__ hist) {
    for (int e = threadIdx.x; e < 4 * kBins; e += kSelThreads) hist[e] = 0;
}

__global__ __launch_bounds__(kSelThreads) void worst_hist_kernel(const float* __restrict__ err,
                                                                 int m, int W, int pass,
                                                                 int* __restrict__ hist,
                                                                 int* __restrict__ state) {
    __shared__ int lh[kBins];
    __shared__ int above[kBins + 1];
    __shared__ int tmp[16];
    __shared__ int st[2];
    uint32_t prefix;
    int remaining;
    state_before(pass, W, hist, state, above, tmp, st, prefix, remaining);

    const int tid = threadIdx.x;
    lh[tid] = 0;
    __syncthreads();
    const int shift = 24 - 8 * pass;
    for (int i = blockIdx.x * kSelThreads + tid; i < m; i += gridDim.x * kSelThreads) {
        const uint32_t key = order_key(err[i]);
        if (pass == 0 || (key >> (shift + 8)) == prefix) atomicAdd(&lh[(key >> shift) & 255u], 1);
    }
    __syncthreads();
    if (lh[tid] != 0) atomicAdd(&hist[pass * kBins + tid], lh[tid]);
}

// cnt[chunk] = (entries above T, entries equal to T) of the chunk
__global__ __launch_bounds__(kSelThreads) void worst_count_kernel(const float* __restrict__ err,
                                                                  int m, int W,
                                                                  int* __restrict__ hist,
                                                                  int* __restrict__ state,
                                                                  int* __restrict__ cnt) {
    __shared__ int above[kBins + 1];
    __shared__ int tmp[16];
    __shared__ int st[2];
    __shared__ int red[2][kSelThreads / 64];
    uint32_t T;
    int need;
    state_before(4, W, hist, state, above, tmp, st, T, need);

    const int tid = threadIdx.x;
    const int i0 = blockIdx.x * kSelChunk + tid * kSelPerThread;
    int gt = 0, eq = 0;
#pragma unroll
    for (int e = 0; e < kSelPerThread; ++e) {
        if (i0 + e < m) {
            const uint32_t key = order_key(err[i0 + e]);
            gt += key > T;
            eq += key == T;
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        gt += __shfl_xor(gt, o, 64);
        eq += __shfl_xor(eq, o, 64);
    }
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = gt;
        red[1][tid >> 6] = eq;
    }
    __syncthreads();
    if (tid == 0) {
        int g = 0, q = 0;
        for (int w = 0; w < kSelThreads / 64; ++w) {
            g += red[0][w];
            q += red[1][w];
        }
        cnt[blockIdx.x * 2] = g;
        cnt[blockIdx.x * 2 + 1] = q;
    }
}

// base[chunk] = exclusive sums of cnt over the chunks before it (one workgroup)
__global__ __launch_bounds__(kSelThreads) void worst_scan_kernel(const int* __restrict__ cnt,
                                                                 int n_chunks,
                                                                 int* __restrict__ base) {
    __shared__ int out[4 * kSelThreads + 1];
    __shared__ int tmp[16];
    for (int which = 0; which < 2; ++which) {
        int carry = 0;
        for (int c0 = 0; c0 < n_chunks; c0 += 4 * kSelThreads) {
            const int n = min(4 * kSelThreads, n_chunks - c0);
            wg_exclusive_scan4([&](int idx) { return cnt[(c0 + idx) * 2 + which]; }, n, out, tmp);
            for (int e = threadIdx.x; e < n; e += kSelThreads) base[(c0 + e) * 2 + which] = carry + out[e];
            carry += out[n];
            __syncthreads();                   // out is rewritten by the next batch
        }
    }
}

// offsets != nullptr: also the set as the grouping of one block (as launch_single_block).
__global__ __launch_bounds__(kSelThreads) void worst_emit_kernel(const float* __restrict__ err,
                                                                 int m, int W,
                                                                 const int* __restrict__ state,
                                                                 const int* __restrict__ base,
                                                                 int32_t* __restrict__ ids, int32_t* __restrict__ counts,
                                                                 int32_t* __restrict__ offsets) {
    __shared__ int cg[kSelThreads], cq[kSelThreads];
    __shared__ int og[kSelThreads + 1], oq[kSelThreads + 1];
    __shared__ int tmp[16];
    const uint32_t T = (uint32_t)state[3 * 2];
    const int need = state[3 * 2 + 1];

    const int tid = threadIdx.x;
    if (offsets != nullptr && blockIdx.x == 0 && tid == 0) {
        counts[0] = W;
        offsets[0] = 0;
        offsets[1] = W;
    }
    const int i0 = blockIdx.x * kSelChunk + tid * kSelPerThread;
    uint32_t key[kSelPerThread];
    int gt = 0, eq = 0;
#pragma unroll
    for (int e = 0; e < kSelPerThread; ++e) {
        key[e] = i0 + e < m ? order_key(err[i0 + e]) : 0u;
        if (i0 + e < m) {
            gt += key[e] > T;
            eq += key[e] == T;
        }
    }
    cg[tid] = gt;
    cq[tid] = eq;
    __syncthreads();
    wg_exclusive_scan4([&](int idx) { return cg[idx]; }, kSelThreads, og, tmp);
    wg_exclusive_scan4([&](int idx) { return cq[idx]; }, kSelThreads, oq, tmp);
    int g_before = base[blockIdx.x * 2] + og[tid];
    int q_before = base[blockIdx.x * 2 + 1] + oq[tid];
#pragma unroll
    for (int e = 0; e < kSelPerThread; ++e) {
        if (i0 + e >= m) break;
        const bool is_gt = key[e] > T, is_eq = key[e] == T;
        if (is_gt || (is_eq && q_before < need)) {
            const int pos = g_before + min(q_before, need);
            if (pos < W) ids[pos] = i0 + e;    // always true; keeps a wrong state from writing past the list
        }
        g_before += is_gt;
        q_before += is_eq;
    }
}

// The same by one workgroup.  Wavefront w holds the entries 64 Q w .. 64 Q (w + 1) - 1, 64 consecutive ones per q, so that
// ballots count them in index order.  Lanes l and l + 32 count in a copy of their own of the 256 bins, in a bank of its
// own: the leading digits (sign and exponent) are nearly all the same.
// counts, offsets: as worst_emit_kernel.
constexpr int kOneWaves = 16;
constexpr int64_t kOneMax = 64 * 32 * kOneWaves;

template <int Q>
__global__ __launch_bounds__(64 * kOneWaves) void worst_one_kernel(const float* __restrict__ err, int m, int W,
                                                                   int32_t* __restrict__ ids, int32_t* __restrict__ counts,
                                                                   int32_t* __restrict__ offsets) {
    constexpr int NTH = 64 * kOneWaves;
    __shared__ int hist[kBins * 32];
    __shared__ int bin[kBins];
    __shared__ int st[2];
    __shared__ int n_gt[kOneWaves], n_eq[kOneWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = wave * 64 * Q + lane;       // entry q of this lane: i0 + 64 q

    uint32_t key[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) key[q] = order_key(err[min(i0 + 64 * q, m - 1)]);
    if (offsets != nullptr && tid == 0) {
        counts[0] = W;
        offsets[0] = 0;
        offsets[1] = W;
    }

    uint32_t prefix = 0;
    int remaining = W;
#pragma unroll 1
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        for (int e = tid; e < kBins * 32; e += NTH) hist[e] = 0;
        if (tid < 2) st[tid] = tid;            // defined whatever happens
        __syncthreads();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const bool in = i0 + 64 * q < m && (pass == 0 || (key[q] >> 8 >> shift) == prefix);
            if (in) atomicAdd(&hist[((key[q] >> shift) & 255u) * 32 + (lane & 31)], 1);
        }
        __syncthreads();
        {                                      // four threads to a bin, each in other banks than its neighbours
            const int b = tid >> 2;
            int s = 0;
#pragma unroll
            for (int c = 0; c < 8; ++c) s += hist[b * 32 + (tid & 3) * 8 + ((c + b) & 7)];
            s += __shfl_xor(s, 1, 64);
            s += __shfl_xor(s, 2, 64);
            if ((tid & 3) == 0) bin[b] = s;
        }
        __syncthreads();
        if (wave == 0) {                       // digits 255 - 4 lane .. 252 - 4 lane
            int own[4], sum = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) sum += own[e] = bin[kBins - 1 - 4 * lane - e];
            int above = sum;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int x = __shfl_up(above, o, 64);
                if (lane >= o) above += x;
            }
            above -= sum;                      // entries with a higher digit
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (above < remaining && remaining <= above + own[e]) {
                    st[0] = (int)((prefix << 8) | (uint32_t)(kBins - 1 - 4 * lane - e));
                    st[1] = remaining - above;
                }
                above += own[e];
            }
        }
        __syncthreads();
        prefix = (uint32_t)st[0];
        remaining = st[1];
        __syncthreads();                       // (st is set anew by the next pass)
    }

    // the keys above `prefix` and the first `remaining` equal to it, in index order
    int gt = 0, eq = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const bool in = i0 + 64 * q < m;
        gt += __popcll(__ballot(in && key[q] > prefix));
        eq += __popcll(__ballot(in && key[q] == prefix));
    }
    if (lane == 0) {
        n_gt[wave] = gt;
        n_eq[wave] = eq;
    }
    __syncthreads();
    int pos = 0, eq_before = 0;
    for (int w = 0; w < wave; ++w) {
        pos += n_gt[w];
        eq_before += n_eq[w];
    }
    pos += min(eq_before, remaining);
    const unsigned long long before = (1ull << lane) - 1ull;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const bool in = i0 + 64 * q < m, is_eq = in && key[q] == prefix;
        const unsigned long long eqs = __ballot(is_eq);
        const bool take = (in && key[q] > prefix) || (is_eq && eq_before + __popcll(eqs & before) < remaining);
        const unsigned long long takes = __ballot(take);
        const int at = pos + __popcll(takes & before);
        if (take && at < W) ids[at] = i0 + 64 * q;         // at < W always (as in worst_emit_kernel)
        pos += __popcll(takes);
        eq_before += __popcll(eqs);
    }
}

}  // namespace

// block: the set also becomes the grouping of one block (ids: ws.perm), as launch_single_block would make it.
hipError_t launch_worst(const float* err, int64_t m, int64_t W, const Workspace& ws, int32_t* ids,
                        hipStream_t st, bool block) {
    if (block && ids != ws.perm) return hipErrorInvalidValue;
    int32_t *counts = block ? ws.counts : nullptr, *offsets = block ? ws.offsets : nullptr;
    if (m <= kOneMax) {
        const auto one = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(1), dim3(64 * kOneWaves), 0, st, err, (int)m, (int)W, ids, counts, offsets);
            return hipGetLastError();
        };
        return m <= kOneMax / 4 ? one(worst_one_kernel<8>) : m <= kOneMax / 2 ? one(worst_one_kernel<16>) : one(worst_one_kernel<32>);
    }
    const int n_chunks = (int)((m + kSelChunk - 1) / kSelChunk);
    const int hist_grid = n_chunks < 1024 ? n_chunks : 1024;
    hipLaunchKernelGGL(worst_clear_kernel, dim3(1), dim3(kSelThreads), 0, st, ws.sel_hist);
    for (int pass = 0; pass < 4; ++pass)
        hipLaunchKernelGGL(worst_hist_kernel, dim3(hist_grid), dim3(kSelThreads), 0, st, err, (int)m,
                           (int)W, pass, ws.sel_hist, ws.sel_state);
    hipLaunchKernelGGL(worst_count_kernel, dim3(n_chunks), dim3(kSelThreads), 0, st, err, (int)m, (int)W,
                       ws.sel_hist, ws.sel_state, ws.sel_cnt);
    hipLaunchKernelGGL(worst_scan_kernel, dim3(1), dim3(kSelThreads), 0, st, ws.sel_cnt, n_chunks,
                       ws.sel_base);
    hipLaunchKernelGGL(worst_emit_kernel, dim3(n_chunks), dim3(kSelThreads), 0, st, err, (int)m, (int)W,
                       ws.sel_state, ws.sel_base, ids, counts, offsets);
    return hipGetLastError();
}

}  // namespace sbo
