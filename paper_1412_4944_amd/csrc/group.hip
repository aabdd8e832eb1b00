// Grouping of the signals by chosen block (Section 3.3: signal lists per base, built
// before the training step) as a deterministic counting sort, entirely on the device:
//   1. per-chunk histograms      (one wavefront per chunk of consecutive signals)
//   2. per-block scan over chunks (one workgroup per block)
//   3. stable scatter            (one wavefront per chunk; offsets = scan of counts)
// Few chunks and blocks: every workgroup of step 3 does step 2 for itself, from all the histograms (the
// launch, 4.5 us, is more than that up to about 10000 histogram entries: 1024 signals, K = 4: 11.5 -> 6.9 us for
// both; at 16384 entries 13.3 -> 14.6).
// Only integer additions are involved and every destination slot is computed, not
// claimed by an atomic, so perm is the unique stable permutation.
#include "sbo_internal.h"
#include "device_utils.h"

#include <mutex>

namespace sbo {

namespace {

constexpr int kMaxK = 1024;
constexpr int kScanInScatter = 8192;           // at most this many histogram entries

// Scratch of launch_group_static (the grouping for callers that must not allocate): the
// per-chunk histograms and per-chunk bases, [2][kStaticChunks][kGroupStaticMaxK] ints = 1 MiB
// on every GPU the library runs on, held until the process ends.
constexpr int kStaticChunks = 1024;            // group_geom() never makes more for m <= 2^20
static __device__ __align__(256) int32_t scratch[2 * kStaticChunks * kGroupStaticMaxK];

// Device address of `scratch` on each GPU (every GPU holds its own copy of the array); looked
// up once per device.  In host code the array's name is only a handle for this lookup.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
int32_t* g_scratch_ptr[kMaxDevices] = {};

hipError_t static_scratch(int32_t** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        int32_t* ptr = nullptr;
        e = hipGetSymbolAddress(reinterpret_cast<void**>(&ptr), HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (ptr == nullptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

// 1. chunk_count[c][j] = number of signals of chunk c that chose block j.
__global__ __launch_bounds__(256) void group_hist_kernel(const int32_t* __restrict__ blk, int m,
                                                         int K, int chunk, int n_chunks,
                                                         int32_t* __restrict__ chunk_count) {
    extern __shared__ int lds[];           // [4][K]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int* cnt = lds + wave * K;
    for (int j = lane; j < K; j += 64) cnt[j] = 0;
    __syncthreads();
    const int c = blockIdx.x * 4 + wave;
    if (c < n_chunks) {
        const int beg = c * chunk;
        const int end = min(m, beg + chunk);
        for (int i = beg + lane; i < end; i += 64) {
            const int b = blk[i];
            if ((unsigned)b < (unsigned)K) atomicAdd(&cnt[b], 1);   // out-of-range ids are dropped
        }
    }
    __syncthreads();
    if (c < n_chunks)
        for (int j = lane; j < K; j += 64) chunk_count[(int64_t)c * K + j] = cnt[j];
}

// 2. chunk_base[c][j] = number of signals of block j in chunks before c; counts[j] = total.
// The histogram entries are set back to zero once read: the coding kernel, which can
// produce them itself, adds into the array.
__global__ __launch_bounds__(256) void group_scan_kernel(int32_t* __restrict__ chunk_count,
                                                         int K, int n_chunks,
                                                         int32_t* __restrict__ chunk_base,
                                                         int32_t* __restrict__ counts) {
    __shared__ int out[4 * 256 + 1];
    __shared__ int tmp[16];
    const int j = blockIdx.x;
    int carry = 0;
    for (int c0 = 0; c0 < n_chunks; c0 += 1024) {
        const int n = min(1024, n_chunks - c0);
        wg_exclusive_scan4([&](int idx) { return chunk_count[(int64_t)(c0 + idx) * K + j]; }, n,
                           out, tmp);
        for (int idx = threadIdx.x; idx < n; idx += 256) {
            chunk_base[(int64_t)(c0 + idx) * K + j] = carry + out[idx];
            chunk_count[(int64_t)(c0 + idx) * K + j] = 0;
        }
        carry += out[n];
        __syncthreads();
    }
    if (threadIdx.x == 0) counts[j] = carry;
}

// 3. perm[offsets[j] + chunk_base[c][j] + rank inside the chunk] = signal id.
// SCAN: chunk_base and counts are not given but formed here from chunk_count (K <= 256), and counts written; the
// workgroup that is the last to have read chunk_count sets it to zero (done: counter, zero between launches;
// nullptr: chunk_count may stay as it is).
template <bool SCAN>
__global__ __launch_bounds__(256) void group_scatter_kernel(const int32_t* __restrict__ blk, int m,
                                                            int K, int chunk, int n_chunks,
                                                            const int32_t* __restrict__ chunk_base,
                                                            int32_t* chunk_count, int* done,
                                                            int32_t* __restrict__ counts,
                                                            int32_t* __restrict__ offsets,
                                                            int32_t* __restrict__ perm) {
    extern __shared__ int lds[];           // off[K+1] | tmp[16] | run[4][K] | SCAN: total[K] | before[K] | flag
    int* off = lds;
    int* tmp = lds + (K + 1);
    int* runs = tmp + 16;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = blockIdx.x * 4 + wave;
    int* run = runs + wave * K;
    const int beg = min(m, c * chunk), end = min(m, beg + chunk);
    int key[8];                                // on their way while the offsets are formed
    load_keys(blk, beg, end, key);
    int ticket = 0;
    if constexpr (SCAN) {
        int *total = runs + 4 * K, *before = total + K;
        for (int j = threadIdx.x; j < 2 * K; j += 256) total[j] = 0;
        __syncthreads();
        const int rows = 256 / K, j = (int)threadIdx.x % K, c0 = (int)blockIdx.x * 4;
        if ((int)threadIdx.x < rows * K) {
            int all = 0, front = 0;
#pragma unroll 8
            for (int r = (int)threadIdx.x / K; r < n_chunks; r += rows) {
                const int v = chunk_count[r * K + j];
                all += v;
                front += r < c0 ? v : 0;
            }
            atomicAdd(&total[j], all);
            atomicAdd(&before[j], front);
        }
        // and of the chunks of the wavefronts before this one
        for (int jj = lane; jj < K; jj += 64) {
            int v = 0;
            for (int w = 0; w < wave; ++w)
                if (c0 + w < n_chunks) v += chunk_count[(c0 + w) * K + jj];
            run[jj] = v;
        }
        __syncthreads();
        if (done != nullptr && threadIdx.x == 0) ticket = atomicAdd(done, 1);      // (looked at when all else is done)
        wg_exclusive_scan4([&](int idx) { return total[idx]; }, K, off, tmp);
        if (blockIdx.x == 0)
            for (int jj = threadIdx.x; jj < K; jj += 256) counts[jj] = total[jj];
        for (int jj = lane; jj < K; jj += 64) run[jj] += off[jj] + before[jj];
    } else {
        wg_exclusive_scan4([&](int idx) { return counts[idx]; }, K, off, tmp);
        if (c < n_chunks)
            for (int j = lane; j < K; j += 64) run[j] = off[j] + chunk_base[(int64_t)c * K + j];
    }
    if (blockIdx.x == 0)
        for (int j = threadIdx.x; j <= K; j += 256) offsets[j] = off[j];
    __builtin_amdgcn_wave_barrier();
    if (c < n_chunks) scatter_chunk(blk, key, beg, end, K, run, perm);
    if constexpr (SCAN)
        if (done != nullptr) {                 // uniform
            int* last = runs + 6 * K;
            if (threadIdx.x == 0) *last = ticket == (int)gridDim.x - 1;
            __syncthreads();
            if (*last) {
                for (int e = threadIdx.x; e < n_chunks * K; e += 256) chunk_count[e] = 0;
                if (threadIdx.x == 0) *done = 0;
            }
        }
}

// scan + scatter from the histograms in chunk_count
hipError_t launch_sort(int K, const int32_t* blk, int64_t m, const GroupGeom& g, int32_t* chunk_count, int32_t* chunk_base,
                       int* done, int32_t* counts, int32_t* offsets, int32_t* perm, hipStream_t st) {
    const unsigned wgs = (unsigned)((g.n_chunks + 3) / 4);
    if (K <= 256 && (int64_t)g.n_chunks * K <= kScanInScatter) {
        hipLaunchKernelGGL(group_scatter_kernel<true>, dim3(wgs), dim3(256), (K + 1 + 16 + 6 * K + 1) * sizeof(int), st, blk,
                           (int)m, K, g.chunk, g.n_chunks, nullptr, chunk_count, done, counts, offsets, perm);
    } else {
        hipLaunchKernelGGL(group_scan_kernel, dim3(K), dim3(256), 0, st, chunk_count, K, g.n_chunks, chunk_base, counts);
        hipLaunchKernelGGL(group_scatter_kernel<false>, dim3(wgs), dim3(256), (K + 1 + 16 + 4 * K) * sizeof(int), st, blk,
                           (int)m, K, g.chunk, g.n_chunks, chunk_base, nullptr, nullptr, counts, offsets, perm);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_group_hist(int K, const int32_t* blk, int64_t m, const Workspace& ws, hipStream_t st) {
    if (K > kMaxK) return hipErrorInvalidValue;
    const GroupGeom g = group_geom(m);
    hipLaunchKernelGGL(group_hist_kernel, dim3((unsigned)((g.n_chunks + 3) / 4)), dim3(256), 4 * K * sizeof(int), st, blk,
                       (int)m, K, g.chunk, g.n_chunks, ws.chunk_count);
    return hipGetLastError();
}

// have_hist: ws.chunk_count already holds the per-chunk histograms (written by the coding
// kernel); otherwise they are computed from blk here.
hipError_t launch_group(int K, const int32_t* blk, int64_t m, const Workspace& ws, bool have_hist,
                        hipStream_t st) {
    if (K > kMaxK) return hipErrorInvalidValue;
    const GroupGeom g = group_geom(m);
    if (!have_hist) {
        hipError_t e = launch_group_hist(K, blk, m, ws, st);
        if (e != hipSuccess) return e;
    }
    return launch_sort(K, blk, m, g, ws.chunk_count, ws.chunk_base, ws.group_done, ws.counts, ws.offsets, ws.perm, st);
}

// The same three kernels with the chunk arrays in the static device array above instead of
// a context's workspace: no allocation anywhere.  m <= kGroupStaticMaxM, K <= kGroupStaticMaxK
// (checked by the caller).  Nothing in the scratch has to start at zero: the histogram kernel
// writes every entry the later kernels read.
hipError_t launch_group_static(int K, const int32_t* blk, int64_t m, int32_t* counts, int32_t* offsets,
                               int32_t* perm, hipStream_t st) {
    if (K < 1 || K > kGroupStaticMaxK || m < 1 || m > kGroupStaticMaxM) return hipErrorInvalidValue;
    int32_t* base = nullptr;
    hipError_t e = static_scratch(&base);
    if (e != hipSuccess) return e;
    const GroupGeom g = group_geom(m);
    if (g.n_chunks > kStaticChunks) return hipErrorInvalidValue;
    int32_t* chunk_count = base;
    int32_t* chunk_base = base + (size_t)kStaticChunks * kGroupStaticMaxK;
    const unsigned wgs = (unsigned)((g.n_chunks + 3) / 4);
    hipLaunchKernelGGL(group_hist_kernel, dim3(wgs), dim3(256), 4 * K * sizeof(int), st, blk, (int)m, K,
                       g.chunk, g.n_chunks, chunk_count);
    return launch_sort(K, blk, m, g, chunk_count, chunk_base, nullptr, counts, offsets, perm, st);
}

}  // namespace sbo
