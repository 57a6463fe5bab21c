// Reductions next to the filter: the sum (and mean) of an FP32 array and the
// 256-bin histogram of a uint8 array.
//
// The paper's `reduction` directive marks scalars that a loop accumulates
// into, so that the iterations may still run in parallel (Sec. II-B.3), and
// OptiML's `sum` becomes a for loop with such a reduction (Sec. III-B). The
// histogram is the indirect increment A[t[i]]++ of the `independent`
// example (Sec. II-B.3), where t[i] repeats: a reduction per bin.
//
// Reassociating a floating-point sum changes its rounding (the paper's
// reproducibility remark, Sec. III-A). The sum here is reproducible: the
// array is cut into fixed chunks of kChunk elements, each chunk is summed in
// float64 by a fixed pattern (thread t of 256 takes float4 groups t, t +
// 256, ... in order, then a fixed pairwise tree over the 256 threads), and
// the chunk sums are added by the same fixed tree. None of this depends on
// the grid size or on timing, so every call on every device gives the same
// bits. Histogram counts are integers: any order is exact.
//
// Both run as two launches over a caller-provided workspace (chunk partials,
// per-block sub-histograms), so nothing is allocated and nothing needs
// zeroing; an array that one workgroup takes alone (a sum of one chunk, a
// histogram of up to kHistUnit bytes) as one.
#include <mutex>

#include "dev_common.h"
#include "pf_internal.h"

namespace pf {
namespace red {

constexpr int kThreads = 256;
constexpr int64_t kChunk = 65536;  // elements per chunk partial (fixed: part of the definition of the result)
constexpr int kSumBlocks = 2048;   // most blocks of the partial-sum launch
constexpr int64_t kHistSpan = 1 << 18;  // bytes per sub-histogram: of the least workspace, of a server task
constexpr int kHistRows = 1024;         // most sub-histograms
constexpr int kHistThreads = 512;
constexpr int kHistDeep = 4;            // 16-byte loads per thread in one batch; the next batch is in flight
constexpr int64_t kHistUnit = 16 * kHistThreads * kHistDeep;  // bytes per workgroup and batch

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// Elements of part c of an n-element array cut into parts of `part` elements.
// From 32-bit comparisons: written as min(part, n - c * part) in 64 bits, the
// compiler (ROCm 7.2) took the minimum from a stale condition bit in
// k_sum_partial, and the last chunk was summed past its end.
__device__ __forceinline__ int part_len(int64_t n, int c, int64_t part) {
    const int last = (int)((n - 1) / part);  // n <= 2^40
    return c < last ? (int)part : (int)(n - c * part);
}

// Fixed pairwise tree over the block's 256 values in LDS; returns the total
// in thread 0.
__device__ __forceinline__ double block_tree(double v, double *s) {
    s[threadIdx.x] = v;
    __syncthreads();
#pragma unroll
    for (int half = kThreads / 2; half > 0; half >>= 1) {
        if ((int)threadIdx.x < half) s[threadIdx.x] = s[threadIdx.x] + s[threadIdx.x + half];
        __syncthreads();
    }
    return s[0];
}

// Sum of one chunk p[0 .. len) (len <= kChunk) by the fixed pattern: thread
// t takes float4 groups t, t + 256, ... in order, then the block tree. The
// total is returned in thread 0. Every caller (single arrays and server
// batches) sums a chunk with this function, so a chunk's bits never depend
// on which launch computed it. STREAM: loads carry the non-temporal hint.
template <bool STREAM = false>
__device__ __forceinline__ double chunk_sum(const float *__restrict__ p, int len, double *s) {
    double acc = 0.0;
    if (len == kChunk) {
        // 64 float4 groups per thread; loads in batches of 16 in flight.
#pragma unroll 1
        for (int k0 = 0; k0 < 64; k0 += 16) {
            f4u q[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const f4u *g = reinterpret_cast<const f4u *>(p + 4 * (threadIdx.x + (k0 + k) * kThreads));
                if constexpr (STREAM) q[k] = __builtin_nontemporal_load(g);
                else q[k] = *g;
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                acc = acc + (double)q[k].x;
                acc = acc + (double)q[k].y;
                acc = acc + (double)q[k].z;
                acc = acc + (double)q[k].w;
            }
        }
    } else {
        // The same order, stopping at len: whole groups in batches in flight,
        // a group past len as zeros (acc is never -0, so adding +0 leaves it as
        // it is), then the elements of the last partial group, which is its
        // thread's last. Element by element, each load waited for, a sum of
        // 4096 elements took 12.3 us (now 3.6 us).
        const int ng = len / 4;
#pragma unroll 1
        for (int k0 = 0; k0 < 64 && k0 * kThreads < ng; k0 += 16) {
            f4u q[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int g = (int)threadIdx.x + (k0 + k) * kThreads;
                q[k] = f4u{0.0f, 0.0f, 0.0f, 0.0f};
                if (g < ng) q[k] = *reinterpret_cast<const f4u *>(p + 4 * g);
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                acc = acc + (double)q[k].x;
                acc = acc + (double)q[k].y;
                acc = acc + (double)q[k].z;
                acc = acc + (double)q[k].w;
            }
        }
        if ((int)threadIdx.x == ng % kThreads)
            for (int e = 4 * ng; e < len; ++e) acc = acc + (double)p[e];
    }
    return block_tree(acc, s);
}

// partial[c] = sum of chunk c, for the chunks this block takes. STREAM from
// 256 MiB up, the size of the last-level cache, where a call cannot find its
// input there: loads carry the non-temporal hint and block b takes the chunks
// b, b + grid, ..., so that the XCDs read one window of the array together
// (a contiguous eighth per XCD: 60 us for 2^26 elements; the window 50 us,
// with the hint 44.6 us = 6.0 TB/s; 2^27: 99, 95 and 84.7 us). Below, a
// contiguous eighth per XCD without the hint is ahead (2^24, inputs partly in
// the cache: 13.1 us; the window 13.3 us, with the hint 15.0 us).
template <bool STREAM>
__global__ __launch_bounds__(kThreads) void k_sum_partial(const float *__restrict__ x, int64_t n,
                                                          double *__restrict__ partial, int nchunks) {
    __shared__ double s[kThreads];
    for (int c = STREAM ? blockIdx.x : xcd_remap(blockIdx.x, gridDim.x); c < nchunks; c += gridDim.x) {
        const double total = chunk_sum<STREAM>(x + c * kChunk, part_len(n, c, kChunk), s);
        if (threadIdx.x == 0) partial[c] = total;
        __syncthreads();
    }
}

// out[0] = sum of the partials (fixed tree), out[1] = out[0] / n.
__device__ __forceinline__ void final_sum(const double *__restrict__ partial, int64_t nchunks, int64_t n,
                                          double *__restrict__ out, double *s) {
    double acc = 0.0;
    for (int64_t c = threadIdx.x; c < nchunks; c += kThreads) acc = acc + partial[c];
    const double total = block_tree(acc, s);
    if (threadIdx.x == 0) {
        out[0] = total;
        out[1] = total / (double)n;
    }
}

__global__ __launch_bounds__(kThreads) void k_sum_final(const double *__restrict__ partial, int64_t nchunks, int64_t n,
                                                        double *__restrict__ out) {
    __shared__ double s[kThreads];
    final_sum(partial, nchunks, n, out, s);
}

// One chunk: its sum is the result (the final launch would add zeros to it).
__global__ __launch_bounds__(kThreads) void k_sum_one(const float *__restrict__ x, int n,
                                                      double *__restrict__ out) {
    __shared__ double s[kThreads];
    const double total = chunk_sum(x, n, s);
    if (threadIdx.x == 0) {
        out[0] = total;
        out[1] = total / (double)n;
    }
}

// sub[b][v]: count of byte value v in the bytes block b takes. The block's
// LDS histogram keeps 32 copies of every bin, interleaved so that copy c of
// bin v is word 32 v + c: lane l counts into copy l mod 32, so the atomics
// of a wave fall into distinct banks whatever the data (a plain 256-word
// histogram serialises lanes whose bins share a bank).
constexpr int kCopies = 32;

// Counts the four bytes of a word into a thread's copy of the histogram.
__device__ __forceinline__ void count_word(uint32_t *mine, uint32_t v) {
    atomicAdd(&mine[kCopies * (v & 0xff)], 1u);
    atomicAdd(&mine[kCopies * ((v >> 8) & 0xff)], 1u);
    atomicAdd(&mine[kCopies * ((v >> 16) & 0xff)], 1u);
    atomicAdd(&mine[kCopies * (v >> 24)], 1u);
}

// Counts the bytes p[0 .. len) into the calling thread's copy of a block
// histogram, taking the whole 16-byte vectors at `first`, first + threads, ..
// (kHistDeep of them), then again `step` vectors on; the next batch is loaded
// while one is counted (46.5 us for the counting of 256 MiB, 49.9 us without). The few bytes
// before the first and after the last aligned vector go to the workgroup
// with `ends` set.
__device__ __forceinline__ void count_bytes(const uint8_t *__restrict__ p, int64_t len, int64_t first, int64_t step,
                                            bool ends, uint32_t *mine) {
    const int head = (int)(-(uintptr_t)p & 15);
    const int64_t nv = (len - head) / 16;  // 0 for len < head
    const uint4 *q = reinterpret_cast<const uint4 *>(p + head);
    if (ends) {
        if ((int)threadIdx.x < head && threadIdx.x < len) atomicAdd(&mine[kCopies * p[threadIdx.x]], 1u);
        const int64_t j = head + 16 * nv + threadIdx.x;
        if (j < len) atomicAdd(&mine[kCopies * p[j]], 1u);
    }
    if (first >= nv) return;
    uint4 v[kHistDeep], w[kHistDeep];
#pragma unroll
    for (int u = 0; u < kHistDeep; ++u) v[u] = q[min(first + u * kHistThreads, nv - 1)];
    for (int64_t i = first; i < nv; i += step) {
#pragma unroll
        for (int u = 0; u < kHistDeep; ++u) w[u] = q[min(i + step + u * kHistThreads, nv - 1)];
#pragma unroll
        for (int u = 0; u < kHistDeep; ++u) {
            if (i + u * kHistThreads < nv) {
                count_word(mine, v[u].x);
                count_word(mine, v[u].y);
                count_word(mine, v[u].z);
                count_word(mine, v[u].w);
            }
            v[u] = w[u];
        }
    }
}

__device__ __forceinline__ void clear_copies(uint32_t *hs) {
    for (int i = threadIdx.x; i < 256 * kCopies; i += kHistThreads) hs[i] = 0u;
    __syncthreads();
}

// o[v] = the block histogram's count of value v (its 32 copies added).
template <class T>
__device__ __forceinline__ void fold_copies(const uint32_t *hs, T *__restrict__ o) {
    __syncthreads();
    for (int v = threadIdx.x; v < 256; v += kHistThreads) {
        uint32_t t = 0;
#pragma unroll
        for (int c = 0; c < kCopies; ++c) t += hs[kCopies * v + ((c + v) & (kCopies - 1))];
        o[v] = t;
    }
}

// Block b takes the units b, b + grid, ... of the array: the workgroups in
// flight read one compact, advancing window of it, whatever its size, and an
// array of a few units already spreads over as many CUs. Bound by HBM from
// about 64 MiB up, by LDS atomics (8 to 10 a clock and CU) within one CU:
// with spans of 256 KiB, as before, a span alone took 13 us. Both launches,
// before -> now, us: 16 KiB 6.4 -> 3.7, 1 MiB 18.3 -> 6.4, 16 MiB 21.7 -> 9.8,
// 64 MiB 22.8 -> 16.4, 256 MiB 62 -> 51.
__global__ __launch_bounds__(kHistThreads) void k_hist_partial(const uint8_t *__restrict__ x, int64_t n,
                                                               uint32_t *__restrict__ sub) {
    __shared__ uint32_t hs[256 * kCopies];
    clear_copies(hs);
    count_bytes(x, n, (int64_t)blockIdx.x * kHistThreads * kHistDeep + threadIdx.x,
                (int64_t)gridDim.x * kHistThreads * kHistDeep, blockIdx.x == 0, hs + (threadIdx.x & (kCopies - 1)));
    fold_copies(hs, sub + (int64_t)blockIdx.x * 256);
}

// One block's array: its counts are the result.
__global__ __launch_bounds__(kHistThreads) void k_hist_one(const uint8_t *__restrict__ x, int64_t n,
                                                           int64_t *__restrict__ hist) {
    __shared__ uint32_t hs[256 * kCopies];
    clear_copies(hs);
    count_bytes(x, n, threadIdx.x, kHistThreads * kHistDeep, true, hs + (threadIdx.x & (kCopies - 1)));
    fold_copies(hs, hist);
}

// hist[v] = sum over rows of sub[row][v] for the 16 values v of this
// workgroup: 16 threads read a row's 64 bytes, 16 rows at a time, then the
// partial sums are added in LDS (integers: exact in any order). One value per
// workgroup, each row read for 4 bytes of it, took 4.7 us at 1024 rows.
constexpr int kFinalBins = 16, kFinalRows = kThreads / kFinalBins;
__device__ __forceinline__ void hist_final(const uint32_t *__restrict__ sub, int64_t rows, int64_t *__restrict__ hist) {
    __shared__ int64_t s[kThreads];
    const int bin = kFinalBins * blockIdx.x + threadIdx.x % kFinalBins;
    int64_t acc = 0;
    for (int64_t b0 = threadIdx.x / kFinalBins; b0 < rows; b0 += 16 * kFinalRows) {
        uint32_t q[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            q[u] = 0u;
            if (b0 + u * kFinalRows < rows) q[u] = sub[(b0 + u * kFinalRows) * 256 + bin];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) acc += q[u];
    }
    s[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x < kFinalBins) {
        int64_t t = 0;
#pragma unroll
        for (int k = 0; k < kFinalRows; ++k) t += s[threadIdx.x + kFinalBins * k];
        hist[bin] = t;
    }
}

__global__ __launch_bounds__(kThreads) void k_hist_final(const uint32_t *__restrict__ sub, int rows,
                                                         int64_t *__restrict__ hist) {
    hist_final(sub, rows, hist);
}

// ---- many arrays in one launch (server batches) -----------------------------
// Task t of a batch is part `part` (a chunk of kChunk floats for a sum, a
// span of kHistSpan bytes for a histogram) of request `req`; its partial
// goes to slot reqs[req].first + part of the batch workspace. Each part is
// reduced by the same device function as in the single-array kernels, so a
// request's result is bit for bit that of pf_sum_f32 / pf_hist256_u8 on the
// same array, whichever batch it lands in.

__global__ __launch_bounds__(kThreads) void k_sum_partial_multi(const ReduceReq *__restrict__ reqs,
                                                                const ReduceTask *__restrict__ tasks, int ntasks,
                                                                double *__restrict__ partial) {
    __shared__ double s[kThreads];
    for (int t = xcd_remap(blockIdx.x, gridDim.x); t < ntasks; t += gridDim.x) {
        const ReduceTask tk = tasks[t];
        const ReduceReq q = reqs[tk.req];
        const double total =
            chunk_sum(global_ptr<const float>(q.in) + tk.part * kChunk, part_len(q.n, tk.part, kChunk), s);
        if (threadIdx.x == 0) partial[q.first + tk.part] = total;
        __syncthreads();
    }
}

// One workgroup per sum request (ids lists them).
__global__ __launch_bounds__(kThreads) void k_sum_final_multi(const ReduceReq *__restrict__ reqs,
                                                              const int32_t *__restrict__ ids,
                                                              const double *__restrict__ partial) {
    __shared__ double s[kThreads];
    const ReduceReq q = reqs[ids[blockIdx.x]];
    final_sum(partial + q.first, (q.n + kChunk - 1) / kChunk, q.n, global_ptr<double>(q.out), s);
}

__global__ __launch_bounds__(kHistThreads) void k_hist_partial_multi(const ReduceReq *__restrict__ reqs,
                                                                     const ReduceTask *__restrict__ tasks, int ntasks,
                                                                     uint32_t *__restrict__ sub) {
    __shared__ uint32_t hs[256 * kCopies];
    for (int t = xcd_remap(blockIdx.x, gridDim.x); t < ntasks; t += gridDim.x) {
        const ReduceTask tk = tasks[t];
        const ReduceReq q = reqs[tk.req];
        clear_copies(hs);
        count_bytes(global_ptr<const uint8_t>(q.in) + tk.part * kHistSpan, part_len(q.n, tk.part, kHistSpan),
                    threadIdx.x, kHistThreads * kHistDeep, true, hs + (threadIdx.x & (kCopies - 1)));
        fold_copies(hs, sub + (q.first + tk.part) * 256);
        __syncthreads();
    }
}

// Workgroup (i, j): values 16 i .. of histogram request ids[j], over its spans.
__global__ __launch_bounds__(kThreads) void k_hist_final_multi(const ReduceReq *__restrict__ reqs,
                                                               const int32_t *__restrict__ ids,
                                                               const uint32_t *__restrict__ sub) {
    const ReduceReq q = reqs[ids[blockIdx.y]];
    hist_final(sub + q.first * 256, (q.n + kHistSpan - 1) / kHistSpan, global_ptr<int64_t>(q.out));
}

}  // namespace red

int64_t reduce_parts(int op, int64_t n) {
    return op == PF_OP_SUM_F32 ? (n + red::kChunk - 1) / red::kChunk : (n + red::kHistSpan - 1) / red::kHistSpan;
}

hipError_t launch_reduce_batch(const ReduceReq *reqs, const int32_t *sum_ids, int nsum, const ReduceTask *sum_tasks,
                               int n_sum_tasks, const int32_t *hist_ids, int nhist, const ReduceTask *hist_tasks,
                               int n_hist_tasks, double *partial, uint32_t *sub, hipStream_t s) {
    hipError_t e = hipSuccess;
    if (nsum > 0) {
        const int grid = std::min(n_sum_tasks, red::kSumBlocks);
        hipLaunchKernelGGL(red::k_sum_partial_multi, dim3(grid), dim3(red::kThreads), 0, s, reqs, sum_tasks,
                           n_sum_tasks, partial);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(red::k_sum_final_multi, dim3(nsum), dim3(red::kThreads), 0, s, reqs, sum_ids, partial);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (nhist > 0) {
        const int grid = std::min(n_hist_tasks, red::kHistRows);
        hipLaunchKernelGGL(red::k_hist_partial_multi, dim3(grid), dim3(red::kHistThreads), 0, s, reqs, hist_tasks,
                           n_hist_tasks, sub);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(red::k_hist_final_multi, dim3(256 / red::kFinalBins, nhist), dim3(red::kThreads), 0, s, reqs, hist_ids, sub);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return e;
}

int64_t sum_chunks(int64_t n) { return (n + red::kChunk - 1) / red::kChunk; }

size_t sum_workspace_bytes(int64_t n) { return (size_t)sum_chunks(n) * sizeof(double); }

size_t hist_workspace_bytes(int64_t n) {
    const int64_t spans = (n + red::kHistSpan - 1) / red::kHistSpan;
    return (size_t)std::min<int64_t>(std::max<int64_t>(spans, 1), red::kHistRows) * 256 * sizeof(uint32_t);
}

// One workgroup per CU, fewer while each has less than a unit. From 2^37
// bytes up all 1024, so that no 32-bit count overflows (2^40 bytes at most).
int64_t hist_rows_wanted(int64_t n) {
    if (n >= ((int64_t)1 << 37)) return red::kHistRows;
    return std::min<int64_t>((n + red::kHistUnit - 1) / red::kHistUnit, std::min(std::max(dev_info().cus, 1), red::kHistRows));
}

// Scratch of pf_sum_f32_noalloc: the chunk partials of sums of up to
// kScratchChunks * kChunk elements, in a file-scope device array (64 KiB on
// each GPU the library runs on, held until the process ends). In host code
// `scratch` names a host-side stand-in, not device memory: host code uses
// only the per-device address that hipGetSymbolAddress returns.
constexpr int64_t kScratchChunks = 8192;
static __device__ __align__(256) double scratch[kScratchChunks];

int64_t sum_noalloc_max() { return kScratchChunks * red::kChunk; }

// The device address of `scratch` on the current device, looked up once per
// device with that device current.
hipError_t sum_scratch(void **ptr) {
    static std::mutex mu;
    static void *addr[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

hipError_t launch_sum(const float *x, int64_t n, double *out, void *workspace, hipStream_t s) {
    const int64_t nchunks = sum_chunks(n);
    if (nchunks == 1) {
        hipLaunchKernelGGL(red::k_sum_one, dim3(1), dim3(red::kThreads), 0, s, x, (int)n, out);
        return hipGetLastError();
    }
    double *partial = static_cast<double *>(workspace);
    const int grid = (int)std::min<int64_t>(nchunks, red::kSumBlocks);
    const bool stream = n >= ((int64_t)1 << 26);
    hipLaunchKernelGGL(stream ? red::k_sum_partial<true> : red::k_sum_partial<false>, dim3(grid), dim3(red::kThreads), 0,
                       s, x, n, partial, (int)nchunks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(red::k_sum_final, dim3(1), dim3(red::kThreads), 0, s, partial, nchunks, n, out);
    return hipGetLastError();
}

hipError_t launch_hist(const uint8_t *x, int64_t n, int64_t *hist, void *workspace, size_t workspace_bytes,
                       hipStream_t s) {
    const int64_t rows = std::min<int64_t>(hist_rows_wanted(n), workspace_bytes / (256 * sizeof(uint32_t)));
    if (n <= red::kHistUnit) {
        hipLaunchKernelGGL(red::k_hist_one, dim3(1), dim3(red::kHistThreads), 0, s, x, n, hist);
        return hipGetLastError();
    }
    uint32_t *sub = static_cast<uint32_t *>(workspace);
    hipLaunchKernelGGL(red::k_hist_partial, dim3((unsigned)rows), dim3(red::kHistThreads), 0, s, x, n, sub);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(red::k_hist_final, dim3(256 / red::kFinalBins), dim3(red::kThreads), 0, s, sub, (int)rows, hist);
    return hipGetLastError();
}

}  // namespace pf
