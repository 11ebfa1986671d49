// Small HBM-bound kernels around the attention kernel:
//   - per-head mean squared error between two attention outputs (the loss of the paper's mask-search
//     algorithm, "STA Mask Search": loss <- MSE(O, O')),
//   - first-minimum selection over a list of patterns per head (same algorithm: keep the pattern whose
//     loss is strictly smaller than the best so far), done where the last pattern's losses are finished,
//   - attention recall from two log-denominators (Sec. 1: fraction of the attention score that falls
//     inside a local window).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "sta_internal.h"

namespace {

constexpr int kThreads = 256;

// Partial sums of the allocation-free per-head MSE entry point: kMseSlices doubles per (batch, head) slab, for
// at most kStaticMseMaxSlabs slabs (512 KB).  Every GPU the library runs on holds its own copy at its own
// address until the process ends.  In host code this name is only a handle for hipGetSymbolAddress; kernels
// receive the device address that call returns.
static __device__ __align__(256) double scratch[sta::kStaticMseMaxSlabs * sta::kMseSlices];
constexpr int kMaxDevices = 64;

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Sum over a workgroup of one double per thread; result valid in thread 0.
__device__ __forceinline__ double block_sum(double x)
{
    __shared__ double part[kThreads / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
#pragma unroll
        for (int i = 0; i < kThreads / 64; ++i) s += part[i];
    return s;
}

// grid = (slices, B*H).  Slice s of slice count S sums the squared differences of 16-byte chunks
// s, s+S, s+2S, ... of one (b,h) slab and writes one double.  chunks = N*D/8 per slab.
__global__ __launch_bounds__(kThreads) void sta_sq_diff_partial_kernel(const uint4 *__restrict__ a,
                                                                       const uint4 *__restrict__ b, size_t chunks,
                                                                       double *__restrict__ partial)
{
    const size_t slab = (size_t)blockIdx.y * chunks;
    const size_t stride = (size_t)gridDim.x * kThreads;
    float acc0 = 0.f, acc1 = 0.f;
    for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < chunks; i += stride) {
        const uint4 x = a[slab + i], y = b[slab + i];
        const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float d0 = bf16_lo(xs[e]) - bf16_lo(ys[e]);
            const float d1 = bf16_hi(xs[e]) - bf16_hi(ys[e]);
            acc0 = fmaf(d0, d0, acc0);
            acc1 = fmaf(d1, d1, acc1);
        }
    }
    const double s = block_sum((double)acc0 + (double)acc1);
    if (threadIdx.x == 0) partial[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
}

// One wave per head: lane i sums slice i of every batch entry (consecutive lanes read consecutive doubles), then the lanes are
// summed in a fixed tree and the sum is divided by the element count.  What bounds it is the latency of its loads.  (One thread
// per head before, B * 64 dependent additions: 24 heads 6.8 us, 19 x 9 slabs 94.)
// best (the last pattern of a list): also the index of the first pattern with the smallest loss, among this one and the
// n_before patterns whose losses stand before it, [n_before][H]; lane i takes the patterns i, i + 64, ..
// (A launch of its own before: 4.5 us.)
static_assert(sta::kMseSlices == 64, "one slice per lane");
__global__ __launch_bounds__(64) void sta_mse_finish_kernel(const double *__restrict__ partial, int B, int H, double inv_count,
                                                            float *mse_per_head, int n_before, int32_t *__restrict__ best)
{
    const int h = blockIdx.x, lane = threadIdx.x;
    double s = 0.0;
#pragma unroll 4
    for (int b = 0; b < B; ++b) s += partial[((size_t)b * H + h) * sta::kMseSlices + lane];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    const float loss = (float)(s * inv_count);
    if (lane == 0) mse_per_head[h] = loss;
    if (best == nullptr) return;
    const float *before = mse_per_head - (size_t)n_before * H + h;
    float minimum = INFINITY;
    int arg = -1;
    for (int p = lane; p <= n_before; p += 64) {
        const float x = p < n_before ? before[(size_t)p * H] : loss;
        if (x < minimum) {
            minimum = x;
            arg = p;
        }
    }
    // the smaller loss, of equal ones the earlier; an arg of -1 (as an unsigned number) comes behind every other
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const float x = __shfl_xor(minimum, off);
        const int a = __shfl_xor(arg, off);
        if (x < minimum || (x == minimum && (uint32_t)a < (uint32_t)arg)) {
            minimum = x;
            arg = a;
        }
    }
    if (lane == 0) best[h] = arg;
}

// grid = (slices, B*H).  recall_i = exp(lse_window_i - lse_full_i); optional per-query output; one partial sum
// per workgroup.
__global__ __launch_bounds__(kThreads) void sta_recall_partial_kernel(const float *__restrict__ lse_window,
                                                                      const float *__restrict__ lse_full, size_t N,
                                                                      float *__restrict__ recall,
                                                                      double *__restrict__ partial)
{
    const size_t base = (size_t)blockIdx.y * N;
    const size_t stride = (size_t)gridDim.x * kThreads;
    float acc = 0.f;
    for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < N; i += stride) {
        const float r = __expf(lse_window[base + i] - lse_full[base + i]);
        if (recall) recall[base + i] = r;
        acc += r;
    }
    const double s = block_sum((double)acc);
    if (threadIdx.x == 0) partial[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
}

// One wave per (batch, head): sum of the slices, one per lane, in a fixed tree.
__global__ __launch_bounds__(64) void sta_recall_finish_kernel(const double *__restrict__ partial, double inv_n,
                                                               float *__restrict__ mean_bh)
{
    double s = partial[(size_t)blockIdx.x * sta::kMseSlices + threadIdx.x];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (threadIdx.x == 0) mean_bh[blockIdx.x] = (float)(s * inv_n);
}

}  // namespace

namespace sta {

hipError_t launch_head_mse(const void *a, const void *b, int B, int H, size_t elems_per_head, double *partial,
                           float *mse_per_head, int n_before, int32_t *best, hipStream_t stream)
{
    const size_t chunks = elems_per_head / 8;
    dim3 grid(kMseSlices, (uint32_t)B * H), block(kThreads);
    const hipError_t e = launch_kernel(sta_sq_diff_partial_kernel, grid, block, stream, static_cast<const uint4 *>(a),
                                       static_cast<const uint4 *>(b), chunks, partial);
    if (e != hipSuccess) return e;
    return launch_kernel(sta_mse_finish_kernel, dim3(H), dim3(64), stream, partial, B, H, 1.0 / ((double)B * (double)elems_per_head),
                         mse_per_head, n_before, best);
}

hipError_t static_mse_scratch(double **out)
{
    static std::mutex mu;
    static double *per_device[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (per_device[dev] == nullptr) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (ptr == nullptr) return hipErrorInvalidSymbol;
        per_device[dev] = static_cast<double *>(ptr);
    }
    *out = per_device[dev];
    return hipSuccess;
}

hipError_t launch_recall(const float *lse_window, const float *lse_full, int BH, size_t N, float *recall, double *partial,
                         float *mean_bh, hipStream_t stream)
{
    const hipError_t e = launch_kernel(sta_recall_partial_kernel, dim3(kMseSlices, BH), dim3(kThreads), stream, lse_window, lse_full, N, recall, partial);
    if (e != hipSuccess) return e;
    return launch_kernel(sta_recall_finish_kernel, dim3(BH), dim3(64), stream, partial, 1.0 / (double)N, mean_bh);
}

}  // namespace sta
