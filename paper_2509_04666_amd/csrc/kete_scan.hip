// Exclusive prefix sums of int32 counts: tile sums, then tile scans whose
// blocks add up the sums before their tile themselves (from kMaxOwnTiles tiles
// on a pass of one block between the two scans the sums); one block does it
// all where that is quicker than a second launch.
#include "kete_internal.hpp"

namespace kete {
namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 4;
constexpr int kTile = kScanThreads * kScanItems;
// A block reads at most four sums a thread; more of them are scanned once.
constexpr int64_t kMaxOwnTiles = 4 * kScanThreads;

// Inclusive scan of one value per thread over a 256-thread block.
__device__ __forceinline__ int block_inclusive(int v, int* sh) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        int u = __shfl_up(v, off, 64);
        if (lane >= off) v += u;
    }
    if (lane == 63) sh[wid] = v;
    __syncthreads();
    int add = 0;
    for (int w = 0; w < wid; ++w) add += sh[w];
    __syncthreads();
    return v + add;
}

__global__ __launch_bounds__(kScanThreads) void k_tile_sums(const int32_t* __restrict__ in, int64_t n,
                                                          int32_t* __restrict__ part) {
    __shared__ int sh[4];
    const int64_t base = (int64_t)blockIdx.x * kTile + threadIdx.x * kScanItems;
    int s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) if (base + k < n) s += in[base + k];
    s = block_inclusive(s, sh);
    if (threadIdx.x == kScanThreads - 1) part[blockIdx.x] = s;
}

// One block of 1024 threads scans a short array, kScanItems values a thread
// at a time: two rounds of it take no longer than one of the two passes, 5 us,
// most of which is the launch.
constexpr int kOneThreads = 1024;
constexpr int kOneRounds = 2;
constexpr int64_t kOneBlock = (int64_t)kOneRounds * kOneThreads * kScanItems;
__global__ __launch_bounds__(kOneThreads) void k_scan_short(const int32_t* in, int64_t n, int32_t* out) {
    __shared__ int sh[kOneThreads / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int carry = 0;
    for (int64_t base = 0; base < n; base += kOneThreads * kScanItems) {
        const int64_t i = base + (int64_t)threadIdx.x * kScanItems;
        int v[kScanItems], s = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) { v[k] = i + k < n ? in[i + k] : 0; s += v[k]; }
        int inc = s;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int u = __shfl_up(inc, off, 64);
            if (lane >= off) inc += u;
        }
        if (lane == 63) sh[wid] = inc;
        __syncthreads();
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < kOneThreads / 64; ++w) {
            before += w < wid ? sh[w] : 0;
            all += sh[w];
        }
        int run = carry + before + inc - s;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            if (i + k < n) out[i + k] = run;
            run += v[k];
        }
        carry += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) out[n] = carry;
}

// One block scans all tile sums (exclusive), carrying a running total.
__global__ __launch_bounds__(kScanThreads) void k_scan_parts(int32_t* __restrict__ part, int64_t np,
                                                           int32_t* __restrict__ total) {
    __shared__ int sh[4];
    __shared__ int carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < np; base += kScanThreads) {
        const int64_t i = base + threadIdx.x;
        const int v = i < np ? part[i] : 0;
        const int inc = block_inclusive(v, sh);
        const int c = carry;
        if (i < np) part[i] = c + inc - v;
        __syncthreads();
        if (threadIdx.x == kScanThreads - 1) carry = c + inc;
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

// With kOwn the tile sums are as k_tile_sums left them.
template <bool kOwn>
__global__ __launch_bounds__(kScanThreads) void k_tile_scan(const int32_t* __restrict__ in, int64_t n,
                                                          const int32_t* __restrict__ part,
                                                          int32_t* __restrict__ out) {
    __shared__ int sh[4];
    int first = 0;
    if constexpr (kOwn) {
        int s = 0;
        for (int64_t i = threadIdx.x; i < (int64_t)blockIdx.x; i += kScanThreads) s += part[i];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
        __syncthreads();
        first = sh[0] + sh[1] + sh[2] + sh[3];
        __syncthreads();
    } else {
        first = part[blockIdx.x];
    }
    const int64_t base = (int64_t)blockIdx.x * kTile + threadIdx.x * kScanItems;
    int v[kScanItems];
    int s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) { v[k] = (base + k < n) ? in[base + k] : 0; s += v[k]; }
    const int inc = block_inclusive(s, sh);
    int run = first + inc - s;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) out[base + k] = run;
        run += v[k];
    }
    if (kOwn && blockIdx.x == gridDim.x - 1 && threadIdx.x == kScanThreads - 1) out[n] = run;
}

}  // namespace

size_t scan_scratch_bytes(int64_t n) {
    const int64_t np = (n + kTile - 1) / kTile;
    return (size_t)(np + 64) * sizeof(int32_t);
}

// out[0..n) = exclusive prefix sums of in, out[n] = total.  `in` may alias `out`.
hipError_t exclusive_scan_i32(const int32_t* in, int32_t* out, int64_t n, void* scratch, hipStream_t s) {
    int32_t* part = (int32_t*)scratch;
    const int64_t np = (n + kTile - 1) / kTile;
    if (n <= kOneBlock) {
        hipLaunchKernelGGL(k_scan_short, dim3(1), dim3(kOneThreads), 0, s, in, n, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_tile_sums, dim3((unsigned)np), dim3(kScanThreads), 0, s, in, n, part);
    if (np <= kMaxOwnTiles) {
        hipLaunchKernelGGL(k_tile_scan<true>, dim3((unsigned)np), dim3(kScanThreads), 0, s, in, n,
                           (const int32_t*)part, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_scan_parts, dim3(1), dim3(kScanThreads), 0, s, part, np, out + n);
    hipLaunchKernelGGL(k_tile_scan<false>, dim3((unsigned)np), dim3(kScanThreads), 0, s, in, n, (const int32_t*)part,
                       out);
    return hipGetLastError();
}

}  // namespace kete
