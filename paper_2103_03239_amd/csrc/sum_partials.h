// The sum of a list of binary64 partial sums by one block, for gfx950 (the last step of a distortion).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moshpit {

constexpr int kSumThreads = 1024;        // at most

// Threads for a list of `count`: one value each as far as they go.
inline uint32_t sum_threads(int64_t count)
{
    return static_cast<uint32_t>(count < kSumThreads ? (count + 63) / 64 * 64 : kSumThreads);
}

// Thread 0 gets the sum; its order depends on `count` and the block's size alone.  A thread requests eight
// values before it adds the first: one block is bound by the latency of its loads (4096 values in steps of 256, each load
// behind the addition before it: 18 us; so: 5).
__device__ __forceinline__ double block_sum(const double *__restrict__ values, int64_t count)
{
    __shared__ double wave_sums[kSumThreads / 64];
    const int32_t step = blockDim.x;
    double acc = 0.0;
    for (int64_t k0 = threadIdx.x; k0 < count; k0 += 8 * step) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t k = k0 + u * step;
            v[u] = values[k < count ? k : 0];
            if (k >= count) v[u] = 0.0;
        }
        acc += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if ((threadIdx.x & 63) == 0) wave_sums[threadIdx.x >> 6] = acc;
    __syncthreads();
    double sum = 0.0;
    if (threadIdx.x == 0)
        for (int32_t w = 0; w < step >> 6; ++w) sum += wave_sums[w];
    return sum;
}

}  // namespace moshpit
