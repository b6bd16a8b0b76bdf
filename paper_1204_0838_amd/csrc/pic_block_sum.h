// Two-stage reductions of the diagnostics: each of at most kSumBlocks
// workgroups sums its share into one row of partials, and one workgroup then
// combines the rows in a fixed order.  One FP64 atomic per wavefront onto a
// few shared words (the earlier form) serialises on them: of 7.7e6 particles
// and 1.9e6 cells, particle sums 417 -> 42 us (20 B per particle: 3.7 TB/s),
// field sums 205 -> 18 us, all diagnostics of an output step 3.67 -> 0.31 ms
// of kernel time.
#pragma once

#include "pic_internal.h"

namespace pic {

constexpr int kSumThreads = 1024;   // 16 wavefronts: one workgroup fills a CU's queue of loads
constexpr int kSumBlocks = 256;     // one per CU; kSumBlocks x K partials fit the diagnostics' 4096 words (K <= 16)

inline int sum_blocks(int64_t n) {
    const int64_t b = (n + kSumThreads - 1) / kSumThreads;
    return (int)(b < 1 ? 1 : (b > kSumBlocks ? kSumBlocks : b));
}

// Words [0, NSUM) of v are summed over the workgroup, words [NSUM, K) take the
// maximum (of values >= 0); the results go to part[blockIdx.x K ..].
template <int NSUM, int K>
__device__ __forceinline__ void block_partials(double (&v)[K], double* __restrict__ part) {
    __shared__ double ws[kSumThreads / 64][K];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double y = __shfl_xor(v[k], o, 64);
            v[k] = k < NSUM ? v[k] + y : fmax(v[k], y);
        }
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < K; ++k) ws[threadIdx.x >> 6][k] = v[k];
    __syncthreads();
    if ((int)threadIdx.x < K) {
        double s = ws[0][threadIdx.x];
        for (int w = 1; w < (int)blockDim.x / 64; ++w) {
            const double y = ws[w][threadIdx.x];
            s = (int)threadIdx.x < NSUM ? s + y : fmax(s, y);
        }
        part[(size_t)blockIdx.x * K + threadIdx.x] = s;
    }
}

// Combine the rows of part (one workgroup of 64 K threads: wavefront k takes
// word k) and hand each result to f(k, value) on one lane.
template <int NSUM, int K, class F>
__device__ __forceinline__ void combine_partials(const double* __restrict__ part, int nb, F f) {
    const int k = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double s = 0.0;
    for (int b = lane; b < nb; b += 64) {
        const double y = part[(size_t)b * K + k];
        s = k < NSUM ? s + y : fmax(s, y);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double y = __shfl_xor(s, o, 64);
        s = k < NSUM ? s + y : fmax(s, y);
    }
    if (lane == 0) f(k, s);
}

}  // namespace pic
