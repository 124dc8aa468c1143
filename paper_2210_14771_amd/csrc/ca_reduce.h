// Column sums of the gradient partials (device code shared by both scorers).
#pragma once

#include "ca_cnn.h"

namespace ca {

constexpr int kReduceThreads = 1024;
constexpr int kReduceCols = 64;   // columns one workgroup sums

// Sums columns [kReduceCols b, kReduceCols (b + 1)) of partial[rows][stride]
// (b: the workgroup) into sums, by kReduceThreads threads; ends with a
// barrier.  stride: a multiple of kReduceCols.  The order is fixed (thread
// rows t, t + 64, ..; then the four rows of a wave; then the waves), so equal
// partials give equal sums.
//
// Bound by memory latency: the partials are 13-26 MB written just before,
// read once.  A wave reads four rows of 256 bytes at a time with eight such
// loads in flight, 16 waves a workgroup: one thread a column walking all 512
// rows (51 and 25 workgroups) took 120 us for the 1-D scorer's 26 MB and
// 379 us for the 2-D scorer's.
__device__ __forceinline__ void column_sums(const float *partial, int rows, int stride,
                                            float *sums)
{
    __shared__ float4 s_wave[kReduceThreads / 64][kReduceCols / 4];
    constexpr int kRows = kReduceThreads * 4 / kReduceCols;   // rows in one sweep
    constexpr int kDeep = 8;
    const int c4 = threadIdx.x & (kReduceCols / 4 - 1);
    const int r0 = threadIdx.x / (kReduceCols / 4);
    const float *p = partial + (int64_t)blockIdx.x * kReduceCols + 4 * c4;
    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int base = r0; base < rows; base += kRows * kDeep) {
        float4 q[kDeep];
#pragma unroll
        for (int k = 0; k < kDeep; ++k) {
            const int r = base + k * kRows;
            q[k] = r < rows ? *reinterpret_cast<const float4 *>(p + (int64_t)r * stride)
                            : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
#pragma unroll
        for (int k = 0; k < kDeep; ++k) {
            v.x += q[k].x;
            v.y += q[k].y;
            v.z += q[k].z;
            v.w += q[k].w;
        }
    }
#pragma unroll
    for (int d = 16; d < 64; d *= 2) {
        v.x += __shfl_xor(v.x, d, 64);
        v.y += __shfl_xor(v.y, d, 64);
        v.z += __shfl_xor(v.z, d, 64);
        v.w += __shfl_xor(v.w, d, 64);
    }
    if ((threadIdx.x & 63) < kReduceCols / 4)
        s_wave[threadIdx.x >> 6][c4] = v;
    __syncthreads();
    if (threadIdx.x < kReduceCols) {
        const float *w = reinterpret_cast<const float *>(&s_wave[0][0]) + threadIdx.x;
        float t = 0.0f;
#pragma unroll
        for (int k = 0; k < kReduceThreads / 64; ++k)
            t += w[k * kReduceCols];
        sums[threadIdx.x] = t;
    }
    __syncthreads();
}

}  // namespace ca
