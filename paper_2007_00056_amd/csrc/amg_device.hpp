// Device-side helpers shared by the gfx950 kernels: wavefront and block
// reductions, XCD-aware block mapping.  Wavefronts are 64 lanes wide on CDNA4.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "amg_index.hpp"

namespace amg {

// Workgroups are dispatched round-robin over the XCDs (block b runs on XCD
// b % 8).  Remapping gives each XCD one contiguous range of logical blocks, so
// rows that share x-vector cache lines share one XCD's L2.
__device__ __forceinline__ int xcd_block(int b, int g) {
    const int xcd = b % kNumXcd, idx = b / kNumXcd;
    const int per = g / kNumXcd, rem = g % kNumXcd;
    return xcd * per + (xcd < rem ? xcd : rem) + idx;
}

// Butterfly sum over groups of W consecutive lanes (W a power of two <= 64);
// every lane of the group ends with the group total, in a fixed order.
template <int W>
__device__ __forceinline__ double group_sum(double s) {
#pragma unroll
    for (int off = W / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, W);
    return s;
}

template <int W>
__device__ __forceinline__ float group_sum(float s) {
#pragma unroll
    for (int off = W / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, W);
    return s;
}

// Deterministic block reduction of NV sums: block b writes its totals to
// part[k * gridDim.x + b].  A separate single-block kernel adds the partials
// in a fixed order (same-address device-scope atomics serialise across the
// XCDs, so no "last block" ticket is used).
template <int NV, int BS>
__device__ __forceinline__ void block_partials(double (&v)[NV], double* part) {
    static_assert(BS % kWave == 0, "block size must be whole waves");
    constexpr int NW = BS / kWave;
    __shared__ double sh[NV][NW];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const double s = group_sum<kWave>(v[k]);
        if (lane == 0) sh[k][wid] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            double s = sh[k][0];
            for (int w = 1; w < NW; ++w) s += sh[k][w];
            part[k * gridDim.x + blockIdx.x] = s;
        }
    }
}

// Sum of np block partials in a fixed order, formed by a whole block of BS
// threads and returned to every thread: lane sums over a stride of BS, the
// wave butterfly, then the waves in order.  Every block that calls it gets
// the same value, so a consumer kernel can finish a reduction itself.
template <int BS>
__device__ __forceinline__ double block_sum_partials(const double* __restrict__ part, int np) {
    static_assert(BS % kWave == 0, "block size must be whole waves");
    constexpr int NW = BS / kWave;
    __shared__ double sh[NW];
    __shared__ double tot;
    double s = 0.0;
    for (int b = threadIdx.x; b < np; b += BS) s += part[b];
    s = group_sum<kWave>(s);
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    if (lane == 0) sh[wid] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = sh[0];
        for (int w = 1; w < NW; ++w) t += sh[w];
        tot = t;
    }
    __syncthreads();
    return tot;
}

}  // namespace amg
