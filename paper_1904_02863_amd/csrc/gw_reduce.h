// Fixed-order block and wave reductions shared by the likelihood kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "gw_internal.h"

namespace gw {

// Fixed-order tree sum of x over the block; every thread gets the total.
// `red` is kBlock doubles of LDS.  All threads must call it.
__device__ __forceinline__ double block_sum(double x, double *red)
{
    red[threadIdx.x] = x;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    const double total = red[0];
    __syncthreads();
    return total;
}

// Sum over the 64 lanes of a wave by a fixed butterfly (lane 0's value is
// the one used).
__device__ __forceinline__ double wave_sum(double x)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

// Column j of an event's per-block partials summed over its n_blocks blocks
// (strided per thread, then a fixed tree): the event-wide sum of quantity j.
__device__ __forceinline__ double column_total(int n_blocks, int per, int j, const double *__restrict__ partials,
                                               double *red)
{
    double x = 0.0;
    for (int b = threadIdx.x; b < n_blocks; b += kBlock) x += partials[(int64_t)b * per + j];
    return block_sum(x, red);
}

}  // namespace gw
