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

// x moved across the lanes of a wave by a DPP control (both halves of the
// double); lanes without a source keep `keep`.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move(double x, double keep)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(keep), __double2loint(x), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(keep), __double2hiint(x), CTRL, ROWS, 0xf, false);
    return __hiloint2double(hi, lo);
}

// Lane 63's value in every lane.
__device__ __forceinline__ double last_lane(double x)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 63),
                            __builtin_amdgcn_readlane(__double2loint(x), 63));
}

// Sum over the 64 lanes of a wave in a fixed order, in every lane: shifts by 1,
// 2, 4, 8 within the rows of 16 lanes, then row ends carried on (register
// moves; the same through LDS permutes took 2.4 us for nine sums at the end of a
// block, where nothing hides their latency).
__device__ __forceinline__ double wave_sum(double x)
{
    x += dpp_move<0x111, 0xf>(x, 0.0);
    x += dpp_move<0x112, 0xf>(x, 0.0);
    x += dpp_move<0x114, 0xf>(x, 0.0);
    x += dpp_move<0x118, 0xf>(x, 0.0);
    x += dpp_move<0x142, 0xa>(x, 0.0);
    x += dpp_move<0x143, 0xc>(x, 0.0);
    return last_lane(x);
}

// Smallest and largest over the 64 lanes, in every lane.
__device__ __forceinline__ double wave_min(double x)
{
    x = fmin(x, dpp_move<0x111, 0xf>(x, x));
    x = fmin(x, dpp_move<0x112, 0xf>(x, x));
    x = fmin(x, dpp_move<0x114, 0xf>(x, x));
    x = fmin(x, dpp_move<0x118, 0xf>(x, x));
    x = fmin(x, dpp_move<0x142, 0xa>(x, x));
    x = fmin(x, dpp_move<0x143, 0xc>(x, x));
    return last_lane(x);
}
__device__ __forceinline__ double wave_max(double x) { return -wave_min(-x); }

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
