// Block reductions for the fused dot products of the CG iteration.  Each block
// writes one partial; a single-block kernel sums the partials in a fixed
// order, so every dot product is reproducible run to run.  (No block waits for
// another and no device-scope fence is issued inside a streaming kernel.)
#pragma once

#include <hip/hip_runtime.h>

namespace hb {

// v + (v of another lane, as the DPP control selects; 0 where it selects none).
template <int CTRL>
__device__ inline double add_dpp(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u), CTRL, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), CTRL, 0xf, 0xf, true);
    return v + __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

// Sum over a wave64, in every lane: by data-parallel moves within rows of 16
// lanes and from row to row (register operations; exchanges through LDS took
// most of a small kernel's reduction time), read back from the last lane.
__device__ inline double wave_sum(double v)
{
    v = add_dpp<0x111>(v);  // row_shr:1
    v = add_dpp<0x112>(v);  // row_shr:2
    v = add_dpp<0x114>(v);  // row_shr:4
    v = add_dpp<0x118>(v);  // row_shr:8: lane 15 of each row holds the row's sum
    v = add_dpp<0x142>(v);  // row_bcast:15: lanes 31 and 63 hold the sums of two rows
    v = add_dpp<0x143>(v);  // row_bcast:31: lane 63 holds the sum
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(u), 63);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(u >> 32), 63);
    return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

// Sum over the whole block (all threads must call it); result valid in every thread.
// `scratch` needs blockDim.x / 64 doubles of shared memory.
__device__ inline double block_sum(double v, double *scratch)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = (blockDim.x + 63) >> 6;
    v = wave_sum(v);
    __syncthreads();  // scratch may still be in use by a previous call
    if (lane == 0) scratch[wave] = v;
    __syncthreads();
    double s = 0.0;
    for (int i = 0; i < nwaves; ++i) s += scratch[i];
    return s;
}

// Workgroups are dispatched to the 8 XCDs of the device in turn (id mod 8).
// Give each XCD a contiguous range of tiles so that tiles sharing data
// (neighbouring elements) are served by the same L2.  A bijection on [0, n).
__host__ __device__ inline int xcd_remap(int bid, int n)
{
    constexpr int X = 8;
    const int per = n / X, rem = n % X;
    const int xcd = bid % X, k = bid / X;
    return xcd * per + (xcd < rem ? xcd : rem) + k;
}

}  // namespace hb
