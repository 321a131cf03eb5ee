// The batched operator over problems of several degrees in one launch: a workgroup
// branches (uniformly) to its item's degree and shape.
//
// For batches whose launches leave compute units idle: a launch per degree then takes
// its few workgroups' latency each (served requests: 10 us at N = 11, 10 at 9, 3 to 5 at
// 7, 5 and 3, one after the other), while here they run side by side: 16 served requests
// 110 -> 90 ms, a batch of 16 problems 5.32 -> 4.52 ms per 50 iterations.  The registers
// are those of the most demanding degree (166: three waves per SIMD, one less than the
// operator has alone at N <= 5), the LDS that of the most demanding one in the list.
#pragma once

#include "ax_impl.h"

namespace hb {

template <typename T, bool MASK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void batch_any_kernel(
    const WorkItem *__restrict__ items, const BatchProb *__restrict__ probs)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char any_lds[];
    __shared__ double red[4];
    const WorkItem it = items[blockIdx.x];
    const int32_t prob = uniform(it.prob), tile = uniform(it.idx);
    const int32_t key = uniform(probs[prob].N) + 16 * uniform(probs[prob].variant);
    T *const lds = reinterpret_cast<T *>(any_lds);
    switch (key) {
// (waves that a degree's shape does not have end here, before its first barrier)
#define HB_ANY(n, v)                                                  \
    case n + 16 * v:                                                  \
        if (threadIdx.x >= Shape<n, v>::threads) return;              \
        return batch_item<n, v, T, MASK>(lds, red, prob, tile, probs);
        HB_ANY(1, 0) HB_ANY(2, 0) HB_ANY(3, 0) HB_ANY(4, 0) HB_ANY(5, 0) HB_ANY(6, 0) HB_ANY(7, 0) HB_ANY(8, 0)
        HB_ANY(9, 0) HB_ANY(10, 0) HB_ANY(11, 0) HB_ANY(12, 0) HB_ANY(13, 0) HB_ANY(14, 0) HB_ANY(15, 0)
        HB_ANY(1, 1) HB_ANY(2, 1) HB_ANY(3, 1) HB_ANY(4, 1) HB_ANY(5, 1) HB_ANY(6, 1) HB_ANY(7, 1)
#undef HB_ANY
    }
}

template <typename T, bool MASK>
hb_status launch_batch_any(const WorkItem *items, int nitems, size_t lds, const BatchProb *probs, hipStream_t s)
{
    batch_any_kernel<T, MASK><<<nitems, 256, lds, s>>>(items, probs);
    HB_HIP(hipGetLastError());
    return HB_OK;
}

}  // namespace hb
