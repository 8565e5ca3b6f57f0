// What the kernels that hold models on chip over several steps share: the barrier in device memory
// among the workgroups of a launch, and the averaging step's arithmetic for one entry.  Internal
// linkage: every translation unit gets its own copy.
#pragma once
#include "lc_internal.h"

namespace lc {
namespace {

// Barrier among the workgroups that add to *ctr, called by one thread per workgroup after a
// workgroup barrier: what the workgroup wrote before is visible to every workgroup that leaves
// the wait.  The wait is bounded; a workgroup that runs out of polls raises the error flag and
// never waits again (it still arrives, so the counts stay right), so the grid always drains.
__device__ __forceinline__ void arrive_and_wait(unsigned* ctr, unsigned target, int spin_limit, unsigned* err,
                                                bool& gave_up) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int polls = 0;
    while (!gave_up) {
        if (polls++ >= spin_limit) {   // a limit of 0 gives up without looking: the host's way to force this path
            gave_up = true;
            atomicOr(err, 1u);
            break;
        }
        const unsigned seen = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (static_cast<int>(seen - target) >= 0) break;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// x_bar = (1/m) sum_i x^(i) of one entry (Sec. 2, the averaging step), summed in double in
// replica order and rounded once: the same arithmetic, bit for bit, as the averaging kernels.
__device__ __forceinline__ float mean_of_replicas(const float* p, int64_t stride, int G) {
    double s = 0.0;
    for (int i0 = 0; i0 < G; i0 += 4) {   // four loads in flight, added in replica order
        float r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i0 + u < G) r[u] = p[(i0 + u) * stride];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i0 + u < G) s += static_cast<double>(r[u]);
    }
    return static_cast<float>(s / static_cast<double>(G));
}

}  // namespace
}  // namespace lc
