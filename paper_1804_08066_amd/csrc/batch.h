// Several tensors in one launch: which of them a workgroup belongs to.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.h"

namespace mqg {

// k with starts[k] <= block < starts[k + 1]; starts[0 .. count): the tensors' first workgroups, in kernel-argument memory and
// not decreasing (an empty tensor starts where the next one does).  One load by all lanes and a count of the starts passed: a
// binary search is a chain of scalar loads, each of which waits for the one before it -- about 0.2 us a step where the
// arguments are cold, which they are in every launch.
// Call with every lane of the wave active.
template <uint32_t ENTRIES>
__device__ __forceinline__ uint32_t tensor_of_block(const uint32_t (&starts)[ENTRIES], const uint32_t count, const uint32_t block) {
    static_assert(ENTRIES <= 64, "one lane per tensor");
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t start = starts[lane < ENTRIES ? lane : ENTRIES - 1u];
    const uint64_t passed = __builtin_amdgcn_ballot_w64(lane < count && start <= block);
    return (uint32_t)__builtin_popcountll(passed) - 1u;   // starts[0] is 0: at least one
}

}  // namespace mqg
