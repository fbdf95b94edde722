// Several tensors in one launch: which of them a workgroup belongs to; and how a whole tensor's range travels from one launch
// to the next.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "encode.h"
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

// Slots of a whole-tensor range (RangeSlots): first element of tile `tile` of `tiles`, the end of that tile, and its slot.
__device__ __forceinline__ uint64_t slot_tile_base(uint32_t tile, uint32_t tiles, uint32_t borrowed) {
    return (uint64_t)tile * kSlotTile - (tile + 1u == tiles ? borrowed : 0u);
}
__device__ __forceinline__ uint64_t slot_tile_end(uint32_t tile, uint32_t tiles, uint32_t borrowed, uint64_t n) {
    return tile + 1u == tiles ? n : slot_tile_base(tile + 1u, tiles, borrowed);
}
// Finder `part` leaves its keys (in thread 0) in every slot.  All lanes of the workgroup; s_keys: two words of LDS.
__device__ __forceinline__ void keys_to_slots(uint32_t* packed, uint64_t n, uint32_t bits, uint32_t borrowed, uint32_t part, uint32_t kl,
                                              uint32_t kh, uint32_t* s_keys) {
    if (threadIdx.x == 0u) {
        s_keys[0] = kl;
        s_keys[1] = kh;
    }
    __syncthreads();
    kl = s_keys[0];
    kh = s_keys[1];
    const uint32_t tiles = (uint32_t)((n + kSlotTile - 1u) / kSlotTile);
    for (uint32_t i = threadIdx.x; i < tiles; i += blockDim.x) {
        uint32_t* slot = packed + (slot_tile_base(i, tiles, borrowed) >> 5) * bits + 2u * part;
        slot[0] = kl;
        slot[1] = kh;
    }
}
// The range from a slot's keys; every wave by itself, all its lanes active.  A barrier must lie between this and the first
// code word that the workgroup stores.
__device__ __forceinline__ float2 range_from_slot(const uint32_t* slot, uint32_t parts) {
    uint32_t kl = 0xFFFFFFFFu, kh = 0u;
    const uint32_t lane = threadIdx.x & 63u;
    for (uint32_t i = lane; i < parts; i += 64u) {
        kl = min(kl, slot[2u * i]);
        kh = max(kh, slot[2u * i + 1u]);
    }
    return encode::range_of_keys(encode::wave_min_from_cells_u32(encode::cell_min_u32(kl), lane),
                                 encode::wave_max_from_cells_u32(encode::cell_max_u32(kh), lane));
}

}  // namespace mqg
