// Internal launch interface between the C-ABI layer (api.hip) and the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mqgrad.h"

namespace mqg {

struct QuantizeArgs {
    const float* grad;       // n floats
    uint64_t n;
    uint32_t bits;           // 1..8
    uint32_t bucket;         // multiple of 32, 32..16384
    int bucket_shift;        // log2(bucket) when bucket is a power of two, else -1
    int scale_mode;          // mqg_scale_mode
    uint32_t key0, key1;     // Philox key = seed
    uint32_t iteration, worker;
    uint64_t elem_base;      // multiple of 8
    const float* scales_in;  // nullable: when set, scales are read, not computed ([min, max] encoding: ONE
                             // (min, max) pair that holds for the whole tensor)
    uint32_t* packed;        // ceil(n*bits/32) words
    float* scales;           // ceil(n/bucket) floats
    uint32_t drop_nan = 0;       // [min, max] ranges: 1: a NaN takes no part, also where a lane holds nothing else (whole-tensor ranges)
    uint32_t stream_codes = 0;   // 1: the code words are stored with the streaming hint instead of agent scope
    uint32_t parts = 0;          // whole-tensor [min, max] ranges that travel in slots (RangeSlots below); scales receives the range
    uint32_t borrowed = 0;
};

// A whole-tensor range found by `parts` workgroups and used by the workgroups of the next launch, one per tile of kSlotTile
// elements: every finder leaves its pair of keys at the front of EVERY user's own code words, and a user folds the pairs it
// finds there before it overwrites them.  No launch in between folds them for all (2 us and 3 us of the caller's time), and
// no memory is needed but the output's.  parts * tiles pairs are written, so this is for small tensors.
constexpr uint32_t kSlotTile = 4096;
struct RangeSlots {
    uint32_t parts;      // 0: does not fit
    uint32_t borrowed;   // elements that the last tile takes from the one before it, so that its words hold the pairs too
};
inline RangeSlots range_slots(uint64_t n, uint32_t bits, uint64_t parts) {
    constexpr uint64_t kMostParts = 128;
    const uint64_t most = 32u * bits < kMostParts ? 32u * bits : kMostParts;   // two tiles' pairs in one tile's words
    if (parts < 2u || parts > most || n <= kSlotTile) return {0u, 0u};
    const uint32_t need = ((64u * (uint32_t)parts + bits - 1u) / bits + 31u) / 32u * 32u;   // elements whose words hold them: at most half a tile
    const uint32_t tail = (uint32_t)((n - 1u) % kSlotTile) + 1u;
    return {(uint32_t)parts, tail >= need ? 0u : (need - tail + 31u) / 32u * 32u};
}

struct AggregateArgs {
    const uint32_t* packed[MQG_MAX_WORKERS];
    const float* scales[MQG_MAX_WORKERS];
    uint32_t W;
    uint64_t n;
    uint32_t bits;
    uint32_t bucket;
    int bucket_shift;
    float neg_c;             // -(lr / W)
    float* params;
    uint32_t per_tensor;     // [min, max] encoding only: every worker has ONE (min, max) pair for the whole tensor
    uint32_t stream_codes;   // the code words are not in this GPU's caches: streaming loads at every width
};

// Server side of the full exchange: quantize the sum over W workers' de-quantized gradients
// (q.grad, q.scales_in unused); the stored bucket range is divided by W.
struct RequantArgs {
    QuantizeArgs q;
    const uint32_t* packed[MQG_MAX_WORKERS];
    const float* scales[MQG_MAX_WORKERS];
    uint32_t W;
};

// Several layer tensors of one model in one launch.  A launch's arguments are copied for every launch, at about 0.45 us of
// the caller's time per KB, so a batch that fits takes the form with room for few (with_few below): the small CNN's two
// launches carry 1.9 KB instead of 4.8.
constexpr uint32_t kMaxBatchTensors = 32, kFewTensors = 12, kFewRanges = 4;   // kFewRanges: one tensor, or the paper's two layers
constexpr uint32_t kMaxBatchPointers = 256, kFewPointers = 96;   // per quantized tensor 2*W pointers, per raw tensor W

struct AggregateTensor {
    uint64_t n;
    float* params;
    uint32_t first_ptr;   // index into ptrs: [W packed][W scales], or [W raw gradients]
    uint32_t raw;         // 1: uncompressed layer
};
struct AggregateBatchHead {
    uint32_t count, W, bits, bucket;
    int bucket_shift;
    float neg_c;
    uint32_t per_tensor;      // [min, max] encoding only: ONE (min, max) pair per worker and tensor
    uint32_t pointers;        // used entries of ptrs
};
template <uint32_t TENSORS, uint32_t POINTERS>
struct AggregateBatch : AggregateBatchHead {
    using Tensor = AggregateTensor;
    using Few = AggregateBatch<kFewTensors, kFewPointers>;
    uint32_t tile_start[TENSORS + 1];   // prefix sums of the tensors' tile counts
    Tensor t[TENSORS];
    const void* ptrs[POINTERS];
    bool few() const { return count <= kFewTensors && pointers <= kFewPointers; }
    void copy_to(Few& f) const {
        static_cast<AggregateBatchHead&>(f) = *this;
        for (uint32_t i = 0; i < kFewTensors; ++i) f.t[i] = t[i];
        for (uint32_t i = 0; i <= kFewTensors; ++i) f.tile_start[i] = tile_start[i];
        for (uint32_t i = 0; i < pointers; ++i) f.ptrs[i] = ptrs[i];
    }
};
using BatchAggregateArgs = AggregateBatch<kMaxBatchTensors, kMaxBatchPointers>;

struct QuantizeTensor {
    const float* grad;
    uint64_t n;
    uint64_t elem_base;
    uint32_t* packed;
    float* scales;
    const float* scales_in;      // nullable: the layer's scales are read, not computed
    uint32_t parts, borrowed;    // as in QuantizeArgs
};
struct QuantizeBatchHead {
    QuantizeArgs common;      // bits, bucket, stream selection, n = elements of all tensors; the other per-tensor fields are taken from t[]
    uint32_t count;
    uint32_t tile_elems;
};
template <uint32_t TENSORS>
struct QuantizeBatch : QuantizeBatchHead {
    using Tensor = QuantizeTensor;
    using Few = QuantizeBatch<kFewTensors>;
    uint32_t tile_start[TENSORS + 1];
    Tensor t[TENSORS];
    bool few() const { return count <= kFewTensors; }
    void copy_to(Few& f) const {
        static_cast<QuantizeBatchHead&>(f) = *this;
        for (uint32_t i = 0; i < kFewTensors; ++i) f.t[i] = t[i];
        for (uint32_t i = 0; i <= kFewTensors; ++i) f.tile_start[i] = tile_start[i];
    }
};
using BatchQuantizeArgs = QuantizeBatch<kMaxBatchTensors>;

// Calls f with the batch, or with its small form where it fits: launch(args) of either type.
template <class Batch, class F>
auto with_few(const Batch& a, F f) {
    if (a.few()) {
        typename Batch::Few small;
        a.copy_to(small);
        return f(small);
    }
    return f(a);
}

uint32_t aggregate_batch_tile();
hipError_t launch_aggregate_tensors(const BatchAggregateArgs& a, uint32_t tiles, hipStream_t stream);
uint32_t quantize_batch_tile(const BatchQuantizeArgs& a);   // elements per workgroup of the kernel the batch will run (reads a.common only)
uint32_t quantize_wave_block_elems(uint32_t bucket, uint32_t bits, uint64_t n);                             // quantize_wave.hip
hipError_t launch_quantize_tensors_wave(const BatchQuantizeArgs& a, uint32_t blocks, hipStream_t stream);
hipError_t launch_quantize_tensors(const BatchQuantizeArgs& a, uint32_t tiles, hipStream_t stream);

hipError_t launch_quantize(const QuantizeArgs& a, hipStream_t stream);
hipError_t launch_requantize(const RequantArgs& a, hipStream_t stream);
bool quantize_wave_supported(const QuantizeArgs& a);          // quantize_wave.hip
hipError_t launch_quantize_wave(const QuantizeArgs& a, hipStream_t stream);
bool quantize_cells_supported(const QuantizeArgs& a);         // quantize_wave.hip: other multiples of 32 up to 4064
hipError_t launch_quantize_cells(const QuantizeArgs& a, hipStream_t stream);
uint32_t quantize_cells_tile_elems(uint32_t bucket);
bool quantize_tensors_cells_supported(const BatchQuantizeArgs& a);
hipError_t launch_quantize_tensors_cells(const BatchQuantizeArgs& a, uint32_t tiles, hipStream_t stream);
bool quantize_minmax_wave_supported(const QuantizeArgs& a);   // quantize_wave.hip
hipError_t launch_quantize_minmax_wave(const QuantizeArgs& a, hipStream_t stream);
bool requantize_wave_supported(const RequantArgs& a);         // quantize_wave.hip
hipError_t launch_requantize_wave(const RequantArgs& a, hipStream_t stream);
hipError_t launch_aggregate(const AggregateArgs& a, hipStream_t stream);
hipError_t launch_aggregate_mean(const AggregateArgs& a, hipStream_t stream);   // a.params receives the mean gradient

// minmax.hip: deterministic [min, max] encoding; `scales` holds (min, max) pairs, 2 floats per bucket
hipError_t launch_quantize_minmax(const QuantizeArgs& a, hipStream_t stream);
hipError_t launch_aggregate_minmax(const AggregateArgs& a, hipStream_t stream);
hipError_t launch_requantize_minmax(const RequantArgs& a, hipStream_t stream);
hipError_t launch_requantize_minmax_tensor(const RequantArgs& a, hipStream_t stream);   // one range per worker and for the mean
// requantize_cells.hip: the re-encoding steps with one cell of 32 elements per lane.  The two passes of the whole-tensor
// one (tile: elements per workgroup), and the bucketed ones: [min, max], and the max-abs range with stochastic rounding
bool tensor_cells_supported(const RequantArgs& a);
uint32_t tensor_cells_tile();
void launch_sum_range_cells(const RequantArgs& a, uint32_t tiles, uint32_t tile, uint32_t* keys, hipStream_t stream);
void launch_requantize_tensor_cells(const RequantArgs& a, uint32_t tiles, uint32_t tile, const float* sum_range, uint32_t borrowed, hipStream_t stream);
bool requantize_minmax_cells_supported(const RequantArgs& a);
hipError_t launch_requantize_minmax_cells(const RequantArgs& a, hipStream_t stream);
bool requantize_centred_cells_supported(const RequantArgs& a);
hipError_t launch_requantize_centred_cells(const RequantArgs& a, hipStream_t stream);
hipError_t launch_tensor_range(const float* grad, uint64_t n, float* range_out, hipStream_t stream);
// the same for several tensors that are encoded next, with their code words as the workgroups' scratch memory
template <uint32_t TENSORS>
struct TensorRanges {
    using Few = TensorRanges<kFewRanges>;
    uint32_t count, bits;
    uint32_t in_slots;                   // set by the launch: tensors of several workgroups have their keys in slots
    RangeSlots slots[TENSORS];           // set by the launch
    const float* grad[TENSORS];
    uint64_t n[TENSORS];                 // 0: no such tensor (or an empty one)
    float* range[TENSORS];               // 2 floats each
    uint32_t* parts[TENSORS];            // the tensor's code words
    uint32_t block_start[TENSORS + 1];   // filled by the launch: prefix sums of the tensors' workgroups
    bool few() const { return count <= kFewRanges; }
    void copy_to(Few& f) const {
        f.count = count;
        f.bits = bits;
        f.in_slots = in_slots;
        for (uint32_t i = 0; i < kFewRanges; ++i) {
            f.slots[i] = slots[i];
            f.grad[i] = grad[i];
            f.n[i] = n[i];
            f.range[i] = range[i];
            f.parts[i] = parts[i];
        }
        for (uint32_t i = 0; i <= kFewRanges; ++i) f.block_start[i] = block_start[i];
    }
};
using TensorRangeBatch = TensorRanges<kMaxBatchTensors>;
hipError_t launch_tensor_ranges(TensorRangeBatch& b, uint32_t count, hipStream_t stream);
hipError_t launch_quantize_minmax_tensor(const QuantizeArgs& a, hipStream_t stream);    // a.scales: the one range; a.bucket unused
uint32_t quantize_minmax_wave_block_elems(uint32_t bucket);                                       // quantize_wave.hip
hipError_t launch_quantize_minmax_tensors_wave(const BatchQuantizeArgs& a, uint32_t blocks, hipStream_t stream);
uint32_t quantize_minmax_batch_tile(uint32_t bucket, int bucket_shift);   // elements per workgroup
hipError_t launch_quantize_minmax_tensors(const BatchQuantizeArgs& a, uint32_t tiles, hipStream_t stream);
uint32_t aggregate_minmax_batch_tile();
hipError_t launch_aggregate_minmax_tensors(const BatchAggregateArgs& a, uint32_t tiles, hipStream_t stream);
hipError_t launch_sum_squares(const float* grad, uint64_t n, double* out, hipStream_t stream);

// Sums of squares of several tensors in one launch, each added up in a fixed order.
constexpr uint32_t kMaxSumTensors = 64;
struct SumSquaresBatch {
    const float* grad[kMaxSumTensors];
    uint64_t n[kMaxSumTensors];
};
uint32_t sum_squares_batch_blocks();   // partial sums (doubles of scratch memory) per tensor
hipError_t launch_sum_squares_batch(const SumSquaresBatch& b, uint32_t count, double* partials, double* out, hipStream_t stream);
// the same with the partial sums in a device array the library holds (no allocation, no workspace argument)
hipError_t launch_sum_squares_batch_static(const SumSquaresBatch& b, uint32_t count, double* out, hipStream_t stream);

}  // namespace mqg
