// The Section 3.2 footnote read literally, on gfx950: a deterministic range-linear encode of a
// gradient to K bits over the [min, max] of each bucket (bucket >= n: one range per tensor, as in the
// paper), the matching server step, and the sum of squares that the "Adaptive" baseline's bit rule
// (Section 4.1) needs.
//
//   encode   mn, mx per bucket;  a = L / (mx - mn);  c = clamp(rint((g - mn) * a), 0, L)
//   decode   value = fma((float)c, (mx - mn) / L, mn)
//   server   acc = sum_w value_w (worker order);  p <- fma(-(lr/W), acc, p)
//
// No random numbers.  Work decomposition as in the stochastic quantizer's workgroup-cooperative
// kernel: a workgroup owns one tile of whole buckets (four float4 per lane, 256 to 1024 lanes, read
// from HBM once), ranges go through LDS with order-preserving integer keys, codes are packed through
// LDS and whole words are stored coalesced.

#include <mutex>
#include <type_traits>

#include "batch.h"
#include "decode.h"
#include "encode.h"
#include "kernels.h"
#include "tile_io.h"

namespace mqg {
namespace {

using namespace encode;
using tile_io::kThreads;

constexpr int kChunk = 8;   // workers whose code loads are in flight together
// The whole-tensor reductions end with one atomic per workgroup on one address; those serialize at
// about 5 ns each and every workgroup arrives at the end together, so the workgroups are few and large:
// 512 of 512 lanes (8 waves per SIMD) read as fast as 2048 of 256 and end 7 us earlier at 100 M elements.
constexpr int kSumThreads = 512;
constexpr uint32_t kSumBlocks = 512;
// Largest tensor that one workgroup encodes in registers, whatever the encoder: the largest bucket.
constexpr uint64_t kOneBucketElems = 16384;
constexpr uint32_t kComputeUnits = 256;

// A workgroup's tile: whole buckets.
struct TileGeometry {
    uint32_t elems;     // buckets * bucket
    uint32_t buckets;
    uint32_t magic;     // ceil(65536 / (bucket / 32)): (cell * magic) >> 16 = cell / (bucket / 32) for a tile's cells (at most 224)
};
// which parts of a tile can lie past its last element: none, whole quads only, or single elements
constexpr int kTailNone = 0, kTailQuads = 1, kTailElements = 2;

// NT lanes own a tile of at most 4*NT*R elements.  ONE: the tile is one bucket (of more than 4096 elements).
template <int R, int NT, bool ONE>
struct Shared {
    static constexpr uint32_t kCap = 4u * NT * R;
    uint32_t words[kCap * 8u / 32u + 4];
    uint32_t kmin[128];
    uint32_t kmax[128];
    float mn[128];
    float a[128];
};

// one HBM pass: the tile of the gradient into registers
template <int R, int NT, int TAIL>
__device__ __forceinline__ void load_grad_tile(const float* __restrict__ g, const uint32_t tile_count, float4 (&x)[R]) {
    const uint32_t tid = threadIdx.x;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const uint32_t el = 4u * (j * NT + tid);
        if (TAIL == kTailNone || el + 4u <= tile_count) {
            const v4f t = __builtin_nontemporal_load(reinterpret_cast<const v4f_a4*>(g + el));
            x[j] = make_float4(t.x, t.y, t.z, t.w);
        } else if (TAIL == kTailQuads) {
            x[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        } else {
            x[j].x = (el + 0u < tile_count) ? g[el + 0] : 0.0f;
            x[j].y = (el + 1u < tile_count) ? g[el + 1] : 0.0f;
            x[j].z = (el + 2u < tile_count) ? g[el + 2] : 0.0f;
            x[j].w = 0.0f;   // el + 3 >= tile_count here
        }
    }
}

template <int R, int NT, bool ONE>
__device__ __forceinline__ void clear_shared(Shared<R, NT, ONE>& sm, uint32_t tile_count, uint32_t b) {
    const uint32_t tid = threadIdx.x;
    const uint32_t nwords = (tile_count * b + 31u) >> 5;
    for (uint32_t i = tid; i < nwords; i += NT) sm.words[i] = 0u;
    if (tid < 128u) {
        sm.kmin[tid] = 0xFFFFFFFFu;
        sm.kmax[tid] = 0u;
    }
}

// buckets that begin inside the tile
template <bool ONE>
__device__ __forceinline__ uint32_t buckets_in_tile(const uint32_t bucket, const TileGeometry& g, const uint32_t tile_count) {
    if (ONE) return 1u;
    return tile_count == g.elems ? g.buckets : (tile_count + bucket - 1u) / bucket;
}

// The tile, once its values are in registers; enters right after the barrier that follows
// clear_shared.  range_div: the stored range is [mn, mx] / range_div (1 for a plain encode, W for the
// server's mean).
// GIVEN: one (min, max) pair for every element, `given` (the whole-tensor range found by an earlier
// pass); no range is reduced and none is stored.
template <int R, int NT, int TAIL, bool ONE, bool GIVEN = false>
__device__ __forceinline__ void encode_minmax_tile(const QuantizeArgs& a, const TileGeometry& g, const uint32_t tile,
                                                   const uint64_t tile_base, const uint32_t tile_count,
                                                   const float4 (&x)[R], const float range_div, Shared<R, NT, ONE>& sm,
                                                   const float2 given = make_float2(0.0f, 0.0f)) {
    const uint32_t tid = threadIdx.x;
    const float inf = __builtin_inff();
    const uint32_t b = a.bits;
    const uint32_t nwords = (tile_count * b + 31u) >> 5;

    const uint32_t nbt = GIVEN ? 1u : buckets_in_tile<ONE>(a.bucket, g, tile_count);
    const uint64_t kb0 = GIVEN ? 0u : (uint64_t)tile * g.buckets;
    uint32_t bl[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const uint32_t el = 4u * (j * NT + tid);
        bl[j] = (GIVEN || ONE) ? 0u : ((el >> 5) * g.magic) >> 16;
    }

    // ---- bucket range: 8-lane cells by DPP; whole waves when a wave's row lies in one bucket -------
    // (every lane of a cell, or of a wave, then holds the same value, and one lane folds it into the
    // bucket's LDS slot: few atomics per slot, since same-address LDS atomics serialize)
    const uint32_t lane = tid & 63u;
    const bool row_in_bucket = ONE || (a.bucket & 255u) == 0u;   // uniform over the launch
    if (!GIVEN) {
    float lo[R], hi[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const uint32_t el = 4u * (j * NT + tid);
        if (TAIL != kTailElements) {
            const bool in = TAIL == kTailNone || el < tile_count;
            lo[j] = quad_min(x[j].x, x[j].y, x[j].z, x[j].w);
            hi[j] = quad_max(x[j].x, x[j].y, x[j].z, x[j].w);
            lo[j] = in ? lo[j] : inf;
            hi[j] = in ? hi[j] : -inf;
        } else {   // elements past the end take no part
            const bool v0 = el + 0u < tile_count, v1 = el + 1u < tile_count;
            const bool v2 = el + 2u < tile_count, v3 = el + 3u < tile_count;
            lo[j] = quad_min(v0 ? x[j].x : inf, v1 ? x[j].y : inf, v2 ? x[j].z : inf, v3 ? x[j].w : inf);
            hi[j] = quad_max(v0 ? x[j].x : -inf, v1 ? x[j].y : -inf, v2 ? x[j].z : -inf, v3 ? x[j].w : -inf);
        }
    }
    if (ONE) {   // the tile is one bucket: fold the lane's rows first
#pragma unroll
        for (int j = 1; j < R; ++j) {
            lo[0] = min_f32(lo[0], lo[j]);
            hi[0] = max_f32(hi[0], hi[j]);
        }
    }
    if (a.drop_nan != 0u) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            lo[j] = min_f32(lo[j], inf);
            hi[j] = max_f32(hi[j], -inf);
        }
    }
    // across lanes on order-preserving integer keys, stage by stage over the rows
    uint32_t kl[R], kh[R];
#pragma unroll
    for (int j = 0; j < (ONE ? 1 : R); ++j) {
        kl[j] = cell_min_u32(order_key(lo[j]));
        kh[j] = cell_max_u32(order_key(hi[j]));
    }
    if (row_in_bucket) {
#pragma unroll
        for (int j = 0; j < (ONE ? 1 : R); ++j) {
            kl[j] = wave_min_from_cells_u32(kl[j], lane);
            kh[j] = wave_max_from_cells_u32(kh[j], lane);
        }
#pragma unroll
        for (int j = 0; j < (ONE ? 1 : R); ++j) {
            const uint32_t row_first = 4u * (j * NT + (tid & ~63u));   // first element of the wave's row
            if (lane == 0u && (TAIL == kTailNone || ONE || row_first < tile_count)) {
                atomicMin(&sm.kmin[bl[j]], kl[j]);
                atomicMax(&sm.kmax[bl[j]], kh[j]);
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const uint32_t el = 4u * (j * NT + tid);
            if ((tid & 7u) == 0u && (TAIL == kTailNone || el < tile_count)) {
                atomicMin(&sm.kmin[bl[j]], kl[j]);
                atomicMax(&sm.kmax[bl[j]], kh[j]);
            }
        }
    }
    }
    __syncthreads();

    const float Lf = (float)((1u << b) - 1u);
    if (tid < nbt) {
        float mn, mx;
        if (GIVEN) {
            mn = given.x;
            mx = given.y;
        } else {
            mn = key_value(sm.kmin[tid]);
            mx = key_value(sm.kmax[tid]);
            if (mn == 0.0f) mn = 0.0f;   // a zero bound is stored as +0
            if (mx == 0.0f) mx = 0.0f;
            a.scales[2u * (kb0 + tid)] = (range_div == 1.0f) ? mn : mn / range_div;
            a.scales[2u * (kb0 + tid) + 1u] = (range_div == 1.0f) ? mx : mx / range_div;
        }
        const float r = mx - mn;
        sm.mn[tid] = mn;
        sm.a[tid] = (r >= 0x1p-96f) ? Lf / r : 0.0f;   // IEEE-correct fp32 division, once per bucket
    }
    __syncthreads();

    // ---- nearest level, packing -----------------------------------------------------------------
    const uint32_t cell_bit = 4u * b * (tid & 7u);            // this lane's bit offset in its 32-element cell
    const uint32_t sh = cell_bit & 31u;
    const uint32_t word_in_cell = cell_bit >> 5;
    const bool straddle = sh + 4u * b > 32u;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const uint32_t ql = j * NT + tid;
        const uint32_t el = 4u * ql;
        const float mn = sm.mn[bl[j]], ai = sm.a[bl[j]];
        uint32_t k0 = nearest_code(x[j].x, mn, ai, Lf);
        uint32_t k1 = nearest_code(x[j].y, mn, ai, Lf);
        uint32_t k2 = nearest_code(x[j].z, mn, ai, Lf);
        uint32_t k3 = nearest_code(x[j].w, mn, ai, Lf);
        if (TAIL == kTailElements) {   // elements past the end contribute zero bits
            if (el + 0u >= tile_count) k0 = 0u;
            if (el + 1u >= tile_count) k1 = 0u;
            if (el + 2u >= tile_count) k2 = 0u;
            if (el + 3u >= tile_count) k3 = 0u;
        }
        const uint32_t v = (((((k3 << b) | k2) << b) | k1) << b) | k0;
        if (TAIL == kTailNone || el < tile_count) {
            const uint32_t w0 = (ql >> 3) * b + word_in_cell;
            atomicOr(&sm.words[w0], v << sh);
            if (straddle) atomicOr(&sm.words[w0 + 1u], v >> (32u - sh));
        }
    }
    __syncthreads();

    uint32_t* __restrict__ out = a.packed + (tile_base >> 5) * b;
    for (uint32_t i = tid; i < nwords; i += NT) __builtin_nontemporal_store(sm.words[i], out + i);
}

// Bucket sizes that are not powers of two (the others take the wave-local kernel in quantize_wave.hip).
template <int R, int NT, int TAIL, bool ONE>
__device__ __forceinline__ void quantize_minmax_loaded(const QuantizeArgs& a, const TileGeometry& g, const uint32_t tile,
                                                       const uint64_t tile_base, const uint32_t tile_count, Shared<R, NT, ONE>& sm) {
    float4 x[R];
    load_grad_tile<R, NT, TAIL>(a.grad + tile_base, tile_count, x);
    clear_shared(sm, tile_count, a.bits);   // while the loads are in flight
    __syncthreads();
    encode_minmax_tile<R, NT, TAIL>(a, g, tile, tile_base, tile_count, x, 1.0f, sm);
}
template <int R, int NT, bool ONE>
__device__ __forceinline__ void quantize_minmax_tile(const QuantizeArgs& a, const TileGeometry& g, const uint32_t tile,
                                                     Shared<R, NT, ONE>& sm) {
    const uint64_t tile_base = (uint64_t)tile * g.elems;
    const uint64_t left = a.n - tile_base;
    const uint32_t tile_count = left < g.elems ? (uint32_t)left : g.elems;
    if ((tile_count & 3u) == 0u) {   // every tile but the one that holds the tensor's ragged end
        quantize_minmax_loaded<R, NT, kTailQuads>(a, g, tile, tile_base, tile_count, sm);
    } else {
        quantize_minmax_loaded<R, NT, kTailElements>(a, g, tile, tile_base, tile_count, sm);
    }
}

template <int R, int NT, bool ONE>
__global__ __launch_bounds__(NT) void quantize_minmax_kernel(const QuantizeArgs a, const TileGeometry g) {
    drop_every_nan();
    __shared__ Shared<R, NT, ONE> sm;
    quantize_minmax_tile(a, g, blockIdx.x, sm);
}

// Several layer tensors in one launch: workgroup -> (tensor, tile of the tensor) through the prefix
// table of tile counts.
template <int R, int NT, bool ONE, class Batch>
__global__ __launch_bounds__(NT) void quantize_minmax_tensors_kernel(const Batch ba, const TileGeometry g) {
    drop_every_nan();
    __shared__ Shared<R, NT, ONE> sm;
    const uint32_t lo = tensor_of_block(ba.tile_start, ba.count, blockIdx.x);
    QuantizeArgs a = ba.common;
    a.grad = ba.t[lo].grad;
    a.n = ba.t[lo].n;
    a.packed = ba.t[lo].packed;
    a.scales = ba.t[lo].scales;
    quantize_minmax_tile(a, g, blockIdx.x - ba.tile_start[lo], sm);
}

// The server's re-encoding step of the full exchange (ReceiveQGThenSendQG): the tile's values are the
// sum over the W workers' de-quantized gradients, decoded from their streams in worker order; the
// stored range is divided by W.  (step, min) of every worker's buckets of the tile sit in an LDS table.
//
// This kernel takes the short launches and the smallest buckets (requantize_minmax_cells_supported).  Bound by latency, that
// of the code words, hidden by more words in flight in short launches and by other waves in long ones.  CH: workers whose
// words are in flight together; left alone the compiler takes 112-117 registers for eight and their table entries (four
// waves per SIMD), with four seven waves fit (MANY and 256 lanes: six, since seven spill).
// us at 4 bits, eight in flight / four:                 (256 lanes, seven waves with 8-16 bytes of scratch memory)
//   bucket 1024, 24 workers, 1 M elements     9.0 /  9.4   (11.1)
//   bucket 4096, 16 workers, 1 M              7.2 /  7.4   ( 8.4)
// MANY: more than CH workers.  Without the loop over them 58 registers do (eight waves).
constexpr int requant_waves(int NT, bool one, int CH, bool many) {
    if (NT == 768) return 6;                     // two workgroups per compute unit
    if (!one && CH == 8) return 4;
    return !one && NT == 256 && many ? 6 : 7;
}
template <int NT, bool ONE, bool STRADDLE, bool ONCE, int CH, bool MANY>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(requant_waves(NT, ONE, CH, MANY), 8))) void requantize_minmax_kernel(const RequantArgs ra, const TileGeometry g) {
    constexpr int R = 4;
    __shared__ Shared<R, NT, ONE> sm;
    extern __shared__ float2 s_tab[];   // [W][buckets of the tile]
    const QuantizeArgs& a = ra.q;
    const uint32_t tid = threadIdx.x;
    const uint64_t tile_base = (uint64_t)blockIdx.x * g.elems;
    const uint64_t left = a.n - tile_base;
    const uint32_t tile_count = left < g.elems ? (uint32_t)left : g.elems;
    const uint32_t b = a.bits;
    const float Lf = (float)((1u << b) - 1u);

    const decode::CodeWindows<R> cw = decode::code_windows<R, NT>(a.n, tile_base, b, tid);
    decode::CodeRegs<R, CH> c;
    decode::fetch_codes<R, CH, ONCE>(ra.packed, ra.W, 0u, cw, c);   // in flight while the table is filled
    const uint32_t nbt = buckets_in_tile<ONE>(a.bucket, g, tile_count);
    const uint64_t kb0 = (uint64_t)blockIdx.x * g.buckets;
    for (uint32_t i = tid; i < ra.W * nbt; i += NT) {
        const uint32_t w = i / nbt, kb = i - w * nbt;
        const float2 rg = reinterpret_cast<const float2*>(ra.scales[w])[kb0 + kb];   // (min, max)
        s_tab[i] = make_float2((rg.y - rg.x) / Lf, rg.x);                            // IEEE-correct fp32 division
    }
    clear_shared(sm, tile_count, b);
    __syncthreads();

    uint32_t bl[R];
    float4 x[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const uint32_t el = 4u * (j * NT + tid);
        bl[j] = ONE ? 0u : ((el >> 5) * g.magic) >> 16;
        if (bl[j] >= nbt) bl[j] = nbt - 1u;   // quads past the end: any valid slot
        x[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    for (uint32_t w0 = 0; w0 < (MANY ? ra.W : 1u); w0 += CH) {
        if (w0 > 0) decode::fetch_codes<R, CH, ONCE>(ra.packed, ra.W, w0, cw, c);
#pragma unroll
        for (int t = 0; t < CH; ++t) {
            if (w0 + t < ra.W) {
                const float2* __restrict__ tw = s_tab + (w0 + t) * nbt;
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const float2 sl = tw[bl[j]];
                    decode::accumulate_quad_minmax<STRADDLE>(c.lo[t][j], cw.sh, b, sl.x, sl.y, x[j]);
                }
            }
        }
    }
    const float Wf = (float)ra.W;
    if (tile_count == Shared<R, NT, ONE>::kCap) {
        encode_minmax_tile<R, NT, kTailNone>(a, g, blockIdx.x, tile_base, tile_count, x, Wf, sm);
    } else if ((tile_count & 3u) == 0u) {   // elements past the end are decoded but take no part
        encode_minmax_tile<R, NT, kTailQuads>(a, g, blockIdx.x, tile_base, tile_count, x, Wf, sm);
    } else {
        encode_minmax_tile<R, NT, kTailElements>(a, g, blockIdx.x, tile_base, tile_count, x, Wf, sm);
    }
}

// ---- the same with ONE range for the whole tensor, as the paper encodes -----------------------------
// The range of the sum is not known until every element has been decoded, so the step takes two passes
// over the W code streams (the fp32 sum still never exists in memory: (2 W + 1) * bits / 8 bytes per
// element in all): pass 1 decodes and leaves each workgroup's min / max keys at the front of packed_out,
// which pass 2 overwrites anyway; one workgroup in between folds them, stores the mean's range and puts
// the sum's range into the first two words of every pass-2 workgroup's own output, where no other
// workgroup writes; pass 2 picks it up there, decodes again and encodes over it.  Three launches.  With
// the keys folded by atomics on one address (and launches to prime, convert and divide them) the step takes 50 us
// instead of 39 at 10 M elements, 12 workers, 4 bits.  That form (range_out as the place of both the keys and the
// sum's range) serves the calls whose packed_out lies over one of the streams they read, where nothing may be
// written before pass 2, and the largest: one workgroup's time grows with the tiles, and so few of very many
// workgroups move a key that the atomics cost little.  us with the fold / with atomics, 4 bits, passes of requantize_cells.hip:
//   elements     1 worker     4          12 workers
//   30 M         21 /  42     37 /  58     76 /  83
//   100 M        55 /  85     98 / 113    236 / 251
//   200 M       100 / 123    201 / 208    486 / 488
//   400 M       191 / 196    398 / 392    950 / 930
// The passes below are those of small tensors (see tensor_cells_supported); larger ones hold a cell per lane.
// Every worker has one (min, max) pair; s_tab[w] = (step, min) of worker w.
template <int NT, bool STRADDLE, bool ONCE>
__device__ __forceinline__ void decode_sum_tile_tensor(const RequantArgs& ra, const uint64_t tile_base, float2* s_tab,
                                                       float4 (&x)[4]) {
    constexpr int R = 4;
    constexpr int CH = 8;
    const uint32_t tid = threadIdx.x;
    const uint32_t b = ra.q.bits;
    const float Lf = (float)((1u << b) - 1u);
    const decode::CodeWindows<R> cw = decode::code_windows<R, NT>(ra.q.n, tile_base, b, tid);
    decode::CodeRegs<R, CH> c;
    decode::fetch_codes<R, CH, ONCE>(ra.packed, ra.W, 0u, cw, c);   // in flight while the table is filled
    if (tid < ra.W) {
        const float2 rg = *reinterpret_cast<const float2*>(ra.scales[tid]);   // (min, max) of worker tid
        s_tab[tid] = make_float2((rg.y - rg.x) / Lf, rg.x);                   // IEEE-correct fp32 division
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < R; ++j) x[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (uint32_t w0 = 0; w0 < ra.W; w0 += CH) {
        if (w0 > 0) decode::fetch_codes<R, CH, ONCE>(ra.packed, ra.W, w0, cw, c);
#pragma unroll
        for (int t = 0; t < CH; ++t) {
            if (w0 + t < ra.W) {
                const float2 sl = s_tab[w0 + t];
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    decode::accumulate_quad_minmax<STRADDLE>(c.lo[t][j], cw.sh, b, sl.x, sl.y, x[j]);
                }
            }
        }
    }
}

// Folds `count` pairs of keys into every lane's own, AHEAD loads of each in flight.
template <int NT, int AHEAD>
__device__ __forceinline__ void fold_pairs(const uint32_t* pairs, const uint32_t count, uint32_t& kl, uint32_t& kh) {
    for (uint32_t i0 = threadIdx.x; i0 < count; i0 += NT * AHEAD) {
        uint32_t l[AHEAD], h[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const uint32_t i = i0 + u * NT < count ? i0 + u * NT : i0;   // past the end: one of its own again
            l[u] = pairs[2u * i];
            h[u] = pairs[2u * i + 1u];
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            kl = min(kl, l[u]);
            kh = max(kh, h[u]);
        }
    }
}

// Folds a workgroup's keys (every lane holds its own) over NT lanes; the result is in thread 0.
template <int NT>
__device__ __forceinline__ void fold_keys(uint32_t& kl, uint32_t& kh, uint32_t* s_lo, uint32_t* s_hi) {
    const uint32_t tid = threadIdx.x;
    kl = wave_min_from_cells_u32(cell_min_u32(kl), tid & 63u);
    kh = wave_max_from_cells_u32(cell_max_u32(kh), tid & 63u);
    if ((tid & 63u) == 0u) {
        s_lo[tid >> 6] = kl;
        s_hi[tid >> 6] = kh;
    }
    __syncthreads();
    if (tid == 0u) {
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) {
            kl = min(kl, s_lo[w]);
            kh = max(kh, s_hi[w]);
        }
    }
}
// Same-address atomics serialize in L2: look first.  The keys only ever move one way, so a stale read can
// cause a needless atomic but never a wrong skip.
__device__ __forceinline__ void fold_into(uint32_t* keys, uint32_t kl, uint32_t kh) {
    if (kl < __atomic_load_n(&keys[0], __ATOMIC_RELAXED)) atomicMin(&keys[0], kl);
    if (kh > __atomic_load_n(&keys[1], __ATOMIC_RELAXED)) atomicMax(&keys[1], kh);
}
// Two floats as the place of the keys: one-thread launches prime them, turn them back into floats and, for
// the mean, divide by W.
__global__ void range_init_kernel(uint32_t* keys) {
    keys[0] = 0xFFFFFFFFu;
    keys[1] = 0u;
}
__global__ void range_finish_kernel(uint32_t* keys) {
    const float2 r = range_of_keys(keys[0], keys[1]);
    keys[0] = __builtin_bit_cast(uint32_t, r.x);
    keys[1] = __builtin_bit_cast(uint32_t, r.y);
}
__global__ void range_divide_kernel(float* range, float Wf) {
    range[0] = range[0] / Wf;
    range[1] = range[1] / Wf;
}

// Both passes: one workgroup per tile of kSumTile elements.  (A loop for a tail without two words of its own in place of
// the borrowed elements below took 96 registers instead of 70, five waves per SIMD instead of seven.)
constexpr int kSumTileThreads = 256;
constexpr uint32_t kSumTile = 4u * kSumTileThreads * 4u;
constexpr uint64_t kMostFoldedTiles = 32768;   // 268 M elements at 8192 per tile

template <int NT, bool STRADDLE, bool ONCE>
__global__ __launch_bounds__(NT) void sum_range_minmax_tensor_kernel(const RequantArgs ra, uint32_t* keys) {
    static_assert(4u * NT * 4u == kSlotTile, "one workgroup per tile");
    constexpr int R = 4;
    constexpr uint32_t kCap = 4u * NT * R;
    __shared__ float2 s_tab[MQG_MAX_WORKERS];
    __shared__ uint32_t s_lo[NT / 64], s_hi[NT / 64], s_keys[2];
    const uint32_t tid = threadIdx.x;
    const uint64_t tile_base = (uint64_t)blockIdx.x * kCap;
    const uint64_t left = ra.q.n - tile_base;
    const uint32_t tile_count = left < kCap ? (uint32_t)left : kCap;
    float4 x[R];
    decode_sum_tile_tensor<NT, STRADDLE, ONCE>(ra, tile_base, s_tab, x);
    const float inf = __builtin_inff();
    float lo = inf, hi = -inf;
#pragma unroll
    for (int j = 0; j < R; ++j) {   // elements past the end take no part
        const uint32_t el = 4u * (j * NT + tid);
        if (el + 0u < tile_count) { lo = fminf(lo, x[j].x); hi = fmaxf(hi, x[j].x); }
        if (el + 1u < tile_count) { lo = fminf(lo, x[j].y); hi = fmaxf(hi, x[j].y); }
        if (el + 2u < tile_count) { lo = fminf(lo, x[j].z); hi = fmaxf(hi, x[j].z); }
        if (el + 3u < tile_count) { lo = fminf(lo, x[j].w); hi = fmaxf(hi, x[j].w); }
    }
    uint32_t kl = order_key(lo), kh = order_key(hi);
    fold_keys<NT>(kl, kh, s_lo, s_hi);
    if (ra.q.parts != 0u) {
        keys_to_slots(ra.q.packed, ra.q.n, ra.q.bits, ra.q.borrowed, blockIdx.x, kl, kh, s_keys);
    } else if (tid == 0u) {
        if (keys != nullptr) {
            fold_into(keys, kl, kh);
        } else {
            ra.q.packed[2u * blockIdx.x] = kl;
            ra.q.packed[2u * blockIdx.x + 1u] = kh;
        }
    }
}

// First element of pass 2's tile `tile` of `tiles`, tile_elems each.  borrowed: elements that the last tile takes from the one before
// it, so that it has two words of its own to find the range of the sum in.
__device__ __forceinline__ uint64_t second_pass_base(uint32_t tile, uint32_t tiles, uint32_t borrowed, uint32_t tile_elems) {
    return (uint64_t)tile * tile_elems - (tile + 1u == tiles ? borrowed : 0u);
}

// One workgroup: all keys are read before the barrier of fold_keys, the words that receive the sum's range
// (they overlap the keys) are written after it.
constexpr int kFoldThreads = 1024;
__global__ __launch_bounds__(kFoldThreads) void fold_sum_range_kernel(uint32_t* packed, const uint32_t tiles, const uint32_t tile_elems, const uint32_t borrowed,
                                                                      const uint32_t bits, float* range, const float Wf) {
    __shared__ uint32_t s_lo[kFoldThreads / 64], s_hi[kFoldThreads / 64];
    __shared__ float2 s_range;
    const uint32_t tid = threadIdx.x;
    uint32_t kl = 0xFFFFFFFFu, kh = 0u;
    fold_pairs<kFoldThreads, 2>(packed, tiles, kl, kh);
    fold_keys<kFoldThreads>(kl, kh, s_lo, s_hi);
    if (tid == 0u) {
        const float2 r = range_of_keys(kl, kh);
        s_range = r;
        range[0] = r.x / Wf;   // the grid of the mean is the grid of the sum scaled by 1 / W
        range[1] = r.y / Wf;
    }
    __syncthreads();
    const float2 r = s_range;
    for (uint32_t i = tid; i < tiles; i += kFoldThreads) {
        uint32_t* slot = packed + (second_pass_base(i, tiles, borrowed, tile_elems) >> 5) * bits;
        slot[0] = __builtin_bit_cast(uint32_t, r.x);
        slot[1] = __builtin_bit_cast(uint32_t, r.y);
    }
}

template <int NT, bool STRADDLE, bool ONCE>
__global__ __launch_bounds__(NT) void requantize_minmax_tensor_kernel(const RequantArgs ra, const float* sum_range,
                                                                      const uint32_t borrowed) {
    constexpr int R = 4;
    constexpr uint32_t kCap = Shared<R, NT, false>::kCap;
    static_assert(kCap == kSumTile, "one workgroup per tile");
    __shared__ Shared<R, NT, false> sm;
    __shared__ float2 s_tab[MQG_MAX_WORKERS];
    const TileGeometry none = {};   // the range is given: no buckets
    const uint64_t tile_base = second_pass_base(blockIdx.x, gridDim.x, borrowed, kSumTile);
    const uint64_t end = blockIdx.x + 1u == gridDim.x ? ra.q.n : second_pass_base(blockIdx.x + 1u, gridDim.x, borrowed, kSumTile);
    const uint32_t tile_count = (uint32_t)(end - tile_base);
    // every lane holds the sum's range before the barrier below; the words are overwritten after it
    const uint32_t* own = ra.q.packed + (tile_base >> 5) * ra.q.bits;
    const float* slot = sum_range != nullptr ? sum_range : reinterpret_cast<const float*>(own);
    float2 range = make_float2(slot[0], slot[1]);
    if (ra.q.parts != 0u) {
        range = range_from_slot(own, ra.q.parts);
        if (blockIdx.x == 0u && threadIdx.x == 0u) {   // the grid of the mean is the grid of the sum scaled by 1 / W
            ra.q.scales[0] = range.x / (float)ra.W;
            ra.q.scales[1] = range.y / (float)ra.W;
        }
    }
    clear_shared(sm, tile_count, ra.q.bits);
    float4 x[R];
    decode_sum_tile_tensor<NT, STRADDLE, ONCE>(ra, tile_base, s_tab, x);   // its barrier also covers clear_shared
    if (tile_count == kCap) {
        encode_minmax_tile<R, NT, kTailNone, false, true>(ra.q, none, 0u, tile_base, tile_count, x, 1.0f, sm, range);
    } else {
        encode_minmax_tile<R, NT, kTailElements, false, true>(ra.q, none, 0u, tile_base, tile_count, x, 1.0f, sm, range);
    }
}

// ---- server step --------------------------------------------------------------------------------
constexpr int kAggR = 2;
constexpr uint32_t kAggTile = 1024u * kAggR;
constexpr uint32_t kMaxBuckets = kAggTile / 32u + 1u;   // buckets a tile can touch

// One tile of one tensor.  The fields of `a` that name the tensor (n, params, packed, scales) are not
// read: the tensor comes in through the arguments, so that one launch can serve several.  raw != nullptr:
// an uncompressed layer whose W fp32 gradients are added in worker order instead of decoded.
struct TileTensor {
    const uint32_t* const* packed;
    const float* const* scales;
    const float* const* raw;
    uint64_t n;
    float* params;
};
struct TileCommon {
    uint32_t W, bits, bucket;
    int bucket_shift;
    uint32_t per_tensor;
    float neg_c;
};
template <bool STRADDLE, bool ONCE>
__device__ __forceinline__ void aggregate_minmax_tile(const TileCommon& a, const TileTensor& t, const uint64_t tile_base,
                                                      float2* s_tab) {
    constexpr int R = kAggR;
    const uint32_t tid = threadIdx.x;
    const uint64_t left = t.n - tile_base;
    const uint32_t tile_count = left < kAggTile ? (uint32_t)left : kAggTile;
    const bool full = tile_count == kAggTile;
    float* __restrict__ p = t.params + tile_base;

    float4 x[R];
    tile_io::load_params<R>(p, tile_count, full, x);
    float4 acc[R];
#pragma unroll
    for (int j = 0; j < R; ++j) acc[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (t.raw != nullptr) {
        tile_io::accumulate_raw<R>(t.raw, a.W, tile_base, tile_count, full, acc);
        tile_io::update_params<R>(p, tile_count, full, a.neg_c, x, acc);
        return;
    }

    const uint32_t b = a.bits;
    const float Lf = (float)((1u << b) - 1u);
    const decode::CodeWindows<R> cw = decode::code_windows<R, kThreads>(t.n, tile_base, b, tid);
    decode::CodeRegs<R, kChunk> c;
    decode::fetch_codes<R, kChunk, ONCE>(t.packed, a.W, 0u, cw, c);   // in flight while the table is filled

    const uint64_t kb0 = tile_base / a.bucket;
    const uint32_t nbt = (uint32_t)((tile_base + tile_count - 1u) / a.bucket - kb0) + 1u;   // <= kMaxBuckets
    const uint32_t first_off = (uint32_t)(tile_base - kb0 * a.bucket);
    uint32_t bl[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const uint32_t eo = 4u * (j * kThreads + tid) + first_off;
        bl[j] = a.bucket_shift >= 0 ? (eo >> a.bucket_shift) : (eo / a.bucket);
        if (bl[j] >= nbt) bl[j] = nbt - 1u;   // quads past the end: any valid slot
    }
    for (uint32_t i = tid; i < a.W * nbt; i += kThreads) {
        const uint32_t w = i / nbt, kb = i - w * nbt;
        const float2 rg = reinterpret_cast<const float2*>(t.scales[w])[a.per_tensor ? 0u : kb0 + kb];   // (min, max)
        s_tab[i] = make_float2((rg.y - rg.x) / Lf, rg.x);                           // IEEE-correct fp32 division
    }
    __syncthreads();

    for (uint32_t w0 = 0; w0 < a.W; w0 += kChunk) {
        if (w0 > 0) decode::fetch_codes<R, kChunk, ONCE>(t.packed, a.W, w0, cw, c);
#pragma unroll
        for (int t = 0; t < kChunk; ++t) {
            if (w0 + t < a.W) {
                const float2* __restrict__ tw = s_tab + (w0 + t) * nbt;
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const float2 sl = tw[bl[j]];
                    decode::accumulate_quad_minmax<STRADDLE>(c.lo[t][j], cw.sh, b, sl.x, sl.y, acc[j]);
                }
            }
        }
    }
    tile_io::update_params<R>(p, tile_count, full, a.neg_c, x, acc);
}

template <bool STRADDLE, bool ONCE>
__global__ __launch_bounds__(kThreads) void aggregate_update_minmax_kernel(const AggregateArgs a) {
    extern __shared__ float2 s_tab[];   // [W][nbt]: (step, min) of each worker's buckets of the tile
    const TileCommon c = {a.W, a.bits, a.bucket, a.bucket_shift, a.per_tensor, a.neg_c};
    const TileTensor t = {a.packed, a.scales, nullptr, a.n, a.params};
    aggregate_minmax_tile<STRADDLE, ONCE>(c, t, (uint64_t)blockIdx.x * kAggTile, s_tab);
}

// Several tensors of a model in one launch: block -> (tensor, tile) through the prefix table of tile
// counts.  A tensor is either encoded (W packed + W range pointers) or raw (W fp32 gradients).
template <bool STRADDLE, bool ONCE, class Batch>
__global__ __launch_bounds__(kThreads) void aggregate_update_minmax_tensors_kernel(const Batch a) {
    extern __shared__ float2 s_tab[];
    const uint32_t lo = tensor_of_block(a.tile_start, a.count, blockIdx.x);
    const AggregateTensor& bt = a.t[lo];
    const void* const* ptrs = a.ptrs + bt.first_ptr;
    const TileCommon c = {a.W, a.bits, a.bucket, a.bucket_shift, a.per_tensor, a.neg_c};
    TileTensor t = {nullptr, nullptr, nullptr, bt.n, bt.params};
    if (bt.raw) {
        t.raw = reinterpret_cast<const float* const*>(ptrs);
    } else {
        t.packed = reinterpret_cast<const uint32_t* const*>(ptrs);
        t.scales = reinterpret_cast<const float* const*>(ptrs + a.W);
    }
    aggregate_minmax_tile<STRADDLE, ONCE>(c, t, (uint64_t)(blockIdx.x - a.tile_start[lo]) * kAggTile, s_tab);
}

// ---- whole-tensor range ---------------------------------------------------------------------------
// The paper encodes a tensor over ONE range.  A workgroup folds its share of the tensor into a pair of
// order-preserving integer keys (exact and order independent); what becomes of the workgroups' keys
// depends on the memory at hand.
// min / max keys of the share of g[0..n) that belongs to workgroup `block` of `nblocks`, in thread 0: contiguous pieces
// of four rows of 2048 elements (one float4 per lane, four in flight), and what is left spread over all.  (Single rows,
// nblocks apart: mqg_tensor_range at 10 M elements 19 us instead of 14, at 100 M 66 instead of 62.)
__device__ __forceinline__ void block_range(const float* __restrict__ g, const uint64_t n, const uint32_t block,
                                            const uint32_t nblocks, uint32_t& kl, uint32_t& kh, uint32_t* s_lo, uint32_t* s_hi) {
    const uint32_t tid = threadIdx.x;
    float lo = __builtin_inff(), hi = -__builtin_inff();
    const v4f_a4* __restrict__ g4 = reinterpret_cast<const v4f_a4*>(g);   // 128-bit loads need dword alignment only
    const uint64_t gtid = (uint64_t)block * kSumThreads + tid;
    const uint64_t stride = (uint64_t)nblocks * kSumThreads;
    const uint64_t nq = n >> 2;
    const auto fold = [&](const v4f t) {
        lo = min_f32(lo, quad_min(t.x, t.y, t.z, t.w));
        hi = max_f32(hi, quad_max(t.x, t.y, t.z, t.w));
    };
    const uint64_t pieces = nq / (4u * kSumThreads);
    for (uint64_t pc = block; pc < pieces; pc += nblocks) {
        const v4f_a4* __restrict__ src = g4 + pc * (4u * kSumThreads) + tid;
        v4f t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = __builtin_nontemporal_load(src + u * kSumThreads);
#pragma unroll
        for (int u = 0; u < 4; ++u) fold(t[u]);
    }
    for (uint64_t q = pieces * (4u * kSumThreads) + gtid; q < nq; q += stride) fold(__builtin_nontemporal_load(g4 + q));
    if (gtid < (n & 3u)) {
        const float v = g[(nq << 2) + gtid];
        lo = min_f32(lo, v);
        hi = max_f32(hi, v);
    }
    kl = order_key(lo);
    kh = order_key(hi);
    fold_keys<kSumThreads>(kl, kh, s_lo, s_hi);
}

// Range alone (two floats are all the memory there is): the workgroups meet in atomics on the two words.
__global__ __launch_bounds__(kSumThreads) void tensor_range_kernel(const float* __restrict__ g, const uint64_t n,
                                                                   uint32_t* keys) {
    drop_every_nan();
    __shared__ uint32_t s_lo[kSumThreads / 64], s_hi[kSumThreads / 64];
    uint32_t kl, kh;
    block_range(g, n, blockIdx.x, gridDim.x, kl, kh, s_lo, s_hi);
    if (threadIdx.x == 0u) fold_into(keys, kl, kh);
}

// Ranges of tensors that are about to be encoded: every workgroup leaves its keys at the front of the
// tensor's code words, which the encoder overwrites afterwards, and one workgroup per tensor folds them:
// no priming launch and no atomics (the encode of 8.8 M elements at 4 bits 15.5 us, 23.1 with atomics; the small CNN's two
// largest layers, 0.9 M elements in all, 4 us for the ranges, 14 with atomics).
// A tensor of one workgroup gets its range at once.
template <class Batch>
__global__ __launch_bounds__(kSumThreads) void tensor_range_parts_kernel(const Batch b) {
    drop_every_nan();
    __shared__ uint32_t s_lo[kSumThreads / 64], s_hi[kSumThreads / 64], s_keys[2];
    const uint32_t k = tensor_of_block(b.block_start, b.count, blockIdx.x);
    const uint32_t block = blockIdx.x - b.block_start[k], nblocks = b.block_start[k + 1u] - b.block_start[k];
    uint32_t kl, kh;
    block_range(b.grad[k], b.n[k], block, nblocks, kl, kh, s_lo, s_hi);
    if (b.in_slots != 0u && nblocks > 1u) {
        keys_to_slots(b.parts[k], b.n[k], b.bits, b.slots[k].borrowed, block, kl, kh, s_keys);
    } else if (threadIdx.x == 0u) {
        if (nblocks == 1u) {
            const float2 r = range_of_keys(kl, kh);
            b.range[k][0] = r.x;
            b.range[k][1] = r.y;
        } else {
            b.parts[k][2u * block] = kl;
            b.parts[k][2u * block + 1u] = kh;
        }
    }
}
constexpr int kFoldPartsThreads = 256;
template <class Batch>
__global__ __launch_bounds__(kFoldPartsThreads) void fold_parts_kernel(const Batch b) {
    __shared__ uint32_t s_lo[kFoldPartsThreads / 64], s_hi[kFoldPartsThreads / 64];
    const uint32_t k = blockIdx.x;
    const uint32_t parts = b.block_start[k + 1u] - b.block_start[k];
    if (parts < 2u) return;
    uint32_t kl = 0xFFFFFFFFu, kh = 0u;
    fold_pairs<kFoldPartsThreads, kSumBlocks / kFoldPartsThreads>(b.parts[k], parts, kl, kh);
    fold_keys<kFoldPartsThreads>(kl, kh, s_lo, s_hi);
    if (threadIdx.x == 0u) {
        const float2 r = range_of_keys(kl, kh);
        b.range[k][0] = r.x;
        b.range[k][1] = r.y;
    }
}

// ---- sum of squares -------------------------------------------------------------------------------
// Squares of fp32 values are exact in fp64; every lane adds its share in fp64, lanes and waves are
// combined by a butterfly and through LDS.  Two ways to finish: mqg_sum_squares adds one fp64 number
// per workgroup to *out with an atomic (its rounding depends on the order in which the workgroups
// arrive: about 1e-16 relative); the batched form stores one partial sum per workgroup and a second
// kernel adds them in a fixed order, which makes the result reproducible to the bit.

__global__ void clear_f64_kernel(double* out) { *out = 0.0; }

// The calling workgroup's share of sum g[i]^2 (workgroup `block` of `nblocks`); the value is returned
// in thread 0.  The order of every addition is a function of (n, nblocks) only.
__device__ __forceinline__ double block_sum_squares(const float* __restrict__ g, const uint64_t n, const uint32_t block,
                                                    const uint32_t nblocks, double* s_part) {
    const uint32_t tid = threadIdx.x;
    const uint64_t gtid = (uint64_t)block * kSumThreads + tid;
    const uint64_t stride = (uint64_t)nblocks * kSumThreads;
    double acc = 0.0;
    const v4f_a4* __restrict__ g4 = reinterpret_cast<const v4f_a4*>(g);   // 128-bit loads need dword alignment only
    const uint64_t nq = n >> 2;
    // a workgroup reads 32 KB contiguous pieces (four float4 per lane in flight), pieces nblocks apart
    const uint64_t pieces = nq / (4u * kSumThreads);
    for (uint64_t pc = block; pc < pieces; pc += nblocks) {
        const v4f_a4* __restrict__ src = g4 + pc * (4u * kSumThreads) + tid;
        v4f t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = __builtin_nontemporal_load(src + u * kSumThreads);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double a0 = (double)t[u].x, a1 = (double)t[u].y, a2 = (double)t[u].z, a3 = (double)t[u].w;
            acc += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
        }
    }
    for (uint64_t q = pieces * (4u * kSumThreads) + gtid; q < nq; q += stride) {   // less than one piece is left
        const v4f t = __builtin_nontemporal_load(g4 + q);
        const double a0 = (double)t.x, a1 = (double)t.y, a2 = (double)t.z, a3 = (double)t.w;
        acc += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
    }
    if (gtid < (n & 3u)) {
        const double v = (double)g[(nq << 2) + gtid];
        acc += v * v;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) acc += __shfl_xor(acc, m, 64);
    if ((tid & 63u) == 0u) s_part[tid >> 6] = acc;
    __syncthreads();
    double t = 0.0;
    if (tid == 0u) {
#pragma unroll
        for (int w = 0; w < kSumThreads / 64; ++w) t += s_part[w];
    }
    return t;
}

__global__ __launch_bounds__(kSumThreads) void sum_squares_kernel(const float* __restrict__ g, const uint64_t n,
                                                                  double* out) {
    __shared__ double s_part[kSumThreads / 64];
    const double t = block_sum_squares(g, n, blockIdx.x, gridDim.x, s_part);
    if (threadIdx.x == 0u) atomicAdd(out, t);
}

// Batched, ordered form.  blockIdx.y = tensor, blockIdx.x = workgroup of the tensor, of kSumBlocks; every workgroup
// stores its partial sum (0 for a workgroup that has nothing to read), nothing is accumulated in memory.  A launch leaves
// out the workgroups past the ones that any of its tensors fills (sum_blocks): 24 tensors of 65,536 elements 17.0 -> 4.4 us.
__global__ __launch_bounds__(kSumThreads) void sum_squares_partial_kernel(const SumSquaresBatch b, double* __restrict__ partials) {
    __shared__ double s_part[kSumThreads / 64];
    const uint32_t k = blockIdx.y;
    const double t = block_sum_squares(b.grad[k], b.n[k], blockIdx.x, kSumBlocks, s_part);
    if (threadIdx.x == 0u) partials[(uint64_t)k * kSumBlocks + blockIdx.x] = t;
}

// Workgroups of kSumBlocks that a tensor fills: block_sum_squares deals out whole pieces of 8192 elements, one each, and
// spreads what is left, less than a piece, over the lanes of the first four.
uint32_t sum_blocks(uint64_t n) {
    const uint64_t pieces = (n >> 2) / (4u * kSumThreads);
    return pieces < 4u ? 4u : (pieces > kSumBlocks ? kSumBlocks : (uint32_t)pieces);
}

// One wave per tensor: lane l adds partials l, l + 64, ... in that order, then the butterfly.  `blocks` of them were
// stored; the others are the 0 of a workgroup without elements, which no sum of squares notices.  All loads are in flight
// before the first addition: one after the other they took 2 us longer.
__global__ __launch_bounds__(64) void sum_squares_finish_kernel(const double* __restrict__ partials, const uint32_t blocks, double* __restrict__ out) {
    const double* __restrict__ p = partials + (uint64_t)blockIdx.x * kSumBlocks;
    double part[kSumBlocks / 64u];
#pragma unroll
    for (uint32_t i = 0; i < kSumBlocks / 64u; ++i) part[i] = 64u * i + threadIdx.x < blocks ? p[64u * i + threadIdx.x] : 0.0;
    double acc = 0.0;
#pragma unroll
    for (uint32_t i = 0; i < kSumBlocks / 64u; ++i) acc += part[i];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) acc += __shfl_xor(acc, m, 64);
    if (threadIdx.x == 0u) out[blockIdx.x] = acc;
}

// Calls f(straddle, once): whether a quad of this width can spill over its word, and whether the code words take
// streaming loads.
template <class F>
void with_codes(uint32_t bits, F f) {
    const bool straddle = (32u % bits) != 0u, once = decode::codes_read_once(bits);
    if (straddle && once) f(std::true_type{}, std::true_type{});
    else if (straddle) f(std::true_type{}, std::false_type{});
    else if (once) f(std::false_type{}, std::true_type{});
    else f(std::false_type{}, std::false_type{});
}

// Workgroup size of a bucket: 4 NT R elements with R = 4, so NT / 64 waves of 1024 elements.  Buckets of more than
// 4096 elements: one per workgroup, the fewest waves that hold it.  Smaller ones: four waves unless five, six or
// seven are filled at least a tenth better by whole buckets (powers of two fill four).  The exchange of 7 M
// elements, 4 workers, 4 bits: bucket 2304 (56 % of four waves, 90 % of five) 44.7 -> 35.4 us at 6 bits, 2752 40.0 ->
// 33.5, 4128 (half of a workgroup of 8192) 40.3 -> 34.1; 4064, which keeps its four waves, 35.9 -> 32.8.
uint32_t tile_waves(uint32_t bucket) {
    if (bucket > 4096u) return (bucket + 1023u) / 1024u;
    uint32_t nw = 4u;
    for (uint32_t w = 5u; w <= 7u; ++w) {   // used fractions, compared by cross-multiplication
        if (((w * 1024u) / bucket) * nw * 10u > ((nw * 1024u) / bucket) * w * 11u) nw = w;
    }
    return nw;
}
TileGeometry tile_geometry(uint32_t bucket, uint32_t waves) {
    const uint32_t buckets = (waves * 1024u) / bucket, cells = bucket / 32u;
    return {buckets * bucket, buckets, (65536u + cells - 1u) / cells};
}
TileGeometry tile_geometry(uint32_t bucket) { return tile_geometry(bucket, tile_waves(bucket)); }
// Calls f(NT, ONE) with the workgroup size as a compile-time constant.
template <class F>
void with_tile_waves(uint32_t bucket, uint32_t nw, F f) {
    using std::integral_constant;
    using several = std::false_type;
    using one = std::true_type;
    if (bucket <= 4096u) {
        switch (nw) {
            case 5: return f(integral_constant<int, 320>{}, several{});
            case 6: return f(integral_constant<int, 384>{}, several{});
            case 7: return f(integral_constant<int, 448>{}, several{});
            default: return f(integral_constant<int, 256>{}, several{});
        }
    }
    if (nw <= 6u) return f(integral_constant<int, 384>{}, one{});
    if (nw <= 8u) return f(integral_constant<int, 512>{}, one{});
    if (nw <= 12u) return f(integral_constant<int, 768>{}, one{});
    return f(integral_constant<int, 1024>{}, one{});
}

template <bool STRADDLE>
hipError_t launch_aggregate_s(const AggregateArgs& a, hipStream_t stream) {
    const uint64_t tiles = (a.n + kAggTile - 1) / kAggTile;
    if (tiles > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const dim3 grid((uint32_t)tiles), block(kThreads);
    const size_t lds = sizeof(float2) * a.W * kMaxBuckets;
    if (decode::codes_read_once(a.bits)) {
        hipLaunchKernelGGL((aggregate_update_minmax_kernel<STRADDLE, true>), grid, block, lds, stream, a);
    } else {
        hipLaunchKernelGGL((aggregate_update_minmax_kernel<STRADDLE, false>), grid, block, lds, stream, a);
    }
    return hipGetLastError();
}

}  // namespace

// ra.scales[w]: worker w's (min, max) pairs; ra.q.scales: (min, max) pairs of the mean
hipError_t launch_requantize_minmax(const RequantArgs& ra, hipStream_t stream) {
    if (ra.q.n == 0) return hipSuccess;
    if (requantize_minmax_cells_supported(ra)) return launch_requantize_minmax_cells(ra, stream);
    // Where every compute unit gets at most one workgroup, four waves of fewer buckets end sooner: bucket 2304, 24 workers,
    // 65,536 elements 9.6 us, with five waves 10.3; at 1 M elements 11.9 and 10.9.
    uint32_t waves = tile_waves(ra.q.bucket);
    if (ra.q.bucket <= 4096u && ra.W > 4u && (ra.q.n - 1u) / tile_geometry(ra.q.bucket, 4u).elems < kComputeUnits) waves = 4u;
    TileGeometry g = tile_geometry(ra.q.bucket, waves);
    const uint32_t max_nb = 4096u / ra.W;   // at most 4096 table entries (32 KB of LDS); >= 64
    if (g.buckets > max_nb) {
        g.buckets = max_nb;
        g.elems = max_nb * ra.q.bucket;
    }
    const uint64_t tiles = (ra.q.n + g.elems - 1) / g.elems;
    if (tiles > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const size_t lds = sizeof(float2) * ra.W * g.buckets;
    with_tile_waves(ra.q.bucket, waves, [&](auto nt, auto one) {
        constexpr int NT = decltype(nt)::value;
        constexpr bool ONE = decltype(one)::value;
        // Eight in flight up to two workgroups of four waves per compute unit (the time with eight / with four at 4 bits, 8
        // workers, bucket 1024: 0.90, 0.89, 0.95, 1.02 at 1, 2, 3, 5 M elements).  More of them come with buckets below 128
        // only; the larger shapes but those above 512 lanes (12320 at 1 M: 1.00) have at most one workgroup per compute unit.
        const bool many_tiles = NT == 256 && tiles > 2u * kComputeUnits;
        with_codes(ra.q.bits, [&](auto straddle, auto once) {
            const auto launch = [&](auto ch, auto many) {
                hipLaunchKernelGGL((requantize_minmax_kernel<NT, ONE, decltype(straddle)::value, decltype(once)::value, decltype(ch)::value, decltype(many)::value>),
                                   dim3((uint32_t)tiles), dim3(NT), lds, stream, ra, g);
            };
            using four = std::integral_constant<int, 4>;
            using eight = std::integral_constant<int, 8>;
            if (ra.W <= 4u) return launch(four{}, std::bool_constant<ONE>{});
            if constexpr (NT <= 512) {
                if (!many_tiles) return launch(eight{}, std::true_type{});
            }
            if constexpr (NT == 256 || NT > 512) launch(four{}, std::true_type{});
        });
    });
    return hipGetLastError();
}

// a.scales: 2 floats (min, max) per bucket; a.scale_mode, key, iteration, worker, elem_base unused
hipError_t launch_quantize_minmax(const QuantizeArgs& a, hipStream_t stream) {
    if (a.n == 0) return hipSuccess;
    if (quantize_minmax_wave_supported(a)) return launch_quantize_minmax_wave(a, stream);   // power-of-two buckets
    if (a.scales_in != nullptr) return hipErrorInvalidValue;   // a given range is tiled with a power-of-two bucket
    const TileGeometry g = tile_geometry(a.bucket);
    const uint64_t tiles = (a.n + g.elems - 1) / g.elems;
    if (tiles > 0x7FFFFFFFull) return hipErrorInvalidValue;
    with_tile_waves(a.bucket, tile_waves(a.bucket), [&](auto nt, auto one) {
        constexpr int NT = decltype(nt)::value;
        hipLaunchKernelGGL((quantize_minmax_kernel<4, NT, decltype(one)::value>), dim3((uint32_t)tiles), dim3(NT), 0, stream, a, g);
    });
    return hipGetLastError();
}

// The tile of the batched encoder.
uint32_t quantize_minmax_batch_tile(uint32_t bucket, int bucket_shift) {
    if (bucket_shift >= 5) return quantize_minmax_wave_block_elems(bucket);
    return tile_geometry(bucket).elems;
}

// a.t[i].scales: (min, max) pairs of tensor i's buckets; a.t[i].scales_in: nullptr, or the ONE (min, max)
// pair of tensor i (then nothing is written to scales and the bucket only shapes the launch: it must be
// a power of two)
hipError_t launch_quantize_minmax_tensors(const BatchQuantizeArgs& a, uint32_t tiles, hipStream_t stream) {
    if (tiles == 0) return hipSuccess;
    if (a.common.bucket_shift >= 5) return launch_quantize_minmax_tensors_wave(a, tiles, stream);
    const TileGeometry g = tile_geometry(a.common.bucket);
    with_tile_waves(a.common.bucket, tile_waves(a.common.bucket), [&](auto nt, auto one) {
        constexpr int NT = decltype(nt)::value;
        with_few(a, [&](const auto& batch) {
            hipLaunchKernelGGL((quantize_minmax_tensors_kernel<4, NT, decltype(one)::value, std::decay_t<decltype(batch)>>), dim3(tiles), dim3(NT), 0, stream, batch, g);
        });
    });
    return hipGetLastError();
}

// range[k][0..1] <- min, max of tensor k, whose encoder will overwrite parts[k].  One piece of block_range per
// workgroup, up to kSumBlocks of them: with 1024 the encode took up to 3 % more from 8.8 M elements on, 5 % at 1 G.
hipError_t launch_tensor_ranges(TensorRangeBatch& b, uint32_t count, hipStream_t stream) {
    constexpr uint64_t kPiece = 16u * kSumThreads;   // elements; 512 words at one bit: two for each workgroup's keys
    uint32_t blocks = 0;
    bool parts = false, fit = true;
    for (uint32_t k = 0; k < kMaxBatchTensors; ++k) {
        b.block_start[k] = blocks;
        b.slots[k] = RangeSlots{0u, 0u};
        if (k >= count || b.n[k] == 0) continue;
        const uint64_t most = b.n[k] / kPiece;
        const uint32_t mine = most < 1u ? 1u : (uint32_t)(most > kSumBlocks ? kSumBlocks : most);
        if (mine > 1u) {
            parts = true;
            b.slots[k] = range_slots(b.n[k], b.bits, mine);
            fit = fit && b.slots[k].parts != 0u;
        }
        blocks += mine;
    }
    b.in_slots = parts && fit ? 1u : 0u;
    b.block_start[kMaxBatchTensors] = blocks;
    if (blocks == 0) return hipSuccess;
    b.count = count;
    with_few(b, [&](const auto& batch) {
        using Batch = std::decay_t<decltype(batch)>;
        hipLaunchKernelGGL((tensor_range_parts_kernel<Batch>), dim3(blocks), dim3(kSumThreads), 0, stream, batch);
        if (parts && !fit) hipLaunchKernelGGL((fold_parts_kernel<Batch>), dim3(count), dim3(kFoldPartsThreads), 0, stream, batch);
    });
    return hipGetLastError();
}

// One range for the whole tensor (a.scales: 2 floats), then the encode over it.  A tensor that one
// workgroup of the encoder holds is one bucket: one launch.
hipError_t launch_quantize_minmax_tensor(const QuantizeArgs& a_in, hipStream_t stream) {
    if (a_in.n == 0) return hipSuccess;
    QuantizeArgs a = a_in;
    a.bucket = 1024u;            // the range is given: the bucket only shapes the launch
    a.bucket_shift = 10;
    if (a.n <= kOneBucketElems) {
        a.drop_nan = 1u;
        while (a.bucket < a.n) {
            a.bucket <<= 1;
            a.bucket_shift += 1;
        }
        return launch_quantize_minmax(a, stream);
    }
    TensorRangeBatch b = {};
    b.grad[0] = a.grad;
    b.n[0] = a.n;
    b.range[0] = a.scales;
    b.parts[0] = a.packed;
    b.bits = a.bits;
    const hipError_t e = launch_tensor_ranges(b, 1u, stream);
    if (e != hipSuccess) return e;
    if (b.in_slots != 0u) {
        a.parts = b.slots[0].parts;
        a.borrowed = b.slots[0].borrowed;
    } else {
        a.scales_in = a.scales;
        a.scales = nullptr;      // not written when the range is given
    }
    return launch_quantize_minmax(a, stream);
}

uint32_t aggregate_minmax_batch_tile() { return kAggTile; }

// a.ptrs: per encoded tensor [W packed][W range arrays], per raw tensor [W fp32 gradients]
hipError_t launch_aggregate_minmax_tensors(const BatchAggregateArgs& a, uint32_t tiles, hipStream_t stream) {
    if (tiles == 0) return hipSuccess;
    const size_t lds = sizeof(float2) * a.W * kMaxBuckets;
    with_codes(a.bits, [&](auto straddle, auto once) {
        with_few(a, [&](const auto& batch) {
            hipLaunchKernelGGL((aggregate_update_minmax_tensors_kernel<decltype(straddle)::value, decltype(once)::value, std::decay_t<decltype(batch)>>),
                               dim3(tiles), dim3(kThreads), lds, stream, batch);
        });
    });
    return hipGetLastError();
}

// a.scales[w]: worker w's (min, max) pairs
hipError_t launch_aggregate_minmax(const AggregateArgs& a, hipStream_t stream) {
    if (a.n == 0) return hipSuccess;
    const bool straddle = (32u % a.bits) != 0u;
    return straddle ? launch_aggregate_s<true>(a, stream) : launch_aggregate_s<false>(a, stream);
}

// ra.scales[w]: worker w's one (min, max) pair; ra.q.scales: the (min, max) pair of the mean (2 floats).
// Pass 1, the fold, pass 2; a tensor that one workgroup holds is one bucket of the bucketed step: one launch.
hipError_t launch_requantize_minmax_tensor(const RequantArgs& ra_in, hipStream_t stream) {
    if (ra_in.q.n == 0) return hipSuccess;
    constexpr int NT = kSumTileThreads;
    if (ra_in.q.n <= kOneBucketElems) {
        RequantArgs one = ra_in;
        one.q.bucket = 4096u;
        one.q.bucket_shift = 12;
        one.q.drop_nan = 1u;
        while (one.q.bucket < one.q.n) {
            one.q.bucket <<= 1;
            one.q.bucket_shift += 1;
        }
        return launch_requantize_minmax(one, stream);
    }
    const bool cells = tensor_cells_supported(ra_in);
    const uint32_t tile = cells ? tensor_cells_tile() : kSumTile;
    const uint64_t tiles = (ra_in.q.n + tile - 1) / tile;
    if (tiles > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const uint64_t words = (ra_in.q.n >> 5) * ra_in.q.bits + (((ra_in.q.n & 31u) * ra_in.q.bits + 31u) >> 5);
    bool atomics = tiles > kMostFoldedTiles;
    for (uint32_t w = 0; w < ra_in.W; ++w) {
        const uint64_t in = reinterpret_cast<uintptr_t>(ra_in.packed[w]), out = reinterpret_cast<uintptr_t>(ra_in.q.packed);
        atomics = atomics || (in < out + 4u * words && out < in + 4u * words);
    }
    const uint64_t tail = ra_in.q.n % tile;
    // small tensors: every workgroup of the second pass folds the keys itself
    RequantArgs ra = ra_in;
    const RangeSlots slots = cells || atomics ? RangeSlots{0u, 0u} : range_slots(ra.q.n, ra.q.bits, tiles);
    ra.q.parts = slots.parts;
    ra.q.borrowed = slots.borrowed;
    const uint32_t borrowed = slots.parts != 0u ? slots.borrowed
                              : !atomics && tail != 0 && tail * ra.q.bits <= 32u ? 64u : 0u;   // 64 elements are two words at one bit
    uint32_t* keys = atomics ? reinterpret_cast<uint32_t*>(ra.q.scales) : nullptr;
    const float* sum_range = atomics ? ra.q.scales : nullptr;
    const dim3 grid((uint32_t)tiles), block(NT);
    if (atomics) hipLaunchKernelGGL(range_init_kernel, dim3(1), dim3(1), 0, stream, keys);
    if (cells) {
        launch_sum_range_cells(ra, (uint32_t)tiles, tile, keys, stream);
    } else {
        with_codes(ra.q.bits, [&](auto straddle, auto once) {
            hipLaunchKernelGGL((sum_range_minmax_tensor_kernel<NT, decltype(straddle)::value, decltype(once)::value>), grid, block, 0, stream, ra, keys);
        });
    }
    if (atomics) {
        hipLaunchKernelGGL(range_finish_kernel, dim3(1), dim3(1), 0, stream, keys);
    } else if (ra.q.parts == 0u) {
        hipLaunchKernelGGL(fold_sum_range_kernel, dim3(1), dim3(kFoldThreads), 0, stream, ra.q.packed, (uint32_t)tiles, tile,
                           borrowed, ra.q.bits, ra.q.scales, (float)ra.W);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (cells) {
        launch_requantize_tensor_cells(ra, (uint32_t)tiles, tile, sum_range, borrowed, stream);
    } else {
        with_codes(ra.q.bits, [&](auto straddle, auto once) {
            hipLaunchKernelGGL((requantize_minmax_tensor_kernel<NT, decltype(straddle)::value, decltype(once)::value>), grid, block, 0, stream, ra,
                               sum_range, borrowed);
        });
    }
    if (atomics) hipLaunchKernelGGL(range_divide_kernel, dim3(1), dim3(1), 0, stream, ra.q.scales, (float)ra.W);
    return hipGetLastError();
}

hipError_t launch_tensor_range(const float* grad, uint64_t n, float* range_out, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    uint32_t* keys = reinterpret_cast<uint32_t*>(range_out);
    hipLaunchKernelGGL(range_init_kernel, dim3(1), dim3(1), 0, stream, keys);
    uint64_t blocks = ((n >> 2) + kSumThreads - 1) / kSumThreads;
    if (blocks < 1) blocks = 1;
    if (blocks > kSumBlocks) blocks = kSumBlocks;
    hipLaunchKernelGGL(tensor_range_kernel, dim3((uint32_t)blocks), dim3(kSumThreads), 0, stream, grad, n, keys);
    hipLaunchKernelGGL(range_finish_kernel, dim3(1), dim3(1), 0, stream, keys);
    return hipGetLastError();
}
uint32_t sum_squares_batch_blocks() { return kSumBlocks; }

// partials: count * kSumBlocks doubles of scratch memory; out: count doubles
hipError_t launch_sum_squares_batch(const SumSquaresBatch& b, uint32_t count, double* partials, double* out, hipStream_t stream) {
    if (count == 0) return hipSuccess;
    uint32_t blocks = 0;
    for (uint32_t k = 0; k < count; ++k) blocks = sum_blocks(b.n[k]) > blocks ? sum_blocks(b.n[k]) : blocks;
    hipLaunchKernelGGL(sum_squares_partial_kernel, dim3(blocks, count), dim3(kSumThreads), 0, stream, b, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sum_squares_finish_kernel, dim3(count), dim3(64), 0, stream, partials, blocks, out);
    return hipGetLastError();
}

// ---- the same with the partial sums in memory that the library itself holds ------------------------
// For callers that cannot allocate (code under graph capture, serving loops): a file-scope device array
// takes the place of the workspace.  Every GPU the library runs on holds its own copy of the array, at
// its own address, until the process ends; the array's name is a host-side handle, not a device address,
// so the address is asked for once per device (with that device current) and kept.
constexpr int kMaxDevices = 64;
static __device__ __align__(256) double scratch[kMaxSumTensors * kSumBlocks];   // 256 KB per GPU

static std::mutex g_scratch_mutex;
static double* g_scratch_ptr[kMaxDevices];   // per device; nullptr until first use on that device

static hipError_t static_scratch(double** ptr) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        double* p = nullptr;
        e = hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (p == nullptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

// No allocation anywhere on this path; the partial sums are all overwritten before they are read, so
// nothing has to be cleared between calls.
hipError_t launch_sum_squares_batch_static(const SumSquaresBatch& b, uint32_t count, double* out, hipStream_t stream) {
    if (count == 0) return hipSuccess;
    if (count > kMaxSumTensors) return hipErrorInvalidValue;
    double* partials = nullptr;
    const hipError_t e = static_scratch(&partials);
    if (e != hipSuccess) return e;
    return launch_sum_squares_batch(b, count, partials, out, stream);
}

hipError_t launch_sum_squares(const float* grad, uint64_t n, double* out, hipStream_t stream) {
    hipLaunchKernelGGL(clear_f64_kernel, dim3(1), dim3(1), 0, stream, out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n == 0) return e;
    uint64_t blocks = ((n >> 2) + kSumThreads - 1) / kSumThreads;
    if (blocks < 1) blocks = 1;
    if (blocks > kSumBlocks) blocks = kSumBlocks;
    hipLaunchKernelGGL(sum_squares_kernel, dim3((uint32_t)blocks), dim3(kSumThreads), 0, stream, grad, n, out);
    return hipGetLastError();
}

}  // namespace mqg
