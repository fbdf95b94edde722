// The server's re-encoding steps of the full exchange (ReceiveQGThenSendQG of Algorithm 1), one cell per lane: the W
// workers' code streams are decoded, added in worker order and encoded again.  Code words are all that these steps
// read or write -- the sum exists in registers only -- so a lane can own a CELL's worth of codes, 32 elements, which
// is `bits` whole words at every width:
//   - a wave's loads of one worker's codes are 64 * bits consecutive words, up to 128 bits per lane and load, and
//     nothing is fetched twice;
//   - the width is a compile-time number, so every code's place in its word is one too;
//   - a lane packs its own words: no staging of the output, no LDS atomics;
//   - buckets are whole cells, so a lane has one step per worker and one range, and a Philox call's eight elements lie
//     in one lane.
// The kernels of quantize_wave.hip and minmax.hip that decode into the layout of fp32 rows (four elements per lane) load
// each code word in up to eight lanes, pack through LDS and, below 5 bits, were bound by LDS gathers.

#include "encode.h"
#include "kernels.h"

#include <type_traits>

namespace mqg {
namespace {

using namespace encode;

constexpr uint32_t kCell = 32;          // elements

// How much there is to do.  kShort: the launch does not fill the chip several times over, and what counts is a wave's own
// chain and how many compute units have a wave: small tiles, many words in flight.  kStream: the streams together exceed
// the last-level cache by so much that streaming loads are faster (size_of).
enum class Size { kShort, kLong, kStream };

typedef float v2f __attribute__((ext_vector_type(2)));
typedef v2u v2u_a4 __attribute__((aligned(4)));

// ---- a lane's words -----------------------------------------------------------------------------------
// At 6 and 8 bits a lane holds two half cells, 64 half cells apart: with whole ones its loads would lie 24 or 32 bytes
// apart, and the second half of each cache line be fetched again.
template <int B>
struct Parts {
    static constexpr int kCount = B == 6 || B == 8 ? 2 : 1;
    static constexpr int kWords = B / kCount;
    static constexpr int kElems = 32 / kCount;
};

template <int N, bool NT>
__device__ __forceinline__ void load_words(const uint32_t* p, uint32_t* w) {
    if constexpr (N >= 4) {
        const v4u_a4* q = reinterpret_cast<const v4u_a4*>(p);
        const v4u t = NT ? __builtin_nontemporal_load(q) : *q;
        w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
        if constexpr (N > 4) load_words<N - 4, NT>(p + 4, w + 4);
    } else if constexpr (N >= 2) {
        const v2u_a4* q = reinterpret_cast<const v2u_a4*>(p);
        const v2u t = NT ? __builtin_nontemporal_load(q) : *q;
        w[0] = t.x; w[1] = t.y;
        if constexpr (N > 2) load_words<N - 2, NT>(p + 2, w + 2);
    } else {
        w[0] = NT ? __builtin_nontemporal_load(p) : *p;
    }
}
// AGENT: written through to memory at once, the line stays in L2 (store_v4u_agent and store_u32_agent); else streaming.
template <int N, bool AGENT>
__device__ __forceinline__ void store_words(uint32_t* p, const uint32_t* w) {
    if constexpr (N >= 4) {
        const v4u t = {w[0], w[1], w[2], w[3]};
        if (AGENT) store_v4u_agent(p, t);
        else __builtin_nontemporal_store(t, reinterpret_cast<v4u_a4*>(p));
        if constexpr (N > 4) store_words<N - 4, AGENT>(p + 4, w + 4);
    } else if constexpr (N >= 2) {
        const v2u t = {w[0], w[1]};
        if (AGENT) store_v2u_agent(p, t);
        else __builtin_nontemporal_store(t, reinterpret_cast<v2u_a4*>(p));
        if constexpr (N > 2) store_words<N - 2, AGENT>(p + 2, w + 2);
    } else {
        if (AGENT) store_u32_agent(p, w[0]);
        else __builtin_nontemporal_store(w[0], p);
    }
}

// Where the lane's parts sit in a tile of `cells` cells (lanes past the last cell stand in for it: they read what it
// reads and write nothing) that starts at element tile_base and ends at tile_end.
template <int B>
struct Window {
    static constexpr int P = Parts<B>::kCount;
    uint64_t tile_word;    // the tile's first word in every stream
    uint32_t word[P];      // first word of the part, from there
    int from[P];           // the part's words are read from here, so that no load leaves the stream (at least kWords long)
    uint32_t cell[P];      // cell of the tile
    uint32_t count[P];     // elements of the part that are the lane's to write

    __device__ __forceinline__ Window(const uint64_t n, const uint64_t tile_base, const uint64_t tile_end, const uint32_t cells) {
        const uint32_t tid = threadIdx.x;
        tile_word = (tile_base >> 5) * B;
        const uint64_t words = (n >> 5) * B + (((n & 31u) * B + 31u) >> 5);
        const uint64_t room = words - tile_word;
        const int last = (int)(room > 0x3FFFFFFFull ? 0x3FFFFFFFu : (uint32_t)room) - Parts<B>::kWords;   // may lie before the tile
        const uint32_t elems = (uint32_t)(tile_end - tile_base);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const uint32_t mine = P == 1 ? tid : (tid >> 6) * 128u + p * 64u + (tid & 63u);
            const uint32_t u = mine < cells * P ? mine : cells * P - 1u;
            word[p] = u * Parts<B>::kWords;
            from[p] = (int)word[p] < last ? (int)word[p] : last;
            cell[p] = u / P;
            const uint32_t el = u * Parts<B>::kElems;
            const uint32_t left = el < elems ? elems - el : 0u;
            count[p] = mine != u ? 0u : (left < (uint32_t)Parts<B>::kElems ? left : (uint32_t)Parts<B>::kElems);
        }
    }
};
template <int B, Size SIZE, bool WHOLE>
__device__ __forceinline__ void fetch(const uint32_t* stream, const Window<B>& at, uint32_t (&w)[B]) {
    constexpr int PW = Parts<B>::kWords;
    const uint32_t* __restrict__ tile = stream + at.tile_word;
#pragma unroll
    for (int p = 0; p < Parts<B>::kCount; ++p) {
        if (WHOLE) load_words<PW, SIZE == Size::kStream>(tile + at.word[p], w + p * PW);
        else load_words<PW, SIZE == Size::kStream>(tile + at.from[p], w + p * PW);
    }
}
// the words of a part that was read from before its first one, in their places (past the end of the stream: any)
template <int B>
__device__ __forceinline__ void settle(const Window<B>& at, const uint32_t (&w)[B], uint32_t (&o)[B]) {
    constexpr int PW = Parts<B>::kWords;
#pragma unroll
    for (int p = 0; p < Parts<B>::kCount; ++p) {
        const uint32_t by = (uint32_t)((int)at.word[p] - at.from[p]);
#pragma unroll
        for (int i = 0; i < PW; ++i) o[p * PW + i] = w[p * PW + i];
        const auto down = [&](auto by_words) {
            constexpr int D = decltype(by_words)::value;
#pragma unroll
            for (int i = 0; i + D < PW; ++i) {
                const uint32_t here = o[p * PW + i], there = o[p * PW + i + D];
                o[p * PW + i] = (by & D) != 0u ? there : here;
            }
        };
        if constexpr (PW > 1) down(std::integral_constant<int, 1>{});
        if constexpr (PW > 2) down(std::integral_constant<int, 2>{});
        if constexpr (PW > 4) down(std::integral_constant<int, 4>{});
    }
}

// ---- decode -------------------------------------------------------------------------------------------
// Constants that stay in vector registers: with a scalar operand an fma, add or and issues at half the rate.
__device__ __forceinline__ float in_vector(float f) {
    asm volatile("" : "+v"(f));
    return f;
}
__device__ __forceinline__ uint32_t in_vector(uint32_t u) {
    asm volatile("" : "+v"(u));
    return u;
}

// Calls f(k, c) for the lane's codes, c = TIMES * code as fp32 (exact; TIMES is a power of two).
// 1, 2, 4 bits: a mask and a shift put every (8 / B)-th code of a word into a byte of its own, and the byte read as a
// FP8 number (E4M3: 0 .. 15 are the multiples of 2^-9 up to 15 * 2^-9) converts two at a time.
// 8 bits: a byte converts in one instruction.  Others: bit field, convert.
template <int B, class F>
__device__ __forceinline__ void for_codes(const uint32_t (&w)[B], const uint32_t byte_mask, const float scale, F f) {
    if constexpr (B == 1 || B == 2 || B == 4) {
        constexpr int PER = 8 / B;       // codes per byte
#pragma unroll
        for (int i = 0; i < B; ++i) {
#pragma unroll
            for (int s = 0; s < PER; ++s) {
                const uint32_t t = (s == 0 ? w[i] : (w[i] >> (s * B))) & byte_mask;
                const v2f lo = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(t, scale, false);
                const v2f hi = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(t, scale, true);
                const int k = i * (32 / B) + s;
                f(k, lo.x);
                f(k + PER, lo.y);
                f(k + 2 * PER, hi.x);
                f(k + 3 * PER, hi.y);
            }
        }
    } else {
#pragma unroll
        for (int k = 0; k < 32; ++k) {
            constexpr uint32_t kMask = (1u << B) - 1u;
            const int i = k * B / 32, sh = k * B % 32;
            uint32_t c;
            if (sh + B > 32) c = __builtin_amdgcn_alignbit(w[i + 1 < B ? i + 1 : i], w[i], sh) & kMask;
            else if (sh + B == 32) c = w[i] >> sh;
            else c = __builtin_amdgcn_ubfe(w[i], sh, B);
            f(k, (float)c);
        }
    }
}
template <int B>
__device__ __forceinline__ uint32_t byte_mask() {
    return in_vector(((1u << B) - 1u) * 0x01010101u);
}

// What adds one worker's codes to the sum's values.
struct MinmaxSum {   // acc <- acc + fma(c, step, min)
    using Step = float2;
    static __device__ __forceinline__ Step step(const float* ranges, const uint64_t k, const float Lf) {
        const float2 rg = reinterpret_cast<const float2*>(ranges)[k];   // (min, max)
        return make_float2((rg.y - rg.x) / Lf, rg.x);                   // IEEE-correct fp32 division
    }
    template <int B>
    struct Consts {
        uint32_t mask;
        float scale;
        __device__ __forceinline__ Consts() : mask(byte_mask<B>()), scale(in_vector(0x1p9f)) {}
    };
    template <int B>
    static __device__ __forceinline__ void add(const uint32_t (&w)[B], const Consts<B>& k, const Step (&s)[Parts<B>::kCount], float (&v)[32]) {
        for_codes<B>(w, k.mask, k.scale, [&](int i, float c) {
            const Step& sm = s[i / Parts<B>::kElems];
            v[i] = v[i] + __builtin_fmaf(c, sm.x, sm.y);
        });
    }
};
struct CentredSum {   // acc <- fma(2c - L, step, acc)
    using Step = float;
    static __device__ __forceinline__ Step step(const float* scales, const uint64_t k, const float Lf) { return scales[k] / Lf; }
    template <int B>
    struct Consts {
        uint32_t mask;
        float scale, minus_top;
        __device__ __forceinline__ Consts()
            : mask(byte_mask<B>()), scale(in_vector(0x1p10f)), minus_top(in_vector(-(float)((1 << B) - 1))) {}
    };
    template <int B>
    static __device__ __forceinline__ void add(const uint32_t (&w)[B], const Consts<B>& k, const Step (&s)[Parts<B>::kCount], float (&v)[32]) {
        for_codes<B>(w, k.mask, k.scale, [&](int i, float c) {
            const float centred = B == 1 || B == 2 || B == 4 ? c + k.minus_top : __builtin_fmaf(c, 2.0f, k.minus_top);   // there c is twice the code
            v[i] = __builtin_fmaf(centred, s[i / Parts<B>::kElems], v[i]);
        });
    }
};

// Workers whose code words are in flight together: as soon as a worker's words are decoded, those of the worker
// in_flight places on are requested in their stead.
template <int B, Size SIZE>
constexpr int in_flight() { return SIZE == Size::kShort ? (B <= 4 ? 8 : 5) : (B == 1 ? 8 : B == 2 ? 4 : 2); }

// v <- the sum over the W workers, in worker order.  table[w * stride + bucket]: worker w's step in the bucket of each
// of the lane's parts; complete after the barrier in here.
template <int B, Size SIZE, bool WHOLE, class Sum>
__device__ __forceinline__ void decode_sum(const RequantArgs& ra, const Window<B>& at, const typename Sum::Step* table, const uint32_t stride,
                                           const uint32_t (&bucket)[Parts<B>::kCount], float (&v)[32]) {
    constexpr int CH = in_flight<B, SIZE>();
    const uint32_t W = ra.W;
    uint32_t c[CH][B];
#pragma unroll
    for (int t = 0; t < CH; ++t) fetch<B, SIZE, WHOLE>(ra.packed[(uint32_t)t < W ? t : W - 1u], at, c[t]);
    const typename Sum::template Consts<B> k;
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = 0.0f;
    __syncthreads();
    const auto add = [&](const uint32_t w, const uint32_t (&words)[B]) {
        typename Sum::Step s[Parts<B>::kCount];
#pragma unroll
        for (int p = 0; p < Parts<B>::kCount; ++p) s[p] = table[w * stride + bucket[p]];
        if constexpr (WHOLE) {
            Sum::template add<B>(words, k, s, v);
        } else {
            uint32_t settled[B];
            settle<B>(at, words, settled);
            Sum::template add<B>(settled, k, s, v);
        }
    };
    uint32_t w0 = 0;
    for (; w0 + CH < W; w0 += CH) {
#pragma unroll
        for (int t = 0; t < CH; ++t) {
            add(w0 + t, c[t]);
            const uint32_t next = w0 + CH + t;
            fetch<B, SIZE, WHOLE>(ra.packed[next < W ? next : W - 1u], at, c[t]);
            __builtin_amdgcn_sched_barrier(0);   // left alone the compiler converts several workers' codes ahead and spills
        }
    }
#pragma unroll
    for (int t = 0; t < CH; ++t) {
        if (w0 + t < W) add(w0 + t, c[t]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// ---- encode -------------------------------------------------------------------------------------------
// bits [k * B, k * B + 32) of the lane's words <- v, which has no bit past the last code it holds
template <int B>
__device__ __forceinline__ void place(uint32_t (&o)[B], const int k, const uint32_t v, const int codes) {
    const int i = k * B / 32, sh = k * B % 32;
    o[i] = sh == 0 ? v : (o[i] | v << sh);
    if (sh + codes * B > 32) o[i + 1 < B ? i + 1 : i] = v >> (32 - sh);
}
template <int B, bool WHOLE, bool AGENT>
__device__ __forceinline__ void store_parts(uint32_t* __restrict__ out, const Window<B>& at, const uint32_t (&o)[B]) {
    constexpr int PW = Parts<B>::kWords;
#pragma unroll
    for (int p = 0; p < Parts<B>::kCount; ++p) {
        uint32_t* __restrict__ dst = out + at.tile_word + at.word[p];
        if (WHOLE) {
            if (at.count[p] != 0u) store_words<PW, AGENT>(dst, o + p * PW);
        } else {
            const uint32_t words = (at.count[p] * B + 31u) >> 5;
#pragma unroll
            for (int i = 0; i < PW; ++i) {
                if ((uint32_t)i < words) store_words<1, AGENT>(dst + i, o + p * PW + i);
            }
        }
    }
}
// is the lane's element k inside the tensor?
template <int B, bool WHOLE>
__device__ __forceinline__ bool inside(const Window<B>& at, const int k) {
    return WHOLE || (uint32_t)(k % Parts<B>::kElems) < at.count[k / Parts<B>::kElems];
}

template <int B, bool WHOLE>
__device__ __forceinline__ void encode_minmax(uint32_t* out, const Window<B>& at, const float (&v)[32], const float (&mn)[Parts<B>::kCount],
                                              const float (&a)[Parts<B>::kCount]) {
    const float Lf = (float)((1 << B) - 1);
    uint32_t o[B];
#pragma unroll
    for (int k = 0; k < 32; ++k) {
        const int p = k / Parts<B>::kElems;
        const uint32_t code = nearest_code(v[k], mn[p], a[p], Lf);
        place<B>(o, k, inside<B, WHOLE>(at, k) ? code : 0u, 1);   // elements past the end contribute zero bits
    }
    store_parts<B, WHOLE, false>(out, at, o);
}
__device__ __forceinline__ float inverse_step(float mn, float mx, float Lf) {
    const float r = mx - mn;
    return (r >= 0x1p-96f) ? Lf / r : 0.0f;   // IEEE-correct fp32 division
}

// Extremes of each part's values; elements past the end take no part (none at all: +inf, -inf), nor does a NaN unless the part
// holds nothing else.  (The rows kernels: unless a quad does.  Sums that are partly not numbers have no specified range.)
template <int B, bool WHOLE>
__device__ __forceinline__ void part_ranges(const float (&v)[32], const Window<B>& at, float (&lo)[Parts<B>::kCount], float (&hi)[Parts<B>::kCount]) {
    constexpr int E = Parts<B>::kElems;
    const float inf = __builtin_inff();
#pragma unroll
    for (int p = 0; p < Parts<B>::kCount; ++p) {
        const int f = p * E;
        lo[p] = inside<B, WHOLE>(at, f) ? v[f] : inf;
        hi[p] = inside<B, WHOLE>(at, f) ? v[f] : -inf;
#pragma unroll
        for (int k = f + 1; k < f + E; ++k) {
            if (WHOLE) {
                if (k + 1 < f + E && ((k - f) & 1)) {
                    asm("v_min3_f32 %0, %1, %2, %0" : "+v"(lo[p]) : "v"(v[k]), "v"(v[k + 1 < 32 ? k + 1 : k]));
                    asm("v_max3_f32 %0, %1, %2, %0" : "+v"(hi[p]) : "v"(v[k]), "v"(v[k + 1 < 32 ? k + 1 : k]));
                } else if ((k - f) & 1) {
                    lo[p] = min_f32(lo[p], v[k]);
                    hi[p] = max_f32(hi[p], v[k]);
                }
            } else {
                lo[p] = min_f32(lo[p], inside<B, WHOLE>(at, k) ? v[k] : inf);
                hi[p] = max_f32(hi[p], inside<B, WHOLE>(at, k) ? v[k] : -inf);
            }
        }
    }
}

// ---- one [min, max] range for the whole tensor ------------------------------------------------------------
// Two passes over the streams, as the range of the sum is known only at the end of the first (see
// launch_requantize_minmax_tensor for where the keys and the range live in between).
__device__ __forceinline__ void fill_tensor_table(const RequantArgs& ra, const float Lf, float2* s_tab) {
    for (uint32_t w = threadIdx.x; w < ra.W; w += blockDim.x) s_tab[w] = MinmaxSum::step(ra.scales[w], 0u, Lf);
}

template <int B, Size SIZE, bool WHOLE>
__device__ __forceinline__ void sum_range_tile(const RequantArgs& ra, uint32_t* keys, const uint64_t tile_base, float2* s_tab,
                                               uint32_t* s_lo, uint32_t* s_hi) {
    const uint32_t tid = threadIdx.x;
    const Window<B> at(ra.q.n, tile_base, WHOLE ? tile_base + blockDim.x * kCell : ra.q.n, blockDim.x);
    fill_tensor_table(ra, (float)((1 << B) - 1), s_tab);
    float v[32], lo[Parts<B>::kCount], hi[Parts<B>::kCount];
    const uint32_t bucket[Parts<B>::kCount] = {};
    decode_sum<B, SIZE, WHOLE, MinmaxSum>(ra, at, s_tab, 1u, bucket, v);
    part_ranges<B, WHOLE>(v, at, lo, hi);
    float l = __builtin_inff(), h = -__builtin_inff();   // a NaN has no part in a tensor's range, whatever the lane holds
#pragma unroll
    for (int p = 0; p < Parts<B>::kCount; ++p) {
        l = min_f32(l, lo[p]);
        h = max_f32(h, hi[p]);
    }
    uint32_t kl = wave_min_from_cells_u32(cell_min_u32(order_key(l)), tid & 63u);
    uint32_t kh = wave_max_from_cells_u32(cell_max_u32(order_key(h)), tid & 63u);
    if ((tid & 63u) == 0u) {
        s_lo[tid >> 6] = kl;
        s_hi[tid >> 6] = kh;
    }
    __syncthreads();
    if (tid == 0u) {
        for (uint32_t w = 1; w < blockDim.x / 64u; ++w) {
            kl = min(kl, s_lo[w]);
            kh = max(kh, s_hi[w]);
        }
        if (keys != nullptr) {   // look first: same-address atomics serialize, and the keys only ever move one way
            if (kl < __atomic_load_n(&keys[0], __ATOMIC_RELAXED)) atomicMin(&keys[0], kl);
            if (kh > __atomic_load_n(&keys[1], __ATOMIC_RELAXED)) atomicMax(&keys[1], kh);
        } else {
            ra.q.packed[2u * blockIdx.x] = kl;
            ra.q.packed[2u * blockIdx.x + 1u] = kh;
        }
    }
}
template <int B, Size SIZE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 8))) void sum_range_cells_kernel(const RequantArgs ra, uint32_t* keys) {
    __shared__ float2 s_tab[MQG_MAX_WORKERS];
    __shared__ uint32_t s_lo[4], s_hi[4];
    const uint64_t tile_base = (uint64_t)blockIdx.x * (blockDim.x * kCell);
    if (tile_base + blockDim.x * kCell <= ra.q.n) sum_range_tile<B, SIZE, true>(ra, keys, tile_base, s_tab, s_lo, s_hi);
    else sum_range_tile<B, SIZE, false>(ra, keys, tile_base, s_tab, s_lo, s_hi);
}

template <int B, Size SIZE, bool WHOLE>
__device__ __forceinline__ void requantize_tensor_tile(const RequantArgs& ra, const float* sum_range, const uint64_t tile_base,
                                                       const uint64_t tile_end, float2* s_tab) {
    constexpr int P = Parts<B>::kCount;
    const float Lf = (float)((1 << B) - 1);
    const Window<B> at(ra.q.n, tile_base, tile_end, blockDim.x);
    // every lane holds the sum's range before the barrier in decode_sum; the words are overwritten after it
    const float* slot = sum_range != nullptr ? sum_range : reinterpret_cast<const float*>(ra.q.packed + at.tile_word);
    const float lowest = in_vector(slot[0]), highest = in_vector(slot[1]);
    fill_tensor_table(ra, Lf, s_tab);
    float v[32];
    const uint32_t bucket[P] = {};
    decode_sum<B, SIZE, WHOLE, MinmaxSum>(ra, at, s_tab, 1u, bucket, v);
    float mn[P], a[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        mn[p] = lowest;
        a[p] = inverse_step(lowest, highest, Lf);
    }
    encode_minmax<B, WHOLE>(ra.q.packed, at, v, mn, a);
}
template <int B, Size SIZE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 8))) void requantize_tensor_cells_kernel(const RequantArgs ra, const float* sum_range, const uint32_t borrowed) {
    __shared__ float2 s_tab[MQG_MAX_WORKERS];
    const uint32_t tile = blockDim.x * kCell;
    const bool last = blockIdx.x + 1u == gridDim.x;
    const uint64_t tile_base = (uint64_t)blockIdx.x * tile - (last ? borrowed : 0u);
    const uint64_t tile_end = last ? ra.q.n : (uint64_t)(blockIdx.x + 1u) * tile - (blockIdx.x + 2u == gridDim.x ? borrowed : 0u);
    if (tile_end - tile_base == tile) requantize_tensor_tile<B, SIZE, true>(ra, sum_range, tile_base, tile_end, s_tab);
    else requantize_tensor_tile<B, SIZE, false>(ra, sum_range, tile_base, tile_end, s_tab);
}

// ---- one range per bucket ------------------------------------------------------------------------------------
// A workgroup owns a tile of whole buckets.  LOCAL: a bucket is 1, 2, 4 .. 64 cells and a wave holds whole ones, so its
// range stays in the wave; otherwise the waves' shares of a bucket meet in one LDS slot behind a barrier.
struct CellTile {
    uint32_t cells, buckets;   // of a tile
    uint32_t bucket_cells;     // bucket / 32
    uint32_t magic;            // ceil(2^20 / bucket_cells)
};
__device__ __forceinline__ uint32_t bucket_of_cell(const CellTile& g, const uint32_t cell) {   // cell / bucket_cells, below 512 cells
    return (cell * g.magic) >> 20;
}
constexpr uint32_t kMostLanes = 512;                      // the largest bucket is 512 cells
constexpr uint32_t kMostSharedBuckets = kMostLanes / 3;   // buckets of a tile that is not LOCAL: at least three cells each

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v) {   // lanes without a source read 0
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
// Maximum over each group of 2^k neighbouring lanes that a bucket is (LOCAL); every lane of the group gets it.
template <int N>
__device__ __forceinline__ void group_max(uint32_t (&m)[N], const uint32_t lanes, const uint32_t lane) {
    if (lanes >= 2u) {
#pragma unroll
        for (int i = 0; i < N; ++i) m[i] = max(m[i], dpp_u32<kDppQuadSwap1>(m[i]));
    }
    if (lanes >= 4u) {
#pragma unroll
        for (int i = 0; i < N; ++i) m[i] = max(m[i], dpp_u32<kDppQuadSwap2>(m[i]));
    }
    if (lanes >= 8u) {
#pragma unroll
        for (int i = 0; i < N; ++i) m[i] = max(m[i], dpp_u32<kDppRowHalfMirror>(m[i]));
    }
    if (lanes >= 16u) {
#pragma unroll
        for (int i = 0; i < N; ++i) m[i] = max(m[i], dpp_u32<kDppRowMirror>(m[i]));
    }
    if (lanes >= 32u) {
#pragma unroll
        for (int i = 0; i < N; ++i) m[i] = max(m[i], swizzle_xor16_u32(m[i]));
    }
    if (lanes >= 64u) {
#pragma unroll
        for (int i = 0; i < N; ++i) m[i] = max(m[i], bpermute_xor32_u32(m[i], lane));
    }
}
// Maximum over the lanes of a bucket up to and including each lane: before = lanes of the wave in front of this one that
// belong to its bucket.  0 is the identity.
template <int N>
__device__ __forceinline__ void segment_max(uint32_t (&m)[N], const uint32_t before, const uint32_t lane) {
    const auto step = [&](auto ctrl, const bool reaches) {
        constexpr int CTRL = decltype(ctrl)::value;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint32_t t = dpp_or_zero<CTRL>(m[i]);
            m[i] = max(m[i], reaches ? t : 0u);
        }
    };
    using std::integral_constant;
    const uint32_t in_row = lane & 15u;
    step(integral_constant<int, 0x111>{}, before >= 1u && in_row >= 1u);   // row_shr:1
    step(integral_constant<int, 0x112>{}, before >= 2u && in_row >= 2u);   // row_shr:2
    step(integral_constant<int, 0x114>{}, before >= 4u && in_row >= 4u);   // row_shr:4
    step(integral_constant<int, 0x118>{}, before >= 8u && in_row >= 8u);   // row_shr:8
    step(integral_constant<int, 0x142>{}, (lane & 16u) != 0u && before > in_row);          // row_bcast:15: rows 1 and 3
    step(integral_constant<int, 0x143>{}, (lane & 32u) != 0u && before > (lane & 31u));    // row_bcast:31: rows 2 and 3
}

// Where a lane holds two half cells (lane l: halves of cells l / 2 and 32 + l / 2 of the wave): maxima of the halves to
// the lanes that stand for the cells, and values of the cells to the halves.
template <int P>
__device__ __forceinline__ uint32_t cell_from_parts(const uint32_t (&m)[P], const uint32_t lane) {
    if constexpr (P == 1) {
        return m[0];
    } else {
        const uint32_t a = max(m[0], dpp_u32<kDppQuadSwap1>(m[0])), b = max(m[1], dpp_u32<kDppQuadSwap1>(m[1]));
        const int from = (int)((lane & 31u) << 3);   // lane 2 (l mod 32), in bytes
        const uint32_t x = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)a), y = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)b);
        return lane < 32u ? x : y;
    }
}
template <int P>
__device__ __forceinline__ void parts_from_cell(const float c, const uint32_t lane, float (&o)[P]) {
    if constexpr (P == 1) {
        o[0] = c;
    } else {
        const int v = __builtin_bit_cast(int, c);
        o[0] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((int)((lane >> 1) << 2), v));
        o[1] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((int)((32u + (lane >> 1)) << 2), v));
    }
}

// The range of the lane's cell's bucket from the parts' maxima m[p][0 .. N), each an unsigned key whose identity is 0.
template <int B, bool LOCAL, int N>
__device__ __forceinline__ void bucket_max(const uint32_t (&m)[N][Parts<B>::kCount], const CellTile& g, const uint32_t cell, const uint32_t bucket,
                                           uint32_t (*s_max)[kMostSharedBuckets], uint32_t (&out)[N]) {
    const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
    for (int i = 0; i < N; ++i) out[i] = cell_from_parts<Parts<B>::kCount>(m[i], lane);
    if constexpr (LOCAL) {
        group_max(out, g.bucket_cells, lane);
    } else {
        const uint32_t in_bucket = cell - bucket * g.bucket_cells;
        segment_max(out, in_bucket < lane ? in_bucket : lane, lane);
        if (lane == 63u || in_bucket + 1u == g.bucket_cells) {   // the wave's last lane of the bucket
#pragma unroll
            for (int i = 0; i < N; ++i) atomicMax(&s_max[i][bucket], out[i]);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < N; ++i) out[i] = s_max[i][bucket];
    }
}

// What the two encodings do with the sum's values.
struct MinmaxCode {
    using Sum = MinmaxSum;
    static constexpr int kKeys = 2;
    static constexpr bool kShortShared = false;   // short launches with buckets across waves: not taken (requantize_minmax_cells_supported)
    template <int B, bool WHOLE>
    static __device__ __forceinline__ void keys(const float (&v)[32], const Window<B>& at, uint32_t (&m)[2][Parts<B>::kCount]) {
        float lo[Parts<B>::kCount], hi[Parts<B>::kCount];
        part_ranges<B, WHOLE>(v, at, lo, hi);
#pragma unroll
        for (int p = 0; p < Parts<B>::kCount; ++p) {
            m[0][p] = ~order_key(lo[p]);
            m[1][p] = order_key(hi[p]);
        }
    }
    template <int B, bool WHOLE>
    static __device__ __forceinline__ void encode(const RequantArgs& ra, const Window<B>& at, const uint64_t, const float (&v)[32], const uint32_t (&key)[2],
                                                  const bool stores, const uint64_t bucket) {
        const float Lf = (float)((1 << B) - 1), Wf = (float)ra.W;
        float lo = key_value(~key[0]), hi = key_value(key[1]);
        if (lo == 0.0f) lo = 0.0f;   // a zero bound is stored as +0
        if (hi == 0.0f) hi = 0.0f;
        if (stores) reinterpret_cast<float2*>(ra.q.scales)[bucket] = make_float2(lo / Wf, hi / Wf);
        const uint32_t lane = threadIdx.x & 63u;
        float mn[Parts<B>::kCount], a[Parts<B>::kCount];
        parts_from_cell<Parts<B>::kCount>(lo, lane, mn);
        parts_from_cell<Parts<B>::kCount>(inverse_step(lo, hi, Lf), lane, a);
        encode_minmax<B, WHOLE>(ra.q.packed, at, v, mn, a);
    }
};
struct CentredCode {
    using Sum = CentredSum;
    static constexpr int kKeys = 1;
    static constexpr bool kShortShared = true;
    template <int B, bool WHOLE>
    static __device__ __forceinline__ void keys(const float (&v)[32], const Window<B>& at, uint32_t (&m)[1][Parts<B>::kCount]) {
        constexpr int E = Parts<B>::kElems;
#pragma unroll
        for (int p = 0; p < Parts<B>::kCount; ++p) {
            float r = 0.0f;
#pragma unroll
            for (int k = p * E; k < p * E + E; k += 2) {   // non-negative floats order like their bit patterns
                const float x = inside<B, WHOLE>(at, k) ? v[k] : 0.0f, y = inside<B, WHOLE>(at, k + 1) ? v[k + 1] : 0.0f;
                asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(r) : "v"(x), "v"(y));
            }
            m[0][p] = __builtin_bit_cast(uint32_t, r);
        }
    }
    template <int B, bool WHOLE>
    static __device__ __forceinline__ void encode(const RequantArgs& ra, const Window<B>& at, const uint64_t tile_base, const float (&v)[32],
                                                  const uint32_t (&key)[1], const bool stores, const uint64_t bucket) {
        constexpr int P = Parts<B>::kCount, E = Parts<B>::kElems;
        const QuantizeArgs& a = ra.q;
        const float halfL = 0.5f * (float)((1 << B) - 1);
        float s = __builtin_bit_cast(float, key[0]);
        if (!(s >= 0x1p-96f)) s = 0.0f;
        if (stores) a.scales[bucket] = s / (float)ra.W;
        float a16[P];
        parts_from_cell<P>((s > 0.0f) ? (halfL / s) * 65536.0f : 0.0f, threadIdx.x & 63u, a16);   // IEEE-correct fp32 division, times 2^16 (exact)
        FixedGrid fg = fixed_grid(B);
        fg.half16 = in_vector(fg.half16);
        uint32_t o[B];
#pragma unroll
        for (int q = 0; q < 4; ++q) {   // one Philox call covers eight consecutive elements
            const int p = 8 * q / E;
            const uint64_t grp = (a.elem_base + tile_base + (uint64_t)(at.word[p] / (Parts<B>::kWords) * E + (8 * q) % E)) >> 3;
            uint32_t h[4];
            philox4x32_10<true>((uint32_t)grp, (uint32_t)(grp >> 32), a.iteration, a.worker, a.key0, a.key1, h);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                uint32_t t[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = 8 * q + 4 * u + e;
                    const uint32_t word = h[2 * u + e / 2];
                    t[e] = round_code_hi(v[k], a16[p], fg, (e & 1) != 0 ? word >> 16 : word & 0xFFFFu);
                    if (!inside<B, WHOLE>(at, k)) t[e] = 0u;   // elements past the end contribute zero bits
                }
                place<B>(o, 8 * q + 4 * u, pack_quad_hi(t[0], t[1], t[2], t[3], B, 2 * B, 3 * B), 4);
            }
        }
        // Written through and kept in L2, where the worker's update reads them next (1 % of the exchange of 25.6 M elements, 8
        // workers, 4 bits); but streaming where a lane's 20 to 28 bytes leave in two or three pieces, each of which would go
        // to memory as a part of a line: us at 25.6 M, 8 workers, bucket 1024, written through / streaming, 5 bits 34.3 / 32.1,
        // 6 bits 38.7 / 34.1, 7 bits 47.6 / 36.6 (3 bits 31.7 / 31.0, and the update 39.0 / 39.5; 8 bits at 100 M 139.9 / 154.4).
        store_parts<B, WHOLE, (B <= 4 || B == 8)>(a.packed, at, o);
    }
};

template <int B, class Code, bool LOCAL, Size SIZE, bool WHOLE>
__device__ __forceinline__ void requantize_cells_tile(const RequantArgs& ra, const CellTile& g, const uint64_t tile_base, typename Code::Sum::Step* s_tab,
                                                      uint32_t (*s_max)[kMostSharedBuckets]) {
    constexpr int P = Parts<B>::kCount;
    const uint32_t tid = threadIdx.x;
    const uint64_t tile_end = WHOLE ? tile_base + g.cells * kCell : ra.q.n;
    const uint32_t buckets = WHOLE ? g.buckets : ((uint32_t)(tile_end - tile_base) + ra.q.bucket - 1u) / ra.q.bucket;   // that begin in the tile
    const uint64_t first_bucket = (uint64_t)blockIdx.x * g.buckets;
    const Window<B> at(ra.q.n, tile_base, tile_end, g.cells);
    const auto bucket_of = [&](const uint32_t cell) {
        const uint32_t k = bucket_of_cell(g, cell);
        return WHOLE || k < buckets ? k : buckets - 1u;   // cells past the end: any
    };
    uint32_t bucket[P];
#pragma unroll
    for (int p = 0; p < P; ++p) bucket[p] = bucket_of(at.cell[p]);
    for (uint32_t i = tid; i < ra.W * buckets; i += blockDim.x) {
        const uint32_t w = i / buckets, k = i - w * buckets;
        s_tab[i] = Code::Sum::step(ra.scales[w], first_bucket + k, (float)((1 << B) - 1));
    }
    if constexpr (!LOCAL) {
        for (uint32_t i = tid; i < g.buckets; i += blockDim.x) {
#pragma unroll
            for (int u = 0; u < Code::kKeys; ++u) s_max[u][i] = 0u;
        }
    }
    float v[32];
    decode_sum<B, SIZE, WHOLE, typename Code::Sum>(ra, at, s_tab, buckets, bucket, v);

    uint32_t m[Code::kKeys][P], key[Code::kKeys];
    Code::template keys<B, WHOLE>(v, at, m);
    const uint32_t cell = tid < g.cells ? tid : g.cells - 1u;   // the cell that this lane stands for
    const uint32_t mine = bucket_of_cell(g, cell);
    bucket_max<B, LOCAL, Code::kKeys>(m, g, cell, mine, s_max, key);
    const bool stores = tid < g.cells && cell == mine * g.bucket_cells && mine < buckets;
    Code::template encode<B, WHOLE>(ra, at, tile_base, v, key, stores, first_bucket + mine);
}
// Waves per SIMD: what the registers of that many words in flight leave without scratch memory.
template <int B, class Code, Size SIZE>
constexpr int bucketed_waves() {
    constexpr bool most = B == 8 && Code::kKeys == 2;
    return SIZE == Size::kShort ? (most ? 3 : 4) : (most ? 5 : 6);
}
template <int B, class Code, bool LOCAL, Size SIZE>
__global__ __launch_bounds__(LOCAL ? 256 : 512) __attribute__((amdgpu_waves_per_eu(bucketed_waves<B, Code, SIZE>(), 8))) void requantize_cells_kernel(const RequantArgs ra, const CellTile g) {
    extern __shared__ float2 s_dyn[];   // [W][buckets of the tile]: steps
    __shared__ uint32_t s_max[LOCAL ? 1 : Code::kKeys][kMostSharedBuckets];
    const uint64_t tile_base = (uint64_t)blockIdx.x * (g.cells * kCell);
    auto* s_tab = reinterpret_cast<typename Code::Sum::Step*>(s_dyn);
    if (tile_base + g.cells * kCell <= ra.q.n) requantize_cells_tile<B, Code, LOCAL, SIZE, true>(ra, g, tile_base, s_tab, s_max);
    else requantize_cells_tile<B, Code, LOCAL, SIZE, false>(ra, g, tile_base, s_tab, s_max);
}

// Calls f(B) with the width as a compile-time constant.
template <class F>
void with_bits(uint32_t bits, F f) {
    using std::integral_constant;
    switch (bits) {
        case 1: return f(integral_constant<int, 1>{});
        case 2: return f(integral_constant<int, 2>{});
        case 3: return f(integral_constant<int, 3>{});
        case 4: return f(integral_constant<int, 4>{});
        case 5: return f(integral_constant<int, 5>{});
        case 6: return f(integral_constant<int, 6>{});
        case 7: return f(integral_constant<int, 7>{});
        default: return f(integral_constant<int, 8>{});
    }
}

constexpr uint64_t kLastLevelCache = 256ull << 20;
// of all workers: the codes, and two floats per bucket (the max-abs range has one, a whole tensor none to speak of)
uint64_t stream_bytes(const RequantArgs& ra) { return ((ra.q.n >> 3) * ra.q.bits + ra.q.n / ra.q.bucket * 8u) * ra.W; }
bool past_cache(const RequantArgs& ra) { return stream_bytes(ra) > kLastLevelCache / 4u * 5u; }
// Where streaming loads begin: with the cache's size at 4, 6 and 8 bits, whose loads leave no gaps; later at 7 and 5 bits, where a
// wave's next load asks for the same cache lines again, and there only where tiles begin with a cache line (power-of-two buckets and
// whole tensors: else neighbours ask again too, and [min, max] takes 8-12 % longer at buckets 352 to 5152).  us of the max-abs step,
// ordinary / streaming loads, inside the exchange (the workers' quantizers just before it) and in a loop of its own, bucket 1024:
//   bits, workers, elements, MB        exchange        alone       |  bits, workers, elements, MB      exchange        alone
//   6     8         50 M     300     64.7 /  66.3   64.1 /  63.4   |  7     4         80 M   280     67.2 /  75.5   63.7 /  71.0
//   6     8        100 M     600    158.9 / 121.2  125.2 / 119.5   |  7     4        100 M   350     96.8 /  97.8   86.0 /  87.2
//   8     8         50 M     400    103.4 /  71.2   84.9 /  77.3   |  7     6         80 M   420    112.5 / 101.9   90.0 /  96.4
//   5    16         35 M     350     86.0 /  82.3   74.5 /  77.1   |  7     4        150 M   525    152.4 / 135.3  121.2 / 127.3
//   5    16         40 M     400     99.4 /  92.1   88.0 /  86.9   |  5    16         50 M   500    131.6 / 112.3  108.1 / 107.1
//   5     8         80 M     400    103.4 / 100.9   91.9 /  95.3   |  5     8        100 M   500    132.8 / 122.9  113.4 / 114.3
//   5     8         70 M     350     88.6 /  90.2   82.5 /  84.7   |  5    24         25 M   375     92.2 /  83.7   79.3 /  79.2
// kShort up to 2^20 elements: above, the large tiles are level or better almost everywhere.  us, small / large tiles: [min, max],
// bucket 2304, 8 workers, 1 bit, 1.05, 1.4 and 2.05 M elements 6.4 / 4.9, 6.7 / 5.1, 6.9 / 6.4; 4096, 16 workers, 1 bit, 1.2 M 8.6 / 6.5;
// max-abs, 1024, 2 workers, 4 bits, 1.6 M 4.3 / 4.0; 2304, 8 workers, 4 bits 7.4 / 5.8; 3 bits, 16 workers, bucket 8192 7.9 / 8.4
Size size_of(const RequantArgs& ra) {
    constexpr uint64_t kShortElems = 1ull << 20;
    if (ra.q.n <= kShortElems) return Size::kShort;
    if (ra.q.bits < 4u) return Size::kLong;
    if ((ra.q.bits & 1u) == 0u) return stream_bytes(ra) > kLastLevelCache ? Size::kStream : Size::kLong;
    const bool streams = ra.q.bits == 7u || ra.W >= 16u ? past_cache(ra) : stream_bytes(ra) > kLastLevelCache / 2u * 3u;
    return streams && ra.q.bucket_shift >= 0 ? Size::kStream : Size::kLong;
}
// Calls f(B, SIZE) with the width and the size as compile-time constants.  SHORT: the form takes launches that are.
template <bool SHORT, class F>
void with_shape(const RequantArgs& ra, F f) {
    const Size size = size_of(ra);
    with_bits(ra.q.bits, [&](auto b) {
        constexpr int B = decltype(b)::value;
        if constexpr (SHORT) {
            if (size == Size::kShort) return f(b, std::integral_constant<Size, Size::kShort>{});
        }
        if constexpr (B >= 4) {
            if (size == Size::kStream) return f(b, std::integral_constant<Size, Size::kStream>{});
        }
        f(b, std::integral_constant<Size, Size::kLong>{});
    });
}

bool local_buckets(const QuantizeArgs& a) { return a.bucket_shift >= 5 && a.bucket <= 64u * kCell; }

// The tile of a bucket size.  Short launches: as few waves as hold a bucket.  Others: up to 256 cells; one bucket where it has more.
// Five waves only where two buckets fill them and four hold one (129 to 160 cells), in long launches: bucket 4128 at 2.5, 8, 16 M
// elements 1.02, 0.92, 0.98 of the time with four.  Where they hold three instead of two (2752) they take 1.28, 1.04, 1.16 of it, and where
// six instead of four (1664) 1.00, 1.05, 1.03: five waves share four SIMDs badly.  At most 4096 steps in LDS.
CellTile cell_tile(const RequantArgs& ra, uint32_t* lanes) {
    const uint32_t bc = ra.q.bucket / kCell;
    const bool local = local_buckets(ra.q);
    uint32_t waves = (bc + 63u) / 64u;
    if (size_of(ra) != Size::kShort && bc <= 256u) {
        waves = bc > 128u && bc <= 160u && ra.q.n > 5ull << 20 ? 5u : 4u;
    }
    uint32_t buckets = (waves * 64u) / bc;
    const uint32_t most = 4096u / ra.W;   // >= 64
    if (buckets > most) buckets = local ? 64u / bc : most;
    const uint32_t cells = buckets * bc;
    *lanes = (cells + 63u) / 64u * 64u;
    return {cells, buckets, bc, ((1u << 20) + bc - 1u) / bc};
}

template <class Code>
hipError_t launch_requantize_cells(const RequantArgs& ra, hipStream_t stream) {
    uint32_t lanes;
    const CellTile g = cell_tile(ra, &lanes);
    const uint64_t elems = (uint64_t)g.cells * kCell;
    const uint64_t tiles = (ra.q.n + elems - 1) / elems;
    if (tiles > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const size_t lds = sizeof(typename Code::Sum::Step) * ra.W * g.buckets;
    const auto launch = [&](auto local, auto b, auto size) {
        hipLaunchKernelGGL((requantize_cells_kernel<decltype(b)::value, Code, decltype(local)::value, decltype(size)::value>), dim3((uint32_t)tiles),
                           dim3(lanes), lds, stream, ra, g);
    };
    if (local_buckets(ra.q)) with_shape<true>(ra, [&](auto b, auto size) { launch(std::true_type{}, b, size); });
    else with_shape<Code::kShortShared>(ra, [&](auto b, auto size) { launch(std::false_type{}, b, size); });
    return hipGetLastError();
}

}  // namespace

// ---- one range for the whole tensor: the passes of launch_requantize_minmax_tensor (minmax.hip) -------------------
// From 1.5 M elements on; below, a wave's chain counts, and that of the rows form is half as long (sixteen elements per
// lane).  us, rows / cells: 3 bits, 12 workers, 1 M elements 12.8 / 14.6, 4 bits 13.8 / 13.1; 2 M 3 bits 15.5 / 15.1; 10 M, 4
// workers, 3 bits 22.9 / 16.6, 4 bits 23.1 / 16.8; 12 workers, 4 bits 41 / 33, 6 bits 51 / 38; 100 M 300 / 236.
// Not at 7 bits with streams past the cache, unless they are few (inside the exchange; size_of has the reason): 2 workers, 250 M
// elements 297 / 259, 4 workers, 120 M 204 / 211, 8 workers, 45 M (315 MB) 132 / 121, 50 M (350) 143 / 155, 100 M 294 / 319, 24
// workers, 20 M 174 / 198.
bool tensor_cells_supported(const RequantArgs& ra) { return ra.q.n > 3ull << 19 && (ra.q.bits != 7u || ra.W <= 4u || !past_cache(ra)); }
uint32_t tensor_cells_tile() { return 256u * kCell; }
void launch_sum_range_cells(const RequantArgs& ra, uint32_t tiles, uint32_t tile, uint32_t* keys, hipStream_t stream) {
    with_shape<false>(ra, [&](auto b, auto size) {
        hipLaunchKernelGGL((sum_range_cells_kernel<decltype(b)::value, decltype(size)::value>), dim3(tiles), dim3(tile / kCell), 0, stream, ra, keys);
    });
}
void launch_requantize_tensor_cells(const RequantArgs& ra, uint32_t tiles, uint32_t tile, const float* sum_range, uint32_t borrowed, hipStream_t stream) {
    with_shape<false>(ra, [&](auto b, auto size) {
        hipLaunchKernelGGL((requantize_tensor_cells_kernel<decltype(b)::value, decltype(size)::value>), dim3(tiles), dim3(tile / kCell), 0, stream, ra, sum_range,
                           borrowed);
    });
}

// ---- one range per bucket -------------------------------------------------------------------------------------------
// us, rows / cells:      64 K           1 M           2 M           10 M          25.6 M elements
//   1024, 8, 4 bits       5.0 /  4.4    5.6 /  4.6    6.5 /  5.5   17.8 / 12.0   36.8 / 25.5
//   1024, 8, 8 bits       5.1 /  4.9    5.6 /  5.0    6.9 /  6.3   20.6 / 15.6   44.3 / 35.9
//   2304, 8, 4 bits       5.2 /  5.4    5.9 /  6.3    7.4 /  6.6   21.3 / 14.0   45.2 / 29.2
//   2304, 16, 2 bits      7.1 /  7.1    7.9 /  8.8   10.0 /  9.4   32.1 / 20.3
//   32, 24, 4 bits       11.7 / 13.4   13.8 / 14.4   15.6 / 20.0   55.0 / 57.4   (a division per lane and worker in either)
//   64, 24, 6 bits       11.3 / 12.4   12.9 / 14.5   15.0 / 17.0
//   1024, 24, 3 bits      9.1 /  9.3    9.4 /  9.9  (1.1 M: 10.8 / 9.8)    128, 24, 3 bits   10.0 / 10.9   11.5 / 13.0
//   128, 24, 6 bits      10.2 / 11.0   12.0 / 12.0                         128, 16, 6 bits    7.9 /  8.2    8.9 /  8.7
//   128, 64, 6 bits      24.2 / 25.4   27.1 / 31.2   31.3 / 32.6           128, 64, 8 bits   23.0 / 21.6   27.1 / 27.9
//   8192, 8, 8 bits              (1.05 M: 5.3 /  5.8)  5.5 /  5.7          8192, 8, 4 bits  (1.05 M: 5.8 / 5.3)
bool requantize_minmax_cells_supported(const RequantArgs& ra) {
    if (ra.q.drop_nan != 0u) return false;   // a whole tensor as one bucket
    // 7 bits past the cache (size_of): 8 workers, bucket 1024, 50 M elements 83.6 / 84.6 inside the exchange, 81.4 / 75.2 alone, 100 M
    // 157.6 / 158.8, 157 / 151; 16 workers, 50 M 146.6 / 152.8, 145.9 / 147.1; but 2304, 8 workers, 100 M 343 / 159
    if (ra.q.bits == 7u && ra.W > 8u && ra.q.bucket_shift >= 0 && past_cache(ra)) return false;
    const bool narrow = ra.q.bucket == 128u && ra.W > 32u && ra.q.bits >= 5u;
    if (ra.q.n <= 1ull << 20) {
        const bool many = ra.q.bits == 3u || (ra.q.bits == 6u && ra.q.bucket == 128u) ? ra.W > 12u : narrow && ra.q.n > 1ull << 19;
        return ra.q.n >= 1ull << 16 && ra.q.bucket >= 128u && local_buckets(ra.q) && !many;
    }
    if (ra.q.n <= 1ull << 21 && (narrow || (ra.q.bucket == 8192u && ra.q.bits == 8u && ra.W <= 16u))) return false;
    return ra.q.bucket >= 128u || ra.W <= 8u;
}
hipError_t launch_requantize_minmax_cells(const RequantArgs& ra, hipStream_t stream) { return launch_requantize_cells<MinmaxCode>(ra, stream); }

// us, the kernels of quantize_wave.hip (power-of-two buckets from 128) or quantize_pack.hip (others) / cells:
//                         64 K           1 M           4 M           10 M          25.6 M elements
//   1024, 8, 1 bit        4.4 /  4.8    4.7 /  5.1    6.6 /  6.7   11.0 / 11.9   23.4 / 26.5
//   1024, 8, 4 bits       4.6 /  4.7    4.8 /  5.1    8.5 /  8.2   15.7 / 12.5   30.9 / 27.2
//   1024, 8, 7 bits       4.7 /  5.3    5.2 /  5.7   10.5 /  8.8   19.6 / 15.3   44.0 / 36.0
//   2304, 8, 4 bits       7.6 /  5.6    7.9 /  6.4   17.6 /  8.9   35.9 / 14.5   85.0 / 33.5
//   64, 8, 4 bits         6.5 /  5.7    6.8 /  6.0                 23.2 / 15.1
//   32, 24, 6 bits       14.6 / 15.6   16.3 / 17.2   (2 M: 18.5 / 22.6)
// and with many workers, cells / rows at 64 K, 700 K, 1.05, 2.2, 3, 4, 5, 6, 8 and 12 M elements:
//   64, 24, 6 bits       1.01  0.97  0.95  1.02  1.04  0.96  0.86  0.84  0.81  0.81
//   64, 48, 4 bits       0.86  0.79  0.85  1.12  1.13  1.01  0.82  0.81  0.77
//   64, 64, 6 bits       1.06  1.16  1.13  1.10  1.09  1.03  0.85  0.88                    64, 64, 2 bits  0.88  0.88  0.85  1.07  1.07  0.95
//   96, 64, 6 bits       0.95  1.03  0.98  0.97  0.95  0.93  0.79  0.78
//   32, 12, 6 bits       1.04  0.98  0.99  0.93  1.09  1.00  0.92  0.89  0.84  0.80
//   32, 24, 4 bits       0.97  0.90  0.91  1.19  1.27  1.16  0.92  0.88  0.84  0.77         32, 24, 8 bits  (8 M) 0.86  1.02
//   32, 32, 8 bits       1.00  1.05  1.27  1.19  1.24  1.14  0.89  0.85  0.91  1.11         32, 32, 3 bits  (12 M) 0.92 (21 M) 0.88
//   32, 48, 4 bits       0.99  0.94  1.12  1.31  1.29  1.11  0.82  0.79  1.07
//   32, 64, 4 bits       0.98  1.14  1.25  1.31  1.23  1.04  1.12  1.20
// Buckets of the rows kernel that begin a new round of it (2^20 elements each) or not, 1.05, 1.3, 2.05, 2.2, 5 and 6 M, cells / rows:
//   1024, 8, 4 bits      1.07  0.92  0.88  0.92  0.88  0.81              1024, 16, 5 bits     1.05  0.89  0.91  0.82  0.80  0.72
//   1024, 16, 3 bits     1.17  1.09  1.03  1.09  1.06  0.95  (3.5 M 0.94, 4.2 M 1.12)         128, 16, 3 bits  1.13  1.05  1.03  0.99  1.00  0.89
//   1024, 2, 3 bits      (1.6 M 0.95, 3 M 0.99, 4.2 M 1.04)              1024, 2, 8 bits      1.00  1.06  0.95  1.04  0.98  0.90
//   1024, 4, 1 bit       1.02  1.00  0.97  1.12  1.06  0.98              1024, 2, 1 bit       (1.6 M 0.94, 2.2 M 1.05, 3 M 1.03)
//   8192, 8, 8 bits      1.08  1.09  1.06  0.89  0.92  0.97              8192, 8, 4 bits      (1.6 M 0.92, 2.2 M 0.83)
// and further on, in the exchange's loop, both in turn:
//                          25.6 M          50 M           100 M elements            16 M           40 M           100 M elements
//   1024, 8, 3 bits     31.3 /  31.7   52.6 /  52.6   103.3 / 104.0   1024, 16   32.8 / 32.2    66.4 /  68.7   169.2 / 174.4
//   1024, 8, 4 bits     34.0 /  29.9   56.6 /  49.4   108.0 /  95.1   512, 16    24.9 / 23.0    69.6 /  68.7   (10 M, 40 M)
//   1024, 8, 5 bits     41.4 /  32.6   71.3 /  54.3   149.9 / 122.9   4096, 24   30.9 / 29.7    97.8 / 100.3   (10 M, 40 M)
//   1024, 8, 6 bits     42.4 /  34.6   77.7 /  64.1   138.9 / 117.5   8192, 8    24.6 / 22.6    48.6 /  45.5   121.5 / 105.8
//   1024, 8, 7 bits     42.5 /  36.8   80.3 /  85.1   152.8 / 158.3   (43 M, 301 MB: 71.3 / 62.4)
//   1024, 8, 8 bits     45.2 /  39.6   81.8 /  71.1   155.8 / 143.1
//   128, 8, 4 bits      36.5 /  31.4   62.0 /  52.0   119.9 / 104.5
//   8192, 8, 4 bits     37.9 /  29.8   63.5 /  49.4   128.5 /  95.1
//   1024, 6, 7 bits: 55 M 74.3 / 62.4, 80 M (420 MB) 105.7 / 101.9; 1024, 16, 7 bits: 22 M 69.0 / 62.4, 25 M (350 MB) 73.5 / 79.1
// (both take a fifth longer in the throttled launches after an idle gap: 4 bits, 100 M, 135-168 / 120-145)
bool requantize_centred_cells_supported(const RequantArgs& ra) {
    if (ra.q.scale_mode != MQG_SCALE_MAXABS || ra.q.n < kCell) return false;   // a lane reads its words at once: the stream must hold as many
    if (requantize_wave_supported(ra)) {
        if (ra.q.bits == 7u && ra.W > 6u && past_cache(ra)) return false;
        if (ra.q.bits == 3u && ra.W > 6u && ra.q.n > 1ull << 24 && ra.q.bucket >= 1024u && ra.q.bucket <= 4096u) return false;
        if (ra.q.bits <= 2u && ra.W > 4u) return false;
        if (ra.q.bucket == 16384u) return ra.q.n > 1ull << 20;
        if (ra.W > 2u && ra.q.bits <= 3u && ra.q.bucket >= 512u && ra.q.bucket <= 4096u) {   // the fourth million is a round of its own to the rows kernel
            return ra.q.n > 11ull << 19 || (ra.q.n > 3ull << 20 && ra.q.n <= 1ull << 22);
        }
        if ((ra.W > 2u && ra.q.bits <= 3u) || (ra.W <= 4u && ra.q.bits == 8u) || (ra.q.bucket == 8192u && ra.q.bits >= 6u)) return ra.q.n > 1ull << 21;
        return ra.q.n > 65ull << 14;
    }
    // a division per bucket, lane and worker where rows share one: the smallest buckets of many workers
    if (ra.q.bucket == 64u) return ra.W <= 24u || ra.q.bits <= 3u || ra.q.n <= 1ull << 19 || ra.q.n > 1ull << 22;
    if (ra.q.bucket > 32u || ra.W <= 8u) return true;
    if (ra.W <= 24u) return ra.q.n > (ra.W <= 12u ? 1ull << 21 : 1ull << 22);
    return ra.q.n > 1ull << 22 && ((ra.W <= 32u && ra.q.bits <= 5u) || (ra.W <= 48u && ra.q.n * ra.W <= 340000000ull));
}
hipError_t launch_requantize_centred_cells(const RequantArgs& ra, hipStream_t stream) { return launch_requantize_cells<CentredCode>(ra, stream); }

}  // namespace mqg
