// libndq, server side (gfx950): DQSG / NDQSG decoders, the fused server loop of
// Algorithm 2, aggregation.  See include/ndq.h for the contract.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "ndq.h"
#include "ndq_device.hpp"
#include "ndq_host.hpp"

namespace ndq {

// ---------------------------------------------------------------------------
// Decoder: Algorithm 1 server block (DQSG) / Algorithm 2 server loop (NDQSG)
// ---------------------------------------------------------------------------
struct DecodeArgs {
    const unsigned char* codes;
    const float* steps;
    const float* side;     // nested modes
    float* out;
    Tiling tl;
    uint64_t index0;
    DitherStream ds;
    Quant qp;
    float side_scale;
};

template <int ROWS> struct DecTile { static constexpr uint32_t N = kWave * 4 * ROWS; };  // outputs per wave
template <int MODE, int ACC> struct DecRows {
    static constexpr int R = ((MODE == kDq || MODE == kDqHalf) && ACC == 0) ? kDecRowsStream : kDecRowsUpdate;
};

enum Acc { kStore = 0, kAccumulate = 1, kAccumulateInPlace = 2 };  // in place: out == side

// Four elements of a row: res = decoded value (stored, or added to ps / ys).
template <int MODE, int ACC>
__device__ __forceinline__ void decode_row(const DecodeArgs& a, uint32_t packed, uint32_t bits,
                                           const float (&ys)[4], const float (&ps)[4], const float (&v)[4],
                                           float step, float inv, float (&res)[4])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t c = __builtin_amdgcn_ubfe(packed, k * bits, bits);   // bit-field extract
        float q, yk = 0.0f;
        if (MODE == kDq || MODE == kDqHalf) {
            q = (float)((int32_t)c + a.qp.q_min);
        } else {
            yk = ys[k] * a.side_scale;
            q = coset_index_f<MODE>((float)c, yk, inv, v[k], a.qp);
        }
        const float val = (MODE == kDqHalf) ? step * q
                                            : shrink<MODE>(index_value(q, step, v[k]), yk, a.qp);
        if (ACC == kStore) res[k] = val;
        else if (ACC == kAccumulate) res[k] = ps[k] + val;
        else res[k] = ys[k] + val;
    }
}

// One wave decodes one tile.  FULL: every element valid, no guards.  STRADDLE:
// the code width does not divide 8, so four codes may cross a 32-bit word.
template <int MODE, int ACC, bool FULL, bool STRADDLE>
__device__ __forceinline__ void decode_tile(const DecodeArgs& a, const TileRef& t, int lane)
{
    const uint32_t bits = a.qp.bits;
    const uint32_t* codes32 = (const uint32_t*)(a.codes + (t.start >> 3) * bits);
    const float* side = a.side + t.start;
    float* out = a.out + t.start;
    const float step = a.steps[t.bucket];
    const float inv = a.qp.alpha * inv_step(step);
    const uint64_t block0 = (a.index0 + t.start) >> 2;

    constexpr int kDecRows = DecRows<MODE, ACC>::R;
    uint32_t packed[kDecRows];
    float4 y[kDecRows], prev[kDecRows];
#pragma unroll
    for (int r = 0; r < kDecRows; ++r) {
        const uint32_t o = (uint32_t)r * kWave * 4 + (uint32_t)lane * 4;
        packed[r] = 0;
        y[r] = make_float4(0.f, 0.f, 0.f, 0.f);
        prev[r] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (FULL || o < t.len) {
            const uint32_t bit = o * bits;
            const uint32_t w = bit >> 5, sh = bit & 31u;
            if (STRADDLE) {
                // read the next word only if a valid code reaches into it (a ragged
                // tail must not touch memory past the stream)
                const uint32_t ncodes = FULL ? 4u : (t.len - o < 4u ? t.len - o : 4u);
                uint64_t window = codes32[w];
                if (sh + ncodes * bits > 32u) window |= (uint64_t)codes32[w + 1] << 32;
                packed[r] = (uint32_t)(window >> sh);
            } else {
                packed[r] = codes32[w] >> sh;
            }
            if (FULL || o + 4 <= t.len) {
                if (MODE == kNestedPow2 || MODE == kNestedAnyM || MODE == kNestedPow2Shrink)
                    y[r] = load_streaming_f4(side + o);
                if (ACC == kAccumulate) prev[r] = load_streaming_f4(out + o);
            } else {
                float ys[4] = {0.f, 0.f, 0.f, 0.f}, ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k)
                    if (o + k < t.len) {
                        if (MODE == kNestedPow2 || MODE == kNestedAnyM || MODE == kNestedPow2Shrink)
                            ys[k] = side[o + k];
                        if (ACC == kAccumulate) ps[k] = out[o + k];
                    }
                y[r] = make_float4(ys[0], ys[1], ys[2], ys[3]);
                prev[r] = make_float4(ps[0], ps[1], ps[2], ps[3]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < kDecRows; ++r) {
        const uint32_t o = (uint32_t)r * kWave * 4 + (uint32_t)lane * 4;
        if (!FULL && o >= t.len) continue;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        if (MODE != kDqHalf) dither4(a.ds, block0 + (o >> 2), v);
        const float ys[4] = {y[r].x, y[r].y, y[r].z, y[r].w};
        const float ps[4] = {prev[r].x, prev[r].y, prev[r].z, prev[r].w};
        float res[4];
        decode_row<MODE, ACC>(a, packed[r], bits, ys, ps, v, step, inv, res);
        if (FULL || o + 4 <= t.len) {
            store_streaming(out + o, res[0], res[1], res[2], res[3]);
        } else {
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k)
                if (o + k < t.len) out[o + k] = res[k];
        }
    }
}

template <int MODE, int ACC, bool STRADDLE>
__global__ __launch_bounds__(kBlock) void decode_kernel(DecodeArgs a)
{
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t tile_id =
        blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    constexpr uint32_t TILE = DecTile<DecRows<MODE, ACC>::R>::N;
    const TileRef t = locate_tile(a.tl, tile_id, TILE);
    if (t.len == TILE) decode_tile<MODE, ACC, true, STRADDLE>(a, t, lane);
    else if (t.len != 0) decode_tile<MODE, ACC, false, STRADDLE>(a, t, lane);
}

// A worker after the other, a short launch waits for each cache line of its arguments: all its waves read a line for the
// first time at the same moment, and the L2 has none of them yet.  So every lane first reads a word of a line of its own,
// which brings the first `bytes` (at most 4,096) into the L2 side by side; nobody waits for it until arguments_read(),
// after the first worker, or the last: a test for the first one inside the loop makes the compiler take the loop apart, which
// chain_kernel gains from (4 x 32 levels 4 to 14 M elements 1 to 4 %), and decode_mean_kernel with few workers, but not with many (kMeanFew).  us without / with it at 0.3, 0.5 and 1.05 M elements: chain_stream_kernel, one row per wave, 2 x 16 levels
// 3.50/3.30 3.70/3.52 4.21/4.01, 8 x 16 levels 6.42/5.62 6.65/5.87 7.20/6.72, 16 levels and 15 x M = 4 at 0.5 M 12.5/10.5; chain_kernel,
// 8 x 100 levels, at 1.05 and 2 M 10.1/8.9 11.7/11.0; decode_mean_kernel, 4 workers, at 0.06, 0.27 and 1.66 M 5.9/5.3 6.3/5.7 10.7/10.5,
// 16 workers 17.7/15.3 18.5/16.9 29.8/29.7.
__device__ __forceinline__ uint32_t read_arguments_ahead(const __attribute__((address_space(4))) void* arguments, uint32_t bytes, int lane)
{
    const uint32_t at = (uint32_t)lane * 64u;
    return ((const __attribute__((address_space(4))) uint32_t*)arguments)[(at < bytes ? at : 0u) / 4u];
}
__device__ __forceinline__ void arguments_read(uint32_t word) { asm volatile("" ::"v"(word)); }

// ---------------------------------------------------------------------------
// Chain decoder: the whole server loop of Algorithm 2 in one pass.  The running
// sum of a lane's elements lives in registers while the workers are folded in
// one after the other; the next worker's code words and step are prefetched
// while the current worker's dither is generated.
// ---------------------------------------------------------------------------
constexpr uint32_t kChainMax = 32;    // workers per launch
#ifndef NDQ_CHAIN_ROWS
#define NDQ_CHAIN_ROWS 2
#endif
constexpr int kChainRows = NDQ_CHAIN_ROWS;   // rows of 8 elements per lane and tile
constexpr uint32_t kChainTile = kWave * kLaneElems * kChainRows;
// Below these numbers of tiles a wave takes one row: two waves per SIMD then hide each other's
// latency where one would wait.  chain_kernel (4 DQSG + 4 nested M = 3: 0.27 M elements 9.8 against
// 12.2 us, 1 M 10.9 / 12.8, 2 M 14.6 / 16.6, 4 M 20.6 / 20.1), chain_stream_kernel (4 workers: 1 M 5.6
// against 6.4, 2 M 8.1 / 8.4, 4 M 12.4 / 10.7).
constexpr uint32_t kShortGeneralTiles = 4096, kShortTiles = 2048;

struct ChainWorker {
    const unsigned char* codes;
    const float* steps;
    uint64_t index0;
    DitherStream ds;
    int32_t q_min;
    uint32_t M;
    float M_f, inv_M_f;
    float alpha, beta;    // nested: shrinkage factor and 1 - alpha^2
    float side_scale;     // 1/(workers folded in before this one); 0 for the first
    uint32_t bits;
    uint32_t mode;        // Mode
    uint32_t first;       // S <- value instead of S + value
};

struct GeneralChainArgs {
    ChainWorker w[kChainMax];
    float* out;
    Tiling tl;
    uint32_t W;
    int continue_sum;     // S starts from out (an earlier group of workers)
    int apply_scale;
    float scale;
    uint32_t row_buckets; // 1: a bucket is one row of a tile (tiling is by tile, a step per row)
    uint32_t num_buckets; // with row_buckets: steps per worker (rows past them decode with step 0)
};

// What is prefetched per worker and row: the step, and a lane's eight codes -- `bits` bytes of
// the stream at any byte address -- as one 64-bit load from there, whatever the code width.
template <int ROWS> struct ChainFetch {
    uint64_t codes[ROWS];
    float step[ROWS];
};

// ROWB: a bucket is one row of the tile (the tiling is by tile and every row has
// its own step); otherwise one step serves the tile.  FULL: every element of the tile is
// valid and the stream goes on for at least eight bytes after it; else lanes near the end
// load the stream's last eight bytes and shift (it has at least eight from a tile's start on:
// its size is a multiple of 16 and a tile starts at a multiple of 8).
template <bool FULL, bool ROWB, int ROWS>
__device__ __forceinline__ void chain_fetch(const GeneralChainArgs& a, const ChainWorker& cw, const TileRef& t,
                                            int lane, ChainFetch<ROWS>& f)
{
    const uint32_t bits = cw.bits;
    const unsigned char* tile = cw.codes + (t.start >> 3) * bits;
    if (ROWB) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const uint32_t b = t.bucket * ROWS + r;                // rows past the last bucket get 0
            f.step[r] = b < a.num_buckets ? cw.steps[b] : 0.0f;
        }
    } else {
        f.step[0] = cw.steps[t.bucket];
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        uint32_t off = (uint32_t)(r * kWave + lane) * bits, shift = 0u;
        if (!FULL) {
            const uint64_t total = (((a.tl.n * bits + 7u) >> 3) + 15u) & ~(uint64_t)15u;
            const uint64_t left = total - (t.start >> 3) * bits - 8u;
            const uint32_t limit = left < 0xFFFFu ? (uint32_t)left : 0xFFFFu;   // (a tile has at most 1,024 bytes)
            if (off > limit) {
                shift = (off - limit) * 8u;
                off = limit;
            }
        }
        __builtin_memcpy(&f.codes[r], tile + off, 8);
        // lanes past the end shift by 64 or more: what they decode is never stored
        if (!FULL) f.codes[r] >>= shift & 63u;
    }
}

// One element of one worker: S + (the worker's decoded value), or that value (FIRST), the side information being S scaled.
// c_f: the code as a float, plus q_min for DQSG.
template <int MODE, bool FIRST>
__device__ __forceinline__ float chain_element(float side_scale, const Quant& qp, float c_f, float v, float step, float inv, float S)
{
    float q = c_f, y = 0.0f;
    if (MODE != kDq) {
        y = S * side_scale;
        q = coset_index_f<MODE>(c_f, y, inv, v, qp);
    }
    const float val = shrink<MODE>(index_value(q, step, v), y, qp);
    return FIRST ? val : S + val;
}

// Folds one worker into the running sum S of a tile.  NARROW: codes of at most
// kFieldAsFloatMaxBits bits, turned into floats with FieldAsFloat.  FIRST: the running sum
// starts with this worker.
template <int MODE, bool NARROW, bool FIRST, bool ROWB, int ROWS>
__device__ __forceinline__ void chain_fold(const ChainWorker& cw, const ChainFetch<ROWS>& f,
                                           uint64_t block0, int lane, float (&S)[ROWS][8])
{
    const uint32_t bits = cw.bits;
    const FieldAsFloat<4> field(NARROW ? bits : 1u, MODE == kDq ? (float)cw.q_min : 0.0f);
    float inv_row[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        inv_row[r] = (ROWB || r == 0) ? cw.alpha * inv_step(f.step[ROWB ? r : 0]) : inv_row[0];
    Quant qp;
    qp.M = cw.M; qp.M_f = cw.M_f; qp.inv_M_f = cw.inv_M_f; qp.q_min = cw.q_min;
    qp.alpha = cw.alpha; qp.beta = cw.beta;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const uint32_t o = (uint32_t)(r * kWave + lane) * kLaneElems;
        const float step = f.step[ROWB ? r : 0], inv = inv_row[r];
        const uint32_t half[2] = {(uint32_t)f.codes[r], (uint32_t)(f.codes[r] >> (4u * bits))};
        float v[8];
        dither8(cw.ds, block0 + (o >> 3), v);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            float c_f;
            if (NARROW) {
                c_f = field.get(half[k >> 2], k & 3);
            } else {
                const uint32_t c = __builtin_amdgcn_ubfe(half[k >> 2], (k & 3) * bits, bits);
                c_f = MODE == kDq ? (float)((int32_t)c + qp.q_min) : (float)c;
            }
            S[r][k] = chain_element<MODE, FIRST>(cw.side_scale, qp, c_f, v[k], step, inv, S[r][k]);
        }
    }
}

template <int MODE, bool FIRST, bool ROWB, int ROWS>
__device__ __forceinline__ void chain_fold_width(const ChainWorker& cw, const ChainFetch<ROWS>& f,
                                                 uint64_t block0, int lane, float (&S)[ROWS][8])
{
    if (cw.bits <= kFieldAsFloatMaxBits) chain_fold<MODE, true, FIRST, ROWB, ROWS>(cw, f, block0, lane, S);
    else chain_fold<MODE, false, FIRST, ROWB, ROWS>(cw, f, block0, lane, S);
}

template <bool FULL, bool ROWB, bool ANYM, int ROWS>
__device__ __forceinline__ void chain_tile(const GeneralChainArgs& a, const TileRef& t, int lane, uint32_t warm)
{
    float S[ROWS][8];
    float* out = a.out + t.start;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const uint32_t o = (uint32_t)(r * kWave + lane) * kLaneElems;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            S[r][k] = 0.0f;
            if (a.continue_sum && (FULL || o + k < t.len)) S[r][k] = out[o + k];
        }
    }
    ChainFetch<ROWS> cur;
    chain_fetch<FULL, ROWB, ROWS>(a, a.w[0], t, lane, cur);
    ChainFetch<ROWS> nxt = cur;
    for (uint32_t w = 0; w < a.W; ++w) {
        const ChainWorker& cw = a.w[w];
        if (w + 1 < a.W) chain_fetch<FULL, ROWB, ROWS>(a, a.w[w + 1], t, lane, nxt);
        const uint64_t block0 = (cw.index0 + t.start) >> 3;
        if (cw.mode == kDq) {
            if (cw.first) chain_fold_width<kDq, true, ROWB, ROWS>(cw, cur, block0, lane, S);
            else chain_fold_width<kDq, false, ROWB, ROWS>(cw, cur, block0, lane, S);
        } else if (cw.mode == kNestedPow2) {
            chain_fold_width<kNestedPow2, false, ROWB, ROWS>(cw, cur, block0, lane, S);
        } else if (cw.mode == kNestedPow2Shrink) {
            chain_fold_width<kNestedPow2Shrink, false, ROWB, ROWS>(cw, cur, block0, lane, S);
        } else if (ANYM) {
            chain_fold_width<kNestedAnyM, false, ROWB, ROWS>(cw, cur, block0, lane, S);
        }
        if (w == 0u) arguments_read(warm);
        cur = nxt;
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const uint32_t o = (uint32_t)(r * kWave + lane) * kLaneElems;
        float res[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) res[k] = a.apply_scale ? a.scale * S[r][k] : S[r][k];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (FULL || o + 4 * j + 4 <= t.len) {
                store_streaming(out + o + 4 * j, res[4 * j], res[4 * j + 1], res[4 * j + 2], res[4 * j + 3]);
            } else {
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k)
                    if (o + 4 * j + k < t.len) out[o + 4 * j + k] = res[4 * j + k];
            }
        }
    }
}

#ifndef NDQ_CHAIN_WAVES_PER_EU
#define NDQ_CHAIN_WAVES_PER_EU 6
#endif
// ANYM: has the code for ratios that are no powers of two.  Plans without such a ratio take the kernel with it too, but for two
// workers that do not shrink, in tiles of two rows: 2 x 32 and 2 x 100 levels at 5.3, 6.6, 8.4 and 14 M elements 8.2/7.8 10.5/9.3 12.9/12.2
// 19.2/17.9 and 8.0/7.8 9.5/9.0 12.8/11.8 18.2/16.9 with / without, but 4 x 32 levels 11.4/12.3 12.6/13.7 15.6/16.9 22.8/25.1, 16 levels and a
// shrinking M = 4 7.9/8.0 9.2/9.4 11.5/11.7 17.0/17.2.
template <bool ROWB, bool ANYM, int ROWS>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(NDQ_CHAIN_WAVES_PER_EU)))
void chain_kernel(GeneralChainArgs a)
{
    constexpr uint32_t TILE = kWave * kLaneElems * ROWS;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t tile_id =
        blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const TileRef t = locate_tile(a.tl, tile_id, TILE);
    uint32_t warm = 0u;
    if (a.W > 1u)
        warm = read_arguments_ahead((const __attribute__((address_space(4))) void*)__builtin_amdgcn_kernarg_segment_ptr(),
                                    a.W * (uint32_t)sizeof(ChainWorker), lane);
    if (t.len == TILE && t.start + TILE + 64u <= a.tl.n) chain_tile<true, ROWB, ANYM, ROWS>(a, t, lane, warm);
    else if (t.len != 0) chain_tile<false, ROWB, ANYM, ROWS>(a, t, lane, warm);
}

// ---------------------------------------------------------------------------
// Chain decoder for short vectors, any plan.  A wave that folds one worker after the other waits, for
// each of them, for its arguments, its codes and forty dependent instructions of Philox: a launch of few
// waves takes W times that, however short the vector.  Here a workgroup takes one row (512 elements) and
// its four waves first do, side by side, all that does not depend on the running sum -- the workers' Philox
// blocks (a wave takes every fourth worker), codes, steps and reciprocals -- and leave it in LDS;
// then a lane folds the workers into two elements, about ten dependent operations each.
// Twice the instructions of the other forms per element, so only as long as the chip is not full
// (short_chain_most has the lines).  WMAX: workers the workgroup's LDS holds.
// ---------------------------------------------------------------------------
typedef const __attribute__((address_space(4))) GeneralChainArgs* GeneralChainArgsPtr;
constexpr uint32_t kShortTile = kWave * kLaneElems;
constexpr uint32_t kShortSteps = kShortTile / 64u;       // buckets a tile can meet: multiples of 64 elements
constexpr uint32_t kShortCodeWords = kShortTile / 4u;    // 32-bit words of a tile's codes, 8 bits each

template <int MODE, bool FIRST>
__device__ __forceinline__ void short_fold(float side_scale, const Quant& qp, const float (&c_f)[2], const float (&v)[2],
                                           float step, float inv, float (&S)[2])
{
#pragma unroll
    for (int k = 0; k < 2; ++k) S[k] = chain_element<MODE, FIRST>(side_scale, qp, c_f[k], v[k], step, inv, S[k]);
}

template <uint32_t WMAX>
__global__ __launch_bounds__(kBlock) void chain_short_kernel(GeneralChainArgs by_value)
{
    const GeneralChainArgsPtr a = (GeneralChainArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    __shared__ __align__(16) uint32_t words_of[WMAX][kBlock];            // Philox words: two elements each
    __shared__ uint32_t codes_of[WMAX][kShortCodeWords + 4u];            // (a window may reach one word further)
    __shared__ float step_of[WMAX][kShortSteps], inv_of[WMAX][kShortSteps];
    constexpr uint32_t MINE = WMAX / kWavesPerBlock;                     // workers a wave prepares
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1u);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint32_t W = a->W, n = (uint32_t)a->tl.n;
    const uint32_t start = blockIdx.x * kShortTile;
    const uint32_t bucket_len = a->tl.bucket_len < n ? (uint32_t)a->tl.bucket_len : n;
    const uint32_t bucket0 = start / bucket_len;

    // lane w holds worker w's parameters: one wait for all of them instead of one per worker
    const uint32_t mine = lane < W ? lane : 0u;
    const uint64_t codes_at = (uint64_t)a->w[mine].codes, index0 = a->w[mine].index0;
    const uint32_t key0 = a->w[mine].ds.key0, key1 = a->w[mine].ds.key1;
    const uint32_t iteration = a->w[mine].ds.step, number = a->w[mine].ds.worker;
    const uint32_t bits_of = a->w[mine].bits, mode_of = a->w[mine].mode;
    const int32_t q_min_of = a->w[mine].q_min;
    const float M_of = a->w[mine].M_f, inv_M_of = a->w[mine].inv_M_f, alpha_of = a->w[mine].alpha;
    const float beta_of = a->w[mine].beta, side_of = a->w[mine].side_scale;
    auto from = [](uint32_t x, uint32_t w) __attribute__((always_inline)) {
        return (uint32_t)__builtin_amdgcn_readlane((int)x, (int)w);
    };
    auto from_f = [&](float x, uint32_t w) __attribute__((always_inline)) {
        return __uint_as_float(from(__float_as_uint(x), w));
    };

    // codes: the tile's share of every stream as aligned words, up to the stream's padded end
    uint32_t code[MINE][2];
#pragma unroll
    for (uint32_t i = 0; i < MINE; ++i) {
        const uint32_t w = i * kWavesPerBlock + wave;
        code[i][0] = code[i][1] = 0u;
        if (w < W) {
            const uint32_t bits = from(bits_of, w);
            const uint32_t total = ((n * (uint64_t)bits + 7u) / 8u + 15u) / 16u * 16u, byte0 = start / 8u * bits;
            const uint64_t at = ((uint64_t)from((uint32_t)(codes_at >> 32), w) << 32 | from((uint32_t)codes_at, w)) + byte0;
            const uint32_t* p = (const uint32_t*)at;
            const uint32_t share = kShortTile / 32u * bits, left = (total - byte0) / 4u;
            const uint32_t have = share < left ? share : left;
            if (lane < have) code[i][0] = p[lane];
            if (lane + kWave < have) code[i][1] = p[lane + kWave];
        }
    }
    if (tid < W * kShortSteps) {
        const uint32_t w = tid / kShortSteps, j = tid % kShortSteps, bucket = bucket0 + j;
        const uint32_t buckets = (n + bucket_len - 1u) / bucket_len;
        const float step = a->w[w].steps[bucket < buckets ? bucket : buckets - 1u];
        step_of[w][j] = step;
        inv_of[w][j] = a->w[w].alpha * inv_step(step);
    }
#pragma unroll
    for (uint32_t i = 0; i < MINE; ++i) {
        const uint32_t w = i * kWavesPerBlock + wave;
        if (w < W) {
            const uint64_t block = (((uint64_t)from((uint32_t)(index0 >> 32), w) << 32 | from((uint32_t)index0, w)) + start) / 8u + lane;
            uint32_t r[4];
            philox4x32_10((uint32_t)block, (uint32_t)(block >> 32), from(iteration, w), from(number, w), from(key0, w),
                          from(key1, w), r);
            *(uint4*)&words_of[w][lane * 4u] = make_uint4(r[0], r[1], r[2], r[3]);
            codes_of[w][lane] = code[i][0];
            codes_of[w][lane + kWave] = code[i][1];
        }
    }
    __syncthreads();

    const uint32_t element = start + 2u * tid;
    const uint32_t my_bucket = (element < n ? element : n - 1u) / bucket_len - bucket0;
    float S[2] = {0.0f, 0.0f};
    for (uint32_t w = 0; w < W; ++w) {
        const uint32_t bits = from(bits_of, w), mode = from(mode_of, w);
        const uint32_t bit = 2u * tid * bits;
        const uint32_t window = __builtin_amdgcn_alignbit(codes_of[w][bit / 32u + 1u], codes_of[w][bit / 32u], bit & 31u);
        const uint32_t word = words_of[w][tid];
        const float step = step_of[w][my_bucket], inv = inv_of[w][my_bucket];
        const float v[2] = {unit_dither(word & 0xFFFFu), unit_dither(word >> 16)};
        const uint32_t c0 = __builtin_amdgcn_ubfe(window, 0u, bits), c1 = __builtin_amdgcn_ubfe(window, bits, bits);
        Quant qp;
        qp.M_f = from_f(M_of, w);
        qp.inv_M_f = from_f(inv_M_of, w);
        qp.alpha = from_f(alpha_of, w);
        qp.beta = from_f(beta_of, w);
        const float side = from_f(side_of, w);
        if (mode == kDq) {
            const int32_t q_min = (int32_t)from((uint32_t)q_min_of, w);
            const float c_f[2] = {(float)((int32_t)c0 + q_min), (float)((int32_t)c1 + q_min)};
            if (w == 0u) short_fold<kDq, true>(side, qp, c_f, v, step, inv, S);
            else short_fold<kDq, false>(side, qp, c_f, v, step, inv, S);
        } else {
            // (shrinking workers of any ratio together, the corrected quotient of a power of two being the product itself: with a
            // branch more the compiler sends the common case through two further jumps per worker)
            const float c_f[2] = {(float)c0, (float)c1};
            if (mode == kNestedPow2) short_fold<kNestedPow2, false>(side, qp, c_f, v, step, inv, S);
            else short_fold<kNestedAnyM, false>(side, qp, c_f, v, step, inv, S);
        }
    }
    if (a->apply_scale) {
        S[0] = a->scale * S[0];
        S[1] = a->scale * S[1];
    }
    float* out = a->out;
    if (element + 1u < n) *(float2*)(out + element) = make_float2(S[0], S[1]);
    else if (element < n) out[element] = S[0];
}

// ---------------------------------------------------------------------------
// Streaming chain decoder for the plans of chain_streams: DQSG workers of one code
// width, then workers that are all alike -- more of them, also of another width after the first, or nested ones of one ratio
// without shrinkage -- with codes of up to 4 bits, and a
// vector cut into whole tiles or rows.  One instantiation of the fold serves every
// worker of a kind, so the sixteen running sums of a lane stay in the same
// registers from the first worker to the store (the general kernel dispatches on
// mode and width after every worker and moves them around each time).  Waves are
// persistent: a wave walks over tiles wave, wave + W, ... and fetches the next
// worker's, and at the end the next tile's, code words while it folds the
// current worker in.
//
// Arithmetic per element of a nested worker, bit for bit that of chain_element with
// kNestedPow2 (every scaling below is by a power of two, which commutes with
// rounding; k and m/M + k are exact or rounded exactly like m + M k):
//   m' = m / M (from the packed field, exact)      y = S * side_scale
//   c  = fma(y, 1/Delta, v)                        k = rint(fma(c, 1/M, -m'))
//   q' = k + m'                                    S = S + Delta * fma(q', M, -v)
// ---------------------------------------------------------------------------
#ifndef NDQ_CHAIN_STREAM_WAVES
#define NDQ_CHAIN_STREAM_WAVES 6
#endif
constexpr int kChainStreamWaves = NDQ_CHAIN_STREAM_WAVES;

// Per-worker parameters as the kernel reads them: through the constant address space (scalar
// loads, no copy of the arguments), with everything that does not depend on the tile worked out
// by the host, and no more than that: a worker is 40 bytes.  A short launch waits for every cache line of its
// arguments (16 workers of 65,536 elements: 11.1 us, with 112 bytes a worker 14.1), a long one spends
// fewer vector instructions on addresses (4 x 2^27: 187 -> 182 us, 16 x 11.2 M: 66.6 -> 65, 8 DQSG workers of 25.6 M:
// 57.5 -> 55, and the plain fold of the one-tile forms, which takes the same dither, 8 x 4.2 M: 15.2 -> 14.0).
struct StreamWorker {
    const unsigned char* codes;
    uint32_t block;       // low word of the number of its first Philox block
    uint32_t extra;       // nested: side_scale, 1/(workers folded in before it), as bits; DQSG: q_min
    PhiloxUniform keys;
};
struct ChainArgs {
    StreamWorker w[kChainMax];
    const float* steps[kChainMax];
    float* out;
    uint64_t n;
    uint64_t bucket_magic;    // bucket of tile t: t * bucket_magic >> bucket_shift (one bucket: 0)
    uint32_t bucket_shift;
    uint32_t tiles;           // whole tiles
    uint32_t W;
    uint32_t dq;              // MIXED: how many of the workers, the first ones, are DQSG
    float ratio, inv_ratio;   // kNestedAnyM: the nested workers' M, and 1/M rounded
    int apply_scale;
    float scale;
};
static_assert(sizeof(ChainArgs) <= 4096, "kernel arguments");
typedef const __attribute__((address_space(4))) ChainArgs* ChainArgsPtr;
typedef const __attribute__((address_space(4))) StreamWorker* StreamWorkerPtr;

// t * magic >> shift is t / d for every t < 2^31: with l = ceil(log2 d) and magic =
// ceil(2^(31 + l) / d) the excess of magic * d over 2^(31 + l) is at most 2^l.
__device__ __forceinline__ uint32_t bucket_of(ChainArgsPtr a, uint32_t tile)
{
    return (uint32_t)((tile * a->bucket_magic) >> a->bucket_shift);
}

__device__ __forceinline__ PhiloxUniform uniform_keys(StreamWorkerPtr w)
{
    return {w->keys.c2, w->keys.c0, w->keys.c2b, w->keys.c3, w->keys.key0, w->keys.key1};
}

// The forms of the kernel (persistent_from has the rule): persistent waves with the
// hand-ordered fold, or one tile per wave -- of two rows, or of one where the vector is so short
// that a wave's own latency is the launch's time (4 workers of 1 M elements: 5.6 us
// against 6.4; 8: 7.3 against 8.4).
enum ChainForm { kPiped = 0, kOneTile = 1, kOneRow = 2 };
template <int FORM> struct ChainStreamTile {
    static constexpr int ROWS = FORM == kOneRow ? 1 : kChainRows;
    static constexpr uint32_t N = kWave * kLaneElems * ROWS;
};

template <int ROWS> struct ChainCodes { uint32_t w[ROWS]; float step; };

// a lane's eight codes of a row: WIDTH bytes
template <int WIDTH>
__device__ __forceinline__ uint32_t lane_codes(const unsigned char* p)
{
    if constexpr (WIDTH == 1) return *p;
    if constexpr (WIDTH == 2) return *(const uint16_t*)p;
    if constexpr (WIDTH == 4) return *(const uint32_t*)p;
    uint16_t low;                     // three bytes at any address, and none behind them
    __builtin_memcpy(&low, p, 2);
    return (uint32_t)low | (uint32_t)p[2] << 16;
}

// The size of a stream of n codes, and what is left of it for the vector's last lane, whose eight codes need not all exist.
// Only for 3-bit codes (16 is no multiple of three) can that be less than the eight codes' bytes.
__device__ __forceinline__ uint64_t stream_bytes(uint64_t n, uint32_t width)
{
    return (((n * width + 7u) >> 3) + 15u) & ~(uint64_t)15u;
}
template <int WIDTH>
__device__ __forceinline__ bool last_lane_is_short(uint64_t n)
{
    return WIDTH == 3 && stream_bytes(n, 3u) - (n - 1u) / 8u * 3u < 3u;
}

// a lane's eight codes of a row: `WIDTH` bytes at a multiple of WIDTH (full tiles).
// `limit`: the largest byte offset inside the tile's codes that may be read (a multiple of
// WIDTH); lanes past it read there instead.  Whole tiles pass 0xFFFFFFFF; for the vector's
// ragged last tile it is the stream's last WIDTH bytes, so that the tile can be fetched and
// folded like a whole one (what lanes past the end compute is never stored).
template <int WIDTH, int ROWS>
__device__ __forceinline__ void stream_fetch(const unsigned char* codes, uint64_t start, int lane, ChainCodes<ROWS>& f,
                                             uint32_t limit = 0xFFFFFFFFu)
{
    const unsigned char* tile = codes + (start >> 3) * WIDTH;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        uint32_t off = (uint32_t)(r * kWave + lane) * WIDTH;
        off = off < limit ? off : limit;
        f.w[r] = lane_codes<WIDTH>(tile + off);
    }
    f.step = 0.0f;     // whole tiles take their steps from the step lanes of the kernel
}

// The same for the vector's ragged last tile of `len` elements: a lane fetches its bytes
// only if its first code exists (they then lie inside the stream, whose size is padded to
// a multiple of 16 bytes: (o/8 + 1) * WIDTH <= the padded size of the tile's codes; three bytes each by itself,
// see last_lane_is_short).
template <int WIDTH, int ROWS>
__device__ __forceinline__ void stream_fetch_ragged(const unsigned char* codes, const float* steps, uint64_t n, uint64_t start,
                                                    uint32_t len, uint32_t bucket, int lane, ChainCodes<ROWS>& f)
{
    const unsigned char* mine = codes + (start >> 3) * WIDTH + (uint32_t)lane * WIDTH;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const unsigned char* p = mine + (uint32_t)(r * kWave) * WIDTH;
        f.w[r] = 0u;
        if ((uint32_t)(r * kWave + lane) * kLaneElems < len) {
            if constexpr (WIDTH == 3) {
                const uint64_t left = stream_bytes(n, 3u) - (uint64_t)(p - codes);
                f.w[r] = p[0];
                if (left > 1u) f.w[r] |= (uint32_t)p[1] << 8;
                if (left > 2u) f.w[r] |= (uint32_t)p[2] << 16;
            } else {
                f.w[r] = lane_codes<WIDTH>(p);
            }
        }
    }
    f.step = steps[bucket];
}

// `block`: low word of the number of the lane's first block (the high word is the same for the whole
// call and part of the keys).
template <int MODE, int WIDTH, bool FIRST, int ROWS>
__device__ __forceinline__ void stream_fold(const PhiloxUniform& keys, uint32_t block, uint32_t extra, float ratio, float inv_ratio,
                                            const ChainCodes<ROWS>& f, float step, float inv, float (&S)[ROWS][8])
{
    constexpr int NF = WIDTH > 2 ? 4 : 8;       // fields of a group that stay inside 23 bits
    // a power-of-two nesting ratio is 2^(code width): M and 1/M are compile-time constants
    constexpr float M_f = (float)(1u << WIDTH), inv_M_f = 1.0f / M_f;
    // DQSG: the code c itself, the index offset q_min going into the dither instead:
    // (c + q_min) - v and c - (v - q_min) are the same exact value rounded once, and
    // v - q_min is exact for |q_min| <= 8 (code widths up to 4 bits); raised by 64.5, the dither
    // leaves c + 64.5 to subtract it from.  Nested: m' = c / M (a ratio that is no power of two: c).
    const FieldScaled<NF> field((uint32_t)WIDTH, MODE == kNestedPow2 ? (uint32_t)WIDTH : 0u, MODE == kDq ? 64.5f : 0.0f);
    Quant qp;                       // (what the coset decoder and `shrink` read of it)
    qp.M_f = ratio;
    qp.inv_M_f = inv_ratio;
    qp.alpha = 1.0f;                // (an infinite running mean becomes NaN, as in chain_kernel: 0 times it is added, which costs 0 to 2 %)
    qp.beta = 0.0f;
    const uint32_t dither_bits = MODE == kDq ? kDitherBits - (extra << 17) : kDitherBits;
    const float side_scale = __uint_as_float(extra);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        PhiloxFlight fl;
        fl.start(keys, block + (uint32_t)(r * kWave));
        fl.run();
        uint32_t words[4];
        fl.words(words);
        const uint32_t lo = f.w[r], hi = f.w[r] >> (NF == 4 ? 4 * WIDTH : 0);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float x = (k & 1) ? dither_raised<true>(words[k >> 1], dither_bits)
                                    : dither_raised<false>(words[k >> 1], dither_bits);
            const float c_f = NF == 8 ? field.get(lo, k) : field.get(k < 4 ? lo : hi, k & 3);
            float val;
            if (MODE == kDq) {
                val = step * (c_f - x);
            } else if (MODE == kNestedAnyM) {
                const float v = x - 64.5f;
                const float y = S[r][k] * side_scale;
                val = shrink<kNestedAnyM>(index_value(coset_index_f<kNestedAnyM>(c_f, y, inv, v, qp), step, v), y, qp);
            } else {
                const float v = x - 64.5f;
                const float y = S[r][k] * side_scale;
                const float c = __builtin_fmaf(y, inv, v);
                const float kk = __builtin_rintf(__builtin_fmaf(c, inv_M_f, -c_f));
                const float qs = kk + c_f;
                const float centred = __builtin_fmaf(qs, M_f, -v);
                val = step * centred;
            }
            S[r][k] = FIRST ? val : S[r][k] + val;
        }
    }
}

// The same fold with fewer and cheaper instructions, in a fixed order, and one Philox
// block (the dither of a later row) advanced by its ten rounds in between.
// Bound by instruction issue (a wave64 fma, add, xor, and: 2.45 cycles of a SIMD; the 32x32
// multiply 4.6; round-to-integer, conversions, 16-bit multiply 4.2, and a binary32 operation
// beside one of these is almost free unless it is a sub-dword (SDWA) form).  133
// vector instructions per row and nested 1-bit worker, 143 before; 4 workers of 2^27
// elements: 204 -> 188 us, 16 workers of 11.2 M: 76 -> 69 us, and no more register spills (with the worker's
// parameters worked out by the host, see StreamWorker, 181 and 65):
// - The dither goes through the mantissa: the bits of 64 + 2^-17 plus twice the cell are
//   the float 64 + (cell + 1/2) 2^-16 (v_mad_u32_u16, which takes the low half of a word; the
//   half-word conversions it replaces are SDWA), and an exact subtraction follows.  DQSG:
//   c - (x - 64.5) = (c + 64.5) - x needs not even that.
// - A 1-bit code j, shifted to bits 23..30, is masked in place: alone in the exponent field
//   it is the float 0 or 2^(2^j - 127), and m' = m/2 comes out of the fma that uses it, as a
//   product with 2^(126 - 2^j).  This fold is divided by M = 2 throughout,
//     c' = fma(y, 1/(M Delta), v/M)   k = rint(c' - m')   q' = k + m'   S = S + (M Delta) (q' - v/M)
//   which is exact, and S that of stream_fold bit for bit, while every step of the tile is 0
//   or in [2^-60, 2^50]: then |S| < 2^60 and |c'| < 2^120.  Tiles with another step are
//   decoded again in the plain form afterwards (step_out_of_range).
// - What the Philox rounds do with wave-uniform operands is done on the host (PhiloxUniform):
//   two of the twenty multiplies, three of the forty other operations.
// - Order: the slow instructions are spread among the float operations (RowProgram); the
//   compiler's own order has them in runs.
__device__ __forceinline__ bool step_out_of_range(float step)
{
    return step > 0x1p50f || (step < 0x1p-60f && step != 0.0f);
}

// The order of a row's instructions, made at compile time: element k runs through its
// stages `lag` steps behind element k - 1, so that at any place operations of about
// (stages / lag) elements and of different kinds stand next to each other; the Philox
// block's multiplies and xors are spread evenly among them.
//   nested  x raised dither  v dither/M  a masked code [b m']  y S/count  c c'  t c' - m'  r rint
//           q + m'  d - v/M  p times M Delta  s added to S
//           a ratio that is no power of two: undivided, and between t and r the quotient of divide_by_ratio in its three
//           pieces Q R N (S and c are finite where the steps are in range, so it needs no fix-up, nor 0 times y added)
//   DQSG    x raised dither  a masked code  b c + 64.5  d minus x  p times Delta  [s added to S]
//   m, X    the next multiply, the next xor of the Philox block
struct RowProgram {
    char op[176];
    uint8_t element[176];
    int n;
};
constexpr RowProgram row_program(const char* stages, int lag)
{
    const char philox[] = "mXmXXmmXXmmXXmmXXmmXXmmXXmmXXmmXXmmXX";
    constexpr int kPhilox = sizeof(philox) - 1;
    int count = 0;
    while (stages[count] != 0) ++count;
    const int own = 8 * count;
    RowProgram p = {};
    int done = 0, advanced = 0;
    for (int t = 0; t < count + 7 * lag; ++t)
        for (int k = 0; k < 8; ++k) {
            const int s = t - lag * k;
            if (s < 0 || s >= count) continue;
            p.op[p.n] = stages[s];
            p.element[p.n++] = (uint8_t)k;
            ++done;
            for (; advanced < done * kPhilox / own; ++advanced) p.op[p.n++] = philox[advanced];
        }
    return p;
}
// Elements two stages apart: 188 us where 1 gives 193 and 3 gives 190 (4 workers, 2^27 elements).
constexpr int kRowLag = 2;

// nested workers with 1-bit codes take the fold divided by M
template <int MODE, int WIDTH> struct RowScaled { static constexpr bool value = MODE == kNestedPow2 && WIDTH == 1; };
// folds that are only right while the steps are in range
template <int MODE, int WIDTH> struct RowRanged { static constexpr bool value = RowScaled<MODE, WIDTH>::value || MODE == kNestedAnyM; };
template <int MODE, int WIDTH, bool FIRST> struct RowOrder {
    static constexpr bool BIT = RowScaled<MODE, WIDTH>::value;
    static constexpr RowProgram program =
        row_program(MODE == kDq ? (FIRST ? "xabdp" : "xabdps") : MODE == kNestedAnyM ? "xvabyctQRNrqdps"
                                : BIT ? "xvayctrqdps" : "xvabyctrqdps", kRowLag);
};

template <int MODE, int WIDTH, bool FIRST>
struct RowFold {
    static constexpr bool BIT = RowOrder<MODE, WIDTH, FIRST>::BIT;
    static constexpr int NF = WIDTH > 2 ? 4 : 8;
    static constexpr float M_f = (float)(1u << WIDTH), inv_M_f = 1.0f / M_f;
    const uint32_t (&words)[4];
    uint32_t code, code_hi, dither_bits;
    float step, inv, side_scale, ratio, inv_ratio;
    float (&S)[8];
    PhiloxFlight& fl;
    float x[8], v[8], m[8], w[8], z[8];

    template <int I> __device__ __forceinline__ void run()
    {
        constexpr char op = RowOrder<MODE, WIDTH, FIRST>::program.op[I];
        constexpr int k = RowOrder<MODE, WIDTH, FIRST>::program.element[I];
        constexpr int j = NF == 8 ? k : (k & 3);
        constexpr float bit_scale = __builtin_bit_cast(float, (uint32_t)(253u - (1u << (k & 7))) << 23);   // 2^(126 - 2^k)
        constexpr uint32_t mask = ((1u << WIDTH) - 1u) << (j * WIDTH);
        constexpr uint32_t base = (150u - j * WIDTH - (MODE == kNestedPow2 ? WIDTH : 0u)) << 23;
        constexpr bool ANY = MODE == kNestedAnyM;
        if constexpr (op == 'm') fl.next_multiply();
        if constexpr (op == 'X') fl.next_xor();
        if constexpr (op == 'x') x[k] = dither_raised<(k & 1) != 0>(words[k >> 1], dither_bits);
        if constexpr (op == 'v') v[k] = x[k] - (BIT ? 64.5f * inv_M_f : 64.5f);
        if constexpr (op == 'a' && BIT) m[k] = __uint_as_float(code & (1u << (23 + k)));
        if constexpr (op == 'a' && !BIT)
            m[k] = __uint_as_float(__builtin_amdgcn_bitop3_b32(NF == 8 || k < 4 ? code : code_hi, mask, base, 0xEA));
        if constexpr (op == 'b') m[k] = m[k] - (__builtin_bit_cast(float, base) - (MODE == kDq ? 64.5f : 0.0f));
        if constexpr (op == 'y') w[k] = S[k] * side_scale;
        if constexpr (op == 'c') w[k] = __builtin_fmaf(w[k], inv, v[k]);
        if constexpr (op == 't') w[k] = ANY ? w[k] - m[k] : BIT ? __builtin_fmaf(m[k], -bit_scale, w[k]) : __builtin_fmaf(w[k], inv_M_f, -m[k]);
        if constexpr (op == 'Q') z[k] = w[k] * inv_ratio;
        if constexpr (op == 'R') w[k] = __builtin_fmaf(-ratio, z[k], w[k]);
        if constexpr (op == 'N') w[k] = __builtin_fmaf(w[k], inv_ratio, z[k]);
        if constexpr (op == 'r') w[k] = __builtin_rintf(w[k]);
        if constexpr (op == 'q') w[k] = ANY ? __builtin_fmaf(w[k], ratio, m[k]) : BIT ? __builtin_fmaf(m[k], bit_scale, w[k]) : w[k] + m[k];
        if constexpr (op == 'd') w[k] = MODE == kDq ? m[k] - x[k] : BIT || ANY ? w[k] - v[k] : __builtin_fmaf(w[k], M_f, -v[k]);
        if constexpr (op == 'p' && FIRST) S[k] = step * w[k];
        if constexpr (op == 'p' && !FIRST) w[k] = step * w[k];
        if constexpr (op == 's') S[k] = S[k] + w[k];
        NDQ_PIN();
    }
    template <int... I> __device__ __forceinline__ void run_all(std::integer_sequence<int, I...>) { (run<I>(), ...); }
};

template <int MODE, int WIDTH, bool FIRST>
__device__ __forceinline__ void fold_row_piped(const uint32_t (&words)[4], uint32_t code, float step, float inv,
                                               uint32_t extra, float ratio, float inv_ratio, float (&S)[8], PhiloxFlight& fl)
{
    using Fold = RowFold<MODE, WIDTH, FIRST>;
    // raised dither: v + 64 (DQSG: v - q_min + 64, so that c minus it is (c + q_min) - v; nested: divided by M)
    const uint32_t dither_bits = MODE == kDq ? kDitherBits - (extra << 17)
                                             : Fold::BIT ? kDitherBits - ((uint32_t)WIDTH << 23) : kDitherBits;
    Fold f = {words, Fold::BIT ? code << 23 : code, code >> (4 * WIDTH), dither_bits, step, inv, __uint_as_float(extra),
              ratio, inv_ratio, S, fl, {}, {}, {}, {}, {}};
    f.run_all(std::make_integer_sequence<int, RowOrder<MODE, WIDTH, FIRST>::program.n>());
}

// Folds a worker's two rows.  While a row is folded the Philox block of the next one is on its
// way: the second row's with this worker's keys, then the next worker's first with its keys.
template <int MODE, int WIDTH, bool FIRST>
__device__ __forceinline__ void stream_fold_piped(const PhiloxUniform& keys, uint32_t block, const PhiloxUniform& keys_next,
                                                  uint32_t block_next, uint32_t extra, float ratio, float inv_ratio,
                                                  const ChainCodes<kChainRows>& f, const float (&step)[kChainRows],
                                                  const float (&inv)[kChainRows], float (&S)[kChainRows][8], PhiloxFlight& fl)
{
#pragma unroll
    for (int r = 0; r < kChainRows; ++r) {
        uint32_t words[4];
        fl.words(words);
        if (r + 1 < kChainRows) fl.start(keys, block + (uint32_t)((r + 1) * kWave));
        else fl.start(keys_next, block_next);
        fold_row_piped<MODE, WIDTH, FIRST>(words, f.w[r], step[r], inv[r], extra, ratio, inv_ratio, S[r], fl);
    }
}

// The ragged last tile with the same folds: lanes past the end decode zeros and store nothing.
template <int RMODE, int W0, int WR, bool MIXED, int ROWS>
__device__ __forceinline__ void stream_ragged_tile(ChainArgsPtr a, uint64_t start, uint32_t len, uint32_t bucket,
                                                   int lane)
{
    const uint32_t W = a->W;
    const uint32_t block = (uint32_t)(start >> 3) + (uint32_t)lane;
    float S[ROWS][8];
    ChainCodes<ROWS> cur, nxt;
    const uint32_t dq = MIXED ? a->dq : 1u;
    auto fetch = [&](uint32_t w) __attribute__((always_inline)) {
        if (MIXED && w < dq) stream_fetch_ragged<W0, ROWS>(a->w[w].codes, a->steps[w], a->n, start, len, bucket, lane, nxt);
        else stream_fetch_ragged<WR, ROWS>(a->w[w].codes, a->steps[w], a->n, start, len, bucket, lane, nxt);
    };
    stream_fetch_ragged<W0, ROWS>(a->w[0].codes, a->steps[0], a->n, start, len, bucket, lane, cur);
    nxt = cur;
    if (W > 1u) fetch(1u);
    stream_fold<kDq, W0, true, ROWS>(uniform_keys(&a->w[0]), a->w[0].block + block, a->w[0].extra, 0.0f, 0.0f, cur, cur.step,
                                     0.0f, S);
    cur = nxt;
    for (uint32_t w = 1; w < W; ++w) {
        if (w + 1u < W) fetch(w + 1u);
        if (MIXED && w < dq)
            stream_fold<kDq, W0, false, ROWS>(uniform_keys(&a->w[w]), a->w[w].block + block, a->w[w].extra, 0.0f, 0.0f, cur,
                                              cur.step, 0.0f, S);
        else
            stream_fold<RMODE, WR, false, ROWS>(uniform_keys(&a->w[w]), a->w[w].block + block, a->w[w].extra, a->ratio, a->inv_ratio,
                                                cur, cur.step, inv_step(cur.step), S);
        cur = nxt;
    }
    float* out = a->out + start;
    const float scale = a->scale;
    const bool apply_scale = a->apply_scale != 0;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const uint32_t o = (uint32_t)(r * kWave + lane) * kLaneElems;
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k)
            if (o + k < len) out[o + k] = apply_scale ? scale * S[r][k] : S[r][k];
    }
}

// The wave's tiles that have a step outside the range fold_row_piped is exact in, decoded
// again in the plain form; `last_too`: and the last tile.
template <int RMODE, int W0, int WR, bool MIXED, bool ROWB>
__device__ __forceinline__ void redo_out_of_range(ChainArgsPtr a, uint32_t first, uint32_t stride,
                                                           uint32_t tiles_all, bool last_too, int lane)
{
    constexpr bool RANGED = RowRanged<RMODE, WR>::value;
    const uint32_t W = a->W;
    const float* my_steps = a->steps[(uint32_t)lane < W ? (uint32_t)lane : W - 1u];
    constexpr int ROWS = ROWB ? 1 : kChainRows;          // rows that share a step
    constexpr uint32_t PART = kWave * kLaneElems * ROWS;
    for (uint32_t tile = first; tile < tiles_all; tile += stride)
        for (uint32_t r = 0; r < kChainTile / PART; ++r) {
            const uint64_t start = (uint64_t)tile * kChainTile + r * PART;
            if (start >= a->n) break;
            const uint32_t bucket = ROWB ? tile * kChainRows + r : bucket_of(a, tile);
            const bool last = last_too && tile + 1u == tiles_all;
            if (!last && (!RANGED || __builtin_amdgcn_ballot_w64(step_out_of_range(my_steps[bucket])) == 0)) continue;
            const uint64_t left = a->n - start;
            stream_ragged_tile<RMODE, W0, WR, MIXED, ROWS>(a, start, left < PART ? (uint32_t)left : PART, bucket, lane);
        }
}

// The one-tile forms of few workers are bound by their stores: a lane's eight results are 32 bytes, so a store of 16 bytes a
// lane half-writes every sector (see PIPED below).  Four neighbouring lanes put their results in order first (quad
// permutations, 24 instructions a row), and the two stores that share 128-byte lines follow each other at once (with the second's
// permutations between them half of the gain is lost): 2 DQSG workers of 5.2 M elements 7.9 -> 6.2 us, 1 + 1 nested of 8.4 M
// 10.9 -> 8.8, 3 DQSG of 8.4 M 10.9 -> 10.2; from four workers on (three with nested ones) the
// instructions cost as much as the stores gain, or 1-2 % more.
__device__ __forceinline__ void store_row_lines(float* row, int lane, const float (&s)[8])
{
    const bool odd = (lane & 1) != 0;
    float front[4], back[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int lo = (int)__float_as_uint(s[k]), hi = (int)__float_as_uint(s[4 + k]);
        // quad_perm [0,0,1,1]: the sixteen results of the first two lanes; [2,2,3,3]: of the other two
        const int fl = __builtin_amdgcn_update_dpp(0, lo, 0x50, 0xF, 0xF, false);
        const int fh = __builtin_amdgcn_update_dpp(0, hi, 0x50, 0xF, 0xF, false);
        const int bl = __builtin_amdgcn_update_dpp(0, lo, 0xFA, 0xF, 0xF, false);
        const int bh = __builtin_amdgcn_update_dpp(0, hi, 0xFA, 0xF, 0xF, false);
        front[k] = __uint_as_float((uint32_t)(odd ? fh : fl));
        back[k] = __uint_as_float((uint32_t)(odd ? bh : bl));
    }
    float* p = row + (lane & ~3) * 8 + (lane & 3) * 4;
    __builtin_amdgcn_sched_barrier(0);        // the two stores next to each other: they share their 128-byte lines
    store_streaming(p, front[0], front[1], front[2], front[3]);
    store_streaming(p + 16, back[0], back[1], back[2], back[3]);
}

// RAGGED: the vector ends in a ragged tile.  An instantiation of its own, because the mere
// presence of that code in the kernel measured 6 % on the main loop (config 5, which has
// no ragged tile: 215 against 203 us) although the loop's instructions are the same.
// Without PIPED one wave folds that tile with guarded code of its own (stream_ragged_tile).
// With PIPED it is one more tile of the loop: its codes are fetched with the lane offsets
// clamped to the end of the stream, it is folded like a whole tile, and only its copy-out is
// guarded (a persistent ragged launch in the plain form is 7-9 % slower than one tile per
// wave at two to three tiles per wave slot, where the piped form is 1-5 % faster).
//
// PIPED (persistent launches of whole tiles): two changes that only pay together.
// (1) A lane's eight consecutive results are 32 bytes of the output, so a 16-byte store per
// lane writes every other 16 bytes of a 2 KB span, and such half-written sectors sustain only
// 2.6 TB/s: with the arithmetic taken out the stores alone took as long as the whole kernel
// (206 us at n = 2^27; 105 us when every store writes 1 KB of consecutive bytes).  The tile
// therefore leaves through the wave's 4 KB of LDS as four stores of consecutive bytes.
// (2) stream_fold_piped: the fold's instructions in a fixed order with the next row's Philox
// block advanced in between.
// It starts one extra Philox block per wave, which a wave with several tiles or many workers to
// fold amortises, and the LDS round trip costs a one-tile wave more than the stores do: the one-tile
// forms keep the plain fold, and persistent_from says from where on this one is taken.
#ifndef NDQ_CHAIN_PIPED_WAVES
#define NDQ_CHAIN_PIPED_WAVES NDQ_CHAIN_STREAM_WAVES
#endif
// LINES: one tile per wave, its results stored with store_row_lines.
// MIXED: the first `dq` workers are DQSG, the rest nested; a loop for each kind.
// ROWB (persistent): a bucket is one row, so a tile has a step for each of its rows.
template <int RMODE, int W0, int WR, bool MIXED, bool ROWB, bool RAGGED, bool LINES, int FORM>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(FORM == kPiped ? NDQ_CHAIN_PIPED_WAVES : kChainStreamWaves, FORM == kPiped ? NDQ_CHAIN_PIPED_WAVES : kChainStreamWaves)))
void chain_stream_kernel(ChainArgs a_by_value)
{
    constexpr bool PIPED = FORM == kPiped;
    constexpr bool TAIL = RAGGED && PIPED;     // the ragged tile runs through the main loop
    constexpr int ROWS = ChainStreamTile<FORM>::ROWS;
    constexpr uint32_t TILE = ChainStreamTile<FORM>::N;
    constexpr bool SCALED = PIPED && RowScaled<RMODE, WR>::value, RANGED = PIPED && RowRanged<RMODE, WR>::value;
    constexpr float kM = SCALED ? (float)(1u << WR) : 1.0f, kInvM = 1.0f / kM;
    const ChainArgsPtr a = (ChainArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t stride = gridDim.x * kWavesPerBlock;
    const uint32_t wave_in_block = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t first = blockIdx.x * kWavesPerBlock + wave_in_block;
    __shared__ __align__(16) float out_stage_all[PIPED ? kWavesPerBlock : 1][PIPED ? TILE : 4];
    float* out_stage = out_stage_all[PIPED ? wave_in_block : 0u];
    const uint32_t tiles = a->tiles;                       // whole tiles: ids 0 .. tiles-1
    const uint32_t tiles_all = TAIL ? tiles + 1u : tiles;  // TAIL: and the ragged one, id `tiles`
    const uint32_t W = a->W, dq = MIXED ? a->dq : 1u;
    float* out_base = a->out;
    const float scale = a->scale;
    const bool apply_scale = __builtin_amdgcn_readfirstlane(a->apply_scale) != 0;
    const float ratio = RMODE == kNestedAnyM ? a->ratio : 0.0f, inv_ratio = RMODE == kNestedAnyM ? a->inv_ratio : 0.0f;
    // The ragged last tile goes first, to a wave that has no whole tile if the grid has one
    // (one tile per wave), else to wave 0: at the start every SIMD is full and hides its
    // latencies; as a kernel of its own, or at the end, it would run alone at a fifth of the rate.
    const uint64_t whole = (uint64_t)tiles * TILE;
    if (RAGGED && !PIPED && whole < a->n && first == (stride > tiles ? tiles : 0u))
        stream_ragged_tile<RMODE, W0, WR, MIXED, ROWS>(a, whole, (uint32_t)(a->n - whole), bucket_of(a, tiles), lane);
    if (first >= tiles_all) return;
    const uint32_t my_tiles = (tiles_all - first + stride - 1u) / stride;
    // TAIL: elements of the ragged tile, and per code width the last byte offset inside its
    // codes that a lane may read: the stream is padded to a multiple of 16 bytes, the tile
    // starts at one, so at least 16 bytes of it exist
    const uint32_t tail_len = TAIL ? (uint32_t)(a->n - whole) : 0u;
    auto tail_limit = [&](uint32_t width) __attribute__((always_inline)) {
        const uint64_t total = ((((uint64_t)a->n * width + 7u) >> 3) + 15u) & ~(uint64_t)15u;
        return (uint32_t)(total - (whole >> 3) * width) - width;
    };
    const uint32_t limit0 = TAIL ? tail_limit((uint32_t)W0) : 0xFFFFFFFFu;
    const uint32_t limitr = TAIL ? tail_limit((uint32_t)WR) : 0xFFFFFFFFu;
    auto limit_for = [&](uint32_t tile_id, uint32_t tail) __attribute__((always_inline)) {
        return (TAIL && tile_id == tiles) ? tail : 0xFFFFFFFFu;
    };
    // a wave's priority (see the end of the loop) steps down at these numbers of tiles done
    const uint32_t lower2 = (my_tiles + 3u) / 4u, lower1 = (my_tiles + 1u) / 2u, lower0 = (3u * my_tiles + 3u) / 4u;
    uint32_t done = 0;
    if (my_tiles > 1u) __builtin_amdgcn_s_setprio(3);

    const StreamWorkerPtr first_worker = &a->w[0], end_worker = &a->w[W];
    constexpr bool WARM = FORM == kOneRow;      // (longer launches: nothing gained)
    uint32_t warm = 0u;
    if (WARM && W > 1u) warm = read_arguments_ahead(a, W * (uint32_t)sizeof(StreamWorker), lane);
    ChainCodes<ROWS> cur;
    stream_fetch<W0, ROWS>(first_worker->codes, (uint64_t)first * TILE, lane, cur, limit_for(first, limit0));
    // PIPED: the dither of the row after the current one is always in flight; here the first row's
    PhiloxUniform keys = uniform_keys(first_worker);
    PhiloxFlight fl;
    if (PIPED) {
        fl.start(keys, first_worker->block + first * (TILE / kLaneElems) + (uint32_t)lane);
        fl.run();
    }
    // Lane w looks after worker w's step: one load and ONE correctly rounded division per tile
    // for all workers (at most 32, one per lane), instead of one per worker in every lane; a
    // worker's step and reciprocal are then read from its lane into scalar registers.
    const float* my_steps = a->steps[(uint32_t)lane < W ? (uint32_t)lane : W - 1u];
    constexpr int STEPS = ROWB ? ROWS : 1;
    auto load_steps = [&](uint32_t tile, float (&to)[STEPS]) __attribute__((always_inline)) {
        if constexpr (ROWB) {
            const uint32_t last = (uint32_t)((a->n - 1u) / (kWave * kLaneElems));
#pragma unroll
            for (int r = 0; r < STEPS; ++r) {
                const uint32_t b = tile * ROWS + (uint32_t)r;
                to[r] = my_steps[b < last ? b : last];       // (a row behind the end is not stored: any step will do)
            }
        } else {
            to[0] = my_steps[bucket_of(a, tile)];
        }
    };
    float steps_ahead[STEPS];
    load_steps(first, steps_ahead);
    bool out_of_range = false;
    for (uint32_t tile = first; tile < tiles_all; tile += stride) {
        const uint64_t start = (uint64_t)tile * TILE;
        // the wave's next tile (after the last one: this one again, unused)
        const uint32_t next = tile + stride < tiles_all ? tile + stride : tile;
        const uint32_t block_here = tile * (TILE / kLaneElems) + (uint32_t)lane;
        const uint32_t block_ahead = next * (TILE / kLaneElems) + (uint32_t)lane;
        float S[ROWS][8];
        float steps_here[STEPS], invs_here[STEPS], scaled_here[STEPS];
#pragma unroll
        for (int r = 0; r < STEPS; ++r) steps_here[r] = steps_ahead[r];
        load_steps(next, steps_ahead);
#pragma unroll
        for (int r = 0; r < STEPS; ++r) {
            invs_here[r] = inv_step(steps_here[r]);
            scaled_here[r] = steps_here[r];
            if (SCALED) {
                invs_here[r] = invs_here[r] * kInvM;
                scaled_here[r] = steps_here[r] * kM;
            }
            if (RANGED) out_of_range = out_of_range || step_out_of_range(steps_here[r]);
        }
        auto from_lane = [](float x, uint32_t w) __attribute__((always_inline)) {
            return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), (int)w));
        };
        // Folds worker `w`, whose codes are in `cur`, and fetches the next worker's, or the first
        // worker's of the next tile.
        // `dq_follows`: MIXED, the next worker is DQSG too.
        auto fold = [&](auto mode, auto width, auto is_first, StreamWorkerPtr w, uint32_t index, bool dq_follows)
            __attribute__((always_inline)) {
            constexpr int MODE = decltype(mode)::value, WIDTH = decltype(width)::value;
            constexpr bool FIRST = decltype(is_first)::value;
            const bool last = w + 1 == end_worker;
            const StreamWorkerPtr wn = last ? first_worker : w + 1;
            const PhiloxUniform keys_next = uniform_keys(wn);
            const uint32_t extra = w->extra, here = w->block + block_here, ahead = wn->block + (last ? block_ahead : block_here);
            const unsigned char* codes_next = wn->codes;
            ChainCodes<ROWS> nxt;
            if (last) stream_fetch<W0, ROWS>(codes_next, (uint64_t)next * TILE, lane, nxt, limit_for(next, limit0));
            else if (MIXED && MODE == kDq && dq_follows) stream_fetch<W0, ROWS>(codes_next, start, lane, nxt, limit_for(tile, limit0));
            else stream_fetch<WR, ROWS>(codes_next, start, lane, nxt, limit_for(tile, limitr));
            float step[ROWS], inv[ROWS];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                step[r] = r < STEPS ? from_lane(MODE == kDq ? steps_here[r % STEPS] : scaled_here[r % STEPS], index) : step[0];
                inv[r] = MODE == kDq ? 0.0f : r < STEPS ? from_lane(invs_here[r % STEPS], index) : inv[0];
            }
            if constexpr (PIPED) stream_fold_piped<MODE, WIDTH, FIRST>(keys, here, keys_next, ahead, extra, ratio, inv_ratio, cur, step, inv, S, fl);
            else stream_fold<MODE, WIDTH, FIRST, ROWS>(keys, here, extra, ratio, inv_ratio, cur, step[0], inv[0], S);
            keys = keys_next;
            cur = nxt;
        };
        fold(std::integral_constant<int, kDq>{}, std::integral_constant<int, W0>{}, std::true_type{}, first_worker, 0u, MIXED && dq > 1u);
        if (WARM) arguments_read(warm);
        uint32_t index = 1u;
        StreamWorkerPtr w = first_worker + 1;
        if constexpr (MIXED)
            for (; index < dq; ++w, ++index)
                fold(std::integral_constant<int, kDq>{}, std::integral_constant<int, W0>{}, std::false_type{}, w, index, index + 1u < dq);
        for (; w != end_worker; ++w, ++index)
            fold(std::integral_constant<int, RMODE>{}, std::integral_constant<int, WR>{}, std::false_type{}, w, index, false);
        float* out = out_base + start;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const uint32_t o = (uint32_t)(r * kWave + lane) * kLaneElems;
            if (apply_scale) {       // wave-uniform
#pragma unroll
                for (int k = 0; k < 8; ++k) S[r][k] = scale * S[r][k];
            }
            if (PIPED) {
                *(float4*)(out_stage + o) = make_float4(S[r][0], S[r][1], S[r][2], S[r][3]);
                *(float4*)(out_stage + o + 4) = make_float4(S[r][4], S[r][5], S[r][6], S[r][7]);
            } else if (LINES) {
                store_row_lines(out + r * kWave * kLaneElems, lane, S[r]);
            } else {
                store_streaming(out + o, S[r][0], S[r][1], S[r][2], S[r][3]);
                store_streaming(out + o + 4, S[r][4], S[r][5], S[r][6], S[r][7]);
            }
        }
        if (PIPED) {
            wave_lds_sync();
            if (TAIL && tile == tiles) {       // the ragged tile: only the elements that exist
#pragma unroll
                for (int j = 0; j < (int)(TILE / (kWave * 4)); ++j) {
                    const uint32_t e = (uint32_t)(j * (kWave * 4) + lane * 4);
                    const float4 x = *(const float4*)(out_stage + e);
                    if (e + 4u <= tail_len) {
                        store_streaming(out + e, x.x, x.y, x.z, x.w);
                    } else {
                        if (e < tail_len) out[e] = x.x;
                        if (e + 1u < tail_len) out[e + 1u] = x.y;
                        if (e + 2u < tail_len) out[e + 2u] = x.z;
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < (int)(TILE / (kWave * 4)); ++j) {
                    const float4 x = *(const float4*)(out_stage + j * (kWave * 4) + lane * 4);
                    store_streaming(out + j * (kWave * 4) + lane * 4, x.x, x.y, x.z, x.w);
                }
            }
            wave_lds_sync();     // the next tile's writes come after these reads
        }
        // the arbiter serves the oldest wave of a SIMD first: lower a wave's priority as it
        // gets ahead, so that the waves of a SIMD finish together
        ++done;
        if (done == lower0) __builtin_amdgcn_s_setprio(0);
        else if (done == lower1) __builtin_amdgcn_s_setprio(1);
        else if (done == lower2) __builtin_amdgcn_s_setprio(2);
    }
    // (the main loop has read the bytes before the end in place of the last lane's if that has less than its three)
    constexpr bool THREE = TAIL && (W0 == 3 || WR == 3);
    const bool last_too = THREE && (last_lane_is_short<W0>(a->n) || last_lane_is_short<WR>(a->n));
    if ((RANGED && __builtin_amdgcn_ballot_w64(out_of_range) != 0) || (THREE && last_too))
        redo_out_of_range<RMODE, W0, WR, MIXED, ROWB>(a, first, stride, tiles_all, last_too, lane);
}

// ---------------------------------------------------------------------------
// Aggregation: Algorithm 1 server, "compute the average"
// ---------------------------------------------------------------------------
constexpr uint32_t kAggMax = 32;
struct AggArgs {
    const float* g[kAggMax];
    float* out;
    uint64_t n;
    uint32_t W;
    int continue_sum;   // start from out (partial sum of an earlier group of workers)
    int finish;         // multiply by scale
    float scale;
};

__global__ __launch_bounds__(kBlock) void aggregate_kernel(AggArgs a)
{
    const uint64_t i4 = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    const uint64_t i = i4 * 4;
    if (i >= a.n) return;
    if (i + 4 <= a.n) {
        float4 acc = a.continue_sum ? *(const float4*)(a.out + i) : make_float4(0.f, 0.f, 0.f, 0.f);
        for (uint32_t w0 = 0; w0 < a.W; w0 += 8) {
            float4 x[8];
#pragma unroll
            for (uint32_t j = 0; j < 8; ++j)
                if (w0 + j < a.W) x[j] = load_streaming_f4(a.g[w0 + j] + i);
#pragma unroll
            for (uint32_t j = 0; j < 8; ++j)
                if (w0 + j < a.W) {
                    acc.x = acc.x + x[j].x; acc.y = acc.y + x[j].y;
                    acc.z = acc.z + x[j].z; acc.w = acc.w + x[j].w;
                }
        }
        if (a.finish) { acc.x = a.scale * acc.x; acc.y = a.scale * acc.y; acc.z = a.scale * acc.z; acc.w = a.scale * acc.w; }
        store_streaming(a.out + i, acc.x, acc.y, acc.z, acc.w);
    } else {
        for (uint64_t e = i; e < a.n; ++e) {
            float acc = a.continue_sum ? a.out[e] : 0.0f;
            for (uint32_t w = 0; w < a.W; ++w) acc = acc + a.g[w][e];
            a.out[e] = a.finish ? a.scale * acc : acc;
        }
    }
}

// ---------------------------------------------------------------------------
// Algorithm 1's server as printed, in one pass: every DQSG worker's gradient is
// reconstructed and kept, and their sum leaves with them.  Bound by the memory it writes, 4 (W + 1)
// bytes per element; decoding and then aggregating reads the 4 W bytes back (W = 4 at
// 1.66 M elements: 4 x 3.9 + 8.2 us, here 10.4; W = 2 at 37 M: 2 x 25 + 71, here 82 = 5.5 TB/s).  A lane owns four consecutive elements per row like the single
// decoders (16-byte stores of consecutive addresses), and the sum stays in its registers.
// ---------------------------------------------------------------------------
constexpr uint32_t kMeanMax = 32;      // workers per launch
constexpr int kMeanRows = 2;           // (1.66 M x 4 / 37 M x 2 elements: 1 row 11.5 / 87, 2 rows 10.4 / 82, 4 rows 10.7 / 79 us)
constexpr uint32_t kMeanTile = kWave * 4 * kMeanRows;
struct MeanWorker {
    const unsigned char* codes;
    const float* steps;
    float* decoded;
    uint64_t index0;
    DitherStream ds;
    int32_t q_min;
    uint32_t bits;
};
struct MeanArgs {
    MeanWorker w[kMeanMax];
    float* out;
    Tiling tl;
    uint32_t W;
    int continue_sum, finish;
    float scale;
    uint32_t bucket_blocks, last_bucket;    // SMALL: 64-element blocks per bucket; index of the last bucket
};
typedef const __attribute__((address_space(4))) MeanArgs* MeanArgsPtr;

// SMALL: buckets shorter than a tile.  The tiles then run over the whole vector, and a lane reads the
// step of its own bucket for every row (its four elements lie in one: a bucket is a multiple of 64):
// with a tile per bucket most lanes have nothing to do (buckets of 64, 11 M elements, one worker / four:
// 67 / 196 us, so 16 / 42; buckets of 320, 30 M x 4: 134 / 108).
//
// the words that hold a lane's four codes of every row (a ragged tail only counts its valid codes), and the steps
template <bool SMALL> struct MeanSteps { static constexpr int N = SMALL ? kMeanRows : 1; };    // per row, or one
template <bool FULL, bool SMALL>
__device__ __forceinline__ void mean_fetch(MeanArgsPtr a, uint32_t w, const TileRef& t, int lane,
                                           const uint32_t (&bucket)[MeanSteps<SMALL>::N],
                                           uint64_t (&window)[kMeanRows], float (&step)[MeanSteps<SMALL>::N])
{
    const uint32_t bits = a->w[w].bits;
    const uint32_t* codes32 = (const uint32_t*)(a->w[w].codes + (t.start >> 3) * bits);
#pragma unroll
    for (int r = 0; r < kMeanRows; ++r) {
        const uint32_t o = (uint32_t)(r * kWave + lane) * 4u;
        window[r] = 0;
        if (FULL || o < t.len) {
            const uint32_t ncodes = FULL ? 4u : (t.len - o < 4u ? t.len - o : 4u);
            const uint32_t word = (o * bits) >> 5, sh = (o * bits) & 31u;
            window[r] = codes32[word];
            if (sh + ncodes * bits > 32u) window[r] |= (uint64_t)codes32[word + 1] << 32;
        }
    }
#pragma unroll
    for (int r = 0; r < MeanSteps<SMALL>::N; ++r) step[r] = a->w[w].steps[bucket[r]];
}

// FEW: see kMeanFew.
template <bool FULL, bool SMALL, bool FEW>
__device__ __forceinline__ void mean_tile(MeanArgsPtr a, const TileRef& t, uint32_t tile_id, int lane)
{
    const uint32_t W = a->W;
    constexpr int STEPS = MeanSteps<SMALL>::N;
    uint32_t bucket[STEPS];
    if constexpr (SMALL) {
#pragma unroll
        for (int r = 0; r < STEPS; ++r) {
            const uint32_t b = (tile_id * (kMeanTile / 64u) + (uint32_t)(r * kWave + lane) / 16u) / a->bucket_blocks;
            bucket[r] = FULL || b < a->last_bucket ? b : a->last_bucket;       // lanes past the end: any step will do
        }
    } else {
        bucket[0] = t.bucket;
    }
    float acc[kMeanRows][4];
#pragma unroll
    for (int r = 0; r < kMeanRows; ++r)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t e = (uint32_t)(r * kWave + lane) * 4u + k;
            acc[r][k] = (a->continue_sum && (FULL || e < t.len)) ? a->out[t.start + e] : 0.0f;
        }
    uint32_t warm = 0u;
    if (W > 1u && a->tl.total_tiles < 4096u) warm = read_arguments_ahead(a, W * (uint32_t)sizeof(MeanWorker), lane);
    uint64_t window[kMeanRows], ahead[kMeanRows];
    float step[STEPS], step_ahead[STEPS] = {};
    mean_fetch<FULL, SMALL>(a, 0u, t, lane, bucket, window, step);
    for (uint32_t w = 0; w < W; ++w) {
        if (w + 1u < W) mean_fetch<FULL, SMALL>(a, w + 1u, t, lane, bucket, ahead, step_ahead);
        const DitherStream ds = {a->w[w].ds.key0, a->w[w].ds.key1, a->w[w].ds.step, a->w[w].ds.worker};
        const uint64_t quad0 = (a->w[w].index0 + t.start) >> 2;
        const uint32_t bits = a->w[w].bits;
        const int32_t q_min = a->w[w].q_min;
        float* decoded = a->w[w].decoded + t.start;
#pragma unroll
        for (int r = 0; r < kMeanRows; ++r) {
            const uint32_t o = (uint32_t)(r * kWave + lane) * 4u;
            const uint32_t packed = (uint32_t)(window[r] >> ((o * bits) & 31u));
            float v[4], res[4];
            dither4(ds, quad0 + (o >> 2), v);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t c = __builtin_amdgcn_ubfe(packed, k * bits, bits);
                res[k] = index_value((float)((int32_t)c + q_min), step[SMALL ? r : 0], v[k]);
                acc[r][k] = acc[r][k] + res[k];
            }
            if (FULL || o + 4u <= t.len) {
                store_streaming(decoded + o, res[0], res[1], res[2], res[3]);
            } else {
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k)
                    if (o + k < t.len) decoded[o + k] = res[k];
            }
        }
        if (FEW && w == 0u) arguments_read(warm);
#pragma unroll
        for (int r = 0; r < kMeanRows; ++r) window[r] = ahead[r];
#pragma unroll
        for (int r = 0; r < STEPS; ++r) step[r] = step_ahead[r];
    }
    if (!FEW) arguments_read(warm);
    float* out = a->out + t.start;
    const float scale = a->scale;
    const bool finish = a->finish != 0;
#pragma unroll
    for (int r = 0; r < kMeanRows; ++r) {
        const uint32_t o = (uint32_t)(r * kWave + lane) * 4u;
        float res[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) res[k] = finish ? scale * acc[r][k] : acc[r][k];
        if (FULL || o + 4u <= t.len) {
            store_streaming(out + o, res[0], res[1], res[2], res[3]);
        } else {
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k)
                if (o + k < t.len) out[o + k] = res[k];
        }
    }
}

// Workers up to which the read of the arguments is waited for after the first of them (see read_arguments_ahead).  After the last over this:
// 2 workers 1.00 to 1.03, 4 0.99 to 1.02 (4 of 3 levels, 1.66 M elements, whole call 22.95 -> 23.10 us), 8 0.98 to 1.05, 12 to 32 0.95 to 1.00.
constexpr uint32_t kMeanFew = 8;

template <bool SMALL, bool FEW>
__global__ __launch_bounds__(kBlock) void decode_mean_kernel(MeanArgs by_value)
{
    const MeanArgsPtr a = (MeanArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const Tiling tl = {a->tl.n, a->tl.bucket_len, a->tl.tiles_per_bucket, a->tl.total_tiles};
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t tile_id =
        blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const TileRef t = locate_tile(tl, tile_id, kMeanTile);
    if (t.len == kMeanTile) mean_tile<true, SMALL, FEW>(a, t, tile_id, lane);
    else if (t.len != 0) mean_tile<false, SMALL, FEW>(a, t, tile_id, lane);
}

// ---------------------------------------------------------------------------
// Host side: dispatch
// ---------------------------------------------------------------------------
template <int MODE, int ACC, bool STRADDLE>
static int run_decode3(DecodeArgs a, uint64_t n, uint32_t bucket, hipStream_t s)
{
    const int rc = make_tiling(n, bucket, DecTile<DecRows<MODE, ACC>::R>::N, &a.tl);
    if (rc != NDQ_OK) return rc;
    return launch((decode_kernel<MODE, ACC, STRADDLE>), dim3(blocks_for(a.tl.total_tiles)), dim3(kBlock), s, a);
}

template <int MODE, bool STRADDLE>
static int run_decode2(const DecodeArgs& a, uint64_t n, uint32_t bucket, int acc, hipStream_t s)
{
    if (acc == kStore) return run_decode3<MODE, kStore, STRADDLE>(a, n, bucket, s);
    if (acc == kAccumulate) return run_decode3<MODE, kAccumulate, STRADDLE>(a, n, bucket, s);
    return run_decode3<MODE, kAccumulateInPlace, STRADDLE>(a, n, bucket, s);
}

template <int MODE>
static int run_decode(const DecodeArgs& a, uint64_t n, uint32_t bucket, int acc, hipStream_t s)
{
    // four b-bit codes sit inside one 32-bit word exactly when 4b divides 32
    const bool straddle = (32u % (4u * a.qp.bits)) != 0u;
    return straddle ? run_decode2<MODE, true>(a, n, bucket, acc, s)
                    : run_decode2<MODE, false>(a, n, bucket, acc, s);
}

static int decode_common(const void* codes, size_t n, uint32_t levels, uint32_t M, bool nested,
                         bool half, float alpha, uint32_t bucket, const float* steps,
                         const ndq_dither* d,
                         const float* side, float side_scale, float* out, int accumulate,
                         void* stream)
{
    DecodeArgs a;
    int rc = make_quant(levels, M, nested, alpha, &a.qp);
    if (rc != NDQ_OK) return rc;
    if (!d) return NDQ_EINVAL;
    if (n == 0) return NDQ_OK;
    if (!codes || !steps || !out || (nested && !side)) return NDQ_EINVAL;
    if (n >= kMaxN) return NDQ_EUNSUPPORTED;
    if (!aligned16(codes) || !aligned16(out) || !aligned4(steps) || (nested && !aligned16(side)))
        return NDQ_EALIGN;
    if (bucket % 64u != 0u || (d->offset & 7u) != 0u) return NDQ_EALIGN;
    if (nested && side != out) {
        // partial overlap of side and out would race between waves
        const uintptr_t s0 = (uintptr_t)side, o0 = (uintptr_t)out, len = (uintptr_t)n * 4u;
        if (s0 < o0 + len && o0 < s0 + len) return NDQ_EINVAL;
    }
    a.codes = (const unsigned char*)codes;
    a.steps = steps;
    a.side = nested ? side : out;
    a.out = out;
    a.index0 = d->offset;
    a.ds = make_stream(d);
    a.side_scale = side_scale;
    hipStream_t s = (hipStream_t)stream;
    int acc = accumulate ? kAccumulate : kStore;
    if (nested && accumulate && side == out) acc = kAccumulateInPlace;
    if (!nested) return half ? run_decode<kDqHalf>(a, n, bucket, acc, s)
                             : run_decode<kDq>(a, n, bucket, acc, s);
    if (is_pow2(M) && alpha == 1.0f) return run_decode<kNestedPow2>(a, n, bucket, acc, s);
    if (is_pow2(M)) return run_decode<kNestedPow2Shrink>(a, n, bucket, acc, s);
    return run_decode<kNestedAnyM>(a, n, bucket, acc, s);
}

// Tiles (of 1,024 elements) from which the persistent form of chain_stream_kernel is taken, for `slots`
// wave slots.  With only a few tiles per wave a fixed share leaves SIMDs idle at the end; the hand-ordered fold makes
// up for it the sooner the more there is to fold.  Persistent time over one tile per wave's
// at 2.1 / 3.2 / 4.2 / 5.2 / 7.5 / 8.4 / 10.5 / 12.5 M elements:
//   1 DQSG    1.14 0.98 0.96 0.87 0.84 0.80 0.76 0.70   bound by its stores
//   2 DQSG    1.11 1.08 1.14 1.05 0.91 0.95 0.88 0.85
//   3 DQSG    1.06 1.04 1.06 1.08 1.04 1.07 0.98 0.98
//   4 DQSG    1.03 1.02 1.05 1.05 1.01 0.97 0.98 0.96
//   8 DQSG    0.99 1.02 1.01 1.02 1.06 1.01 1.00 0.99
//   2 (1 nested) 1.13 1.04 1.15 1.15 1.03 1.12 1.00 1.00
//   3 (2 nested) 1.09 1.05 1.11 1.06 1.05 1.04 1.02 1.00
//   4 (3 nested) 1.09 1.03 1.10 1.08 1.06 1.04 1.01 0.99
//   8 (7 nested) 1.02 1.00 1.03 1.03 1.01 1.01 1.00 1.01
//   16 (15 nested) 0.98 0.98 1.01 1.01 1.00 1.00 1.00 0.99
// Just above one tile per slot every plan takes it: a second round of one-tile waves is
// nearly empty (6.4 M: 2 workers 0.93 to 0.99, 3 DQSG 0.99, 4 DQSG 1.02, 4 with nested ones 1.06).
static uint32_t persistent_from(uint32_t W, bool all_dq, uint32_t slots)
{
    if (W == 1u) return kShortTiles;
    if (all_dq) return W == 2u || W >= 8u ? slots : slots / 2u * 3u;
    return W <= 3u ? 2u * slots : W < 8u ? slots : kShortTiles;
}

// The same for the rarer plans (see chain_streams), at 2.2 / 3.1 / 4.3 / 5.3 / 6.5 / 7.7 / 8.6 / 10.8 / 12.9 M elements:
//   3 bits, 1 DQSG   1.08 1.07 1.01 0.94 0.91 0.92 0.91 0.84 0.81
//           2 DQSG   1.05 1.04 1.05 1.07 1.00 0.99 0.97 0.98 0.94
//           4 DQSG   1.02 0.95 0.97 1.02 0.97 0.97 0.97 0.91 0.92
//           8 DQSG   0.97 0.88 0.93 0.96 0.91 0.95 0.94 0.87 0.90
//   1 + 1 nested     1.19 1.18 1.14 1.13 1.03 1.02 1.02 1.00 0.97
//   2 + 2            1.11 1.07 1.09 1.07 1.07 1.06 1.05 1.02 1.00
//   4 + 4            1.07 1.05 1.06 1.04 1.04 1.03 1.03 1.01 1.02
//   8 + 8            1.02 1.02 0.99 1.03 1.02 1.03 1.02 0.99 1.02
//   M = 3, 4 + 4     1.09 1.07 1.04 1.04 1.01 1.02 1.00 1.00 1.00
//          1 + 7     1.00 1.00 1.00 0.98 0.97 0.96 0.96 0.96 0.95
//          1 + 15    0.96 0.95 0.95 0.95 0.94 0.95 0.95 0.94 0.94
// (a second round that is nearly empty costs them no more than the persistent form does).  Buckets of a row, over one row per
// wave:  4 DQSG 1.15 1.08 1.04 0.99 1.00 0.99 0.99 0.95 0.93    1 + 1 1.19 1.09 1.04 0.99 0.97 0.94 0.93 0.89 0.86
//        M = 3, 1 + 1 1.42 1.33 1.25 1.16 1.09 1.04 1.01 0.96 0.96    8 + 8 1.16 1.03 1.08 0.96 1.04 1.00 1.01 0.98 0.98
static uint32_t rarer_persistent_from(uint32_t W, uint32_t dq, bool any_ratio, bool row_buckets, uint32_t slots)
{
    if (row_buckets) return slots / 3u * 4u;
    if (dq == W) return W == 1u ? slots / 4u * 3u : W < 8u ? slots : kShortTiles;
    return any_ratio && W - dq >= 7u ? kShortTiles : slots / 3u * 5u;
}

template <int RMODE, int W0, int WR, bool MIXED, bool ROWB = false>
static int launch_chain_stream(ChainArgs& a, uint64_t bucket_len, hipStream_t s)
{
    // Persistent waves, kChainStreamWaves on every SIMD, every wave with the same number of tiles (give or
    // take one), or one tile per wave: see persistent_from.
    const uint32_t slots = 1024u * kChainStreamWaves;
    const uint32_t full = (uint32_t)(a.n / kChainTile);
    const StreamTuning& tuning = stream_tuning();
    constexpr bool RARER = MIXED || W0 == 3 || ROWB;     // (see chain_streams)
    constexpr bool TWO_WIDTHS = RMODE == kDq && W0 != WR;
    // buckets of one row: ROWB has the persistent form only
    const bool rows_only = bucket_len < kChainTile && !ROWB;
    const uint32_t from = RARER ? rarer_persistent_from(a.W, RMODE == kDq ? a.W : a.dq, RMODE == kNestedAnyM, ROWB, slots)
                                : persistent_from(a.W, RMODE == kDq, slots);
    const bool persistent =
        full != 0u && !rows_only && (tuning.threshold_from_env ? full >= tuning.min_tiles_per_wave * slots
                                                               : full >= from || (!RARER && full >= slots && full < slots + slots / 16u));
    // Few workers of the rarer plans store whole lines from fewer tiles on: rows / tiles at 1.0, 1.3, 1.6, 2.0 M elements
    //   2 workers   4.63/4.67  5.32/5.05  5.79/5.13  6.12/5.40 (3-bit and a 2-bit nested)  4.35/4.39  4.70/4.69  5.06/4.73  5.42/4.94
    //   3           5.13/5.88  5.91/6.00  6.32/6.19  6.68/6.72                             4.76/5.17  5.17/5.54  5.79/5.49  6.10/5.68
    // Four and more workers of them take rows for longer, 3-bit DQSG ones almost until the chip holds a tile per wave slot: a second
    // round of rows is as full as the tiles' first.  chain_kernel / rows / tiles at 2.1, 2.4, 2.7, 3.6, 4.7 and 5.4 M elements
    //   4 x 8 levels                  7.0/6.2/7.4  7.8/6.9/8.7  8.3/7.6/8.5  9.2/9.1/9.4  11.2/10.4/11.1  12.4/11.8/10.4
    //   7 x 8 levels                  10.2/9.0/10.6  11.4/10.0/12.3  12.6/11.0/12.3  13.8/12.6/14.4  17.4/14.8/16.7  19.5/16.8/16.2
    //   4 x 16 levels, 4 x M = 4      13.3/10.9/11.4  13.6/11.4/11.7  15.2/12.8/11.7  17.0/14.6/14.1
    //   4 x 5 levels, 4 x M = 3       14.6/12.3/13.7  14.9/13.0/13.9  16.6/14.6/13.8  18.6/17.5/16.6
    //   16 levels, 7 x M = 8          14.2/13.1/14.8  14.5/13.6/15.2  16.2/15.2/15.1  17.9/18.1/18.1
    //   16 levels, 15 x M = 8         27.3/24.8/30.6  27.2/25.3/31.0  30.6/27.8/30.3  33.0/32.0/34.3  (tiles vary by a seventh with the length)
    const uint32_t rows_below = !RARER || a.W == 1u ? kShortTiles : a.W == 2u ? 1280u : a.W == 3u ? 1536u : RMODE == kDq ? 4864u
                                : RMODE == kNestedPow2 && WR == 3 && a.W >= 12u ? 4096u : 2600u;
    const bool short_vector = !persistent && (full < rows_below || rows_only);
    const uint32_t tile = short_vector ? ChainStreamTile<kOneRow>::N : kChainTile;
    // the rarer plans have the kernels with a ragged last tile only: a whole one takes its place
    const uint32_t tiles = (uint32_t)((RARER ? a.n - 1u : a.n) / tile);
    if (tiles == 0u || (ROWB && !persistent)) return 1;
    a.tiles = tiles;
    // (see bucket_of; a bucket is a multiple of the tile.  A tile's number times the magic stays below 2^63)
    const uint64_t per_bucket = bucket_len / tile;
    uint32_t log2 = 0u;
    while (((uint64_t)1 << log2) < per_bucket) ++log2;
    a.bucket_shift = 31u + log2;
    a.bucket_magic = ROWB || bucket_len == a.n ? 0u : (((uint64_t)1 << a.bucket_shift) + per_bucket - 1u) / per_bucket;
    const bool ragged = (uint64_t)tiles * tile < a.n;     // one more wave takes the ragged last tile
    const uint32_t all = tiles + (ragged ? 1u : 0u);
    // (a grid has fewer than 2^32 threads: close to 2^35 elements a wave takes two rows, in chain_kernel)
    if (rows_only && blocks_for(all) > 0xFFFFFFFFu / (uint32_t)kBlock) return 1;
    const dim3 grid(persistent ? persistent_blocks(all, 1024u * NDQ_CHAIN_PIPED_WAVES) : blocks_for(all)), block(kBlock);
    auto run = [&](auto lines, auto form) {
        constexpr bool LINES = decltype(lines)::value;
        constexpr int FORM = decltype(form)::value;
        if constexpr (RARER) return launch((chain_stream_kernel<RMODE, W0, WR, MIXED, ROWB, true, LINES, FORM>), grid, block, s, a);
        else return ragged ? launch((chain_stream_kernel<RMODE, W0, WR, MIXED, ROWB, true, LINES, FORM>), grid, block, s, a)
                           : launch((chain_stream_kernel<RMODE, W0, WR, MIXED, ROWB, false, LINES, FORM>), grid, block, s, a);
    };
    if (persistent) return run(std::false_type{}, std::integral_constant<int, kPiped>{});
    if constexpr (!ROWB) {
        // Rows of long vectors store whole lines, whatever they fold: halves / lines at 2.2, 4 and 16.8 M elements, 2 x 16 levels
        // 5.7/5.0 8.2/6.7 19.1/16.6, 8 x 16 levels 10.3/9.9 14.4/13.8 43.6/42.5, 4 levels and 3 x M = 2 7.9/7.4 11.5/10.5 31.4/30.5.
        if constexpr (!TWO_WIDTHS)
            if (rows_only && full >= (rows_below < kShortTiles ? rows_below : kShortTiles)) return run(std::true_type{}, std::integral_constant<int, kOneRow>{});
        if (short_vector) {
            // (a launch of rows is bound by its stores only with one worker: 2 M elements 4.4 -> 4.0 us; 2 of 1.6 M 4.1 -> 4.2)
            if constexpr (RMODE == kDq && W0 == WR)
                if (a.W == 1u) return run(std::true_type{}, std::integral_constant<int, kOneRow>{});
            return run(std::false_type{}, std::integral_constant<int, kOneRow>{});
        }
        return a.W < (RMODE == kDq ? 4u : 3u) ? run(std::true_type{}, std::integral_constant<int, kOneTile>{})
                                              : run(std::false_type{}, std::integral_constant<int, kOneTile>{});
    }
    return 1;
}

// The plans the streaming kernel has.
enum ChainPlan { kNoStream = 0,
                 kPurePlan = 1,     // all DQSG (the first may have another width), or one DQSG worker and nested ones; codes of 1, 2 and 4 bits
                 // The rarer plans: several DQSG workers and then nested ones, 3-bit codes, or a ratio that is no power of two;
                 // codes of 2 to 4 bits and of 1 to 3.  In kernels of their own, so that the others' stay as they are.  chain_kernel / this, us, at 1.05, 4 and
                 // 16.8 M elements: 1 x 8 levels 4.1/3.4 6.8/5.6 21.2/13.3, 8 x 8 levels 10.0/7.5 17.5/14.4 50.7/38.2, 8 levels and M = 4
                 // 4.9/4.5 7.5/6.8 19.5/16.9, 2 x 16 levels and 2 x M = 8 6.7/5.7 11.4/10.1 31.8/27.3, 8 x 16 levels and 8 x M = 4
                 // 17.5/12.9 34.4/26.6 113.9/84.2, 16 levels and 15 x M = 8 17.8/15.1 37.2/33.9 130/103, 4 x 5 levels and 4 x M = 3
                 // 11.5/9.1 22.2/18.6 65.9/52.3, 16 levels and 3 x M = 3 7.4/5.8 14.4/11.6 39.0/31.9.
                 // Buckets of one row, any of these plans, at 2.2, 4 and 16.8 M: 4 x 16 levels 8.4/6.6 10.6/9.0 29.7/22.9, 16 levels and
                 // 15 x M = 4 26.1/21.7 37.1/30.7 131/99.7, 16 levels and M = 4 6.0/5.4 7.4/7.1 21.1/17.5.
                 kMixedPlan = 2 };

// Whether it has the plan and the tiling; *dq are the DQSG workers and *wr the code width of the workers after them.
static ChainPlan chain_streams(const GeneralChainArgs& a, uint32_t bucket, uint32_t* dq, uint32_t* wr)
{
    if (a.continue_sum) return kNoStream;
    if (!(bucket == 0u || bucket % kChainTile == 0u || bucket == kWave * kLaneElems)) return kNoStream;
    const uint32_t w0 = a.w[0].bits;
    uint32_t first = 0u;
    while (first < a.W && a.w[first].mode == kDq && a.w[first].bits == w0) ++first;
    if (first == 0u || w0 > 4u) return kNoStream;
    *dq = first;
    *wr = first < a.W ? a.w[first].bits : w0;
    auto pure_width = [](uint32_t bits) { return bits == 1u || bits == 2u || bits == 4u; };
    // DQSG workers of two widths, the first one's and the others' (buckets of one row: chain_kernel).  chain_kernel / this, us, at
    // 1.05, 4.2 and 25.6 M elements: 4 and 16 levels 4.2/3.5 6.9/5.6 29.0/20.9, 4 and 3 x 16 levels 5.5/4.3 10.1/8.3 41.4/32.4,
    // 2 and 7 x 4 levels 8.0/6.0 17.9/13.9 68.8/54.8
    const bool two_widths = first == 1u && a.W > 1u && a.w[1].mode == kDq;
    const bool any_ratio = first < a.W && a.w[first].mode == kNestedAnyM;
    for (uint32_t j = first; j < a.W; ++j) {
        if (a.w[j].mode != (two_widths ? kDq : any_ratio ? kNestedAnyM : kNestedPow2) || a.w[j].bits != *wr) return kNoStream;
        if (!two_widths && (a.w[j].alpha != 1.0f || a.w[j].M != a.w[first].M)) return kNoStream;
    }
    if (two_widths && (a.row_buckets || !pure_width(w0) || !pure_width(*wr))) return kNoStream;
    // the high word of the dither's block number is the same for the whole call (it changes every 2^35 elements)
    for (uint32_t j = 0; j < a.W; ++j)
        if ((a.w[j].index0 >> 35) != ((a.w[j].index0 + a.tl.n - 1u) >> 35)) return kNoStream;
    if (two_widths) {
        *dq = a.W;
        return kPurePlan;
    }
    if (first == a.W) return w0 == 3u ? kMixedPlan : kPurePlan;
    if (any_ratio) return w0 >= 2u && *wr <= 3u ? kMixedPlan : kNoStream;
    if (first == 1u && pure_width(w0) && pure_width(*wr)) return kPurePlan;
    return w0 >= 2u && *wr <= 3u ? kMixedPlan : kNoStream;
}

// Runs the streaming kernel for a plan that chain_streams accepts; returns 1 when the vector holds no whole tile.
static int run_chain_stream(const GeneralChainArgs& a, uint32_t bucket, ChainPlan plan, uint32_t dq, uint32_t wr, hipStream_t s)
{
    const uint32_t w0 = a.w[0].bits;
    ChainArgs b;
    for (uint32_t j = 0; j < a.W; ++j) {
        const ChainWorker& cw = a.w[j];
        StreamWorker& sw = b.w[j];
        sw.codes = cw.codes;
        sw.block = (uint32_t)(cw.index0 >> 3);
        sw.extra = (uint32_t)cw.q_min;
        if (cw.mode != kDq) __builtin_memcpy(&sw.extra, &cw.side_scale, 4);
        sw.keys = philox_uniform(cw.ds, (uint32_t)(cw.index0 >> 35));
        b.steps[j] = cw.steps;
    }
    b.out = a.out;
    b.n = a.tl.n;
    b.W = a.W;
    b.dq = dq;
    b.ratio = a.w[a.W - 1u].M_f;
    b.inv_ratio = a.w[a.W - 1u].inv_M_f;
    b.apply_scale = a.apply_scale;
    b.scale = a.scale;
    // (a bucket that holds the whole vector is no different from none)
    const uint64_t bucket_len = bucket != 0u && bucket < b.n ? bucket : b.n;
    auto run = [&](auto rmode, auto first, auto rest, auto mixed) {
        constexpr int RMODE = decltype(rmode)::value, W0 = decltype(first)::value, WR = decltype(rest)::value;
        constexpr bool MIXED = decltype(mixed)::value;
        // buckets of one row, persistent: one DQSG worker is the mixed plan that has one
        if constexpr (W0 >= 2 && (RMODE == kDq ? W0 == WR : WR <= 3))
            if (bucket_len < kChainTile) {
                const int rc = launch_chain_stream<RMODE, W0, WR, RMODE != kDq, true>(b, bucket_len, s);
                if (rc != 1) return rc;
            }
        return launch_chain_stream<RMODE, W0, WR, MIXED>(b, bucket_len, s);
    };
    constexpr std::integral_constant<int, kDq> all_dq{};
    constexpr std::integral_constant<int, kNestedPow2> nested{};
    constexpr std::integral_constant<int, kNestedAnyM> any_ratio{};
    constexpr std::integral_constant<int, 1> b1{};
    constexpr std::integral_constant<int, 2> b2{};
    constexpr std::integral_constant<int, 3> b3{};
    constexpr std::integral_constant<int, 4> b4{};
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    if (dq == a.W && w0 != wr) {
        if (w0 == 1u) return wr == 2u ? run(all_dq, b1, b2, no) : run(all_dq, b1, b4, no);
        if (w0 == 2u) return wr == 1u ? run(all_dq, b2, b1, no) : run(all_dq, b2, b4, no);
        return wr == 1u ? run(all_dq, b4, b1, no) : run(all_dq, b4, b2, no);
    }
    if (dq == a.W)
        return w0 == 1u ? run(all_dq, b1, b1, no) : w0 == 2u ? run(all_dq, b2, b2, no) : w0 == 3u ? run(all_dq, b3, b3, no)
                                                                                                : run(all_dq, b4, b4, no);
    if (plan == kPurePlan) {
        auto rest = [&](auto first) {
            return wr == 1u ? run(nested, first, b1, no) : wr == 2u ? run(nested, first, b2, no) : run(nested, first, b4, no);
        };
        return w0 == 1u ? rest(b1) : w0 == 2u ? rest(b2) : rest(b4);
    }
    if (a.w[a.W - 1u].mode == kNestedAnyM) {
        auto rest = [&](auto first) { return wr == 2u ? run(any_ratio, first, b2, yes) : run(any_ratio, first, b3, yes); };
        return w0 == 2u ? rest(b2) : w0 == 3u ? rest(b3) : rest(b4);
    }
    auto rest = [&](auto first) {
        return wr == 1u ? run(nested, first, b1, yes) : wr == 2u ? run(nested, first, b2, yes) : run(nested, first, b3, yes);
    };
    return w0 == 2u ? rest(b2) : w0 == 3u ? rest(b3) : rest(b4);
}

// Longest vector chain_short_kernel takes.  A workgroup keeps all workers of a row in LDS, so a compute unit holds six of
// them for up to 16 workers and three for more: the lines lie about where these rounds end.  Time over the other kernel's,
// launches replayed from a graph / one call after the other, at 131 k, 262 k, 393 k, 459 k elements
//   against chain_stream_kernel   2 workers     1.05/1.03  1.15/1.04  1.14/1.02  1.23/1.05   (3.0 against 2.7 us)
//                                 3             0.97/1.03  1.05/1.03  1.15/1.06  1.20/1.06
//                                 4             0.93/0.98  0.98/0.98  1.09/1.02  1.19/1.08
//                                 8             0.83/0.82  0.90/0.87  1.00/0.94  1.15/1.04
//                                 16            0.75/0.71  0.80/0.75  0.95/0.85  1.10/0.98
//                                 20 to 32      0.71/0.64  0.77/0.70  0.88/0.83  1.27/1.19
// and at 262 k, 393 k, 524 k, 655 k, 786 k, 918 k, 983 k
//   against chain_kernel          2             0.92/0.99  0.94/0.98  1.02/1.00  1.06/1.01  1.14/1.06  1.17/1.08  1.19/1.10
//                                 3             0.80/0.89  0.89/0.89  0.97/0.94  1.04/0.97  1.07/1.02  1.13/1.06  1.18/1.07
//                                 4             0.73/0.79  0.82/0.83  0.89/0.89  0.94/0.92  0.99/0.96  1.06/1.01  1.12/1.04
//                                 6, 8          0.64/0.66  0.72/0.71  0.81/0.77  0.86/0.84  0.94/0.89  1.02/0.96  1.09/1.03
//                                 12, 16        0.56/0.51  0.66/0.57  0.76/0.67  0.80/0.76  0.89/0.86  0.98/0.95  1.06/1.03
//                                 20 to 32      0.53/0.46  0.60/0.54  0.81/0.77  0.86/0.85  0.96/0.95  1.12/1.12  1.19/1.19
// at 131 k, 262 k, 393 k, 458 k, 524 k, 655 k, 786 k (as far as the lines are near)
//   against chain_stream_kernel, the rarer plans
//     3-bit DQSG      2   0.98/1.02 1.08/1.05 1.16/1.09
//                     3   0.87/0.94 0.96/0.98 1.06/1.06
//                     4   0.78/0.94 0.86/0.96 0.95/0.99 1.05/1.05
//                     6   0.76/0.86 0.83/0.93 0.90/0.96 0.99/1.03
//                     8   0.66/0.76 0.72/0.80 0.82/0.88 0.92/0.96 0.95/0.98 1.00/0.99 1.10/1.09
//                     16  0.57/0.64 0.63/0.68 0.75/0.78 0.87/0.88 0.87/0.88 0.95/0.96 1.07/1.08
//                     20  0.56/0.59 0.61/0.63 0.74/0.75 1.04/1.04
//     half nested,    2   0.96/1.01 1.06/1.00 1.12/1.09
//     1 or 2 bits     3   0.94/1.02 1.00/1.00 1.08/1.06
//                     4   0.87/0.98 0.93/0.98 1.03/1.02 1.12/1.06
//                     8   0.77/0.84 0.85/0.90 0.96/0.97 1.08/1.07
//                     16  0.68/0.74 0.74/0.79 0.88/0.89 1.01/1.02
//                     20  0.67/0.70 0.73/0.76 0.87/0.88 1.25/1.25
//     half M = 3      2   0.95/1.01 1.04/1.03 1.11/1.10
//                     4   0.81/0.92 0.87/0.95 0.96/0.97 1.06/1.08
//                     8   0.69/0.78 0.77/0.84 0.87/0.92 1.00/1.00 1.00/1.04
//                     16  0.61/0.67 0.68/0.71 0.80/0.82 0.93/0.95 0.94/0.95 0.97/0.97 1.11/1.10
//                     20  0.60/0.63 0.66/0.67 0.79/0.80 1.13/1.13
//     15 of M = 8     16  0.56/0.59 0.61/0.63 0.71/0.72 0.82/0.83 0.83/0.83 0.86/0.85 0.97/0.97
// One worker alone has nothing to wait for twice.  (A streaming threshold from the environment means that
// kernel, whatever the length.)
// `dq` DQSG workers, then nested ones with codes of `wr` bits.
static uint32_t short_chain_most(uint32_t W, ChainPlan plan, uint32_t dq, uint32_t wr, bool any_ratio)
{
    if (plan == kNoStream) return W < 2u ? 0u : 131072u * (W > 16u ? 6u : W < 6u ? W + 1u : 7u);
    if (stream_tuning().threshold_from_env) return 0u;
    if (plan == kPurePlan) return W < 4u ? 0u : 196608u + 12288u * (W < 16u ? W : 16u);
    if (W < 4u) return 131072u * (W - 1u);
    // (longer folds gain the more by being prepared side by side)
    if (W > 16u) return 3u * 131072u;
    if (dq == W) return 131072u * (W >= 8u ? 5u : 3u);
    return 131072u * (W < 12u ? 3u : any_ratio ? 5u : wr == 3u ? 6u : 3u);
}

}  // namespace ndq

extern "C" {

int ndq_dq_decode(const void* codes, size_t n, uint32_t levels, uint32_t bucket,
                  const float* steps, const ndq_dither* d, float* out, int accumulate,
                  void* stream)
{
    return ndq::decode_common(codes, n, levels, 0u, false, false, 1.0f, bucket, steps, d, nullptr,
                              1.0f, out, accumulate, stream);
}

int ndq_dq_decode_half(const void* codes, size_t n, uint32_t levels, uint32_t bucket,
                       const float* steps, float* out, int accumulate, void* stream)
{
    const ndq_dither none = {0u, 0u, 0u, 0u};   // no dither is regenerated
    return ndq::decode_common(codes, n, levels, 0u, false, true, 1.0f, bucket, steps, &none,
                              nullptr, 1.0f, out, accumulate, stream);
}

int ndq_nested_decode(const void* codes, size_t n, uint32_t M, float alpha, uint32_t bucket,
                      const float* steps, const ndq_dither* d, const float* side,
                      float side_scale, float* out, int accumulate, void* stream)
{
    // `levels` plays no part in decoding: the step travels in `steps`
    return ndq::decode_common(codes, n, 2u, M, true, false, alpha, bucket, steps, d, side,
                              side_scale, out, accumulate, stream);
}

int ndq_aggregate(const float* const* gs, uint32_t W, size_t n, float scale, float* out,
                  void* stream)
{
    using namespace ndq;
    if (!gs || W < 1u || W > 1024u) return NDQ_EINVAL;
    if (n == 0) return NDQ_OK;
    if (!out) return NDQ_EINVAL;
    if (n >= kMaxN) return NDQ_EUNSUPPORTED;
    if (!aligned16(out)) return NDQ_EALIGN;
    for (uint32_t w = 0; w < W; ++w) {
        if (!gs[w]) return NDQ_EINVAL;
        if (!aligned16(gs[w])) return NDQ_EALIGN;
        if (W > kAggMax && gs[w] == out) return NDQ_EINVAL;
    }
    const uint64_t threads = (n + 3) / 4;
    const uint64_t blocks = (threads + kBlock - 1) / kBlock;
    if (blocks >= ((uint64_t)1 << 31)) return NDQ_EUNSUPPORTED;
    for (uint32_t w0 = 0; w0 < W; w0 += kAggMax) {
        AggArgs a;
        a.W = (W - w0 < kAggMax) ? W - w0 : kAggMax;
        for (uint32_t j = 0; j < kAggMax; ++j) a.g[j] = j < a.W ? gs[w0 + j] : nullptr;
        a.out = out;
        a.n = n;
        a.continue_sum = w0 != 0u;
        a.finish = w0 + kAggMax >= W;
        a.scale = scale;
        if (launch(aggregate_kernel, dim3((uint32_t)blocks), dim3(kBlock), (hipStream_t)stream, a) != NDQ_OK)
            return NDQ_ELAUNCH;
    }
    return NDQ_OK;
}

int ndq_decode_mean(const ndq_worker* workers, float* const* decoded, uint32_t W, size_t n, uint32_t bucket,
                    float scale, float* out, void* stream)
{
    using namespace ndq;
    if (!workers || !decoded || W < 1u || W > 1024u) return NDQ_EINVAL;
    for (uint32_t p = 0; p < W; ++p)
        if (workers[p].kind != NDQ_WORKER_DQ || workers[p].levels_or_M < 2u || workers[p].levels_or_M > 256u)
            return NDQ_EINVAL;
    if (n == 0) return NDQ_OK;
    if (!out) return NDQ_EINVAL;
    if (n >= kMaxN) return NDQ_EUNSUPPORTED;
    if (!aligned16(out) || bucket % 64u != 0u) return NDQ_EALIGN;
    for (uint32_t p = 0; p < W; ++p) {
        const ndq_worker& wk = workers[p];
        if (!wk.codes || !wk.steps || !decoded[p]) return NDQ_EINVAL;
        if (!aligned16(wk.codes) || !aligned16(decoded[p]) || !aligned4(wk.steps) || (wk.dither.offset & 7u) != 0u)
            return NDQ_EALIGN;
        // a partial sum waits in `out` between launches (one launch: a lane writes `out` last)
        if (W > kMeanMax && decoded[p] == out) return NDQ_EINVAL;
    }
    // vectors that overlap by a part would race between waves (the same vector twice: a lane writes it in order)
    uintptr_t begin[1025];
    for (uint32_t p = 0; p < W; ++p) begin[p] = (uintptr_t)decoded[p];
    begin[W] = (uintptr_t)out;
    std::sort(begin, begin + W + 1u);
    for (uint32_t p = 0; p < W; ++p)
        if (begin[p] != begin[p + 1u] && begin[p + 1u] - begin[p] < 4u * n) return NDQ_EINVAL;
    MeanArgs a;
    // (tiles of the whole vector: their 64-element blocks are numbered in 32 bits.  One worker alone is bound
    // by its stores, and with three quarters of its lanes busy does no worse: 384 elements, 30 M 37.6 us
    // against 43.5; two workers or more gain, four 116 -> 108)
    const bool small = bucket != 0u && bucket < kMeanTile && (W > 1u || bucket < 384u) && n < ((uint64_t)1 << 37);
    int rc = make_tiling(n, bucket, kMeanTile, &a.tl);
    if (rc == NDQ_OK && small) rc = make_tiling(n, 0u, kMeanTile, &a.tl);
    if (rc != NDQ_OK) return rc;
    a.bucket_blocks = small ? bucket / 64u : 1u;
    a.last_bucket = small ? (uint32_t)((n + bucket - 1u) / bucket) - 1u : 0u;
    a.out = out;
    a.scale = scale;
    for (uint32_t p0 = 0; p0 < W; p0 += kMeanMax) {
        a.W = (W - p0 < kMeanMax) ? W - p0 : kMeanMax;
        a.continue_sum = p0 != 0u;
        a.finish = p0 + kMeanMax >= W;
        for (uint32_t j = 0; j < a.W; ++j) {
            const ndq_worker& wk = workers[p0 + j];
            a.w[j] = {(const unsigned char*)wk.codes, wk.steps, decoded[p0 + j], wk.dither.offset,
                      make_stream(&wk.dither), -(int32_t)(wk.levels_or_M / 2u), code_bits(wk.levels_or_M)};
        }
        const dim3 grid(blocks_for(a.tl.total_tiles)), block(kBlock);
        auto* kernel = a.W <= kMeanFew ? (small ? decode_mean_kernel<true, true> : decode_mean_kernel<false, true>)
                                       : (small ? decode_mean_kernel<true, false> : decode_mean_kernel<false, false>);
        if (launch(kernel, grid, block, (hipStream_t)stream, a) != NDQ_OK) return NDQ_ELAUNCH;
    }
    return NDQ_OK;
}

int ndq_decode_chain(const ndq_worker* workers, uint32_t W, size_t n, uint32_t bucket,
                     float scale, float* out, void* stream)
{
    using namespace ndq;
    if (!workers || W < 1u || W > 1024u) return NDQ_EINVAL;
    if (workers[0].kind != NDQ_WORKER_DQ) return NDQ_EINVAL;   // nothing to decode against yet
    for (uint32_t p = 0; p < W; ++p) {
        const ndq_worker& wk = workers[p];
        if (wk.kind != NDQ_WORKER_DQ && wk.kind != NDQ_WORKER_NESTED) return NDQ_EINVAL;
        if (wk.levels_or_M < 2u || wk.levels_or_M > 256u) return NDQ_EINVAL;
        if (wk.kind == NDQ_WORKER_NESTED && !(wk.alpha > 0.0f && wk.alpha <= 1.0f)) return NDQ_EINVAL;
    }
    if (n == 0) return NDQ_OK;
    if (!out) return NDQ_EINVAL;
    if (n >= kMaxN) return NDQ_EUNSUPPORTED;
    if (!aligned16(out) || bucket % 64u != 0u) return NDQ_EALIGN;
    for (uint32_t p = 0; p < W; ++p) {
        const ndq_worker& wk = workers[p];
        if (!wk.codes || !wk.steps) return NDQ_EINVAL;
        if (!aligned16(wk.codes) || !aligned4(wk.steps) || (wk.dither.offset & 7u) != 0u)
            return NDQ_EALIGN;
    }
    GeneralChainArgs a;
    // buckets of exactly one row share a tile, each row with its own step
    a.row_buckets = (kChainRows > 1 && bucket == kWave * kLaneElems) ? 1u : 0u;
    a.num_buckets = a.row_buckets ? (uint32_t)ndq_num_buckets(n, bucket) : 0u;   // n < 2^40: fits
    int rc = make_tiling(n, a.row_buckets ? kChainTile : bucket, kChainTile, &a.tl);
    if (rc != NDQ_OK) return rc;
    const bool short_vector = a.tl.total_tiles < kShortGeneralTiles;
    Tiling short_tl = a.tl;
    if (short_vector && (rc = make_tiling(n, bucket, kWave * kLaneElems, &short_tl)) != NDQ_OK) return rc;
    a.out = out;
    a.scale = scale;
    for (uint32_t p0 = 0; p0 < W; p0 += kChainMax) {
        a.W = (W - p0 < kChainMax) ? W - p0 : kChainMax;
        a.continue_sum = p0 != 0u;
        a.apply_scale = (p0 + kChainMax >= W) && scale != 1.0f;
        for (uint32_t j = 0; j < a.W; ++j) {
            const ndq_worker& wk = workers[p0 + j];
            const bool nested = wk.kind == NDQ_WORKER_NESTED;
            Quant qp;
            make_quant(nested ? 2u : wk.levels_or_M, wk.levels_or_M, nested, wk.alpha, &qp);
            ChainWorker& cw = a.w[j];
            cw.codes = (const unsigned char*)wk.codes;
            cw.steps = wk.steps;
            cw.index0 = wk.dither.offset;
            cw.ds = make_stream(&wk.dither);
            cw.q_min = qp.q_min;
            cw.M = qp.M;
            cw.M_f = qp.M_f;
            cw.inv_M_f = qp.inv_M_f;
            cw.alpha = qp.alpha;
            cw.beta = qp.beta;
            cw.side_scale = (p0 + j) ? 1.0f / (float)(p0 + j) : 0.0f;
            cw.bits = qp.bits;
            cw.mode = !nested ? kDq
                              : (!is_pow2(wk.levels_or_M) ? kNestedAnyM
                                 : (wk.alpha == 1.0f ? kNestedPow2 : kNestedPow2Shrink));
            cw.first = (p0 + j) == 0u;
        }
        hipStream_t hs = (hipStream_t)stream;
        uint32_t dq = 0u, wr = 0u;
        const ChainPlan plan = W <= kChainMax ? chain_streams(a, bucket, &dq, &wr) : kNoStream;
        if (W <= kChainMax && n <= short_chain_most(W, plan, dq, wr, plan != kNoStream && a.w[W - 1u].mode == kNestedAnyM)) {
            a.tl.bucket_len = bucket != 0u ? bucket : n;
            const dim3 grid((uint32_t)((n + kShortTile - 1u) / kShortTile)), block(kBlock);
            return W <= 8u ? launch(chain_short_kernel<8>, grid, block, hs, a)
                           : W <= 16u ? launch(chain_short_kernel<16>, grid, block, hs, a)
                                      : launch(chain_short_kernel<32>, grid, block, hs, a);
        }
#ifndef NDQ_NO_STREAM_CHAIN
        if (plan != kNoStream) {
            const int rc_stream = run_chain_stream(a, bucket, plan, dq, wr, hs);
            if (rc_stream != 1) return rc_stream;
        }
#endif
        if (short_vector) {
            a.tl = short_tl;
            a.row_buckets = 0u;
        }
        const dim3 grid(blocks_for(a.tl.total_tiles)), block(kBlock);
        // (see chain_kernel; the first worker of a later launch can be any)
        auto plain = [&](uint32_t j) { return a.w[j].mode == kDq || a.w[j].mode == kNestedPow2; };
        const bool two_workers = a.W == 2u && plain(0u) && plain(1u);
        const int rc_launch = short_vector ? launch((chain_kernel<false, true, 1>), grid, block, hs, a)
                              : a.row_buckets && two_workers ? launch((chain_kernel<true, false, kChainRows>), grid, block, hs, a)
                              : a.row_buckets ? launch((chain_kernel<true, true, kChainRows>), grid, block, hs, a)
                              : two_workers ? launch((chain_kernel<false, false, kChainRows>), grid, block, hs, a)
                                            : launch((chain_kernel<false, true, kChainRows>), grid, block, hs, a);
        if (rc_launch != NDQ_OK) return NDQ_ELAUNCH;
    }
    return NDQ_OK;
}

}  // extern "C"
