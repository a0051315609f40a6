// libndq, worker side (gfx950): max-norm scale factors, DQSG / NDQSG encoders.
// See include/ndq.h for the contract.
//
// Every kernel of the library is a streaming pass: a wave owns a tile of
// consecutive elements at a time (one tile per wave in the short-vector kernels,
// tile after tile in the persistent ones), loads it with 16-byte loads,
// regenerates the dither with Philox in registers and writes coalesced vectors.
// Nothing is a contraction, so no MFMA; LDS only transposes the small packed
// codes into stream order and, for buckets of two or four tiles, carries the
// tile maxima between the waves of a workgroup.
#include <hip/hip_runtime.h>

#include <string.h>

#include <type_traits>
#include <utility>

#include "ndq.h"
#include "ndq_device.hpp"
#include "ndq_host.hpp"

namespace ndq {

// ---------------------------------------------------------------------------
// Encoder: Algorithm 1 worker block (DQSG) / Algorithm 2 worker block (NDQSG)
// ---------------------------------------------------------------------------
// One vector to encode.
struct EncodeJob {
    const void* g;
    unsigned char* codes;
    float* steps;          // written (fused, preset, handed over) or already there (two-pass)
    const float* step_in;  // where a step that is not found here is read: `steps`, or the one handed over
    uint64_t index0;       // dither offset of element 0
    DitherStream ds;
};

// What a wave works with: its vector, and what all vectors of the launch share.
struct EncodeArgs : EncodeJob {
    Tiling tl;
    uint64_t total_bytes;  // size of the packed stream incl. zero padding
    Quant qp;
    float preset_step;     // > 0: bucket == 0 with a caller-set step
    uint32_t rows_log2;    // MULTI: a bucket is 2^rows_log2 rows of a tile
    uint32_t num_buckets;  // MULTI: buckets in the call (steps to write)
    uint32_t waves_log2;   // FUSED, not MULTI: a bucket is 2^waves_log2 tiles of one workgroup
    uint32_t through;      // binary32, buckets: how codes of 1 and 2 bits are stored
};

// A launch encodes up to kEncJobs vectors of one length, type and quantizer (blockIdx.y, or
// the tiles of all of them in turn in the streaming kernel): the vectors of a group of
// workers, or the one of a single call.
constexpr uint32_t kEncJobs = 16;
struct EncodeBatch {
    EncodeArgs common;     // its EncodeJob part is unused
    EncodeJob job[kEncJobs];
    uint32_t jobs;
};
// read through the constant address space: scalar loads, no copy of the arguments
typedef const __attribute__((address_space(4))) EncodeBatch* EncodeBatchPtr;

__device__ __forceinline__ void select_job(EncodeArgs& a, EncodeBatchPtr b, uint32_t j)
{
    a.g = b->job[j].g;
    a.codes = b->job[j].codes;
    a.steps = b->job[j].steps;
    a.step_in = b->job[j].step_in;
    a.index0 = b->job[j].index0;
    a.ds.key0 = b->job[j].ds.key0;
    a.ds.key1 = b->job[j].ds.key1;
    a.ds.step = b->job[j].ds.step;
    a.ds.worker = b->job[j].ds.worker;
}

__device__ __forceinline__ EncodeArgs common_args(EncodeBatchPtr b)
{
    EncodeArgs a;
    a.tl.n = b->common.tl.n;
    a.tl.bucket_len = b->common.tl.bucket_len;
    a.tl.tiles_per_bucket = b->common.tl.tiles_per_bucket;
    a.tl.total_tiles = b->common.tl.total_tiles;
    a.total_bytes = b->common.total_bytes;
    a.qp.q_min_f = b->common.qp.q_min_f;
    a.qp.q_max_f = b->common.qp.q_max_f;
    a.qp.q_min = b->common.qp.q_min;
    a.qp.levels = b->common.qp.levels;
    a.qp.M = b->common.qp.M;
    a.qp.M_f = b->common.qp.M_f;
    a.qp.inv_M_f = b->common.qp.inv_M_f;
    a.qp.bits = b->common.qp.bits;
    a.qp.pack_bias = b->common.qp.pack_bias;
    a.qp.alpha = b->common.qp.alpha;
    a.qp.beta = b->common.qp.beta;
    a.preset_step = b->common.preset_step;
    a.rows_log2 = b->common.rows_log2;
    a.num_buckets = b->common.num_buckets;
    a.waves_log2 = b->common.waves_log2;
    a.through = b->common.through;
    return a;
}

template <int DT> struct EncRows { static constexpr int R = kEncLoads / Elem<DT>::V; };
template <int DT> struct EncTile { static constexpr uint32_t N = kWave * kLaneElems * EncRows<DT>::R; };

// A tile in registers: a lane owns 8 consecutive elements per row (one Philox
// block, and 8 codes = `bits` whole bytes of the stream).
template <int DT> struct TileRegs { typename Elem<DT>::Row row[EncRows<DT>::R]; };

// Issues all 16-byte loads of a tile back to back.  FULL: every element of the
// tile is valid, no guards; otherwise elements past the end read as zero.
template <int DT, bool FULL, bool KEEP = false>
__device__ __forceinline__ void load_tile(const void* g, const TileRef& t, int lane, TileRegs<DT>& regs)
{
    using T = Elem<DT>;
    const typename T::scalar* tile = (const typename T::scalar*)g + t.start;
#pragma unroll
    for (int r = 0; r < EncRows<DT>::R; ++r)
        regs.row[r] = load_row<DT, FULL, KEEP>(tile, (uint32_t)(r * kWave + lane) * kLaneElems, t.len);
}

// folds the lane's share of a tile into its running max |g|
template <int DT>
__device__ __forceinline__ typename Elem<DT>::maxacc lane_max(typename Elem<DT>::maxacc m,
                                                               const TileRegs<DT>& regs)
{
#pragma unroll
    for (int r = 0; r < EncRows<DT>::R; ++r) m = Elem<DT>::max_update(m, regs.row[r]);
    return m;
}

// max |g| over the tile a wave holds (Sec. 3.1 eq. (2)), the same in every lane
template <int DT>
__device__ __forceinline__ float tile_max(const TileRegs<DT>& regs)
{
    using T = Elem<DT>;
    return wave_max(T::max_final(lane_max<DT>(T::max_init(), regs)));
}

// One wave encodes the tile it holds: finds the step, quantizes, and leaves the
// packed codes in `stage` in stream order.  FULL: no guards anywhere.  FUSED: the
// step comes from `kappa`, the max-norm of the tile's bucket, found in registers.
// MULTI (with FUSED): the bucket is a whole number of rows and several buckets
// share the tile, each with its own step.
// REFILL: a row's registers are loaded again while the row is processed, with the same row of
// the whole tile at `refill` (lane `refill_lane`'s share), so that one set of registers holds
// the current tile and, by the end, the next one.
// GIVEN: `kappa` is the step itself, and the caller writes it.
template <int DT, int MODE, bool FUSED, bool FULL, bool MULTI, int BITSW = 0, bool REFILL = false, bool GIVEN = false>
__device__ __forceinline__ void encode_tile(const EncodeArgs& a, const TileRef& t, uint32_t tile_id,
                                            typename std::conditional<REFILL, TileRegs<DT>, const TileRegs<DT>>::type& regs,
                                            float kappa, bool writes_step, unsigned char* stage, int lane,
                                            const void* refill = nullptr, int refill_lane = 0)
{
    using T = Elem<DT>;
    constexpr int ROWS = EncRows<DT>::R;
    const uint32_t bits = BITSW ? (uint32_t)BITSW : a.qp.bits;   // BITSW: the code width, known at compile time
    auto& raw = regs.row;

    // 1/step per row (alpha/step for a nested worker that shrinks), wave-uniform
    float inv_row[ROWS];
    if (FUSED && MULTI) {
        // A bucket is 1, 2 or 4 rows (Sec. 3.1 eq. (2) per bucket): a lane's share of its rows is merged
        // first, then there is one wave-wide maximum per bucket, and lane r does the two divisions of
        // the bucket that starts at row r, all of them at once.
        const uint32_t rl = a.rows_log2, group_mask = (1u << rl) - 1u;
        typename T::maxacc m[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) m[r] = T::max_update(T::max_init(), raw[r]);
        if (rl != 0u) {
#pragma unroll
            for (int r = 0; r < ROWS; r += 2) m[r] = T::max_merge(m[r], m[r + 1]);
        }
        if (rl == 2u) {
#pragma unroll
            for (int r = 0; r + 2 < ROWS; r += 4) m[r] = T::max_merge(m[r], m[r + 2]);
        }
        float kappas = 0.0f;
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            if (((uint32_t)r & group_mask) == 0u) {   // first row of a bucket
                const float kappa_r = wave_max(T::max_final(m[r]));
                kappas = lane == r ? kappa_r : kappas;
            }
        const float steps = step_from_kappa(kappas, a.qp.levels), invs = a.qp.alpha * inv_step(steps);
        const uint32_t bucket = t.bucket * ((uint32_t)ROWS >> rl) + ((uint32_t)lane >> rl);
        if (lane < ROWS && ((uint32_t)lane & group_mask) == 0u && bucket < a.num_buckets) a.steps[bucket] = steps;
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            inv_row[r] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(invs), r & ~(int)group_mask));
    } else {
        float step;
        if (GIVEN) {
            step = kappa;
        } else if (FUSED) {
            step = step_from_kappa(kappa, a.qp.levels);
            if (REFILL) a.steps[t.bucket] = step;     // every lane, the same value: no branch around the store
            else if (lane == 0 && writes_step) a.steps[t.bucket] = step;
        } else {
            step = a.preset_step > 0.0f ? a.preset_step : a.step_in[t.bucket];
            // one step for the whole vector, preset or handed over: the worker's transmitted step
            if (tile_id == 0 && lane == 0) a.steps[0] = step;
        }
        const float inv_all = a.qp.alpha * inv_step(step);   // alpha = 1 unless a nested worker shrinks
#pragma unroll
        for (int r = 0; r < ROWS; ++r) inv_row[r] = inv_all;
    }
    const uint64_t block0 = (a.index0 + t.start) >> 3;

#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const uint32_t o = (uint32_t)(r * kWave + lane) * kLaneElems;
        const float inv = inv_row[r];
        float v[8];
        dither8(a.ds, block0 + (o >> 3), v);
        // REFILL: the row is widened to binary32 first and its registers are loaded again right
        // here, at one fixed place per row between the dither and the quantizer (measured: 5 %
        // faster than leaving the load's place to the compiler, which batches two rows' loads
        // and issues them later; earlier, before the dither, is slower too).
        float gw[8];
        if constexpr (REFILL) {
#pragma unroll
            for (int k = 0; k < 8; ++k) gw[k] = T::get(raw[r], k);
            asm volatile("" : "+v"(gw[0]), "+v"(gw[1]), "+v"(gw[2]), "+v"(gw[3]), "+v"(gw[4]), "+v"(gw[5]), "+v"(gw[6]), "+v"(gw[7]));
            raw[r] = load_row<DT, true>(refill, (uint32_t)(r * kWave + refill_lane) * kLaneElems, EncTile<DT>::N);
            __builtin_amdgcn_sched_barrier(0);
        }
        auto elem = [&](int i) __attribute__((always_inline)) { return REFILL ? gw[i] : T::get(raw[r], i); };
        uint32_t quad[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t chunk = 0;
            if (MODE == kDqNarrow) {
                // codes of <= 6 bits: sum (q_k - q_min) 2^(k b) stays an exact float below 2^24
                float acc = a.qp.pack_bias;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float q = dq_index_f(elem(4 * h + k), inv, v[4 * h + k], a.qp);
                    if (!FULL && o + 4 * h + k >= t.len) q = a.qp.q_min_f;
                    acc = __builtin_fmaf(q, __uint_as_float((127u + k * bits) << 23), acc);
                }
                chunk = (uint32_t)acc;
            } else if (MODE == kNestedAnyMBounded) {
                // residues of <= 6 bits packed like the narrow DQSG codes: exact float fma's
                float acc = 0.0f;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float m = nested_residue_f(elem(4 * h + k), inv, v[4 * h + k], a.qp);
                    if (!FULL && o + 4 * h + k >= t.len) m = 0.0f;
                    acc = __builtin_fmaf(m, __uint_as_float((127u + k * bits) << 23), acc);
                }
                chunk = (uint32_t)acc;
            } else if (MODE == kNestedPow2Bounded) {
                // each code enters at the top of the word and moves down as the next
                // ones arrive: one funnel shift per code keeps exactly its low `bits` bits
                uint32_t acc = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    uint32_t low = nested_low_bits(elem(4 * h + k), inv, v[4 * h + k]);
                    if (!FULL && o + 4 * h + k >= t.len) low = 0;
                    acc = __builtin_amdgcn_alignbit(low, acc, bits);
                }
                chunk = acc >> (32u - 4u * bits);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    uint32_t c = encode_one<MODE>(elem(4 * h + k), inv, v[4 * h + k], a.qp);
                    if (!FULL && o + 4 * h + k >= t.len) c = 0;
                    chunk |= c << (k * bits);
                }
            }
            quad[h] = chunk;
        }
        // eight consecutive codes -> `bits` bytes at byte (o/8)*bits of the tile's stream
        const uint64_t chunk8 = (uint64_t)quad[0] | ((uint64_t)quad[1] << (4 * bits));
        unsigned char* p = stage + (o >> 3) * bits;
        switch (bits) {
            case 1: *p = (unsigned char)chunk8; break;
            case 2: *(uint16_t*)p = (uint16_t)chunk8; break;
            case 3:
                if (BITSW == 3) {
                    // four lanes' twelve bytes leave as three words: lane j of the four takes what is
                    // left of its own 24 bits and the first of its neighbour's
                    const int here = (int)(uint32_t)chunk8;
                    const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(0, here, 0xF9, 0xF, 0xF, false);   // quad_perm [1,2,3,3]
                    const uint32_t j = (uint32_t)lane & 3u;
                    const uint32_t word = (uint32_t)here >> (8u * j) | next << (24u - 8u * j);
                    if (j != 3u) *(uint32_t*)(p + j) = word;          // at byte 12 (lane / 4) + 4 j of the row
                } else {
                    p[0] = (unsigned char)chunk8; p[1] = (unsigned char)(chunk8 >> 8); p[2] = (unsigned char)(chunk8 >> 16);
                }
                break;
            case 4: *(uint32_t*)p = (uint32_t)chunk8; break;
            case 8: *(uint64_t*)p = chunk8; break;
            default:
                for (uint32_t k = 0; k < bits; ++k) p[k] = (unsigned char)(chunk8 >> (8 * k));
        }
    }
    if (lane == 0) *(uint64_t*)(stage + (size_t)EncTile<DT>::N / 8 * bits) = 0;  // pad unit
}

// Copies a tile's packed codes from the wave's stage to the stream, 8 bytes per lane.  BUCKETS: a step per bucket
// (which stores: see store_through).
template <int DT, bool BUCKETS>
__device__ __forceinline__ void stage_to_stream(const EncodeArgs& a, const TileRef& t, uint32_t bits,
                                                const unsigned char* stage, int lane)
{
    const uint64_t byte0 = (t.start >> 3) * bits;                 // tile start is a multiple of 64
    const bool last = t.start + t.len == a.tl.n;
    const uint64_t nbytes = last ? a.total_bytes - byte0 : (uint64_t)(t.len >> 3) * bits;
    const uint32_t units = (uint32_t)(nbytes >> 3);
    uint64_t* dst = (uint64_t*)(a.codes + byte0);
    const uint64_t* src = (const uint64_t*)stage;
    if (DT == 1 || !BUCKETS || bits > 2u || a.through != 0u) {
        for (uint32_t u = lane; u < units; u += kWave) store_through(dst + u, src[u]);
    } else {
        for (uint32_t u = lane; u < units; u += kWave) dst[u] = src[u];
    }
}

// Occupancy target.  The bfloat16 encoder is bound by instruction issue with a
// burst of loads at the start of every tile; eight waves per SIMD (64 registers)
// hide that burst better than four (+8 % measured).  The binary32 encoder moves
// twice the bytes per element and measured best with the registers it asks for.
#ifndef NDQ_ENC_WAVES_BF16
#define NDQ_ENC_WAVES_BF16 8
#endif
template <int DT> struct EncWaves { static constexpr int W = DT == 1 ? NDQ_ENC_WAVES_BF16 : 4; };
// FUSED: the bucket fits one tile.  MULTI: several buckets to a tile.  BLOCK: the
// bucket is 2 or 4 tiles, all held by the waves of one workgroup.  In all three
// the max-norm is found in registers and the step written; otherwise the step is
// the preset one or read from `steps` (written by the max-norm pass, or handed over).
// BITSW: the code width when it is one of 1 to 4 (the packing and the store of a
// row's codes are then straight-line code: 56 registers instead of 100 in binary32, half the instructions);
// 0: any width, read from the arguments.
// (MULTI reduces a bucket's rows in a lane before it reduces them across the wave, and divides for all buckets
// of a tile at once: with the known width, 4 x 11.2 M bfloat16 in buckets of 1,024, the iteration 47.4 -> 41.8 us.)
template <int DT, int MODE, bool FUSED, bool MULTI, bool BLOCK, int BITSW>
__device__ __forceinline__ void encode_wave(const EncodeArgs& a, const TileRef& t, uint32_t tile_id, int wave, int lane,
                                            unsigned char* stage, float (&part)[kWavesPerBlock])
{
    constexpr uint32_t TILE = EncTile<DT>::N;
    const uint32_t bits = BITSW ? (uint32_t)BITSW : a.qp.bits;
    if (BLOCK) {
        // A bucket of 2 or 4 tiles lies inside one workgroup (tile ids are consecutive
        // and buckets start at multiples of their length): the waves exchange their
        // tile maxima through LDS.  Every wave of the workgroup reaches the barrier,
        // also one whose tile is empty.
        TileRegs<DT> regs;
        if (t.len == TILE) load_tile<DT, true>(a.g, t, lane, regs);
        else if (t.len != 0) load_tile<DT, false>(a.g, t, lane, regs);
        float kappa = 0.0f;
        if (t.len != 0) kappa = tile_max<DT>(regs);
        if (lane == 0) part[wave] = kappa;
        __syncthreads();
        const uint32_t group = 1u << a.waves_log2, first = (uint32_t)wave & ~(group - 1u);
        kappa = part[first];
        for (uint32_t w = 1; w < group; ++w) kappa = __builtin_fmaxf(kappa, part[first + w]);
        const bool writes_step = (uint32_t)wave == first;
        if (t.len == TILE)
            encode_tile<DT, MODE, true, true, false, BITSW>(a, t, tile_id, regs, kappa, writes_step, stage, lane);
        else if (t.len != 0)
            encode_tile<DT, MODE, true, false, false, BITSW>(a, t, tile_id, regs, kappa, writes_step, stage, lane);
    } else if (t.len == TILE) {
        TileRegs<DT> regs;
        load_tile<DT, true>(a.g, t, lane, regs);
        const float kappa = (FUSED && !MULTI) ? tile_max<DT>(regs) : 0.0f;
        encode_tile<DT, MODE, FUSED, true, MULTI, BITSW>(a, t, tile_id, regs, kappa, true, stage, lane);
    } else if (t.len != 0) {
        TileRegs<DT> regs;
        load_tile<DT, false>(a.g, t, lane, regs);
        const float kappa = (FUSED && !MULTI) ? tile_max<DT>(regs) : 0.0f;
        encode_tile<DT, MODE, FUSED, false, MULTI, BITSW>(a, t, tile_id, regs, kappa, true, stage, lane);
    }
    wave_lds_sync();     // a wave copies out only the stage it filled itself
    if (t.len != 0) stage_to_stream<DT, FUSED>(a, t, bits, stage, lane);
}

template <int DT, int MODE, bool FUSED, bool MULTI, bool BLOCK, int BITSW = 0>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(EncWaves<DT>::W)))
void encode_kernel(EncodeBatch by_value)
{
    const EncodeBatchPtr batch = (EncodeBatchPtr)__builtin_amdgcn_kernarg_segment_ptr();
    EncodeArgs a = common_args(batch);
    select_job(a, batch, blockIdx.y);
    constexpr uint32_t TILE = EncTile<DT>::N;
    __shared__ __align__(16) unsigned char stage_all[kWavesPerBlock][TILE + 8];
    __shared__ float part[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);   // wave-uniform
    const uint32_t tile_id = blockIdx.x * kWavesPerBlock + wave;
    const TileRef t = locate_tile(a.tl, tile_id, TILE);
    encode_wave<DT, MODE, FUSED, MULTI, BLOCK, BITSW>(a, t, tile_id, wave, lane, stage_all[wave], part);
}

// ---------------------------------------------------------------------------
// Encoder for short vectors: the vectors of ALL quantizers of a call in one launch (a launch of few
// waves takes 3 to 5 us whatever it does), each workgroup going by its vector's mode and code width.
//   FORM  kFormBucket: a bucket is at most a tile   kFormMulti: several share one   kFormBlock: 2 or 4 tiles
//         kFormVector: one step for the whole vector
// kFormVector, step from the vector's own max-norm: the workgroup reduces the parts of the max-norm pass by
// itself, which spares the launch between (absmax_finish_kernel).  The codes will overwrite the parts, so every
// workgroup has a copy of them to itself, at the start of the codes it is going to write
// (ShortShare; absmax_copies_kernel writes all the copies).
// ---------------------------------------------------------------------------
//         kFormLong: the same for long binary32 vectors of several quantizers, whose steps are all in memory: what
//         is spared is the end of one launch and the start of the next (1 + 15 workers of 11.2 M: see run_long)
enum ShortForm { kFormBucket = 0, kFormMulti = 1, kFormBlock = 2, kFormVector = 3, kFormLong = 4 };
struct ShortJob : EncodeJob {
    Quant qp;
    uint64_t total_bytes;
    float preset_step;
    uint32_t variant;      // 8 * mode + code width
    uint32_t parts;        // kFormVector: parts to reduce; 0: the step is preset or in memory
    uint32_t levels;       // the parts' step: levels of the vector that chose it
    uint32_t writes;       // kFormLong: 0 when the step already lies where it would be written
};
struct ShortBatch {
    ShortJob job[kEncJobs];
    Tiling tl;
    uint32_t rows_log2, num_buckets, waves_log2;
    uint32_t groups;       // kFormVector: workgroups per vector
};
typedef const __attribute__((address_space(4))) ShortBatch* ShortBatchPtr;
static_assert(sizeof(ShortBatch) <= 4096, "kernel arguments");

// kFormVector: the tiles of workgroup `group` of `groups`, as even as whole tiles go, so that also the last
// one, which ends with the vector, has codes enough to hold its copy of the parts.
struct ShortShare {
    uint32_t first, count;
    __host__ __device__ __forceinline__ ShortShare(uint32_t tiles, uint32_t groups, uint32_t group)
    {
        const uint32_t base = tiles / groups, extra = tiles - base * groups;
        first = group * base + (group < extra ? group : extra);
        count = base + (group < extra ? 1u : 0u);
    }
};

template <int DT, int FORM, int MODE, int BITSW>
__device__ __forceinline__ void encode_short(const EncodeArgs& a, const TileRef& t, uint32_t tile_id, int wave, int lane,
                                             unsigned char* stage, float (&part)[kWavesPerBlock], uint32_t parts,
                                             uint32_t levels, uint32_t writes, const float* copy)
{
    if constexpr (FORM != kFormVector && FORM != kFormLong) {
        encode_wave<DT, MODE, true, FORM == kFormMulti, FORM == kFormBlock, BITSW>(a, t, tile_id, wave, lane, stage, part);
    } else {
        constexpr uint32_t TILE = EncTile<DT>::N;
        TileRegs<DT> regs;
        if (t.len == TILE) load_tile<DT, true, FORM == kFormVector>(a.g, t, lane, regs);
        else if (t.len != 0) load_tile<DT, false, FORM == kFormVector>(a.g, t, lane, regs);
        float step;
        if (FORM == kFormVector && parts != 0u) {
            const float mine = wave_max((uint32_t)threadIdx.x < parts ? copy[threadIdx.x] : 0.0f);
            if (lane == 0) part[wave] = mine;
            __syncthreads();     // and the copy has been read: the codes may take its place
            float all = part[0];
#pragma unroll
            for (int w = 1; w < kWavesPerBlock; ++w) all = __builtin_fmaxf(all, part[w]);
            step = step_from_kappa(all, levels);
        } else {
            step = a.preset_step > 0.0f ? a.preset_step : a.step_in[0];
        }
        if (tile_id == 0u && lane == 0 && (FORM == kFormVector || writes != 0u)) a.steps[0] = step;
        if (t.len == TILE) encode_tile<DT, MODE, false, true, false, BITSW, false, true>(a, t, tile_id, regs, step, false, stage, lane);
        else if (t.len != 0) encode_tile<DT, MODE, false, false, false, BITSW, false, true>(a, t, tile_id, regs, step, false, stage, lane);
        wave_lds_sync();
        if (t.len != 0) stage_to_stream<DT, false>(a, t, BITSW, stage, lane);
    }
}

// The variants a workgroup may meet.  (A step that is not the vector's own comes with kFormVector only.)
template <int FORM> struct ShortVariants {
    using list = std::integer_sequence<int, 8 * kDqNarrow + 1, 8 * kDqNarrow + 2, 8 * kDqNarrow + 3, 8 * kDqNarrow + 4,
                                       8 * kNestedPow2Bounded + 1, 8 * kNestedPow2Bounded + 2, 8 * kNestedPow2Bounded + 3,
                                       8 * kNestedPow2Bounded + 4, 8 * kNestedAnyMBounded + 2, 8 * kNestedAnyMBounded + 3>;
};
template <> struct ShortVariants<kFormVector> {
    using list = std::integer_sequence<int, 8 * kDqNarrow + 1, 8 * kDqNarrow + 2, 8 * kDqNarrow + 3, 8 * kDqNarrow + 4,
                                       8 * kNestedPow2Bounded + 1, 8 * kNestedPow2Bounded + 2, 8 * kNestedPow2Bounded + 3,
                                       8 * kNestedPow2Bounded + 4, 8 * kNestedAnyMBounded + 2, 8 * kNestedAnyMBounded + 3,
                                       8 * kNestedPow2 + 1, 8 * kNestedPow2 + 2, 8 * kNestedPow2 + 3, 8 * kNestedPow2 + 4>;
};
template <> struct ShortVariants<kFormLong> : ShortVariants<kFormVector> {};
template <int... V>
constexpr bool short_variant(uint32_t variant, std::integer_sequence<int, V...>) { return ((variant == (uint32_t)V) || ...); }

template <int DT, int FORM, int... V>
__device__ __forceinline__ void encode_short_any(uint32_t variant, std::integer_sequence<int, V...>, const EncodeArgs& a,
                                                 const TileRef& t, uint32_t tile_id, int wave, int lane, unsigned char* stage,
                                                 float (&part)[kWavesPerBlock], uint32_t parts, uint32_t levels,
                                                 uint32_t writes, const float* copy)
{
    (void)((variant == (uint32_t)V
                ? (encode_short<DT, FORM, V / 8, V % 8>(a, t, tile_id, wave, lane, stage, part, parts, levels, writes, copy), true)
                : false) || ...);
}

template <int DT, int FORM>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(EncWaves<DT>::W)))
void encode_short_kernel(ShortBatch by_value)
{
    const ShortBatchPtr batch = (ShortBatchPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const __attribute__((address_space(4))) ShortJob* job = &batch->job[blockIdx.y];
    EncodeArgs a;
    a.g = job->g;
    a.codes = job->codes;
    a.steps = job->steps;
    a.step_in = job->step_in;
    a.index0 = job->index0;
    a.ds.key0 = job->ds.key0; a.ds.key1 = job->ds.key1; a.ds.step = job->ds.step; a.ds.worker = job->ds.worker;
    a.tl.n = batch->tl.n;
    a.tl.bucket_len = batch->tl.bucket_len;
    a.tl.tiles_per_bucket = batch->tl.tiles_per_bucket;
    a.tl.total_tiles = batch->tl.total_tiles;
    a.total_bytes = job->total_bytes;
    a.qp.q_min_f = job->qp.q_min_f; a.qp.q_max_f = job->qp.q_max_f; a.qp.q_min = job->qp.q_min;
    a.qp.levels = job->qp.levels; a.qp.M = job->qp.M; a.qp.M_f = job->qp.M_f; a.qp.inv_M_f = job->qp.inv_M_f;
    a.qp.bits = job->qp.bits; a.qp.pack_bias = job->qp.pack_bias; a.qp.alpha = job->qp.alpha; a.qp.beta = job->qp.beta;
    a.preset_step = job->preset_step;
    a.rows_log2 = batch->rows_log2;
    a.num_buckets = batch->num_buckets;
    a.waves_log2 = batch->waves_log2;
    a.through = 0u;           // (launches of few codes)
    constexpr uint32_t TILE = EncTile<DT>::N;
    __shared__ __align__(16) unsigned char stage_all[kWavesPerBlock][TILE / 2 + 8];      // at most 4 bits a code
    __shared__ float part[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    uint32_t tile_id = blockIdx.x * kWavesPerBlock + wave;
    const float* copy = nullptr;
    if (FORM == kFormVector) {
        const ShortShare share(a.tl.total_tiles, batch->groups, blockIdx.x);
        tile_id = (uint32_t)wave < share.count ? share.first + wave : a.tl.total_tiles;
        copy = (const float*)(a.codes + (uint64_t)share.first * (TILE / 8u) * a.qp.bits);
    }
    const TileRef t = locate_tile(a.tl, tile_id, TILE);
    encode_short_any<DT, FORM>(job->variant, typename ShortVariants<FORM>::list{}, a, t, tile_id, wave, lane, stage_all[wave],
                               part, job->parts, job->levels, job->writes, copy);
}

// The same for a full tile that is not the vector's last, with the code width known
// at compile time: a fixed number of store instructions, so that the compiler can
// count the memory operations in flight between a tile's loads and its use.
template <int DT, int BITSW>
__device__ __forceinline__ void stage_to_stream_full(const EncodeArgs& a, const TileRef& t,
                                                     const unsigned char* stage, int lane)
{
    constexpr uint32_t units = EncTile<DT>::N / 64u * BITSW;       // 8-byte units: a multiple of 64 for bfloat16 tiles
    uint64_t* dst = (uint64_t*)(a.codes + (t.start >> 3) * BITSW);
    const uint64_t* src = (const uint64_t*)stage;
    if constexpr (units % kWave == 0u) {
#pragma unroll
        for (uint32_t u = 0; u < units; u += kWave) store_through(dst + u + lane, src[u + lane]);
    } else {
        static_assert(units < (uint32_t)kWave, "a partial store only for less than one unit per lane");
        if ((uint32_t)lane < units) store_through(dst + lane, src[lane]);
    }
}

// ---------------------------------------------------------------------------
// Streaming encoder for vectors whose buckets are tiles (the max-norm found in
// registers): every wave
// walks over the tiles wave, wave + W, wave + 2W, ... (W = waves in the grid).
// One set of registers holds the current tile and, by the end of it, the next
// one: as soon as a row is quantized its registers are loaded again with the
// same row of the wave's next tile, so the loads leave one row at a time
// instead of a tile at a time, and a row has the rest of the tile's arithmetic
// (the first) down to the copy-out (the last) to arrive.  Measured against two
// register sets with the whole next tile requested at the start of the current
// one: 49.7 against 52.6 us (1-bit nested) and 57.5 against 59.9 us (2-bit
// DQSG) at 2^27 bfloat16 elements; with the registers this frees, 5, 6 or 8
// waves per SIMD are slower than 4 (55, 55, 54 us), and so are 3 and 2.
// No wave is ever new: the instruction arbiter serves older waves first, so in
// a one-tile-per-wave grid a new wave crawls through its address arithmetic,
// its loads and its max-norm behind busy neighbours, and the SIMD idles
// whenever those neighbours run out at the same time.
// ---------------------------------------------------------------------------
#ifndef NDQ_STREAM_WAVES
#define NDQ_STREAM_WAVES 4
#endif
constexpr int kStreamWaves = NDQ_STREAM_WAVES;   // per SIMD

template <int DT>
__device__ __forceinline__ TileRef stream_tile_ref(uint32_t tile_id)
{
    TileRef t;
    t.start = (uint64_t)tile_id * EncTile<DT>::N;
    t.len = EncTile<DT>::N;
    t.bucket = tile_id;
    return t;
}

template <int DT, int MODE, int BITSW>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kStreamWaves, kStreamWaves)))
void encode_stream_kernel(EncodeBatch by_value, uint32_t full_tiles)
{
    constexpr uint32_t TILE = EncTile<DT>::N;
    __shared__ __align__(16) unsigned char stage_all[kWavesPerBlock][TILE + 8];
    const EncodeBatchPtr batch = (EncodeBatchPtr)__builtin_amdgcn_kernarg_segment_ptr();
    EncodeArgs a = common_args(batch);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    unsigned char* stage = stage_all[wave];
    const uint32_t stride = gridDim.x * kWavesPerBlock;
    const uint32_t first = blockIdx.x * kWavesPerBlock + wave;
    const uint32_t jobs = batch->jobs;
    const uint32_t all_tiles = jobs * full_tiles;      // job after job: tile `t` of job j is j * full_tiles + t
    if (first < all_tiles) {
        // Every pass over a tile issues exactly one load per row, also the last one (then of the
        // vector's first 16 bytes per row, all lanes alike: one cache line, no traffic to speak
        // of), and the code width is a compile-time constant, so that the number of memory
        // operations in flight at every wait is known at compile time: they complete in order,
        // and a wait must cover a row's load but not the loads and stores issued after it.
        TileRegs<DT> regs;
        uint32_t cur = first, job = first / full_tiles, tile = first - job * full_tiles;
        // The arbiter serves the oldest wave of a SIMD first, so left alone the waves of a
        // SIMD finish one after the other and the last one runs alone, at a third of the
        // SIMD's rate.  Lower a wave's priority as it gets ahead: they finish together.
        const uint32_t my_tiles = (all_tiles - first + stride - 1) / stride;
        uint32_t done = 0;
        __builtin_amdgcn_s_setprio(3);
        select_job(a, batch, job);
        load_tile<DT, true>(a.g, stream_tile_ref<DT>(tile), lane, regs);
        for (;;) {
            const uint32_t nxt = cur + stride;
            const bool more = nxt < all_tiles;
            uint32_t next_job = job, next_tile = tile + stride;
            while (next_tile >= full_tiles && more) { next_tile -= full_tiles; ++next_job; }
            const void* next_g = batch->job[more ? next_job : job].g;
            const TileRef t = stream_tile_ref<DT>(tile);
            const float kappa = tile_max<DT>(regs);
            wave_lds_sync();     // the previous tile's copy-out has read the stage
            encode_tile<DT, MODE, true, true, false, BITSW, true>(
                a, t, tile, regs, kappa, true, stage, lane,
                (const typename Elem<DT>::scalar*)next_g + (uint64_t)(more ? next_tile : 0u) * TILE, more ? lane : 0);
            wave_lds_sync();
            stage_to_stream_full<DT, BITSW>(a, t, stage, lane);
            if (!more) break;
            ++done;
            const uint32_t quarter = 4u * done / my_tiles;
            if (quarter == 1u) __builtin_amdgcn_s_setprio(2);
            else if (quarter == 2u) __builtin_amdgcn_s_setprio(1);
            else if (quarter >= 3u) __builtin_amdgcn_s_setprio(0);
            cur = nxt; job = next_job; tile = next_tile;
            select_job(a, batch, job);
        }
    }
    // the ragged last tile of every vector, if there is one, by the wave whose turn it would be
    if (full_tiles < a.tl.total_tiles) {
        for (uint32_t j = 0; j < jobs; ++j) {
            if ((all_tiles + j) % stride != first) continue;
            select_job(a, batch, j);
            const TileRef t = locate_tile(a.tl, full_tiles, TILE);
            if (t.len != 0) {
                TileRegs<DT> regs;
                load_tile<DT, false>(a.g, t, lane, regs);
                const float kappa = tile_max<DT>(regs);
                wave_lds_sync();
                encode_tile<DT, MODE, true, false, false, BITSW>(a, t, full_tiles, regs, kappa, true, stage, lane);
                wave_lds_sync();
                stage_to_stream<DT, true>(a, t, BITSW ? (uint32_t)BITSW : a.qp.bits, stage, lane);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Max-norm per bucket (two-pass path and ndq_absmax)
// ---------------------------------------------------------------------------
struct AbsmaxBatch {
    const void* g[kEncJobs];        // blockIdx.y: vectors of one length and type
    uint32_t* kappa_bits[kEncJobs]; // K words each
    uint32_t levels[kEncJobs];
    float* parts[kEncJobs];         // absmax_span_kernel: K * blocks_per_bucket floats each; null: atomics
    Tiling tl;
    uint64_t K;                     // buckets per vector
    uint64_t parts_bytes;           // memory behind each of `parts`
    uint32_t blocks_per_bucket;     // absmax_span_kernel
};
typedef const __attribute__((address_space(4))) AbsmaxBatch* AbsmaxBatchPtr;

// absmax_copies_kernel
struct CopiesBatch {
    const void* g[kEncJobs];           // blockIdx.y: the vectors that choose their step
    unsigned char* codes[kEncJobs];    // the vectors that quantize with one of those steps, their own included:
    uint32_t bits[kEncJobs];           // where their workgroups' copies lie follows from their code width
    uint32_t source[kEncJobs];         // ... and whose parts they are (blockIdx.y)
    uint32_t users, groups;            // how many such vectors, and workgroups the encoder has for each
    Tiling tl;
};
typedef const __attribute__((address_space(4))) CopiesBatch* CopiesBatchPtr;

__global__ void fill_zero_kernel(AbsmaxBatch by_value)
{
    const AbsmaxBatchPtr b = (AbsmaxBatchPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < b->K) b->kappa_bits[blockIdx.y][i] = 0u;
}

// levels != 0: the bucket's step is wanted, not its max-norm.  The step rule is monotone in
// kappa (an exact doubling, one correctly rounded division, a threshold), so the maximum of
// the parts' steps is the step of the maximum: each part converts before its atomic, and no
// pass over the buckets is needed afterwards.
__device__ __forceinline__ uint32_t absmax_word(float m, uint32_t levels)
{
    // non-negative floats order like their bit patterns
    return __float_as_uint(levels ? step_from_kappa(m, levels) : m);
}

template <int DT, bool KEEP>
__global__ __launch_bounds__(kBlock) void absmax_kernel(AbsmaxBatch by_value)
{
    constexpr uint32_t TILE = EncTile<DT>::N;
    const AbsmaxBatchPtr b = (AbsmaxBatchPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const Tiling tl = {b->tl.n, b->tl.bucket_len, b->tl.tiles_per_bucket, b->tl.total_tiles};
    const void* g = b->g[blockIdx.y];
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t tile_id =
        blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const TileRef t = locate_tile(tl, tile_id, TILE);
    if (t.len == 0) return;
    TileRegs<DT> regs;
    if (t.len == TILE) load_tile<DT, true, KEEP>(g, t, lane, regs);
    else load_tile<DT, false, KEEP>(g, t, lane, regs);
    const float m = tile_max<DT>(regs);
    if (lane == 0) atomicMax(b->kappa_bits[blockIdx.y] + t.bucket, absmax_word(m, b->levels[blockIdx.y]));
}

// The same for buckets of many tiles (a whole vector at the extreme): a workgroup's
// waves stride over the bucket's tiles with the running max in registers, and each
// workgroup leaves one float.  Atomics on one address are served one after the other,
// about 18 ns each (a vector of 11 M binary32 elements: 11.5 us with 256 workgroups, 12,
// 18 and 27 us with 512, 1,024 and 1,365, which is the number that streams fastest), so an
// encoder's pass stores its parts and absmax_finish_kernel reduces them; the parts
// lie in the vector's code stream, which the encoder overwrites afterwards.
// ndq_absmax has no such memory: few workgroups, one atomic each.  A workgroup with a bucket to itself
// writes the word.
template <int DT, bool KEEP>
__global__ __launch_bounds__(kBlock) void absmax_span_kernel(AbsmaxBatch by_value)
{
    using T = Elem<DT>;
    constexpr uint32_t TILE = EncTile<DT>::N;
    const AbsmaxBatchPtr b = (AbsmaxBatchPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const Tiling tl = {b->tl.n, b->tl.bucket_len, b->tl.tiles_per_bucket, b->tl.total_tiles};
    const void* g = b->g[blockIdx.y];
    const uint32_t blocks_per_bucket = b->blocks_per_bucket;
    __shared__ float part[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t bucket = blockIdx.x / blocks_per_bucket;
    const uint32_t first = (blockIdx.x - bucket * blocks_per_bucket) * kWavesPerBlock + wave;
    const uint32_t stride = blocks_per_bucket * kWavesPerBlock;
    typename T::maxacc acc = T::max_init();
    for (uint32_t j = first; j < tl.tiles_per_bucket; j += stride) {
        const TileRef t = locate_tile(tl, bucket * tl.tiles_per_bucket + j, TILE);
        if (t.len == 0) break;   // past the end of the vector: so are this wave's later tiles
        TileRegs<DT> regs;
        if (t.len == TILE) load_tile<DT, true, KEEP>(g, t, lane, regs);
        else load_tile<DT, false, KEEP>(g, t, lane, regs);
        acc = lane_max<DT>(acc, regs);
    }
    const float m = wave_max(T::max_final(acc));
    if (lane == 0) part[wave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        float all = part[0];
#pragma unroll
        for (int w = 1; w < kWavesPerBlock; ++w) all = __builtin_fmaxf(all, part[w]);
        float* parts = b->parts[blockIdx.y];
        uint32_t* word = b->kappa_bits[blockIdx.y] + bucket;
        if (blocks_per_bucket == 1u) *word = absmax_word(all, b->levels[blockIdx.y]);
        else if (parts) parts[blockIdx.x] = all;
        else atomicMax(word, absmax_word(all, b->levels[blockIdx.y]));
    }
}

// The same for one bucket per vector whose encoder is encode_short_kernel: the workgroup's part goes to
// every workgroup of the encoder that needs it.
template <int DT>
__global__ __launch_bounds__(kBlock) void absmax_copies_kernel(CopiesBatch by_value)
{
    using T = Elem<DT>;
    constexpr uint32_t TILE = EncTile<DT>::N;
    const CopiesBatchPtr b = (CopiesBatchPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const Tiling tl = {b->tl.n, b->tl.bucket_len, b->tl.tiles_per_bucket, b->tl.total_tiles};
    const void* g = b->g[blockIdx.y];
    __shared__ float part[kWavesPerBlock];
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    typename T::maxacc acc = T::max_init();
    for (uint32_t j = blockIdx.x * kWavesPerBlock + wave; j < tl.total_tiles; j += gridDim.x * kWavesPerBlock) {
        const TileRef t = locate_tile(tl, j, TILE);
        TileRegs<DT> regs;
        if (t.len == TILE) load_tile<DT, true, true>(g, t, lane, regs);
        else load_tile<DT, false, true>(g, t, lane, regs);
        acc = lane_max<DT>(acc, regs);
    }
    const float m = wave_max(T::max_final(acc));
    if (lane == 0) part[wave] = m;
    __syncthreads();
    float all = part[0];
#pragma unroll
    for (int w = 1; w < kWavesPerBlock; ++w) all = __builtin_fmaxf(all, part[w]);
    const uint32_t groups = b->groups;
    for (uint32_t u = 0; u < b->users; ++u) {
        if (b->source[u] != blockIdx.y) continue;
        const uint32_t tile_bytes = TILE / 8u * b->bits[u];
        for (uint32_t e = threadIdx.x; e < groups; e += kBlock)
            ((float*)(b->codes[u] + (uint64_t)ShortShare(tl.total_tiles, groups, e).first * tile_bytes))[blockIdx.x] = all;
    }
}

// The step of one bucket from the parts absmax_span_kernel left.
__global__ __launch_bounds__(kBlock) void absmax_finish_kernel(AbsmaxBatch by_value)
{
    const AbsmaxBatchPtr b = (AbsmaxBatchPtr)__builtin_amdgcn_kernarg_segment_ptr();
    const uint32_t count = b->blocks_per_bucket;
    const float* parts = b->parts[blockIdx.y] + (size_t)blockIdx.x * count;
    __shared__ float part[kWavesPerBlock];
    float m = 0.0f;
    for (uint32_t i = threadIdx.x; i < count; i += kBlock) m = __builtin_fmaxf(m, parts[i]);
    m = wave_max(m);
    if ((threadIdx.x & (kWave - 1)) == 0u) part[threadIdx.x / kWave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        float all = part[0];
#pragma unroll
        for (int w = 1; w < kWavesPerBlock; ++w) all = __builtin_fmaxf(all, part[w]);
        b->kappa_bits[blockIdx.y][blockIdx.x] = absmax_word(all, b->levels[blockIdx.y]);
    }
}

// ---------------------------------------------------------------------------
// Host side: dispatch
// ---------------------------------------------------------------------------
// Whether the pass leaves its lines in the caches for the encoder (its loads are cached instead of
// streaming).  `bytes`: the vectors of the launch, all of which are read before the first encoder runs.
// binary32 (steps for the whole vector): 25.6 M elements 37.2 us against 42.7 streaming, 8 x 11 M 124.5 /
// 137, 16 x 8 M (512 MiB) 191.5 / 200.5, 200 M (763 MiB) 285 / 290; beyond that the cached loads themselves are
// the slower ones: 300 M 442 / 433, 16 x 25 M 605 / 585, 393 M in 3,000 buckets 585 / 572.
// bfloat16: 11 M (22 MB, within the L2s) 14.8 / 15.7, 25.6 M 27.9 / 25.3, 4 x 11 M 41.4 / 38.7, 300 M 238 / 217.
// ndq_absmax, which no encoder follows: at 2^27 binary32 elements, buckets of 2,048, 89.4 / 86.9.
template <int DT>
static bool absmax_keeps(uint64_t bytes, bool encoder_follows)
{
    const uint64_t most = DT == 1 ? (uint64_t)32 << 20 : encoder_follows ? (uint64_t)768 << 20 : (uint64_t)256 << 20;
    return bytes <= most;
}

// b: vectors, words, levels, tiling and (for an encoder) memory for the parts are set.
template <int DT, bool KEEP>
static int run_absmax_loads(AbsmaxBatch& b, uint32_t jobs, hipStream_t s)
{
    // Many tiles per bucket: workgroups that stride over one, at any number of buckets (3,000 buckets of
    // 64 tiles, binary32: 572 us against 602 with an atomic per tile, of 32 tiles 288 / 298).  With
    // memory for the parts a full chip of waves; with atomics one workgroup per compute unit; a workgroup that
    // has a bucket to itself writes its word.  What counts are the tiles that hold elements: a bucket may
    // be longer than the whole vector.
    constexpr uint32_t kSpanMinTiles = 16;
    // (binary32 with streaming loads is the only one to gain from twice the workgroups: 250 M elements 366 ->
    // 361 us, 16 x 25 M 595 -> 585; cached, 25.6 M 37.2 -> 38.9; bfloat16, 60 M 50.5 -> 52.1)
    const uint32_t target = !b.parts[0] ? 256u : DT == 0 && !KEEP ? 4096u : 2048u;
    const uint64_t tiles = b.K == 1u ? (b.tl.n + EncTile<DT>::N - 1u) / EncTile<DT>::N : b.tl.tiles_per_bucket;
    if (tiles >= kSpanMinTiles) {
        uint32_t per_bucket = (uint32_t)(target / (b.K * jobs));
        const uint32_t most = blocks_for((uint32_t)tiles);
        if (per_bucket > most) per_bucket = most;
        // a part is 4 bytes.  A workgroup has a tile, 256 bytes of 1-bit codes, so the parts always fit
        // (K >= 2: only the last bucket is short, and the others have 16 tiles); no plan may write past them
        if (b.parts[0] && per_bucket > b.parts_bytes / (4u * b.K)) per_bucket = (uint32_t)(b.parts_bytes / (4u * b.K));
        if (per_bucket < 1u) per_bucket = 1u;
        b.blocks_per_bucket = per_bucket;
        const bool parts = b.parts[0] && per_bucket > 1u, atomics = !b.parts[0] && per_bucket > 1u;
        if (atomics && launch(fill_zero_kernel, dim3((uint32_t)((b.K + 255) / 256), jobs), dim3(256), s, b) != NDQ_OK)
            return NDQ_ELAUNCH;
        if (launch((absmax_span_kernel<DT, KEEP>), dim3((uint32_t)b.K * per_bucket, jobs), dim3(kBlock), s, b) != NDQ_OK)
            return NDQ_ELAUNCH;
        return parts ? launch(absmax_finish_kernel, dim3((uint32_t)b.K, jobs), dim3(kBlock), s, b) : NDQ_OK;
    }
    if (launch(fill_zero_kernel, dim3((uint32_t)((b.K + 255) / 256), jobs), dim3(256), s, b) != NDQ_OK)
        return NDQ_ELAUNCH;
    return launch((absmax_kernel<DT, KEEP>), dim3(blocks_for((uint32_t)(tiles * b.K)), jobs), dim3(kBlock), s, b);
}

template <int DT>
static int run_absmax(AbsmaxBatch& b, uint32_t jobs, hipStream_t s)
{
    const uint64_t bytes = b.tl.n * sizeof(typename Elem<DT>::scalar) * jobs;
    return absmax_keeps<DT>(bytes, b.parts[0] != nullptr) ? run_absmax_loads<DT, true>(b, jobs, s)
                                                          : run_absmax_loads<DT, false>(b, jobs, s);
}

// Waves of the streaming kernel: kStreamWaves on each of the 1,024 SIMDs.
constexpr uint32_t kStreamSlots = 1024u * kStreamWaves;

template <int DT, int MODE, int BITSW>
static int launch_stream(const EncodeBatch& b, uint32_t full_tiles, hipStream_t s)
{
    const uint32_t blocks = persistent_blocks(full_tiles * b.jobs, kStreamSlots);
    return launch((encode_stream_kernel<DT, MODE, BITSW>), dim3(blocks), dim3(kBlock), s, b, full_tiles);
}

// Tiles of a launch from which the streaming kernel is the faster one (bfloat16; the time of one tile per wave is what
// has come down since it was made, by code widths known at compile time).  One tile per wave over this, encoder calls on
// vectors that are in no cache, at 4 x 8.4 M, 4 x 11.2 M, 67 M, 2 x 50 M, 8 x 16 M, 3 x 134 M elements (2 to 24 tiles per wave slot):
//   buckets of a tile   4 levels 1.02 0.98 1.07 1.00 0.99         2 levels 0.98 0.97 1.02 1.00 1.01
//                       16 levels 1.00 0.99 1.02 1.06 1.07        M = 2 0.97 0.95 1.05 1.00 1.00     M = 4 0.95 0.91 1.00 0.99 0.99 1.05
// (us persistent, buckets of a tile, 4 levels 17.4 23.4 30.0 44.3 54.7.)  Buckets smaller than a tile and codes of 3 bits gain 3
// to 5 % by it at 8 x 16 M and lose as much below 2 x 50 M: they are left to the other kernel.  So are vectors with one step, which
// it had too: one tile per wave over this at 34, 41, 50, 60, 75, 100, 134, 200 and 268 M elements, 4 levels 0.94 0.93 1.00 1.00 1.00 0.99 0.98
// 0.97 0.97, 2 levels 0.96 0.96 0.98 0.96 0.99 1.00 0.99 0.97 0.96, 16 levels 0.99 0.94 0.97 0.96 0.96 0.98 0.98 0.97 0.98, M = 4 0.93 0.94 1.00
// 0.99 1.00 1.00 0.99 0.98 0.97 (4 to 6 whole rounds of 2-bit codes: 1.02).
static uint64_t stream_from_tiles(bool nested, uint32_t bits)
{
    const StreamTuning& tuning = stream_tuning();
    if (tuning.threshold_from_env) return (uint64_t)tuning.min_tiles_per_wave * kStreamSlots;
    return (nested && bits == 2u ? 16u : 3u) * kStreamSlots;
}

// The streaming kernel serves vectors whose buckets are tiles (a ragged last one aside), in the quantizer modes and code
// widths of the common configurations.  Returns 1 when it does not apply.
template <int DT, int MODE>
static int try_stream(const EncodeBatch& b, bool fused, bool multi, uint32_t bucket, hipStream_t s)
{
    const EncodeArgs& a = b.common;
    constexpr uint32_t TILE = EncTile<DT>::N;
    // binary32 input: one tile per wave is faster at every length (2^27 elements: 112 against 120 us,
    // 25.6 M: 22.8 against 23.2; its tile carries half the arithmetic of a bfloat16 tile per byte, so
    // the kernel is nearer to a plain copy, which gains nothing from persistence)
    if constexpr (DT == 0 || (MODE != kDqNarrow && MODE != kNestedPow2Bounded)) {
        return 1;
    } else {
    if (multi || a.waves_log2 != 0u) return 1;
    if (bucket != TILE || !fused) return 1;
    const uint32_t full_tiles = (uint32_t)(a.tl.n / TILE);
    const uint32_t bits = a.qp.bits;
    const uint64_t all_tiles = (uint64_t)full_tiles * b.jobs;
    if (full_tiles == 0u || all_tiles < stream_from_tiles(MODE != kDqNarrow, bits) || all_tiles >= ((uint64_t)1 << 31))
        return 1;
    if (bits != 1u && bits != 2u && bits != 4u) return 1;
    if (bits == 1u) return launch_stream<DT, MODE, 1>(b, full_tiles, s);
    if (bits == 2u) return launch_stream<DT, MODE, 2>(b, full_tiles, s);
    return launch_stream<DT, MODE, 4>(b, full_tiles, s);
    }
}

// Whether a mode has instantiations of its own for code width BITS: the narrow DQSG and power-of-two nested codes
// (1 to 4 bits), other nesting ratios from 3 to 8 (2 and 3 bits).
template <int MODE, int BITS>
constexpr bool kWidthKnown = MODE == kNestedAnyMBounded ? BITS == 2 || BITS == 3
                                                        : MODE == kDqNarrow || MODE == kNestedPow2Bounded || MODE == kNestedPow2;

template <int DT, int MODE, bool FUSED, bool MULTI, bool BLOCK>
static int launch_encode(const EncodeBatch& b, hipStream_t s)
{
    const dim3 grid(blocks_for(b.common.tl.total_tiles), b.jobs), block(kBlock);
    const uint32_t bits = b.common.qp.bits;
    if constexpr (kWidthKnown<MODE, 1>)
        if (bits == 1u) return launch((encode_kernel<DT, MODE, FUSED, MULTI, BLOCK, 1>), grid, block, s, b);
    // (bfloat16, M = 3, buckets shorter than a row: 4 x 11 M in buckets of 64 1,338 us with the width read from the arguments and
    // 1,445 with it known, of 192 454 and 486; from a row on known is the better one)
    const bool short_bucket = DT == 1 && MODE == kNestedAnyMBounded && b.common.tl.bucket_len < kWave * kLaneElems;
    if constexpr (kWidthKnown<MODE, 2>)
        if (bits == 2u && !short_bucket) return launch((encode_kernel<DT, MODE, FUSED, MULTI, BLOCK, 2>), grid, block, s, b);
    if constexpr (kWidthKnown<MODE, 3>)
        if (bits == 3u) return launch((encode_kernel<DT, MODE, FUSED, MULTI, BLOCK, 3>), grid, block, s, b);
    if constexpr (kWidthKnown<MODE, 4>)
        if (bits == 4u) return launch((encode_kernel<DT, MODE, FUSED, MULTI, BLOCK, 4>), grid, block, s, b);
    return launch((encode_kernel<DT, MODE, FUSED, MULTI, BLOCK, 0>), grid, block, s, b);
}

template <int DT, int MODE>
static int run_encode(const EncodeBatch& b, bool fused, bool multi, uint32_t bucket, hipStream_t s)
{
#ifndef NDQ_NO_STREAM_ENCODER
    const int rc = try_stream<DT, MODE>(b, fused, multi, bucket, s);
    if (rc != 1) return rc;
#endif
    if constexpr (MODE == kNestedPow2) {      // a step that is not the bucket's own comes with bucket == 0
        return launch_encode<DT, MODE, false, false, false>(b, s);
    } else {
        if (b.common.waves_log2 != 0u) return launch_encode<DT, MODE, true, false, true>(b, s);
        if (multi) return launch_encode<DT, MODE, true, true, false>(b, s);
        return fused ? launch_encode<DT, MODE, true, false, false>(b, s) : launch_encode<DT, MODE, false, false, false>(b, s);
    }
}

// One vector's call, checked and planned.  Vectors whose plans agree in everything but the
// EncodeJob part share a launch.
struct EncodePlan {
    EncodeArgs a;
    int mode;
    bool fused, multi;
    bool two_pass;       // the steps come from a max-norm pass of their own
    bool handed;         // the step is read from memory the caller named
};

static bool same_launch(const EncodePlan& p, const EncodePlan& q)
{
    return p.mode == q.mode && p.two_pass == q.two_pass && p.a.preset_step == q.a.preset_step &&
           memcmp(&p.a.qp, &q.a.qp, sizeof(Quant)) == 0;   // (length, type and bucket are the call's)
}

// job.step_in != nullptr: one step for the whole vector, read from device memory when the
// kernels run (bucket and delta are then not used, nor `levels` to derive a step).
static int plan_encode(const ndq_encode_job& job, int dt, size_t n, float delta, uint32_t bucket, EncodePlan* plan)
{
    EncodeArgs& a = plan->a;
    const bool nested = job.kind == NDQ_WORKER_NESTED;
    const uint32_t levels = job.levels;
    int rc = make_quant(levels, job.M, nested, job.alpha, &a.qp);
    if (rc != NDQ_OK) return rc;
    if (dt != NDQ_F32 && dt != NDQ_BF16) return NDQ_EINVAL;
    if (n == 0) return NDQ_OK;
    if (!job.g || !job.codes_out || !job.steps_out) return NDQ_EINVAL;
    if (!(delta == delta)) return NDQ_EINVAL;
    if (n >= kMaxN) return NDQ_EUNSUPPORTED;
    if (!aligned16(job.g) || !aligned16(job.codes_out) || !aligned4(job.steps_out)) return NDQ_EALIGN;
    if (job.step_in && !aligned4(job.step_in)) return NDQ_EALIGN;
    if (bucket % 64u != 0u || (job.dither.offset & 7u) != 0u) return NDQ_EALIGN;

    const uint32_t tile = dt == NDQ_F32 ? EncTile<0>::N : EncTile<1>::N;
    // buckets of 1, 2 or 4 whole rows (2, 4 or 8 to a tile) share tiles: the tiling is
    // that of tile-sized buckets and the kernel finds a max-norm per group of rows
    constexpr uint32_t row = kWave * kLaneElems;
    const bool multi = bucket != 0u && bucket < tile && tile % bucket == 0u && bucket % row == 0u &&
                       bucket / row <= 4u && (bucket / row & (bucket / row - 1u)) == 0u;
    rc = make_tiling(n, multi ? tile : bucket, tile, &a.tl);
    if (rc != NDQ_OK) return rc;
    a.rows_log2 = multi ? (bucket / row == 1u ? 0u : bucket / row == 2u ? 1u : 2u) : 0u;
    // buckets of 2 or 4 tiles: the waves of one workgroup hold the whole bucket
    const bool block_fused = kWavesPerBlock == 4 && (bucket == 2u * tile || bucket == 4u * tile);
    a.waves_log2 = block_fused ? (bucket == 2u * tile ? 1u : 2u) : 0u;
    a.num_buckets = (uint32_t)((n + (bucket ? bucket : n) - 1) / (bucket ? bucket : n));
    a.g = job.g;
    a.codes = (unsigned char*)job.codes_out;
    a.steps = job.steps_out;
    a.step_in = job.step_in ? job.step_in : job.steps_out;
    a.index0 = job.dither.offset;
    a.total_bytes = packed_bytes(n, a.qp.bits);
    a.ds = make_stream(&job.dither);
    a.preset_step = (bucket == 0u && delta > 0.0f && !job.step_in) ? delta : 0.0f;

    plan->multi = multi;
    plan->fused = (bucket != 0u && bucket <= tile) || block_fused;   // (multi implies fused)
    plan->two_pass = !job.step_in && !plan->fused && a.preset_step == 0.0f;
    plan->handed = job.step_in != nullptr;
#ifndef NDQ_NARROW_MAX_BITS
#define NDQ_NARROW_MAX_BITS 6u
#endif
    // a step derived from the data bounds |g/Delta|; a caller's step (preset, or in device memory) does not
    const bool own_step = a.preset_step == 0.0f && !job.step_in;
    plan->mode = !nested ? (a.qp.bits <= NDQ_NARROW_MAX_BITS ? kDqNarrow : kDq)
                         : (!is_pow2(job.M) ? ((!own_step || a.qp.bits > 6u) ? kNestedAnyM : kNestedAnyMBounded)
                                            : (!own_step ? kNestedPow2 : kNestedPow2Bounded));
    return NDQ_OK;
}

template <int DT>
static int run_encode_mode(const EncodeBatch& b, const EncodePlan& p, uint32_t bucket, hipStream_t s)
{
    if (p.mode == kDqNarrow) return run_encode<DT, kDqNarrow>(b, p.fused, p.multi, bucket, s);
    if (p.mode == kDq) return run_encode<DT, kDq>(b, p.fused, p.multi, bucket, s);
    if (p.mode == kNestedPow2) return run_encode<DT, kNestedPow2>(b, p.fused, p.multi, bucket, s);
    if (p.mode == kNestedPow2Bounded) return run_encode<DT, kNestedPow2Bounded>(b, p.fused, p.multi, bucket, s);
    if (p.mode == kNestedAnyMBounded) return run_encode<DT, kNestedAnyMBounded>(b, p.fused, p.multi, bucket, s);
    return run_encode<DT, kNestedAnyM>(b, p.fused, p.multi, bucket, s);
}

// Whether encode_short_kernel takes a batch; it then answers *rc.  Worth it while a launch more counts: encoder
// calls, us, this / a launch per quantizer, W vectors of n elements:
//   binary32, buckets of 1,024     8 + 8   61 k 5.4/8.9    267 k 7.1/11.4   1.05 M 14.8/17.4   1.66 M 23.3/25.2   3 M 40.5/40.4
//   bfloat16, buckets of 4,096     8 + 8   61 k 5.3/10.5   267 k 6.9/12.9   1.05 M 10.1/13.4   1.66 M 15.0/19.6   3 M 24.3/27.5
// so buckets up to 16,384 tiles in all.  A step per vector: this over the max-norm pass with its closing kernel and the
// encoders after it (binary32: one launch of those too, see run_long), and in brackets where it is not taken:
//   binary32   1        61 k 0.88   267 k 0.89   1.05 M 0.91   1.66 M 0.95  (2.2 M 1.05)
//              2        61 k 0.84   267 k 0.85   1.05 M 0.89   1.3 M 0.94   1.66 M 1.02
//              4        61 k 0.87   267 k 0.90   660 k 0.85    800 k 1.04   1.05 M 0.94  (1.3 M 1.09)
//              8        61 k 0.86   267 k 0.85   530 k 1.02   (800 k 1.08   930 k 1.10)
//              16       61 k 0.93   267 k 0.92   400 k 0.97   (530 k 1.10)
//              1 + 1    61 k 0.83   267 k 0.88   1.05 M 0.87   1.66 M 0.98
//              4 + 4    61 k 0.85   267 k 0.85   530 k 0.99   (800 k 1.04   930 k 1.06)
//      shared step      61 k 0.97   267 k 0.94   530 k 1.01   (800 k 1.08)
//      1 + 15 shared   (61 k 1.11   267 k 1.09   530 k 1.10)
//   bfloat16   1        61 k 0.91   267 k 0.94   1.05 M 0.93   2.2 M 0.96   3 M 0.99     (4.5 M 1.08)
//              4        61 k 0.91   267 k 0.93   1.05 M 0.91   1.66 M 1.04  (2.2 M 1.03)
//              16       61 k 0.95   267 k 0.94   530 k 0.98    800 k 1.03   (930 k 1.12)
//              1 + 1    61 k 0.62   267 k 0.62   1.05 M 0.64   2.2 M 0.72   3 M 0.79
//              4 + 4    61 k 0.63   267 k 0.62   1.05 M 0.76   1.66 M 0.86
//      1 + 15 shared    61 k 0.77   267 k 0.72   800 k 0.96    1.05 M 1.07
// What it costs are the copies: the more of them, the fewer workgroups the pass has (kShortCopies), and where one of those
// takes the tiles of three workgroups of the encoder, or of two and the others of one, it is what everything waits for.
constexpr uint32_t kShortBucketTiles = 16384, kShortVectorTiles = 6144;
template <int DT> constexpr uint32_t kShortOneQuantizerTiles = DT == 0 ? 4096 : 3200;
// Copies of parts to write, at most: every one is a store to a line of its own.  Iterations of 4 x 1.66 M elements, us, with at
// most 16 k / 32 k / 64 k / 128 k copies: 22.2-23.7 / 22.1 / 22.8-23.1 / 24.1-24.4, with absmax_finish_kernel 22.2; 4 x 900 k: 14.5-15.6 /
// 13.9 / 13.5-14.7 / 14.7, 15.1.
constexpr uint32_t kShortCopies = 32768;

static ShortJob short_job(const EncodePlan& p)
{
    ShortJob job;
    static_cast<EncodeJob&>(job) = p.a;
    job.qp = p.a.qp;
    job.total_bytes = p.a.total_bytes;
    job.preset_step = p.a.preset_step;
    job.variant = 8u * (uint32_t)p.mode + p.a.qp.bits;
    job.parts = 0u;
    job.levels = 0u;
    job.writes = p.two_pass ? 0u : 1u;
    return job;
}

// Long binary32 vectors with one step each, of several quantizers, after the max-norm passes.  Iterations, a launch
// per quantizer / this: 1 + 15 workers of 11.2 M elements 211 / 208.8 us, 1 + 7 of 4 M 65.4 / 62.2, 1 + 3 39.5 / 34.3, 1 + 1
// 27.4 / 22.0.  bfloat16 has the streaming kernel.  Whether it applies; it then answers *rc.
static bool run_long(const EncodePlan* plans, uint32_t jobs, int dt, uint32_t bucket, hipStream_t s, int* rc)
{
    if (dt != NDQ_F32 || bucket != 0u) return false;
    bool one_quantizer = true;
    for (uint32_t j = 0; j < jobs; ++j) {
        if (!short_variant(8u * (uint32_t)plans[j].mode + plans[j].a.qp.bits, ShortVariants<kFormLong>::list{})) return false;
        one_quantizer = one_quantizer && plans[j].a.qp.M == plans[0].a.qp.M && plans[j].a.qp.bits == plans[0].a.qp.bits;
    }
    if (one_quantizer) return false;
    ShortBatch b;
    for (uint32_t j = 0; j < jobs; ++j) b.job[j] = short_job(plans[j]);
    b.tl = plans[0].a.tl;
    b.rows_log2 = b.waves_log2 = 0u;
    b.num_buckets = 1u;
    b.groups = blocks_for(b.tl.total_tiles);
    *rc = launch((encode_short_kernel<0, kFormLong>), dim3(b.groups, jobs), dim3(kBlock), s, b);
    return true;
}

template <int DT>
static bool run_short(const EncodePlan* plans, uint32_t jobs, uint32_t bucket, hipStream_t s, int* rc)
{
    constexpr uint32_t TILE = EncTile<DT>::N;
    const EncodeArgs& first = plans[0].a;
    const bool vector = bucket == 0u;
    const uint64_t all_tiles = (uint64_t)first.tl.total_tiles * jobs;
    if (all_tiles > (vector ? kShortVectorTiles : kShortBucketTiles)) return false;
    if (!vector && !plans[0].fused) return false;       // (the form of a bucket is the same for all)
    // (a streaming threshold from the environment means that kernel, whatever the length: see try_stream)
    if (DT == 1 && stream_tuning().threshold_from_env && bucket == TILE) return false;
    bool one_quantizer = true, several = false;
    uint32_t sources = 0u;
    for (uint32_t j = 0; j < jobs; ++j) {
        const uint32_t variant = 8u * (uint32_t)plans[j].mode + plans[j].a.qp.bits;
        if (!(vector ? short_variant(variant, ShortVariants<kFormVector>::list{})
                     : short_variant(variant, ShortVariants<kFormBucket>::list{})))
            return false;
        one_quantizer = one_quantizer && plans[j].a.qp.M == first.qp.M && plans[j].a.qp.bits == first.qp.bits;
        several = several || (!same_launch(plans[0], plans[j]) && plans[0].two_pass == plans[j].two_pass);
        if (vector && plans[j].two_pass) ++sources;
    }
    if (sources == 0u && !several) return false;
    if (vector && one_quantizer && all_tiles > kShortOneQuantizerTiles<DT>) return false;
    ShortBatch b[2];        // the vectors of the first launch, and those of a second one
    uint32_t count[2] = {0u, 0u};
    CopiesBatch m;
    m.users = 0u;
    uint32_t chosen = 0u, narrow = 4u;
    for (uint32_t j = 0; j < jobs; ++j) {
        // A vector that is handed the step of one that chooses it here finds the step itself, from
        // parts like that one's, if the quantizers differ (the workers of Algorithm 2); the others that have
        // their step in memory or from the caller wait for a launch of their own where anything chooses.
        uint32_t source = kEncJobs, k = 0u;
        if (vector)
            for (uint32_t i = 0; i < jobs; ++i) {
                if (!plans[i].two_pass) continue;
                if (i == j || (!one_quantizer && i < j && plans[j].handed && plans[j].a.step_in == plans[i].a.steps)) source = k;
                ++k;
            }
        const uint32_t launch_of = source == kEncJobs && sources != 0u ? 1u : 0u;
        ShortJob& job = b[launch_of].job[count[launch_of]++];
        job = short_job(plans[j]);
        if (source == kEncJobs) continue;
        if (plans[j].two_pass) {
            m.g[chosen++] = plans[j].a.g;
            job.levels = plans[j].a.qp.levels;
        } else {
            for (uint32_t u = 0; u < m.users; ++u)
                if (m.source[u] == source) { job.levels = b[0].job[u].levels; break; }
        }
        m.codes[m.users] = plans[j].a.codes;
        m.bits[m.users] = plans[j].a.qp.bits;
        m.source[m.users++] = source;
        if (plans[j].a.qp.bits < narrow) narrow = plans[j].a.qp.bits;
    }
    const uint32_t tiles = first.tl.total_tiles, groups = blocks_for(tiles);
    if (sources != 0u) {
        // a copy of the parts fits the shortest share of the narrowest codes, the last one's; the
        // pass keeps a workgroup per compute unit, or one for every four of the encoder's
        const ShortShare last(tiles, groups, groups - 1u);
        const uint64_t bytes = packed_bytes(first.tl.n, narrow) - (uint64_t)last.first * (TILE / 8u) * narrow;
        uint32_t parts = groups < (uint32_t)kBlock ? groups : (uint32_t)kBlock;
        if (parts > bytes / 4u) parts = (uint32_t)(bytes / 4u);
        if (parts > kShortCopies / (groups * m.users)) parts = kShortCopies / (groups * m.users);
        if (parts == 0u || (4u * parts < groups && parts * sources < 256u)) return false;
        // no more than two of the encoder's workgroups for one of the pass, unless all have the same number: with one quantizer,
        // or binary32, a launch is all there is to spare
        if ((DT == 0 || one_quantizer) && 2u * parts < groups && groups % parts != 0u) return false;
        if (DT == 0 && m.users > 8u && sources < m.users) return false;
        for (uint32_t u = 0; u < m.users; ++u) b[0].job[u].parts = parts;
        m.tl = first.tl;
        m.groups = groups;
        *rc = launch(absmax_copies_kernel<DT>, dim3(parts, sources), dim3(kBlock), s, m);
        if (*rc != NDQ_OK) return true;
    }
    for (uint32_t i = 0; i < 2u; ++i) {
        if (count[i] == 0u) continue;
        b[i].tl = first.tl;
        b[i].rows_log2 = first.rows_log2;
        b[i].num_buckets = first.num_buckets;
        b[i].waves_log2 = first.waves_log2;
        b[i].groups = groups;
        const dim3 grid(groups, count[i]), block(kBlock);
        *rc = vector ? launch((encode_short_kernel<DT, kFormVector>), grid, block, s, b[i])
              : first.waves_log2 != 0u ? launch((encode_short_kernel<DT, kFormBlock>), grid, block, s, b[i])
              : plans[0].multi ? launch((encode_short_kernel<DT, kFormMulti>), grid, block, s, b[i])
                               : launch((encode_short_kernel<DT, kFormBucket>), grid, block, s, b[i]);
        if (*rc != NDQ_OK) return true;
    }
    return true;
}

// Up to kEncJobs planned vectors: first the max-norm passes of those that need one, all in
// one launch, then the encoders, one launch for all vectors of a kind.  Launches of many
// vectors instead of one per vector: a launch ramps up and drains once, and the next
// vector's loads overlap with this one's arithmetic.
static int run_plans(const EncodePlan* plans, uint32_t jobs, int dt, uint32_t bucket, hipStream_t s)
{
    int rc_short;
    if (dt == NDQ_F32 ? run_short<0>(plans, jobs, bucket, s, &rc_short) : run_short<1>(plans, jobs, bucket, s, &rc_short))
        return rc_short;
    AbsmaxBatch m;
    uint32_t need = 0;
    for (uint32_t j = 0; j < jobs; ++j) {
        if (!plans[j].two_pass) continue;
        m.g[need] = plans[j].a.g;
        m.kappa_bits[need] = (uint32_t*)plans[j].a.steps;
        m.levels[need] = plans[j].a.qp.levels;
        m.parts[need] = (float*)plans[j].a.codes;
        m.parts_bytes = need == 0u || plans[j].a.total_bytes < m.parts_bytes ? plans[j].a.total_bytes : m.parts_bytes;
        ++need;
    }
    if (need != 0u) {
        m.tl = plans[0].a.tl;
        m.K = plans[0].a.num_buckets;
        const int rc = dt == NDQ_F32 ? run_absmax<0>(m, need, s) : run_absmax<1>(m, need, s);
        if (rc != NDQ_OK) return rc;
    }
    if (run_long(plans, jobs, dt, bucket, s, &rc_short)) return rc_short;
    bool done[kEncJobs] = {};
    for (uint32_t j = 0; j < jobs; ++j) {
        if (done[j]) continue;
        EncodeBatch b;
        b.common = plans[j].a;
        b.jobs = 0u;
        for (uint32_t k = j; k < jobs; ++k) {
            if (done[k] || !same_launch(plans[j], plans[k])) continue;
            b.job[b.jobs++] = plans[k].a;
            done[k] = true;
        }
        // (where narrow codes go straight through the L2: see store_through)
        b.common.through = b.common.tl.n * b.jobs * b.common.qp.bits >= 120000000u ? 1u : 0u;
        const int rc = dt == NDQ_F32 ? run_encode_mode<0>(b, plans[j], bucket, s)
                                     : run_encode_mode<1>(b, plans[j], bucket, s);
        if (rc != NDQ_OK) return rc;
    }
    return NDQ_OK;
}

// What a worker writes: its steps and its code stream.
struct Written {
    uintptr_t steps, steps_end, codes, codes_end;
    bool changes_steps;      // false: the step handed over is the one it would write
};
static Written written(const EncodePlan& p)
{
    const uintptr_t steps = (uintptr_t)p.a.steps, codes = (uintptr_t)p.a.codes;
    return {steps, steps + 4u * (uintptr_t)p.a.num_buckets, codes, codes + (uintptr_t)p.a.total_bytes,
            !(p.handed && p.a.step_in == p.a.steps)};
}
static bool inside(uintptr_t x, uintptr_t begin, uintptr_t end) { return x + 4u > begin && x < end; }

// run_plans makes the max-norm passes of all its vectors first and one launch of many encoders;
// the bytes have to be those of one call after the other.  True: `later` must not share a
// run_plans with `earlier`, because one of them reads a step the other one writes (a step from a
// max-norm pass is there before every encoder) or both write the same memory.
static bool must_wait(const EncodePlan& earlier, const EncodePlan& later)
{
    const Written a = written(earlier), b = written(later);
    const uintptr_t reads_a = (uintptr_t)earlier.a.step_in, reads_b = (uintptr_t)later.a.step_in;
    if (later.handed && ((inside(reads_b, a.steps, a.steps_end) && a.changes_steps && !earlier.two_pass) ||
                         inside(reads_b, a.codes, a.codes_end)))
        return true;
    if (earlier.handed && ((inside(reads_a, b.steps, b.steps_end) && b.changes_steps) ||
                           inside(reads_a, b.codes, b.codes_end)))
        return true;
    return (b.changes_steps && a.steps < b.steps_end && b.steps < a.steps_end) ||
           (a.codes < b.codes_end && b.codes < a.codes_end) || (a.steps < b.codes_end && b.codes < a.steps_end) ||
           (b.changes_steps && a.codes < b.steps_end && b.steps < a.codes_end);
}

// one vector
static int encode_single(const ndq_encode_job& job, int dt, size_t n, float delta, uint32_t bucket, void* stream)
{
    EncodePlan p;
    const int rc = plan_encode(job, dt, n, delta, bucket, &p);
    if (rc != NDQ_OK || n == 0) return rc;
    return run_plans(&p, 1u, dt, bucket, (hipStream_t)stream);
}

static bool encode_job_from(ndq_encode_job* job, const void* g, const float* step_in, uint32_t levels, uint32_t M,
                            bool nested, float alpha, const ndq_dither* d, void* codes_out, float* steps_out)
{
    if (!d) return false;
    job->g = g;
    job->codes_out = codes_out;
    job->steps_out = steps_out;
    job->step_in = step_in;
    job->kind = nested ? NDQ_WORKER_NESTED : NDQ_WORKER_DQ;
    job->levels = levels;
    job->M = M;
    job->alpha = alpha;
    job->dither = *d;
    return true;
}

}  // namespace ndq

extern "C" {

int ndq_absmax(const void* g, int dt, size_t n, uint32_t bucket, float* kappa_out,
               void* stream)
{
    using namespace ndq;
    if (dt != NDQ_F32 && dt != NDQ_BF16) return NDQ_EINVAL;
    if (!kappa_out) return NDQ_EINVAL;
    if (n >= kMaxN) return NDQ_EUNSUPPORTED;
    if (!aligned4(kappa_out) || bucket % 64u != 0u) return NDQ_EALIGN;
    hipStream_t s = (hipStream_t)stream;
    AbsmaxBatch b;
    b.g[0] = g;
    b.kappa_bits[0] = (uint32_t*)kappa_out;
    b.levels[0] = 0u;
    b.parts[0] = nullptr;
    b.parts_bytes = 0;
    b.K = bucket ? (n + bucket - 1) / bucket : 1;
    if (n == 0) {   // one (empty) bucket: its max-norm is 0
        if (bucket != 0u) return NDQ_OK;
        return launch(fill_zero_kernel, dim3(1), dim3(256), s, b);
    }
    if (!g) return NDQ_EINVAL;
    if (!aligned16(g)) return NDQ_EALIGN;
    const uint32_t tile = dt == NDQ_F32 ? EncTile<0>::N : EncTile<1>::N;
    int rc = make_tiling(n, bucket, tile, &b.tl);
    if (rc != NDQ_OK) return rc;
    return dt == NDQ_F32 ? run_absmax<0>(b, 1u, s) : run_absmax<1>(b, 1u, s);
}

int ndq_encode_check(const ndq_encode_job* jobs, uint32_t W, int dt, size_t n, float delta, uint32_t bucket)
{
    using namespace ndq;
    if (!jobs || W < 1u || W > 1024u) return NDQ_EINVAL;
    EncodePlan plan;
    for (uint32_t w = 0; w < W; ++w) {
        if (jobs[w].kind != NDQ_WORKER_DQ && jobs[w].kind != NDQ_WORKER_NESTED) return NDQ_EINVAL;
        if (jobs[w].step_in && bucket != 0u) return NDQ_EINVAL;     // one step belongs to one bucket
        const int rc = plan_encode(jobs[w], dt, n, delta, bucket, &plan);
        if (rc != NDQ_OK) return rc;
    }
    return NDQ_OK;
}

int ndq_encode_workers(const ndq_encode_job* jobs, uint32_t W, int dt, size_t n, float delta, uint32_t bucket,
                       void* stream)
{
    using namespace ndq;
    const int rc_check = ndq_encode_check(jobs, W, dt, n, delta, bucket);
    if (rc_check != NDQ_OK) return rc_check;
    EncodePlan plans[kEncJobs];
    if (n == 0) return NDQ_OK;
    for (uint32_t w0 = 0; w0 < W;) {
        uint32_t count = 0;
        for (; w0 + count < W && count < kEncJobs; ++count) {
            plan_encode(jobs[w0 + count], dt, n, delta, bucket, &plans[count]);
            bool waits = false;
            for (uint32_t k = 0; k < count; ++k) waits = waits || must_wait(plans[k], plans[count]);
            if (waits) break;
        }
        const int rc = run_plans(plans, count, dt, bucket, (hipStream_t)stream);
        if (rc != NDQ_OK) return rc;
        w0 += count;
    }
    return NDQ_OK;
}

int ndq_dq_encode(const void* g, int dt, size_t n, float delta, uint32_t levels,
                  uint32_t bucket, const ndq_dither* d, void* codes_out, float* steps_out,
                  void* stream)
{
    ndq_encode_job job;
    if (!ndq::encode_job_from(&job, g, nullptr, levels, 0u, false, 1.0f, d, codes_out, steps_out)) return NDQ_EINVAL;
    return ndq::encode_single(job, dt, n, delta, bucket, stream);
}

int ndq_dq_encode_with_step(const void* g, int dt, size_t n, const float* step_in, uint32_t levels,
                            const ndq_dither* d, void* codes_out, float* steps_out, void* stream)
{
    ndq_encode_job job;
    if (!step_in && n != 0) return NDQ_EINVAL;
    if (!ndq::encode_job_from(&job, g, step_in, levels, 0u, false, 1.0f, d, codes_out, steps_out)) return NDQ_EINVAL;
    return ndq::encode_single(job, dt, n, 0.0f, 0u, stream);
}

int ndq_nested_encode(const void* g, int dt, size_t n, float delta, uint32_t levels,
                      uint32_t M, float alpha, uint32_t bucket, const ndq_dither* d,
                      void* codes_out, float* steps_out, void* stream)
{
    ndq_encode_job job;
    if (!ndq::encode_job_from(&job, g, nullptr, levels, M, true, alpha, d, codes_out, steps_out)) return NDQ_EINVAL;
    return ndq::encode_single(job, dt, n, delta, bucket, stream);
}

int ndq_nested_encode_with_step(const void* g, int dt, size_t n, const float* step_in, uint32_t M,
                                float alpha, const ndq_dither* d, void* codes_out, float* steps_out,
                                void* stream)
{
    ndq_encode_job job;
    if (!step_in && n != 0) return NDQ_EINVAL;
    // the number of fine levels only ever served to derive a step: any valid value will do
    if (!ndq::encode_job_from(&job, g, step_in, 2u, M, true, alpha, d, codes_out, steps_out)) return NDQ_EINVAL;
    return ndq::encode_single(job, dt, n, 0.0f, 0u, stream);
}

}  // extern "C"
