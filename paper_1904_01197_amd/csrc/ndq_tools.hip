// libndq, beyond the headline path (gfx950): entropy of an index stream, dense
// base-L stream, sigma_z^2 estimate and Thm 4's parameter helpers, size rules and
// status text.  See include/ndq.h for the contract.
#include <hip/hip_runtime.h>

#include <math.h>

#include <mutex>

#include "ndq.h"
#include "ndq_device.hpp"
#include "ndq_host.hpp"

namespace ndq {

// ---------------------------------------------------------------------------
// Histogram and entropy of an index stream (Sec. 4: the bit rate after entropy
// coding is reported through the entropy of the transmitted indices).
// Few, large workgroups in both kernels: every workgroup ends with one atomic per
// bin on the same few addresses, and those serialize.
//
// Codes of 3 to 8 bits: a thread reads units of 32 codes (= BITS consecutive
// 32-bit words, the next unit already in flight) and takes the codes out with
// shifts known at compile time.  Counting: 32 copies of the workgroup's histogram
// in LDS, a lane adding to copy (lane mod 32) -- the word index is
// code * 32 + copy, so the 32 lanes that LDS serves together always fall into 32
// different banks, whatever the distribution of the codes (index streams are
// heavily peaked); the two halves of a wave are served one after the other anyway.
// ---------------------------------------------------------------------------
constexpr uint32_t kHistThreads = 1024;
constexpr uint32_t kHistBlocks = 256;
constexpr uint32_t kHistCopies = 32;

// The call is one launch when a word holds its ticket (the entropy's eight bytes, or those of the bin that is derived) and the
// stream is not a long one of 1 or 2 bits (kSmallCleared).
// Nobody has cleared the bins (a launch of its own for that costs the call 1.5 to 2.5 us: 25.6 M codes of 4 bits
// 12.8 -> 11.0, 1 M 7.6 -> 6.1, 0.2 M of 5 bits 7.4 -> 5.8), so whoever finds the ticket without the call's tag puts it
// there, clears the bins and says so.  That is the first workgroup, which counts nothing, while the others count; a
// workgroup that wants to add and finds nothing done yet does it itself.  So one waits only for a workgroup that runs
// and waits for nobody (after kOpenPolls looks, which takes two calls that wrongly share their results, it goes on).
// Every workgroup draws a ticket, so none comes after the last one, when the tag is gone.  A workgroup that is alone
// stores its counts (0.2 M codes of 2 bits 6.8 -> 4.2 us).
//
// The workgroup that finishes last closes the histogram: it fills in a bin that was left to be derived and computes
// the entropy.  A workgroup's atomics on the histogram all come from its FIRST WAVE: that wave's fence waits for
// them before the workgroup's ticket, and no barrier would (it does not wait for
// atomics that return nothing, so another wave's could still be in flight when the ticket is
// drawn; letting every wave wait for its own takes 10.8 -> 12.0 us at 4 M 7-bit codes, this nothing).
// (A fence per thread would write
// back and invalidate the L2 sixteen times per workgroup while the others still stream through it.)
// Every thread calls last_workgroup.  The one that draws the last ticket therefore finds all counts in
// memory; it reads them with atomics of device scope, like the additions that made them.
constexpr unsigned long long kTicketBits = 0xFFFFull;       // the low bits of the word: tickets drawn (a workgroup each, and the opening one)
constexpr unsigned long long kOpening = 0x8000ull;          // ... or this, while the bins are being cleared
static_assert(kHistBlocks + 1u < kOpening, "tickets");
constexpr uint32_t kOpenPolls = 1u << 18;                   // of about a microsecond each

// What the first wave of a workgroup knows of the opening.  All functions are called by that whole wave.
struct HistogramOpening {
    unsigned long long* hist;
    unsigned long long* ticket;
    unsigned long long tag, look;
    uint32_t first_bin, nbins;
    bool open;
    __device__ __forceinline__ HistogramOpening(unsigned long long* hist_, uint32_t first_bin_, uint32_t nbins_,
                                                unsigned long long* ticket_, unsigned long long tag_)
        : hist(hist_), ticket(ticket_), tag(tag_), look(0ull), first_bin(first_bin_), nbins(nbins_), open(false) {}
    // A look between two rounds of counting: by the end it has been seen that the bins are clear.  (Looks at the end, when
    // everyone else draws tickets, queue up with those: 25.6 M codes of 4 bits 13.0 us with them alone, 11.3 so.  Codes of
    // 1 and 2 bits have few workgroups and rounds, and a look among those rounds costs more than it spares: 8.6 / 9.1.)
    __device__ __forceinline__ void glance()
    {
        if (open) return;
        look = __hip_atomic_load(ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        open = (look & ~kTicketBits) == tag && (look & kOpening) == 0ull;
    }
    // Returns when the bins are clear.
    __device__ __forceinline__ void await()
    {
#pragma unroll 1
        for (uint32_t poll = 0; !open && poll < kOpenPolls; ++poll) {
            glance();
            if ((look & ~kTicketBits) != tag) clear();
            else if (!open) __builtin_amdgcn_s_sleep(1);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");       // (the additions that follow are atomics of device scope)
    }
    __device__ __forceinline__ void clear()
    {
        const uint32_t lane = threadIdx.x & (kWave - 1u);
        int first = 0;
        if (lane == 0u)
            first = __hip_atomic_compare_exchange_strong(ticket, &look, tag | kOpening, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
        if (__builtin_amdgcn_readfirstlane(first) == 0) return;
        for (uint32_t b = first_bin + lane; b < nbins; b += kWave)
            __hip_atomic_store(hist + b, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __threadfence();             // the wave's stores, before the word says that they are done
        if (lane == 0u) __hip_atomic_store(ticket, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

__device__ __forceinline__ bool last_workgroup(unsigned long long* ticket, unsigned long long tag, uint32_t* flag)
{
    __syncthreads();
    if (threadIdx.x == 0u) {
        __threadfence();
        *flag = atomicAdd(ticket, 1ull) == tag + (unsigned long long)gridDim.x - 1ull ? 1u : 0u;
        __threadfence();
    }
    __syncthreads();
    return *flag != 0u;
}

// -sum p log2 p over at most 256 bins, binary64, fixed reduction order; called by all
// threads of one workgroup of at least 256 threads.  derive_bin0 (at most 4 bins):
// bin 0 was not counted and is what the other bins leave of n.  (In a workgroup that is alone every thread reads the bin
// that it has stored.)
__device__ __forceinline__ void close_histogram(unsigned long long* hist, uint32_t nbins, uint64_t n,
                                                double* entropy_out, bool derive_bin0, double* term,
                                                unsigned long long* few)
{
    const uint32_t tid = threadIdx.x;
    unsigned long long h = 0ull;
    if (tid < nbins && !(derive_bin0 && tid == 0u))
        h = __hip_atomic_load(hist + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (derive_bin0) {
        if (tid >= 1u && tid < nbins) few[tid] = h;
        __syncthreads();
        if (tid == 0u) {
            unsigned long long rest = n;
            for (uint32_t b = 1; b < nbins; ++b) rest -= few[b];
            hist[0] = rest;
            h = rest;
        }
    }
    if (!entropy_out) return;     // (the same for every thread)
    double t = 0.0;
    if (tid < nbins && h) {
        const double p = (double)h / (double)n;
        t = -p * log2(p);
    }
    // pairs that are 128, 64, ... 1 apart: across waves through LDS, then within the first
    t += 0.0;                     // (what absent bins add: -0 becomes 0)
    if (nbins > (uint32_t)kWave) {
        if (tid < 256u) term[tid] = t;
        __syncthreads();
        if (tid < 128u) term[tid] += term[tid + 128u];
        __syncthreads();
        if (tid < 64u) t = term[tid] + term[tid + 64u];
    }
    for (int s = 32; s >= 1; s >>= 1) t += __shfl_down(t, s, kWave);
    if (tid == 0u) entropy_out[0] = t;
}

template <int BITS>
__device__ __forceinline__ void load_unit(const uint32_t* __restrict__ words, uint64_t u, uint32_t (&w)[BITS])
{
    const uint32_t* p = words + u * BITS;
    if constexpr (BITS % 4 == 0) {      // 16-byte aligned: the stream is, and so is every unit
#pragma unroll
        for (int k = 0; k < BITS / 4; ++k) {
            const uint4 x = reinterpret_cast<const uint4*>(p)[k];
            w[4 * k] = x.x; w[4 * k + 1] = x.y; w[4 * k + 2] = x.z; w[4 * k + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < BITS; ++k) w[k] = p[k];
    }
}

// Codes of 3 and 4 bits are counted two at a time, by the value of the pair: half the LDS
// additions, which bound long streams (call of 134 M codes 29.4 -> 22.4 us, of 25.6 M 14.9 -> 14.2
// us at 4 bits, 29.5 -> 21.6 and 14.7 -> 13.6 at 3, on the full grid).  Pairs of wider codes would need 128 KB of
// LDS or more.
template <int BITS>
__global__ __launch_bounds__(kHistThreads) void histogram_kernel(const uint32_t* __restrict__ words, uint64_t n,
                                                                 unsigned long long* hist, double* entropy_out,
                                                                 unsigned long long tag)
{
    constexpr uint32_t NB = 1u << BITS;
    constexpr uint32_t MASK = NB - 1u;
    constexpr bool PAIRS = BITS <= 4;
    constexpr uint32_t SLOTS = PAIRS ? NB * NB : NB;
    constexpr int SLOT_BITS = PAIRS ? 2 * BITS : BITS;
    __shared__ uint32_t cnt[SLOTS * kHistCopies];
    __shared__ uint32_t single[NB];                 // the last n mod 32 codes
    __shared__ unsigned long long total[PAIRS || NB > kWave ? NB : 1];
    __shared__ double term[256];
    __shared__ uint32_t flag;
    const uint32_t tid = threadIdx.x;
    // the entropy's eight bytes hold the ticket until the last workgroup writes the entropy there
    unsigned long long* ticket = reinterpret_cast<unsigned long long*>(entropy_out);
    const bool alone = ticket && gridDim.x == 1u, opens = ticket && gridDim.x != 1u && blockIdx.x == 0u;
    HistogramOpening opening(hist, 0u, NB, ticket, tag);
    if (opens && tid < kWave) opening.await();
    const bool watches = ticket && !alone && !opens && __builtin_amdgcn_readfirstlane(tid / kWave) == 0u;
    for (uint32_t i = tid; i < SLOTS * kHistCopies; i += kHistThreads) cnt[i] = 0u;
    if (tid < NB) single[tid] = 0u;
    __syncthreads();

    const uint32_t copy = tid & (kHistCopies - 1u);
    const uint64_t units = n >> 5;                  // whole units; the last n mod 32 codes below
    const uint32_t first_counter = ticket && !alone ? 1u : 0u;
    const uint64_t stride = (uint64_t)(gridDim.x - first_counter) * kHistThreads;
    uint64_t u = opens ? units : (uint64_t)(blockIdx.x - first_counter) * kHistThreads + tid;
    uint32_t w[BITS], ahead[BITS];
    if (u < units) load_unit<BITS>(words, u, w);
    while (u < units) {
        const uint64_t un = u + stride;
        if (un < units) load_unit<BITS>(words, un, ahead);
#pragma unroll
        for (int j = 0; j < 32 * BITS / SLOT_BITS; ++j) {
            const int bit = j * SLOT_BITS, k = bit >> 5, sh = bit & 31;
            uint32_t slot = w[k] >> sh;
            if (sh + SLOT_BITS > 32) slot |= w[k + 1] << (32 - sh);
            atomicAdd(&cnt[(slot & (SLOTS - 1u)) * kHistCopies + copy], 1u);     // result unused: a plain LDS add
        }
#pragma unroll
        for (int k = 0; k < BITS; ++k) w[k] = ahead[k];
        if (watches) opening.glance();
        u = un;
    }
    const uint32_t rest = (uint32_t)(n & 31u);
    if (blockIdx.x == first_counter && tid < rest) {
        // one code per thread; a code that crosses into the next word is a valid code,
        // so that word lies inside the stream
        const uint64_t bit = ((units << 5) + tid) * BITS;
        const uint64_t k = bit >> 5;
        const uint32_t sh = (uint32_t)(bit & 31u);
        uint32_t code = words[k] >> sh;
        if (sh + BITS > 32u) code |= words[k + 1] << (32u - sh);
        atomicAdd(&single[code & MASK], 1u);
    }
    __syncthreads();
    if constexpr (PAIRS) {
        // a wave per code (sixteen waves, at most sixteen codes): the lanes of one half take the
        // pairs whose low code it is, those of the other half the pairs whose high code it is;
        // a lane keeps to its copy, so a half never meets in a bank.  One wave adds all totals with
        // one instruction, which reaches the bins' cache line as one request: sixteen waves adding
        // one each queue there (45 us a call against 14 at 25.6 M codes of 4 bits).
        const uint32_t code = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid & (kWave - 1u);
        if (code < NB) {
            const uint32_t first = lane < kHistCopies ? code : code * NB;
            const uint32_t step = lane < kHistCopies ? NB : 1u;
            unsigned long long sum = lane == 0u ? single[code] : 0u;
#pragma unroll
            for (uint32_t o = 0; o < NB; ++o) sum += cnt[(first + o * step) * kHistCopies + copy];
            for (int off = 32; off >= 1; off >>= 1) sum += __shfl_down(sum, off, kWave);
            if (lane == 0u) total[code] = sum;
        }
        __syncthreads();
        if (alone) {
            if (tid < NB) hist[tid] = total[tid];
        } else if (tid < kWave) {
            if (watches) opening.await();
            if (tid < NB && total[tid]) atomicAdd(hist + tid, total[tid]);
        }
    } else {
        if (watches) opening.await();
        // (64 bins or fewer: the first wave's own; more: it takes them over through LDS)
        if (tid < NB) {
            unsigned long long sum = single[tid];
            for (uint32_t c = 0; c < kHistCopies; ++c)
                sum += cnt[tid * kHistCopies + ((c + tid) & (kHistCopies - 1u))];
            if constexpr (NB > kWave) total[tid] = sum;
            else if (alone) hist[tid] = sum;
            else if (sum) atomicAdd(hist + tid, sum);
        }
        if constexpr (NB > kWave) {
            __syncthreads();
            if (tid < kWave) {
#pragma unroll
                for (uint32_t b = tid; b < NB; b += kWave)
                    if (total[b] && !alone) atomicAdd(hist + b, total[b]);
            }
            if (alone && tid < NB) hist[tid] = total[tid];
        }
    }
    if (ticket && (alone || last_workgroup(ticket, tag, &flag)))
        close_histogram(hist, NB, n, entropy_out, false, term, nullptr);
}

// 1- and 2-bit codes: a thread takes 16 bytes (128 or 64 codes) at a time, eight
// such loads in flight, and counts with population counts.  Few, large workgroups
// (at most kSmallBlocks of kSmallThreads), because every workgroup ends with one
// atomic per bin on the same few addresses and those serialize.  A thread sees at
// most n / 2^18 + 1024 codes (n < 2^40), a wave 64 times that: 32-bit counts up to
// the wave's sum, 64-bit ones across waves.
constexpr uint32_t kSmallBlocks = 256;
static_assert(kSmallBlocks < kOpening, "tickets");
// Counting workgroups from which a launch of its own clears the bins: the workgroups of a stream this long all end at once, and
// their looks at the ticket's word then queue up with the additions and tickets on the same line (and have no rounds to go
// between).  us cleared by a launch / by the first workgroup, 2-bit codes, 60, 80, 100, 130, 160, 300 and 1500 M (115, 153, 191, 248,
// 256 workgroups): 11.1/10.8 12.8/12.6 14.1/14.5 17.4/20.1 18.0/24.1 22.7/28.1 76.4/78.5; 1-bit codes, 130, 160, 200 and 300 M (124,
// 153, 191, 256): 10.9/10.4 12.4/12.4 13.8/14.6 17.8/21.4.
constexpr uint32_t kSmallCleared = 160;
constexpr uint32_t kSmallThreads = 1024;
constexpr int kSmallInFlight = 8;

template <int BITS>
__device__ __forceinline__ void count_small(uint32_t w, uint32_t& c1, uint32_t& c2, uint32_t& c3)
{
    if (BITS == 1) {
        c1 += __builtin_popcount(w);
    } else {
        const uint32_t lo = w & 0x55555555u, hi = (w >> 1) & 0x55555555u;
        c1 += __builtin_popcount(lo & ~hi);
        c2 += __builtin_popcount(hi & ~lo);
        c3 += __builtin_popcount(lo & hi);
    }
}

template <int BITS>
__device__ __forceinline__ void count_small(const uint4& x, uint32_t& c1, uint32_t& c2, uint32_t& c3)
{
    count_small<BITS>(x.x, c1, c2, c3); count_small<BITS>(x.y, c1, c2, c3);
    count_small<BITS>(x.z, c1, c2, c3); count_small<BITS>(x.w, c1, c2, c3);
}

// (the code width is a template parameter: as a run-time value it put a branch around every
// word's counting, and the loop then waited for all its loads before the first count)
template <int BITS>
__global__ __launch_bounds__(kSmallThreads) void histogram_small_kernel(const uint4* __restrict__ vec, uint64_t n,
                                                                        unsigned long long* hist,
                                                                        double* entropy_out, unsigned long long tag)
{
    constexpr uint32_t bits = BITS;
    __shared__ uint32_t part[3][kSmallThreads / 64];
    __shared__ double term[256];
    __shared__ unsigned long long few[4];
    __shared__ uint32_t flag;
    const uint32_t tid = threadIdx.x;
    // bins 1..3 (or bin 1) are counted; bin 0 is not: its eight bytes hold the
    // ticket, and the last workgroup writes there what the other bins leave of n
    // (no tag: the bins have been cleared by a launch of its own, and tickets count from 0)
    constexpr uint32_t nbins = 1u << BITS;
    const bool alone = gridDim.x == 1u, cleared = tag == 0ull, opens = !alone && !cleared && blockIdx.x == 0u;
    HistogramOpening opening(hist, 1u, nbins, hist, tag);
    if (opens && tid < kWave) opening.await();
    const bool watches = !alone && !cleared && !opens && __builtin_amdgcn_readfirstlane(tid / kWave) == 0u;
    // whole 16-byte vectors here; the last, partial one (the stream is allocated in
    // multiples of 16 bytes) is masked to its valid bits below.  Bits masked away
    // read as code 0, and bin 0 is n minus the other bins anyway.
    const uint64_t vectors = (n * bits) >> 7;
    const uint32_t first_counter = alone || cleared ? 0u : 1u;
    const uint64_t stride = (uint64_t)(gridDim.x - first_counter) * kSmallThreads;
    uint32_t c[3] = {0u, 0u, 0u};
    uint64_t u = opens ? vectors : (uint64_t)(blockIdx.x - first_counter) * kSmallThreads + tid;
    for (; u + (kSmallInFlight - 1) * stride < vectors; u += kSmallInFlight * stride) {
        uint4 x[kSmallInFlight];
#pragma unroll
        for (int j = 0; j < kSmallInFlight; ++j) x[j] = vec[u + (uint64_t)j * stride];
#pragma unroll
        for (int j = 0; j < kSmallInFlight; ++j) count_small<BITS>(x[j], c[0], c[1], c[2]);
    }
    for (; u < vectors; u += stride) count_small<BITS>(vec[u], c[0], c[1], c[2]);
    const uint32_t tail_bits = (uint32_t)((n * bits) & 127u);
    if (blockIdx.x == first_counter && tid == 0 && tail_bits != 0u) {
        const uint4 x = vec[vectors];
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (uint32_t j = 0; j < 4u; ++j) {
            const uint32_t have = tail_bits > 32u * j ? tail_bits - 32u * j : 0u;
            const uint32_t mask = have >= 32u ? 0xffffffffu : ((1u << have) - 1u);
            count_small<BITS>(w[j] & mask, c[0], c[1], c[2]);
        }
    }
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        for (int off = 32; off >= 1; off >>= 1) c[b] += __shfl_down(c[b], off, 64);
        if ((tid & 63u) == 0u) part[b][tid >> 6] = c[b];
    }
    __syncthreads();
    if (watches) opening.await();
    if (tid >= 1u && tid < nbins) {
        unsigned long long sum = 0u;
        for (uint32_t w = 0; w < kSmallThreads / 64u; ++w) sum += part[tid - 1u][w];
        if (alone) hist[tid] = sum;
        else if (sum) atomicAdd(hist + tid, sum);
    }
    if (alone || last_workgroup(hist, tag, &flag)) close_histogram(hist, nbins, n, entropy_out, true, term, few);
}

// For what nobody holds a ticket of, and long streams: clears the bins and, when an entropy is wanted, its eight bytes (+0.0: the
// entropy of an empty stream).
__global__ void clear_histogram_kernel(unsigned long long* hist, uint32_t nbins, unsigned long long* entropy_bits)
{
    if (threadIdx.x < nbins) hist[threadIdx.x] = 0ull;
    if (threadIdx.x == 0u && entropy_bits) entropy_bits[0] = 0ull;
}

// ---------------------------------------------------------------------------
// Dense base-L stream (Sec. 4 Table 1 counts log2 L bits per index): K indices
// per 32-bit word as the number sum_j c_j L^j.  Transcoders between the
// fixed-width stream and the dense one.  A thread owns P dense words = P K
// indices = TB = P K BITS / 8 whole bytes of the fixed-width stream, so no two threads
// share a byte; they sit in its registers as one bit string with every index at a place known
// at compile time.  Both streams move between memory and LDS sixteen bytes at a time.
//
// Bound by the digits' arithmetic: a digit at a time is a multiply and a shift or two for each of K, so D
// digits are taken together, through a table of their 2^(D BITS) codes (packing) or L^D values
// (unpacking) that the workgroup makes first: K / D multiplications or divisions a word.  Four words a
// thread where that is a whole number of 32-bit words (more waves for the same stream), else eight.
// us, packing + unpacking, before (a digit at a time; other L than 3 and 5 byte by byte, with eight words a
// thread) and now: 25.6 M indices of three levels 4.8 + 6.3, 4.1 + 4.3; five 5.2 + 7.3, 5.2 + 6.7; six 12.8 + 15.9,
// 5.9 + 6.7; 1.5 M of twelve 7.3 + 7.4, 3.1 + 3.1.  (Packing three levels by the table: 4.5.)
// ---------------------------------------------------------------------------
struct DenseArgs {
    unsigned char* fixed;     // fixed-width stream (read by pack, written by unpack)
    uint32_t* dense;          // dense stream (written by pack, read by unpack)
    uint64_t n;               // indices
    uint64_t fixed_total;     // its padded size
    uint64_t dense_total;     // padded size in words
    uint32_t levels;
    uint32_t group;           // levels^D
    // division of a 32-bit number by `group` through one high multiply (division by
    // an invariant integer, round-up method): with l = ceil(log2 group) and
    // magic = floor(2^32 (2^l - group) / group) + 1, for every 32-bit x
    // x / group = (t + ((x - t) >> 1)) >> (l - 1), t = high word of x * magic
    uint32_t magic, shift;
};

constexpr uint32_t kDenseBlock = 256;

// LC: the number of levels when it is known at compile time (the level counts of the paper's own
// experiments, three and five), else 0.
template <uint32_t LC, uint32_t K, uint32_t BITS> struct DenseForm {
    static constexpr uint32_t D = BITS == 1u ? 8u : BITS == 2u ? (K == 20u ? 5u : 4u) : BITS == 3u ? 3u : BITS <= 5u ? 2u : 1u;
    static constexpr uint32_t G = K / D, R = K % D;                 // whole groups of digits, and digits left over
    static constexpr uint32_t PACK_D = LC ? 1u : D;                 // (packing: by a constant L a digit is a shift and an addition)
    static constexpr uint32_t P = K * BITS % 8u == 0u ? 4u : 8u;    // dense words per thread
    static constexpr uint32_t TB = P * K * BITS / 8u;               // a thread's bytes of the fixed-width stream
    static constexpr uint32_t NX = (TB + 3u) / 4u;                  // as 32-bit words
    static constexpr uint32_t NR = TB % 4u == 0u ? NX : TB / 4u + 2u;   // aligned words that cover them at any offset
    static constexpr uint32_t FIXED_WORDS = kDenseBlock * TB / 4u;  // per workgroup (256 * TB is a multiple of 16)
    static constexpr uint32_t DENSE_WORDS = kDenseBlock * P;
    static constexpr uint32_t CODES = 1u << (D * BITS);             // entries of either table: L^D <= CODES
    static constexpr uint32_t power(uint32_t e) { return e == 0u ? 1u : LC * power(e - 1u); }
    static_assert(P * K * BITS % 8u == 0u && FIXED_WORDS % 4u == 0u && CODES <= 1024u, "partition");
    static __device__ __forceinline__ uint32_t group(const DenseArgs& a) { return LC ? power(D) : a.group; }
    static __device__ __forceinline__ uint32_t divide(uint32_t x, const DenseArgs& a)
    {
        if (LC) return x / power(D);
        const uint32_t t = __umulhi(x, a.magic);
        return (t + ((x - t) >> 1)) >> a.shift;
    }
};

// bytes of the fixed-width stream that belong to this workgroup (a multiple of 16, like its first byte
// and the stream's size)
template <uint32_t TB>
__device__ __forceinline__ uint32_t dense_block_bytes(const DenseArgs& a, uint64_t block_byte0)
{
    constexpr uint64_t share = (uint64_t)kDenseBlock * TB;
    if (block_byte0 >= a.fixed_total) return 0u;
    const uint64_t left = a.fixed_total - block_byte0;
    return (uint32_t)(left < share ? left : share);
}

// keeps the first `valid_bits` bits of a bit string held in NX words
template <uint32_t NX>
__device__ __forceinline__ void keep_bits(uint32_t (&x)[NX], uint32_t valid_bits)
{
#pragma unroll
    for (uint32_t i = 0; i < NX; ++i) {
        const uint32_t have = valid_bits > 32u * i ? valid_bits - 32u * i : 0u;
        x[i] &= have >= 32u ? 0xffffffffu : ((1u << have) - 1u);
    }
}

// bits of the thread's share that belong to indices below n
template <uint32_t K, uint32_t BITS, uint32_t P>
__device__ __forceinline__ uint32_t dense_valid_bits(const DenseArgs& a, uint64_t first_word)
{
    const uint64_t first = first_word * K;
    if (first >= a.n) return 0u;
    const uint64_t left = a.n - first;
    return left >= P * K ? P * K * BITS : (uint32_t)left * BITS;
}

// the `width` <= 10 bits from `bit` on
template <uint32_t NX>
__device__ __forceinline__ uint32_t window_of(const uint32_t (&x)[NX], uint32_t bit, uint32_t width)
{
    const uint32_t k = bit >> 5, sh = bit & 31u;
    uint32_t c = x[k] >> sh;
    if (sh + width > 32u) c |= x[k + 1] << (32u - sh);
    return c & ((1u << width) - 1u);
}

template <uint32_t LC, uint32_t K, uint32_t BITS>
__global__ __launch_bounds__(kDenseBlock) void dense_pack_kernel(DenseArgs a)
{
    using F = DenseForm<LC, K, BITS>;
    constexpr uint32_t D = F::PACK_D, G = K / D, R = K % D, CODES = 1u << (D * BITS);
    __shared__ __align__(16) uint32_t fixed_stage[F::FIXED_WORDS], dense_stage[F::DENSE_WORDS];
    __shared__ uint16_t value_of[D > 1u ? CODES : 1u];
    const uint32_t tid = threadIdx.x;
    const uint64_t block_byte0 = (uint64_t)blockIdx.x * kDenseBlock * F::TB;
    const uint64_t block_w0 = (uint64_t)blockIdx.x * F::DENSE_WORDS;
    const uint32_t vectors_in = dense_block_bytes<F::TB>(a, block_byte0) / 16u;
    const uint4* fixed128 = reinterpret_cast<const uint4*>(a.fixed + block_byte0);
    uint4* stage128 = reinterpret_cast<uint4*>(fixed_stage);
    for (uint32_t i = tid; i < F::FIXED_WORDS / 4u; i += kDenseBlock)
        stage128[i] = i < vectors_in ? fixed128[i] : make_uint4(0u, 0u, 0u, 0u);
    if constexpr (D > 1u) {
        const uint32_t L = LC ? LC : a.levels;
        for (uint32_t e = tid; e < CODES; e += kDenseBlock) {
            uint32_t v = 0u;
#pragma unroll
            for (int d = (int)D - 1; d >= 0; --d) v = v * L + ((e >> (d * BITS)) & ((1u << BITS) - 1u));
            value_of[e] = (uint16_t)v;      // (an index that is not below L counts like any other)
        }
    }
    __syncthreads();

    // the thread's TB bytes, from the aligned words around them
    const uint32_t byte0 = tid * F::TB;
    uint32_t r[F::NR], x[F::NX];
#pragma unroll
    for (uint32_t i = 0; i < F::NR; ++i) {
        const uint32_t w = byte0 / 4u + i;
        r[i] = F::TB % 4u == 0u || w < F::FIXED_WORDS ? fixed_stage[w] : 0u;
    }
    if constexpr (F::TB % 4u == 0u) {
#pragma unroll
        for (uint32_t i = 0; i < F::NX; ++i) x[i] = r[i];
    } else {
#pragma unroll
        for (uint32_t i = 0; i < F::NX; ++i) x[i] = __builtin_amdgcn_alignbyte(r[i + 1], r[i], byte0 & 3u);
    }
    // indices at or beyond n count as digit 0, whatever the padding holds
    keep_bits<F::NX>(x, dense_valid_bits<K, BITS, F::P>(a, block_w0 + (uint64_t)tid * F::P));

    const uint32_t group = LC ? F::power(D) : a.group;
    uint32_t value[F::P];
#pragma unroll
    for (uint32_t j = 0; j < F::P; ++j) {
        uint32_t v = 0u;
        if (R != 0u) {
            const uint32_t c = window_of<F::NX>(x, (j * K + G * D) * BITS, R * BITS);
            v = D > 1u ? value_of[c] : c;
        }
#pragma unroll
        for (int g = (int)G - 1; g >= 0; --g) {        // highest digits first
            const uint32_t c = window_of<F::NX>(x, (j * K + (uint32_t)g * D) * BITS, D * BITS);
            v = v * group + (D > 1u ? value_of[c] : c);
        }
        value[j] = v;
    }
    uint4* mine = reinterpret_cast<uint4*>(dense_stage + tid * F::P);
#pragma unroll
    for (uint32_t j = 0; j < F::P; j += 4u) mine[j / 4u] = make_uint4(value[j], value[j + 1u], value[j + 2u], value[j + 3u]);
    __syncthreads();
    const uint4* out128 = reinterpret_cast<const uint4*>(dense_stage);
    uint4* dense128 = reinterpret_cast<uint4*>(a.dense + block_w0);
    for (uint32_t i = tid; i < F::DENSE_WORDS / 4u; i += kDenseBlock)
        if (block_w0 + 4u * i < a.dense_total) dense128[i] = out128[i];      // dense_total is a multiple of 4
}

template <uint32_t LC, uint32_t K, uint32_t BITS>
__global__ __launch_bounds__(kDenseBlock) void dense_unpack_kernel(DenseArgs a)
{
    using F = DenseForm<LC, K, BITS>;
    __shared__ __align__(16) uint32_t fixed_stage[F::FIXED_WORDS], dense_stage[F::DENSE_WORDS];
    __shared__ uint16_t codes_of[F::D > 1u ? F::CODES : 1u];
    const uint32_t tid = threadIdx.x;
    const uint64_t block_byte0 = (uint64_t)blockIdx.x * kDenseBlock * F::TB;
    const uint64_t block_w0 = (uint64_t)blockIdx.x * F::DENSE_WORDS;
    const uint4* dense128 = reinterpret_cast<const uint4*>(a.dense + block_w0);
    uint4* in128 = reinterpret_cast<uint4*>(dense_stage);
    for (uint32_t i = tid; i < F::DENSE_WORDS / 4u; i += kDenseBlock)
        in128[i] = block_w0 + 4u * i < a.dense_total ? dense128[i] : make_uint4(0u, 0u, 0u, 0u);
    const uint32_t group = F::group(a);
    if constexpr (F::D > 1u) {
        // the codes of every value below L^D, written by the thread that has the codes: no division
        const uint32_t L = LC ? LC : a.levels;
        for (uint32_t e = tid; e < F::CODES; e += kDenseBlock) {
            uint32_t v = 0u;
            bool below = true;
#pragma unroll
            for (int d = (int)F::D - 1; d >= 0; --d) {
                const uint32_t c = (e >> (d * BITS)) & ((1u << BITS) - 1u);
                below = below && c < L;
                v = v * L + c;
            }
            if (below) codes_of[v] = (uint16_t)e;
        }
    }
    __syncthreads();

    uint32_t value[F::P], x[F::NX];
    const uint4* mine = reinterpret_cast<const uint4*>(dense_stage + tid * F::P);
#pragma unroll
    for (uint32_t j = 0; j < F::P; j += 4u) {
        const uint4 w = mine[j / 4u];
        value[j] = w.x; value[j + 1u] = w.y; value[j + 2u] = w.z; value[j + 3u] = w.w;
    }
#pragma unroll
    for (uint32_t i = 0; i < F::NX; ++i) x[i] = 0u;
    auto put = [&](uint32_t bit, uint32_t width, uint32_t c) __attribute__((always_inline)) {
        const uint32_t k = bit >> 5, sh = bit & 31u;
        x[k] |= c << sh;
        if (sh + width > 32u) x[k + 1] |= c >> (32u - sh);
    };
#pragma unroll
    for (uint32_t j = 0; j < F::P; ++j) {
        uint32_t v = value[j];
#pragma unroll
        for (uint32_t g = 0; g < F::G + (F::R != 0u ? 1u : 0u); ++g) {
            const uint32_t q = F::divide(v, a), rest = v - q * group;       // below L^D whatever the word holds
            uint32_t c = F::D > 1u ? codes_of[rest] : rest;
            const uint32_t digits = g < F::G ? F::D : F::R;
            if (g == F::G) c &= (1u << (F::R * BITS)) - 1u;
            put((j * K + g * F::D) * BITS, digits * BITS, c);
            v = q;
        }
    }
    keep_bits<F::NX>(x, dense_valid_bits<K, BITS, F::P>(a, block_w0 + (uint64_t)tid * F::P));

    const uint32_t byte0 = tid * F::TB;
    if constexpr (F::TB % 4u == 0u) {
#pragma unroll
        for (uint32_t i = 0; i < F::NX; ++i) fixed_stage[byte0 / 4u + i] = x[i];
    } else {
        unsigned char* bytes = reinterpret_cast<unsigned char*>(fixed_stage) + byte0;
#pragma unroll
        for (uint32_t i = 0; i < F::TB; ++i) bytes[i] = (unsigned char)(x[i / 4u] >> (8u * (i & 3u)));
    }
    __syncthreads();
    const uint32_t vectors_out = dense_block_bytes<F::TB>(a, block_byte0) / 16u;
    const uint4* stage128 = reinterpret_cast<const uint4*>(fixed_stage);
    uint4* fixed128 = reinterpret_cast<uint4*>(a.fixed + block_byte0);
    for (uint32_t i = tid; i < vectors_out; i += kDenseBlock) fixed128[i] = stage128[i];
}

// Launches the transcoder whose level count, or digits per word and code width, are those of the call.
template <uint32_t LC, uint32_t K, uint32_t BITS>
static int launch_dense(DenseArgs& a, bool pack, hipStream_t s)
{
    using F = DenseForm<LC, K, BITS>;
    a.group = 1u;
    for (uint32_t d = 0; d < F::D; ++d) a.group *= a.levels;
    uint32_t log2 = 0u;
    while ((1u << log2) < a.group) ++log2;
    a.magic = (uint32_t)((((uint64_t)1 << 32) * (((uint64_t)1 << log2) - a.group)) / a.group + 1u);
    a.shift = log2 - 1u;                        // group >= 2
    const uint64_t blocks = pack ? (a.dense_total + F::DENSE_WORDS - 1u) / F::DENSE_WORDS
                                 : (a.fixed_total + 4u * F::FIXED_WORDS - 1u) / (4u * F::FIXED_WORDS);
    if (blocks >= ((uint64_t)1 << 31)) return NDQ_EUNSUPPORTED;
    const dim3 grid((uint32_t)blocks), block(kDenseBlock);
    return pack ? launch((dense_pack_kernel<LC, K, BITS>), grid, block, s, a)
                : launch((dense_unpack_kernel<LC, K, BITS>), grid, block, s, a);
}

// every (digits per word, code width) that a level count from 2 to 256 has
static int run_dense(DenseArgs& a, uint32_t k, uint32_t bits, bool pack, hipStream_t s)
{
    if (a.levels == 3u) return launch_dense<3, 20, 2>(a, pack, s);
    if (a.levels == 5u) return launch_dense<5, 13, 3>(a, pack, s);
    switch (16u * k + bits) {
    case 16u * 32u + 1u: return launch_dense<0, 32, 1>(a, pack, s);
    case 16u * 16u + 2u: return launch_dense<0, 16, 2>(a, pack, s);
    case 16u * 12u + 3u: return launch_dense<0, 12, 3>(a, pack, s);
    case 16u * 11u + 3u: return launch_dense<0, 11, 3>(a, pack, s);
    case 16u * 10u + 3u: return launch_dense<0, 10, 3>(a, pack, s);
    case 16u * 10u + 4u: return launch_dense<0, 10, 4>(a, pack, s);
    case 16u * 9u + 4u: return launch_dense<0, 9, 4>(a, pack, s);
    case 16u * 8u + 4u: return launch_dense<0, 8, 4>(a, pack, s);
    case 16u * 7u + 5u: return launch_dense<0, 7, 5>(a, pack, s);
    case 16u * 6u + 5u: return launch_dense<0, 6, 5>(a, pack, s);
    case 16u * 6u + 6u: return launch_dense<0, 6, 6>(a, pack, s);
    case 16u * 5u + 6u: return launch_dense<0, 5, 6>(a, pack, s);
    case 16u * 5u + 7u: return launch_dense<0, 5, 7>(a, pack, s);
    case 16u * 4u + 7u: return launch_dense<0, 4, 7>(a, pack, s);
    case 16u * 4u + 8u: return launch_dense<0, 4, 8>(a, pack, s);
    default: return NDQ_EUNSUPPORTED;      // cannot happen
    }
}

// ---------------------------------------------------------------------------
// sum_i (a_i - b_i)^2 in binary64 (the sigma_z^2 estimate behind Thm 4's parameter
// choice).  A fixed grid and fixed orders of adding, so that the result does not depend on scheduling.
//
// One launch: every workgroup leaves its sum in a slot of the workspace and the last one of the grid collects
// them (with a launch of its own for that, replayed from a graph, 11 M elements take 17.5 us, so 16.7; 0.1 M 4.4 and 4.2).
// Nobody has cleared the workspace, so a slot says by itself whether it is filled: two words, each half of the
// sum beside half of the call's tag.  The other workgroups wait for nothing, so the collector's wait ends; a slot that
// has not come after kSqPolls looks (two calls that wrongly share a workspace, a workgroup that is kept from running) it works
// out by itself.  A call replayed from a graph has the same tag, so no slot is left filled: the collector empties what it has seen and
// marks the words it gave up on as closed, and whoever comes to a word second, the collector or its workgroup, empties it.
// ---------------------------------------------------------------------------
constexpr uint32_t kSqBlocks = 512;
constexpr uint32_t kSqThreads = 512;
constexpr uint32_t kSqPolls = 1u << 18;          // of about a microsecond each
static_assert(kSqBlocks == kSqThreads, "a thread of the collector per slot");

struct SqSlot { uint64_t word[2]; };

// Workgroup `block`'s slot.  `skip`, one more than are needed, is left out: the one a result inside the workspace lies in.
__device__ __forceinline__ SqSlot* slot_of(SqSlot* slots, uint32_t block, uint32_t skip) { return slots + block + (block >= skip ? 1u : 0u); }

// what a word with this half of the tag holds once the collector has given it up
__device__ __forceinline__ uint64_t closed_word(uint32_t half) { return (uint64_t)~half << 32 | (uint32_t)~half; }

// the workgroup's sum, in its first thread
__device__ __forceinline__ double block_sum(double x, double* sh)
{
    const uint32_t tid = threadIdx.x;
    __syncthreads();                             // (sh may still be read from the time before)
    sh[tid] = x;
    __syncthreads();
    for (uint32_t s = kSqThreads / 2u; s >= 1; s >>= 1) {
        if (tid < s) sh[tid] += sh[tid + s];
        __syncthreads();
    }
    return sh[0];
}

// the sum of workgroup `block` of the grid, called by all threads of a workgroup
__device__ __forceinline__ double sqdiff_share(const float* __restrict__ a, const float* __restrict__ b, uint64_t n,
                                               uint32_t block, double* sh)
{
    const uint64_t n4 = n >> 2;
    double acc = 0.0;
    for (uint64_t i = (uint64_t)block * kSqThreads + threadIdx.x; i < n4; i += (uint64_t)kSqBlocks * kSqThreads) {
        const float4 x = ((const float4*)a)[i], y = ((const float4*)b)[i];
        const double d0 = (double)x.x - (double)y.x, d1 = (double)x.y - (double)y.y;
        const double d2 = (double)x.z - (double)y.z, d3 = (double)x.w - (double)y.w;
        acc += d0 * d0; acc += d1 * d1; acc += d2 * d2; acc += d3 * d3;
    }
    if (block == 0u && threadIdx.x < (n & 3u)) {       // the last n mod 4 elements
        const uint64_t i = (n4 << 2) + threadIdx.x;
        const double d = (double)a[i] - (double)b[i];
        acc += d * d;
    }
    return block_sum(acc, sh);
}

__global__ __launch_bounds__(kSqThreads) void sqdiff_kernel(const float* __restrict__ a, const float* __restrict__ b,
                                                            uint64_t n, SqSlot* slots, uint32_t skip, uint64_t tag,
                                                            uint32_t polls, double* out)
{
    __shared__ double sh[kSqThreads];
    __shared__ uint32_t missing[kSqBlocks];
    const uint32_t tid = threadIdx.x;
    const uint32_t half[2] = {(uint32_t)tag, (uint32_t)(tag >> 32)};
    const double total = sqdiff_share(a, b, n, blockIdx.x, sh);
    if (blockIdx.x != kSqBlocks - 1u) {
        if (tid == 0u) {
            const uint64_t bits = (uint64_t)__double_as_longlong(total);
            const uint64_t filled[2] = {bits >> 32 << 32 | half[0], bits << 32 | half[1]};
            uint64_t* word = slot_of(slots, blockIdx.x, skip)->word;
            const uint64_t before[2] = {exchange_through(&word[0], filled[0]), exchange_through(&word[1], filled[1])};
#pragma unroll
            for (int w = 0; w < 2; ++w)
                if (before[w] == closed_word(half[w])) store_through(&word[w], 0u);
        }
        return;
    }
    double mine = total;                         // (its own sum has no slot to go through)
    const bool own = tid == kSqBlocks - 1u;
    bool have = own;
    uint64_t* word = slot_of(slots, own ? 0u : tid, skip)->word;
    for (uint32_t poll = 0; !have && poll < polls; ++poll) {
        const uint64_t w0 = load_through(&word[0]), w1 = load_through(&word[1]);
        have = (uint32_t)w0 == half[0] && (uint32_t)w1 == half[1];
        if (have) mine = __longlong_as_double((long long)(w0 >> 32 << 32 | w1 >> 32));
        else __builtin_amdgcn_s_sleep(1);
    }
    missing[tid] = have ? 0u : 1u;
    if (!own) {
#pragma unroll
        for (int w = 0; w < 2; ++w)
            if (have || (uint32_t)exchange_through(&word[w], closed_word(half[w])) == half[w]) store_through(&word[w], 0u);
    }
    if (__syncthreads_count(have ? 0 : 1) != 0)
        for (uint32_t block = 0; block < kSqBlocks; ++block) {
            if (missing[block] == 0u) continue;
            const double share = sqdiff_share(a, b, n, block, sh);
            if (tid == block) mine = share;
        }
    const double sum = block_sum(mine, sh);
    if (tid == 0u) out[0] = sum;
}

// Slots of ndq_sqdiff_static: one per workgroup, in
// memory the library owns (8 KB on every GPU it runs on, until the process ends).
// In host code this name is only a handle for hipGetSymbolAddress; the kernels get
// the per-device address kept in g_scratch_ptr.
static __device__ __align__(256) SqSlot scratch[kSqBlocks];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static SqSlot* g_scratch_ptr[kMaxDevices];   // address of `scratch` on each device, looked up once

// Address of `scratch` on the current device (null: the runtime refused).
static SqSlot* scratch_on_current_device()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        g_scratch_ptr[dev] = (SqSlot*)p;
    }
    return g_scratch_ptr[dev];
}

// Looks at a slot before the collector works it out.  NDQ_COLLECT_POLLS, read once per process, sets it, so that
// tests can make the collector do all of them (0).
static uint32_t collector_polls()
{
    static const uint32_t polls = [] {
        const char* e = getenv("NDQ_COLLECT_POLLS");
        return e ? (uint32_t)strtoul(e, nullptr, 10) : kSqPolls;
    }();
    return polls;
}

// Argument checks and the launch shared by ndq_sqdiff and ndq_sqdiff_static.
static int sqdiff_common(const float* a, const float* b, size_t n, SqSlot* slots, double* out, void* stream)
{
    if (!out) return NDQ_EINVAL;
    if (n != 0 && (!a || !b)) return NDQ_EINVAL;
    if (n >= kMaxN) return NDQ_EUNSUPPORTED;
    if (((uintptr_t)slots & 7u) || ((uintptr_t)out & 7u)) return NDQ_EALIGN;
    if (n != 0 && (!aligned16(a) || !aligned16(b))) return NDQ_EALIGN;
    // a result may lie inside the workspace
    const uintptr_t inside = (uintptr_t)out - (uintptr_t)slots;
    const uint32_t skip = inside < kSqBlocks * sizeof(SqSlot) ? (uint32_t)(inside / sizeof(SqSlot)) : kSqBlocks - 1u;
    // (an emptied slot holds no tag: neither half is 0)
    return launch(sqdiff_kernel, dim3(kSqBlocks), dim3(kSqThreads), (hipStream_t)stream, a, b, (uint64_t)n, slots, skip,
                  call_tag() | 0x100000001u, collector_polls(), out);
}

}  // namespace ndq

extern "C" {

uint32_t ndq_code_bits(uint32_t levels_or_M) { return ndq::code_bits(levels_or_M); }

size_t ndq_packed_bytes(size_t n, uint32_t bits) { return ndq::packed_bytes(n, bits); }

size_t ndq_num_buckets(size_t n, uint32_t bucket)
{
    return bucket ? (n + bucket - 1u) / bucket : 1u;
}

int ndq_code_entropy(const void* codes, size_t n, uint32_t bits, uint64_t* hist_out,
                     double* entropy_out, void* stream)
{
    using namespace ndq;
    if (bits < 1u || bits > 8u || !hist_out) return NDQ_EINVAL;
    if (n >= kMaxN) return NDQ_EUNSUPPORTED;
    if (((uintptr_t)hist_out & 7u) != 0u || ((uintptr_t)entropy_out & 7u) != 0u) return NDQ_EALIGN;
    if (n != 0 && !codes) return NDQ_EINVAL;
    if (n != 0 && !aligned16(codes)) return NDQ_EALIGN;
    hipStream_t s = (hipStream_t)stream;
    const uint32_t nbins = 1u << bits;
    // a ticket's word: bin 0 of a narrow stream, else the entropy's; a count is below 2^40 and an entropy not negative, so
    // neither is taken for a tag
    const bool ticket = n != 0u && (bits <= 2u || entropy_out);
    const unsigned long long tag = (call_tag() | (uint64_t)1 << 63) & ~kTicketBits;
    if (!ticket && launch(clear_histogram_kernel, dim3(1), dim3(256), s, (unsigned long long*)hist_out, nbins,
                          (unsigned long long*)entropy_out) != NDQ_OK)
        return NDQ_ELAUNCH;
    if (n == 0) return NDQ_OK;
    if (bits <= 2u) {
        const uint64_t vectors = ((uint64_t)n * bits) >> 7;
        uint64_t blocks = (vectors + kSmallInFlight * kSmallThreads - 1) / (kSmallInFlight * kSmallThreads);
        if (blocks > kSmallBlocks) blocks = kSmallBlocks;
        if (blocks == 0u) blocks = 1u;
        const bool cleared = blocks >= kSmallCleared;
        if (cleared && launch(clear_histogram_kernel, dim3(1), dim3(256), s, (unsigned long long*)hist_out, nbins,
                              (unsigned long long*)nullptr) != NDQ_OK)
            return NDQ_ELAUNCH;
        if (blocks > 1u && !cleared) ++blocks;           // and the one that opens the histogram
        return launch(bits == 1u ? histogram_small_kernel<1> : histogram_small_kernel<2>, dim3((uint32_t)blocks), dim3(kSmallThreads),
                      s, (const uint4*)codes, (uint64_t)n, (unsigned long long*)hist_out, entropy_out, cleared ? 0ull : tag);
    }
    const uint64_t units = (uint64_t)n >> 5;
    uint64_t blocks = (units + kHistThreads - 1) / kHistThreads;
    if (blocks < (uint64_t)kHistBlocks * kHistBlocks) {
        // A workgroup's closing atomics cost the call 25 ns, a round of units about
        // 0.6 us, so 0.025 B + 0.6 blocks / B is smallest at B = sqrt(24 blocks).  Against the full grid:
        // 4-bit calls of 4 M codes 9.3 -> 8.2 us, 25.6 M 14.2 -> 12.1, 134 M 22.4 both; 5-bit ones of 4 M 9.8 -> 8.0,
        // 25.6 M 16.0 -> 14.1; 8-bit 10.4 -> 8.9, 17.0 -> 15.3, 100 M 28.1 both.
        uint64_t fewer = (uint64_t)sqrt(24.0 * (double)blocks);
        if (fewer < blocks) blocks = fewer;
    }
    if (blocks > kHistBlocks) blocks = kHistBlocks;
    if (blocks == 0u) blocks = 1u;
    if (ticket && blocks > 1u) ++blocks;     // and the one that opens the histogram
    const dim3 grid((uint32_t)blocks), block(kHistThreads);
    const uint32_t* words = (const uint32_t*)codes;
    unsigned long long* h = (unsigned long long*)hist_out;
    switch (bits) {
    case 3: return launch(histogram_kernel<3>, grid, block, s, words, (uint64_t)n, h, entropy_out, tag);
    case 4: return launch(histogram_kernel<4>, grid, block, s, words, (uint64_t)n, h, entropy_out, tag);
    case 5: return launch(histogram_kernel<5>, grid, block, s, words, (uint64_t)n, h, entropy_out, tag);
    case 6: return launch(histogram_kernel<6>, grid, block, s, words, (uint64_t)n, h, entropy_out, tag);
    case 7: return launch(histogram_kernel<7>, grid, block, s, words, (uint64_t)n, h, entropy_out, tag);
    default: return launch(histogram_kernel<8>, grid, block, s, words, (uint64_t)n, h, entropy_out, tag);
    }
}

uint32_t ndq_dense_group(uint32_t levels)
{
    if (levels < 2u || levels > 256u) return 0u;
    uint32_t k = 0u;
    uint64_t power = 1u;
    while (power * levels <= ((uint64_t)1 << 32)) { power *= levels; ++k; }
    return k;
}

size_t ndq_dense_bytes(size_t n, uint32_t levels)
{
    const uint32_t k = ndq_dense_group(levels);
    if (!k) return 0u;
    const size_t words = (n + k - 1u) / k;
    return (words * 4u + 15u) / 16u * 16u;
}

static int dense_common(const void* fixed, const void* dense, size_t n, uint32_t levels, bool pack,
                        void* stream)
{
    using namespace ndq;
    DenseArgs a;
    const uint32_t k = ndq_dense_group(levels);
    if (!k) return NDQ_EINVAL;
    if (n == 0) return NDQ_OK;
    if (!fixed || !dense) return NDQ_EINVAL;
    if (n >= kMaxN) return NDQ_EUNSUPPORTED;
    if (!aligned16(fixed) || !aligned16(dense)) return NDQ_EALIGN;
    const uint32_t bits = code_bits(levels);
    a.fixed = (unsigned char*)fixed;
    a.dense = (uint32_t*)dense;
    a.n = n;
    a.levels = levels;
    a.fixed_total = packed_bytes(n, bits);
    a.dense_total = ndq_dense_bytes(n, levels) / 4u;
    return run_dense(a, k, bits, pack, (hipStream_t)stream);
}

int ndq_dense_pack(const void* codes, size_t n, uint32_t levels, void* dense_out, void* stream)
{
    return dense_common(codes, dense_out, n, levels, true, stream);
}

int ndq_dense_unpack(const void* dense, size_t n, uint32_t levels, void* codes_out, void* stream)
{
    return dense_common(codes_out, dense, n, levels, false, stream);
}

double ndq_alpha_for_equal_variance(double delta1, double sigma_z2)
{
    const double arg = 1.0 - delta1 * delta1 / (12.0 * sigma_z2);
    return arg > 0.0 ? sqrt(arg) : 0.0;
}

double ndq_decode_error_bound(double delta1, uint32_t M, double alpha, double sigma_z2)
{
    const double delta2 = (double)M * delta1;
    return delta1 * delta1 / (3.0 * delta2 * delta2) + 4.0 * alpha * alpha * sigma_z2 / (delta2 * delta2);
}

uint32_t ndq_nesting_ratio_for_error(double delta1, double alpha, double sigma_z2, double p_max)
{
    if (!(delta1 > 0.0) || !(alpha >= 0.0 && alpha <= 1.0) || !(sigma_z2 >= 0.0) || !(p_max > 0.0))
        return 0;
    // bound(M) = c / M^2 with c = 1/3 + 4 alpha^2 sigma_z^2 / Delta_1^2: start at
    // the real-valued root and let the bound itself settle the last unit.
    const double c = 1.0 / 3.0 + 4.0 * alpha * alpha * sigma_z2 / (delta1 * delta1);
    const double root = sqrt(c / p_max);
    if (!(root <= 257.0)) return 0;
    uint32_t M = root < 2.0 ? 2u : (uint32_t)root;
    while (M > 2 && ndq_decode_error_bound(delta1, M - 1, alpha, sigma_z2) <= p_max) --M;
    while (M <= 256 && ndq_decode_error_bound(delta1, M, alpha, sigma_z2) > p_max) ++M;
    return M <= 256 ? M : 0;
}

size_t ndq_sqdiff_workspace(void) { return ndq::kSqBlocks * sizeof(ndq::SqSlot); }

int ndq_sqdiff(const float* a, const float* b, size_t n, double* workspace, double* out,
               void* stream)
{
    if (!workspace) return NDQ_EINVAL;
    return ndq::sqdiff_common(a, b, n, (ndq::SqSlot*)workspace, out, stream);
}

int ndq_sqdiff_static(const float* a, const float* b, size_t n, double* out, void* stream)
{
    if (n >= ndq::kMaxN) return NDQ_EUNSUPPORTED;   // beyond what the fixed grid is sized for
    ndq::SqSlot* slots = ndq::scratch_on_current_device();
    if (!slots) return NDQ_ELAUNCH;
    return ndq::sqdiff_common(a, b, n, slots, out, stream);
}

const char* ndq_strerror(int rc)
{
    switch (rc) {
        case NDQ_OK: return "success";
        case NDQ_EINVAL: return "invalid argument (null pointer, levels or M outside [2,256], overlapping buffers, bad W)";
        case NDQ_EALIGN: return "alignment violated (16-byte data pointers, bucket multiple of 64, offset multiple of 8)";
        case NDQ_EUNSUPPORTED: return "vector too long for one call";
        case NDQ_ELAUNCH: return "the HIP runtime refused a kernel launch";
        default: return "unknown ndq status";
    }
}

}  // extern "C"
