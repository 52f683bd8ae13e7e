// gv_compact.h -- three-way compaction of track outputs into the
// per-particle-type queues (the stage baskets and survivor stack of
// Sec. 2.1.1-2.1.2, realised as queues in HBM): stable across the whole
// launch (look-back) or stable within each block (arrival-order reservation).
//
// Every input slot expands to at most three outputs (the surviving track and
// two secondaries), each bound for one of three queues.  Output order in a
// queue is the order of the expanded input stream: input slot, then
// (survivor, child 0, child 1).  One pass, no atomics deciding order:
//   1. per wave: ballot + popcount of the two bits of each thread's per-queue
//      count (0..3) gives the wave-exclusive offset and the wave total;
//   2. per block: wave totals through LDS;
//   3. across blocks: single-pass decoupled look-back over the chunk index,
//      one wave reading 64 predecessors per round (chunks are claimed in
//      increasing order, so every predecessor is owned by a running
//      workgroup); status words carry an epoch so they never need clearing
//      between launches.
#pragma once
#include "gv_common.h"

namespace gv {

// status word: [epoch:30 | flag:2 | value:32]; flag 1 = aggregate, 2 = inclusive prefix
constexpr uint64_t kFlagAgg = 1ull, kFlagInc = 2ull;
// bound on the polls of one look-back window (each poll sleeps ~64 cycles);
// past it the error flag is raised and the launch completes with a wrong count
constexpr uint32_t kMaxSpins = 1u << 22;
constexpr uint32_t kEpochBits = (1u << 30) - 1u;
__device__ __forceinline__ uint64_t pack_status(uint32_t epoch, uint64_t flag, uint32_t v)
{
    return ((uint64_t)(epoch & kEpochBits) << 34) | (flag << 32) | v;
}

template <int BLOCK> struct ScanShared {
    int wtot[3][BLOCK / 64];
    int prefix[3];
    int total[3];
    int ticket;
};

// exclusive offsets of this thread's counts within the block, and block totals
template <int BLOCK>
__device__ __forceinline__ void block_scan3(const int cnt[3], int excl[3], int tot[3], ScanShared<BLOCK>& sh)
{
    constexpr int NW = BLOCK / 64;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    int wex[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const uint64_t b0 = __ballot(cnt[q] & 1), b1 = __ballot(cnt[q] & 2);
        wex[q] = __popcll(b0 & lt) + 2 * __popcll(b1 & lt);
        if (lane == 0) sh.wtot[q][wid] = __popcll(b0) + 2 * __popcll(b1);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int v = sh.wtot[q][w];
            before += w < wid ? v : 0;
            all += v;
        }
        excl[q] = before + wex[q];
        tot[q] = all;
    }
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += (uint32_t)__shfl_xor((int)v, off, 64);
    return v;
}

// Exclusive prefix of queue q for `chunk`: wave 0 reads the status words of
// the 64 preceding chunks at once, finds the nearest inclusive prefix by
// ballot and adds the aggregates up to it; a window without an inclusive
// prefix is summed whole and the window moves 64 chunks back.
__device__ __forceinline__ uint32_t lookback_queue(const uint64_t* status, uint32_t chunk, uint32_t epoch, int q,
                                                   uint32_t* err)
{
    const int lane = threadIdx.x & 63;
    uint32_t excl = 0;
    long long hi = (long long)chunk - 1;
    uint32_t spins = 0;
    while (hi >= 0) {
        const long long j = hi - lane;
        uint64_t s = pack_status(epoch, kFlagInc, 0);   // before chunk 0: an inclusive zero
        if (j >= 0) s = __hip_atomic_load(status + (size_t)j * 3 + q, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
        const bool ok = (uint32_t)(s >> 34) == (epoch & kEpochBits) && ((s >> 32) & 3ull) != 0;
        const bool inc = ok && ((s >> 32) & 3ull) == kFlagInc;
        const uint64_t inc_mask = __ballot(inc);
        const uint64_t bad_mask = __ballot(!ok);
        const int first_inc = inc_mask ? __ffsll((unsigned long long)inc_mask) - 1 : 64;
        const uint64_t need = first_inc >= 63 ? ~0ull : ((2ull << first_inc) - 1ull);
        if ((bad_mask & need) && ++spins < kMaxSpins) {
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        if (bad_mask & need) atomicOr(err, 2u);   // gave up waiting: missing values count as zero
        spins = 0;
        const uint32_t v = (((need >> lane) & 1ull) && ok) ? (uint32_t)s : 0u;
        excl += wave_sum(v);
        if (first_inc < 64) break;
        hi -= 64;
    }
    return excl;
}

// Publish this chunk's aggregates, look back for the exclusive prefix of each
// queue, publish the inclusive prefix.  Called by all threads; wave 0 does the
// work; the result lands in sh.prefix / sh.total.
template <int BLOCK>
__device__ __forceinline__ void lookback3(uint64_t* status, uint32_t chunk, uint32_t epoch, const int tot[3],
                                          ScanShared<BLOCK>& sh, uint32_t* err)
{
    if (threadIdx.x < 64) {
        const int q = threadIdx.x;
        // this lane's queue total, selected without indexing a register array
        const uint32_t mine = (uint32_t)(q == 0 ? tot[0] : (q == 1 ? tot[1] : tot[2]));
        if (q < 3)
            __hip_atomic_store(status + (size_t)chunk * 3 + q,
                               pack_status(epoch, chunk == 0 ? kFlagInc : kFlagAgg, mine), __ATOMIC_RELEASE,
                               __HIP_MEMORY_SCOPE_AGENT);
        uint32_t e0 = 0, e1 = 0, e2 = 0;
        if (chunk > 0) {
            e0 = lookback_queue(status, chunk, epoch, 0, err);
            e1 = lookback_queue(status, chunk, epoch, 1, err);
            e2 = lookback_queue(status, chunk, epoch, 2, err);
        }
        const uint32_t ex = q == 0 ? e0 : (q == 1 ? e1 : e2);
        if (q < 3) {
            if (chunk > 0)
                __hip_atomic_store(status + (size_t)chunk * 3 + q, pack_status(epoch, kFlagInc, ex + mine),
                                   __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            sh.prefix[q] = (int)ex;
            sh.total[q] = (int)mine;
        }
    }
    __syncthreads();
}

// Arrival-order placement: the block reserves its output range in each queue
// with one atomic add on the queue's counter; the queue ends up holding the
// blocks' outputs in the order the reservations landed, each block's outputs
// in slot order.  No block waits for another.  A reservation that runs past
// `cap` sets bit 0 of *err (stores beyond cap are skipped by the caller).
template <int BLOCK>
__device__ __forceinline__ void reserve3(uint32_t* count_out, uint32_t cap, const int tot[3], ScanShared<BLOCK>& sh,
                                         uint32_t* err)
{
    if (threadIdx.x < 3) {
        const int q = threadIdx.x;
        const uint32_t mine = (uint32_t)(q == 0 ? tot[0] : (q == 1 ? tot[1] : tot[2]));
        uint32_t base = 0;
        if (mine) {
            base = atomicAdd(count_out + q, mine);
            if ((uint64_t)base + mine > cap) atomicOr(err, 1u);
        }
        sh.prefix[q] = (int)base;
        sh.total[q] = (int)mine;
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// The same compaction of codes already in memory (gv_compact3_noalloc), in two
// launches: each block counts its inputs' codes per queue, then each block adds
// up the totals of the blocks before it and places its own.  Codes are read
// twice, but nothing waits: the single-pass look-back is for callers whose
// counts are expensive to form again (the step kernel), and took 475 us for the
// same million (3,907 chunks of 256 in one chain of look-backs).
// One million inputs take 10.6 us this way, most of it the two launches; millions
// of them are bound by HBM.
// A thread takes ITEMS inputs in a row (16 from 2^20 inputs on: 48 bytes, three
// 16-byte loads, and few enough blocks that adding up their totals is cheap;
// 4 below, so that 100,000 inputs still fill the chip) and the block's outputs
// go through LDS, so that each queue's run is written in order.  Up to 8,192
// inputs (eight blocks of 4 per thread) the blocks count the codes before theirs
// themselves (ALONE) and one launch is enough: 100 inputs 4.5 us, 8,000 7.3 us,
// where two launches take 7.9 us at any size up to 100,000 (16 inputs per thread
// there took 10.9 us for 100, unrolled over too few lanes).
// ---------------------------------------------------------------------------
constexpr int kPartBlock = 256;
constexpr unsigned long long kPartBad = 1ull << 48;   // beside three 16-bit counts: a code outside [-1, 2]

// the codes of ITEMS inputs, four to a word; inputs past n read as -1
template <int ITEMS, bool ALIGNED>
__device__ __forceinline__ void part_load(const int8_t* codes, long long i0, long long n, uint32_t w[3 * ITEMS / 4])
{
    constexpr int W = 3 * ITEMS / 4;
    if (ALIGNED && i0 + ITEMS <= n) {
        if constexpr (ITEMS == 16) {
            const uint4* p = reinterpret_cast<const uint4*>(codes + 3 * i0);
#pragma unroll
            for (int k = 0; k < W / 4; ++k) {
                const uint4 v = p[k];
                w[4 * k] = v.x;
                w[4 * k + 1] = v.y;
                w[4 * k + 2] = v.z;
                w[4 * k + 3] = v.w;
            }
        } else {
            const uint32_t* p = reinterpret_cast<const uint32_t*>(codes + 3 * i0);
#pragma unroll
            for (int k = 0; k < W; ++k) w[k] = p[k];
        }
        return;
    }
    if (!ALIGNED && i0 > 0 && i0 + ITEMS + 1 < n) {
        // at any address: the words that hold the codes, shifted into place.  They
        // begin up to 3 bytes before and end up to 4 bytes after them, in codes of
        // other inputs.  (Byte by byte, 8,192 inputs took 12.9 us instead of 8.0.)
        const uintptr_t at = (uintptr_t)(codes + 3 * i0);
        const uint32_t* p = reinterpret_cast<const uint32_t*>(at & ~(uintptr_t)3);
        uint32_t v[W + 1];
#pragma unroll
        for (int k = 0; k <= W; ++k) v[k] = p[k];
#pragma unroll
        for (int k = 0; k < W; ++k) w[k] = __builtin_amdgcn_alignbyte(v[k + 1], v[k], (uint32_t)at);
        return;
    }
#pragma unroll
    for (int k = 0; k < W; ++k) {
        uint32_t v = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const long long at = 3 * i0 + 4 * k + b;
            v |= (uint32_t)(uint8_t)(at < 3 * n ? codes[at] : (int8_t)-1) << (8 * b);
        }
        w[k] = v;
    }
}

// codes per queue, 16 bits each (at most 3 * ITEMS * kPartBlock = 12,288 in a block)
template <int W> __device__ __forceinline__ unsigned long long part_count(const uint32_t w[W], bool& bad)
{
    unsigned long long c = 0;
#pragma unroll
    for (int k = 0; k < 4 * W; ++k) {
        const int q = (int)(int8_t)(w[k / 4] >> (8 * (k % 4)));
        c += (q >= 0 && q <= 2) ? 1ull << (16 * (q & 3)) : 0ull;
        bad |= q < -1 || q > 2;
    }
    return c;
}

template <int ITEMS, bool ALIGNED>
__global__ void __launch_bounds__(kPartBlock) k_part_count(const int8_t* codes, long long n, unsigned long long* totals)
{
    __shared__ unsigned long long sum[kPartBlock / 64];
    const long long i0 = ((long long)blockIdx.x * kPartBlock + threadIdx.x) * ITEMS;
    uint32_t w[3 * ITEMS / 4];
    part_load<ITEMS, ALIGNED>(codes, i0, n, w);
    bool bad = false;
    unsigned long long c = part_count<3 * ITEMS / 4>(w, bad);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    if (__any(bad)) c |= kPartBad;
    if ((threadIdx.x & 63) == 0) sum[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0, f = 0;
        for (int k = 0; k < kPartBlock / 64; ++k) {
            t += sum[k] & (kPartBad - 1);
            f |= sum[k] & kPartBad;
        }
        totals[blockIdx.x] = t | f;
    }
}

template <int ITEMS, bool ALIGNED, bool ALONE>
__global__ void __launch_bounds__(kPartBlock) k_part_place(const int8_t* codes, long long n, int* index,
                                                           uint32_t* counts, const unsigned long long* totals)
{
    constexpr int kWaves = kPartBlock / 64;
    __shared__ unsigned long long wsum[kWaves];
    __shared__ uint32_t before[kWaves][3];
    __shared__ uint32_t flag;
    __shared__ int out[3 * ITEMS * kPartBlock];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const long long i0 = ((long long)blockIdx.x * kPartBlock + threadIdx.x) * ITEMS;
    uint32_t w[3 * ITEMS / 4];
    part_load<ITEMS, ALIGNED>(codes, i0, n, w);
    bool bad = false;
    const unsigned long long mine = part_count<3 * ITEMS / 4>(w, bad);
    // inclusive scan of the wavefront's counts
    unsigned long long inc = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long v = __shfl_up(inc, off, 64);
        inc += lane >= off ? v : 0ull;
    }
    if (threadIdx.x == 0) flag = 0;
    if (lane == 63) wsum[wid] = inc;
    // totals of the blocks before this one
    uint32_t p[3] = {0, 0, 0};
    bool any_bad = bad;
    for (uint32_t j = threadIdx.x; j < (ALONE ? blockIdx.x * kPartBlock : blockIdx.x); j += kPartBlock) {
        unsigned long long t;
        if constexpr (ALONE) {
            uint32_t v[3 * ITEMS / 4];
            part_load<ITEMS, ALIGNED>(codes, (long long)j * ITEMS, n, v);
            t = part_count<3 * ITEMS / 4>(v, any_bad);
        } else {
            t = totals[j];
            any_bad |= (t & kPartBad) != 0;
        }
        p[0] += (uint32_t)t & 0xffffu;
        p[1] += (uint32_t)(t >> 16) & 0xffffu;
        p[2] += (uint32_t)(t >> 32) & 0xffffu;
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const uint32_t v = wave_sum(p[q]);
        if (lane == 0) before[wid][q] = v;
    }
    __syncthreads();
    if (__any(any_bad) && lane == 0) atomicOr(&flag, 4u);
    unsigned long long excl = inc - mine, tot = 0;
    uint32_t base[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        excl += k < wid ? wsum[k] : 0ull;
        tot += wsum[k];
#pragma unroll
        for (int q = 0; q < 3; ++q) base[q] += before[k][q];
    }
    const uint32_t t0 = (uint32_t)tot & 0xffffu, t1 = (uint32_t)(tot >> 16) & 0xffffu,
                   t2 = (uint32_t)(tot >> 32) & 0xffffu;
    // this block's outputs in LDS: queue 0's, then 1's, then 2's
    uint32_t at[3] = {(uint32_t)excl & 0xffffu, t0 + ((uint32_t)(excl >> 16) & 0xffffu),
                      t0 + t1 + ((uint32_t)(excl >> 32) & 0xffffu)};
#pragma unroll
    for (int k = 0; k < 3 * ITEMS; ++k) {
        const int q = (int)(int8_t)(w[k / 4] >> (8 * (k % 4)));
        const int v = (int)(i0 + k / 3) * 4 + k % 3;
        if (q == 0) out[at[0]++] = v;
        else if (q == 1) out[at[1]++] = v;
        else if (q == 2) out[at[2]++] = v;
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < t0 + t1 + t2; k += kPartBlock) {
        const uint32_t q = k < t0 ? 0u : k < t0 + t1 ? 1u : 2u;
        const uint32_t first = q == 0 ? 0u : q == 1 ? t0 : t0 + t1;
        const uint32_t b = q == 0 ? base[0] : q == 1 ? base[1] : base[2];
        index[(long long)q * 3 * n + b + (k - first)] = out[k];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        counts[0] = base[0] + t0;
        counts[1] = base[1] + t1;
        counts[2] = base[2] + t2;
        counts[3] = flag;
    }
}

}  // namespace gv
