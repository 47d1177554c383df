// Small device helpers shared by the kernel files of libdfamin.
#pragma once

#include "dfamin_internal.h"

namespace dfamin {
namespace {

__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

// Multiply-xorshift mixing of 32-bit words into a 64-bit hash.
__device__ __forceinline__ uint64_t mix_step(uint64_t h, uint32_t w) {
    h ^= w;
    h *= 0x9E3779B97F4A7C15ull;
    h ^= h >> 32;
    return h;
}
__device__ __forceinline__ uint64_t mix_final(uint64_t h) {
    h ^= h >> 29;
    h *= 0xBF58476D1CE4E5B9ull;
    h ^= h >> 32;
    return h;
}
constexpr uint64_t kHashSeed = 0x6A09E667F3BCC909ull;

__device__ __forceinline__ size_t global_tid() {
    return static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
}
__device__ __forceinline__ size_t grid_stride() {
    return static_cast<size_t>(gridDim.x) * blockDim.x;
}

// Workgroup sum of per-thread values, added with one atomic per workgroup to
// one of kSpread counters (consecutive workgroups use different lines).
// Every thread of the workgroup must call it.
// The tiles (of `tile` states, covering n states) that this workgroup
// handles, as first, end and step.  Workgroups are dispatched to the 8 XCDs
// round-robin; with a grid that is a multiple of 8, each XCD takes one
// contiguous eighth of the tiles, so in a union (whose transitions stay
// inside each operand) the gathers of an XCD stay inside one operand, a
// footprint half as large for its L2.  Other grids stride over all tiles.
struct TileRange {
    size_t first, end, step;
};

__device__ __forceinline__ TileRange xcd_tiles(size_t n, size_t tile) {
    const size_t tiles = (n + tile - 1) / tile;
    TileRange t{blockIdx.x, tiles, gridDim.x};
    if (gridDim.x % 8 == 0) {
        const size_t x = blockIdx.x % 8;
        t.first = tiles * x / 8 + blockIdx.x / 8;
        t.end = tiles * (x + 1) / 8;
        t.step = gridDim.x / 8;
    }
    return t;
}

template <uint32_t NT = kBlock>  // threads of the workgroup
__device__ __forceinline__ void wg_add_spread(uint32_t *counters, int word, uint32_t v) {
    __shared__ uint32_t part[NT / 64];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    __syncthreads();
    if (lane_id() == 0) part[threadIdx.x / 64] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t s = 0;
#pragma unroll
        for (int w = 0; w < static_cast<int>(NT / 64); ++w) s += part[w];
        if (s) atomicAdd(counters + (blockIdx.x % kSpread) * kSpreadStride + word, s);
    }
}

// Sets *flag = 1 (a plain store: every writer stores the same value) if any
// active lane has `pred`; skips the store once the flag reads as set.
__device__ __forceinline__ void wave_set_flag(uint32_t *flag, bool pred) {
    const unsigned long long m = __ballot(pred);
    if (m == 0) return;
    const int leader = __ffsll(static_cast<unsigned long long>(m)) - 1;
    if (static_cast<int>(lane_id()) == leader && *flag == 0u) *flag = 1u;
}

__device__ __forceinline__ unsigned long long wave_or64(unsigned long long v) {
    uint32_t lo = static_cast<uint32_t>(v), hi = static_cast<uint32_t>(v >> 32);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        lo |= __shfl_xor(lo, d, 64);
        hi |= __shfl_xor(hi, d, 64);
    }
    return (static_cast<unsigned long long>(hi) << 32) | lo;
}


__device__ __forceinline__ bool rows_equal(const uint32_t *__restrict__ sig, size_t W, size_t a,
                                           size_t b) {
    const uint32_t *ra = sig + a * W;
    const uint32_t *rb = sig + b * W;
    // eight words at a time: their loads are in flight together, and none
    // is past the row (W is uniform)
    for (size_t i = 0; i < W; i += 8) {
        uint32_t va[8], vb[8];
#pragma unroll
        for (size_t j = 0; j < 8; ++j) {
            va[j] = vb[j] = 0;
            if (i + j < W) {
                va[j] = ra[i + j];
                vb[j] = rb[i + j];
            }
        }
        bool eq = true;
#pragma unroll
        for (size_t j = 0; j < 8; ++j) eq &= va[j] == vb[j];
        if (!eq) return false;
    }
    return true;
}

// The columns a kernel reads, resolved once per thread: the column list
// does not change during a launch, and holding the pointers in registers
// keeps the compiler from reloading the list after every store.
template <int KC>
struct ColPtrs {
    const uint32_t *c[KC > 0 ? KC : 1];
    __device__ __forceinline__ ColPtrs(const uint32_t *cols, const uint32_t *colmap, size_t N) {
#pragma unroll
        for (int j = 0; j < KC; ++j) c[j] = cols + static_cast<size_t>(colmap[j]) * N;
    }
};

// What the end of a round leaves: whether the round ran, and (in thread 0) the
// rounds so far and whether the refinement has stopped.
struct RoundOutcome {
    bool ran, done;
    uint32_t rounds;
};

__device__ __forceinline__ void wait_for_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Tells the host (page-locked memory) that a round has ended: the number of
// rounds; with details, first the blocks and gains so far; once the refinement
// has stopped, the whole round state.
// Every thread of the workgroup calls it, after ctl has been written by
// thread 0.  The stores bypass the caches, so waiting for them orders them; a
// system-scope release would write back the XCD's L2 as well, which cost 5 us
// a round.  The wait itself is a round trip to the host's memory, 1.5 us: it is
// left to the rounds that have something to order.
__device__ __forceinline__ void report_round(const RoundCtl *ctl, HostProgress *host,
                                             uint32_t details, const RoundOutcome &o) {
    if (!host) return;
    const bool done = __syncthreads_or(o.done) != 0;
    if (done || details) __syncthreads();  // (thread 0's stores to ctl)
    if (done) {
        constexpr uint32_t words = sizeof(RoundCtl) / sizeof(uint32_t);
        const uint32_t *src = reinterpret_cast<const uint32_t *>(ctl);
        uint32_t *dst = reinterpret_cast<uint32_t *>(&host->ctl);
        for (uint32_t i = threadIdx.x; i < words; i += blockDim.x)
            __hip_atomic_store(dst + i, src[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    } else if (details) {
        for (uint32_t i = threadIdx.x; i < kActiveHist; i += blockDim.x)
            __hip_atomic_store(&host->gain_hist[i], ctl->gain_hist[i], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
        if (threadIdx.x == 0) {
            __hip_atomic_store(&host->blocks, ctl->prev_count, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(&host->active_sum, ctl->active_sum, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    if (done || details) {
        wait_for_stores();
        __syncthreads();
    }
    if (threadIdx.x == 0)
        __hip_atomic_store(&host->progress, o.rounds | (done ? kProgressDone : 0u),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Marks block `id` as having two or more members after round r.
__device__ __forceinline__ void mark_multi(uint32_t *multi, uint32_t id, uint32_t tag) {
    if (multi[id] != tag) multi[id] = tag;
}

// Sets the summary bits of the groups holding a changed state, from a wave's
// changed-id mask (states first .. first + 63, first a multiple of 64).
__device__ __forceinline__ void set_summary(unsigned long long *sum, size_t first,
                                            unsigned long long cm) {
    constexpr uint32_t G = 1u << kSumShift;  // states per bit
    unsigned long long bits = 0;
    if constexpr (G >= 64) {
        bits = cm ? 1ull : 0ull;
    } else {
#pragma unroll
        for (uint32_t g = 0; g < 64 / G; ++g)
            if ((cm >> (g * G)) & ((1ull << G) - 1ull)) bits |= 1ull << g;
    }
    if (bits) atomicOr(sum + (first >> kSumWordShift), bits << ((first >> kSumShift) & 63));
}

// Whether state t's group is marked in a summary.
__device__ __forceinline__ bool summary_bit(const unsigned long long *sum, uint32_t t) {
    return ((sum[t >> kSumWordShift] >> ((t >> kSumShift) & 63)) & 1ull) != 0;
}

}  // namespace
}  // namespace dfamin
