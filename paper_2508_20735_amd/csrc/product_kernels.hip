// Breadth-first exploration of the synchronous product of two DFAs on the
// GPU: the naive Hopcroft-Karp of Section 4, where the relation is the plain
// set of reached pairs (a lock-free hash set of 64-bit keys p << 32 | q in
// HBM) and no transitive closure is maintained.  Inclusion L(A) <= L(B) is
// refuted by a reached pair with p accepting in A and q rejecting in B;
// equivalence by a pair with exactly one accepting side.
#include "device_common.h"

namespace dfamin {
namespace {

constexpr unsigned long long kEmpty = ~0ull;

// Slot of a pair key: the library's key mixing over its two 32-bit halves.
__device__ __forceinline__ uint64_t pair_hash(uint64_t key) {
    return mix_final(mix_step(mix_step(kHashSeed, static_cast<uint32_t>(key >> 32)),
                              static_cast<uint32_t>(key)));
}

// Inserts key, whose slot s held e when it was read; returns true if the key
// was not present.
__device__ __forceinline__ bool set_insert_from(unsigned long long *tab, uint64_t mask,
                                                unsigned long long key, uint64_t s,
                                                unsigned long long e) {
    for (;;) {
        if (e == key) return false;
        if (e == kEmpty) {
            const unsigned long long prev = atomicCAS(tab + s, kEmpty, key);
            if (prev == kEmpty) return true;
            if (prev == key) return false;
        }
        s = (s + 1) & mask;
        e = __hip_atomic_load(tab + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__device__ __forceinline__ bool set_insert(unsigned long long *tab, uint64_t mask,
                                           unsigned long long key) {
    const uint64_t s = pair_hash(key) & mask;
    return set_insert_from(tab, mask, key, s,
                           __hip_atomic_load(tab + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Whether pair (p, q) refutes the property.
__device__ __forceinline__ bool refutes(const ProductArgs &a, uint32_t p, uint32_t q) {
    const bool fa = a.accA[p] != 0, fb = a.accB[q] != 0;
    return a.mode == 0 ? (fa && !fb) : (fa != fb);
}

__global__ __launch_bounds__(64) void k_product_reset(ProductCtl *ctl, unsigned long long count,
                                                      uint32_t frontier_size) {
    if (blockIdx.x != 0) return;
    for (uint32_t i = threadIdx.x; i <= kProductBatch; i += 64) ctl->size[i] = i ? 0u : frontier_size;
    if (threadIdx.x == 0) {
        ctl->count = count;
        ctl->narrow_levels = 0;
        ctl->refuted = 0;
    }
}

// One level of the search (level j of a batch): the frontier of ctl->size[j]
// pairs expands into `next`, ctl->size[j + 1] = the new pairs.  The level
// does nothing (and leaves size[j + 1] zero, so the levels after it do
// nothing either) when its frontier is empty, a pair was refuted before, or
// it could outgrow `next` or half of the visited set: the host then makes
// room.
//
// Bound by random accesses: the two rows, two acceptance bytes and one
// probe per pair and letter.  A workgroup appends its new pairs of up to
// kLetters letters with one atomic: one atomic per wave and letter on the
// single counter made a level of 806,000 pairs and 4 letters 608 us (50,000
// atomics, about 12 ns each); this one takes about 120.
constexpr uint32_t kLetters = 4;

__global__ __launch_bounds__(kBlock) void k_product_level(ProductArgs a,
                                                          const unsigned long long *frontier,
                                                          unsigned long long *next,
                                                          uint64_t next_cap, uint32_t j) {
    __shared__ uint32_t wsum[kBlock / 64];
    __shared__ uint32_t at;
    ProductCtl *ctl = a.ctl;
    const uint32_t n = ctl->size[j];
    unsigned long long total = ctl->count;
    for (uint32_t i = 1; i <= j; ++i) total += ctl->size[i];
    const unsigned long long most = static_cast<unsigned long long>(n) * a.k;
    // (uniform over the grid, but for a refutation found meanwhile by this
    // level itself, which makes its new pairs worthless)
    const bool skip = n == 0 || ctl->err || ctl->refuted || most > next_cap ||
                      (total + most) * 2 > a.visited_cap;
    if (__syncthreads_or(skip)) return;
    const uint32_t lane = lane_id(), wave = threadIdx.x / 64;
    const uint64_t mask = a.visited_cap - 1;
    // rows of a multiple of 4 letters at 16-byte aligned addresses are read
    // 16 bytes at a time
    const bool wide = a.k % 4 == 0 && ((reinterpret_cast<uintptr_t>(a.dA) |
                                        reinterpret_cast<uintptr_t>(a.dB)) & 15u) == 0;
    for (size_t base = static_cast<size_t>(blockIdx.x) * kBlock; base < n;
         base += static_cast<size_t>(gridDim.x) * kBlock) {
        const size_t i = base + threadIdx.x;
        const unsigned long long key = i < n ? frontier[i] : 0ull;
        const uint32_t p = static_cast<uint32_t>(key >> 32), q = static_cast<uint32_t>(key);
        bool live = i < n;
        if (live && refutes(a, p, q)) {
            ctl->refuted = j + 1;
            live = false;
        }
        const uint32_t *ra = a.dA + static_cast<size_t>(p) * a.k;
        const uint32_t *rb = a.dB + static_cast<size_t>(q) * a.k;
        for (uint32_t c0 = 0; c0 < a.k; c0 += kLetters) {
            const uint32_t m = a.k - c0 < kLetters ? a.k - c0 : kLetters;
            uint32_t ta[kLetters], tb[kLetters];
            if (wide) {
                const uint4 va = *reinterpret_cast<const uint4 *>(ra + c0);
                const uint4 vb = *reinterpret_cast<const uint4 *>(rb + c0);
                ta[0] = va.x, ta[1] = va.y, ta[2] = va.z, ta[3] = va.w;
                tb[0] = vb.x, tb[1] = vb.y, tb[2] = vb.z, tb[3] = vb.w;
            } else {
#pragma unroll
                for (uint32_t c = 0; c < kLetters; ++c) {
                    ta[c] = ra[c0 + (c < m ? c : 0u)];
                    tb[c] = rb[c0 + (c < m ? c : 0u)];
                }
            }
            // every letter's first probe is in flight before one is resolved
            unsigned long long nk[kLetters], e[kLetters];
            uint64_t s[kLetters];
#pragma unroll
            for (uint32_t c = 0; c < kLetters; ++c) {
                nk[c] = (static_cast<unsigned long long>(ta[c]) << 32) | tb[c];
                s[c] = pair_hash(nk[c]) & mask;
                e[c] = nk[c];
                if (live && c < m)
                    e[c] = __hip_atomic_load(a.visited + s[c], __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
            }
            bool fresh[kLetters];
            uint32_t mine = 0;
#pragma unroll
            for (uint32_t c = 0; c < kLetters; ++c) {
                fresh[c] = live && c < m && set_insert_from(a.visited, mask, nk[c], s[c], e[c]);
                mine += fresh[c] ? 1u : 0u;
            }
            // the workgroup's new pairs, thread by thread
            uint32_t x = mine;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t y = __shfl_up(x, d, 64);
                if (lane >= static_cast<uint32_t>(d)) x += y;
            }
            if (lane == 63) wsum[wave] = x;
            __syncthreads();
            uint32_t before = 0, all = 0;
#pragma unroll
            for (uint32_t w = 0; w < kBlock / 64; ++w) {
                before += w < wave ? wsum[w] : 0u;
                all += wsum[w];
            }
            if (threadIdx.x == 0 && all) at = atomicAdd(&ctl->size[j + 1], all);
            __syncthreads();
            // (at most n * k new pairs, which `next` holds)
            size_t slot = static_cast<size_t>(all ? at : 0u) + before + x - mine;
#pragma unroll
            for (uint32_t c = 0; c < kLetters; ++c)
                if (fresh[c]) next[slot++] = nk[c];
        }
    }
}

// One workgroup expands levels while the frontier times k fits an LDS queue
// (long, thin explorations such as C_n's products, where a launch and a host
// round trip per level would dominate).  Pairs are inserted into the same
// HBM set as by k_product_level; new pairs go to the other LDS queue.  Stops
// when the frontier is empty, a refuting pair is expanded, the next
// frontier could overflow the queue or half of the visited set, or after
// max_levels levels; the remaining frontier is written back to `frontier`,
// ctl->size[0] receives its size and ctl->count the pairs added.
__global__ __launch_bounds__(kProductNarrowThreads) void k_product_narrow(
    ProductArgs a, unsigned long long *frontier, uint32_t max_levels) {
    __shared__ unsigned long long buf[2][kProductNarrowCap];
    __shared__ uint32_t next_size, refuted;
    ProductCtl *ctl = a.ctl;
    if (ctl->err || ctl->refuted) return;
    const uint32_t tx = threadIdx.x;
    const uint64_t mask = a.visited_cap - 1;
    uint32_t s = ctl->size[0];
    unsigned long long total = ctl->count;
    if (static_cast<uint64_t>(s) * a.k > kProductNarrowCap) return;
    for (uint32_t i = tx; i < s; i += kProductNarrowThreads) buf[0][i] = frontier[i];
    if (tx == 0) refuted = 0;
    __syncthreads();  // every thread has read the control words
    uint32_t cur = 0, levels = 0;
    for (;;) {
        const uint64_t most = static_cast<uint64_t>(s) * a.k;
        if (s == 0 || levels == max_levels || most > kProductNarrowCap ||
            (total + most) * 2 > a.visited_cap)
            break;
        if (tx == 0) next_size = 0;
        __syncthreads();
        for (uint32_t i = tx; i < s; i += kProductNarrowThreads) {
            const unsigned long long key = buf[cur][i];
            const uint32_t p = static_cast<uint32_t>(key >> 32), q = static_cast<uint32_t>(key);
            if (refutes(a, p, q)) {
                refuted = 1;
                continue;
            }
            for (uint32_t c = 0; c < a.k; ++c) {
                const unsigned long long nk =
                    (static_cast<unsigned long long>(a.dA[static_cast<size_t>(p) * a.k + c]) << 32) |
                    a.dB[static_cast<size_t>(q) * a.k + c];
                // at most s * k fresh pairs <= kProductNarrowCap
                if (set_insert(a.visited, mask, nk)) buf[cur ^ 1u][atomicAdd(&next_size, 1u)] = nk;
            }
        }
        __syncthreads();
        ++levels;
        const uint32_t n = next_size;
        const bool stop = refuted != 0;
        __syncthreads();  // every thread has read next_size before it is reset
        if (stop) {
            s = 0;
            break;
        }
        total += n;
        s = n;
        cur ^= 1u;
    }
    for (uint32_t i = tx; i < s; i += kProductNarrowThreads) frontier[i] = buf[cur][i];
    if (tx == 0) {
        ctl->size[0] = s;
        ctl->count = total;
        ctl->narrow_levels = levels;
        if (refuted) ctl->refuted = kProductNarrowRefuted;
    }
}

__global__ __launch_bounds__(kBlock) void k_visited_clear(unsigned long long *tab, uint64_t cap) {
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < cap;
         i += static_cast<size_t>(gridDim.x) * blockDim.x)
        tab[i] = kEmpty;
}

__global__ void k_product_start(ProductArgs a, unsigned long long *frontier,
                                unsigned long long key) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    set_insert(a.visited, a.visited_cap - 1, key);
    frontier[0] = key;
}

__global__ __launch_bounds__(kBlock) void k_rehash(const unsigned long long *old_tab, uint64_t old_cap,
                                                    unsigned long long *new_tab, uint64_t new_cap) {
    for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < old_cap;
         i += static_cast<size_t>(gridDim.x) * blockDim.x) {
        const unsigned long long key = old_tab[i];
        if (key != kEmpty) set_insert(new_tab, new_cap - 1, key);
    }
}

unsigned grid_for(size_t work) {
    size_t g = (work + kBlock - 1) / kBlock;
    if (g == 0) g = 1;
    if (g > (1u << 20)) g = 1u << 20;
    return static_cast<unsigned>(g);
}

}  // namespace

void launch_product_reset(ProductCtl *ctl, uint64_t count, uint32_t frontier_size,
                          hipStream_t s) {
    launch_kernel(k_product_reset, dim3(1), dim3(64), 0, s, ctl,
                  static_cast<unsigned long long>(count), frontier_size);
}

void launch_product_start(const ProductArgs &a, unsigned long long *frontier,
                          unsigned long long key, hipStream_t s) {
    launch_kernel(k_product_start, dim3(1), dim3(64), 0, s, a, frontier, key);
}

void launch_product_level(const ProductArgs &a, const unsigned long long *frontier,
                          unsigned long long *next, uint64_t next_cap, uint32_t level,
                          uint32_t groups, hipStream_t s) {
    launch_kernel(k_product_level, dim3(groups), dim3(kBlock), 0, s, a, frontier, next, next_cap,
                  level);
}

void launch_product_narrow(const ProductArgs &a, unsigned long long *frontier,
                           uint32_t max_levels, hipStream_t s) {
    launch_kernel(k_product_narrow, dim3(1), dim3(kProductNarrowThreads), 0, s, a, frontier,
                  max_levels);
}

void launch_visited_clear(unsigned long long *visited, uint64_t cap, hipStream_t s) {
    launch_kernel(k_visited_clear, dim3(grid_for(cap)), dim3(kBlock), 0, s, visited, cap);
}

void launch_rehash(const unsigned long long *old_tab, uint64_t old_cap,
                   unsigned long long *new_tab, uint64_t new_cap, hipStream_t s) {
    launch_kernel(k_rehash, dim3(grid_for(old_cap)), dim3(kBlock), 0, s, old_tab, old_cap,
                       new_tab, new_cap);
}

}  // namespace dfamin
