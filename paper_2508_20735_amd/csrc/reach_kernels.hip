// Reachability from the start state (breadth-first search) and the
// sub-automaton of the reachable states, for minimisation restricted to the
// reachable part (the usual minimal DFA; the paper itself prunes nothing,
// Section 2).
//
// The search keeps a mark byte per state (0 unvisited, 1 settled, 2 / 3 in
// the frontier of an even / odd level) and a frontier queue.  A frontier of
// at most kNarrowCap / k states is expanded inside one workgroup, level after
// level, with both queues in LDS (long thin searches, such as chains, then
// cost no launch per level; an atomic on the mark's word dedupes within the
// workgroup).  A larger frontier is expanded by dense levels: every state is
// scanned, the frontier ones expand, and unvisited targets get the next
// level's mark by plain stores (several writers store the same value), so
// wide levels use no atomics on the visited set.  Every state is marked once,
// so both loops end.
//
// The host queues a narrow launch and several dense levels at a time; each
// decides on the device whether it still has work (the marks that the level
// before it stored, the target check), so the host waits once per batch of
// levels, not once per level.
#include <algorithm>

#include "device_common.h"

namespace dfamin {
namespace {

constexpr uint32_t kNarrowThreads = 1024;
constexpr uint32_t kNarrowCap = 4096;  // LDS queue entries (two queues: 32 KB)

// *err = 1 if some target is >= n (every later step indexes with targets).
__global__ __launch_bounds__(kBlock) void k_check_targets(const uint32_t *__restrict__ delta,
                                                          uint64_t total, uint32_t n,
                                                          uint32_t *err) {
    bool bad = false;
    for (uint64_t i = global_tid(); i < total; i += grid_stride()) bad |= delta[i] >= n;
    wave_set_flag(err, bad);
}

// Marks t as settled if it is unvisited; true for the one caller that did.
// (While the narrow kernel runs, every mark is 0 or 1.)
__device__ __forceinline__ bool settle(uint8_t *mark, uint32_t t) {
    if (__hip_atomic_load(mark + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) return false;
    const uint32_t sh = 8 * (t & 3);
    uint32_t *w = reinterpret_cast<uint32_t *>(mark) + (t >> 2);
    return ((atomicOr(w, 1u << sh) >> sh) & 0xFFu) == 0;
}

// One workgroup: expands levels while the frontier times k fits kNarrowCap,
// then leaves the frontier in qa / sizes[0].  The search starts at `start`
// (init), or continues from qa.
__global__ __launch_bounds__(kNarrowThreads) void k_bfs_narrow(ReachArgs a, uint32_t start,
                                                               uint32_t init) {
    __shared__ uint32_t buf[2][kNarrowCap];
    __shared__ uint32_t sz[2];
    if (*a.err) return;
    const uint32_t tx = threadIdx.x;
    const uint32_t k = a.k;
    uint32_t s = init ? 1u : a.sizes[0];
    if (!init && static_cast<uint64_t>(s) * k > kNarrowCap) return;  // the host checked; stay safe
    if (init) {
        if (tx == 0) {
            buf[0][0] = start;
            a.mark[start] = 1;
        }
    } else {
        for (uint32_t i = tx; i < s; i += kNarrowThreads) buf[0][i] = a.qa[i];
    }
    if (tx == 0) sz[0] = s;
    __syncthreads();
    uint32_t cur = 0;
    for (;;) {
        s = sz[cur];
        // uniform: every thread read the same size after the barrier
        if (s == 0 || static_cast<uint64_t>(s) * k > kNarrowCap) break;
        const uint32_t nxt = cur ^ 1u;
        if (tx == 0) sz[nxt] = 0;
        __syncthreads();
        const uint32_t work = s * k;
        for (uint32_t i = tx; i < work; i += kNarrowThreads) {
            const uint32_t q = buf[cur][i / k];
            const uint32_t t = a.delta[static_cast<size_t>(q) * k + (i % k)];
            // at most one entry per (state, letter) pair: pos < s * k <= kNarrowCap
            if (settle(a.mark, t)) buf[nxt][atomicAdd(&sz[nxt], 1u)] = t;
        }
        __syncthreads();
        cur = nxt;
    }
    s = sz[cur];
    for (uint32_t i = tx; i < s; i += kNarrowThreads) a.qa[i] = buf[cur][i];
    if (tx == 0) a.sizes[0] = s;
}

// Queue -> marks: the listed states become the frontier of a dense level
// (nothing to do while the frontier still suits the narrow kernel).
__global__ __launch_bounds__(kBlock) void k_bfs_list_to_marks(ReachArgs a, uint8_t f) {
    if (*a.err) return;
    const uint32_t s = a.sizes[0];
    if (static_cast<uint64_t>(s) * a.k <= kNarrowCap) return;
    for (size_t i = global_tid(); i < s; i += grid_stride()) a.mark[a.qa[i]] = f;
}

// One dense level: states marked f expand (unvisited targets get nf) and
// settle.  The level's counters receive the number of marks stored (an
// upper bound of the new states: two lanes may store the same target; zero
// iff none was stored).  Level j of a batch writes counter set j; it runs if
// the level before it stored more than the narrow kernel takes (after_list:
// if the listed frontier is that large; the first level of a batch that
// continues dense levels always runs).
//
// Bound by the frontier's rows and their random mark reads (the marks fit
// L2).  S states per thread, a word of marks at a time; the count goes out as
// one atomic per workgroup, spread over kBfsSpread lines: one atomic per
// wave on a single word made a level of 2^20 states 190 us (16,384 waves,
// about 11 ns each); this one takes about 12.
template <int KC>
__global__ __launch_bounds__(kBlock) void k_bfs_dense(ReachArgs a, uint8_t f, uint8_t nf,
                                                      uint32_t level, uint32_t after_list) {
    __shared__ uint32_t part[kBlock / 64];
    if (*a.err) return;
    if (after_list) {
        if (static_cast<uint64_t>(a.sizes[0]) * a.k <= kNarrowCap) return;
    } else if (level > 0) {
        const uint32_t *prev = a.stored + (level - 1) * kBfsSetWords;
        uint32_t v = lane_id() < kBfsSpread ? prev[lane_id() * kBfsStride] : 0u;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
        if (static_cast<uint64_t>(v) * a.k <= kNarrowCap) return;  // uniform over the grid
    }
    constexpr int S = 4;  // states per thread: one word of marks
    uint32_t stored = 0;
    const size_t words = (static_cast<size_t>(a.n) + S - 1) / S;
    for (size_t i = global_tid(); i < words; i += grid_stride()) {
        const uint32_t m = reinterpret_cast<const uint32_t *>(a.mark)[i];
        bool act[S];
        bool any = false;
#pragma unroll
        for (int u = 0; u < S; ++u) {
            act[u] = ((m >> (8 * u)) & 0xFFu) == f && i * S + u < a.n;
            any |= act[u];
        }
        if (!any) continue;
        // letters in groups of KC: the row entries of every state, then
        // their marks, are loaded together before any store (an idle state
        // reads its word's first active one's row again)
        size_t q[S], busy = 0;
#pragma unroll
        for (int u = S - 1; u >= 0; --u)
            if (act[u]) busy = i * S + u;
#pragma unroll
        for (int u = 0; u < S; ++u) q[u] = act[u] ? i * S + u : busy;
        for (uint32_t j0 = 0; j0 < a.k; j0 += KC) {
            uint32_t t[S][KC];
            uint8_t mk[S][KC];
#pragma unroll
            for (int u = 0; u < S; ++u)
#pragma unroll
                for (int j = 0; j < KC; ++j)
                    t[u][j] = a.delta[q[u] * a.k + (j0 + j < a.k ? j0 + j : j0)];
#pragma unroll
            for (int u = 0; u < S; ++u)
#pragma unroll
                for (int j = 0; j < KC; ++j) mk[u][j] = a.mark[t[u][j]];
#pragma unroll
            for (int u = 0; u < S; ++u)
#pragma unroll
                for (int j = 0; j < KC; ++j)
                    if (act[u] && mk[u][j] == 0) {
                        a.mark[t[u][j]] = nf;
                        ++stored;
                    }
        }
#pragma unroll
        for (int u = 0; u < S; ++u)
            if (act[u]) a.mark[i * S + u] = 1;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) stored += __shfl_xor(stored, d, 64);
    if (lane_id() == 0) part[threadIdx.x / 64] = stored;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t sum = 0;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) sum += part[w];
        if (sum)
            atomicAdd(a.stored + level * kBfsSetWords + (blockIdx.x % kBfsSpread) * kBfsStride, sum);
    }
}

// Marks -> queue: the states marked f settle and are listed in qa (one
// append atomic per wave); sizes[0], zero on entry, = their number.
__global__ __launch_bounds__(kBlock) void k_bfs_marks_to_list(ReachArgs a, uint8_t f) {
    const uint32_t lane = lane_id();
    for (size_t base = static_cast<size_t>(blockIdx.x) * kBlock; base < a.n;
         base += static_cast<size_t>(gridDim.x) * kBlock) {
        const size_t q = base + threadIdx.x;
        const bool hit = q < a.n && a.mark[q] == f;
        const unsigned long long m = __ballot(hit);
        if (m == 0) continue;
        const int leader = __ffsll(static_cast<unsigned long long>(m)) - 1;
        uint32_t pos = 0;
        if (static_cast<int>(lane) == leader)
            pos = atomicAdd(a.sizes, static_cast<uint32_t>(__popcll(m)));
        pos = __shfl(pos, leader, 64);
        if (hit) {
            const unsigned long long below = lane ? (m & ((1ull << lane) - 1ull)) : 0ull;
            a.qa[pos + static_cast<uint32_t>(__popcll(below))] = static_cast<uint32_t>(q);
            a.mark[q] = 1;
        }
    }
}

// The counters of a batch of dense levels start at zero.
__global__ __launch_bounds__(kBlock) void k_bfs_reset(ReachArgs a, uint32_t list) {
    for (uint32_t i = threadIdx.x; i < kBfsBatch * kBfsSetWords; i += kBlock) a.stored[i] = 0;
    if (list && threadIdx.x == 0) a.sizes[0] = 0;
}

// Sub-automaton: row i is the reachable state orig[i], targets renumbered.
__global__ __launch_bounds__(kBlock) void k_sub_dfa(const uint32_t *__restrict__ delta,
                                                    const uint8_t *__restrict__ acc, uint32_t k,
                                                    const uint32_t *__restrict__ orig,
                                                    const uint32_t *__restrict__ dense,
                                                    const uint32_t *m_dev,
                                                    uint32_t *__restrict__ sub_delta,
                                                    uint8_t *__restrict__ sub_acc) {
    const uint64_t m = *m_dev;
    const uint64_t work = m * k;
    for (uint64_t i = global_tid(); i < work; i += grid_stride()) {
        const uint64_t row = i / k;
        const uint32_t q = orig[row];
        sub_delta[i] = dense[delta[static_cast<size_t>(q) * k + (i % k)]];
        if (i % k == 0) sub_acc[row] = acc[q];
    }
}

// block_out[q] = orig[sub_block[dense[q]]] for reachable q, kUnreachable
// otherwise (sub_block is canonical, and dense keeps the original order, so
// the result is the smallest reachable state of the block).
__global__ __launch_bounds__(kBlock) void k_reach_expand(const uint8_t *mark, size_t n,
                                                         const uint32_t *dense,
                                                         const uint32_t *orig,
                                                         const uint32_t *sub_block,
                                                         uint32_t *block_out) {
    for (size_t q = global_tid(); q < n; q += grid_stride())
        block_out[q] = mark[q] ? orig[sub_block[dense[q]]] : 0xFFFFFFFFu;
}

unsigned grid_of(uint64_t work, unsigned cap = 8192) {
    uint64_t g = (work + kBlock - 1) / kBlock;
    if (g == 0) g = 1;
    if (g > cap) g = cap;
    return static_cast<unsigned>(g);
}

}  // namespace

void launch_check_targets(const uint32_t *delta, uint64_t total, uint32_t n, uint32_t *err,
                          hipStream_t s) {
    launch_kernel(k_check_targets, dim3(grid_of(total)), dim3(kBlock), 0, s, delta, total, n,
                       err);
}

void launch_bfs_narrow(const ReachArgs &a, uint32_t start, bool init, hipStream_t s) {
    launch_kernel(k_bfs_narrow, dim3(1), dim3(kNarrowThreads), 0, s, a, start, init ? 1u : 0u);
}

void launch_bfs_list_to_marks(const ReachArgs &a, uint8_t f, hipStream_t s) {
    // the frontier's size is known on the device only: at most kNarrowCap
    // states per letter step of the narrow kernel
    launch_kernel(k_bfs_list_to_marks, dim3(grid_of(std::min(a.n, kNarrowCap))), dim3(kBlock), 0, s,
                  a, f);
}

void launch_bfs_dense(const ReachArgs &a, uint8_t f, uint8_t nf, uint32_t level, bool after_list,
                      hipStream_t s) {
    const dim3 grid(grid_of((static_cast<uint64_t>(a.n) + 3) / 4, 4096)), block(kBlock);
    const uint32_t al = after_list ? 1u : 0u;
    if (a.k <= 2)
        launch_kernel(k_bfs_dense<2>, grid, block, 0, s, a, f, nf, level, al);
    else
        launch_kernel(k_bfs_dense<4>, grid, block, 0, s, a, f, nf, level, al);
}

void launch_bfs_marks_to_list(const ReachArgs &a, uint8_t f, hipStream_t s) {
    launch_kernel(k_bfs_marks_to_list, dim3(grid_of(a.n)), dim3(kBlock), 0, s, a, f);
}

void launch_bfs_reset(const ReachArgs &a, bool list, hipStream_t s) {
    launch_kernel(k_bfs_reset, dim3(1), dim3(kBlock), 0, s, a, list ? 1u : 0u);
}

uint32_t bfs_narrow_cap() { return kNarrowCap; }

void launch_sub_dfa(const uint32_t *delta, const uint8_t *acc, uint32_t k, const uint32_t *orig,
                    const uint32_t *dense, const uint32_t *m_dev, uint32_t m_host,
                    uint32_t *sub_delta, uint8_t *sub_acc, hipStream_t s) {
    launch_kernel(k_sub_dfa, dim3(grid_of(static_cast<uint64_t>(m_host) * k)), dim3(kBlock),
                       0, s, delta, acc, k, orig, dense, m_dev, sub_delta, sub_acc);
}

void launch_reach_expand(const uint8_t *mark, size_t n, const uint32_t *dense,
                         const uint32_t *orig, const uint32_t *sub_block, uint32_t *block_out,
                         hipStream_t s) {
    launch_kernel(k_reach_expand, dim3(grid_of(n)), dim3(kBlock), 0, s, mark, n, dense,
                       orig, sub_block, block_out);
}

}  // namespace dfamin
