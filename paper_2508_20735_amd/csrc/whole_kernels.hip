// A small refinement whole inside one workgroup, for calls on one DFA or one
// pair (the batched calls run many of them, batch_kernels.hip).
//
// A DFA of a few thousand states has no work for a device; its call is a
// chain of launches and host waits.  Here one workgroup of 1,024 threads
// keeps everything in LDS: the transitions (16-bit), two id arrays (16-bit)
// and the grouping table, so every access of a round is an LDS access and a
// round costs two barriers.  The same launch writes the canonical ids and the
// quotient, and its figures go to page-locked host memory, so the call is
// one launch and one wait.  Measured on MI355X, a call that minimises 1,009
// states, 4 letters, with the quotient: 116 us with a launch per round, 43 us
// here (20 of them in the kernel).
//
// Rounds are those of Section 3.3, Algorithm 4, as in the other paths; keys
// are compared in full.  A refinement that is not decided after max_rounds
// rounds (a chain) leaves no result: the caller takes another path.
#include "device_common.h"

namespace dfamin {
namespace {

constexpr uint32_t kWaves = kWholeThreads / 64;
constexpr uint32_t kEpochBits = 4;
constexpr uint32_t kRoundsPerClear = (1u << kEpochBits) - 1;  // epochs 1 .. 15

// Exclusive prefix sum over the workgroup's threads; `total` = the sum.
__device__ __forceinline__ uint32_t wg_prefix(uint32_t v, uint32_t *red, uint32_t &total) {
    uint32_t x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, 64);
        if (lane_id() >= static_cast<uint32_t>(d)) x += y;
    }
    __syncthreads();  // the last use of red is over
    if (lane_id() == 63) red[threadIdx.x / 64] = x;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) {
        before += w < threadIdx.x / 64 ? red[w] : 0u;
        total += red[w];
    }
    return before + x - v;
}

// A row of KC 16-bit targets in LDS, read in one piece.
template <int KC>
struct alignas(2 * KC) Row {
    uint16_t t[KC];
};

template <int KC>
__global__ __launch_bounds__(kWholeThreads) void k_whole(WholeArgs a) {
    extern __shared__ __align__(16) uint8_t lds[];
    __shared__ uint32_t red[kWaves];
    __shared__ uint32_t claims[2], moved;
    const uint32_t tx = threadIdx.x;
    const unsigned long long t0 = wall_clock64();
    const uint32_t n = a.na + a.nb, k = a.k;
    const uint32_t T = a.slots;
    uint32_t *table = reinterpret_cast<uint32_t *>(lds);
    Row<KC> *rows = reinterpret_cast<Row<KC> *>(table + T);
    uint16_t *ida = reinterpret_cast<uint16_t *>(rows + n);
    uint16_t *idb = ida + n;
    // transitions (numbered in the union; a target outside its operand
    // becomes the operand's first state and fails the call), acceptance
    bool bad = false, acc = false, rej = false;
    uint32_t moves = 0;
    for (uint32_t i = tx; i < n; i += kWholeThreads) {
        const bool in_b = i >= a.na;
        const uint32_t off = in_b ? a.na : 0u, lim = in_b ? a.nb : a.na;
        const uint32_t *r = (in_b ? a.db : a.da) + static_cast<size_t>(i - off) * k;
        uint32_t t[KC];
        if (KC % 4 == 0 && a.wide) {  // (k == KC)
#pragma unroll
            for (int j = 0; j < KC; j += 4) {
                const uint4 v = *reinterpret_cast<const uint4 *>(r + j);
                t[j] = v.x;
                t[j + 1] = v.y;
                t[j + 2] = v.z;
                t[j + 3] = v.w;
            }
        } else {  // (fewer letters than KC: the first one fills up)
#pragma unroll
            for (int j = 0; j < KC; ++j) t[j] = r[j < static_cast<int>(k) ? j : 0];
        }
        const bool f = (in_b ? a.ab[i - off] : a.aa[i]) != 0;
        Row<KC> row;
#pragma unroll
        for (int j = 0; j < KC; ++j) {
            const bool out = t[j] >= lim;
            bad |= out;
            const uint32_t g = off + (out ? 0u : t[j]);
            row.t[j] = static_cast<uint16_t>(g);
            moves |= g != i ? 1u << j : 0u;
        }
        rows[i] = row;
        ida[i] = f ? 1 : 0;
        acc |= f;
        rej |= !f;
    }
    for (uint32_t s = tx; s < T; s += kWholeThreads) table[s] = 0;
    if (tx == 0) {
        claims[0] = claims[1] = 0;
        moved = 0;
    }
    uint32_t prev = (__syncthreads_or(acc) ? 1u : 0u) + (__syncthreads_or(rej) ? 1u : 0u);
    const bool failed = __syncthreads_or(bad) != 0;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) moves |= __shfl_xor(moves, d, 64);
    if (lane_id() == 0 && moves) atomicOr(&moved, moves);
    uint16_t *cur = ida, *nxt = idb;
    uint32_t round = 0, changing = 0;
    bool stable = false, separated = false;
    while (!failed && !stable && !separated && round < a.max_rounds) {
        // entry = (epoch:4 | tag:12 | representative:16); entries of older
        // epochs are empty, and the table is cleared when the epochs run out
        if (round && round % kRoundsPerClear == 0) {
            for (uint32_t s = tx; s < T; s += kWholeThreads) table[s] = 0;
            __syncthreads();
        }
        const uint32_t epoch = round % kRoundsPerClear + 1;
        uint32_t mine = 0;
        for (uint32_t i = tx; i < n; i += kWholeThreads) {
            const Row<KC> row = rows[i];
            const uint32_t w0 = cur[i];
            uint32_t w[KC];
#pragma unroll
            for (int j = 0; j < KC; ++j) w[j] = cur[row.t[j]];
            uint64_t h = mix_step(kHashSeed, w0);
#pragma unroll
            for (int j = 0; j < KC; ++j) h = mix_step(h, w[j]);
            h = mix_final(h);
            const uint32_t tag = (epoch << 12) | static_cast<uint32_t>(h >> 52);
            const uint32_t want = (tag << 16) | i;
            uint32_t s = static_cast<uint32_t>(h) & (T - 1);
            uint32_t id = i;
            uint32_t e =
                __hip_atomic_load(table + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            // (at least half of the slots stay empty: the probe ends)
            for (;;) {
                if ((e >> (32 - kEpochBits)) != epoch) {
                    const uint32_t was = atomicCAS(table + s, e, want);
                    if (was == e) {
                        ++mine;
                        break;
                    }
                    e = was;
                    continue;
                }
                if ((e >> 16) == tag) {
                    const uint32_t o = e & 0xFFFFu;
                    const Row<KC> ro = rows[o];
                    bool eq = cur[o] == w0;
#pragma unroll
                    for (int j = 0; j < KC; ++j) eq &= cur[ro.t[j]] == w[j];
                    if (eq) {
                        id = o;
                        break;
                    }
                }
                s = (s + 1) & (T - 1);
                e = __hip_atomic_load(table + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            nxt[i] = static_cast<uint16_t>(id);
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) mine += __shfl_xor(mine, d, 64);
        if (lane_id() == 0 && mine) atomicAdd(claims + (round & 1u), mine);
        __syncthreads();  // ids and count of the round
        const uint32_t count = claims[round & 1u];
        // the next round's counter: last read before the barrier of this
        // round, next added to after the barrier below
        if (tx == 0) claims[(round + 1) & 1u] = 0;
        __syncthreads();
        ++round;
        stable = count == prev;
        changing += stable ? 0u : 1u;
        prev = count;
        uint16_t *sw = cur;
        cur = nxt;
        nxt = sw;
        separated = a.nb && cur[a.eq_a] != cur[a.eq_b];
    }
    if (tx == 0) {
        WholeResult r{};
        r.err = failed ? 1u : 0u;
        r.done = stable || separated ? 1u : 0u;
        r.rounds = round;
        r.changing = changing;
        r.blocks = prev;
        r.separated = separated ? 1u : 0u;
        r.stable = stable ? 1u : 0u;
        r.moves = moved;
        r.ticks = wall_clock64() - t0;
        *a.result = r;
    }
    if (failed || a.nb || !stable) return;  // (uniform)
    // canonical ids: the smallest member, in the table's words
    __syncthreads();
    uint32_t *minof = table;
    for (uint32_t i = tx; i < n; i += kWholeThreads) minof[i] = ~0u;
    __syncthreads();
    for (uint32_t i = tx; i < n; i += kWholeThreads) atomicMin(minof + cur[i], i);
    __syncthreads();
    uint16_t *canon = nxt;
    for (uint32_t i = tx; i < n; i += kWholeThreads) {
        const uint32_t b = minof[cur[i]];
        canon[i] = static_cast<uint16_t>(b);
        a.block_out[i] = b;
    }
    if (!a.qdelta) {
        if (tx == 0) a.result->ticks = wall_clock64() - t0;
        return;
    }
    // dense numbers of the leaders (dense = cur's words), and the leaders in
    // order (lead_of: in the table's second half, T >= 2n)
    __syncthreads();
    uint16_t *dense = cur;
    uint16_t *lead_of = reinterpret_cast<uint16_t *>(table + n);
    uint32_t base = 0;
    for (uint32_t i0 = 0; i0 < n; i0 += kWholeThreads) {
        const uint32_t i = i0 + tx;
        const bool lead = i < n && canon[i] == i;
        uint32_t total;
        const uint32_t d = base + wg_prefix(lead ? 1u : 0u, red, total);
        if (lead) {
            dense[i] = static_cast<uint16_t>(d);
            lead_of[d] = static_cast<uint16_t>(i);
        }
        base += total;
    }
    __syncthreads();
    const uint32_t entries = base * k;
    for (uint32_t e = tx; e < entries; e += kWholeThreads) {
        const uint32_t b = e / k, j = e - b * k;
        const uint32_t l = lead_of[b];
        a.qdelta[e] = dense[canon[rows[l].t[j]]];
        if (j == 0) a.qacc[b] = a.aa[l] ? 1 : 0;
    }
    if (tx == 0) {
        a.result->qstart = dense[canon[a.start]];
        a.result->ticks = wall_clock64() - t0;
    }
}

}  // namespace

uint32_t whole_lds_bytes(uint32_t n, uint32_t k) {
    return whole_slots(n) * 4u + n * (2u * direct_width(k) + 4u);
}

void launch_whole(const WholeArgs &a, hipStream_t s) {
    const uint32_t lds = whole_lds_bytes(a.na + a.nb, a.k);
    const dim3 grid(1), block(kWholeThreads);
    switch (direct_width(a.k)) {
        case 1: launch_kernel(k_whole<1>, grid, block, lds, s, a); break;
        case 2: launch_kernel(k_whole<2>, grid, block, lds, s, a); break;
        case 4: launch_kernel(k_whole<4>, grid, block, lds, s, a); break;
        case 8: launch_kernel(k_whole<8>, grid, block, lds, s, a); break;
        default: launch_kernel(k_whole<16>, grid, block, lds, s, a); break;
    }
}

}  // namespace dfamin
