// Batched refinement of small DFAs inside single workgroups.
//
// One workgroup refines one job at a time: a DFA (minimisation) or the
// disjoint union of two DFAs (equivalence), with the whole signature loop of
// Section 3.3 (Algorithm 4: signature = own block id and the successors'
// block ids; equal signatures form the next blocks; stop when the block
// count does not grow) on the device.  Block ids and the grouping table sit
// in LDS, and the transitions too where they fit (16 bits a target), so
// every access of a round is an LDS access; rounds are separated by workgroup
// barriers, with no launch and no host round trip per round.  Workgroups take
// jobs from a counter, largest first.
//
// Bound by the longest job, a chain of rounds that each wait for LDS.  1,024
// threads and transitions in LDS, instead of 256 that read them from the L2,
// measured on MI355X: 589 DFAs of 64 to 4,096 states 198 -> 59 us, 272 pairs
// 550 -> 152 us.  Thousands of jobs of at most 1,024 states go to workgroups of
// 256 threads instead, six to a CU (kSmallFewJobs in api.hip).
//
// Ids inside a round are the index of the state that first claimed its
// signature's slot; the final ids are made canonical (smallest member) in
// LDS.  The round counts are those of plain signature rounds from the
// initial partition {F, Q \ F}, as in the segmented path; a pair stops at the
// round that separates its start states.
#include "device_common.h"

namespace dfamin {
namespace {

constexpr uint32_t kEpochBits = 4;
constexpr uint32_t kRoundsPerClear = (1u << kEpochBits) - 1;  // epochs 1 .. 15

__host__ __device__ __forceinline__ uint32_t small_table_slots(uint32_t n) {
    uint32_t t = 64;
    while (t < 2 * n) t <<= 1;
    return t;
}

template <int KC>
struct alignas(2 * KC) SmallRow {
    uint16_t t[KC];
};

// The transitions of a job's states, numbered in the union: in LDS, or read
// from the caller's arrays.  A target outside its DFA becomes the DFA's state
// 0 and sets `bad` (the call then fails; no access leaves the job's arrays);
// with fewer letters than KC the first one fills up.
template <int KC>
struct SmallRows {
    const SmallJob &J;
    const SmallRow<KC> *staged;  // nullptr: not in LDS

    __device__ __forceinline__ SmallRow<KC> load(uint32_t i, bool &bad) const {
        const bool in_b = i >= J.na;
        const uint32_t off = in_b ? J.na : 0u, lim = in_b ? J.nb : J.na;
        const uint32_t *r = (in_b ? J.delta_b : J.delta_a) + static_cast<size_t>(i - off) * J.k;
        uint32_t t[KC];
#pragma unroll
        for (int j = 0; j < KC; ++j) t[j] = r[j < static_cast<int>(J.k) ? j : 0];
        SmallRow<KC> row;
#pragma unroll
        for (int j = 0; j < KC; ++j) {
            const bool out = t[j] >= lim;
            bad |= out;
            row.t[j] = static_cast<uint16_t>(off + (out ? 0u : t[j]));
        }
        return row;
    }
    __device__ __forceinline__ SmallRow<KC> operator[](uint32_t i) const {
        bool bad = false;
        return staged ? staged[i] : load(i, bad);
    }
};

template <int KC, uint32_t NT>
__device__ __forceinline__ void small_job(const SmallJob &J, uint8_t *lds, uint32_t lds_bytes,
                                          uint32_t *claims, uint32_t max_rounds,
                                          uint32_t *out_blocks, SmallResult *results,
                                          uint32_t *err) {
    const uint32_t tx = threadIdx.x, n = J.na + J.nb, T = small_table_slots(n);
    // LDS: table (T words), two id arrays of n halves, the rows
    uint32_t *table = reinterpret_cast<uint32_t *>(lds);
    const uint32_t halves = (n + 7) & ~7u;
    uint16_t *ida = reinterpret_cast<uint16_t *>(table + T);
    uint16_t *idb = ida + halves;
    SmallRow<KC> *rows = reinterpret_cast<SmallRow<KC> *>(idb + halves);
    const bool staged = 4 * T + 4 * halves + n * sizeof(SmallRow<KC>) <= lds_bytes;
    const SmallRows<KC> R{J, staged ? rows : nullptr};
    bool bad = false, acc = false, rej = false;
    for (uint32_t i = tx; i < n; i += NT) {
        const SmallRow<KC> row = R.load(i, bad);
        if (staged) rows[i] = row;
        const bool f = (i < J.na ? J.acc_a[i] : J.acc_b[i - J.na]) != 0;
        ida[i] = f ? 1 : 0;
        acc |= f;
        rej |= !f;
    }
    for (uint32_t s = tx; s < T; s += NT) table[s] = 0;
    if (tx == 0) claims[0] = claims[1] = 0;
    uint32_t prev = (__syncthreads_or(acc) ? 1u : 0u) + (__syncthreads_or(rej) ? 1u : 0u);
    if (__syncthreads_or(bad) && tx == 0) *err = 1u;
    uint16_t *cur = ida, *nxt = idb;
    uint32_t round = 0, changing = 0, limit = 0;
    for (;;) {
        // entry = (epoch:4 | tag:12 | representative:16); entries of older
        // epochs are empty, and the table is cleared when the epochs run out
        if (round && round % kRoundsPerClear == 0) {
            for (uint32_t s = tx; s < T; s += NT) table[s] = 0;
            __syncthreads();
        }
        const uint32_t epoch = round % kRoundsPerClear + 1;
        uint32_t mine = 0;
        for (uint32_t i = tx; i < n; i += NT) {
            const SmallRow<KC> row = R[i];
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
                    const SmallRow<KC> ro = R[o];
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
        uint16_t *sw = cur;
        cur = nxt;
        nxt = sw;
        // stable: the same partition as before, with state ids
        if (count == prev) break;
        prev = count;
        ++changing;
        // a pair is decided once its start states are separated (the
        // refinement never merges them again)
        if (J.nb && cur[J.start_a] != cur[J.na + J.start_b]) break;
        if (max_rounds && round >= max_rounds) {
            limit = 1;
            break;
        }
    }
    if (J.nb == 0) {
        // canonical ids (smallest member) in the table's words
        uint32_t *minof = table;
        for (uint32_t i = tx; i < n; i += NT) minof[i] = ~0u;
        __syncthreads();
        for (uint32_t i = tx; i < n; i += NT) atomicMin(minof + cur[i], i);
        __syncthreads();
        uint32_t *out = out_blocks + J.out;
        for (uint32_t i = tx; i < n; i += NT) out[i] = minof[cur[i]];
    }
    if (tx == 0) {
        SmallResult r;
        r.num_blocks = prev;
        r.rounds = round;
        r.changing = changing;
        r.verdict = J.nb ? (cur[J.start_a] == cur[J.na + J.start_b] ? 1u : 0u) : 0u;
        r.limit = limit;
        results[J.index] = r;
    }
    __syncthreads();
}

// (1,024 threads: registers for two workgroups a CU, with a few words spilled;
// small workgroups have six a CU without that)
template <uint32_t NT>
__global__ __launch_bounds__(NT, NT == kSmallThreads ? 8 : 1) void k_small_refine(const SmallJob *__restrict__ jobs,
                                                     uint32_t njobs, uint32_t *next_job,
                                                     uint32_t *out_blocks, SmallResult *results,
                                                     uint32_t max_rounds, uint32_t *err,
                                                     uint32_t lds_bytes) {
    extern __shared__ __align__(16) uint8_t lds[];
    __shared__ uint32_t job_id, claims[2];
    for (;;) {
        if (threadIdx.x == 0) job_id = atomicAdd(next_job, 1u);
        __syncthreads();
        const uint32_t j = job_id;
        __syncthreads();  // every thread has read job_id before it changes
        if (j >= njobs) return;
        const SmallJob J = jobs[j];
        if (J.k <= 2)
            small_job<2, NT>(J, lds, lds_bytes, claims, max_rounds, out_blocks, results, err);
        else if (J.k <= 4)
            small_job<4, NT>(J, lds, lds_bytes, claims, max_rounds, out_blocks, results, err);
        else if (J.k <= 8)
            small_job<8, NT>(J, lds, lds_bytes, claims, max_rounds, out_blocks, results, err);
        else
            small_job<16, NT>(J, lds, lds_bytes, claims, max_rounds, out_blocks, results, err);
    }
}

__global__ void k_small_reset(uint32_t *next_job, uint32_t *err) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        next_job[0] = next_job[1] = 0;
        *err = 0;
    }
}

}  // namespace

uint32_t small_refine_lds_bytes(uint32_t n) {
    return small_table_slots(n) * 4u + 2u * ((n + 7) & ~7u) * 2u;
}

uint32_t small_rows_lds_bytes(uint32_t n, uint32_t k) {
    return n * 2u * (k <= 2 ? 2u : k <= 4 ? 4u : k <= 8 ? 8u : 16u);
}

int small_refine_max_groups(uint32_t threads, uint32_t lds_bytes, int device_cus) {
    int per_cu = 0;
    const hipError_t e =
        threads == kSmallThreads
            ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_small_refine<kSmallThreads>,
                                                           kSmallThreads, lds_bytes)
            : hipOccupancyMaxActiveBlocksPerMultiprocessor(
                  &per_cu, k_small_refine<kSmallFewThreads>, kSmallFewThreads, lds_bytes);
    return e == hipSuccess && per_cu > 0 ? per_cu * device_cus : 0;
}

void launch_small_reset(uint32_t *next_job, uint32_t *err, hipStream_t s) {
    launch_kernel(k_small_reset, dim3(1), dim3(64), 0, s, next_job, err);
}

void launch_small_refine(const SmallJob *jobs, uint32_t njobs, uint32_t threads, uint32_t groups,
                         uint32_t lds_bytes, uint32_t *next_job, uint32_t *out_blocks, SmallResult *results,
                         uint32_t max_rounds, uint32_t *err, hipStream_t s) {
    if (threads == kSmallThreads)
        launch_kernel(k_small_refine<kSmallThreads>, dim3(groups), dim3(kSmallThreads), lds_bytes,
                      s, jobs, njobs, next_job, out_blocks, results, max_rounds, err, lds_bytes);
    else
        launch_kernel(k_small_refine<kSmallFewThreads>, dim3(groups), dim3(kSmallFewThreads),
                      lds_bytes, s, jobs, njobs, next_job, out_blocks, results, max_rounds, err,
                      lds_bytes);
}

}  // namespace dfamin
