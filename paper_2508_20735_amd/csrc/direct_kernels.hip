// Signature rounds of ordinary-sized refinements: one launch per round.
//
// A refinement of up to some hundred thousand states is bound by launches,
// not by memory: its ids and table sit in L2, a kernel that does nothing
// takes 4.5 us of the stream, and the general path spends four kernels on a
// round (marking, signatures, grouping, round end), three more to lay the
// transitions out symbol-major, and a host wait for the letters' flags.
// Here a round is one kernel:
//   - it reads the transition rows straight from the caller's row-major
//     arrays (of one DFA, or of the two operands of a union),
//   - it groups the states of a workgroup in an LDS table by their keys, and
//     one state per local group in the HBM table; the key of the table's
//     representative is computed again from the round's ids, which do not
//     change during the round, so no key is ever written to memory,
//   - a state alone in its block after the round before keeps its id,
//   - the block count goes to a counter of the round; the next round reads
//     the last two and does nothing if they agree (stable) or an earlier
//     round stopped, or if an equivalence's start states have separated.
// k_direct_end turns the counters into the round state that the general path
// keeps, so that a refinement that is not stable after these rounds goes on
// there.  Keys are always compared in full, so grouping is exact.
//
// Measured on MI355X, a round of 100,000 states with 4 letters: 20 us in four
// launches before, 8 us here.
#include "device_common.h"

namespace dfamin {
namespace {

constexpr unsigned long long kEmptyLds = ~0ull;
constexpr uint32_t kDirectLds = 2 * kBlock;  // LDS table slots (load <= 1/2)
constexpr uint64_t kDirectEagerEdges = uint64_t(1) << 19;

// The ids a round starts from: the acceptance of the state in the first
// round, the last round's block ids afterwards.
template <int KC, bool FIRST>
struct Keys {
    const DirectArgs &a;
    const uint32_t *X;

    // State q's row, the number of states of its operand and their offset.
    __device__ __forceinline__ const uint32_t *row(uint32_t q, uint32_t &n, uint32_t &off) const {
        const bool in_b = q >= a.na;
        n = in_b ? a.nb : a.na;
        off = in_b ? a.na : 0u;
        return (in_b ? a.db : a.da) + static_cast<size_t>(q - off) * a.k;
    }
    // Targets of q, numbered in the union; one outside its operand becomes
    // the operand's first state and sets `bad` (the call then fails).  With
    // fewer letters than KC the first one fills up (a repeated key component
    // changes no comparison, and loads without branches stay in flight
    // together).
    __device__ __forceinline__ void targets(uint32_t q, uint32_t *t, bool &bad) const {
        uint32_t n, off;
        const uint32_t *r = row(q, n, off);
        if (KC % 4 == 0 && a.wide) {  // (k == KC)
#pragma unroll
            for (int j = 0; j < KC; j += 4) {
                const uint4 v = *reinterpret_cast<const uint4 *>(r + j);
                t[j] = v.x;
                t[j + 1] = v.y;
                t[j + 2] = v.z;
                t[j + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < KC; ++j) t[j] = r[j < static_cast<int>(a.k) ? j : 0];
        }
#pragma unroll
        for (int j = 0; j < KC; ++j) {
            const bool out = t[j] >= n;
            bad |= out;
            t[j] = off + (out ? 0u : t[j]);
        }
    }
    __device__ __forceinline__ uint32_t id(uint32_t q) const {
        if constexpr (FIRST)
            return (q >= a.na ? a.ab[q - a.na] : a.aa[q]) != 0 ? 1u : 0u;
        else
            return X[q];
    }
    __device__ __forceinline__ void ids(const uint32_t *t, uint32_t *w) const {
#pragma unroll
        for (int j = 0; j < KC; ++j) w[j] = id(t[j]);
    }
    // Whether state q's key is (w0, w).
    __device__ __forceinline__ bool equal(uint32_t q, uint32_t w0, const uint32_t *w) const {
        uint32_t t[KC], v[KC];
        bool bad = false;
        const uint32_t v0 = id(q);
        targets(q, t, bad);
        ids(t, v);
        bool eq = v0 == w0;
#pragma unroll
        for (int j = 0; j < KC; ++j) eq &= v[j] == w[j];
        return eq;
    }
};

// Sum of the 16 counters of a slot: every lane of the wave gets it.
__device__ __forceinline__ unsigned long long slot_sum(const DirectArgs &a, uint32_t slot) {
    const unsigned long long v =
        lane_id() < kDirectSpread ? a.cnt[(slot * kDirectSpread + lane_id()) * kDirectStride] : 0ull;
    uint32_t lo = static_cast<uint32_t>(v), hi = static_cast<uint32_t>(v >> 32);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        lo += __shfl_xor(lo, d, 64);
        hi += __shfl_xor(hi, d, 64);
    }
    return (static_cast<unsigned long long>(hi) << 32) | lo;
}

// Blocks when round r starts (the acceptance classes before round 0); 0 if
// the round before it did not run.
__device__ __forceinline__ uint32_t blocks_before(const DirectArgs &a, uint32_t r) {
    if (r == 0) return (a.flags[1] ? 1u : 0u) + (a.flags[2] ? 1u : 0u);
    return static_cast<uint32_t>(slot_sum(a, r - 1));
}

template <int KC, bool FIRST>
__global__ __launch_bounds__(kBlock) void k_direct_round(DirectArgs a, uint32_t r) {
    __shared__ unsigned long long ltab[kDirectLds];
    __shared__ uint32_t lkey[kBlock * (KC + 1)];
    __shared__ uint32_t gid[kBlock];
    __shared__ uint32_t lsize[kBlock];
    __shared__ uint32_t part[kBlock / 64];
    const uint32_t tx = threadIdx.x;
    const uint32_t *__restrict__ X = (r & 1u) ? a.blockB : a.blockA;
    uint32_t *__restrict__ Y = (r & 1u) ? a.blockA : a.blockB;
    const Keys<KC, FIRST> K{a, X};
    const uint32_t q = blockIdx.x * kBlock + tx;
    const bool valid = q < a.N;
    const uint32_t qs = valid ? q : 0u;  // (idle lanes read the first state)
    // Small rounds are a chain of dependent loads: everything that the round
    // may need is loaded before the stop test, which would add its own two in
    // front.  Larger ones test first and read the rows of refined states only
    // (rounds of 300,007 states with 16 letters that have nothing to do: 24 us
    // the first way, 5 the second).
    const bool eager = FIRST || static_cast<uint64_t>(a.N) * a.k <= kDirectEagerEdges;
    auto stopped = [&]() -> bool {  // (uniform over the grid)
        const uint32_t now = blocks_before(a, r), last = blocks_before(a, r - 1);
        return now == 0 || now == last || (a.check_eq && X[a.eq_a] != X[a.eq_b]);
    };
    if constexpr (!FIRST) {
        if (!eager && stopped()) return;
    }
    const uint32_t w0 = K.id(qs);
    uint32_t t[KC], w[KC];
    bool bad = false;
    // a block of one member after the last round stays one (its id is the
    // state itself)
    bool act = valid;
    if constexpr (!FIRST) act = valid && (w0 != q || a.multi[qs] == r);
    if (eager || act) {
        K.targets(qs, t, bad);
        K.ids(t, w);
    }
    if constexpr (!FIRST) {
        if (eager && stopped()) return;
    }
    for (uint32_t i = tx; i < kDirectLds; i += kBlock) ltab[i] = kEmptyLds;
    lsize[tx] = 0;
    uint64_t h = 0;
    uint32_t moves = 0;  // letters that move the state
    if (act) {
        if constexpr (FIRST) {
#pragma unroll
            for (int j = 0; j < KC; ++j) moves |= t[j] != q ? 1u << j : 0u;
        }
        h = mix_step(kHashSeed, w0);
        lkey[tx * (KC + 1)] = w0;
#pragma unroll
        for (int j = 0; j < KC; ++j) {
            lkey[tx * (KC + 1) + 1 + j] = w[j];
            h = mix_step(h, w[j]);
        }
        h = mix_final(h);
    }
    if constexpr (FIRST) {
        wave_set_flag(a.flags + 0, valid && bad);
        wave_set_flag(a.flags + 1, valid && w0 != 0);
        wave_set_flag(a.flags + 2, valid && w0 == 0);
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) moves |= __shfl_xor(moves, d, 64);
        // (plain loads: a stale zero only repeats the store)
        if (lane_id() < a.k && ((moves >> lane_id()) & 1u) && a.flags[3 + lane_id()] == 0u)
            a.flags[3 + lane_id()] = 1u;
    }
    __syncthreads();
    // the workgroup's states by key
    uint32_t lead = tx;
    if (act) {
        const uint32_t ltag = static_cast<uint32_t>(h >> 32);
        uint32_t s = static_cast<uint32_t>(h) & (kDirectLds - 1);
        for (;;) {
            unsigned long long e =
                __hip_atomic_load(ltab + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (e == kEmptyLds) {
                const unsigned long long want = (static_cast<unsigned long long>(ltag) << 32) | tx;
                const unsigned long long prev = atomicCAS(ltab + s, kEmptyLds, want);
                if (prev == kEmptyLds) break;
                e = prev;
            }
            if (static_cast<uint32_t>(e >> 32) == ltag) {
                const uint32_t o = static_cast<uint32_t>(e);
                bool eq = lkey[o * (KC + 1)] == w0;
#pragma unroll
                for (int j = 0; j < KC; ++j) eq &= lkey[o * (KC + 1) + 1 + j] == w[j];
                if (eq) {
                    lead = o;
                    break;
                }
            }
            s = (s + 1) & (kDirectLds - 1);
        }
        if (lead != tx) lsize[lead] = 1;  // (every writer stores the same)
    }
    __syncthreads();
    // one state per local group in the HBM table: entry = (epoch:8 | tag:24)
    // << 32 | representative, as in the general path (the table is never more
    // than half full, so a probe always reaches an empty slot).  Probes may
    // read a cached, older value: a slot only changes from empty to its final
    // value within a round, and the CAS on a stale empty one fails and
    // returns the value stored.
    bool claimed = false;
    if (act && lead == tx) {
        const uint32_t epoch = r + 1;
        const uint32_t tag = (epoch << 24) | static_cast<uint32_t>(h >> 40);
        const unsigned long long want = (static_cast<unsigned long long>(tag) << 32) | q;
        uint64_t s = h & a.mask;
        unsigned long long e =
            __hip_atomic_load(a.table + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        uint32_t id;
        for (;;) {
            if (static_cast<uint32_t>(e >> 56) != epoch) {
                const unsigned long long prev = atomicCAS(a.table + s, e, want);
                if (prev == e) {
                    claimed = true;
                    id = q;
                    break;
                }
                e = prev;
                continue;
            }
            if (static_cast<uint32_t>(e >> 32) == tag && K.equal(static_cast<uint32_t>(e), w0, w)) {
                id = static_cast<uint32_t>(e);
                break;
            }
            s = (s + 1) & a.mask;
            e = __hip_atomic_load(a.table + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
        gid[tx] = id;
        if (!claimed || lsize[tx]) mark_multi(a.multi, id, r + 1);
    }
    __syncthreads();
    if (valid) Y[q] = act ? gid[lead] : q;
    // blocks (claims and kept singletons) and refined states of the round:
    // at most kBlock each, summed together
    uint32_t v = (claimed || (valid && !act) ? 1u : 0u) | (act ? 1u << 16 : 0u);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    if (lane_id() == 0) part[tx / 64] = v;
    __syncthreads();
    if (tx == 0) {
        uint32_t sum = 0;
#pragma unroll
        for (int i = 0; i < kBlock / 64; ++i) sum += part[i];
        atomicAdd(a.cnt + (r * kDirectSpread + blockIdx.x % kDirectSpread) * kDirectStride,
                  (static_cast<unsigned long long>(sum >> 16) << 32) | (sum & 0xFFFFu));
    }
}

// One workgroup: the round state after the rounds that ran, of `launched`.
__global__ __launch_bounds__(kBlock) void k_direct_end(DirectArgs a, uint32_t launched) {
    static_assert(kDirectMaxRounds * kDirectSpread == kBlock, "one counter per thread");
    __shared__ uint32_t count[kDirectMaxRounds], refined[kDirectMaxRounds];
    RoundCtl *ctl = a.ctl;
    const unsigned long long v = a.cnt[threadIdx.x * kDirectStride];
    uint32_t c = static_cast<uint32_t>(v), act = static_cast<uint32_t>(v >> 32);
#pragma unroll
    for (int d = kDirectSpread / 2; d >= 1; d >>= 1) {
        c += __shfl_xor(c, d, 64);
        act += __shfl_xor(act, d, 64);
    }
    if (threadIdx.x % kDirectSpread == 0) {
        count[threadIdx.x / kDirectSpread] = c;
        refined[threadIdx.x / kDirectSpread] = act;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    uint32_t rounds = 0, changing = 0, prev = (a.flags[1] ? 1u : 0u) + (a.flags[2] ? 1u : 0u);
    uint32_t stable = 0, gain = 0;
    unsigned long long active = 0;
    // (a round that did not run counted no block)
    for (; rounds < launched && count[rounds]; ++rounds) {
        gain = count[rounds] - prev;
        prev = count[rounds];
        stable = gain == 0 ? 1u : 0u;
        changing += stable ? 0u : 1u;
        active += refined[rounds];
        ctl->gain_hist[rounds % kActiveHist] = gain;
        ctl->active_hist[rounds % kActiveHist] = refined[rounds];
    }
    const uint32_t *ids = ((rounds - 1) & 1u) ? a.blockA : a.blockB;
    const uint32_t separated = a.check_eq && ids[a.eq_a] != ids[a.eq_b] ? 1u : 0u;
    ctl->round = rounds;
    ctl->prev_count = prev;
    ctl->last_gain = gain;
    ctl->last_active = rounds ? refined[rounds - 1] : 0;
    ctl->changing = changing;
    ctl->stable = stable;
    ctl->separated = separated;
    // (a bad target: nothing that follows may use the targets)
    ctl->done = a.flags[0] ? 0u : stable | separated;
    ctl->limit = 0;
    ctl->max_rounds = 0;
    ctl->eq_a = a.eq_a;
    ctl->eq_b = a.eq_b;
    ctl->check_eq = a.check_eq;
    ctl->pattern_first = 0;
    ctl->packed_second = 0;
    ctl->all_active_until = 0;
    // the next round refines every state of a multi-state block
    ctl->full_until = rounds;
    ctl->last_changed = a.N;
    ctl->last_claims = 0;
    ctl->active_sum = active;
    ctl->pb_rounds = 0;
    ctl->part_rounds = 0;
}

// The general path goes on after `rounds` rounds: the singleton bits, and as
// the states refined in the round before just those singletons, whose ids it
// then copies to the other block buffer (which may still hold older ones).
__global__ __launch_bounds__(kBlock) void k_direct_singles(DirectArgs a, uint32_t rounds,
                                                           unsigned long long *single,
                                                           unsigned long long *active) {
    const uint32_t *ids = ((rounds - 1) & 1u) ? a.blockA : a.blockB;
    const uint32_t q = blockIdx.x * kBlock + threadIdx.x;
    const bool s = q < a.N && ids[q] == q && a.multi[q] != rounds;
    const unsigned long long m = __ballot(s);
    if (lane_id() == 0 && q < a.N) {
        single[q >> 6] = m;
        active[q >> 6] = m;
    }
}

// Canonical ids of a refinement that direct rounds have decided, queued
// behind them before the host knows (nothing to do if they have not).
__global__ __launch_bounds__(kBlock) void k_direct_canon(DirectArgs a, uint32_t *maxs) {
    if (!a.ctl->done) return;
    const uint32_t *__restrict__ ids = ((a.ctl->round - 1) & 1u) ? a.blockA : a.blockB;
    const uint32_t q = blockIdx.x * kBlock + threadIdx.x;
    if (q < a.N) atomicMax(maxs + ids[q], ~q);
}

__global__ __launch_bounds__(kScanTile) void k_direct_leaders(DirectArgs a, const uint32_t *maxs,
                                                              uint32_t *__restrict__ out,
                                                              uint32_t *partials) {
    __shared__ uint32_t wsum[kScanTile / 64];
    if (!a.ctl->done) return;
    const uint32_t *__restrict__ ids = ((a.ctl->round - 1) & 1u) ? a.blockA : a.blockB;
    const uint32_t q = blockIdx.x * kScanTile + threadIdx.x;
    uint32_t b = ~0u;
    if (q < a.N) {
        b = ~maxs[ids[q]];
        out[q] = b;
    }
    const unsigned long long m = __ballot(q < a.N && b == q);
    if (lane_id() == 0) wsum[threadIdx.x / 64] = static_cast<uint32_t>(__popcll(m));
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t sum = 0;
        for (uint32_t i = 0; i < kScanTile / 64; ++i) sum += wsum[i];
        partials[blockIdx.x] = sum;
    }
}

template <int KC>
void direct_round(const DirectArgs &a, uint32_t r, hipStream_t s) {
    const dim3 grid((a.N + kBlock - 1) / kBlock), block(kBlock);
    if (r == 0)
        launch_kernel(k_direct_round<KC, true>, grid, block, 0, s, a, r);
    else
        launch_kernel(k_direct_round<KC, false>, grid, block, 0, s, a, r);
}

}  // namespace

void launch_direct_round(const DirectArgs &a, uint32_t r, hipStream_t s) {
    switch (direct_width(a.k)) {
        case 1: direct_round<1>(a, r, s); break;
        case 2: direct_round<2>(a, r, s); break;
        case 4: direct_round<4>(a, r, s); break;
        case 8: direct_round<8>(a, r, s); break;
        default: direct_round<16>(a, r, s); break;
    }
}

void launch_direct_end(const DirectArgs &a, uint32_t launched, hipStream_t s) {
    launch_kernel(k_direct_end, dim3(1), dim3(kBlock), 0, s, a, launched);
}

void launch_direct_canonical(const DirectArgs &a, uint32_t *scratch_max, uint32_t *out,
                             uint32_t *partials, hipStream_t s) {
    launch_kernel(k_direct_canon, dim3((a.N + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a,
                  scratch_max);
    launch_kernel(k_direct_leaders, dim3((a.N + kScanTile - 1) / kScanTile), dim3(kScanTile), 0, s,
                  a, static_cast<const uint32_t *>(scratch_max), out, partials);
}

void launch_direct_singles(const DirectArgs &a, uint32_t rounds, unsigned long long *single,
                           unsigned long long *active, hipStream_t s) {
    launch_kernel(k_direct_singles, dim3((a.N + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a,
                  rounds, single, active);
}

}  // namespace dfamin
