// Batched refinement, one launch per round: many DFAs (or equivalence pairs)
// refined side by side, each a segment with blocks, counts and a verdict of
// its own.  The rounds are those of the direct kernels (direct_kernels.hip):
// a state's key is computed from the caller's row and the last round's ids
// and never stored, a workgroup groups its tile in LDS and then one state per
// local group in a table in memory.  What the segments add:
//   - every DFA starts at a multiple of the tile, so a workgroup's states
//     belong to one DFA: its row pointer, letters and segment are uniform;
//   - every segment has a table of its own, so the accesses of a tile fall
//     into the few hundred kilobytes of ids, marks and table of its segment,
//     and a contiguous eighth of the tiles goes to each XCD, whose L2 then
//     holds them;
//   - a segment's block count goes to a ring of four counters; a round that
//     finds the last two equal (stable), or a pair's start states separated,
//     does nothing for the segment, and the segment's first tile records it.
//     A decided segment costs its tiles three loads a round, one behind the
//     other: the tile's part, its segment, the segment's end.
//
// Table entries carry a 20-bit epoch that the workspace counts on from call
// to call, so the tables are cleared once in a million rounds.
//
// Bound by L2 requests and, where most keys differ, by the atomics of the
// table.  Measured on MI355X, 1,024 random DFAs of 64 to 65,536 states and 2 to
// 8 letters, 9.87 million states in the segments: the call takes 2.83 ms, 3.81
// in the general path's five passes over signature rows; 512 pairs 6.17 ms,
// 7.29.  Batches whose parts have at most 65,536 states and 8 letters, and 896
// states on average, are faster with their ids in LDS (staged rounds, below);
// these rounds remain for the others.
#include "device_common.h"

namespace dfamin {
namespace {

constexpr unsigned long long kEmptyLds = ~0ull;
constexpr uint32_t kTileLds = 2 * kBlock;

// Whether segment s is decided when round r starts (r >= 1), and what it has
// then: blocks, and the rounds that changed its partition.
__device__ __forceinline__ bool segd_decided(const SegdArgs &a, const SegdSeg &S, uint32_t s,
                                             uint32_t r, const uint32_t *X, uint32_t &blocks,
                                             uint32_t &changing) {
    const uint32_t now = a.cnt[((r - 1) & 3u) * a.nseg + s];
    const uint32_t last = r == 1 ? static_cast<uint32_t>(__popc(a.classes[s]))
                                 : a.cnt[((r - 2) & 3u) * a.nseg + s];
    blocks = now;
    changing = now == last ? r - 1 : r;
    return now == last || (a.pairs && X[S.eq_a] != X[S.eq_b]);
}

__device__ __forceinline__ void segd_record(const SegdArgs &a, uint32_t s, uint32_t rounds,
                                            uint32_t blocks, uint32_t changing) {
    a.done[s] = rounds;
    a.blocks[s] = blocks;
    a.changing[s] = changing;
    atomicAdd(&a.ctl->ndone, 1u);
}

// The tile of this workgroup: workgroups go to the 8 XCDs round-robin, and
// each XCD takes a contiguous eighth (the grid is a multiple of 8).
__device__ __forceinline__ bool segd_tile(uint32_t tiles, uint32_t &tile) {
    const uint32_t x = blockIdx.x % 8, i = blockIdx.x / 8;
    const uint32_t lo = static_cast<uint32_t>(static_cast<uint64_t>(tiles) * x / 8);
    const uint32_t hi = static_cast<uint32_t>(static_cast<uint64_t>(tiles) * (x + 1) / 8);
    tile = lo + i;
    return tile < hi;
}

// Keys of the states of a segment: part P holds the tile's states, O the
// pair's other operand (P itself for a single DFA).
template <int KC, bool FIRST>
struct SegdKeys {
    const SegdPart &P, &O;
    const uint32_t *X;

    // (a target out of range becomes the DFA's first state and sets `bad`;
    // with fewer letters than KC the first one fills up)
    __device__ __forceinline__ void targets(uint32_t q, uint32_t *t, bool &bad) const {
        const bool own = q - P.off < P.n;
        const uint32_t n = own ? P.n : O.n, off = own ? P.off : O.off, k = P.k;
        const uint32_t *r = (own ? P.delta : O.delta) + static_cast<size_t>(q - off) * k;
        if (KC % 4 == 0 && (P.wide & O.wide)) {  // (k == KC)
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
            for (int j = 0; j < KC; ++j) t[j] = r[j < static_cast<int>(k) ? j : 0];
        }
#pragma unroll
        for (int j = 0; j < KC; ++j) {
            const bool out = t[j] >= n;
            bad |= out;
            t[j] = off + (out ? 0u : t[j]);
        }
    }
    __device__ __forceinline__ uint32_t id(uint32_t q) const {
        if constexpr (FIRST) {
            const bool own = q - P.off < P.n;
            return (own ? P.acc[q - P.off] : O.acc[q - O.off]) != 0 ? 1u : 0u;
        } else {
            return X[q];
        }
    }
    __device__ __forceinline__ void ids(const uint32_t *t, uint32_t *w) const {
#pragma unroll
        for (int j = 0; j < KC; ++j) w[j] = id(t[j]);
    }
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

template <int KMAX>
struct SegdLds {
    unsigned long long tab[kTileLds];
    uint32_t key[kBlock * (KMAX + 1)];
    uint32_t gid[kBlock];
    uint32_t shared[kBlock];  // another state of the tile has the key
    uint32_t part[kBlock / 64];
};

// One round of a tile (uniform: the whole workgroup).
template <int KC, int KMAX, bool FIRST>
__device__ __forceinline__ void segd_tile_round(const SegdArgs &a, const SegdPart &P,
                                                const SegdPart &O, const SegdSeg &S, uint32_t s,
                                                uint32_t tile, uint32_t r, uint32_t epoch,
                                                SegdLds<KMAX> &L) {
    const uint32_t tx = threadIdx.x;
    const uint32_t *__restrict__ X = (r & 1u) ? a.blockB : a.blockA;
    uint32_t *__restrict__ Y = (r & 1u) ? a.blockA : a.blockB;
    const SegdKeys<KC, FIRST> K{P, O, X};
    const uint32_t q = tile * kBlock + tx;
    const bool valid = q - P.off < P.n;
    const uint32_t qs = valid ? q : P.off;
    const uint32_t w0 = K.id(qs);
    uint32_t t[KC], w[KC];
    bool bad = false;
    // a block of one member after the last round stays one (its id is the
    // state itself)
    bool act = valid;
    if constexpr (!FIRST) act = valid && (w0 != q || a.multi[qs] == r);
    if (__syncthreads_or(act) == 0) {  // (the tile's states are all singletons)
        if (valid) Y[q] = q;
        if (tx == 0)
            atomicAdd(a.cnt + (r & 3u) * a.nseg + s, min(P.n - (tile * kBlock - P.off), kBlock + 0u));
        return;
    }
    if (act) {
        K.targets(qs, t, bad);
        K.ids(t, w);
    }
    for (uint32_t i = tx; i < kTileLds; i += kBlock) L.tab[i] = kEmptyLds;
    L.shared[tx] = 0;
    uint64_t h = 0;
    uint32_t moves = 0;  // letters that move the state
    if (act) {
        if constexpr (FIRST) {
#pragma unroll
            for (int j = 0; j < KC; ++j) moves |= t[j] != q ? 1u << j : 0u;
        }
        h = mix_step(kHashSeed, w0);
        L.key[tx * (KC + 1)] = w0;
#pragma unroll
        for (int j = 0; j < KC; ++j) {
            L.key[tx * (KC + 1) + 1 + j] = w[j];
            h = mix_step(h, w[j]);
        }
        h = mix_final(h);
    }
    if constexpr (FIRST) {
        wave_set_flag(&a.ctl->err, valid && bad);
        const uint32_t cls = (__ballot(valid && w0 != 0) ? 1u : 0u) | (__ballot(valid && w0 == 0) ? 2u : 0u);
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) moves |= __shfl_xor(moves, d, 64);
        moves &= (1u << P.k) - 1u;
        if (lane_id() == 0) {
            // (plain reads: an older value only repeats the atomic)
            if (cls & ~a.classes[s]) atomicOr(a.classes + s, cls);
            if (moves & ~a.ctl->moves) atomicOr(&a.ctl->moves, moves);
        }
    }
    __syncthreads();
    uint32_t lead = tx;
    if (act) {
        const uint32_t ltag = static_cast<uint32_t>(h >> 32);
        uint32_t sl = static_cast<uint32_t>(h) & (kTileLds - 1);
        for (;;) {
            unsigned long long e =
                __hip_atomic_load(L.tab + sl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (e == kEmptyLds) {
                const unsigned long long want = (static_cast<unsigned long long>(ltag) << 32) | tx;
                const unsigned long long prev = atomicCAS(L.tab + sl, kEmptyLds, want);
                if (prev == kEmptyLds) break;
                e = prev;
            }
            if (static_cast<uint32_t>(e >> 32) == ltag) {
                const uint32_t o = static_cast<uint32_t>(e);
                bool eq = L.key[o * (KC + 1)] == w0;
#pragma unroll
                for (int j = 0; j < KC; ++j) eq &= L.key[o * (KC + 1) + 1 + j] == w[j];
                if (eq) {
                    lead = o;
                    break;
                }
            }
            sl = (sl + 1) & (kTileLds - 1);
        }
        if (lead != tx) L.shared[lead] = 1;  // (every writer stores the same)
    }
    __syncthreads();
    // one state per local group in the segment's table: entry = (epoch:20 |
    // tag:12) << 32 | representative; entries of other epochs are empty, and
    // the table is never more than half full.  Probes may read a cached,
    // older value: within a round a slot changes once, from empty to its
    // final value, and the CAS on a stale empty one fails and returns it.
    bool claimed = false;
    if (act && lead == tx) {
        unsigned long long *table = a.table + S.table;
        const uint32_t tag = (epoch << 12) | static_cast<uint32_t>(h >> 52);
        const unsigned long long want = (static_cast<unsigned long long>(tag) << 32) | q;
        uint32_t sl = static_cast<uint32_t>(h) & S.mask;
        unsigned long long e =
            __hip_atomic_load(table + sl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        uint32_t id;
        for (;;) {
            if (static_cast<uint32_t>(e >> 44) != epoch) {
                const unsigned long long prev = atomicCAS(table + sl, e, want);
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
            sl = (sl + 1) & S.mask;
            e = __hip_atomic_load(table + sl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
        L.gid[tx] = id;
        if (!claimed || L.shared[tx]) mark_multi(a.multi, id, r + 1);
    }
    __syncthreads();
    if (valid) Y[q] = act ? L.gid[lead] : q;
    // blocks (claims and kept singletons) and refined states, summed together
    uint32_t v = (claimed || (valid && !act) ? 1u : 0u) | (act ? 1u << 16 : 0u);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    if (lane_id() == 0) L.part[tx / 64] = v;
    __syncthreads();
    if (tx == 0) {
        uint32_t sum = 0;
#pragma unroll
        for (int i = 0; i < kBlock / 64; ++i) sum += L.part[i];
        atomicAdd(a.cnt + (r & 3u) * a.nseg + s, sum & 0xFFFFu);
        atomicAdd(a.ctl->active + (blockIdx.x % kSegdSpread) * kSegdStride,
                  static_cast<unsigned long long>(sum >> 16));
    }
}

template <int KMAX, bool FIRST>
__global__ __launch_bounds__(kBlock) void k_segd_round(SegdArgs a, uint32_t r, uint32_t epoch) {
    __shared__ SegdLds<KMAX> L;
    uint32_t tile;
    if (!segd_tile(a.tiles, tile)) return;
    const uint32_t p = a.tile_part[tile];
    const SegdPart P = a.parts[p];
    const uint32_t s = P.seg;
    if constexpr (!FIRST) {
        if (a.done[s]) return;
    }
    const SegdSeg S = a.segs[s];
    const bool first_tile = tile == S.first_tile;
    if constexpr (!FIRST) {
        const uint32_t *X = (r & 1u) ? a.blockB : a.blockA;
        uint32_t blocks, changing;
        // (the same for every workgroup of the segment)
        if (segd_decided(a, S, s, r, X, blocks, changing)) {
            if (first_tile && threadIdx.x == 0) segd_record(a, s, r, blocks, changing);
            return;
        }
    }
    // the counter of the next round (last read two rounds ago)
    if (first_tile && threadIdx.x == 0) a.cnt[((r + 1) & 3u) * a.nseg + s] = 0;
    const SegdPart O = a.pairs ? a.parts[p ^ 1u] : P;
    if (P.k <= 2)
        segd_tile_round<2, KMAX, FIRST>(a, P, O, S, s, tile, r, epoch, L);
    else if (P.k <= 4)
        segd_tile_round<4, KMAX, FIRST>(a, P, O, S, s, tile, r, epoch, L);
    else if (KMAX == 8 || P.k <= 8)
        segd_tile_round<8, KMAX, FIRST>(a, P, O, S, s, tile, r, epoch, L);
    else if constexpr (KMAX > 8)
        segd_tile_round<16, KMAX, FIRST>(a, P, O, S, s, tile, r, epoch, L);
}

// ---------------------------------------------------------------- staged rounds
//
// Parts of up to 65,536 states, in two launches a round and with no access to
// a table in memory (an atomic to a random word costs the chip 1 / 14 G/s):
//   keys   a workgroup holds all the ids that its states' successors can have
//          in LDS (two bytes each), so the gathers are LDS accesses.  It
//          packs each refined state and its key into an entry of 17-bit
//          numbers (8 to 24 bytes), sorted by the key's bucket within groups
//          of 2,048 states, and stores the state as its own id;
//   groups a workgroup groups a bucket's entries, about 6,144 of them if the
//          keys differ, in an LDS table, and stores the id of the states that
//          found their key there.
// A workgroup of the first kind takes up to 8,192 states of a part, so that
// staging the ids (256 KB in a row) costs less than the gathers would (about
// one address a clock and CU).  A pair's ids need 17 bits if its union is
// larger than the window; the top bits then lie in an array of their own.
// A bucket's runs lie in the groups of its segment, so entries of one key can
// overflow nothing: they only make that bucket longer.
//
// Measured on MI355X (the batches above, whole calls): 2.83 -> 1.24 ms, and
// 6.17 -> 2.80 ms for the pairs.  A round that refines all 9.87 million states
// takes 147 + 153 us, the tile rounds' 988 us.  Of the keys' time a sixth is
// staging, the rest latency with one workgroup a CU (loading a group's rows
// while the one before it is sorted: 158 -> 147 us); more entries in flight in
// the groups' launch change nothing.
//
// Round 0 gathers acceptance bytes instead: a key is a pattern of letters + 1
// bits, grouped by direct index, in LDS and then (once per pattern) in a
// small table of the segment's.  It stores the targets in 16 bits for the
// later rounds.

// Marks the block of a state as one of several (read in the next round); the
// mark's eight bits make a block look shared again after 256 rounds, which
// only refines it once for nothing.
__device__ __forceinline__ void mark_shared(uint8_t *shared, uint32_t id, uint32_t tag) {
    if (shared[id] != (tag & 255u)) shared[id] = static_cast<uint8_t>(tag);
}

constexpr uint32_t kIdBits = 17;
constexpr uint32_t kIdMask = (1u << kIdBits) - 1;

// A row of 16-bit targets, padded to a power of two: one aligned access.
template <int K>
struct alignas(2 * (K <= 2 ? K : K <= 4 ? 4 : 8)) StagedRow {
    uint16_t t[K <= 2 ? K : K <= 4 ? 4 : 8];
};

template <int K>
__device__ __forceinline__ StagedRow<K> *staged_row(const SegdArgs &a, const SegdPart &P,
                                                    uint32_t q) {
    return reinterpret_cast<StagedRow<K> *>(a.rows + P.rows) + (q - P.off);
}

// A state and its key, 17 bits each; numbers count from the segment's start.
template <int K>
struct alignas(staged_words(K) == 4 ? 16 : staged_words(K) % 2 ? 4 : 8) StagedEntry {
    static constexpr int W = staged_words(K);
    uint32_t w[W];

    template <int I>
    __device__ __forceinline__ void put(uint32_t v) {
        constexpr int at = I * kIdBits / 32, sh = I * kIdBits % 32;
        w[at] |= v << sh;
        if constexpr (sh + kIdBits > 32) w[at + 1] |= v >> (32 - sh);
    }
    __device__ __forceinline__ uint32_t state() const { return w[0] & kIdMask; }
    __device__ __forceinline__ bool same_key(const StagedEntry &o) const {
        bool eq = ((w[0] ^ o.w[0]) >> kIdBits) == 0;
#pragma unroll
        for (int i = 1; i < W; ++i) eq &= w[i] == o.w[i];
        return eq;
    }
    __device__ __forceinline__ uint64_t hash() const {
        uint64_t h = mix_step(kHashSeed, w[0] >> kIdBits);
#pragma unroll
        for (int i = 1; i < W; ++i) h = mix_step(h, w[i]);
        return mix_final(h);
    }
};

// The ids of the window's states, in the segment: low halves, and their bit
// 16 four to a byte (if any can be set).
struct StagedIds {
    const uint16_t *lo;
    const uint8_t *hi;
    bool big;
    __device__ __forceinline__ uint32_t operator[](uint32_t i) const {
        uint32_t v = lo[i];
        if (big) v |= ((hi[i >> 2] >> (i & 3u)) & 1u) << 16;
        return v;
    }
};

template <int K, int I>
__device__ __forceinline__ void staged_put(StagedEntry<K> &e, const StagedIds &ids, uint32_t own,
                                           const StagedRow<K> &row) {
    if constexpr (I < K) {
        e.template put<I + 2>(ids[own + row.t[I]]);
        staged_put<K, I + 1>(e, ids, own, row);
    }
}

// The entries of a chunk.  base: the window's first state.
template <int K>
__device__ __forceinline__ void staged_keys(const SegdArgs &a, const SegdPart &P,
                                            const SegdSeg &S, const StagedIds &ids, uint32_t base,
                                            const SegdChunk &C, uint32_t end, uint32_t r,
                                            uint32_t *hist, uint32_t *pre, uint32_t *Y,
                                            uint32_t &blocks, uint32_t &active) {
    constexpr int U = kStagedGroup / kStagedThreads;
    const uint32_t tx = threadIdx.x, own = P.off - base, nb = S.mask;
    const uint32_t seg0 = S.first_tile * kBlock;
    StagedEntry<K> *out = reinterpret_cast<StagedEntry<K> *>(a.entries + S.table);
    uint32_t group = C.group;
    // rows and marks of a group are loaded while the one before it is sorted
    StagedRow<K> next_row[U];
    uint8_t next_mark[U];
    auto fetch = [&](uint32_t q0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t q = q0 + u * kStagedThreads + tx;
            const uint32_t qs = q < end ? q : C.first;
            next_mark[u] = a.shared[qs];
            next_row[u] = *staged_row<K>(a, P, qs);
        }
    };
    fetch(C.first);
    for (uint32_t q0 = C.first; q0 < end; q0 += kStagedGroup, ++group) {
        if (tx < nb) hist[tx] = 0;
        StagedEntry<K> e[U];
        uint32_t bucket[U], rank[U];
        bool act[U];
        {
            StagedRow<K> row[U];
            uint8_t m[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                row[u] = next_row[u];
                m[u] = next_mark[u];
            }
            if (q0 + kStagedGroup < end) fetch(q0 + kStagedGroup);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t q = q0 + u * kStagedThreads + tx;
                const uint32_t w0 = ids[(q < end ? q : q0) - base];
                act[u] = q < end && (w0 != q - seg0 || m[u] == (r & 255u));
                e[u] = StagedEntry<K>{};
                e[u].template put<0>(q - seg0);
                e[u].template put<1>(w0);
                staged_put<K, 0>(e[u], ids, own, row[u]);
                if (q < end) Y[q] = q;
                blocks += q < end && !act[u] ? 1u : 0u;
                active += act[u] ? 1u : 0u;
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            bucket[u] = rank[u] = 0;
            if (nb > 1) {
                if (!act[u]) continue;
                bucket[u] = __umulhi(static_cast<uint32_t>(e[u].hash() >> 32), nb);
                rank[u] = atomicAdd(hist + bucket[u], 1u);
            } else {
                const unsigned long long am = __ballot(act[u]);
                uint32_t at = 0;
                if (lane_id() == 0) at = atomicAdd(hist, static_cast<uint32_t>(__popcll(am)));
                rank[u] = __shfl(at, 0, 64) +
                          static_cast<uint32_t>(__popcll(am & ((1ull << lane_id()) - 1)));
            }
        }
        __syncthreads();
        if (tx <= nb) {
            uint32_t before = 0;
            for (uint32_t b = 0; b < tx; ++b) before += hist[b];
            pre[tx] = before;
            a.offs[S.offs + group * (nb + 1) + tx] = static_cast<uint16_t>(before);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (act[u]) out[q0 - seg0 + pre[bucket[u]] + rank[u]] = e[u];
    }
}

// Sums of a workgroup (valid in thread 0).
__device__ __forceinline__ uint32_t staged_sum(uint32_t v, uint32_t *red) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    __syncthreads();
    if (lane_id() == 0) red[threadIdx.x / 64] = v;
    __syncthreads();
    uint32_t s = 0;
#pragma unroll
    for (uint32_t i = 0; i < kStagedThreads / 64; ++i) s += red[i];
    return s;
}

__global__ __launch_bounds__(kStagedThreads) void k_staged_keys(SegdArgs a, uint32_t r) {
    extern __shared__ __align__(16) uint8_t lds[];
    __shared__ uint32_t red[kStagedThreads / 64];
    __shared__ uint32_t hist[kStagedMaxBuckets], pre[kStagedMaxBuckets + 1];
    uint32_t chunk;
    if (!segd_tile(a.nchunks, chunk)) return;
    const SegdChunk C = a.chunks[chunk];
    const SegdPart P = a.parts[C.part];
    const uint32_t s = P.seg, tx = threadIdx.x;
    if (a.done[s]) return;
    const SegdSeg S = a.segs[s];
    const uint32_t seg0 = S.first_tile * kBlock;
    const uint32_t *__restrict__ X = (r & 1u) ? a.blockB : a.blockA;
    uint32_t *__restrict__ Y = (r & 1u) ? a.blockA : a.blockB;
    uint32_t was, changing;
    if (segd_decided(a, S, s, r, X, was, changing)) {
        if (C.first == seg0 && tx == 0) segd_record(a, s, r, was, changing);
        return;
    }
    if (C.first == seg0 && tx == 0) a.cnt[((r + 1) & 3u) * a.nseg + s] = 0;
    const uint32_t end = min(C.first + a.chunk_groups * kStagedGroup, P.off + P.n);
    uint32_t blocks = 0, active = 0;
    bool any = false;
    for (uint32_t q = C.first + tx; q < end; q += kStagedThreads)
        any |= X[q] != q || a.shared[q] == (r & 255u);
    if (__syncthreads_or(any) == 0) {  // (all of them are singletons)
        for (uint32_t q = C.first + tx; q < end; q += kStagedThreads) {
            Y[q] = q;
            ++blocks;
        }
        const uint32_t starts =
            (end - C.first + kStagedGroup - 1) / kStagedGroup * (S.mask + 1);
        if (tx < starts) a.offs[S.offs + C.group * (S.mask + 1) + tx] = 0;
    } else {
        const SegdPart O = a.pairs ? a.parts[C.part ^ 1u] : P;
        const bool big = max(P.off + P.n, O.off + O.n) - seg0 > kStagedWindow;
        uint16_t *lo = reinterpret_cast<uint16_t *>(lds);
        uint8_t *hi = lds + 2 * a.window;
        // (the part starts at a multiple of the tile, and whole tiles are
        // allocated)
        for (uint32_t i = 4 * tx; i < P.n; i += 4 * kStagedThreads) {
            const uint4 v = *reinterpret_cast<const uint4 *>(X + P.off + i);
            const uint32_t x = v.x - seg0, y = v.y - seg0, z = v.z - seg0, w = v.w - seg0;
            *reinterpret_cast<uint2 *>(lo + i) =
                make_uint2((x & 0xFFFFu) | (y << 16), (z & 0xFFFFu) | (w << 16));
            if (big)
                hi[i >> 2] = static_cast<uint8_t>(((x >> 16) & 1u) | (((y >> 16) & 1u) << 1) |
                                                  (((z >> 16) & 1u) << 2) |
                                                  (((w >> 16) & 1u) << 3));
        }
        const StagedIds ids{lo, hi, big};
        __syncthreads();
        switch (P.k) {
#define STAGED_KEYS(K) \
    staged_keys<K>(a, P, S, ids, P.off, C, end, r, hist, pre, Y, blocks, active)
            case 1: STAGED_KEYS(1); break;
            case 2: STAGED_KEYS(2); break;
            case 3: STAGED_KEYS(3); break;
            case 4: STAGED_KEYS(4); break;
            case 5: STAGED_KEYS(5); break;
            case 6: STAGED_KEYS(6); break;
            case 7: STAGED_KEYS(7); break;
            default: STAGED_KEYS(8); break;
#undef STAGED_KEYS
        }
    }
    // (at most 8,192 of each)
    const uint32_t sum = staged_sum(blocks | active << 16, red);
    if (tx == 0) {
        if (sum & 0xFFFFu) atomicAdd(a.cnt + (r & 3u) * a.nseg + s, sum & 0xFFFFu);
        if (sum >> 16)
            atomicAdd(a.ctl->active + (blockIdx.x % kSegdSpread) * kSegdStride,
                      static_cast<unsigned long long>(sum >> 16));
    }
}

constexpr uint32_t kStagedProbes = 1024;      // slots that a key may take
constexpr uint32_t kStagedGroups = 128;  // most groups of a segment

// Groups the m entries of a bucket; runs: entry i of it is entry
// i + at[g] of the segment, g its run (first[g] <= i).
template <int K>
__device__ __forceinline__ uint32_t staged_bucket(const SegdArgs &a, const SegdSeg &S,
                                                  const uint32_t *first, const uint32_t *at,
                                                  uint32_t groups, uint32_t m, uint32_t r,
                                                  uint32_t *tab, uint32_t *left) {
    constexpr int U = 2;
    constexpr uint32_t NT = kStagedThreads;
    const uint32_t tx = threadIdx.x, seg0 = S.first_tile * kBlock;
    uint32_t *__restrict__ Y = (r & 1u) ? a.blockA : a.blockB;
    const StagedEntry<K> *ent = reinterpret_cast<const StagedEntry<K> *>(a.entries + S.table);
    const uint32_t T = min(kStagedSlots, max(256u, 2 * m));
    for (uint32_t i = tx; i < (m + 31) / 32; i += NT) left[i] = 0;
    uint32_t claims = 0;
    // One pass, but for a table that fills up (which takes twice a bucket's
    // share of different keys): an entry that finds neither its key nor a
    // free slot is left to the next pass, with an empty table.  All entries
    // of a key probe the same slots, so a pass settles all of them or none.
    for (bool again = false;; again = true) {
        for (uint32_t i = tx; i < T; i += NT) tab[i] = ~0u;
        __syncthreads();
        bool more = false;
        for (uint32_t i0 = 0; i0 < m; i0 += U * NT) {
            StagedEntry<K> e[U];
            uint32_t loc[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t i = min(i0 + u * NT + tx, m - 1);
                uint32_t lo = 0, hi = groups;
                while (hi - lo > 1) {
                    const uint32_t mid = (lo + hi) / 2;
                    if (first[mid] <= i)
                        lo = mid;
                    else
                        hi = mid;
                }
                loc[u] = i + at[lo];
                e[u] = ent[loc[u]];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t i = i0 + u * NT + tx;
                if (i >= m) continue;
                if (again && !((left[i / 32] >> (i % 32)) & 1u)) continue;
                const uint64_t h = e[u].hash();
                // (not all ones, which with the last entry is a free slot)
                const uint32_t tag = min(static_cast<uint32_t>(h >> 32) & 0x7FFFu, 0x7FFEu);
                uint32_t sl = __umulhi(static_cast<uint32_t>(h), T);
                bool settled = false;
                for (uint32_t probe = 0; probe < kStagedProbes; ++probe) {
                    uint32_t o = __hip_atomic_load(tab + sl, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (o == ~0u) {
                        o = atomicCAS(tab + sl, ~0u, (tag << kIdBits) | loc[u]);
                        if (o == ~0u) {
                            ++claims;
                            settled = true;
                            break;
                        }
                    }
                    if ((o >> kIdBits) == tag) {
                        const StagedEntry<K> rep = ent[o & kIdMask];
                        if (rep.same_key(e[u])) {
                            const uint32_t id = seg0 + rep.state();
                            Y[seg0 + e[u].state()] = id;
                            mark_shared(a.shared, id, r + 1);
                            settled = true;
                            break;
                        }
                    }
                    sl = sl + 1 == T ? 0u : sl + 1;
                }
                if (!settled) {
                    more = true;
                    atomicOr(left + i / 32, 1u << (i % 32));
                } else if (again) {
                    atomicAnd(left + i / 32, ~(1u << (i % 32)));
                }
            }
        }
        if (__syncthreads_or(more) == 0) return claims;
    }
}

__global__ __launch_bounds__(kStagedThreads) void k_staged_group(SegdArgs a, uint32_t r) {
    extern __shared__ __align__(16) uint8_t lds[];
    __shared__ uint32_t red[kStagedThreads / 64];
    __shared__ uint32_t first[kStagedGroups], at[kStagedGroups], total;
    uint32_t index;
    if (!segd_tile(a.nbuckets, index)) return;
    const SegdBucket b = a.buckets[index];
    if (a.done[b.seg]) return;  // (recorded by this round's first launch, if decided)
    const SegdSeg S = a.segs[b.seg];
    const uint32_t p = a.pairs ? 2 * b.seg : b.seg, tx = threadIdx.x;
    const SegdPart P = a.parts[p];
    if (tx < 64) {
        // two groups to a lane: where their runs start, and how long they are
        const uint32_t own = (P.n + kStagedGroup - 1) / kStagedGroup;
        const uint32_t seg0 = S.first_tile * kBlock;
        const uint32_t second = a.pairs ? a.parts[p + 1].off - seg0 : 0u;
        uint32_t len[2], start[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t g = 2 * tx + u;
            len[u] = start[u] = 0;
            if (g < S.groups) {
                const uint16_t *o = a.offs + S.offs + g * (S.mask + 1) + b.bucket;
                const uint32_t from = o[0], to = o[1];
                len[u] = to - from;
                start[u] = from + (g < own ? g * kStagedGroup
                                           : second + (g - own) * kStagedGroup);
            }
        }
        uint32_t x = len[0] + len[1];
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(x, d, 64);
            if (tx >= static_cast<uint32_t>(d)) x += y;
        }
        uint32_t before = x - len[0] - len[1];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            first[2 * tx + u] = before;
            at[2 * tx + u] = start[u] - before;
            before += len[u];
        }
        if (tx == 63) total = x;
    }
    __syncthreads();
    const uint32_t m = total;
    if (m == 0) return;
    uint32_t *tab = reinterpret_cast<uint32_t *>(lds), *left = tab + kStagedSlots;
    uint32_t claims = 0;
    switch (P.k) {
#define STAGED_BUCKET(K) claims = staged_bucket<K>(a, S, first, at, S.groups, m, r, tab, left)
        case 1: STAGED_BUCKET(1); break;
        case 2: STAGED_BUCKET(2); break;
        case 3: STAGED_BUCKET(3); break;
        case 4: STAGED_BUCKET(4); break;
        case 5: STAGED_BUCKET(5); break;
        case 6: STAGED_BUCKET(6); break;
        case 7: STAGED_BUCKET(7); break;
        default: STAGED_BUCKET(8); break;
#undef STAGED_BUCKET
    }
    const uint32_t sum = staged_sum(claims, red);
    if (tx == 0) atomicAdd(a.cnt + (r & 3u) * a.nseg + b.seg, sum);
}

// Patterns of a chunk: the representatives in LDS (rep, by pattern), whether
// a pattern has several states there, and the letters that move a state.
template <int K>
__device__ __forceinline__ void staged_patterns(const SegdArgs &a, const SegdPart &P,
                                                const uint8_t *acc, uint32_t first, uint32_t end,
                                                uint32_t *rep, uint32_t *shared, uint16_t *pat,
                                                uint32_t &moves, uint32_t &cls, bool &bad) {
    constexpr int U = 2;
    for (uint32_t q0 = first; q0 < end; q0 += U * kStagedThreads) {
        uint32_t t[U][K];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t q = q0 + u * kStagedThreads + threadIdx.x;
            const uint32_t *r =
                P.delta + static_cast<size_t>((q < end ? q : first) - P.off) * K;
            if (K % 4 == 0 && P.wide) {
#pragma unroll
                for (int j = 0; j < K; j += 4) {
                    const uint4 v = *reinterpret_cast<const uint4 *>(r + j);
                    t[u][j] = v.x;
                    t[u][j + 1] = v.y;
                    t[u][j + 2] = v.z;
                    t[u][j + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int j = 0; j < K; ++j) t[u][j] = r[j];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t q = q0 + u * kStagedThreads + threadIdx.x;
            if (q >= end) continue;
            uint32_t p = acc[q - P.off] != 0 ? 1u : 0u;
            cls |= p ? 1u : 2u;
            StagedRow<K> row{};
#pragma unroll
            for (int j = 0; j < K; ++j) {
                // (a target out of range fails the call)
                const bool out = t[u][j] >= P.n;
                bad |= out;
                const uint32_t i = out ? 0u : t[u][j];
                row.t[j] = static_cast<uint16_t>(i);
                p |= (acc[i] != 0 ? 2u : 0u) << j;
                moves |= i != q - P.off ? 1u << j : 0u;
            }
            *staged_row<K>(a, P, q) = row;
            pat[q - first] = static_cast<uint16_t>(p);
            // (read first: a pattern that is there costs no atomic)
            uint32_t o = __hip_atomic_load(rep + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (o == ~0u) o = atomicCAS(rep + p, ~0u, q);
            if (o != ~0u) shared[p] = 1;
        }
    }
}

__global__ __launch_bounds__(kStagedThreads) void k_staged_first(SegdArgs a) {
    extern __shared__ __align__(16) uint8_t lds[];
    __shared__ uint32_t red[kStagedThreads / 64];
    __shared__ uint32_t rep[kStagedPatterns], gid[kStagedPatterns], shared[kStagedPatterns];
    uint32_t chunk;
    if (!segd_tile(a.nchunks, chunk)) return;
    const SegdChunk C = a.chunks[chunk];
    const SegdPart P = a.parts[C.part];
    const uint32_t s = P.seg, tx = threadIdx.x;
    const SegdSeg S = a.segs[s];
    const bool first_chunk = C.first == S.first_tile * kBlock;
    if (first_chunk && tx == 0) a.cnt[a.nseg + s] = 0;  // the counter of round 1
    const uint32_t end = min(C.first + a.chunk_groups * kStagedGroup, P.off + P.n);
    uint32_t *__restrict__ Y = a.blockB;
    uint16_t *pat = reinterpret_cast<uint16_t *>(lds);
    // acceptance, words where they are aligned (at the same alignment in LDS)
    const uint32_t lead = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(P.acc) & 3u);
    uint8_t *acc = lds + 2 * a.chunk_groups * kStagedGroup + lead;
    {
        const uint32_t head = min((4u - lead) & 3u, P.n);
        const uint32_t words = (P.n - head) / 4;
        for (uint32_t i = tx; i < words; i += kStagedThreads)
            reinterpret_cast<uint32_t *>(acc + head)[i] =
                reinterpret_cast<const uint32_t *>(P.acc + head)[i];
        if (tx < head) acc[tx] = P.acc[tx];
        for (uint32_t i = head + 4 * words + tx; i < P.n; i += kStagedThreads) acc[i] = P.acc[i];
    }
    for (uint32_t i = tx; i < kStagedPatterns; i += kStagedThreads) {
        rep[i] = ~0u;
        shared[i] = 0;
    }
    __syncthreads();
    uint32_t moves = 0, cls = 0;
    bool bad = false;
    switch (P.k) {
        case 1: staged_patterns<1>(a, P, acc, C.first, end, rep, shared, pat, moves, cls, bad); break;
        case 2: staged_patterns<2>(a, P, acc, C.first, end, rep, shared, pat, moves, cls, bad); break;
        case 3: staged_patterns<3>(a, P, acc, C.first, end, rep, shared, pat, moves, cls, bad); break;
        case 4: staged_patterns<4>(a, P, acc, C.first, end, rep, shared, pat, moves, cls, bad); break;
        case 5: staged_patterns<5>(a, P, acc, C.first, end, rep, shared, pat, moves, cls, bad); break;
        case 6: staged_patterns<6>(a, P, acc, C.first, end, rep, shared, pat, moves, cls, bad); break;
        case 7: staged_patterns<7>(a, P, acc, C.first, end, rep, shared, pat, moves, cls, bad); break;
        default: staged_patterns<8>(a, P, acc, C.first, end, rep, shared, pat, moves, cls, bad); break;
    }
    wave_set_flag(&a.ctl->err, bad);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        moves |= __shfl_xor(moves, d, 64);
        cls |= __shfl_xor(cls, d, 64);
    }
    if (lane_id() == 0) {
        // (plain reads: an older value only repeats the atomic)
        if (cls & ~a.classes[s]) atomicOr(a.classes + s, cls);
        if (moves & ~a.ctl->moves) atomicOr(&a.ctl->moves, moves);
    }
    __syncthreads();
    uint32_t blocks = 0;
    if (tx < kStagedPatterns && rep[tx] != ~0u) {
        const uint32_t q = rep[tx];
        // (a word: the representative's number in the segment + 1)
        const uint32_t seg0 = S.first_tile * kBlock;
        uint32_t was = atomicCAS(a.patterns + s * kStagedPatterns + tx, 0u, q - seg0 + 1);
        if (!was) {
            ++blocks;
            was = q - seg0 + 1;
        }
        const uint32_t id = seg0 + was - 1;
        gid[tx] = id;
        if (!blocks || shared[tx]) mark_shared(a.shared, id, 1);
    }
    __syncthreads();
    for (uint32_t q = C.first + tx; q < end; q += kStagedThreads) Y[q] = gid[pat[q - C.first]];
    const uint32_t sum = staged_sum(blocks, red);
    if (tx == 0) {
        atomicAdd(a.cnt + s, sum);
        atomicAdd(a.ctl->active + (blockIdx.x % kSegdSpread) * kSegdStride,
                  static_cast<unsigned long long>(end - C.first));
    }
}

// The segments that are decided after r rounds are recorded; with `last`, the
// others too, as not stable.
__global__ __launch_bounds__(kBlock) void k_segd_decide(SegdArgs a, uint32_t r, uint32_t last) {
    const uint32_t s = static_cast<uint32_t>(global_tid());
    if (s >= a.nseg || a.done[s]) return;
    const uint32_t *X = (r & 1u) ? a.blockB : a.blockA;
    uint32_t blocks, changing;
    const bool d = segd_decided(a, a.segs[s], s, r, X, blocks, changing);
    if (!d && !last) return;
    if (!d) a.ctl->limit = 1;
    segd_record(a, s, r, blocks, changing);
}

// The block ids of a decided segment.
__device__ __forceinline__ const uint32_t *segd_final(const SegdArgs &a, uint32_t s) {
    return ((a.done[s] - 1) & 1u) ? a.blockA : a.blockB;
}

// Canonical ids, as the maximum of ~q per id in a zeroed scratch (segments
// whose blocks are all single states need none).
__global__ __launch_bounds__(kBlock) void k_segd_canon(SegdArgs a, uint32_t *maxs) {
    uint32_t tile;
    if (!segd_tile(a.tiles, tile)) return;
    const SegdPart P = a.parts[a.tile_part[tile]];
    const uint32_t q = tile * kBlock + threadIdx.x;
    if (q - P.off >= P.n || a.blocks[P.seg] == P.n) return;
    atomicMax(maxs + segd_final(a, P.seg)[q], ~q);
}

__global__ __launch_bounds__(kBlock) void k_segd_output(SegdArgs a, const uint32_t *maxs,
                                                         uint32_t *__restrict__ out) {
    uint32_t tile;
    if (!segd_tile(a.tiles, tile)) return;
    const SegdPart P = a.parts[a.tile_part[tile]];
    const uint32_t q = tile * kBlock + threadIdx.x;
    const uint32_t i = q - P.off;
    if (i >= P.n) return;
    out[P.out + i] = a.blocks[P.seg] == P.n ? i : ~maxs[segd_final(a, P.seg)[q]] - P.off;
}

__global__ __launch_bounds__(kBlock) void k_segd_verdicts(SegdArgs a, int32_t *verdicts) {
    const uint32_t s = static_cast<uint32_t>(global_tid());
    if (s >= a.nseg) return;
    const uint32_t *ids = segd_final(a, s);
    verdicts[s] = ids[a.segs[s].eq_a] == ids[a.segs[s].eq_b] ? 1 : 0;
}

dim3 tile_grid(const SegdArgs &a) { return dim3((a.tiles + 7) / 8 * 8); }

}  // namespace

void launch_segd_round(const SegdArgs &a, uint32_t r, uint32_t epoch, bool wide_letters,
                       hipStream_t s) {
    const dim3 grid = tile_grid(a), block(kBlock);
    if (wide_letters) {
        if (r == 0)
            launch_kernel(k_segd_round<16, true>, grid, block, 0, s, a, r, epoch);
        else
            launch_kernel(k_segd_round<16, false>, grid, block, 0, s, a, r, epoch);
    } else {
        if (r == 0)
            launch_kernel(k_segd_round<8, true>, grid, block, 0, s, a, r, epoch);
        else
            launch_kernel(k_segd_round<8, false>, grid, block, 0, s, a, r, epoch);
    }
}

void launch_staged_round(const SegdArgs &a, uint32_t r, hipStream_t s) {
    const dim3 chunks((a.nchunks + 7) / 8 * 8), buckets((a.nbuckets + 7) / 8 * 8);
    const dim3 block(kStagedThreads);
    if (r == 0) {
        const uint32_t lds = 2 * a.chunk_groups * kStagedGroup + a.max_n + 4;
        launch_kernel(k_staged_first, chunks, block, lds, s, a);
    } else {
        launch_kernel(k_staged_keys, chunks, block, 2 * a.window + a.window / 4, s, a, r);
        launch_kernel(k_staged_group, buckets, block, 4 * kStagedSlots + a.max_states / 8 + 4, s,
                      a, r);
    }
}

void launch_segd_decide(const SegdArgs &a, uint32_t r, bool last, hipStream_t s) {
    launch_kernel(k_segd_decide, dim3((a.nseg + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a, r,
                  last ? 1u : 0u);
}

void launch_segd_output(const SegdArgs &a, uint32_t *scratch_max, uint32_t *out, hipStream_t s) {
    launch_kernel(k_segd_canon, tile_grid(a), dim3(kBlock), 0, s, a, scratch_max);
    launch_kernel(k_segd_output, tile_grid(a), dim3(kBlock), 0, s, a,
                  static_cast<const uint32_t *>(scratch_max), out);
}

void launch_segd_verdicts(const SegdArgs &a, int32_t *verdicts, hipStream_t s) {
    launch_kernel(k_segd_verdicts, dim3((a.nseg + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a,
                  verdicts);
}

}  // namespace dfamin
