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
//     A decided segment costs its tiles one load a round.
//
// Table entries carry a 20-bit epoch that the workspace counts on from call
// to call, so the tables are cleared once in a million rounds.
//
// Bound by L2 requests (the successor ids of a state, then its table slot).
// Measured on MI355X, 1,024 random DFAs of 64 to 65,536 states and 2 to 8
// letters, 9.87 million states in the segments: the call takes 2.83 ms, 3.81 in
// the general path's five passes over signature rows; 512 pairs 6.17 ms, 7.29.
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
