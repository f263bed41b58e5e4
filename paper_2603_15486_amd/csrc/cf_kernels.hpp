// cf_kernels.hpp -- gfx950 kernels of the cuckoo filter.
//
// One lane per key, wave64, grid-stride loops over any grid; the host picks
// the launch shape (one key per thread for queries and deletes up to a cap,
// a smaller grid with several keys per thread for inserts).  Occupancy
// counts follow Sec. 4.3's hierarchy: wave shuffle, LDS, one atomic per
// block.  Insertion defers the eviction search of keys whose two buckets
// are full to a second pass of the same block (see insert_kernel).
#pragma once

#include "cf_bulk_plan.hpp"
#include "cf_device.hpp"

namespace cfk {

constexpr int kBlock = 256;
constexpr int kRefill = 16;  // free lanes of a wave that take new searches together
constexpr int kStripes = 32;  // occupancy counter stripes, one 128-byte line each

// Device-side counters.  The occupancy count is striped over kStripes
// separate lines: blocks add to stripe (blockIdx mod kStripes), so the one
// atomic per block of Sec. 4.3's hierarchical tally never piles up on a
// single address (device-scope atomics execute at the memory side on this
// part and same-address ones serialise).  The failure counter doubles as the
// cursor of the dropped-tag log; failures are rare.
struct alignas(128) Stripe {
    unsigned long long v;
    unsigned long long pad[15];
};

struct Counters {
    Stripe count[kStripes];
    unsigned long long failures;
    unsigned long long total;  // sum of the stripes, written by sum_counts_kernel
};

// ------------------------------------------ entries of a partitioned insert
// (cf_bulk.hpp; packed as cf_bulk_plan.hpp says)
struct Raw {  // as loaded: a key, or an entry's words
    uint64_t a;
    uint32_t b;
};

// What a partitioned insert left over (see insert_kernel).
struct NoRest {};
struct Rest {
    Ents list;               // part p's entries at p * cap
    const uint32_t *list_n;  // how many; behind them the overflow list's length
    const uint32_t *ovl;     // the overflow list: keys' indices
    uint32_t cap, parts, split, extra;
    uint32_t shift;          // parts of 2^shift buckets
    uint32_t ncursors;
    uint32_t *cursors;       // the pass's cursors, to be cleared for the next one
};

struct LostLog {
    unsigned long long *bucket;
    uint32_t *tag;
    unsigned long long cap;
};

// Sum v over the block and add it to the block's count stripe with one
// atomic.  Every thread of the block must call it.
template <int BT = kBlock>
__device__ __forceinline__ void block_add(Counters *ctr, unsigned long long v) {
    __shared__ unsigned long long part[BT / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) part[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long s = 0;
#pragma unroll
        for (int k = 0; k < BT / 64; ++k) s += part[k];
        if (s) atomicAdd(&ctr->count[blockIdx.x % kStripes].v, s);
    }
    __syncthreads();
}

// ------------------------------------------------------------------ query

// Alg. 2: probe i1, and i2 only when i1 misses.
template <class G, int HASH, int POL>
__global__ __launch_bounds__(kBlock) void query_kernel(const typename G::W *__restrict__ table,
                                                       Place pl,
                                                       const uint64_t *__restrict__ keys,
                                                       uint64_t n, uint8_t *__restrict__ found) {
    const uint64_t stride = uint64_t(gridDim.x) * kBlock;
    for (uint64_t i = uint64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += stride) {
        const uint64_t key = __builtin_nontemporal_load(keys + i);
        const Derived d = derive<G, HASH, POL>(key, pl);
        Bucket<G> bk;
        load_bucket<G>(table, d.i1, bk);
        bool hit = bk.contains(d.t1);
        if (!hit) {
            load_bucket<G>(table, d.i2, bk);
            hit = bk.contains(d.t2);
        }
        __builtin_nontemporal_store(uint8_t(hit), found + i);
    }
}

// ----------------------------------------------------------------- delete

// Alg. 3: remove one copy from i1, else from i2; the occupancy count drops
// by the block's number of successes.
template <class G, int HASH, int POL>
__global__ __launch_bounds__(kBlock) void delete_kernel(typename G::W *__restrict__ table,
                                                        Place pl,
                                                        const uint64_t *__restrict__ keys,
                                                        uint64_t n, uint8_t *__restrict__ ok,
                                                        Counters *ctr) {
    unsigned long long removed = 0;
    const uint64_t stride = uint64_t(gridDim.x) * kBlock;
    for (uint64_t i = uint64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += stride) {
        const uint64_t key = __builtin_nontemporal_load(keys + i);
        const Derived d = derive<G, HASH, POL>(key, pl);
        Bucket<G> bk;
        load_bucket<G>(table, d.i1, bk);
        bool done = try_remove<G>(table, d.i1, d.t1, bk);
        if (!done) {
            load_bucket<G>(table, d.i2, bk);
            done = try_remove<G>(table, d.i2, d.t2, bk);
        }
        removed += done;
        if (ok) ok[i] = uint8_t(done);
    }
    // count -= removed, as the two's-complement addition of -removed
    block_add(ctr, 0ull - removed);
}

// --------------------------------------------------- insert: eviction search

// Candidates whose other buckets a grouped breadth-first search loads at
// once: as many as 128 bytes of buckets hold, at most b/2.
template <class G>
constexpr int probe_width() {
    constexpr int bytes = G::B * G::F / 8;
    constexpr int fit = bytes >= 128 ? 1 : 128 / bytes;
    return fit < G::B / 2 ? fit : G::B / 2;
}

// Sec. 4.6.1 breadth-first heuristic, one level at a time.  At each level the
// candidates are the b/2 slots of the current bucket starting at a random
// slot; the first whose fingerprint has an empty slot in its other bucket is
// moved there and the carried fingerprint takes its place.  Failing that, the
// last candidate is displaced and carried to its other bucket.  The move is
// done displacement first: the carried fingerprint replaces the candidate
// with a CAS that only succeeds while the slot still holds the candidate,
// then the candidate is inserted into its other bucket.  If that bucket
// filled up in the meantime the candidate is simply carried on, as after a
// displacement.  `tag` is always the carried fingerprint as it is written in
// `cur` (the choice bit of the offset policy flips with every move).
// The insert kernels that use it are compiled at -O1: built at -O2 or -O3
// they lost fingerprints under heavy contention (one-launch fills of a
// 2^20-slot table), a loss that appears with the backend's Early Machine
// LICM run over the kernel and goes away without it; see the one-launch
// contention tests.
//
// PW (probe width) candidates have their other buckets loaded together, then
// the first of them (in candidate order) with an empty slot is moved, so the
// choice is the one a candidate-by-candidate probe makes on an unchanged
// table; only the number of dependent loads per level drops, from b/2 to
// b/(2 PW), at the price of loading a group's buckets whole.  PW = 1 is the
// candidate-by-candidate probe, which the single-filter insert kernel uses
// on large tables, where it is bound by memory requests and whole groups
// only add reads; tables of a few MiB measured faster with probe_width (the
// launchers choose by table size).
//
// What bounds a search is its chain of dependent memory accesses (half a
// microsecond and up for a load, more than one for a device-scope CAS), so a
// level hands the bucket it ends in to the next one: the displaced last
// candidate's other bucket was just probed and found full, and within an
// insert launch a full bucket stays full, so neither it nor the next level's
// current bucket is loaded again.  A level that displaces is then one round
// of probes and one CAS.

// One search in flight.
template <class G>
struct Search {
    uint64_t rs;      // its stream of random draws
    uint32_t cur;     // the bucket the carried fingerprint is to enter
    uint32_t tag;     // ... as it is written there
    uint32_t n;       // levels done
    uint32_t kicks;
    bool have;        // cb holds cur's words, seen full
    Bucket<G> cb;
};

template <class G>
__device__ __forceinline__ void search_start(Search<G> &st, Derived d, uint64_t rs) {
    // masks, not selects: a select becomes an indexed access to d in memory
    const uint32_t second = 0u - uint32_t(splitmix_at(rs, 0) & 1);
    st.rs = rs;
    st.cur = (d.i1 & ~second) | (d.i2 & second);
    st.tag = (d.t1 & ~second) | (d.t2 & second);
    st.n = 0;
    st.kicks = 0;
    st.have = false;
}

// One level; true once the carried fingerprint is stored.  KEEP: probed
// buckets stay in registers, for the move that follows and for the next
// level.  Without it they are loaded again where they are needed: the set's
// kernels hold the code of several bucket sizes and measured no gain, and
// their persistent form would fit fewer blocks (256 threads, 16-bit
// fingerprints: 5 waves per SIMD for 6).
template <class G, int HASH, int POL, int PW, bool KEEP>
__device__ __forceinline__ bool bfs_level(typename G::W *table, const Place &pl, Search<G> &st) {
    using W = typename G::W;
    constexpr int HALF = G::B / 2;
    static_assert(PW >= 1 && HALF % PW == 0, "probe width must divide b/2");
    ++st.n;
    if (!st.have) {
        load_bucket<G>(table, st.cur, st.cb);
        if (st.cb.has_empty() && try_insert<G>(table, st.cur, st.tag, st.cb) >= 0) return true;
    }
    const int r0 = int(splitmix_at(st.rs, st.n) % uint64_t(G::B));
    Bucket<G> last;       // the last candidate's other bucket,
    uint32_t last_c = 0;  // and the candidate (0: it has no other bucket)
    for (int j0 = 0; j0 < HALF; j0 += PW) {
        Bucket<G> ab[PW];  // the group's other buckets,
        uint32_t cv[PW];   // and its candidates
        uint32_t ok = 0;
#pragma unroll
        for (int q = 0; q < PW; ++q) {
            cv[q] = st.cb.slot((r0 + j0 + q) % G::B);
            uint32_t moved = cv[q];
            const uint32_t a = move_tag<G, HASH, POL>(st.cur, moved, pl);
            if constexpr (KEEP) {
                // no branch around the load, so that a group's loads go out together
                if (a == st.cur) cv[q] = 0;
                load_bucket<G>(table, cv[q] != 0 ? a : st.cur, ab[q]);
            } else if (cv[q] != 0 && a != st.cur) {
                Bucket<G> b;
                load_bucket<G>(table, a, b);
                if (b.has_empty()) ok |= 1u << q;
            }
        }
        if constexpr (KEEP) {
#pragma unroll
            for (int q = 0; q < PW; ++q) ok |= (cv[q] != 0 && ab[q].has_empty() ? 1u : 0u) << q;
        }
        if constexpr (KEEP) {
            last = ab[PW - 1];
            last_c = cv[PW - 1];
        }
        // in candidate order, the move of the first that takes it (the probed
        // value: the move happens only while the slot holds it)
        while (ok) {
            const int q = __builtin_ctz(ok);
            ok &= ok - 1u;
            const int s = (r0 + j0 + q) % G::B;
            uint32_t c = 0;
            Bucket<G> mb{};
#pragma unroll
            for (int k = 0; k < PW; ++k) {
                c |= cv[k] & (0u - uint32_t(k == q));
                if constexpr (KEEP) {
                    const W mask = W(0) - W(k == q);
#pragma unroll
                    for (int w = 0; w < G::WPB; ++w) mb.w[w] |= ab[k].w[w] & mask;
                }
            }
            uint32_t moved = c;
            const uint32_t a = move_tag<G, HASH, POL>(st.cur, moved, pl);
            if (!replace_slot_if<G>(table, st.cur, s, c, st.tag, st.cb)) continue;
            ++st.kicks;
            if constexpr (!KEEP) load_bucket<G>(table, a, mb);
            if (try_insert<G>(table, a, moved, mb) >= 0) return true;
            st.tag = moved;  // `a` filled up meanwhile: carry the candidate from there
            st.cur = a;
            st.cb = mb;
            st.have = KEEP;
            return false;
        }
    }
    const uint32_t ev = swap_slot<G>(table, st.cur, (r0 + HALF - 1) % G::B, st.tag, st.cb);
    ++st.kicks;
    if (ev == 0) return true;
    st.tag = ev;
    st.cur = move_tag<G, HASH, POL>(st.cur, st.tag, pl);
    st.have = KEEP;
    if (KEEP && ev == last_c) st.cb = last;
    else load_bucket<G>(table, st.cur, st.cb);
    return st.cb.has_empty() && try_insert<G>(table, st.cur, st.tag, st.cb) >= 0;
}

// One step of Alg. 1's eviction chain: displace a random slot, carry the
// displaced fingerprint to its other bucket, try there.
template <class G, int HASH, int POL, bool KEEP>
__device__ __forceinline__ bool dfs_level(typename G::W *table, const Place &pl,
                                          Search<G> &st) {
    const int s = int(splitmix_at(st.rs, ++st.n) % uint64_t(G::B));
    if (!st.have) load_bucket<G>(table, st.cur, st.cb);
    const uint32_t ev = swap_slot<G>(table, st.cur, s, st.tag, st.cb);
    ++st.kicks;
    if (ev == 0) return true;
    st.tag = ev;
    st.cur = move_tag<G, HASH, POL>(st.cur, st.tag, pl);
    st.have = KEEP;
    load_bucket<G>(table, st.cur, st.cb);
    return try_insert<G>(table, st.cur, st.tag, st.cb) >= 0;
}

// A whole search by one lane; false: the bound was reached, and st.cur and
// st.tag are the fingerprint dropped.
template <class G, int HASH, int POL, int PW, bool KEEP>
__device__ __forceinline__ bool evict_bfs(typename G::W *table, const Place &pl,
                                          Search<G> &st, uint32_t max_evict) {
    while (st.n < max_evict)
        if (bfs_level<G, HASH, POL, PW, KEEP>(table, pl, st)) return true;
    return false;
}

template <class G, int HASH, int POL, bool KEEP>
__device__ __forceinline__ bool evict_dfs(typename G::W *table, const Place &pl,
                                          Search<G> &st, uint32_t max_evict) {
    while (st.n < max_evict)
        if (dfs_level<G, HASH, POL, KEEP>(table, pl, st)) return true;
    return false;
}

// ------------------------------------------------------------------ insert

// One launch per batch, in two passes per block.
//  1. Direct pass (Alg. 1 phase 1) over the block's grid-stride share of the
//     keys.  Keys whose two buckets are full go to the block's own segment of
//     the eviction queue, queue[blockIdx * seg ...], through a wave-aggregated
//     LDS counter: no global atomic is involved in the hand-off.
//  2. Eviction pass (BFS of Sec. 4.6.1 or the random walk of Alg. 1) over
//     that segment.
// Within an insert launch slots only ever go from EMPTY to full (evictions
// replace a fingerprint in place), so a queued key's two buckets are still
// full when its eviction starts: this is one legal interleaving of the
// paper's concurrent insert.  Deferring evictions keeps the common path's
// wave64 lanes free of eviction-chain divergence, and blocks in different
// passes overlap the read-heavy direct work with the atomic-heavy evictions.
//
// With R = Rest the launch takes what a partitioned insert left over
// (cf_bulk.hpp) instead of keys [0, n): block b runs the searches of its share
// of one part's list, entries in a full i2 whose i1 is full too, and the last
// rest.extra blocks take shares of the overflow list from the start.  The
// entries' draws come from index, bucket and tag (their keys lie scattered
// in memory, a request each).  The keys' flags and kick counts already hold
// 1 and 0 then, so only what differs is written (single bytes at random
// places cost a request each as well).
template <class G, int HASH, int EVICT, int POL, int PW, class R>
__global__ __launch_bounds__(kBlock) void insert_kernel(
    typename G::W *__restrict__ table, Place pl, const uint64_t *__restrict__ keys,
    uint64_t n, uint8_t *__restrict__ ok, uint32_t *__restrict__ kicks, Counters *ctr,
    uint32_t *__restrict__ queue, uint64_t seg, LostLog log, uint32_t max_evict,
    uint64_t seed, R rest) {
    constexpr bool left = std::is_same<R, Rest>::value;
    __shared__ uint32_t s_qn, s_take;
    if (threadIdx.x == 0) s_qn = s_take = 0;
    __syncthreads();
    uint32_t *myq = queue + uint64_t(blockIdx.x) * seg;
    unsigned long long placed = 0;
    uint64_t stride = uint64_t(gridDim.x) * kBlock;
    uint64_t i = uint64_t(blockIdx.x) * kBlock + threadIdx.x;
    const uint32_t *ovl = nullptr;  // a share of the overflow list
    uint32_t part = 0;
    uint64_t ent0 = 0, ents = 0;    // a share of a part's list
    if constexpr (left) {
        for (; i < rest.ncursors; i += stride) rest.cursors[i] = 0;
        const uint32_t lists = rest.parts * rest.split;
        const bool searches = blockIdx.x < lists;
        part = searches ? blockIdx.x / rest.split : rest.parts;
        const uint64_t share = searches ? blockIdx.x % rest.split : blockIdx.x - lists;
        const uint64_t of = searches ? rest.split : rest.extra;
        const uint64_t len = rest.list_n[part];
        const uint64_t lo = len * share / of;
        const uint64_t have = len * (share + 1) / of - lo;
        i = threadIdx.x;
        stride = kBlock;
        if (searches) {
            ent0 = uint64_t(part) * rest.cap + lo;
            ents = have;
            n = 0;
        } else {
            ovl = rest.ovl + lo;
            myq = queue + lo;
            seg = n = have;
        }
    }
    const int lane = threadIdx.x & 63;
    for (; i < n; i += stride) {
        const uint64_t at = left ? ovl[i] : i;
        const uint64_t key = __builtin_nontemporal_load(keys + at);
        const Derived d = derive<G, HASH, POL>(key, pl);
        Bucket<G> bk;
        load_bucket<G>(table, d.i1, bk);
        bool done = try_insert<G>(table, d.i1, d.t1, bk) >= 0;
        if (!done) {
            load_bucket<G>(table, d.i2, bk);
            done = try_insert<G>(table, d.i2, d.t2, bk) >= 0;
        }
        placed += done;
        if (!left) {
            if (ok) ok[at] = uint8_t(done);
            if (kicks) kicks[at] = 0;
        }
        const uint64_t need = __ballot(!done);
        if (need) {
            const int leader = __builtin_ctzll(need);
            uint32_t base = 0;
            if (lane == leader) base = atomicAdd(&s_qn, uint32_t(__popcll(need)));
            base = __shfl(base, leader, 64);
            const uint32_t pos = base + uint32_t(__popcll(need & ((1ull << lane) - 1ull)));
            if (!done && pos < seg) myq[pos] = uint32_t(at);
        }
    }
    __syncthreads();
    const uint32_t qn = ents ? uint32_t(ents) : s_qn < seg ? s_qn : uint32_t(seg);
    Search<G> st;
    uint32_t idx = 0;
    auto begin = [&](uint32_t q) {
        if constexpr (left) {
            if (ents) {
                const Ent e = unpack_ent<G::F>(rest.list.a[ent0 + q],
                                               G::F == 32 ? rest.list.b[ent0 + q] : 0u);
                idx = e.idx;
                Derived d;
                d.i2 = (part << rest.shift) + e.bucket;
                d.t1 = d.t2 = e.tag;
                d.i1 = move_tag<G, HASH, POL>(d.i2, d.t1, pl);
                search_start(st, d,
                             (uint64_t(e.tag) << 32) ^ (uint64_t(d.i2) << 20) ^ idx ^ seed);
                return;
            }
        }
        idx = myq[q];
        const uint64_t key = keys[idx];
        search_start(st, derive<G, HASH, POL>(key, pl), key ^ seed);
    };
    auto end = [&](bool done) {
        placed += done;
        if (!done) {
            const unsigned long long slot = atomicAdd(&ctr->failures, 1ull);
            if (slot < log.cap) {
                log.bucket[slot] = st.cur;
                log.tag[slot] = st.tag;
            }
        }
        if (ok && !(left && done)) ok[idx] = uint8_t(done);
        if (kicks && !(left && st.kicks == 0)) kicks[idx] = st.kicks;
    };
    if constexpr (EVICT == 1) {
        // Every step of the random walk is the same few accesses in every
        // lane, so one lane takes one key after another (the scheme below
        // measured 2-3% slower).
        for (uint32_t q = threadIdx.x; q < qn; q += kBlock) {
            begin(q);
            end(evict_dfs<G, HASH, POL, false>(table, pl, st, max_evict));
        }
    } else {
        // A wave steps its lanes' searches level by level, and lanes whose
        // search ended take the next queued keys together once a quarter of
        // the wave is free (taking a key is two dependent loads, which the
        // others wait for).  Searches differ in length by an order of
        // magnitude; run to the end by 64 lanes side by side, most lanes wait
        // for the longest (64 MiB build at load 0.9: 2195 -> 1728 us).
        // A wave takes at most its share of a short queue: lanes on different
        // paths of a level run one path after another, so few lanes in each
        // of four waves end sooner than many in one (2 MiB build: 144 -> 134
        // us).
        constexpr bool KEEP = G::B * G::F <= 256;  // larger buckets would cost waves in flight
        constexpr uint32_t NW = kBlock / 64;
        const uint32_t share = (qn + NW - 1) / NW;
        bool busy = false, more = qn != 0;
        while (true) {
            const uint64_t idle = __ballot(!busy);
            if (more && __popcll(idle) >= kRefill) {
                const int leader = __builtin_ctzll(idle);
                const uint32_t free = uint32_t(__popcll(idle));
                const uint32_t take = free < share ? free : share;
                uint32_t base = 0;
                if (lane == leader) base = atomicAdd(&s_take, take);
                base = __shfl(base, leader, 64);
                more = base + take < qn;
                const uint32_t k = uint32_t(__popcll(idle & ((1ull << lane) - 1ull)));
                const uint32_t q = base + k;
                if (!busy && k < take && q < qn) {
                    begin(q);
                    busy = true;
                }
            }
            if (__ballot(busy) == 0) break;  // nothing taken: the queue is empty
            if (!busy) continue;
            bool done = false;
            if (st.n < max_evict) done = bfs_level<G, HASH, POL, PW, KEEP>(table, pl, st);
            if (!done && st.n < max_evict) continue;
            busy = false;
            end(done);
        }
    }
    block_add(ctr, placed);
}

// ------------------------------------------------------------- utilities

// Occupancy recount after an import: non-empty slots over the whole table.
template <class G>
__global__ __launch_bounds__(kBlock) void recount_kernel(const typename G::W *__restrict__ table,
                                                         uint64_t nwords, Counters *ctr) {
    using W = typename G::W;
    constexpr W HI = lane_repeat<W, G::F>(W(1)) << (G::F - 1);
    unsigned long long c = 0;
    const uint64_t stride = uint64_t(gridDim.x) * kBlock;
    for (uint64_t i = uint64_t(blockIdx.x) * kBlock + threadIdx.x; i < nwords; i += stride) {
        const W nz = ~zero_lanes<W, G::F>(table[i]) & HI;
        if constexpr (sizeof(W) == 8) c += __popcll(nz);
        else c += __popc(nz);
    }
    block_add(ctr, c);
}

__device__ __forceinline__ void clear_counters(Counters *ctr) {
    const int t = threadIdx.x;
    if (t < kStripes) ctr->count[t].v = 0;
    if (t == 0) {
        ctr->failures = 0;
        ctr->total = 0;
    }
}

static __global__ void clear_counters_kernel(Counters *ctr) { clear_counters(ctr); }

// total = sum of the count stripes (one wave).
static __global__ void sum_counts_kernel(Counters *ctr) {
    unsigned long long v = threadIdx.x < kStripes ? ctr->count[threadIdx.x].v : 0ull;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if (threadIdx.x == 0) ctr->total = v;
}

// An empty filter: table and counters.
static __global__ __launch_bounds__(kBlock) void reset_kernel(uint64_t *__restrict__ p, uint64_t n,
                                                              Counters *ctr) {
    const uint64_t stride = uint64_t(gridDim.x) * kBlock;
    if (blockIdx.x == 0) clear_counters(ctr);
    for (uint64_t i = uint64_t(blockIdx.x) * kBlock + threadIdx.x; i < n; i += stride) p[i] = 0;
}

}  // namespace cfk
