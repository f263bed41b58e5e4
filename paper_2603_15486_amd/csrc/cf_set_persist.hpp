// cf_set_persist.hpp -- the persistent form of a filter set's mixed batch:
// one cooperative launch runs the whole batch (partition, queries, deletes,
// inserts) with grid-wide barriers between the phases, instead of a
// partition launch and one launch per (phase, class).
//
// The phases and their order are those of cf_set.h's batch semantics: every
// query sees its filter as it was before the batch (Sec. 4.4: a query must
// not overlap a write), then all deletes run, then all inserts (inserts and
// deletes never overlap, which the delete's fetch-AND relies on).  Within a
// phase each block takes chunks c = blockIdx, blockIdx + grid, ... and runs
// every bin of that phase in the chunk, dispatching on the bin's bucket size
// b at run time; the per-bin work is the class kernels' own (query_bin,
// delete_bin, insert_bin).  A set qualifies when all its filters share the
// fingerprint width, hash and placement (any mix of b).
//
// Grid barrier.  Every block must be resident at once, which the cooperative
// launch guarantees (it refuses a grid that cannot be).  The blocks are split
// into kBarrierGroups groups (block k in group k mod kBarrierGroups), each
// with an arrival counter and a generation word on lines of their own:
// device-scope atomics on one address are performed one after another at
// the memory side, so a single counter for a grid of a thousand blocks would
// cost a thousand serialised round trips per barrier, and a thousand blocks
// polling one word queue on one memory channel.  Each block's thread 0
// publishes the block's writes (agent-scope release) and adds one to its
// group's counter; the last of a group resets it and adds one to the top
// counter; the last group's last block resets that and advances every
// group's generation (release).  The others poll their group's generation
// (agent-scope acquire), sleeping about a microsecond between polls.  The
// wait is bounded: past `limit` ticks of the constant-rate wall clock, or
// once another block has given up, the block marks the control block's
// error word and leaves the kernel without touching the batch again.  A block
// never enters a phase unless the barrier before it completed, so an
// abandoned batch does no out-of-order work; a marked error also makes later
// launches return at once until the host clears the control block
// (cf_set_set_shape).
#pragma once

#include "cf_set_kernels.hpp"
#include "cf_set_requests.hpp"

namespace cfs {

// Control block of the persistent path, one per set; each word on its own
// 128-byte line.  Zeroed at creation and when the host clears an error.
constexpr uint32_t kBarrierGroups = 32;

struct alignas(128) CtlWord {
    unsigned int v;
    unsigned int pad[31];
};

// Wall-clock ticks of the last batch: [0] when block 0 started, [k] when
// barrier k (k = 1, 2, 3: after the partition, the queries, the deletes)
// completed; written by block 0 and by each barrier's releaser.
struct alignas(128) CtlStamps {
    unsigned long long t[4];
    unsigned long long pad[12];
};

struct PersistCtl {
    CtlWord top;                        // groups arrived at the current barrier
    CtlWord error;                      // 1 once a barrier wait gave up
    CtlWord arrive[kBarrierGroups];     // blocks of each group arrived
    CtlWord gen[kBarrierGroups];        // barriers completed, per group
    CtlStamps stamp;
};

// The classes a launch covers (all of one hash and placement, and of one f
// unless the kernel is for any): their numbers in the set, bucket sizes b and
// fingerprint widths f.
struct ClassB {
    uint8_t b[kMaxClasses];
    uint8_t f[kMaxClasses];
    uint8_t id[kMaxClasses];
    uint32_t n;
};

__device__ __forceinline__ unsigned int ld_relaxed(const unsigned int *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned int add_relaxed(unsigned int *p) {
    return __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void st_relaxed(unsigned int *p, unsigned int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The grid barrier described above.  Returns false if the block must leave
// (this or another block gave up).  Every thread of the block calls it; `gen`
// is the block's count of completed barriers (the same in every thread).
// Ordering is by fences around relaxed atomics: an agent-scope release fence
// writes the L2's dirty lines back and an acquire fence invalidates the
// L2's lines that other agents' caches may have changed, so they are issued
// once per arrival and once after the wait, never per poll (an acquiring
// poll would invalidate the L2 of every waiting block's compute unit again
// and again, under the blocks of that L2 still working).  Each arrival is a
// release fence then a relaxed add; the group's last and the last group
// acquire what came before them (the adds form one release sequence per
// counter) and release it on; the waiters acquire after their poll sees the
// generation move.
__device__ __forceinline__ bool grid_sync(PersistCtl *ctl, unsigned int &gen, uint64_t limit,
                                          int stamp) {
    __shared__ int s_ok;
    __syncthreads();
    if (threadIdx.x == 0) {
        int ok = 1;
        const uint32_t ngroups = gridDim.x < kBarrierGroups ? gridDim.x : kBarrierGroups;
        const uint32_t g = blockIdx.x % kBarrierGroups;
        const uint32_t members = (gridDim.x - g + kBarrierGroups - 1) / kBarrierGroups;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // this block's writes first
        bool released = false;
        if (add_relaxed(&ctl->arrive[g].v) == members - 1) {  // the group's last
            // reset for the next barrier, then acquire the group and release
            // it (with the reset) to the top counter
            st_relaxed(&ctl->arrive[g].v, 0u);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
            if (add_relaxed(&ctl->top.v) == ngroups - 1) {  // the last group: release all
                st_relaxed(&ctl->top.v, 0u);
                ctl->stamp.t[stamp] = wall_clock64();
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
                for (uint32_t k = 0; k < ngroups; ++k) st_relaxed(&ctl->gen[k].v, gen + 1);
                released = true;
            }
        }
        if (!released) {
            // A poll is a device-coherent load served past the L2; a waiting
            // block sleeps about a microsecond between polls and looks at the
            // error word only every 16th time.
            const uint64_t t0 = wall_clock64();
            uint32_t polls = 0;
            while (ld_relaxed(&ctl->gen[g].v) == gen) {
                if (wall_clock64() - t0 > limit ||
                    ((++polls & 15u) == 0 && ld_relaxed(&ctl->error.v))) {
                    st_relaxed(&ctl->error.v, 1u);
                    ok = 0;
                    break;
                }
                __builtin_amdgcn_s_sleep(32);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // the other blocks' writes
        s_ok = ok;
    }
    __syncthreads();
    gen += 1;
    return s_ok != 0;
}

template <int F, int HASH, int POL, int BT, int BMAX>
__global__ __launch_bounds__(BT) void persist_kernel(Batch bt, const SetFilter *__restrict__ filters,
                                                     const uint8_t *__restrict__ cls, ClassB cb,
                                                     uint32_t nfilters, uint32_t ncls,
                                                     uint32_t chunk, Scratch sc, PersistCtl *ctl,
                                                     uint64_t limit, uint32_t wave_bfs) {
    __shared__ uint32_t hist[kMaxBins + 1];
    __shared__ uint32_t base[kMaxBins + 1];
    __shared__ int lds[kLdsFilters];
    __shared__ uint32_t s_qn;
    __shared__ unsigned int s_gen;
    __shared__ int s_err;
    if (threadIdx.x == 0) {
        if (blockIdx.x == 0) ctl->stamp.t[0] = wall_clock64();
        s_err = int(ld_relaxed(&ctl->error.v));
        s_gen = ld_relaxed(&ctl->gen[blockIdx.x % kBarrierGroups].v);
    }
    __syncthreads();
    if (s_err) return;  // an earlier batch was abandoned: nothing runs until cleared
    unsigned int gen = s_gen;
    const uint32_t nb = 3 * ncls;
    const uint64_t n = batch_n(bt);
    const uint64_t nchunks = (n + chunk - 1) / chunk;
    Tally<BT> tally{lds, nfilters};

    // phase 0: sort every chunk by (kind, class)
    for (uint64_t cid = blockIdx.x; cid < nchunks; cid += gridDim.x)
        partition_chunk<BT>(bt, n, cls, nfilters, ncls, chunk, cid, sc, hist, base);
    if (!grid_sync(ctl, gen, limit, 1)) return;

    // phase 1: queries (Alg. 2)
    for (uint64_t cid = blockIdx.x; cid < nchunks; cid += gridDim.x) {
        const uint32_t *seg = sc.sorted + cid * chunk;
        for (uint32_t c = 0; c < ncls; ++c) {
            uint32_t b0, b1;
            bin_range(sc, nb, cid, c, b0, b1);
            if (b0 < b1)
                with_b<F, BMAX>(cb.f[c], cb.b[c], [&](auto g) {
                    query_bin<decltype(g), HASH, POL, BT>(ChunkSrc{bt, seg, cid * chunk}, filters, b0, b1);
                });
        }
    }
    if (!grid_sync(ctl, gen, limit, 2)) return;

    // phase 2: deletes (Alg. 3)
    tally.init();
    for (uint64_t cid = blockIdx.x; cid < nchunks; cid += gridDim.x) {
        const uint32_t *seg = sc.sorted + cid * chunk;
        for (uint32_t c = 0; c < ncls; ++c) {
            uint32_t b0, b1;
            bin_range(sc, nb, cid, ncls + c, b0, b1);
            if (b0 < b1)
                with_b<F, BMAX>(cb.f[c], cb.b[c], [&](auto g) {
                    delete_bin<decltype(g), HASH, POL, BT>(ChunkSrc{bt, seg, cid * chunk}, filters, b0, b1, tally);
                });
        }
    }
    tally.flush(filters);
    if (!grid_sync(ctl, gen, limit, 3)) return;

    // phase 3: inserts (Alg. 1 with the eviction search of Sec. 4.6.1)
    tally.init();
    for (uint64_t cid = blockIdx.x; cid < nchunks; cid += gridDim.x) {
        const uint64_t at = cid * chunk;
        for (uint32_t c = 0; c < ncls; ++c) {
            uint32_t b0, b1;
            bin_range(sc, nb, cid, 2 * ncls + c, b0, b1);
            if (b0 < b1)  // uniform across the block: insert_bin has block barriers
                with_b<F, BMAX>(cb.f[c], cb.b[c], [&](auto g) {
                    insert_bin<decltype(g), HASH, POL, BT>(ChunkSrc{bt, sc.sorted + at, at}, filters,
                                                           b0, b1, sc.queue + at + b0, &s_qn,
                                                           tally, wave_bfs);
                });
        }
    }
    tally.flush(filters);
}

// ------------------------------------------------ one launch per phase
// The class-kernel form with the classes of each phase fused into one
// launch: grid = chunks x classes, block k working on the bin of the launch's
// class k mod cb.n in chunk k / cb.n, with that class's b chosen at run time
// (with_b).  A set whose classes differ in f, hash or placement has one such
// launch per phase and group of classes that agree, or for small batches per
// group that agrees in hash and placement (F = 0: f chosen per block too).
// The queries of every class run side by side in one launch, then every
// delete, then every insert, all on the caller's stream: no side streams,
// and a captured batch is a straight chain of four kernels (partition and
// three phases) if all classes agree.  Bins beyond the batch's chunks are empty (the
// partition writes empty offsets for them), and a block with an empty bin
// returns at once, before any barrier.

// The partition and the queries of the launch's classes in one: a chunk's
// operations are loaded once, in order, and sorted by bin in LDS; the queries
// run from LDS, their flags are collected there and written in order, and
// what the later launches need (every other operation's entry and the bin
// starts) goes to the scratch as in partition_chunk.  Apart, the partition
// read every kind and id twice and the queries then fetched entry, id and key
// one behind another from scattered places before their first probe.
// Per 2^22 operations over 256 filters: 19 + 130 us apart, 134 together, 26 of
// them before the first probe (a batch of invalid operations).  512 threads:
// with 256 and chunks of 1024 to 4096 the batch took 259-277 us for 257.
// LDS per block: 13 bytes per operation of the chunk.
constexpr int kFrontBlock = 512;
constexpr int kFrontItems = int(kMaxChunk) / kFrontBlock;
inline size_t front_lds(uint32_t chunk) { return size_t(chunk) * 13; }

template <int F, int HASH, int POL, int BMAX>
__global__ __launch_bounds__(kFrontBlock) void phase_front_kernel(
    Batch bt, const SetFilter *__restrict__ filters, const uint8_t *__restrict__ cls, ClassB cb,
    uint32_t nfilters, uint32_t ncls, uint32_t chunk, Scratch sc) {
    extern __shared__ __align__(16) uint8_t front_mem[];
    uint64_t *s_key = reinterpret_cast<uint64_t *>(front_mem);
    uint32_t *s_ent = reinterpret_cast<uint32_t *>(s_key + chunk);
    uint8_t *s_res = reinterpret_cast<uint8_t *>(s_ent + chunk);
    __shared__ uint32_t hist[kMaxBins + 1], base[kMaxBins + 2];
    __shared__ uint8_t s_b[kMaxClasses];  // b of the launch's classes, 0: not one of them
    __shared__ uint8_t s_f[kMaxClasses];
    const uint64_t n = batch_n(bt);
    const uint64_t lo = uint64_t(blockIdx.x) * chunk;
    const uint32_t have = lo >= n ? 0u : n - lo < chunk ? uint32_t(n - lo) : chunk;
    const uint32_t nb = 3 * ncls, t = threadIdx.x;
    for (uint32_t j = t; j <= nb; j += kFrontBlock) hist[j] = 0;
    if (t < kMaxClasses) s_b[t] = 0;
    __syncthreads();
    if (t < cb.n) {
        s_b[cb.id[t]] = cb.b[t];
        s_f[cb.id[t]] = cb.f[t];
    }
    uint64_t key[kFrontItems];
    uint32_t fid[kFrontItems], bin[kFrontItems], rank[kFrontItems];
#pragma unroll
    for (int k = 0; k < kFrontItems; ++k) {
        const uint32_t j = uint32_t(k) * kFrontBlock + t;
        bin[k] = ~0u;
        if (j < have) {
            bin[k] = bt.ops[lo + j];
            fid[k] = bt.fids[lo + j];
            key[k] = bt.keys[lo + j];
        }
    }
#pragma unroll
    for (int k = 0; k < kFrontItems; ++k)
        if (bin[k] != ~0u) {
            uint32_t x = nb;
            if (bin[k] <= 2u && fid[k] < nfilters) {
                const uint32_t c = cls[fid[k]];
                if (c < ncls) x = bin[k] * ncls + c;  // 0xFF: filter detached
            }
            bin[k] = x;
            rank[k] = atomicAdd(&hist[x], 1u);
        }
    __syncthreads();
    if (t < 64) {  // bin starts: one wave, at most 49 bins
        const uint32_t mine = t <= nb ? hist[t] : 0u;
        uint32_t inc = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = __shfl_up(inc, d, 64);
            if (t >= uint32_t(d)) inc += o;
        }
        if (t <= nb) {
            base[t] = inc - mine;
            sc.binoff[uint64_t(blockIdx.x) * (nb + 1) + t] = inc - mine;
        }
    }
    __syncthreads();
    const uint32_t nq = base[ncls];  // queries come first
#pragma unroll
    for (int k = 0; k < kFrontItems; ++k)
        if (bin[k] != ~0u) {
            const uint32_t j = uint32_t(k) * kFrontBlock + t;
            const uint32_t p = base[bin[k]] + rank[k];
            s_ent[p] = sorted_entry(fid[k], j);
            if (p < nq) s_key[p] = key[k];
        }
    __syncthreads();
    for (uint32_t p = t; p < have; p += kFrontBlock) sc.sorted[lo + p] = s_ent[p];
    uint32_t c = 0;
    for (uint32_t p = t; p < nq; p += kFrontBlock) {
        while (p >= base[c + 1]) ++c;
        const uint32_t v = s_ent[p];
        bool hit = false;
        with_b<F, BMAX>(s_f[c], s_b[c], [&](auto g) {
            hit = query_one<decltype(g), HASH, POL>(filters[v / kMaxChunk], s_key[p]);
        });
        s_res[v & (kMaxChunk - 1)] = uint8_t(hit);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kFrontItems; ++k) {
        if (bin[k] == ~0u) continue;
        const uint32_t j = uint32_t(k) * kFrontBlock + t;
        if (bin[k] == nb) bt.results[lo + j] = 0xFF;
        else if (bin[k] < ncls && s_b[bin[k]]) bt.results[lo + j] = s_res[j];
    }
}

template <int F, int HASH, int POL, int BMAX>
__global__ __launch_bounds__(kBlock) void phase_query_kernel(Batch bt,
                                                             const SetFilter *__restrict__ filters,
                                                             ClassB cb, uint32_t ncls,
                                                             uint32_t chunk, Scratch sc) {
    const uint64_t cid = blockIdx.x / cb.n;
    const uint32_t c = blockIdx.x % cb.n;
    uint32_t b0, b1;
    bin_range(sc, 3 * ncls, cid, cb.id[c], b0, b1);
    if (b0 >= b1) return;
    const uint32_t *seg = sc.sorted + cid * chunk;
    with_b<F, BMAX>(cb.f[c], cb.b[c], [&](auto g) {
        query_bin<decltype(g), HASH, POL, kBlock>(ChunkSrc{bt, seg, cid * chunk}, filters, b0, b1);
    });
}

template <int F, int HASH, int POL, int BMAX>
__global__ __launch_bounds__(kBlock) void phase_delete_kernel(Batch bt,
                                                              const SetFilter *__restrict__ filters,
                                                              ClassB cb, uint32_t nfilters,
                                                              uint32_t ncls, uint32_t chunk,
                                                              Scratch sc) {
    __shared__ int lds[kLdsFilters];
    const uint64_t cid = blockIdx.x / cb.n;
    const uint32_t c = blockIdx.x % cb.n;
    uint32_t b0, b1;
    bin_range(sc, 3 * ncls, cid, ncls + cb.id[c], b0, b1);
    if (b0 >= b1) return;  // the same in every thread of the block
    Tally<kBlock> tally{lds, nfilters};
    tally.init();
    const uint32_t *seg = sc.sorted + cid * chunk;
    with_b<F, BMAX>(cb.f[c], cb.b[c], [&](auto g) {
        delete_bin<decltype(g), HASH, POL, kBlock>(ChunkSrc{bt, seg, cid * chunk}, filters, b0, b1, tally);
    });
    tally.flush(filters);
}

template <int F, int HASH, int POL, int BMAX>
__global__ __launch_bounds__(kBlock) void phase_insert_kernel(Batch bt,
                                                              const SetFilter *__restrict__ filters,
                                                              ClassB cb, uint32_t nfilters,
                                                              uint32_t ncls, uint32_t chunk,
                                                              Scratch sc, uint32_t wave_bfs) {
    __shared__ int lds[kLdsFilters];
    __shared__ uint32_t s_qn;
    const uint64_t cid = blockIdx.x / cb.n;
    const uint32_t c = blockIdx.x % cb.n;
    uint32_t b0, b1;
    bin_range(sc, 3 * ncls, cid, 2 * ncls + cb.id[c], b0, b1);
    if (b0 >= b1) return;  // the same in every thread of the block
    Tally<kBlock> tally{lds, nfilters};
    tally.init();
    const uint64_t at = cid * chunk;
    with_b<F, BMAX>(cb.f[c], cb.b[c], [&](auto g) {
        insert_bin<decltype(g), HASH, POL, kBlock>(ChunkSrc{bt, sc.sorted + at, at}, filters, b0, b1,
                                                   sc.queue + at + b0, &s_qn, tally, wave_bfs);
    });
    tally.flush(filters);
}

// Host launchers of the three phase kernels for one (f, hash, placement).
// grid = chunks x classes of the launch; ncls = classes of the set.
struct PhaseLaunch {
    void (*front)(Batch, const SetFilter *, const uint8_t *cls, ClassB, uint32_t nfilters,
                  uint32_t ncls, uint32_t chunk, Scratch, int chunks, hipStream_t) = nullptr;
    void (*query)(Batch, const SetFilter *, ClassB, uint32_t ncls, uint32_t chunk, Scratch,
                  int grid, hipStream_t) = nullptr;
    void (*del)(Batch, const SetFilter *, ClassB, uint32_t nfilters, uint32_t ncls,
                uint32_t chunk, Scratch, int grid, hipStream_t) = nullptr;
    void (*ins)(Batch, const SetFilter *, ClassB, uint32_t nfilters, uint32_t ncls,
                uint32_t chunk, Scratch, uint32_t wave_bfs, int grid, hipStream_t) = nullptr;
    void (*req_query)(const ReqSpan &, const ReqEntry *, const SetFilter *, int grid,
                      hipStream_t) = nullptr;
    void (*req_del)(const ReqSpan &, const ReqEntry *, const SetFilter *, uint32_t nfilters,
                    int grid, hipStream_t) = nullptr;
    void (*req_ins)(const ReqSpan &, const ReqEntry *, const SetFilter *, uint32_t nfilters,
                    uint32_t *queue, uint32_t wave_bfs, int grid, hipStream_t) = nullptr;
};

template <int F, int HASH, int POL, int BMAX>
struct PhaseInst {
    static void front(Batch bt, const SetFilter *fl, const uint8_t *cls, ClassB cb, uint32_t nf,
                      uint32_t ncls, uint32_t chunk, Scratch sc, int chunks, hipStream_t s) {
        phase_front_kernel<F, HASH, POL, BMAX><<<chunks, kFrontBlock, front_lds(chunk), s>>>(
            bt, fl, cls, cb, nf, ncls, chunk, sc);
    }
    static void query(Batch bt, const SetFilter *fl, ClassB cb, uint32_t ncls, uint32_t chunk,
                      Scratch sc, int grid, hipStream_t s) {
        phase_query_kernel<F, HASH, POL, BMAX><<<grid, kBlock, 0, s>>>(bt, fl, cb, ncls, chunk, sc);
    }
    static void del(Batch bt, const SetFilter *fl, ClassB cb, uint32_t nf, uint32_t ncls,
                    uint32_t chunk, Scratch sc, int grid, hipStream_t s) {
        phase_delete_kernel<F, HASH, POL, BMAX><<<grid, kBlock, 0, s>>>(bt, fl, cb, nf, ncls, chunk, sc);
    }
    static void ins(Batch bt, const SetFilter *fl, ClassB cb, uint32_t nf, uint32_t ncls,
                    uint32_t chunk, Scratch sc, uint32_t wave_bfs, int grid, hipStream_t s) {
        phase_insert_kernel<F, HASH, POL, BMAX>
            <<<grid, kBlock, 0, s>>>(bt, fl, cb, nf, ncls, chunk, sc, wave_bfs);
    }
    static void req_query(const ReqSpan &sp, const ReqEntry *tab, const SetFilter *fl, int grid,
                          hipStream_t s) {
        req_query_kernel<F, HASH, POL, BMAX><<<grid, kBlock, 0, s>>>(sp, tab, fl);
    }
    static void req_del(const ReqSpan &sp, const ReqEntry *tab, const SetFilter *fl, uint32_t nf,
                        int grid, hipStream_t s) {
        req_delete_kernel<F, HASH, POL, BMAX><<<grid, kBlock, 0, s>>>(sp, tab, fl, nf);
    }
    static void req_ins(const ReqSpan &sp, const ReqEntry *tab, const SetFilter *fl, uint32_t nf,
                        uint32_t *queue, uint32_t wave_bfs, int grid, hipStream_t s) {
        req_insert_kernel<F, HASH, POL, BMAX>
            <<<grid, kBlock, 0, s>>>(sp, tab, fl, nf, queue, wave_bfs);
    }
};

// Fills the query and delete launchers (INSERT = false) or the insert
// launcher (INSERT = true) of L for sets whose buckets have at most bmax
// slots; false for an unknown hash or placement.
template <int F, bool INSERT, int BMAX>
bool pick_phase_fb(uint32_t hash, uint32_t placement, PhaseLaunch &L) {
    if (hash > 1 || placement > 1) return false;
    auto fill = [&](auto inst) {
        using I = decltype(inst);
        if constexpr (INSERT) {
            L.ins = &I::ins;
            if constexpr (F != 0) L.req_ins = &I::req_ins;
        } else {
            L.front = &I::front;
            L.query = &I::query;
            L.del = &I::del;
            if constexpr (F != 0) {
                L.req_query = &I::req_query;
                L.req_del = &I::req_del;
            }
        }
    };
    if (hash == 0)
        placement ? fill(PhaseInst<F, 0, 1, BMAX>{}) : fill(PhaseInst<F, 0, 0, BMAX>{});
    else
        placement ? fill(PhaseInst<F, 1, 1, BMAX>{}) : fill(PhaseInst<F, 1, 0, BMAX>{});
    return true;
}

// Launchers for classes of any f (no request kernels): query and delete in
// cf_set_any.hip, insert in cf_set_insi_any.hip (built at -O1).
bool pick_phase_any(uint32_t hash, uint32_t placement, PhaseLaunch &out);
bool pick_phase_insert_any(uint32_t hash, uint32_t placement, PhaseLaunch &out);

template <int F, bool INSERT>
bool pick_phase_f(uint32_t hash, uint32_t placement, uint32_t bmax, PhaseLaunch &L) {
    return bmax <= 16 ? pick_phase_fb<F, INSERT, 16>(hash, placement, L)
                      : pick_phase_fb<F, INSERT, 32>(hash, placement, L);
}

// Per fingerprint width: query and delete in cf_set_inst_f*.hip, insert in
// cf_set_persist_insi_f*.hip (built at -O1).  The request kernels' launchers
// (cf_set_requests.hpp) come with them.
bool pick_phase_f8(uint32_t hash, uint32_t placement, uint32_t bmax, PhaseLaunch &out);
bool pick_phase_f16(uint32_t hash, uint32_t placement, uint32_t bmax, PhaseLaunch &out);
bool pick_phase_f32(uint32_t hash, uint32_t placement, uint32_t bmax, PhaseLaunch &out);
bool pick_phase_insert_f8(uint32_t hash, uint32_t placement, uint32_t bmax,
                          PhaseLaunch &out);
bool pick_phase_insert_f16(uint32_t hash, uint32_t placement, uint32_t bmax,
                          PhaseLaunch &out);
bool pick_phase_insert_f32(uint32_t hash, uint32_t placement, uint32_t bmax,
                          PhaseLaunch &out);

// Host side: the kernel for the set's (f, hash, placement) at each block size.
constexpr int kPersistBlocks[2] = {256, 512};

struct PersistLaunch {
    const void *kern[2] = {nullptr, nullptr};  // block of kPersistBlocks[k] threads
};

template <int F, int HASH, int POL, int BMAX>
void fill_persist(PersistLaunch &L) {
    L.kern[0] = reinterpret_cast<const void *>(&persist_kernel<F, HASH, POL, 256, BMAX>);
    L.kern[1] = reinterpret_cast<const void *>(&persist_kernel<F, HASH, POL, 512, BMAX>);
}

template <int F, int BMAX>
bool pick_persist_fb(uint32_t hash, uint32_t placement, PersistLaunch &L) {
    if (hash > 1 || placement > 1) return false;
    if (hash == 0) placement ? fill_persist<F, 0, 1, BMAX>(L) : fill_persist<F, 0, 0, BMAX>(L);
    else placement ? fill_persist<F, 1, 1, BMAX>(L) : fill_persist<F, 1, 0, BMAX>(L);
    return true;
}

// The kernels for a set whose buckets have at most bmax slots.
template <int F>
bool pick_persist_f(uint32_t hash, uint32_t placement, uint32_t bmax, PersistLaunch &L) {
    return bmax <= 16 ? pick_persist_fb<F, 16>(hash, placement, L)
                      : pick_persist_fb<F, 32>(hash, placement, L);
}

// Per fingerprint width, in cf_set_persist_insi_f*.hip (built at -O1 like
// every unit with insert code).
bool pick_persist_f8(uint32_t hash, uint32_t placement, uint32_t bmax, PersistLaunch &out);
bool pick_persist_f16(uint32_t hash, uint32_t placement, uint32_t bmax, PersistLaunch &out);
bool pick_persist_f32(uint32_t hash, uint32_t placement, uint32_t bmax, PersistLaunch &out);

}  // namespace cfs
