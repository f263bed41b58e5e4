// cf_set_requests.hpp -- a batch of whole requests on a filter set, run
// without laying it out as a mixed batch.
//
// A request is one kind of operation on one filter for an array of keys, so
// the host can order a batch's requests by phase and class itself, and no
// device pass has to gather their keys into one array, sort them by bin and
// scatter the flags back (three passes that took a quarter of a batch of
// 2^22 operations: 97 of 390 us).  The kernels here walk a table of requests
// in that order: positions [j0, j1) of the batch belong to one class, a block
// takes kReqOps of them, finds the requests that cover its stretch and reads
// keys and writes flags in the requests' own arrays, in order.  One launch
// per phase and group of classes that share f, hash and placement, with the
// class's b chosen per block.
#pragma once

#include "cf_set_kernels.hpp"

namespace cfs {

// A request as the kernels see it: its keys, flags and filter, and its first
// position in the batch; the table is sorted by position.
struct ReqEntry {
    const uint64_t *keys;
    uint8_t *results;
    uint32_t off;
    uint32_t fid;
};

// Positions per block: a burst of 1024 requests of 1..2^20 keys took 4.49-4.56
// ms with 512, 4.54 with 1024 and 4.93 with 2048 (7.96 laid out).
constexpr uint32_t kReqOps = 1024;

// One launch: its classes' bucket sizes, and per class the first block, the
// positions [j0, j1) and the table entries [e0, e1).
struct ReqSpan {
    uint32_t n;
    uint8_t b[kMaxClasses];
    uint32_t blk[kMaxClasses];
    uint32_t j0[kMaxClasses], j1[kMaxClasses];
    uint32_t e0[kMaxClasses], e1[kMaxClasses];
};

// Run fn(Geom<f, b>{}) for the bucket sizes the library compiles, up to
// BMAX slots, and fingerprints of f = F bits, or of any width if F = 0.  A
// kernel holds the code of every geometry it may meet and takes the registers
// of the largest: the 32-slot insert path alone limits a kernel to 4 waves
// per SIMD, so sets whose buckets have at most 16 slots get kernels without
// it (BMAX = 16), and kernels for any width are for batches whose launches
// cost more than their work.
template <int F, int BMAX, class Fn>
__device__ __forceinline__ void with_b(uint32_t f, uint32_t b, Fn &&fn) {
    if constexpr (F == 0) {
        if (f == 8) with_b<8, BMAX>(f, b, fn);
        else if (f == 16) with_b<16, BMAX>(f, b, fn);
        else if (f == 32) with_b<32, BMAX>(f, b, fn);
    } else {
        switch (b) {
            case 4: fn(cfk::Geom<F, 4>{}); break;
            case 8: fn(cfk::Geom<F, 8>{}); break;
            case 16: fn(cfk::Geom<F, 16>{}); break;
            case 32:
                if constexpr (BMAX >= 32) fn(cfk::Geom<F, 32>{});
                break;
            default: break;
        }
    }
}

__device__ __forceinline__ uint32_t find_entry(const ReqEntry *tab, uint32_t lo, uint32_t hi,
                                               uint32_t p) {
    while (hi - lo > 1) {  // the last entry of [lo, hi) with off <= p
        const uint32_t mid = (lo + hi) >> 1;
        if (tab[mid].off <= p) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The requests that cover a block's stretch, entries [lo, hi).
struct ReqSrc {
    const ReqEntry *tab;
    uint32_t lo, hi;
    __device__ __forceinline__ Op get(uint32_t p) const {
        const ReqEntry &e = tab[find_entry(tab, lo, hi, p)];
        const uint32_t k = p - e.off;
        return Op{e.fid, e.keys[k], e.results + k};
    }
};

// This block's class, stretch [p0, p1) and requests.  Every thread of the
// block calls it.
__device__ __forceinline__ ReqSrc req_block(const ReqSpan &sp, const ReqEntry *tab, uint32_t &c,
                                            uint32_t &p0, uint32_t &p1) {
    __shared__ uint32_t s_e[2];
    c = 0;
    while (c + 1 < sp.n && blockIdx.x >= sp.blk[c + 1]) ++c;
    p0 = sp.j0[c] + (blockIdx.x - sp.blk[c]) * kReqOps;
    p1 = sp.j1[c] - p0 < kReqOps ? sp.j1[c] : p0 + kReqOps;
    if (threadIdx.x < 2)
        s_e[threadIdx.x] = find_entry(tab, sp.e0[c], sp.e1[c], threadIdx.x ? p1 - 1 : p0);
    __syncthreads();
    return ReqSrc{tab, s_e[0], s_e[1] + 1};
}

template <int F, int HASH, int POL, int BMAX>
__global__ __launch_bounds__(kBlock) void req_query_kernel(ReqSpan sp,
                                                           const ReqEntry *__restrict__ tab,
                                                           const SetFilter *__restrict__ filters) {
    uint32_t c, p0, p1;
    const ReqSrc src = req_block(sp, tab, c, p0, p1);
    with_b<F, BMAX>(F, sp.b[c], [&](auto g) {
        query_bin<decltype(g), HASH, POL, kBlock>(src, filters, p0, p1);
    });
}

template <int F, int HASH, int POL, int BMAX>
__global__ __launch_bounds__(kBlock) void req_delete_kernel(ReqSpan sp,
                                                            const ReqEntry *__restrict__ tab,
                                                            const SetFilter *__restrict__ filters,
                                                            uint32_t nfilters) {
    __shared__ int lds[kLdsFilters];
    uint32_t c, p0, p1;
    const ReqSrc src = req_block(sp, tab, c, p0, p1);
    Tally<kBlock> tally{lds, nfilters};
    tally.init();
    with_b<F, BMAX>(F, sp.b[c], [&](auto g) {
        delete_bin<decltype(g), HASH, POL, kBlock>(src, filters, p0, p1, tally);
    });
    tally.flush(filters);
}

// queue: as many entries as the batch has positions.
template <int F, int HASH, int POL, int BMAX>
__global__ __launch_bounds__(kBlock) void req_insert_kernel(ReqSpan sp,
                                                            const ReqEntry *__restrict__ tab,
                                                            const SetFilter *__restrict__ filters,
                                                            uint32_t nfilters, uint32_t *queue,
                                                            uint32_t wave_bfs) {
    __shared__ int lds[kLdsFilters];
    __shared__ uint32_t s_qn;
    uint32_t c, p0, p1;
    const ReqSrc src = req_block(sp, tab, c, p0, p1);
    Tally<kBlock> tally{lds, nfilters};
    tally.init();
    with_b<F, BMAX>(F, sp.b[c], [&](auto g) {
        insert_bin<decltype(g), HASH, POL, kBlock>(src, filters, p0, p1, queue + p0, &s_qn, tally,
                                                   wave_bfs);
    });
    tally.flush(filters);
}

}  // namespace cfs
