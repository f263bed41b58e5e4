// cf_bulk.hpp -- partitioned insertion of a batch that is large against the
// table (part of the single-filter insert; cf_api.hip chooses when).
//
// What bounds the one-launch insert of a large batch is one device-scope CAS
// per key: atomics execute at the memory side at 20-27 G/s whatever the
// table's size, while the bytes a build needs (keys, flags, table) take a
// tenth of that time.  So the batch is first grouped by table part (a
// contiguous range of buckets that fits in LDS), then one block per part
// loads the part, tries every key's primary bucket with LDS compare-and-swaps
// and stores the part back: the direct attempt of Alg. 1 in i1 without a
// single global atomic and with the table read and written once, in order.
// Keys whose i1 was full go to the part's list, and insert_kernel takes those
// lists through i2 and the eviction search.  For the table this is one legal
// interleaving of the concurrent insert: every attempt in an i1 happens
// before any attempt in an i2.
//
//  bulk_split_kernel    keys -> entries grouped by bin (bin = i1 >> shift)
//  bulk_resplit_kernel  (tables of many parts) entries of one bin -> parts
//  bulk_insert_kernel    one part in LDS: the attempts in i1
//  insert_kernel        the lists left over (Rest)
//
// Bins and parts hold a fixed number of entries, sized by the host from the
// mean of a uniform hash plus eight standard deviations.  Entries beyond it
// (many copies of one key) go to one overflow list instead, which
// insert_kernel runs from the start, so a skewed batch is slower but never
// wrong.
#pragma once

#include "cf_kernels.hpp"

namespace cfk {

constexpr int kSplitBlock = 512;
constexpr int kSplitItems = 8;                            // entries per thread and tile
constexpr int kSplitTile = kSplitBlock * kSplitItems;
constexpr uint32_t kMaxBulkBins = 1024;
constexpr uint32_t kBulkSegs = 8;                         // one per XCD, see bulk_split_kernel
constexpr int kPlaceBlock = 1024;
constexpr int kPlaceItems = 4;
constexpr uint32_t kBulkIdxBits = 27;                     // keys of one partitioned pass
constexpr uint64_t kMaxBulkKeys = 1ull << kBulkIdxBits;

// One entry: the tag as written in i1, the key's index in the pass, and the
// low bits of i1 (its place within the bin).  8 bytes for fingerprints of 8
// and 16 bits (tag | index | bucket bits, so 64 - 27 - f of the latter), and
// 12 bytes in two arrays for 32-bit ones.
struct Ents {
    uint64_t *a;
    uint32_t *b;  // f = 32 only: the index
};

struct Ent {
    uint32_t tag, idx, bucket;
};

struct Raw {  // as loaded: a key, or an entry's words
    uint64_t a;
    uint32_t b;
};

template <int F>
__device__ __forceinline__ uint64_t pack_ent(const Ent &e) {
    if constexpr (F == 32) return uint64_t(e.tag) | (uint64_t(e.bucket) << 32);
    else
        return uint64_t(e.tag) | (uint64_t(e.idx) << F) |
               (uint64_t(e.bucket) << (F + kBulkIdxBits));
}

template <int F>
__device__ __forceinline__ Ent unpack_ent(uint64_t a, uint32_t b) {
    if constexpr (F == 32) return Ent{uint32_t(a), b, uint32_t(a >> 32)};
    else
        return Ent{uint32_t(a) & ((1u << F) - 1u),
                   uint32_t(a >> F) & ((1u << kBulkIdxBits) - 1u),
                   uint32_t(a >> (F + kBulkIdxBits))};
}

// Append one index per active lane to a list behind a global counter.
__device__ __forceinline__ void append_wave(uint32_t *list, uint32_t *count, uint32_t v) {
    const uint64_t on = __ballot(1);
    const int lane = threadIdx.x & 63;
    const int leader = __builtin_ctzll(on);
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(count, uint32_t(__popcll(on)));
    base = __shfl(base, leader, 64);
    list[base + uint32_t(__popcll(on & ((1ull << lane) - 1ull)))] = v;
}

// Group a tile of `have` <= kSplitTile entries by bin in LDS and copy each
// bin's run to its place behind the bin's cursor.  read(j) loads entry j,
// make(raw, j, bin) decodes it.  Every thread of the block calls it.
// LDS: one tile of staging and three words per bin; the staging makes the
// copies runs of consecutive addresses (tile / bins entries each).  All of a
// thread's loads go out before the first is used.
template <int F, class Read, class Make>
__device__ __forceinline__ void split_tile(uint8_t *lds, uint32_t have, uint32_t nbins,
                                           uint32_t *cursor, const Ents &out, uint64_t first_run,
                                           uint32_t cap, uint32_t *ovl, uint32_t *ovl_n,
                                           Read read, Make make) {
    uint64_t *sa = reinterpret_cast<uint64_t *>(lds);
    uint32_t *sb = reinterpret_cast<uint32_t *>(sa + kSplitTile);
    uint16_t *sbin = reinterpret_cast<uint16_t *>(sb + (F == 32 ? kSplitTile : 0));
    uint32_t *hist = reinterpret_cast<uint32_t *>(sbin + kSplitTile);
    uint32_t *off = hist + nbins;
    uint32_t *gb = off + nbins;
    __shared__ uint32_t wsum[kSplitBlock / 64];
    const uint32_t t = threadIdx.x;
    Raw raw[kSplitItems];
#pragma unroll
    for (int k = 0; k < kSplitItems; ++k) {
        const uint32_t j = uint32_t(k) * kSplitBlock + t;
        raw[k] = read(j < have ? j : have - 1);
    }
    for (uint32_t j = t; j < nbins; j += kSplitBlock) hist[j] = 0;
    __syncthreads();
    Ent e[kSplitItems];
    uint32_t bin[kSplitItems], rank[kSplitItems];
#pragma unroll
    for (int k = 0; k < kSplitItems; ++k) {
        const uint32_t j = uint32_t(k) * kSplitBlock + t;
        bin[k] = ~0u;
        if (j < have) {
            e[k] = make(raw[k], j, bin[k]);
            rank[k] = atomicAdd(&hist[bin[k]], 1u);
        }
    }
    __syncthreads();
    // exclusive scan of the counts: per thread `per` consecutive bins, then
    // over the wave, then over the waves' sums
    const uint32_t per = (nbins + kSplitBlock - 1) / kSplitBlock;
    const uint32_t j0 = t * per;
    uint32_t mine = 0;
    for (uint32_t q = 0; q < per; ++q)
        if (j0 + q < nbins) mine += hist[j0 + q];
    uint32_t inc = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(inc, d, 64);
        if ((t & 63) >= uint32_t(d)) inc += o;
    }
    if ((t & 63) == 63) wsum[t >> 6] = inc;
    __syncthreads();
    uint32_t acc = inc - mine;
    for (uint32_t w = 0; w < (t >> 6); ++w) acc += wsum[w];
    for (uint32_t q = 0; q < per; ++q) {
        const uint32_t j = j0 + q;
        if (j >= nbins) break;
        off[j] = acc;
        if (hist[j]) gb[j] = atomicAdd(&cursor[j], hist[j]);
        acc += hist[j];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSplitItems; ++k)
        if (bin[k] != ~0u) {
            const uint32_t p = off[bin[k]] + rank[k];
            sa[p] = pack_ent<F>(e[k]);
            if constexpr (F == 32) sb[p] = e[k].idx;
            sbin[p] = uint16_t(bin[k]);
        }
    __syncthreads();
    const uint32_t total = off[nbins - 1] + hist[nbins - 1];
    for (uint32_t p = t; p < total; p += kSplitBlock) {
        const uint32_t j = sbin[p];
        const uint32_t g = gb[j] + (p - off[j]);
        if (g < cap) {
            const uint64_t at = (first_run + j) * cap + g;
            out.a[at] = sa[p];
            if constexpr (F == 32) out.b[at] = sb[p];
        } else {
            append_wave(ovl, ovl_n, unpack_ent<F>(sa[p], F == 32 ? sb[p] : 0u).idx);
        }
    }
}

// Bytes of dynamic LDS of the two split kernels.
inline size_t split_lds(int f, uint32_t nbins) {
    return size_t(kSplitTile) * (8 + (f == 32 ? 4 : 0) + 2) + size_t(nbins) * 12;
}

// First level: keys [0, n) to bins of 2^shift buckets.  Each bin has
// kBulkSegs runs with a cursor each, picked by block number mod 8: blocks are
// dealt to the XCDs in that order, so a run is filled from one XCD (its L2
// merges neighbouring tiles' stores) and a cursor sees an eighth of the
// tiles' atomics.  The flags and kick counts of a key placed in i1 (1 and 0)
// are written here, in order, for every key; the later kernels only write
// where they differ.
template <int F, int HASH, int POL>
__global__ __launch_bounds__(kSplitBlock) void bulk_split_kernel(
    const uint64_t *__restrict__ keys, uint32_t n, Place pl, uint32_t shift, uint32_t nbins,
    uint32_t *__restrict__ cursor, Ents out, uint32_t cap, uint8_t *__restrict__ ok,
    uint32_t *__restrict__ kicks, uint32_t *__restrict__ ovl, uint32_t *__restrict__ ovl_n) {
    extern __shared__ __align__(16) uint8_t bulk_lds[];
    const uint32_t lo = blockIdx.x * uint32_t(kSplitTile);
    const uint32_t have = n - lo < uint32_t(kSplitTile) ? n - lo : uint32_t(kSplitTile);
    const uint32_t x = blockIdx.x % kBulkSegs;
    split_tile<F>(
        bulk_lds, have, nbins, cursor + x * nbins, out, uint64_t(x) * nbins, cap, ovl, ovl_n,
        [&](uint32_t j) { return Raw{__builtin_nontemporal_load(keys + lo + j), 0u}; },
        [&](const Raw &r, uint32_t j, uint32_t &bin) {
            const Derived d = derive<Geom<F, 32>, HASH, POL>(r.a, pl);
            if (ok) ok[lo + j] = 1;
            if (kicks) kicks[lo + j] = 0;
            bin = d.i1 >> shift;
            return Ent{d.t1, lo + j, d.i1 & ((1u << shift) - 1u)};
        });
}

// Second level: the entries of bin c (its kBulkSegs runs of at most cap_in)
// to the bin's 2^fine parts.  Block = one tile of one run.
template <int F>
__global__ __launch_bounds__(kSplitBlock) void bulk_resplit_kernel(
    Ents in, const uint32_t *__restrict__ in_n, uint32_t nbins, uint32_t cap_in, uint32_t tiles,
    uint32_t shift, uint32_t fine, uint32_t *__restrict__ cursor, Ents out, uint32_t cap,
    uint32_t *__restrict__ ovl, uint32_t *__restrict__ ovl_n) {
    extern __shared__ __align__(16) uint8_t bulk_lds[];
    const uint32_t run = blockIdx.x / tiles;
    const uint32_t have = in_n[run] < cap_in ? in_n[run] : cap_in;
    const uint32_t lo = (blockIdx.x % tiles) * uint32_t(kSplitTile);
    if (lo >= have) return;
    const uint32_t c = run % nbins;
    const uint64_t base = uint64_t(run) * cap_in + lo;
    split_tile<F>(
        bulk_lds, have - lo < uint32_t(kSplitTile) ? have - lo : uint32_t(kSplitTile), 1u << fine,
        cursor + (c << fine), out, uint64_t(c) << fine, cap, ovl, ovl_n,
        [&](uint32_t j) {
            return Raw{__builtin_nontemporal_load(in.a + base + j), F == 32 ? in.b[base + j] : 0u};
        },
        [&](const Raw &r, uint32_t, uint32_t &bin) {
            Ent e = unpack_ent<F>(r.a, r.b);
            bin = e.bucket >> shift;
            e.bucket &= (1u << shift) - 1u;
            return e;
        });
}

// One part (2^shift buckets from bucket part << shift on, the last part cut
// at m) in LDS: load, try every entry's bucket, store.  An entry whose bucket
// is full goes to the part's list; the overflow list's length goes behind the
// lists' lengths, since the next launch clears the cursors.  runs / stride: the part's entries lie in
// `runs` runs, run r at (r * stride + part) * cap with count in_n[same].
template <class G>
__global__ __launch_bounds__(kPlaceBlock) void bulk_insert_kernel(
    typename G::W *__restrict__ table, uint64_t m, uint32_t shift, Ents in,
    const uint32_t *__restrict__ in_n, uint32_t runs, uint32_t stride, uint32_t cap,
    uint32_t *__restrict__ list, uint32_t *__restrict__ list_n, uint32_t list_cap,
    const uint32_t *__restrict__ ovl_n, Counters *ctr) {
    using W = typename G::W;
    extern __shared__ __align__(16) uint8_t bulk_lds[];
    __shared__ uint32_t s_n;
    W *part = reinterpret_cast<W *>(bulk_lds);
    const uint64_t b0 = uint64_t(blockIdx.x) << shift;
    const uint32_t nb = uint32_t(m - b0 < (1ull << shift) ? m - b0 : (1ull << shift));
    const uint32_t words = nb * G::WPB;
    W *home = table + b0 * G::WPB;
    // 16-byte moves (parts start at multiples of 16 bytes: 2^shift buckets of
    // at least 4 bytes, shift >= 2), then what is left of a cut last part
    constexpr uint32_t WPV = 16 / sizeof(W);
    const uint32_t vecs = words / WPV;
    const ulonglong2 *gv = reinterpret_cast<const ulonglong2 *>(home);
    ulonglong2 *lv = reinterpret_cast<ulonglong2 *>(part);
    for (uint32_t j = threadIdx.x; j < vecs; j += kPlaceBlock) lv[j] = gv[j];
    for (uint32_t j = vecs * WPV + threadIdx.x; j < words; j += kPlaceBlock) part[j] = home[j];
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    unsigned long long placed = 0;
    const int lane = threadIdx.x & 63;
    uint32_t *mylist = list + uint64_t(blockIdx.x) * list_cap;
    for (uint32_t r = 0; r < runs; ++r) {
        const uint64_t run = uint64_t(r) * stride + blockIdx.x;
        const uint32_t have = in_n[run] < cap ? in_n[run] : cap;
        const uint64_t base = run * cap;
        // kPlaceItems entries of a thread are loaded before the first is used
        for (uint32_t i0 = threadIdx.x; i0 < have; i0 += kPlaceItems * kPlaceBlock) {
            Raw raw[kPlaceItems];
#pragma unroll
            for (int k = 0; k < kPlaceItems; ++k) {
                const uint32_t i = i0 + uint32_t(k) * kPlaceBlock;
                const uint64_t at = base + (i < have ? i : i0);
                raw[k] = Raw{__builtin_nontemporal_load(in.a + at), G::F == 32 ? in.b[at] : 0u};
            }
#pragma unroll
            for (int k = 0; k < kPlaceItems; ++k) {
                if (i0 + uint32_t(k) * kPlaceBlock >= have) break;
                const Ent e = unpack_ent<G::F>(raw[k].a, raw[k].b);
                Bucket<G> bk;
                load_bucket<G>(part, e.bucket, bk);
                const bool done = try_insert<G>(part, e.bucket, e.tag, bk) >= 0;
                placed += done;
                const uint64_t need = __ballot(!done);
                if (need) {
                    const int leader = __builtin_ctzll(need);
                    uint32_t at = 0;
                    if (lane == leader) at = atomicAdd(&s_n, uint32_t(__popcll(need)));
                    at = __shfl(at, leader, 64);
                    if (!done)
                        mylist[at + uint32_t(__popcll(need & ((1ull << lane) - 1ull)))] = e.idx;
                }
            }
        }
    }
    __syncthreads();
    ulonglong2 *hv = reinterpret_cast<ulonglong2 *>(home);
    for (uint32_t j = threadIdx.x; j < vecs; j += kPlaceBlock) hv[j] = lv[j];
    for (uint32_t j = vecs * WPV + threadIdx.x; j < words; j += kPlaceBlock) home[j] = part[j];
    if (threadIdx.x == 0) {
        list_n[blockIdx.x] = s_n;
        if (blockIdx.x == 0) list_n[gridDim.x] = *ovl_n;
    }
    block_add<kPlaceBlock>(ctr, placed);
}

}  // namespace cfk
