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
// Keys whose i1 was full are grouped again by the part of their i2 and tried
// there the same way, and insert_kernel takes those left over through the
// eviction search.  For the table this is one legal interleaving of the
// concurrent insert: every attempt in an i1 happens before any attempt in an
// i2, and those before any eviction.
//
//  bulk_split_kernel    keys -> entries grouped by bin (bin = i1 >> shift)
//  bulk_resplit_kernel  (tables of many parts) entries of one bin -> parts
//  bulk_insert_kernel   one part in LDS: the attempts in its buckets
//  bulk_move_kernel     entries left over -> grouped by bin of their i2;
//                       then resplit and insert again
//  insert_kernel        the searches of the entries left over (Rest)
//
// Measured, builds of 2 MiB (b = 4, f = 16), 64 MiB (b = 4, f = 8) and 512 MiB
// (b = 16, f = 16) from one batch: 190, 3766 and 12476 us direct, 135, 1731
// and 5840 us this way.  The kernels are streams: of a pass of 2^27 keys on
// 512 MiB the split takes 478 us (17 bytes a key: 4.5 TB/s), the resplit 548
// (3.7 TB/s), the placement 487 on an empty table and 745 on a half-full one
// (8 bytes an entry and the table twice: 4.4 and 2.9 TB/s), where a copy
// reaches 4.9 TB/s.
//
// Bins and parts hold a fixed number of entries, sized by the host from the
// mean of a uniform hash plus eight standard deviations.  Entries beyond it
// (many copies of one key) go to one overflow list instead, which
// insert_kernel runs from the start, so a skewed batch is never wrong.  It is
// seldom slower than the one-launch insert: with a tenth of the keys copies, 4
// to 4096 of each, side by side or spread, the builds to 0.75 (b = 4) or 0.8
// took, in one launch -> partitioned: 512 MiB (b = 16, f = 16) 8.8-336 -> 3.7-123
// ms, 64 MiB (b = 4, f = 8) 2.6-78 -> 1.0-57, 8 MiB (b = 16, f = 16) 0.2-14 ->
// 0.1-4.7 (the long ones are searches of copies that cannot be stored).  The
// exception is 1 and 2 MiB with b = 4 where 9 to 24 copies lie side by side and 2 to 7%
// of the batch fails: 545-910 -> 625-1010 us.
#pragma once

#include "cf_kernels.hpp"

namespace cfk {

// A part of 64 KiB leaves room for two blocks on a compute unit, one loading
// or storing while the other places; parts of 32 KiB (with 512 or 1024
// threads) built the 512 MiB table 8-13% slower.
constexpr int kPlaceBlock = 1024;
constexpr int kPlaceItems = 4;

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

// Entries left over in the parts' lists, moved to their other bucket and
// grouped by its bin.  Block = one part's list.
template <int F, int HASH, int POL>
__global__ __launch_bounds__(kSplitBlock) void bulk_move_kernel(
    Ents list, const uint32_t *__restrict__ list_n, uint32_t list_cap, Place pl,
    uint32_t part_shift, uint32_t shift, uint32_t nbins, uint32_t *__restrict__ cursor, Ents out,
    uint32_t cap, uint32_t *__restrict__ ovl, uint32_t *__restrict__ ovl_n) {
    extern __shared__ __align__(16) uint8_t bulk_lds[];
    const uint32_t have = list_n[blockIdx.x];
    const uint32_t x = blockIdx.x % kBulkSegs;
    const uint32_t b0 = blockIdx.x << part_shift;
    for (uint32_t lo = 0; lo < have; lo += kSplitTile) {
        const uint64_t base = uint64_t(blockIdx.x) * list_cap + lo;
        split_tile<F>(
            bulk_lds, have - lo < uint32_t(kSplitTile) ? have - lo : uint32_t(kSplitTile), nbins,
            cursor + x * nbins, out, uint64_t(x) * nbins, cap, ovl, ovl_n,
            [&](uint32_t j) { return Raw{list.a[base + j], F == 32 ? list.b[base + j] : 0u}; },
            [&](const Raw &r, uint32_t, uint32_t &bin) {
                Ent e = unpack_ent<F>(r.a, r.b);
                const uint32_t b = move_tag<Geom<F, 32>, HASH, POL>(b0 + e.bucket, e.tag, pl);
                bin = b >> shift;
                e.bucket = b & ((1u << shift) - 1u);
                return e;
            });
        __syncthreads();
    }
}

// Alg. 1's TryInsert in LDS, word by word from the scan's start (the slots are
// those try_insert takes): a bucket read whole costs a wave 64 x 32 bytes of
// LDS bandwidth where the first word mostly has room (placing 2^27 keys in an
// empty table: 697 -> 487 us).
template <class G>
__device__ __forceinline__ bool lds_insert(typename G::W *part, uint32_t bucket, uint32_t tag) {
    using W = typename G::W;
    W *base = part + bucket * G::WPB;
    const int start = scan_start<G>(tag);
    for (int k = 0; k < G::WPB; ++k) {
        W *at = base + ((start + k) & (G::WPB - 1));
        W w = *at;
        for (W z = zero_lanes<W, G::F>(w); z; z = zero_lanes<W, G::F>(w)) {
            const int sh = lowest_bit(z) / G::F * G::F;
            const W old = cas_word(at, w, W(w | (W(tag) << sh)));
            if (old == w) return true;
            w = old;
        }
    }
    return false;
}

// A part that gets fewer entries than one per so many bytes is not staged:
// its entries (no other block has any in it) are tried in place.  Staging
// costs its bytes twice at the streaming rate, an entry in place a line read
// and a CAS, 70 ps.
constexpr uint32_t kStageBytes = 160;

// One part (2^shift buckets from bucket part << shift on, the last part cut
// at m) in LDS: load, try every entry's bucket, store.  An entry whose bucket
// is full goes to the part's list; the overflow list's length goes behind the
// lists' lengths, since the next launch clears the cursors.  runs / stride: the part's entries lie in
// `runs` runs, run r at (r * stride + part) * cap with count in_n[same].
template <class G>
__global__ __launch_bounds__(kPlaceBlock) void bulk_insert_kernel(
    typename G::W *__restrict__ table, uint64_t m, uint32_t shift, Ents in,
    const uint32_t *__restrict__ in_n, uint32_t runs, uint32_t stride, uint32_t cap,
    Ents list, uint32_t *__restrict__ list_n, uint32_t list_cap,
    const uint32_t *__restrict__ ovl_n, Counters *ctr) {
    using W = typename G::W;
    extern __shared__ __align__(16) uint8_t bulk_lds[];
    __shared__ uint32_t s_n;
    W *part = reinterpret_cast<W *>(bulk_lds);
    const uint64_t b0 = uint64_t(blockIdx.x) << shift;
    const uint32_t nb = uint32_t(m - b0 < (1ull << shift) ? m - b0 : (1ull << shift));
    const uint32_t words = nb * G::WPB;
    W *home = table + b0 * G::WPB;
    // the runs end to end: run r holds the part's entries [s_run[r], s_run[r + 1])
    __shared__ uint32_t s_run[kBulkSegs + 1];
    if (threadIdx.x == 0) {
        uint32_t acc = 0;
        for (uint32_t r = 0; r < runs; ++r) {
            s_run[r] = acc;
            const uint32_t c = in_n[uint64_t(r) * stride + blockIdx.x];
            acc += c < cap ? c : cap;
        }
        s_run[runs] = acc;
        s_n = 0;
    }
    __syncthreads();
    const uint32_t total = s_run[runs];
    // 16-byte moves (parts start at multiples of 16 bytes: 2^shift buckets of
    // at least 4 bytes, shift >= 2), then what is left of a cut last part
    constexpr uint32_t WPV = 16 / sizeof(W);
    const uint32_t vecs = words / WPV;
    ulonglong2 *hv = reinterpret_cast<ulonglong2 *>(home);
    ulonglong2 *lv = reinterpret_cast<ulonglong2 *>(part);
    const bool staged = uint64_t(total) * kStageBytes >= uint64_t(words) * sizeof(W);
    if (staged) {
        for (uint32_t j = threadIdx.x; j < vecs; j += kPlaceBlock) lv[j] = hv[j];
        for (uint32_t j = vecs * WPV + threadIdx.x; j < words; j += kPlaceBlock)
            part[j] = home[j];
    }
    __syncthreads();
    unsigned long long placed = 0;
    const int lane = threadIdx.x & 63;
    const uint64_t mine = uint64_t(blockIdx.x) * list_cap;
    auto place = [&](auto in_lds) {
        // kPlaceItems entries of a thread are loaded before the first is used
        for (uint32_t i0 = threadIdx.x; i0 < total; i0 += kPlaceItems * kPlaceBlock) {
            Raw raw[kPlaceItems];
#pragma unroll
            for (int k = 0; k < kPlaceItems; ++k) {
                const uint32_t j = i0 + uint32_t(k) * kPlaceBlock;
                const uint32_t i = j < total ? j : i0;
                uint32_t r = 0;
                while (i >= s_run[r + 1]) ++r;
                const uint64_t at = (uint64_t(r) * stride + blockIdx.x) * cap + (i - s_run[r]);
                raw[k] = Raw{__builtin_nontemporal_load(in.a + at), G::F == 32 ? in.b[at] : 0u};
            }
#pragma unroll
            for (int k = 0; k < kPlaceItems; ++k) {
                if (i0 + uint32_t(k) * kPlaceBlock >= total) break;
                const Ent e = unpack_ent<G::F>(raw[k].a, raw[k].b);
                bool done;
                if constexpr (decltype(in_lds)::value) {
                    done = lds_insert<G>(part, e.bucket, e.tag);
                } else {
                    Bucket<G> bk;
                    load_bucket<G>(home, e.bucket, bk);
                    done = try_insert<G>(home, e.bucket, e.tag, bk) >= 0;
                }
                placed += done;
                const uint64_t need = __ballot(!done);
                if (need) {
                    const int leader = __builtin_ctzll(need);
                    uint32_t at = 0;
                    if (lane == leader) at = atomicAdd(&s_n, uint32_t(__popcll(need)));
                    at = __shfl(at, leader, 64);
                    if (!done) {
                        const uint64_t to =
                            mine + at + uint32_t(__popcll(need & ((1ull << lane) - 1ull)));
                        list.a[to] = raw[k].a;
                        if constexpr (G::F == 32) list.b[to] = raw[k].b;
                    }
                }
            }
        }
    };
    if (staged) place(std::true_type{});
    else place(std::false_type{});
    __syncthreads();
    if (staged) {
        for (uint32_t j = threadIdx.x; j < vecs; j += kPlaceBlock) hv[j] = lv[j];
        for (uint32_t j = vecs * WPV + threadIdx.x; j < words; j += kPlaceBlock)
            home[j] = part[j];
    }
    if (threadIdx.x == 0) {
        list_n[blockIdx.x] = s_n;
        if (blockIdx.x == 0) list_n[gridDim.x] = *ovl_n;
    }
    block_add<kPlaceBlock>(ctr, placed);
}

}  // namespace cfk
