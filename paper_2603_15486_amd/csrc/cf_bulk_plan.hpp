// cf_bulk_plan.hpp -- the host arithmetic of the partitioned insert
// (cf_bulk.hpp): which batches go partitioned, the layout of a pass, and the
// packing of an entry.  Plain C++ without HIP, so that a host program can
// evaluate every plan and check that what it addresses is there.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace cfk {

// 44 KiB of staging for 8-byte entries: three blocks on a compute unit.
constexpr int kSplitBlock = 512;
constexpr int kSplitItems = 8;                            // entries per thread and tile
constexpr int kSplitTile = kSplitBlock * kSplitItems;
constexpr uint32_t kBulkSegs = 8;                         // one per XCD, see bulk_split_kernel

constexpr uint32_t kBulkIdxBits = 27;  // keys of one pass
constexpr uint64_t kMaxBulkKeys = 1ull << kBulkIdxBits;

// ------------------------------------------------------------------ entries

// One entry: the tag as written in its bucket, the key's index in the pass, and
// the low bits of the bucket (its place within the bin).  8 bytes for fingerprints of 8
// and 16 bits (tag | index | bucket bits, see bulk_bucket_bits), and
// 12 bytes in two arrays for 32-bit ones.
struct Ents {
    uint64_t *a;
    uint32_t *b;  // f = 32 only: the index
};

struct Ent {
    uint32_t tag, idx, bucket;
};

// Bits of the bucket that an entry has room for.
constexpr uint32_t bulk_bucket_bits(uint32_t f) { return f == 32 ? 32 : 64 - kBulkIdxBits - f; }

template <int F>
constexpr __attribute__((always_inline)) uint64_t pack_ent(const Ent &e) {
    if constexpr (F == 32) return uint64_t(e.tag) | (uint64_t(e.bucket) << 32);
    else
        return uint64_t(e.tag) | (uint64_t(e.idx) << F) |
               (uint64_t(e.bucket) << (F + kBulkIdxBits));
}

template <int F>
constexpr __attribute__((always_inline)) Ent unpack_ent(uint64_t a, uint32_t b) {
    if constexpr (F == 32) return Ent{uint32_t(a), b, uint32_t(a >> 32)};
    else
        return Ent{uint32_t(a) & ((1u << F) - 1u),
                   uint32_t(a >> F) & ((1u << kBulkIdxBits) - 1u),
                   uint32_t(a >> (F + kBulkIdxBits))};
}

// Bytes of dynamic LDS of the split kernels: a tile's staging and three words
// per bin.
inline uint64_t split_lds(int f, uint32_t nbins) {
    return uint64_t(kSplitTile) * (8 + (f == 32 ? 4 : 0) + 2) + uint64_t(nbins) * 12;
}

}  // namespace cfk

namespace cfl {

// The table a batch goes into: m buckets of b slots of f bits.
struct BulkTable {
    uint64_t m;
    uint32_t b, f;
    uint64_t slots() const { return m * b; }
    uint64_t bucket_bytes() const { return uint64_t(b) * f / 8; }
    uint64_t bytes() const { return m * bucket_bytes(); }
};

// Layout of one pass of `len` keys.
struct BulkPlan {
    uint32_t shift, parts;      // parts of 2^shift buckets
    uint32_t bins, fine;        // bins of 2^fine parts; fine = 0: a bin is a part
    uint32_t cap1, cap2;        // entries per run of a bin, per part (fine > 0)
    uint32_t list_cap;
    uint64_t cursors;           // cursors and overflow count; zero between passes
    uint64_t o_cur, o_listn, o_a, o_a32, o_b, o_b32, o_list, o_list32, o_ovl, bytes;
};

constexpr uint64_t kPartBytes = 64 << 10;
constexpr uint64_t kMinPartBytes = 1 << 10;
constexpr uint32_t kWantParts = 256;
// Up to this many parts one level of grouping, although a tile then leaves
// runs of four entries: 32 MiB (b = 16, f = 16) 291 us with one level and 329
// with two, 64 MiB 551 and 586 (b = 4, f = 8: 1731 and 1862), but 128 MiB 1274
// and 1110.  Also the most bins a split kernel is launched with (its LDS).
constexpr uint32_t kOneLevelBins = 1024;

inline uint32_t bulk_cap(double mean) {
    return (uint32_t(mean + 8 * std::sqrt(mean) + 16) + 15u) & ~15u;
}

inline BulkPlan bulk_plan(const BulkTable &t, uint64_t len) {
    const uint64_t m = t.m, bucket = t.bucket_bytes();
    BulkPlan p{};
    while ((bucket << (p.shift + 1)) <= kPartBytes) ++p.shift;
    auto parts_at = [&](uint32_t s) { return (m + (1ull << s) - 1) >> s; };
    while (parts_at(p.shift) < kWantParts && (bucket << p.shift) > kMinPartBytes) --p.shift;
    p.parts = uint32_t(parts_at(p.shift));
    while (p.parts > kOneLevelBins && (1u << (2 * p.fine)) < p.parts) ++p.fine;
    p.bins = (p.parts + (1u << p.fine) - 1) >> p.fine;
    const double share = double(1ull << (p.shift + p.fine)) / double(m);  // of a bin
    const uint64_t tiles = (len + cfk::kSplitTile - 1) / cfk::kSplitTile;
    const uint64_t per_run = (tiles + cfk::kBulkSegs - 1) / cfk::kBulkSegs * cfk::kSplitTile;
    p.cap1 = bulk_cap(std::min(1.0, share) * double(std::min(per_run, len)));
    p.cap2 = p.fine ? bulk_cap(double(len) * double(1ull << p.shift) / double(m)) : 0;
    p.list_cap = p.fine ? p.cap2 : cfk::kBulkSegs * p.cap1;
    const uint64_t wide = t.f == 32 ? 4 : 0;
    const uint64_t n1 = uint64_t(p.bins) * cfk::kBulkSegs * p.cap1;
    const uint64_t n2 = uint64_t(p.parts) * p.cap2;
    const uint64_t lists = uint64_t(p.parts) * p.list_cap;
    auto take = [&](uint64_t bytes) {
        const uint64_t o = p.bytes;
        p.bytes += (bytes + 255) & ~uint64_t(255);
        return o;
    };
    p.cursors = 2 * (uint64_t(p.bins) * cfk::kBulkSegs + (p.fine ? p.parts : 0)) + 1;
    p.o_cur = take(p.cursors * 4);
    p.o_listn = take((uint64_t(p.parts) + 1) * 4);
    // the first level's entries, and later (they are used up by then) the
    // eviction queue of the overflow list
    p.o_a = take(n1 * 8);  // n1 >= len
    p.o_a32 = take(n1 * wide);
    p.o_b = take(n2 * 8);
    p.o_b32 = take(n2 * wide);
    p.o_list = take(lists * 8);
    p.o_list32 = take(lists * wide);
    p.o_ovl = take(len * 4);
    return p;
}

// Whether an entry has room for a bucket's place within its bin, and the split
// kernels' LDS for a bin's counters.  Tables of 2^31 slots, the largest whose
// batches go partitioned, need up to all of an entry's 21 bits (2^29 buckets
// of 4 x 16 bits), one bucket more 22: a bucket whose top bit is lost would
// be another one.
inline bool bulk_fits(const BulkTable &t, const BulkPlan &p) {
    return p.shift + p.fine <= cfk::bulk_bucket_bits(t.f) && p.bins <= kOneLevelBins &&
           (1u << p.fine) <= kOneLevelBins;
}

// Whether a batch of n goes partitioned.  It then costs a fixed chain of
// launches (40 us) and the table read and written twice, which must be less
// than a CAS per key.  Measured, direct -> partitioned:
//  - from empty, 2^19 keys 46-63 -> 41-47 us, 2^18 keys 39-45 -> 35-46: no
//    gain below 2^19 keys;
//  - an eighth of the slots at load 0 / 0.5 / 0.8, 32 MiB of 32-bit
//    fingerprints (2^20 keys) 53 / 73 / 152 -> 56 / 71 / 127 us, 512 MiB of
//    16-bit ones (2^25 keys) 1363 / 1367 / 1751 -> 611 / 759 / 1357;
//  - a sixteenth on 512 MiB 687 / 694 / 958 -> 450 / 549 / 983, on 4 GiB
//    (2^27 keys), where direct requests cost more, 6.8 / 6.9 / 9.9 -> 3.6 /
//    4.4 / 8.2 ms; a thirty-second on 512 MiB 357 / 361 / 542 -> 374 / 457 /
//    630.
// A batch of more than twice the slots, most of which must fail, goes direct:
// its failing searches need more blocks than a small table has parts.
inline bool bulk_wanted(const BulkTable &t, uint64_t n) {
    if (n < (1ull << 19) || n / 2 > t.slots()) return false;
    const uint64_t share = n < (1ull << 20)            ? 4
                           : n < (1ull << 22)          ? 8
                           : t.bytes() < (2ull << 30) ? 12
                                                       : 16;
    const uint64_t len = std::min(n, cfk::kMaxBulkKeys);
    return len * share >= t.slots() && bulk_fits(t, bulk_plan(t, len));
}

// The largest batch of at most n keys that goes partitioned, 0 if none does:
// up to twice the slots the rule only gets easier with more keys.
inline uint64_t bulk_most(const BulkTable &t, uint64_t n) {
    const uint64_t most = std::min(n, 2 * t.slots() + 1);
    return bulk_wanted(t, most) ? most : 0;
}

}  // namespace cfl
