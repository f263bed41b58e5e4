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

// The table a batch goes into: m buckets of b slots of f bits, filled by the
// breadth-first search or (walk) the random walk.
struct BulkTable {
    uint64_t m;
    uint32_t b, f;
    bool walk;
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
// than a CAS per key, so the rule is a line of table bytes per key.  The host
// does not know how full the table is, and the gain is least where it is
// fullest (the searches cost the same either way, and those of a partitioned
// batch have fewer blocks to overlap with), so each line lies where a batch
// still gains that ends at load 0.86 / 0.91 / 0.945 / 0.955 (b = 4 / 8 / 16 /
// 32).  Measured at the lines, direct time over partitioned time, the least over
// b and the loads 0, 0.5 and the highest, and the mean (against the library
// before it had this path no least is below 0.98):
//   keys         f   breadth-first          random walk
//   2^19         8    4 B  0.98  1.09        4 B  0.94  1.10
//               16    4 B  1.02  1.09        4 B  0.98  1.08
//   3 * 2^18     8    4 B  1.07  1.22        4 B  1.01  1.21
//               16    6 B  0.97  1.08        6 B  0.95  1.08
//   2^20         8    8 B  1.05  1.41        8 B  0.97  1.30
//               16    8 B  0.98  1.22        8 B  0.99  1.22
//               32    6 B  1.03  1.09        6 B  0.97  1.07   b < 32
//   3 * 2^19     8    8 B  1.08  1.56        8 B  1.06  1.49
//               16   12 B  0.98  1.28        8 B  1.00  1.37
//               32    8 B  1.03  1.22        8 B  0.96  1.20   b < 32
//   2^21         8    8 B  1.19  1.78        8 B  0.97  1.68
//               16   16 B  1.14  1.54       12 B  0.99  1.49
//               32   16 B  1.00  1.32        8 B  1.09  1.43
//   2^22         8   12 B  1.28  1.79       12 B  1.05  1.72
//               16   24 B  1.13  1.46       12 B  1.09  1.67
//               32   16 B  1.01  1.39        8 B  1.14  1.66
//   2^24         8   12 B  1.15  1.92       12 B  1.02  1.95
//               16   24 B  1.06  1.42       12 B  1.06  1.86
//               32   16 B  1.09  1.38        8 B  1.17  1.63
//   2^26, 2 GiB 16   32 B  1.07  1.41       32 B  1.03  1.41
//   2^27, 2 GiB  8   16 B  1.25  1.92       16 B  1.19  1.89
//               32   16 B  1.23  1.52       16 B  1.21  1.51
// and beyond them: 16 bits 2^19 keys 8 B 0.87 and 0.93, 2^20 16 B 0.96 and 0.96;
// random walk 2^22 16 B 0.97, 24 B on 512 MiB 0.95; 32 bits (entries of 12
// bytes) 2^19 keys 5 B 0.88 to 1.00, 2^20 b = 32 (a bucket is a whole line) 6 B
// 0.91 and 0.93, 2^22 24 B 0.97, random walk 16 B 0.90, 2^25 keys on 2 GiB 64 B
// 0.72 and 0.71.  Below 2^19 keys nothing is gained (2^18 from empty 39-45 ->
// 35-46 us).
// A batch of more than twice the slots, most of which must fail, goes direct:
// its failing searches need more blocks than a small table has parts.
inline uint32_t bulk_bytes_per_key(const BulkTable &t, uint64_t n) {
    const int band = n < (3ull << 18)            ? 0
                     : n < (1ull << 20)          ? 1
                     : n < (3ull << 19)          ? 2
                     : n < (1ull << 21)          ? 3
                     : n < (1ull << 22)          ? 4
                     : t.bytes() < (2ull << 30) ? 5
                                                 : 6;
    constexpr uint8_t most[2][3][7] = {
        {{4, 4, 8, 8, 8, 12, 16}, {4, 6, 8, 12, 16, 24, 32}, {0, 0, 6, 8, 16, 16, 16}},
        {{4, 4, 8, 8, 8, 12, 16}, {4, 6, 8, 8, 12, 12, 32}, {0, 0, 6, 8, 8, 8, 16}}};
    if (t.f == 32 && t.b == 32 && band < 4) return 0;
    return most[t.walk][t.f == 8 ? 0 : t.f == 16 ? 1 : 2][band];
}

inline bool bulk_wanted(const BulkTable &t, uint64_t n) {
    if (n < (1ull << 19) || n / 2 > t.slots()) return false;
    const uint64_t len = std::min(n, cfk::kMaxBulkKeys);
    return len * bulk_bytes_per_key(t, n) >= t.bytes() && bulk_fits(t, bulk_plan(t, len));
}

// The largest batch of at most n keys that goes partitioned, 0 if none does,
// and the smallest that does if `most` does: up to twice the slots the rule
// only gets easier with more keys.
inline uint64_t bulk_most(const BulkTable &t, uint64_t n) {
    const uint64_t most = std::min(n, 2 * t.slots() + 1);
    return bulk_wanted(t, most) ? most : 0;
}

inline uint64_t bulk_least(const BulkTable &t, uint64_t most) {
    uint64_t no = 0;
    while (most - no > 1) {
        const uint64_t mid = no + (most - no) / 2;
        (bulk_wanted(t, mid) ? most : no) = mid;
    }
    return most;
}

}  // namespace cfl
