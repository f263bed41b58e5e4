// cf_launch.hpp -- host-side launchers of the single-filter kernels for one
// (f, b, hash, eviction policy, placement) instantiation, shared by the
// translation units of libcf.so.  The instantiations live in cf_inst_f*.hip,
// one translation unit per fingerprint width so that they compile in
// parallel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cf.h"
#include "cf_bulk.hpp"
#include "cf_kernels.hpp"

namespace cfl {

struct Launchers {
    void (*query)(const void *table, const cfk::Place &pl, const uint64_t *keys, uint64_t n,
                  uint8_t *found, int grid, hipStream_t s);
    void (*del)(void *table, const cfk::Place &pl, const uint64_t *keys, uint64_t n,
                uint8_t *okv, cfk::Counters *ctr, int grid, hipStream_t s);
    void (*ins)(void *table, const cfk::Place &pl, const uint64_t *keys, uint64_t n,
                uint8_t *okv, uint32_t *kicks, cfk::Counters *ctr, uint32_t *queue, uint64_t seg,
                cfk::LostLog log, uint32_t max_evict, uint64_t seed, const cfk::Rest *rest,
                bool grouped, int grid, hipStream_t s);
    // the partitioned insert (cf_bulk.hpp)
    void (*split)(const uint64_t *keys, uint32_t n, const cfk::Place &pl, uint32_t shift,
                  uint32_t nbins, uint32_t *cursor, cfk::Ents out, uint32_t cap, uint8_t *okv,
                  uint32_t *kicks, uint32_t *ovl, uint32_t *ovl_n, hipStream_t s);
    void (*resplit)(cfk::Ents in, const uint32_t *in_n, uint32_t nbins, uint32_t cap_in,
                    uint32_t shift, uint32_t fine, uint32_t *cursor, cfk::Ents out, uint32_t cap,
                    uint32_t *ovl, uint32_t *ovl_n, hipStream_t s);
    void (*move)(cfk::Ents list, const uint32_t *list_n, uint32_t list_cap, const cfk::Place &pl,
                 uint32_t part_shift, uint32_t shift, uint32_t nbins, uint32_t *cursor,
                 cfk::Ents out, uint32_t cap, uint32_t *ovl, uint32_t *ovl_n, int parts,
                 hipStream_t s);
    void (*place)(void *table, uint64_t m, uint32_t shift, cfk::Ents in, const uint32_t *in_n,
                  uint32_t runs, uint32_t stride, uint32_t cap, cfk::Ents list, uint32_t *list_n,
                  uint32_t list_cap, const uint32_t *ovl_n, cfk::Counters *ctr, int parts,
                  hipStream_t s);
    void (*recount)(const void *table, uint64_t nwords, cfk::Counters *ctr, int grid,
                    hipStream_t s);
    uint64_t words_per_bucket;  // in units of the geometry's word type
    uint64_t word_bytes;
};

// Whether an insert launch of n keys on a table of that many bytes loads each
// group of candidates' other buckets together (cfk::probe_width) in the
// breadth-first search, or probes candidate by candidate.
// By table size, measured on one-launch fills at load 0.95: 2 MiB 6.6 -> 7.25
// Gops/s and 8 MiB 13.8 -> 14.3-14.7 grouped.  The 64 MiB eviction-stress
// table (4-byte buckets, to load 0.98) was 2-5% slower grouped, and the
// 512 MiB and 4 GiB tables, whose probes are HBM requests, 3% (the 4 GiB
// step's inserts 15%).
constexpr uint64_t kGroupedProbeBytes = uint64_t(16) << 20;
constexpr uint64_t kGroupedKeys = uint64_t(1) << 19;
inline bool grouped_probe(uint64_t table_bytes, uint64_t n) {
    return table_bytes <= kGroupedProbeBytes || n <= kGroupedKeys;
}

// Launchers for p's geometry, hash, eviction policy and placement; false if
// unsupported.  pick_launchers dispatches on f to the per-width tables
// (pick_launchers_f*: query, delete, recount; pick_insert_f*: insert).
bool pick_launchers(const cf_params &p, Launchers &out);
bool pick_launchers_f8(const cf_params &p, Launchers &out);
bool pick_launchers_f16(const cf_params &p, Launchers &out);
bool pick_launchers_f32(const cf_params &p, Launchers &out);
bool pick_insert_f8(const cf_params &p, Launchers &out);
bool pick_insert_f16(const cf_params &p, Launchers &out);
bool pick_insert_f32(const cf_params &p, Launchers &out);

// Checks every field of p (what cf_create documents); on failure records
// the message, prefixed by `who` when it is not empty, and returns the
// status.
cf_status check_params(const cf_params &p, const char *who);

// The kernels' view of p's placement (p already checked).
inline cfk::Place make_place(const cf_params &p) {
    cfk::Place pl{};
    if (p.placement == CF_PLACE_OFFSET) {
        pl.m = uint32_t(p.num_buckets);
        pl.m1 = pl.m - 1;
        pl.mdiv = cfk::fastmod_constant(pl.m);
        pl.m1div = pl.m1 ? cfk::fastmod_constant(pl.m1) : 0;
    } else {
        pl.mmask = uint32_t(p.num_buckets - 1);
    }
    return pl;
}

// Queue entries an insert launch of `len` keys needs with `grid` blocks, and
// the per-block segment length.
inline uint64_t insert_segment(uint64_t len, int grid) {
    const uint64_t per = uint64_t(grid) * cfk::kBlock;
    return ((len + per - 1) / per) * cfk::kBlock;
}

}  // namespace cfl
