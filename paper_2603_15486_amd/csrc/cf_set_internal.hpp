// cf_set_internal.hpp -- what other translation units of the library may
// ask of a filter set beyond its C ABI (include/cf_set.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cf_set.h"

namespace cfs {

// Number of filters the set was created with (0 for NULL).
uint32_t filter_count(const cf_set *set);

// Scratch lanes.  A batch of requests uses the eviction queue of one lane;
// batches on different lanes may be in flight at once and overlap on the
// device, as long as they touch disjoint filters (the caller orders batches
// that share a filter).  Lane 0 is the set's own scratch, which
// cf_set_execute, graphs and cf_set_apply use.  reserve_lanes makes lanes
// 1 .. n-1 (synchronous; set-up only).
uint32_t lane_count(const cf_set *set);
cf_status reserve_lanes(cf_set *set, uint32_t n);

// A batch of whole requests on one lane: every query, then every delete, then
// every insert, all on `stream` (cf_set_requests.hpp).  The requests' filters
// are attached and their keys sum to at most max_batch.  h_tab (pinned) and
// d_tab: room for one ReqEntry per request, the caller's until the batch has
// completed.
struct ReqEntry;
struct Request {
    uint32_t fid, op;
    const uint64_t *keys;
    uint8_t *results;
    uint64_t n;
};
cf_status requests_lane(cf_set *set, uint32_t lane, const Request *reqs, uint32_t count,
                        ReqEntry *h_tab, ReqEntry *d_tab, hipStream_t stream);
uint64_t req_entry_bytes();

// cf_set_apply on one lane.
cf_status apply_lane(cf_set *set, uint32_t lane, uint32_t fid, uint32_t op, const uint64_t *keys,
                     uint64_t n, uint8_t *results, hipStream_t stream);

}  // namespace cfs
