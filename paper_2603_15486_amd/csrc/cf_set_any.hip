// cf_set_any.hip -- the query and delete phase kernels for classes of any
// fingerprint width (small batches on sets that mix widths).
#include "cf_set_persist.hpp"

bool cfs::pick_phase_any(uint32_t hash, uint32_t placement, PhaseLaunch &out) {
    return pick_phase_fb<0, false, 32>(hash, placement, out);
}
