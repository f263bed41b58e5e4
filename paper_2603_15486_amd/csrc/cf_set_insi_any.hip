// cf_set_insi_any.hip -- the insert phase kernel for classes of any
// fingerprint width (built at -O1, see the build script).
#include "cf_set_persist.hpp"

bool cfs::pick_phase_insert_any(uint32_t hash, uint32_t placement, PhaseLaunch &out) {
    return pick_phase_fb<0, true, 32>(hash, placement, out);
}
