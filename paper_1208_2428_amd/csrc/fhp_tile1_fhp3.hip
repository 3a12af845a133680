// fhp_tile1_fhp3.hip -- the tiled pass (kernels in fhp_tile.h) with one word per
// thread for FHP-III (its own translation unit: see fhp_tile1.hip).
#include "fhp_tile.h"

namespace fhp {

hipError_t launch_tiles_1_fhp3(uint32_t grid, uint32_t nt, bool force, const uint64_t* in, uint64_t* out,
                               const uint64_t* S, const TileArgs& a, hipStream_t st) {
    return force ? launch_tile1<true, kRulesFHP3>(grid, nt, in, out, S, a, st)
                 : launch_tile1<false, kRulesFHP3>(grid, nt, in, out, S, a, st);
}

}  // namespace fhp
