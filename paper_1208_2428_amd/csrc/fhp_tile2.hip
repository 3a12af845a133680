// fhp_tile2.hip -- the tiled pass (kernels in fhp_tile.h) with two words per
// thread.  Scheduled kernel by kernel for the fewest registers (build.py), which
// keeps each row's collision together: us per step, FHP-III 4096^2 3.26 -> 2.85
// and 4096 x 2048 2.08 -> 1.91 with forcing, FHP-II 6016 x 6000 3.11 -> 3.06
// without, 4096^2 and 8192 x 8128 the same.
#include "fhp_tile.h"

namespace fhp {

hipError_t launch_tiles_2(uint32_t grid, uint32_t nt, bool force, uint32_t rules, const uint64_t* in,
                          uint64_t* out, const uint64_t* S, const TileArgs& a, hipStream_t st) {
    const bool solid = S != nullptr || a.walls;
#define FHP_TILE2(FORCE, RULES)                                                    \
    (solid ? launch_tile2<FORCE, true, RULES>(grid, nt, in, out, S, a, st)         \
           : launch_tile2<FORCE, false, RULES>(grid, nt, in, out, S, a, st))
    if (rules == kRulesFHP1) return force ? FHP_TILE2(true, kRulesFHP1) : FHP_TILE2(false, kRulesFHP1);
    if (rules == kRulesFHP3) return force ? FHP_TILE2(true, kRulesFHP3) : FHP_TILE2(false, kRulesFHP3);
    return force ? FHP_TILE2(true, kRulesFHP2) : FHP_TILE2(false, kRulesFHP2);
#undef FHP_TILE2
}

}  // namespace fhp
