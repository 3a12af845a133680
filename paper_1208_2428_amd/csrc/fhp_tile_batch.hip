// fhp_tile_batch.hip -- the tiled pass (kernels in fhp_tile.h) over the tiles
// of many lattices, scheduled as fhp_tile2.hip: us per step of 60 and 512
// lattices 9.7 -> 9.5 and 61 -> 59.5, with forcing 10.4 -> 10.1 and the same,
// FHP-III with forcing 17.6 -> 16.3 and 124 -> 117 (without 15.5 -> 16.0 and
// 102 -> 104).
#include "fhp_tile.h"

namespace fhp {

hipError_t launch_tile_items(uint32_t items_n, bool force, bool solid, uint32_t rules,
                             const TileMember* members, const TileItem* items, uint32_t done,
                             uint32_t launches, uint32_t n, uint32_t tail, hipStream_t st) {
    if (items_n == 0) return hipSuccess;
    if (n == 0 || n + tail > kTileMaxSteps) return hipErrorInvalidValue;
    const dim3 grid(items_n), block(kTileBatchThreads);
#define FHP_TILES(FORCE, SOLID, RULES)                                                             \
    hipLaunchKernelGGL((k_tiles<FORCE, SOLID, RULES>), grid, block, 0, st, members, items, done, \
                       launches, n, tail)
#define FHP_TILES_R(RULES)                              \
    do {                                                \
        if (force && solid) FHP_TILES(true, true, RULES); \
        else if (force) FHP_TILES(true, false, RULES);  \
        else if (solid) FHP_TILES(false, true, RULES);  \
        else FHP_TILES(false, false, RULES);            \
    } while (0)
    if (rules == kRulesFHP1) FHP_TILES_R(kRulesFHP1);
    else if (rules == kRulesFHP3) FHP_TILES_R(kRulesFHP3);
    else FHP_TILES_R(kRulesFHP2);
#undef FHP_TILES_R
#undef FHP_TILES
    return hipGetLastError();
}

}  // namespace fhp
