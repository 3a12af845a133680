// fhp_tile1.hip -- the tiled pass (kernels in fhp_tile.h) with one word per
// thread for FHP-I and FHP-II, and the launch of a tiled pass.  Scheduled for
// instruction-level parallelism kernel by kernel (build.py): few waves per SIMD
// wait on one another, us per step 320 x 96 0.54 -> 0.51, 512^2 0.56 -> 0.54,
// 1024 x 512 0.62 -> 0.59, 1984 x 1030 0.75 -> 0.74, 256^2 the same.  FHP-III,
// 2 to 3.5% slower that way, is in fhp_tile1_fhp3.hip.
#include "fhp_tile.h"

namespace fhp {

hipError_t launch_tiles_1(uint32_t grid, uint32_t nt, bool force, uint32_t rules, const uint64_t* in,
                          uint64_t* out, const uint64_t* S, const TileArgs& a, hipStream_t st) {
    if (rules == kRulesFHP1)
        return force ? launch_tile1<true, kRulesFHP1>(grid, nt, in, out, S, a, st)
                     : launch_tile1<false, kRulesFHP1>(grid, nt, in, out, S, a, st);
    if (rules == kRulesFHP3) return launch_tiles_1_fhp3(grid, nt, force, in, out, S, a, st);
    return force ? launch_tile1<true, kRulesFHP2>(grid, nt, in, out, S, a, st)
                 : launch_tile1<false, kRulesFHP2>(grid, nt, in, out, S, a, st);
}

hipError_t launch_tile(const TilePlan& P, uint32_t steps, const uint64_t* in, uint64_t* out,
                       const Lattice& L, const Dyn& D, uint64_t t, hipStream_t st) {
    TileArgs a;
    a.H = L.H;
    a.wd = L.wd;
    a.C = P.C;
    a.out_words = tile_out_words(P.C, L.wd);
    a.tiles_x = tiles_per_row(P.C, L.wd);
    a.T = P.T;
    a.halo = tile_halo(steps);
    a.steps = steps;
    a.walls = L.walls;
    a.ps = L.ps;
    a.t0 = t;
    a.key_chir = D.key_chir;
    a.key_force = D.key_force;
    a.thr_force = D.thr_force;
    a.chi_and = (D.chir_mode == FHP_CHIR_HASH) ? ~0u : 0u;
    a.chi_or = (D.chir_mode == FHP_CHIR_ONE) ? ~0u : 0u;
    // What the kernels assume: whole pairs of rows, and halo words that
    // `steps` nodes of error do not cross.
    if (!P.R || steps == 0 || steps > kTileMaxSteps || (P.T & 1) || P.T == 0 ||
        (P.C != L.wd && P.C < 3))
        return hipErrorInvalidValue;
    const uint32_t rows = a.T + 2 * a.halo;
    const uint32_t nt = tile_threads(P.R, rows, P.C);
    const uint64_t grid = (uint64_t)((L.H + a.T - 1) / a.T) * a.tiles_x;
    if (nt > kTileMaxThreads || grid > 0x7fffffffull) return hipErrorInvalidValue;
    a.split = nt / 2;
    const bool force = D.thr_force != 0;
    if (P.R == 1) return launch_tiles_1((uint32_t)grid, nt, force, D.rules, in, out, L.S, a, st);
    return launch_tiles_2((uint32_t)grid, nt, force, D.rules, in, out, L.S, a, st);
}

}  // namespace fhp
