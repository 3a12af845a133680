// fhp_tile_plan.h -- host-side choice of the tiled pass's shape, and the tables
// of a launch over many lattices (plain C++: also built on the host alone to be
// checked).
//
// A tile holds rows = T + 2 halo rows of C words; one workgroup steps it n
// times and stores its T x out_words own words.  Deeper launches spread the
// launch, the loads and the stores over more steps but recompute more halo;
// larger tiles recompute less of it but leave fewer workgroups.  The choice is
// the cheapest shape under a model of a launch's time (tile_plan).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace fhp {

constexpr uint32_t kTileMaxSteps = 32;  // deepest tiled launch
constexpr uint32_t kTileMaxThreads = 1024;
constexpr uint32_t kTileBatchThreads = 512;  // workgroup of a launch over many lattices

struct TilePlan {
    uint32_t R;  // rows per thread (0: no plan)
    uint32_t T;  // rows a tile stores (even)
    uint32_t C;  // words per row of a tile (= wd: full rows, periodic)
    uint32_t n;  // most steps per launch
    double us;   // modelled time of all launches
};

inline uint32_t tile_halo(uint32_t steps) { return (steps + 1) & ~1u; }

// Threads of a tile of `rows` rows of C words.  With one row per thread the
// even and the odd rows' threads each start at a wave.
inline uint32_t tile_threads(uint32_t R, uint32_t rows, uint32_t C) {
    const uint32_t half = (rows / 2 * C + 63) / 64 * 64;
    return R == 1 ? 2 * half : half;
}

// Whether the wave whose first thread is `thread` has a word of a tile of two rows
// per thread.
constexpr bool tile_wave_words(uint32_t thread, uint32_t rows, uint32_t C) { return thread < rows / 2 * C; }

inline uint32_t tile_out_words(uint32_t C, uint32_t wd) { return C == wd ? C : C - 2; }
inline uint32_t tiles_per_row(uint32_t C, uint32_t wd) {
    const uint32_t o = tile_out_words(C, wd);
    return (wd + o - 1) / o;
}

// The cheapest shape for `steps` steps of an H x wd-word lattice on `cus`
// compute units.  A step costs a SIMD `work` rows of 64 words: its waves (a
// workgroup's count rounded up to four, one per SIMD: 7 waves cost more than
// 8) times the rows each holds, less those that no longer matter.
//  - Workgroups that have their compute unit to themselves (all tiles in one
//    round, or 1024 threads of two rows): 3.5 us and 0.15 per wave of a SIMD,
//    and a step 0.1 us + 0.22 us a row with one row per thread; 5.5 us, 0.06
//    + 0.25 with two.
//  - Two workgroups per compute unit, one working while the other waits at its
//    barrier: 3 us, and per round 2.1 us + 0.225 or 0.212 us a row (0.235 or
//    0.26 where a single round starts them all together).  Rounds end by
//    halves, a workgroup per compute unit.
// Fitted to launches of 22 lattices from 64^2 to 12288 x 8192 (FHP-II with
// forcing; FHP-III takes 2.2 or 1.9 times the arithmetic, no forcing 0.87).  Measured
// us per step of the shape it picks, and of the fastest of all that it
// considers for 960 steps: 256^2 0.50, 0.50; 512^2 0.55, 0.55; 1024^2 0.67, 0.66;
// 3072^2 1.31, 1.31; 4096^2 1.81, 1.81; 8192 x 8128 6.25, 6.24.
inline TilePlan tile_plan(uint32_t H, uint32_t wd, uint32_t cus, bool fhp3, bool force, uint64_t steps) {
    TilePlan best{};
    uint64_t best_lines = 0;
    auto consider = [&](uint32_t R, uint32_t C, uint32_t threads, uint32_t n) {
        const uint32_t halo = tile_halo(n);
        // the most rows whose threads fit (an even number of waves for R = 1)
        const uint32_t fit = R == 1 ? threads / 128 * 64 / C : threads / C;
        if (2 * fit < 2 * halo + 2) return;
        uint32_t T = std::min(2 * fit - 2 * halo, H);
        const uint32_t ty = (H + T - 1) / T;
        T = ((H + ty - 1) / ty + 1) & ~1u;  // the same number of tiles, even ones
        const uint32_t rows = T + 2 * halo, waves = tile_threads(R, rows, C) / 64;
        const uint64_t grid = (uint64_t)ty * tiles_per_row(C, wd);
        const uint64_t per_cu = (grid + cus - 1) / cus;
        // rows beyond those that still matter are skipped, wave by wave where
        // a wave's rows are many (one word per thread)
        const uint32_t whole = R == 1 ? std::min(128 / C, rows) : R;
        const double live = std::min(1.0, (double)(T + n - 1 + whole) / rows);
        const double alu = (fhp3 ? (R == 1 ? 2.2 : 1.9) : 1.0) * (force ? 1.0 : 0.87);
        const double row = live * ((waves + 3) / 4) * R;  // of one workgroup, on each SIMD
        // LDS: 160 KB hold two workgroups, but one of 1024 threads with R = 2
        // (and registers one of more than 768 with R = 1)
        const bool two = R == 1 ? threads <= (fhp3 ? 640u : 768u) : threads <= 512;
        double launch, step;
        if (per_cu == 1 || !two) {
            launch = (R == 1 ? 3.5 + 0.15 * ((waves + 3) / 4) : 5.5) * per_cu;
            step = per_cu * (R == 1 ? 0.1 + std::max(row, 1.0) * 0.22 * alu : 0.06 + std::max(row, 2.0) * 0.25 * alu);
        } else {
            const double x = (double)grid / (2.0 * cus);
            const double rounds = x <= 1.0 ? 1.0 : 0.5 * (double)((grid + cus - 1) / cus) + 0.13;
            launch = 3.0 + 2.1 * rounds;
            const double c = x <= 1.0 ? (R == 1 ? 0.235 : 0.26) : (R == 1 ? 0.225 : 0.212);
            step = rounds * 2 * row * c * alu;
        }
        const uint64_t launches = (steps + n - 1) / n;
        const double us = launches * launch + (double)steps * step;
        // Calls of two or three steps are mostly loads and stores, which the
        // model has no term for: of shapes it finds equal, the one whose runs
        // of words touch the fewest lines of 16 words (a run at any word:
        // C + 15 words of them on average).  Against the first one found 6%
        // faster over 290 lattices of two steps each, 3% of three: 2048^2
        // 6.4 -> 5.1 us, 1536 x 2048 6.1 -> 5.2.
        const uint32_t cut = C == wd ? 0 : 15;
        const uint64_t lines = grid * (rows * (uint64_t)(C + cut) + T * (uint64_t)(tile_out_words(C, wd) + cut));
        if (best.R == 0 || us < best.us || (steps <= 3 && us == best.us && lines < best_lines)) {
            best_lines = lines;
            best.R = R;
            best.T = T;
            best.C = C;
            best.n = n;
            best.us = us;
        }
    };
    const uint32_t depths[] = {8, 10, 12, 16, 20, 24, 28, kTileMaxSteps};
    const uint32_t widths[] = {5, 6, 8, 10, 13, 15, 18, 24, 34, 0};  // 0: full rows
    uint32_t last_n = 0;
    for (uint32_t n : depths) {
        n = (uint32_t)std::min<uint64_t>(n, steps);
        if (n == last_n) break;
        last_n = n;
        uint32_t last_C = 0;
        for (uint32_t w : widths) {
            if (w ? w >= wd : wd > 66) continue;
            // the fewest tiles of at most w words, evened out
            const uint32_t k = w ? (wd + w - 3) / (w - 2) : 1;
            const uint32_t C = w ? (wd + k - 1) / k + 2 : wd;
            if (C == last_C || (w && C >= wd)) continue;
            last_C = C;
            for (uint32_t t : {256u, 512u, 768u, 1024u}) consider(1, C, t, n);
            for (uint32_t t : {512u, 1024u}) consider(2, C, t, n);
        }
    }
    return best;
}

// Shape of one lattice's tiles in a launch over many (two rows per thread,
// workgroups of kTileBatchThreads): the fewest rows of 64 words updated per
// step, tiles x live waves x 2 (`work`).
struct TileShape {
    uint32_t T, C;
    uint32_t tiles;
    double work;
};

inline TileShape tile_shape(uint32_t H, uint32_t wd, uint32_t n) {
    TileShape best{0, 0, 0, 0.0};
    const uint32_t halo = tile_halo(n);
    const uint32_t widths[] = {5, 6, 8, 10, 13, 15, 18, 24, 34, 0};  // 0: full rows
    for (uint32_t w : widths) {
        if (w ? w >= wd : wd > 66) continue;
        const uint32_t k = w ? (wd + w - 3) / (w - 2) : 1;
        const uint32_t C = w ? (wd + k - 1) / k + 2 : wd;
        if (w && C >= wd) continue;
        const uint32_t fit = kTileBatchThreads / C;
        if (2 * fit < 2 * halo + 2) continue;
        uint32_t T = std::min(2 * fit - 2 * halo, H);
        const uint32_t ty = (H + T - 1) / T;
        T = ((H + ty - 1) / ty + 1) & ~1u;
        const uint32_t rows = T + 2 * halo, tiles = ty * tiles_per_row(C, wd);
        const double live = std::min(1.0, (double)(T + n + 1) / rows);
        const double work = (double)tiles * (tile_threads(2, rows, C) / 64) * live * 2;
        if (!best.T || work < best.work) best = {T, C, tiles, work};
    }
    return best;
}

// One lattice of a tiled launch over many, and one tile of it.
struct TileMember {
    uint64_t* buf[2];
    const uint64_t* S;
    uint64_t ps, t0, key_chir, key_force;
    uint32_t thr_force, chi_and, chi_or;
    uint32_t H, wd, walls, cur;
    uint32_t steps;  // steps it may still run (kNoStepLimit: no limit)
    uint32_t T, C, out_words, tiles_x;
};
struct TileItem {
    uint32_t m, tile;
};
constexpr uint32_t kNoStepLimit = 0xffffffffu;

// Steps that a launch of n steps runs of a lattice whose table entry allows
// `steps`: n, or all it has left where that is at most n + tail, or none where
// an earlier launch ran its last ones.  `done` steps and `launches` launches
// lie between the tables and this launch, all with this tail: a lattice that
// has at most `tail` left then had at most n + tail before the last one.
constexpr uint32_t tile_item_steps(uint32_t steps, uint32_t done, uint32_t launches, uint32_t n, uint32_t tail) {
    if (steps <= done) return 0;
    const uint32_t left = steps - done;
    if (launches && left <= tail) return 0;
    return left <= n + tail ? left : n;
}

}  // namespace fhp
