// fhp_tile_plan.h -- host-side choice of the tiled pass's shape (plain C++:
// also built on the host alone to be checked).
//
// A tile holds rows = T + 2 halo rows of C words; one workgroup steps it n
// times and stores its T x out_words own words.  Deeper launches spread the
// launch, the loads and the stores over more steps but recompute more halo;
// larger tiles recompute less of it but leave fewer workgroups.  The choice is
// the cheapest shape under a model of a launch's time,
//   A + rounds B + n (rounds L + work c)  microseconds,
// rounds = workgroups a compute unit runs one after the other, work = rows of
// 64 words a SIMD updates per step.  Its constants are fitted to 900 measured
// launches of 20 lattices from 64^2 to 16384^2 (model over measured 0.85 to
// 1.15 for 80% of them).  Over those lattices the shape it picks is within 10%
// of the fastest one measured, 1% in the median: 256^2 0.54 us per step (the
// fastest 0.53), 1024^2 0.75 (0.74), 2048^2 1.04 (1.04), 4096^2 2.20 (2.11),
// 8192 x 8128 8.3 (7.5).
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

inline uint32_t tile_out_words(uint32_t C, uint32_t wd) { return C == wd ? C : C - 2; }
inline uint32_t tiles_per_row(uint32_t C, uint32_t wd) {
    const uint32_t o = tile_out_words(C, wd);
    return (wd + o - 1) / o;
}

// Model constants by rows per thread: FHP-I and FHP-II with forcing, FHP-III.
struct TileModel {
    double A, B, L, c;
};
constexpr TileModel kTileModel[2][2] = {{{0.0, 7.7, 0.0, 0.33}, {1.9, 8.2, 0.0, 0.266}},
                                        {{4.8, 4.1, 0.07, 0.55}, {0.4, 9.5, 0.62, 0.40}}};

// The cheapest shape for `steps` steps of an H x wd-word lattice on `cus`
// compute units.  Without forcing a step has 0.8 times the arithmetic.
inline TilePlan tile_plan(uint32_t H, uint32_t wd, uint32_t cus, bool fhp3, bool force, uint64_t steps) {
    TilePlan best{};
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
        // workgroups a compute unit holds: by registers 24 waves (R = 2 and
        // FHP-III: 20 and 16), by its 160 KB of LDS 80 bytes (R = 2: 112) per
        // thread of the kernel's size
        const uint32_t lds = R == 1 ? (threads <= 256 ? 8 : threads <= 512 ? 4 : 2)
                                    : (threads <= 320 ? 4 : threads <= 640 ? 2 : 1);
        const uint32_t regs = (fhp3 ? 16u : R == 1 ? 24u : 20u) / waves;
        const uint32_t held = std::max(1u, std::min(lds, regs));
        const uint64_t per_cu = (grid + cus - 1) / cus;
        const double rounds = (double)((per_cu + held - 1) / held);
        // rows beyond those that still matter are skipped wave by wave
        const double live = std::min(1.0, (double)(T + n - 1 + R) / rows);
        const double work = std::max(live * ((per_cu * waves + 3) / 4), 1.0) * R;
        const TileModel& m = kTileModel[fhp3][R - 1];
        const double launch = m.A + m.B * rounds;
        const double step = m.L * rounds + work * m.c * (force ? 1.0 : 0.8);
        const uint64_t launches = (steps + n - 1) / n;
        const double us = launches * launch + (double)steps * step;
        if (best.R == 0 || us < best.us) {
            best.R = R;
            best.T = T;
            best.C = C;
            best.n = n;
            best.us = us;
        }
    };
    const uint32_t depths[] = {8, 12, 16, 20, 24, 28, kTileMaxSteps};
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
            for (uint32_t t : {256u, 384u, 512u, 640u, 768u, 1024u}) consider(1, C, t, n);
            for (uint32_t t : {320u, 512u, 640u, 768u, 1024u}) consider(2, C, t, n);
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

}  // namespace fhp
