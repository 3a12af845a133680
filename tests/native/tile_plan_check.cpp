// Checks the tiled pass's shapes (fhp_tile_plan.h) against what its kernels
// assume, over lattices from one word to the widest ones.
#include <cstdio>
#include <cstdlib>

#include "fhp_tile_plan.h"

using namespace fhp;

static long checked = 0;

#define REQUIRE(c)                                                                              \
    do {                                                                                        \
        if (!(c)) {                                                                             \
            printf("FAILED %s: H %u wd %u n %llu T %u C %u\n", #c, H, wd, (unsigned long long)n, T, C); \
            exit(1);                                                                            \
        }                                                                                       \
    } while (0)

// Every word of the lattice is stored by exactly one tile, the threads fit the
// workgroup, and the halo covers the steps.
static void shape(uint32_t H, uint32_t wd, uint64_t n, uint32_t R, uint32_t T, uint32_t C, uint32_t depth,
                  uint32_t max_threads, uint64_t tiles) {
    REQUIRE(T >= 2 && T % 2 == 0);
    REQUIRE(C == wd || (C >= 3 && C < wd));
    REQUIRE(depth >= 1 && depth <= kTileMaxSteps);
    const uint32_t halo = tile_halo(depth), rows = T + 2 * halo;
    REQUIRE(halo >= depth && halo % 2 == 0);
    const uint32_t nt = tile_threads(R, rows, C);
    REQUIRE(nt % 64 == 0 && nt >= 64 && nt <= max_threads);
    // entries: every pair of rows has C of them in each parity's (R = 1) or the
    // pairs' (R = 2) part of the workgroup's LDS entries
    REQUIRE(rows / 2 * C <= (R == 1 ? nt / 2 : nt));
    if (R == 1) REQUIRE(nt / 2 % 64 == 0);
    const uint32_t o = tile_out_words(C, wd), tx = tiles_per_row(C, wd);
    REQUIRE((uint64_t)tx * o >= wd && (uint64_t)(tx - 1) * o < wd);
    const uint32_t ty = (H + T - 1) / T;
    REQUIRE(tiles == 0 || tiles == (uint64_t)tx * ty);
    checked++;
}

int main() {
    const uint32_t Hs[] = {2, 4, 6, 8, 10, 34, 64, 96, 254, 256, 1030, 2048, 4090, 8128, 16384, 65536};
    const uint32_t wds[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 16, 31, 32, 33, 63, 64, 65, 66, 67, 127, 128, 192, 512, 1024};
    for (uint32_t H : Hs)
        for (uint32_t wd : wds) {
            if ((uint64_t)H * wd > 1u << 23) continue;
            for (uint64_t n : {1ull, 2ull, 3ull, 5ull, 9ull, 16ull, 31ull, 32ull, 33ull, 500ull, 100000ull})
                for (int rules = 0; rules < 4; rules++) {
                    const TilePlan p = tile_plan(H, wd, 256, rules & 1, rules & 2, n);
                    const uint32_t T = p.T, C = p.C;
                    REQUIRE(p.R == 1 || p.R == 2);
                    REQUIRE(p.n <= n);
                    shape(H, wd, n, p.R, p.T, p.C, p.n, kTileMaxThreads, 0);
                }
            for (uint32_t n = 1; n <= 32; n++) {
                const TileShape s = tile_shape(H, wd, n);
                if (!s.T) continue;  // bands then
                shape(H, wd, n, 2, s.T, s.C, n, kTileBatchThreads, s.tiles);
            }
        }
    printf("OK %ld shapes\n", checked);
    return 0;
}
