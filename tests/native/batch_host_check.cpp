// The host side of batches, pools and uploads (libfhp.so over the stand-in of
// hip_standin.h): what the tables hold when a kernel that reads them is
// launched, and the order of calls.  The first argument names the check.
#include <stdio.h>
#include <sys/mman.h>

#include "../../include/fhp.h"
#include "../../paper_1208_2428_amd/csrc/fhp_groups.h"
#include "../../paper_1208_2428_amd/csrc/fhp_tile_plan.h"
#include "hip_standin.h"

#define REQUIRE(c)                                                           \
    do {                                                                     \
        if (!(c)) {                                                          \
            printf("FAILED line %d: %s (%s)\n", __LINE__, #c, fhp_last_error()); \
            exit(1);                                                         \
        }                                                                    \
    } while (0)

namespace {

std::vector<fhp_params> lattices;  // of the batch, or the pool's jobs
long tile_launches, band_launches, sim_tiles, sim_sweeps;  // of batches and pools; of single lattices
uint32_t sweep_bands;  // of the last single lattice's sweep
bool all_tiled;  // every step of the check is a tiled one: the kernel's rule keeps tiled_time
std::map<const uint64_t*, uint64_t> tiled_time;  // by a lattice's first buffer

fhp_params params(uint32_t W, uint32_t H) {
    fhp_params p;
    memset(&p, 0, sizeof(p));
    p.abi_version = FHP_ABI_VERSION;
    p.width = W;
    p.height = H;
    p.seed = 7;
    p.fill = 0.3;
    return p;
}

uint64_t* device(size_t bytes) {  // zeros; pages nobody writes cost nothing
    void* p = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED) exit(2);
    return (uint64_t*)p;
}

// Every tile of every member once, each member's shape one its lattice can have.
void check_tiles(const standin::Launch& l) {
    const auto* M = standin::arg<const fhp::TileMember*>(l, 0);
    const auto* it = standin::arg<const fhp::TileItem*>(l, 1);
    const uint32_t n = standin::arg<uint32_t>(l, 4) + standin::arg<uint32_t>(l, 5);
    std::vector<std::vector<int>> seen;
    for (uint32_t i = 0; i < l.grid; i++) {
        const uint32_t m = it[i].m;
        REQUIRE(m < lattices.size());
        REQUIRE(M[m].H >= 2 && M[m].wd >= 1 && M[m].T >= 2 && M[m].T % 2 == 0 && M[m].tiles_x >= 1);
        const uint32_t tiles = (M[m].H + M[m].T - 1) / M[m].T * M[m].tiles_x;
        if (seen.size() <= m) seen.resize(m + 1);
        seen[m].resize(tiles);
        REQUIRE(it[i].tile < tiles && !seen[m][it[i].tile]++);
        REQUIRE(fhp::tile_threads(2, M[m].T + 2 * fhp::tile_halo(n), M[m].C) <= fhp::kTileBatchThreads);
        REQUIRE(M[m].out_words == fhp::tile_out_words(M[m].C, M[m].wd));
    }
    for (size_t m = 0; m < seen.size(); m++) {
        for (int k : seen[m]) REQUIRE(k == 1);
        if (!all_tiled) continue;
        const uint32_t k = fhp::tile_item_steps(M[m].steps, standin::arg<uint32_t>(l, 2), standin::arg<uint32_t>(l, 3),
                                                standin::arg<uint32_t>(l, 4), standin::arg<uint32_t>(l, 5));
        uint64_t& t = tiled_time[M[m].buf[0]];
        REQUIRE(k == 0 || t == M[m].t0 + standin::arg<uint32_t>(l, 2));
        t += k;
    }
}

void check_bands(const standin::Launch& l) {
    const auto* g = standin::arg<const fhp::GroupDesc*>(l, 2);
    const auto* w = standin::arg<const fhp::WaveDesc*>(l, 3);
    bool known = false;
    for (auto& p : lattices) known |= p.width / 64 == g[0].wd;
    REQUIRE(known && g[0].nwaves >= 1 && g[0].T >= 2 && w[g[0].first_wave].m < lattices.size());
}

void launched(const standin::Launch& l) {
    if (l.name.find("k_tiles") != std::string::npos) {
        tile_launches++;
        check_tiles(l);
    } else if (l.name.find("k_batchILi") != std::string::npos) {
        band_launches++;
        check_bands(l);
    }
    sim_tiles += l.name.find("k_tile1") != std::string::npos || l.name.find("k_tile2") != std::string::npos;
    if (l.name.find("k_stepk") != std::string::npos) sim_sweeps++, sweep_bands = l.grid;
}

struct BatchOf {
    fhp_batch* b = nullptr;
    uint64_t* ws;
    size_t bytes = 0;
    BatchOf() {
        REQUIRE(!fhp_batch_workspace_bytes(lattices.data(), (uint32_t)lattices.size(), &bytes));
        ws = device(bytes);
        REQUIRE(!fhp_batch_create(lattices.data(), (uint32_t)lattices.size(), ws, bytes, nullptr, &b));
    }
    ~BatchOf() {
        fhp_batch_destroy(b);
        munmap(ws, bytes);
    }
    void step(uint64_t n) { REQUIRE(!fhp_batch_step(b, n)); }
    void tiling(uint32_t depth) { REQUIRE(!fhp_batch_set_tiling(b, depth, 0, 0, 1)); }
};

// Tiles are launched over tiles' tables whatever was set or asked in between.
void retile() {
    for (int i = 0; i < 3; i++) lattices.push_back(params(320, 96 + 32 * i));
    for (uint32_t depth : {0u, 3u}) {
        BatchOf a;
        a.step(16);
        a.tiling(depth);
        if (depth) a.step(7);
        a.tiling(0);
        a.step(16);
        a.step(5);
        a.tiling(0);
        a.step(3);
    }
    BatchOf z;
    z.step(16);
    z.step(0);
    z.step(16);
    REQUIRE(tile_launches == 4 + 4 + 2);
}

// Calls of one kind after another write no tables and wait for nothing, on
// bands as on tiles.
void repeat() {
    auto quiet = [](BatchOf& a, uint64_t n, bool tiles) {
        a.step(n);
        a.step(n);
        const standin::Counts c = standin::counts;
        const long t = tile_launches;
        for (int i = 0; i < 4; i++) a.step(n);
        REQUIRE(standin::counts.copies == c.copies && standin::counts.waits == c.waits);
        REQUIRE((tile_launches > t) == tiles);
    };
    // words that bands take in calls of one pass
    for (int i = 0; i < 30; i++) lattices.push_back(params(4096, 4096));
    {
        BatchOf a;
        quiet(a, 5, false);
        quiet(a, 16, true);
        quiet(a, 3, false);
        quiet(a, 40, true);
        // a single shallow call keeps the tiles
        const standin::Counts c = standin::counts;
        a.step(5);
        a.step(40);
        REQUIRE(standin::counts.copies == c.copies);
    }
    // a member too large for tiles
    lattices.assign(1, params(16384, 16384));
    lattices.push_back(params(64, 64));
    {
        BatchOf a;
        for (uint64_t n : {5, 16, 40}) quiet(a, n, false);
    }
    lattices.assign(3, params(320, 96));
    BatchOf a;
    for (uint64_t n : {5, 16, 3, 40}) quiet(a, n, true);
}

// Bands or tiles, by the members' shapes and the steps of a call or tick.
void routes() {
    auto batch = [](uint32_t n, uint32_t W, uint32_t H, uint32_t rules, uint64_t steps) {
        lattices.assign(n, params(W, H));
        for (auto& p : lattices) p.rules = rules;
        BatchOf a;
        const long t = tile_launches;
        a.step(steps);
        return tile_launches > t;
    };
    for (uint64_t steps : {3, 4, 5}) REQUIRE(!batch(30, 4096, 4096, FHP_RULES_FHP2, steps));
    for (uint64_t steps : {1, 2, 6, 9, 10}) REQUIRE(batch(30, 4096, 4096, FHP_RULES_FHP2, steps));
    for (uint64_t steps : {2, 3}) REQUIRE(!batch(30, 4096, 4096, FHP_RULES_FHP3, steps));
    for (uint64_t steps : {1, 4}) REQUIRE(batch(30, 4096, 4096, FHP_RULES_FHP3, steps));
    REQUIRE(batch(28, 4096, 4096, FHP_RULES_FHP2, 5));   // fewer rounds
    REQUIRE(!batch(60, 2048, 4096, FHP_RULES_FHP2, 5));  // rows of 32 words: a whole pass only
    REQUIRE(batch(60, 2048, 4096, FHP_RULES_FHP2, 3));
    REQUIRE(batch(60, 1984, 4096, FHP_RULES_FHP2, 5));   // rows that leave lanes idle
    REQUIRE(batch(60, 4096, 2018, FHP_RULES_FHP2, 5));   // one band of 2018 rows
    auto pool = [](uint32_t n, uint32_t W, uint32_t H, uint32_t passes) {
        lattices.assign(n, params(W, H));
        size_t bytes = 0;
        REQUIRE(!fhp_pool_workspace_bytes(n, n * H, (size_t)n * W * H * 2, &bytes));
        uint64_t* arena = device(bytes);
        fhp_pool* pl = nullptr;
        REQUIRE(!fhp_pool_create(arena, bytes, n, n * H, nullptr, &pl));
        uint32_t slot;
        for (auto& p : lattices) REQUIRE(!fhp_pool_admit(pl, &p, 100, &slot));
        const long t = tile_launches;
        REQUIRE(!fhp_pool_tick(pl, passes));
        fhp_pool_destroy(pl);
        munmap(arena, bytes);
        return tile_launches > t;
    };
    for (uint32_t n : {94, 128, 153, 300}) REQUIRE(!pool(n, 2048, 1024, 1));
    for (uint32_t n : {1, 93, 129, 152}) REQUIRE(pool(n, 2048, 1024, 1));
    REQUIRE(pool(300, 2048, 1024, 2) && pool(300, 1984, 1024, 1) && pool(300, 1024, 2048, 1));
    REQUIRE(pool(300, 2048, 1018, 1));
    // on bands, jobs left with fewer steps than a pass end in one launch each
    for (uint64_t rest : {1, 2, 3, 4}) {
        lattices.assign(130, params(2048, 1024));
        size_t bytes = 0;
        REQUIRE(!fhp_pool_workspace_bytes(130, 130 * 32, (size_t)130 * 2048 * 1024 * 2, &bytes));
        uint64_t* arena = device(bytes);
        fhp_pool* pl = nullptr;
        REQUIRE(!fhp_pool_create(arena, bytes, 130, 130 * 32, nullptr, &pl) && !fhp_pool_set_tiling(pl, 0, 32, 0));
        uint32_t slot, done = 0, list[130];
        for (auto& p : lattices) REQUIRE(!fhp_pool_admit(pl, &p, 5 + rest, &slot));
        const standin::Counts c = standin::counts;
        REQUIRE(!fhp_pool_tick(pl, 1) && !fhp_pool_done(pl, list, 130, &done) && done == 130);
        REQUIRE(standin::counts.launches == c.launches + 2 + 130);  // header and bands; the rests
        fhp_pool_destroy(pl);
        munmap(arena, bytes);
    }
}

// Waves with words of a tile are as many as the shapes' model counts.
void waves() {
    for (uint32_t H : {8u, 64u, 96u, 1030u, 4096u})
        for (uint32_t wd : {1u, 2u, 5u, 16u, 31u, 64u, 128u})
            for (uint32_t n = 1; n <= 16; n++) {
                const fhp::TileShape s = fhp::tile_shape(H, wd, n);
                if (!s.T) continue;
                const uint32_t rows = s.T + 2 * fhp::tile_halo(n);
                uint32_t with = 0;
                for (uint32_t t = 0; t < fhp::kTileBatchThreads; t += 64)
                    with += fhp::tile_wave_words(t, rows, s.C);
                REQUIRE(64 * with == fhp::tile_threads(2, rows, s.C));
            }
}

// A pool's jobs: what the kernel runs of each in every tick is what the host
// counts, also while ended jobs stay resident.
void jobs() {
    all_tiled = true;
    for (uint32_t passes = 1; passes <= 5; passes++) {
        lattices.clear();
        tiled_time.clear();
        for (uint32_t i = 0; i < 40; i++) lattices.push_back(params(64 + 64 * (i % 3), 8 + 2 * i));
        size_t bytes = 0;
        REQUIRE(!fhp_pool_workspace_bytes(64, 4096, 64 << 20, &bytes));
        uint64_t* arena = device(bytes);
        fhp_pool* pl = nullptr;
        REQUIRE(!fhp_pool_create(arena, bytes, 64, 4096, nullptr, &pl));
        std::vector<uint32_t> slots;
        uint64_t longest = 0;
        for (uint32_t i = 0; i < lattices.size(); i++) {
            const uint64_t steps = i < 36 ? 1 + i : 20 * i;
            uint32_t slot;
            REQUIRE(!fhp_pool_admit(pl, &lattices[i], steps, &slot));
            slots.push_back(slot);
            longest = std::max(longest, steps);
        }
        uint32_t n_done = 0, done[64];
        for (uint64_t t = 0; t <= longest + 20; t += 5 * passes) {
            uint32_t k;
            REQUIRE(!fhp_pool_tick(pl, passes) && !fhp_pool_done(pl, done, 64, &k));
            n_done += k;
            std::map<uint64_t, int> kernel, host;
            for (auto& q : tiled_time) kernel[q.second]++;
            for (uint32_t slot : slots) {
                fhp_sim* s;
                uint64_t now;
                REQUIRE(!fhp_pool_member(pl, slot, &s) && !fhp_time(s, &now));
                host[now]++;
            }
            REQUIRE(kernel == host);
        }
        REQUIRE(n_done == lattices.size());
        // nothing is launched once all jobs have ended
        const standin::Counts c = standin::counts;
        for (int i = 0; i < 4; i++) REQUIRE(!fhp_pool_tick(pl, passes));
        REQUIRE(standin::counts.launches == c.launches && standin::counts.copies == c.copies);
        fhp_pool_destroy(pl);
        munmap(arena, bytes);
    }
}

struct SimOf {
    fhp_sim* s = nullptr;
    uint64_t* ws;
    size_t bytes = 0;
    SimOf(const fhp_params& p) {
        REQUIRE(!fhp_workspace_bytes(&p, &bytes));
        ws = device(bytes);
        REQUIRE(!fhp_create(&p, ws, bytes, nullptr, &s));
    }
    ~SimOf() {
        fhp_destroy(s);
        munmap(ws, bytes);
    }
    // one launch of n steps: whether it was a sweep
    bool swept(uint64_t n) {
        const long t = sim_tiles, w = sim_sweeps;
        REQUIRE(!fhp_step(s, n) && sim_tiles + sim_sweeps == t + w + 1);
        return sim_sweeps > w;
    }
};

// A state goes up at once, not behind a kernel: every chunk is copied, packed
// and waited for, the note of obstacles cleared in between and read at the end.
void upload() {
    SimOf a(params(256, 256));
    const std::vector<uint8_t> state(256 * 256);
    standin::order.clear();
    REQUIRE(!fhp_set_state(a.s, state.data(), state.size(), 0));
    REQUIRE(standin::order == "cflwclwcw");
}

// Calls of two and three steps (FHP-III: two): one sweep where its bands fill
// the device evenly, else tiles, of wide runs of words.
void shallow() {
    struct {
        uint32_t W, H;
        bool sweep;
    } const cases[] = {{4096, 4096, true}, {4032, 4090, true},  {3456, 4096, true},  {4096, 3442, true},
                       {4096, 4608, true}, {4096, 2048, true},  {4096, 4610, false}, {4032, 4098, false},
                       {4096, 3438, false}, {4096, 2046, false}, {4160, 4032, false}, {2048, 2048, false},
                       {320, 96, false},   {8192, 2048, false}};
    for (auto& c : cases)
        for (uint32_t rules : {FHP_RULES_FHP2, FHP_RULES_FHP1, FHP_RULES_FHP3}) {
            fhp_params p = params(c.W, c.H);
            p.rules = rules;
            SimOf a(p);
            for (uint64_t n : {2, 3}) REQUIRE(a.swept(n) == (c.sweep && (n == 2 || rules != FHP_RULES_FHP3)));
            REQUIRE(!a.swept(4));
            REQUIRE(!fhp_set_depth(a.s, 3) && a.swept(2));
        }
    for (uint32_t wd : {16, 24, 28, 31, 32, 40, 48, 64, 110, 128})
        for (uint32_t H : {1024, 2048, 3072, 4096, 8192})
            for (uint64_t n : {2, 3}) REQUIRE(fhp::tile_plan(H, wd, 256, false, true, n).C >= 10);
}

// Tall lattices of narrow rows: bands of 32 rows in passes of two steps, and in
// light ones of four; other passes and wider rows take bands by rounds.
void tall() {
    struct {
        uint32_t W, H, rules;
        double force;
        uint64_t n;
        bool thirty_two;
    } const cases[] = {
        {384, 500000, 0, 1e-3, 2, true},  {384, 500000, 0, 1e-3, 3, false},  {384, 500000, 0, 1e-3, 4, false},
        {384, 500000, 0, 0.0, 4, true},   {384, 500000, 1, 1e-3, 4, true},   {384, 500000, 2, 1e-3, 2, true},
        {384, 500000, 0, 0.0, 5, false},  {512, 524288, 0, 1e-3, 2, true},   {512, 524288, 0, 0.0, 4, false},
        {768, 300000, 0, 1e-3, 2, true},  {832, 250000, 0, 1e-3, 2, false},  {832, 250000, 0, 0.0, 4, false},
    };
    for (auto& c : cases) {
        fhp_params p = params(c.W, c.H);
        p.rules = c.rules;
        p.force_rate = c.force;
        SimOf a(p);
        REQUIRE(a.swept(c.n));
        REQUIRE((sweep_bands == (c.H + 31) / 32) == c.thirty_two);
    }
    // rows of 64 words, two steps: whole rounds of three waves per SIMD
    SimOf a(params(4096, 65536));
    REQUIRE(a.swept(2));
    const uint32_t rounds = (sweep_bands + 3071) / 3072;
    REQUIRE(sweep_bands > rounds * 3072 - 3072 / 20);
}

}  // namespace

int main(int argc, char** argv) {
    standin::on_launch = launched;
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "retile") retile();
    else if (what == "repeat") repeat();
    else if (what == "waves") waves();
    else if (what == "routes") routes();
    else if (what == "jobs") jobs();
    else if (what == "upload") upload();
    else if (what == "shallow") shallow();
    else if (what == "tall") tall();
    else return 2;
    printf("OK %ld tiled launches, %ld launches of bands\n", tile_launches, band_launches);
    return 0;
}
