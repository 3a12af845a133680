// fhp_tile.h -- the tiled pass: many FHP time steps per launch, for lattices
// too small to fill the device with sweeping bands (fhp_stepk.h).
//
// Decomposition.  A workgroup owns a tile: T rows of the lattice and `halo`
// rows above and below, over full rows (periodic) or over C words of which
// the outer one on each side is halo.  Every thread holds one or two words of
// the tile (rows of one column) in registers for the whole launch; a step
// reads the neighbours' words from LDS, streams, collides and publishes its
// own words in the other of two LDS slots, so that a step costs one barrier.
// The halo loses a row and a node per step; after `steps` steps the tile's own
// words are stored.  Steps are a loop: one kernel runs any number of them.
// Waves none of whose rows matter any more skip a step.
//
// What bounds it.  A step takes a wave about 120 VALU instructions per word
// (FHP-II with forcing), 4.9 cycles each with four waves per SIMD, and the
// barrier between publishing and reading, which leaves the SIMD idle unless
// another workgroup has work; per launch 3 to 5 us of launch, loads and
// stores (an empty launch takes 1.7).  The sweep (3 to 5 steps per launch on
// these lattices) pays those and the latency of its level chain every few
// steps: 256^2 1.68 -> 0.52 us per step, 1024^2 2.0 -> 0.67, 2048^2 2.1 ->
// 0.83, 4096^2 2.9 -> 1.8, 8192 x 8128 10.1 -> 6.2, 12288 x 8192 12.8 -> 9.0
// (lattices above 12288^2 nodes stay with the sweep).
//
// Horizontal neighbours are LDS entries of the same row, so any row width
// packs its threads densely; vertical ones are entries of the rows above and
// below.  One word per thread: a thread's row parity decides which of its
// planes shift; the even rows' threads fill the first waves and the odd rows'
// the others, so that the parity is uniform in a wave.  Two words per thread
// (an even row and the odd one below) halve the barriers and a quarter of the
// LDS accesses per word (a step of four waves per SIMD of each takes 0.9 us
// with one word, 1.7 with two), and need tiles of twice the rows: better from
// about 3000^2 on.
#pragma once

#include "fhp_device.h"
#include "fhp_internal.h"
#include "fhp_sweep.h"
#include "fhp_tile_plan.h"

namespace fhp {

struct TileArgs {
    uint32_t H, wd;       // rows, words per row of the lattice
    uint32_t C;           // words per row of a tile
    uint32_t out_words;   // words of a tile row that it stores (C, or C - 2 with halo words)
    uint32_t tiles_x;     // tiles per row of the lattice
    uint32_t T, halo;     // rows a tile stores; rows above and below (even, >= steps)
    uint32_t steps;
    uint32_t split;       // one word per thread: first thread of the odd rows (a multiple of 64)
    uint32_t walls;
    uint64_t ps;
    uint64_t t0;
    uint64_t key_chir, key_force, thr_force;
    uint32_t chi_and, chi_or;
};

namespace {

__device__ __forceinline__ uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Tile of workgroup b of nb.  Workgroups go round-robin to the eight dies (b to
// b mod 8); die x takes the x-th contiguous run of tiles, so that the lines a
// tile shares with its neighbours come through one L2: launches of one step
// 2048^2 9.0 -> 4.5 us, 4096^2 12.0 -> 7.4, 8192 x 8128 46 -> 25.
__device__ __forceinline__ uint32_t tile_of(uint32_t b, uint32_t nb) {
    const uint32_t q = nb >> 3, r = nb & 7, x = b & 7;
    return x * q + min(x, r) + (b >> 3);
}
// The same in runs of 16 of many lattices' tiles: dies stay level where whole
// lattices have no work left.
__device__ __forceinline__ uint32_t tile_item_of(uint32_t b, uint32_t nb) {
    if ((b | 127u) >= nb) return b;  // the last, partial group of 128
    return (b & ~127u) + (b & 7) * 16 + (b >> 3 & 15);
}

// Where a thread stands: its (first) row and column of the tile, the lattice's
// row and word, and the rows of its wave (from its first thread's to its last
// one's, or to the tile's last row where that one has no word).  At the
// tile's edges the neighbour is the thread's own word: those results are
// never stored.
struct TilePlace {
    bool valid, full;
    uint32_t c, row, ty, tx, y, w;
    uint32_t cl, cr;  // columns beside it
    uint32_t row_lo, row_hi;
};

// tile: the tile's number in the lattice, row by row.
__device__ __forceinline__ TilePlace tile_place(const TileArgs& a, uint32_t tile, bool valid, uint32_t row,
                                                uint32_t c, uint32_t rows_each) {
    TilePlace p;
    p.valid = valid;
    p.c = c;
    p.row = row;
    p.full = a.tiles_x == 1;
    p.ty = tile / a.tiles_x;
    p.tx = tile - p.ty * a.tiles_x;
    p.y = (p.ty * a.T + row + a.H - a.halo % a.H) % a.H;
    p.w = p.full ? c : (p.tx * a.out_words + c + a.wd - 1) % a.wd;
    p.cl = c ? c - 1 : (p.full ? a.C - 1 : 0);
    p.cr = c + 1 < a.C ? c + 1 : (p.full ? 0 : c);
    p.row_lo = uniform(row);
    const bool last_on = __builtin_amdgcn_readlane((uint32_t)valid, 63) != 0;
    p.row_hi = last_on ? __builtin_amdgcn_readlane(row, 63) + rows_each - 1 : a.T + 2 * a.halo - 1;
    return p;
}

// Whether the thread's row `row` is one of those its tile stores.
__device__ __forceinline__ bool tile_stores(const TileArgs& a, const TilePlace& p) {
    const uint32_t ry = p.row - a.halo, oc = p.full ? p.c : p.c - 1;
    return p.valid && ry < a.T && p.ty * a.T + ry < a.H && oc < a.out_words &&
           (p.full || p.tx * a.out_words + oc < a.wd);
}

// Steps that the wave takes part in: step st matters to the tile's own rows
// only within steps - 1 - st rows of them.
__device__ __forceinline__ uint32_t tile_live_steps(const TileArgs& a, const TilePlace& p) {
    const uint32_t below = a.halo > p.row_hi ? a.halo - p.row_hi : 0;
    const uint32_t last = a.halo + a.T - 1;
    const uint32_t above = p.row_lo > last ? p.row_lo - last : 0;
    const uint32_t off = max(below, above);
    return off < a.steps ? a.steps - off : 0;
}

// Runs step(slot to read, slot to write) for every step that the wave takes
// part in; it keeps the barriers of the others.  (Skipping inside the step
// cost 30 registers: the state then flows through both branches.)
template <class Slot, class F>
__device__ __forceinline__ void tile_loop(const TileArgs& a, const TilePlace& p, Slot* slots, F&& step) {
    const uint32_t live = tile_live_steps(a, p);
    uint32_t st = 0;
    for (; st + 2 <= live; st += 2) {
        step(slots[0], slots[1]);
        step(slots[1], slots[0]);
    }
    if (st < live) step(slots[0], slots[1]);
    for (st = live; st < a.steps; st++) lds_barrier();
}

// ---------------------------------------------------------------------------
// One word per thread.

// An LDS slot for NT entries: planes 0, 1, 3, 4, and the halves of planes 2
// and 5 that the neighbouring words shift in.
template <int NT>
struct WordSlot {
    uint64_t p0[NT], p1[NT], p3[NT], p4[NT];
    uint32_t h2[NT], l5[NT];
};

// The steps of a thread whose row has parity ODD.
template <bool ODD, int NT, bool FORCE, int RULES>
__device__ __forceinline__ void tile1_steps(WordSlot<NT>* slots, const TileArgs& a, const TilePlace& at,
                                            uint64_t s, uint64_t p[7]) {
    const uint64_t base_y = row_term(0, at.y);
    const uint64_t base_chi = word_base(a.key_chir, at.w) + base_y;
    const uint64_t base_frc = word_base(a.key_force, at.w) + base_y;
    uint32_t chi_and = a.chi_and;  // kept in a vector register (see chir_word)
    asm("" : "+v"(chi_and));
    // Entries of the even rows, from 0, and of the odd ones, from split: a
    // wave's are consecutive.  (With the rows in order it used every second
    // run of C entries, half of the banks: 4% slower on 256^2 to 1024^2.)
    const uint32_t pairs = (a.T + 2 * a.halo) / 2, er = at.row / 2;
    const uint32_t e = er * a.C + at.c, me = ODD ? a.split + e : e;
    const uint32_t up = ODD ? e : er ? a.split + e - a.C : me;
    const uint32_t dn = !ODD ? a.split + e : er + 1 < pairs ? e + a.C : me;
    const uint32_t left = me - at.c + at.cl, right = me - at.c + at.cr;
    // the words beside those above and below, on the side this parity shifts in
    const uint32_t side = ODD ? at.cr : at.cl;
    const uint32_t upn = up - at.c + side, dnn = dn - at.c + side;
    const uint64_t t_step = row_term(1, 0);
    uint64_t tq = row_term(a.t0, 0);
    auto put = [&](WordSlot<NT>& L) __attribute__((always_inline)) {
        if (!at.valid) return;
        L.p0[me] = p[0];
        L.p1[me] = p[1];
        L.p3[me] = p[3];
        L.p4[me] = p[4];
        L.h2[me] = hi32(p[2]);
        L.l5[me] = lo32(p[5]);
    };
    put(slots[0]);
    tile_loop(a, at, slots, [&](WordSlot<NT>& L, WordSlot<NT>& next) __attribute__((always_inline)) {
        const uint64_t R = in_sgprs(tq);
        tq += t_step;
        // One hash covers the writes' latency before the barrier, the other
        // the reads' after it.
        const uint64_t chi = chir_word(mix64(base_chi + R), chi_and, a.chi_or);
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();
        const uint64_t u3 = L.p3[up], u4 = L.p4[up], d0 = L.p0[dn], d1 = L.p1[dn];
        const uint32_t c2 = L.h2[left], c5 = L.l5[right];
        const uint32_t cu = ODD ? ((const uint32_t*)L.p4)[2 * upn] : ((const uint32_t*)L.p3)[2 * upn + 1];
        const uint32_t cd = ODD ? ((const uint32_t*)L.p0)[2 * dnn] : ((const uint32_t*)L.p1)[2 * dnn + 1];
        __builtin_amdgcn_sched_barrier(0);
        uint64_t coin = 0;
        uint32_t upm = 0;
        if (FORCE) {
            const uint64_t hf = mix64(base_frc + R);
            coin = coin_bit(hf);
            upm = coin_up(hf, a.thr_force);
        }
        uint64_t n[7];
        n[3] = ODD ? u3 : rotl1(u3, cu);
        n[4] = ODD ? rotr1(u4, cu) : u4;
        n[0] = ODD ? rotr1(d0, cd) : d0;
        n[1] = ODD ? d1 : rotl1(d1, cd);
        n[2] = rotl1(p[2], c2);
        n[5] = rotr1(p[5], c5);
        n[6] = p[6];
        update<RULES>(n, s, chi, coin, upm, p);
        put(next);
    });
}

template <int NT, bool FORCE, int RULES>
__global__ void __launch_bounds__(NT) k_tile1(const uint64_t* __restrict__ in, uint64_t* __restrict__ out,
                                              const uint64_t* __restrict__ S, TileArgs a) {
    __shared__ WordSlot<NT> slots[2];
    const uint32_t half = (a.T + 2 * a.halo) / 2 * a.C;  // words of one parity
    const uint32_t tid = threadIdx.x;
    const bool odd = uniform(tid) >= a.split;
    const uint32_t e = tid - (odd ? a.split : 0);
    const bool valid = e < half;
    const uint32_t er = valid ? e / a.C : 0, c = valid ? e - er * a.C : 0;
    const TilePlace at = tile_place(a, tile_of(blockIdx.x, gridDim.x), valid, 2 * er + (odd ? 1u : 0u), c, 1);
    const size_t idx = (size_t)at.y * a.wd + at.w;
    uint64_t p[7];
#pragma unroll
    for (int k = 0; k < 7; k++) p[k] = in[k * a.ps + idx];
    uint64_t s = S ? S[idx] : 0ull;
    if (a.walls && (at.y == 0 || at.y == a.H - 1)) s = ~0ull;
    if (odd) tile1_steps<true, NT, FORCE, RULES>(slots, a, at, s, p);
    else tile1_steps<false, NT, FORCE, RULES>(slots, a, at, s, p);
    if (tile_stores(a, at)) {
#pragma unroll
        for (int k = 0; k < 7; k++) out[k * a.ps + idx] = p[k];
    }
}

// ---------------------------------------------------------------------------
// Two words per thread: an even row (e) and the odd row below it (o).

// An LDS slot for NT entries: what the thread above (e0, e1), the one below
// (o3, o4) and those beside (halves; of both rows in one word, the even
// row's in its low half) read.
template <int NT>
struct PairSlot {
    uint64_t e0[NT], e1[NT], o3[NT], o4[NT];
    uint64_t h2[NT], l5[NT];
    uint32_t o1[NT], e4[NT];
};

// Waves per SIMD the compiler is to make room for.
template <int RULES>
constexpr int pair_waves() {
    return RULES == kRulesFHP3 ? 4 : 5;
}

// One tile of a lattice from `in` to `out`.  SOLID: the lattice has obstacles
// or walls.
template <int NT, bool FORCE, bool SOLID, int RULES>
__device__ __forceinline__ void tile2(PairSlot<NT>* slots, const uint64_t* __restrict__ in,
                                      uint64_t* __restrict__ out, const uint64_t* __restrict__ S,
                                      const TileArgs& a, uint32_t tile) {
    const uint32_t rows = a.T + 2 * a.halo;
    const uint32_t tid = threadIdx.x;
    const bool valid = tid < rows / 2 * a.C;
    const uint32_t g = valid ? tid / a.C : 0, c = valid ? tid - g * a.C : 0;
    // H, T and halo are even: the pair never straddles the lattice's last row
    const TilePlace at = tile_place(a, tile, valid, 2 * g, c, 2);
    const size_t idx = (size_t)at.y * a.wd + at.w;
    uint64_t pe[7], po[7];
#pragma unroll
    for (int k = 0; k < 7; k++) {
        pe[k] = in[k * a.ps + idx];
        po[k] = in[k * a.ps + idx + a.wd];
    }
    uint64_t se = 0, so = 0;
    if (SOLID && S) se = S[idx], so = S[idx + a.wd];
    if (SOLID && a.walls && at.y == 0) se = ~0ull;
    if (SOLID && a.walls && at.y + 2 == a.H) so = ~0ull;
    const uint64_t base_y = row_term(0, at.y);
    const uint64_t base_chi = word_base(a.key_chir, at.w) + base_y;
    const uint64_t base_frc = word_base(a.key_force, at.w) + base_y;
    uint32_t chi_and = a.chi_and;
    asm("" : "+v"(chi_and));
    const uint32_t me = g * a.C + c;
    const uint32_t left = me - c + at.cl, right = me - c + at.cr;
    const uint32_t up = g ? me - a.C : me, dn = 2 * g + 2 < rows ? me + a.C : me;
    const uint32_t upl = up - c + at.cl, dnr = dn - c + at.cr;
    const uint64_t t_step = row_term(1, 0), row_step = row_term(0, 1);
    uint64_t tq = row_term(a.t0, 0);
    auto put = [&](PairSlot<NT>& L) __attribute__((always_inline)) {
        if (!valid) return;
        L.e0[me] = pe[0];
        L.e1[me] = pe[1];
        L.o3[me] = po[3];
        L.o4[me] = po[4];
        L.h2[me] = ((uint64_t)hi32(po[2]) << 32) | hi32(pe[2]);
        L.l5[me] = ((uint64_t)lo32(po[5]) << 32) | lo32(pe[5]);
        L.o1[me] = hi32(po[1]);
        L.e4[me] = lo32(pe[4]);
    };
    put(slots[0]);
    tile_loop(a, at, slots, [&](PairSlot<NT>& L, PairSlot<NT>& next) __attribute__((always_inline)) {
        const uint64_t Re = in_sgprs(tq), Ro = in_sgprs(tq + row_step);
        tq += t_step;
        uint64_t coine = 0, coino = 0;
        uint32_t upe = 0, upo = 0;
        auto force = [&](uint64_t R, uint64_t& coin, uint32_t& upm) __attribute__((always_inline)) {
            if (!FORCE) return;
            const uint64_t hf = mix64(base_frc + R);
            coin = coin_bit(hf);
            upm = coin_up(hf, a.thr_force);
        };
        // three hashes cover the writes' latency before the barrier, the
        // fourth the reads' after it
        const uint64_t chie = chir_word(mix64(base_chi + Re), chi_and, a.chi_or);
        const uint64_t chio = chir_word(mix64(base_chi + Ro), chi_and, a.chi_or);
        force(Re, coine, upe);
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();
        const uint64_t o3 = L.o3[up], o4 = L.o4[up], e0 = L.e0[dn], e1 = L.e1[dn];
        const uint64_t h2 = L.h2[left], l5 = L.l5[right];
        const uint32_t o1c = L.o1[left], e4c = L.e4[right];
        const uint32_t o3c = ((const uint32_t*)L.o3)[2 * upl + 1], e0c = ((const uint32_t*)L.e0)[2 * dnr];
        __builtin_amdgcn_sched_barrier(0);
        force(Ro, coino, upo);
        uint64_t n[7], m[7];
        n[0] = po[0];
        n[1] = rotl1(po[1], o1c);
        n[2] = rotl1(pe[2], lo32(h2));
        n[3] = rotl1(o3, o3c);
        n[4] = o4;
        n[5] = rotr1(pe[5], lo32(l5));
        n[6] = pe[6];
        m[0] = rotr1(e0, e0c);
        m[1] = e1;
        m[2] = rotl1(po[2], hi32(h2));
        m[3] = pe[3];
        m[4] = rotr1(pe[4], e4c);
        m[5] = rotr1(po[5], hi32(l5));
        m[6] = po[6];
        update<RULES>(n, se, chie, coine, upe, pe);
        update<RULES>(m, so, chio, coino, upo, po);
        put(next);
    });
    if (tile_stores(a, at)) {
#pragma unroll
        for (int k = 0; k < 7; k++) {
            out[k * a.ps + idx] = pe[k];
            out[k * a.ps + idx + a.wd] = po[k];
        }
    }
}

template <int NT, bool FORCE, bool SOLID, int RULES>
__global__ void __launch_bounds__(NT, pair_waves<RULES>()) k_tile2(const uint64_t* __restrict__ in,
                                                                   uint64_t* __restrict__ out,
                                                                   const uint64_t* __restrict__ S,
                                                                   TileArgs a) {
    __shared__ PairSlot<NT> slots[2];
    tile2<NT, FORCE, SOLID, RULES>(slots, in, out, S, a, tile_of(blockIdx.x, gridDim.x));
}

// Tiles of many lattices in one launch: workgroup b takes item b.  How many
// steps its lattice takes part with: tile_item_steps.
template <bool FORCE, bool SOLID, int RULES>
__global__ void __launch_bounds__(kTileBatchThreads, pair_waves<RULES>())
    k_tiles(const TileMember* __restrict__ members, const TileItem* __restrict__ items, uint32_t done,
            uint32_t launches, uint32_t n, uint32_t tail) {
    __shared__ PairSlot<kTileBatchThreads> slots[2];
    const TileItem it = items[tile_item_of(blockIdx.x, gridDim.x)];
    const TileMember& M = members[it.m];
    TileArgs a;
    a.steps = tile_item_steps(M.steps, done, launches, n, tail);
    if (!a.steps) return;
    a.H = M.H;
    a.wd = M.wd;
    a.C = M.C;
    a.out_words = M.out_words;
    a.tiles_x = M.tiles_x;
    a.T = M.T;
    a.halo = (a.steps + 1) & ~1u;  // tile_halo
    // A launch has kTileBatchThreads threads, whatever its tiles take: waves
    // without a word only keep the barriers, one per step (a 64^2 lattice has
    // words for one wave of eight).
    if (!tile_wave_words(uniform(threadIdx.x), a.T + 2 * a.halo, a.C)) {
        for (uint32_t st = 0; st < a.steps; st++) lds_barrier();
        return;
    }
    a.split = 0;
    a.walls = M.walls;
    a.ps = M.ps;
    a.t0 = M.t0 + done;
    a.key_chir = M.key_chir;
    a.key_force = M.key_force;
    a.thr_force = M.thr_force;
    a.chi_and = M.chi_and;
    a.chi_or = M.chi_or;
    const uint32_t cur = (M.cur ^ launches) & 1;
    tile2<kTileBatchThreads, FORCE, SOLID, RULES>(slots, M.buf[cur], M.buf[cur ^ 1], M.S, a, it.tile);
}

// Picks the kernel with the fewest LDS entries that hold nt threads.
template <bool FORCE, int RULES>
hipError_t launch_tile1(uint32_t grid, uint32_t nt, const uint64_t* in, uint64_t* out, const uint64_t* S,
                        const TileArgs& a, hipStream_t st) {
    if (nt <= 256)
        hipLaunchKernelGGL((k_tile1<256, FORCE, RULES>), dim3(grid), dim3(nt), 0, st, in, out, S, a);
    else if (nt <= 512)
        hipLaunchKernelGGL((k_tile1<512, FORCE, RULES>), dim3(grid), dim3(nt), 0, st, in, out, S, a);
    else if (nt <= 1024)
        hipLaunchKernelGGL((k_tile1<1024, FORCE, RULES>), dim3(grid), dim3(nt), 0, st, in, out, S, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

template <bool FORCE, bool SOLID, int RULES>
hipError_t launch_tile2(uint32_t grid, uint32_t nt, const uint64_t* in, uint64_t* out, const uint64_t* S,
                        const TileArgs& a, hipStream_t st) {
    if (nt <= 512)
        hipLaunchKernelGGL((k_tile2<512, FORCE, SOLID, RULES>), dim3(grid), dim3(nt), 0, st, in, out, S, a);
    else if (nt <= 1024)
        hipLaunchKernelGGL((k_tile2<1024, FORCE, SOLID, RULES>), dim3(grid), dim3(nt), 0, st, in, out, S, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace

// The kernels of one and of two words per thread (fhp_tile1.hip and
// fhp_tile1_fhp3.hip, fhp_tile2.hip: translation units of their own, which
// compile in parallel and under schedules of their own).
hipError_t launch_tiles_1(uint32_t grid, uint32_t nt, bool force, uint32_t rules, const uint64_t* in,
                          uint64_t* out, const uint64_t* S, const TileArgs& a, hipStream_t st);
hipError_t launch_tiles_1_fhp3(uint32_t grid, uint32_t nt, bool force, const uint64_t* in, uint64_t* out,
                               const uint64_t* S, const TileArgs& a, hipStream_t st);
hipError_t launch_tiles_2(uint32_t grid, uint32_t nt, bool force, uint32_t rules, const uint64_t* in,
                          uint64_t* out, const uint64_t* S, const TileArgs& a, hipStream_t st);
// Tiles of many lattices (fhp_tile_batch.hip); solid: any lattice has
// obstacles or walls.
hipError_t launch_tile_items(uint32_t items_n, bool force, bool solid, uint32_t rules,
                             const TileMember* members, const TileItem* items, uint32_t done,
                             uint32_t launches, uint32_t n, uint32_t tail, hipStream_t st);

}  // namespace fhp
