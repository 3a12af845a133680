// fhp_device.h -- per-word FHP arithmetic shared by the gfx950 kernels.
//
// Every function works on 64 nodes at once: bit b of a uint64 word is node
// x = 64w + b of one row, and a node's seven channels live in seven such words
// (bit-planes).  All functions are pure bit logic; they compile for the device
// and for the host (the host build is used only to check them exhaustively).
//
// Model: arXiv:1208.2428, Sec. 2 (seven channels, motion then scattering,
// bounce-back at boundary nodes, forcing by exchanging bits 2 and 5).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define FHP_HD __host__ __device__ __forceinline__

namespace fhp {

constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kTagInit = 1, kTagChir = 2, kTagForce = 3;

// SplitMix64 finaliser (Steele, Lea & Flood, OOPSLA 2014).
FHP_HD uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Output number n+1 of SplitMix64 started from state key.
FHP_HD uint64_t hash64(uint64_t key, uint64_t n) { return mix64(key + (n + 1) * kGamma); }

// Hash counter of (t, row, 64-node word): t*2^40 + y*2^20 + w.
FHP_HD uint64_t counter(uint64_t t, uint64_t y, uint64_t w) { return (t << 40) + (y << 20) + w; }

// The same hash split into a per-word and a per-row part, so that a kernel
// forms the SplitMix64 state with one 64-bit add:
//   key + (t*2^40 + y*2^20 + w + 1)*gamma = word_base(key, w) + row_term(t, y)  (mod 2^64).
FHP_HD uint64_t word_base(uint64_t key, uint64_t w) { return key + (w + 1) * kGamma; }
FHP_HD uint64_t row_term(uint64_t t, uint64_t y) { return ((t << 40) + (y << 20)) * kGamma; }

// Three-input bit function: bit i of the result is bit (a_i b_i c_i) of the
// truth table TT, i.e. TT = f(0xF0, 0xCC, 0xAA).  One v_bitop3_b32 on gfx950.
constexpr uint32_t kA = 0xF0, kB = 0xCC, kC = 0xAA;

template <uint32_t TT>
FHP_HD uint32_t lop3(uint32_t a, uint32_t b, uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_bitop3_b32(a, b, c, TT & 0xFF);
#else
    uint32_t r = 0;
    for (uint32_t i = 0; i < 8; i++)
        if ((TT >> i) & 1) r |= ((i & 4) ? a : ~a) & ((i & 2) ? b : ~b) & ((i & 1) ? c : ~c);
    return r;
#endif
}

FHP_HD uint32_t mux3(uint32_t s, uint32_t x, uint32_t y) {  // s ? x : y
    return lop3<(kA & kB) | (~kA & kC)>(s, x, y);
}
FHP_HD uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) {
    return lop3<(kA & kB) | (kA & kC) | (kB & kC)>(a, b, c);
}
FHP_HD uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return lop3<kA ^ kB ^ kC>(a, b, c); }
FHP_HD uint32_t or3(uint32_t a, uint32_t b, uint32_t c) { return lop3<kA | kB | kC>(a, b, c); }

// Rule sets (the values of fhp_params.rules).
constexpr int kRulesFHP2 = 0, kRulesFHP1 = 1, kRulesFHP3 = 2;

// Collisions of 32 nodes after streaming (fluid nodes) and bounce-back (solid
// nodes).  a[0..5] moving channels, a[6] rest, s solid, chi chirality.
//
// Every rule is applied as flips, shared by as many channels as possible:
//   o_j = a_j ^ E_k ^ V_class
// with one mask E_k per pair of opposite channels (k = j mod 3, the channels k
// and k+3) and one mask V per parity class (even channels 0, 2, 4, odd
// channels 1, 3, 5; neighbouring channels lie in different classes, channels
// 120 degrees apart in the same one).  With y_k = a_k ^ a_{k+3}:
//   bounce-back of a solid node exchanges the channels of every pair:
//     E_k = y_k;
//   R1, a head-on pair alone (rest particle a spectator) turns by +60 deg
//     (chi = 1) or -60 deg (chi = 0): its own pair and the one it turns to
//     flip; each pair is all set or all clear, so that is every k but the one
//     left alone: E_k = ~(chi ? a_{k+1} : a_{k+2});
//   R2, {0,2,4} <-> {1,3,5}: every y_k is set and all six flip: E_k = y_k;
//   R3, one particle c plus rest <-> {c-1, c+1} without rest.  One class is
//     empty.  E_k = y_k, plus the whole empty class flips: E_k moves each
//     particle to its opposite channel, and flipping the empty class turns
//     what has arrived there into what has to be there.
// So one select (Q: E_k = y_k) serves the bounce, R2 and R3.  The flips of
// the three pairs add up to Q times the parity of the six channels, which
// gives the third one from the other two.

// E_k from d_k = Q & y_k and R1's select (r1) and pick (m_k): see above.
FHP_HD uint32_t pair_flip(uint32_t d, uint32_t r1, uint32_t m) {
    return lop3<(kA | (kB & ~kC)) & 0xFF>(d, r1, m);
}

// Class counts of the six moving channels: even class 2 ce + se, odd class
// 2 co + so.
struct ClassCounts {
    uint32_t se, ce, so, co;
};

FHP_HD ClassCounts class_counts(const uint32_t a[7]) {
    return {xor3(a[0], a[2], a[4]), maj3(a[0], a[2], a[4]), xor3(a[1], a[3], a[5]),
            maj3(a[1], a[3], a[5])};
}

// R1's select: one particle in each class (c1: its first part) and the two
// opposite each other, which is a_0 = a_3 and a_2 = a_5.
FHP_HD uint32_t opposite(uint32_t c1, const uint32_t a[7]) {
    const uint32_t c2 = lop3<kA & ~(kB ^ kC)>(c1, a[0], a[3]);
    return lop3<kA & ~(kB ^ kC)>(c2, a[2], a[5]);
}

// The pair flips of a[0..5] for selects q (Q) and r1, x = parity of the six.
FHP_HD void pair_flips(const uint32_t a[7], uint32_t q, uint32_t r1, uint32_t x, uint32_t chi,
                       uint32_t E[3]) {
    const uint32_t d0 = lop3<kA & (kB ^ kC)>(q, a[0], a[3]);
    const uint32_t d1 = lop3<kA & (kB ^ kC)>(q, a[1], a[4]);
    E[0] = pair_flip(d0, r1, mux3(chi, a[1], a[2]));
    E[1] = pair_flip(d1, r1, mux3(chi, a[2], a[0]));
    E[2] = xor3(E[0], E[1], q & x);
}

// FHP-I: R1 and R2 whatever the rest particle, which never changes.
// 26 operations.
FHP_HD void collide_fhp1(const uint32_t a[7], uint32_t s, uint32_t chi, uint32_t o[7]) {
    const ClassCounts n = class_counts(a);
    const uint32_t x = n.se ^ n.so;
    const uint32_t w = lop3<~(kA ^ kB) & (kA ^ kC)>(n.se, n.ce, n.so);  // e in {0, 3}, x
    const uint32_t q = lop3<kA & ~(kB ^ kC)>(w, n.so, n.co) | s;        // and o in {0, 3}: R2
    const uint32_t e1 = lop3<kA & ~kB & ~kC>(n.se, n.ce, s);            // e = 1, fluid
    const uint32_t r1 = opposite(lop3<kA & kB & ~kC>(e1, n.so, n.co), a);
    uint32_t E[3];
    pair_flips(a, q, r1, x, chi, E);
#pragma unroll
    for (int j = 0; j < 6; j++) o[j] = a[j] ^ E[j % 3];
    o[6] = a[6];
}

// FHP-II: R1, R2 without rest particle, R3.  32 operations (44 when each
// channel selects among its neighbours' values).  Te, To: one class is empty
// and the other (even, odd) holds a colliding number: one particle with a
// rest particle (R3), two (R3) or three (R2) without.  R2's total is odd and
// has no rest particle, R3's parity equals the rest bit, so R3 on a fluid node
// is T with x = rest.
FHP_HD void collide_fhp2(const uint32_t a[7], uint32_t s, uint32_t chi, uint32_t o[7]) {
    const uint32_t r = a[6];
    const ClassCounts n = class_counts(a);
    const uint32_t x = n.se ^ n.so;
    const uint32_t ue = lop3<(kC & kA & ~kB) | (~kC & kB)>(n.se, n.ce, r);  // r ? e = 1 : e >= 2
    const uint32_t uo = lop3<(kC & kA & ~kB) | (~kC & kB)>(n.so, n.co, r);
    const uint32_t te = lop3<kA & ~kB & ~kC>(ue, n.so, n.co);
    const uint32_t to = lop3<kA & ~kB & ~kC>(uo, n.se, n.ce);
    const uint32_t q = or3(te, to, s);
    const uint32_t f = lop3<~(kA ^ kB) & ~kC>(x, r, s);
    const uint32_t vo = te & f, ve = to & f;  // the empty class flips
    const uint32_t e1 = lop3<kA & kB & ~kC>(n.se, n.so, n.ce);
    // s takes the place of co, which the opposite pair implies: with a_0 = a_3
    // and a_2 = a_5 the classes differ in channels 1 and 4 alone, and equal
    // parities make those equal too
    const uint32_t r1 = opposite(e1 & ~s, a);
    uint32_t E[3];
    pair_flips(a, q, r1, x, chi, E);
#pragma unroll
    for (int j = 0; j < 6; j++) o[j] = xor3(a[j], E[j % 3], (j & 1) ? vo : ve);
    o[6] = lop3<kA ^ (kB | kC)>(r, vo, ve);
}

// Collision-saturated FHP-III.  Nodes of mass >= 4 are handled through their
// complement b (particle-hole duality: T(s) = ~T(~s), so the flips of s are
// those of ~s); the rules below therefore meet mass <= 3 only: FHP-II, R1 with
// or without rest, plus for every spectator position j the cycle
// A_j -> B_j -> C_j -> A_j (chi = 1; reversed for chi = 0) with
//   A_j = {j, j+1, j+4}, B_j = {j, j+2, j+5}, C_j = {j+1, j+5} + rest.
// A_j and B_j are a head-on pair and a spectator: y_k is set for the
// spectator's pair alone, and the pair is the next one (A) or the one before
// (B).  The flips:
//   A_j <-> B_j (select D): the pair turns, E_k = ~y_k;
//   A_j, B_j -> C_j (select F): the class holding two empties, and the
//     channel of the other class between those two flips;
//   C_j -> A_j (chi = 1), B_j (chi = 0): in the empty class every channel
//     whose neighbour at +1 (chi = 1) or -1 (chi = 0) is set flips, in the
//     other the particle whose other one lies at +2 or -2.
// F and C flip the rest particle.  Bounce-back flips commute with the
// complement, so solid nodes need no care there.
FHP_HD void collide_fhp3(const uint32_t a[7], uint32_t s, uint32_t chi, uint32_t o[7]) {
    const ClassCounts n0 = class_counts(a);
    const uint32_t x = n0.se ^ n0.so;  // the complement keeps the parity of six channels
    const uint32_t c0 = n0.se & n0.so;
    const uint32_t n1 = xor3(n0.ce, n0.co, c0), n2 = maj3(n0.ce, n0.co, c0);
    // mass >= 4: four or more moving particles, or three with a rest particle
    const uint32_t cm = lop3<(kA & kB & kC)>(x, n1, a[6]) | n2;
    uint32_t b[7];
#pragma unroll
    for (int c = 0; c < 7; c++) b[c] = a[c] ^ cm;
    const uint32_t r = b[6];
    // a class of three channels with e particles has 3 - e after the
    // complement, which flips both bits of e
    const uint32_t se = n0.se ^ cm, ce = n0.ce ^ cm, so = n0.so ^ cm, co = n0.co ^ cm;
    // at most three particles: two or three in one class (ce, co exclude each
    // other); with a rest particle at most two move
    const uint32_t two = ce | co;
    const uint32_t r3 = lop3<(kA & kB) | (~kA & ~kB & kC)>(r, x, two);
    const uint32_t r3f = r3 & ~s;
    const uint32_t vo = lop3<kA & (kB | kC)>(r3f, se, ce);  // the empty class flips
    const uint32_t ve = lop3<kA & (kB | kC)>(r3f, so, co);
    const uint32_t C = lop3<kA & kB & ~kC>(r, two, s);
    const uint32_t xf = x & ~s;
    const uint32_t z = lop3<kA & ~(kB ^ kC)>(xf, ce, se);
    const uint32_t q = or3(z & two, r3, s);  // z & two: R2
    const uint32_t y0 = b[0] ^ b[3], y1 = b[1] ^ b[4];
    const uint32_t p21 = lop3<kA & kB & ~kC>(xf, two, z);   // two and one
    const uint32_t p3 = lop3<kA & ~(kB & kC)>(p21, y0, y1);  // with a head-on pair
    const uint32_t isA = mux3(y0, b[1], mux3(y1, b[2], b[0]));
    const uint32_t D = lop3<kA & ~(kB ^ kC)>(p3, isA, chi);
    const uint32_t F = p3 & ~D;
    const uint32_t r1 = opposite(lop3<kA & kB & ~kC>(se, so, s), b);
    uint32_t E[3];
    E[0] = pair_flip(mux3(y0, q, D), r1, mux3(chi, b[1], b[2]));
    E[1] = pair_flip(mux3(y1, q, D), r1, mux3(chi, b[2], b[0]));
    E[2] = xor3(E[0], E[1], q & x);
    // F and C: the class holding two (even: ge, odd: go); h1, h0 pick C's side.
    // With two of three channels p, q', c of a class set, c is ~(p & q').  R3
    // is disjoint from both: with h1 and h0 set, its flip of the empty class is
    // the other class's term below whatever the neighbours hold.
    const uint32_t g = F | C;
    const uint32_t h1 = lop3<(kA & kB) | kC>(C, chi, r3f), h0 = lop3<(kA & ~kB) | kC>(C, chi, r3f);
    const uint32_t g2[2] = {g & ce, g & co};
    const uint32_t e2[2] = {g2[1] | ve, g2[0] | vo};
#pragma unroll
    for (int j = 0; j < 6; j++) {
        const uint32_t gs = g2[j & 1], gn = e2[j & 1];
        const uint32_t am = b[(j + 5) % 6], ap = b[(j + 1) % 6];
        const uint32_t p2 = b[(j + 2) % 6], m2 = b[(j + 4) % 6];
        // two in the other class: F: A & B, C: chi ? B : A; R3: 1
        const uint32_t u = lop3<(kA | kB) & kC>(am, h1, gn);
        const uint32_t wn = lop3<kA & (kB | kC)>(u, ap, h0);
        // two in this class: F: its particles, C: chi ? ~m2 : ~p2 -- of the
        // two terms at most one is set
        const uint32_t t1 = lop3<~kA & ~kB & kC & 0xFF>(p2, h1, gs);
        const uint32_t t0 = lop3<~kA & ~kB & kC & 0xFF>(m2, h0, gs);
        o[j] = xor3(xor3(a[j], E[j % 3], wn), t1, t0);
    }
    o[6] = a[6] ^ or3(r3f, F, C);
}

// Update of 32 nodes after streaming: collision (fluid) or bounce-back
// (solid) of rule set RULES, then forcing: bits 5 -> 2 where the coin is up,
// on fluid nodes with o5 set and o2 clear.  coin has at most one bit; up is
// all ones (the coin counts) or zero (it does not).
template <int RULES = kRulesFHP2>
FHP_HD void update32(const uint32_t a[7], uint32_t s, uint32_t chi, uint32_t coin, uint32_t up,
                     uint32_t o[7]) {
    if constexpr (RULES == kRulesFHP3) {
        collide_fhp3(a, s, chi, o);
    } else if constexpr (RULES == kRulesFHP2) {
        collide_fhp2(a, s, chi, o);
    } else {
        collide_fhp1(a, s, chi, o);
    }
    const uint32_t cf = lop3<kA & ~kB & kC>(coin, s, up);
    const uint32_t o5 = lop3<kA & ~(kB & ~kC)>(o[5], cf, o[2]);
    const uint32_t o2 = lop3<kA | (kB & kC)>(o[2], cf, o[5]);
    o[5] = o5;
    o[2] = o2;
}

// 64-node version: the two 32-bit halves independently.
template <int RULES = kRulesFHP2>
FHP_HD void update(const uint64_t a[7], uint64_t solid, uint64_t chi, uint64_t coin, uint32_t up,
                   uint64_t o[7]) {
    uint32_t lo[7], hi[7], olo[7], ohi[7];
    for (int c = 0; c < 7; c++) {
        lo[c] = (uint32_t)a[c];
        hi[c] = (uint32_t)(a[c] >> 32);
    }
    update32<RULES>(lo, (uint32_t)solid, (uint32_t)chi, (uint32_t)coin, up, olo);
#if defined(__HIP_DEVICE_COMPILE__)
    // The halves are independent; interleaving them buys no speed on a
    // wave-serial SIMD but nearly doubles the live values (FHP-II at depth 4:
    // 243 VGPRs interleaved, 188 apart).  An empty asm that makes the high
    // inputs depend on the low result keeps them apart.
#pragma unroll
    for (int c = 0; c < 7; c++) asm volatile("" : "+v"(hi[c]) : "v"(olo[c]));
#endif
    update32<RULES>(hi, (uint32_t)(solid >> 32), (uint32_t)(chi >> 32), (uint32_t)(coin >> 32), up,
                    ohi);
    for (int c = 0; c < 7; c++) o[c] = ((uint64_t)ohi[c] << 32) | olo[c];
}

// The same with a coin word that is up wherever it has a bit.
template <int RULES = kRulesFHP2>
FHP_HD void update(const uint64_t a[7], uint64_t solid, uint64_t chi, uint64_t coin, uint64_t o[7]) {
    update<RULES>(a, solid, chi, coin, ~0u, o);
}

// Forcing coin of one 64-node word, h = H(key_force, counter): the coin of
// node h>>58 is up when (h mod 2^32) < thr, thr = floor(f * 2^38) < 2^32.
// The blocked kernels keep it as that node's bit (coin_bit) and a mask that
// is all ones when the coin is up (coin_up); the forcing step folds the mask
// into a bit function it evaluates anyway.
FHP_HD uint64_t coin_bit(uint64_t h) { return 1ull << (h >> 58); }
FHP_HD uint32_t coin_up(uint64_t h, uint64_t thr) { return ((uint32_t)h < (uint32_t)thr) ? ~0u : 0u; }
FHP_HD uint64_t coin_word(uint64_t h, uint64_t thr) { return coin_up(h, thr) ? coin_bit(h) : 0ull; }

// Chirality word of a chirality mode: (h & m_and) | m_or on each 32-bit half
// (m_and, m_or are all ones or all zeros).  With m_and in a vector register
// each half is one three-input bit function.
FHP_HD uint64_t chir_word(uint64_t h, uint32_t m_and, uint32_t m_or) {
    const uint32_t lo = lop3<(kA & kB) | kC>((uint32_t)h, m_and, m_or);
    const uint32_t hi = lop3<(kA & kB) | kC>((uint32_t)(h >> 32), m_and, m_or);
    return ((uint64_t)hi << 32) | lo;
}

}  // namespace fhp
