// smap_bits.hpp -- the bit-level pieces of the automata's generations and of EDM's
// root: packing, the masks of a word's cells, the sliced counts and rules.
// Host and device code, so that a host check runs these expressions themselves.
#pragma once

#include <stdint.h>
#include <string.h>

#include "smap_decode.hpp"

namespace smap {

SMAP_HD uint32_t float_bits(float f)
{
    uint32_t u;
    memcpy(&u, &f, 4);
    return u;
}
SMAP_HD float bits_float(uint32_t u)
{
    float f;
    memcpy(&f, &u, 4);
    return f;
}

SMAP_HD int32_t clamp31(int32_t v) { return v < 0 ? 0 : (v > 31 ? 31 : v); }

// c plus the dot product of the 4 bytes of a and b.
SMAP_HD uint32_t dot4(uint32_t a, uint32_t b, uint32_t c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_udot4(a, b, c, false);
#else
    for (int k = 0; k < 32; k += 8) c += (a >> k & 255u) * (b >> k & 255u);
    return c;
#endif
}

// Cells of a word inside the simplex, in two parts for a column of words: the
// cells x .. x+31 with x >= 0, and, given those, the cells of row y of which
// number `last` (possibly negative or beyond 31) is the last inside.
SMAP_HD uint32_t ca2k_left_bits(int32_t x)
{
    return x <= -32 ? 0u : ~0u << clamp31(-x);
}
SMAP_HD uint32_t ca2k_row_bits(uint32_t left, int32_t last, int32_t y)
{
    const uint32_t past = 0xFFFFFFFEu << clamp31(last);     // the cells after the last
    const uint32_t none = (uint32_t)((last | y) >> 31);             // no cell at all
    return left & ~past & ~none;
}

// 4 bits -> four 0/1 bytes (bit k -> byte k): bit k of v times 2^(7j)
// lands on bit k + 7j, a multiple of 8 only for j = k, with no carries.
SMAP_HD uint32_t unpack4(uint32_t v) { return ((v & 0xFu) * 0x00204081u) & 0x01010101u; }

// Sixteen bytes -> 16 bits, bit k = bit 0 of byte k: dot products of the
// 0/1 bytes with powers of two, eight bytes per accumulator.
SMAP_HD uint32_t pack16(uint32_t x, uint32_t y, uint32_t z, uint32_t w)
{
    uint32_t lo = dot4(x & 0x01010101u, 0x08040201u, 0u);
    lo = dot4(y & 0x01010101u, 0x80402010u, lo);
    uint32_t hi = dot4(z & 0x01010101u, 0x08040201u, 0u);
    hi = dot4(w & 0x01010101u, 0x80402010u, hi);
    return lo | (hi << 8);
}

// One 3-input logic operation; the immediate is the function of the bit
// patterns A, B, C (of the three inputs).
constexpr uint32_t kBitA = 0xF0u, kBitB = 0xCCu, kBitC = 0xAAu;
template <uint32_t F>
SMAP_HD uint32_t bit3(uint32_t a, uint32_t b, uint32_t c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_bitop3_b32(a, b, c, F & 0xFFu);
#else
    uint32_t r = 0u;                            // the set rows of the truth table
    for (uint32_t i = 0; i < 8; ++i)
        if (F >> i & 1u) r |= (i & 4u ? a : ~a) & (i & 2u ? b : ~b) & (i & 1u ? c : ~c);
    return r;
#endif
}
SMAP_HD uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return bit3<kBitA ^ kBitB ^ kBitC>(a, b, c); }
SMAP_HD uint32_t maj3(uint32_t a, uint32_t b, uint32_t c)
{
    return bit3<(kBitA & kBitB) | (kBitC & (kBitA ^ kBitB))>(a, b, c);
}

// B3/S23 on 32 cells: the horizontal 3-sums (lo, hi bits) of the rows above,
// at and below them, and the cells themselves.  The 3x3 sum with the centre is
// T = a + 2 (k + b) + 4 m; next = (T == 3) | (T == 4 & alive).
SMAP_HD uint32_t life_bits(uint32_t p0, uint32_t p1, uint32_t c0, uint32_t c1, uint32_t n0,
                                              uint32_t n1, uint32_t alive)
{
    const uint32_t a = xor3(p0, c0, n0), k = maj3(p0, c0, n0);
    const uint32_t b = xor3(p1, c1, n1), m = maj3(p1, c1, n1);
    const uint32_t t3 = bit3<(kBitA ^ kBitB) & ~kBitC>(k, b, m);                  // T - a == 2
    const uint32_t t4 = bit3<~(kBitA ^ kBitB) & (kBitA ^ kBitC)>(k, b, m);        // T - a == 4
    const uint32_t s = t4 & alive;
    return bit3<(kBitA & kBitB) | (~kBitA & kBitC)>(a, t3, s);
}

// In-plane 3x3 sum q + 2 (k + t) + 4 m of 32 cells.
struct Ca3kSum {
    uint32_t q, k, t, m;
};

// B6/S567 from three planes' sums and the cells themselves (which are dead
// outside `left`); the result's bits outside `left` and `keep` are cleared.
SMAP_HD uint32_t ca3k_rule(const Ca3kSum &a, const Ca3kSum &b, const Ca3kSum &c, uint32_t alive,
                                              uint32_t left, uint32_t keep)
{
    // T = t0 + 2 t1 + 4 t2 + 8 t3 + 16 t4 (at most 27, the centre included)
    const uint32_t t0 = xor3(a.q, b.q, c.q), u = maj3(a.q, b.q, c.q);
    const uint32_t k = xor3(a.k, b.k, c.k), ck = maj3(a.k, b.k, c.k);
    const uint32_t t = xor3(a.t, b.t, c.t), ct = maj3(a.t, b.t, c.t);
    const uint32_t t1 = xor3(u, k, t), cu = maj3(u, k, t);
    const uint32_t m = xor3(a.m, b.m, c.m), cm = maj3(a.m, b.m, c.m);
    const uint32_t v = xor3(ck, ct, cu), cv = maj3(ck, ct, cu);
    const uint32_t t2 = m ^ v, cw = m & v;
    const uint32_t t3 = xor3(cm, cv, cw), t4 = maj3(cm, cv, cw);
    const uint32_t e67 = bit3<kBitA & kBitB & ~kBitC>(t1, t2, t3);          // T = 6 or 7 (mod 16)
    const uint32_t e89 = bit3<~kBitA & ~kBitB & kBitC>(t1, t2, t3);         // T = 8 or 9
    const uint32_t born = bit3<kBitA & ~kBitB & kBitC>(e67, t0, left);      // T = 6
    const uint32_t stay = bit3<kBitA | (kBitB & ~kBitC)>(e67, e89, t0);     // T = 6, 7 or 8
    const uint32_t next = bit3<(kBitA & kBitB) | (~kBitA & kBitC)>(alive, stay, born);
    return bit3<kBitA & ~kBitB & kBitC>(next, t4, keep);
}

}  // namespace smap
