// Host check of the kernels' own bit-level code (csrc/smap_bits.hpp and the root
// of csrc/smap_edm.hpp), each against its plain definition.
#include <cmath>
#include <cstdio>
#include <limits>
#include <random>

#include "../../paper_2208_11617_amd/csrc/smap_edm.hpp"

using namespace smap;

static long bad = 0;
static void expect(bool ok, const char *what, double a, double b)
{
    if (!ok && ++bad < 20) std::printf("%s: %.9g %.9g\n", what, a, b);
}

static void packing()
{
    std::mt19937 rng(1);
    for (uint32_t bits = 0; bits < 65536; ++bits) {
        uint32_t w[4] = {};
        for (int k = 0; k < 16; ++k)                     // only bit 0 of a byte counts
            w[k / 4] |= ((rng() & 0xFEu) | (bits >> k & 1u)) << (8 * (k % 4));
        expect(pack16(w[0], w[1], w[2], w[3]) == bits, "pack16", bits, 0);
    }
    for (uint32_t v = 0; v < 256; ++v)
        for (int k = 0; k < 4; ++k) expect((unpack4(v) >> (8 * k) & 255u) == (v >> k & 1u), "unpack4", v, k);
}

static void masks()
{
    for (int x = -70; x < 40; ++x) {
        const uint32_t left = ca2k_left_bits(x);
        for (int y : {-2147483647, -2, -1, 0, 5}) {
            for (int last = -4; last < 70; ++last) {
                uint32_t want = 0;
                for (int b = 0; b < 32; ++b) want |= (uint32_t)(x + b >= 0 && b <= last && y >= 0) << b;
                expect(ca2k_row_bits(left, last, y) == want, "row_bits", x, last);
            }
        }
    }
}

static void logic()
{
    for (uint32_t i = 0; i < 8; ++i) {
        const uint32_t a = i >> 2, b = i >> 1 & 1u, c = i & 1u;
        expect((xor3(a, b, c) & 1u) == ((a + b + c) & 1u), "xor3", i, 0);
        expect((maj3(a, b, c) & 1u) == (a + b + c) >> 1, "maj3", i, 0);
    }
    for (uint32_t p = 0; p < 4; ++p)
        for (uint32_t c = 0; c < 4; ++c)
            for (uint32_t n = 0; n < 4; ++n)
                for (uint32_t alive = 0; alive < 2; ++alive) {
                    const uint32_t t = p + c + n;
                    const uint32_t got = life_bits(p & 1, p >> 1, c & 1, c >> 1, n & 1, n >> 1, alive) & 1u;
                    expect(got == (uint32_t)(t == 3 || (t == 4 && alive)), "life", t, alive);
                }
    for (uint32_t i = 0; i < 1u << 15; ++i) {             // three sums of four bits, alive, left, keep
        const auto sum = [&](int o) { return Ca3kSum{i >> o & 1, i >> (o + 1) & 1, i >> (o + 2) & 1, i >> (o + 3) & 1}; };
        const Ca3kSum a = sum(0), b = sum(4), c = sum(8);
        uint32_t t = 0;
        for (const Ca3kSum &s : {a, b, c}) t += s.q + 2 * (s.k + s.t) + 4 * s.m;
        const uint32_t alive = i >> 12 & 1, left = i >> 13 & 1, keep = i >> 14 & 1;
        if (alive && !left) continue;                      // cells outside are dead
        if (t > 27) continue;
        const uint32_t want = keep && ((t == 6 && left) || (alive && (t == 7 || t == 8)));
        expect((ca3k_rule(a, b, c, alive, left, keep) & 1u) == want, "ca3 rule", t, alive);
    }
}

static void roots()
{
    const float inf = std::numeric_limits<float>::infinity();
    const auto check = [&](float x) {
        const float want = std::sqrt(x);
        for (const float s : {std::nextafter(want, 0.0f), want, std::nextafter(want, inf)})
            expect(root_rounded(x, s) == want, "root", x, s);
    };
    for (uint32_t b = float_bits(1.0f); b < float_bits(4.0f); b += 3) check(bits_float(b));
    const uint32_t lo = (127u - 100u) << 23, hi = float_bits(inf);
    for (uint32_t k = 0; k < 200000; ++k) {                // both ends of the range, and over all of it
        check(bits_float(lo + k));
        check(bits_float(hi - 1 - k));
        check(bits_float(lo + (uint32_t)((uint64_t)k * (hi - 1 - lo) / 200000)));
    }
    std::mt19937 rng(2);
    for (int k = 0; k < 200000; ++k) {                     // squares and their neighbours
        const float r = bits_float(((127u - 49u) << 23) + rng() % ((49u + 62u) << 23));
        const float x = r * r;
        check(x);
        check(std::nextafter(x, 0.0f));
        check(std::nextafter(x, inf));
    }
    expect(root_rounded(0.0f, 0.0f) == 0.0f, "root of 0", 0, 0);
    expect(root_rounded(inf, inf) == inf, "root of inf", 0, 0);
    expect(std::isnan(root_rounded(std::nanf(""), std::nanf(""))), "root of nan", 0, 0);
}

int main()
{
    packing();
    masks();
    logic();
    roots();
    std::printf("bad=%ld\n", bad);
    return bad != 0;
}
