// smap_steps.hpp -- host planner of the 3-D passes of several generations: how
// the columns of the 3-simplex are cut into pieces, and their order.  Pure host
// integer code; no HIP calls.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <tuple>
#include <vector>

#include "smap_decode.hpp"

namespace smap {

// Generations of one pass at most.
constexpr int kCa3kMaxGens = 16;

// Pieces of one H launch: x tile, y tile (10 bits each) and piece (12 bits).
constexpr int kCa3kUnits = 768;
struct Ca3kUnits {
    uint32_t unit[kCa3kUnits];
};

constexpr int ca3k_rho(int w, int gens) { return (w - 2 * gens) / 16 * 16; }

// Pieces of at most rz planes in the columns of rho x rho cells of Delta_n^3:
// s + 1 columns are n - rho s + 1 planes high.
inline int64_t steps3_pieces(int64_t n, int rho, int64_t rz)
{
    int64_t c = 0;
    for (int64_t s = 0; s * rho <= n; ++s) c += (s + 1) * ((n - rho * s + rz) / rz);
    return c;
}

// Launch plan of a pass of `gens` generations over Delta_n^3.
struct Steps3Plan {
    int w, rho, rz;                // region side, column side, planes of a piece at most
    int64_t slots;                 // workgroups the chip holds at once
    std::vector<uint32_t> units;   // H: the pieces (Ca3kUnits), tallest first
};

// W: 128-cell regions keep more of what they step; below n = 384 they leave
// too few columns, and the planes of a generation, one after another, are the
// time.  Measured (us; 64, 128): n = 200, 8 generations 16, 25 and 16: 36, 64;
// n = 301: 22, 29 and 51, 72; n = 400: 32, 36 and 81, 83; n = 450: 39, 40 and 112,
// 91; n = 512: 50, 46 and 166, 105.
// rz: a workgroup is counted as filling a CU (two do with 64-cell regions and
// up to 4 generations; with more, and with 128-cell regions up to 4, two would
// fit as well, but are not counted on), and a pass over the chip takes the time of a piece, rz planes
// and about 2 gens more to fill and drain the pipeline of generations; so the
// pieces are made as tall as 1 to 8 whole rounds over the chip's 256 CUs allow,
// whichever is shortest.  n = 1024, 16 generations: 340 us with 256
// pieces, 372 with 512, 501 with 1024; 547 with pieces of 48 planes.
// With more columns than r rounds hold (one round from n of 2100 to 2450 on) the
// search ends at whole columns, which cost more than the r rounds counted; from
// about n = 3250 on they are taken all the same, and are the faster cut:
// columns of all heights, tallest first, end together, and each fills and
// drains the pipeline once.  Whole columns against the best 4 to 8 rounds (ms):
// n = 3300, 9 generations 7.0, 9.8; n = 3750, 8: 12.1, 12.1 and 16: 12.1, 14.7;
// n = 4500, 8: 17.3, 20.6 and 1: 19.2, 20.5.
inline Steps3Plan steps3_plan(int64_t n, int gens)
{
    Steps3Plan S;
    S.w = n < 384 ? 64 : 128;
    S.rho = ca3k_rho(S.w, gens);
    S.slots = S.w == 64 && gens <= 4 ? 512 : 256;
    int64_t best = 0;
    for (int64_t r = 1; r <= 8; ++r) {
        int64_t lo = 1, hi = n + 1;                  // the lowest pieces of which there are at most r rounds
        while (lo < hi) {
            const int64_t mid = (lo + hi) / 2;
            if (steps3_pieces(n, S.rho, mid) <= r * S.slots) hi = mid;
            else lo = mid + 1;
        }
        const int64_t cost = r * (lo + 2 * gens);
        if (r == 1 || cost < best) {
            best = cost;
            S.rz = (int)lo;
        }
    }
    return S;
}

// The pieces of an H pass from the host run of the H map over the columns (P:
// its plan).  More than one round over the chip: tallest first.  One round:
// every piece runs at once, and neighbouring columns share the lines at their
// seams and their halos, so the pieces of one height index go row by row, an
// eighth of them to each XCD (n = 900: 1 generation 137 -> 120 us, 8 151 -> 139,
// 16 level; n = 512, 2: 34.5 -> 31.9).
inline void steps3_units(const Plan &P, Steps3Plan &S)
{
    struct Piece {
        int32_t height, k;
        uint32_t x, y;
    };
    std::vector<Piece> v;
    for (uint32_t w = 0; w < P.total; ++w) {
        int32_t t[4] = {0, 0, 0, 0};
        if (!decode_h<2>(P, w, t)) continue;
        const int32_t height = P.n - P.rho * (t[0] + t[1]) + 1;
        const int32_t pieces = (height + S.rz - 1) / S.rz, each = (height + pieces - 1) / pieces;
        for (int32_t k = 0; k * each < height; ++k)
            v.push_back({std::min(each, height - k * each), k, (uint32_t)t[0], (uint32_t)t[1]});
    }
    const bool once = (int64_t)v.size() <= S.slots;
    if (once)
        std::sort(v.begin(), v.end(), [](const Piece &a, const Piece &b) {
            return std::tie(a.k, a.y, a.x) < std::tie(b.k, b.y, b.x);
        });
    else
        std::stable_sort(v.begin(), v.end(), [](const Piece &a, const Piece &b) { return a.height > b.height; });
    S.units.reserve(v.size());
    for (uint32_t L = 0; L < v.size(); ++L) {
        const Piece &q = v[once ? xcd_remap(L, (uint32_t)v.size()) : L];
        S.units.push_back(q.x | q.y << 10 | (uint32_t)q.k << 20);
    }
}

}  // namespace smap
