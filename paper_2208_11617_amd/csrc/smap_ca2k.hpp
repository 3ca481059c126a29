// smap_ca2k.hpp -- several Life generations (B3/S23) per pass over HBM.
//
// The paper's automaton test runs a fixed number of steps (Section 5.1).
// One launch here advances every cell of Delta_n^2 by `gens` <= 32
// generations: a workgroup takes a rho x rho tile plus a halo of
// (W - rho) / 2 >= gens cells on each side, W x W cells in all (cells outside
// the simplex, or outside the box, are dead), steps the whole region `gens`
// times on chip, and writes the tile.  Each generation the band of cells
// whose neighbourhood reached outside the region grows inward by one, so
// after `gens` generations the tile itself is exact.
//
// The region lives in registers, one bit per cell: a lane holds a column of
// R words (32 cells along x each), XL lanes stand side by side along x, and
// the 64 / XL lane groups of a wave and the waves of the workgroup stand
// below one another.  A word's neighbours along x come from the next lanes
// (DPP row shifts; what enters at the region's edge is never used by the
// tile), the rows above and below a lane's run from the neighbouring groups
// through LDS, two words each way per generation, with one barrier.  The
// neighbour count is bit-sliced: a row's horizontal 3-sum is a full adder
// over the row and its copies shifted by one cell, three such 2-bit numbers
// are added by two more full adders, and the rule works on the carries as
// they are: about 14 operations (two 3-input logic operations per full
// adder) step 32 cells.
//
// Bound: HBM up to about 16 generations a pass, the VALU above.  A region kept
// in LDS and read back for every generation (256-cell tiles in 320-cell
// regions) took 288 us for 32 generations at n = 16384 and 60 us for 17 at
// n = 3001; this form takes 109 and 10 us.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "smap_bits.hpp"
#include "smap_ca2.hpp"
#include "smap_decode.hpp"

namespace smap {

// Generations of one pass at most.
constexpr int kCa2kMaxGens = 32;

// XL lanes of 32 cells side by side, R rows per lane, NW waves.
template <int XL, int R, int NW>
struct Ca2kShape {
    static constexpr int W = 32 * XL;                // cells per region row; region rows
    static constexpr int NG = (64 / XL) * NW;        // lane groups, one below the other
    static constexpr int NT = 64 * NW;
    static constexpr int RPI = NT / (2 * XL);        // rows the workgroup loads at once, 16 cells a lane
    static constexpr int LB = W / RPI < 8 ? W / RPI : 8;   // pieces in flight per lane
    static_assert(64 % XL == 0 && NG * R == W && W % (RPI * LB) == 0 && W > 2 * kCa2kMaxGens, "bad CA2K shape");
};

// Tile side that leaves a halo of at least `gens` cells in a region of W
// cells: a multiple of 16, so that the tile is stored in whole 16-cell pieces.
constexpr int ca2k_rho(int w, int gens) { return (w - 2 * gens) / 16 * 16; }

template <int XL, int R, int NW, bool SAFE>
__device__ __forceinline__ void ca2k_tile(const Plan &P, const uint8_t *__restrict__ in,
                                          uint8_t *__restrict__ out, const int32_t *t, int gens)
{
    using Sh = Ca2kShape<XL, R, NW>;
    constexpr int W = Sh::W, NG = Sh::NG, RPI = Sh::RPI, LB = Sh::LB;
    __shared__ uint32_t stage[W][XL];               // the region as bits, while it is loaded and stored
    __shared__ uint32_t edge[2][2][NG][XL];         // [generation parity][first row, last row][group][word]
    const int32_t n = P.n, rho = P.rho;
    const int32_t x0 = t[0] * rho, y0 = t[1] * rho;
    if (x0 + y0 > n) return;                    // uniform: BB tile outside the simplex
    const int32_t halo = (W - rho) / 2;
    const int64_t pitch = P.stride[1];
    const int64_t total = pitch * pitch;
    const int xl = threadIdx.x % XL, grp = threadIdx.x / XL;
    const int32_t xs = x0 - halo, ys = y0 - halo;   // the region's first cell
    const int32_t x = xs + 32 * xl, y = ys + grp * R;   // the lane's first cell

    // 1. Load, 16 cells per lane: consecutive lanes take consecutive pieces of
    //    a row, LB pieces per lane in flight.  A piece with no simplex cell
    //    reads the buffer's first 16 bytes (from n = 15 on a 16-byte access
    //    that starts at a simplex cell stays inside the buffer; below, the
    //    byte-safe loads are used); one that starts left of the box is loaded
    //    from x = 0 and its bits shifted.  The bits go through LDS to the lane
    //    that owns their word.
    {
        const int32_t xc = xs + 16 * (int)(threadIdx.x % (2 * XL)), xa = max(xc, 0);
        const int32_t rt = threadIdx.x / (2 * XL);
        const uint32_t left = ca2k_left_bits(xc);
        const uint32_t up16 = (uint32_t)min(max(-xc, 0), 31);
#pragma unroll 1
        for (int r0 = 0; r0 < W; r0 += RPI * LB) {
            uint4 v[LB];
#pragma unroll
            for (int k = 0; k < LB; ++k) {
                const int32_t yr = ys + r0 + k * RPI + rt;
                const bool has = (yr >= 0) & (xc > -16) & (xa <= n - yr);
                if constexpr (SAFE) {
                    v[k] = make_uint4(0u, 0u, 0u, 0u);
                    if (has) {
                        const int64_t rb = (int64_t)yr * pitch;
                        v[k].x = ld_masked(in + rb, xa, yr, n, total - rb);
                        v[k].y = ld_masked(in + rb, xa + 4, yr, n, total - rb);
                        v[k].z = ld_masked(in + rb, xa + 8, yr, n, total - rb);
                        v[k].w = ld_masked(in + rb, xa + 12, yr, n, total - rb);
                    }
                } else {
                    const int64_t at = (int64_t)yr * pitch + xa;
                    v[k] = *reinterpret_cast<const uint4 *>(in + (has ? at : 0));
                }
            }
#pragma unroll
            for (int k = 0; k < LB; ++k) {
                const int r = r0 + k * RPI + rt;
                const int32_t yr = ys + r;
                const uint32_t w = (pack16(v[k].x, v[k].y, v[k].z, v[k].w) << up16) & ca2k_row_bits(left, n - yr - xc, yr);
                reinterpret_cast<uint16_t *>(&stage[r][0])[threadIdx.x % (2 * XL)] = (uint16_t)w;
            }
        }
    }
    lds_barrier();
    uint32_t a[R];
#pragma unroll
    for (int r = 0; r < R; ++r) a[r] = stage[grp * R + r][xl];
    uint32_t keep[R];                               // the words' cells inside the simplex
#pragma unroll
    for (int r = 0; r < R; ++r) keep[r] = ca2k_row_bits(ca2k_left_bits(x), n - y - r - x, y + r);

    // 2. Generations.  A region that lies inside the simplex needs no mask.
    const bool interior = xs >= 0 && ys >= 0 && xs + ys + 2 * (W - 1) <= n;   // uniform
    auto hsum = [&](uint32_t c, uint32_t &s0, uint32_t &s1) {
        const uint32_t l = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0x111, 0xf, 0xf, true);   // row_shr:1
        const uint32_t r = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0x101, 0xf, 0xf, true);   // row_shl:1
        const uint32_t L = __builtin_amdgcn_alignbit(c, l, 31);    // cell x-1
        const uint32_t Rt = __builtin_amdgcn_alignbit(r, c, 1);    // cell x+1
        s0 = xor3(L, c, Rt);
        s1 = maj3(L, c, Rt);
    };
    const int up = max(grp - 1, 0), down = min(grp + 1, NG - 1);   // (the region's own edge rows go stale)
    auto generations = [&](auto masked) {
        for (int g = 0; g < gens; ++g) {
            uint32_t(*e)[NG][XL] = edge[g & 1];
            e[0][grp][xl] = a[0];
            e[1][grp][xl] = a[R - 1];
            lds_barrier();
            const uint32_t above = e[1][up][xl], below = e[0][down][xl];
            uint32_t p0, p1, c0, c1;
            hsum(above, p0, p1);
            hsum(a[0], c0, c1);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                uint32_t n0, n1;
                hsum(r + 1 < R ? a[r + 1] : below, n0, n1);
                uint32_t res = life_bits(p0, p1, c0, c1, n0, n1, a[r]);
                if constexpr (decltype(masked)::value) res &= keep[r];
                a[r] = res;
                p0 = c0; p1 = c1;
                c0 = n0; c1 = n1;
            }
        }
    };
    if (interior) generations(std::false_type{});
    else generations(std::true_type{});

    // 3. Store, again 16 cells per lane with consecutive lanes along a row;
    //    the tile starts `halo` bits into the region.
#pragma unroll
    for (int r = 0; r < R; ++r) stage[grp * R + r][xl] = a[r];
    lds_barrier();
    const int bit = halo + 16 * (int)(threadIdx.x % (2 * XL));   // region bit of the lane's first cell
    const int32_t xo = x0 + bit - halo;
    if (bit + 16 > halo + rho) return;
    const int wd = bit >> 5, sh = bit & 31;
    const int wn = min(wd + 1, XL - 1);               // (unused where the piece lies in one word)
#pragma unroll 2
    for (int r = threadIdx.x / (2 * XL); r < rho; r += RPI) {
        const int32_t yr = y0 + r;
        const int32_t v = n - yr - xo + 1;           // simplex cells from xo on
        if (v <= 0) break;
        const uint32_t w = __builtin_amdgcn_alignbit(stage[halo + r][wn], stage[halo + r][wd], sh);
        uint32_t w4[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w4[i] = unpack4(w >> (4 * i));
        uint8_t *row = out + (int64_t)yr * pitch;
        if (v >= 16) {
            *reinterpret_cast<uint4 *>(row + xo) = make_uint4(w4[0], w4[1], w4[2], w4[3]);
        } else {
            st_tail(row + xo, w4[0], w4[1], w4[2], w4[3], v);
        }
    }
}

template <int XL, int R, int NW, bool BB, bool SAFE>
__global__ __launch_bounds__(64 * NW, XL >= 16 ? 6 : 8) void k_ca2k(const Plan P, const uint8_t *__restrict__ in,
                                                     uint8_t *__restrict__ out, int gens)
{
    int32_t t[4] = {0, 0, 0, 0};
    const WgId g = wg_id(P);
    if (BB) {
        decode_bb(P, g.x, g.y, 0, t);
    } else {
        if (!decode_h<2>(P, g.x, t)) return;
    }
    ca2k_tile<XL, R, NW, SAFE>(P, in, out, t, gens);
}

}  // namespace smap
