// smap_ca3k.hpp -- several B6/S567 generations per pass over HBM (3-D).
//
// The paper's automaton test runs a fixed number of steps (Section 5.1);
// this is that loop on the 3-simplex, blocked in time.  One launch advances
// every cell of Delta_n^3 by `gens` <= 16 generations.  The (x_1, x_2) plane
// is cut into tiles of rho x rho cells, those that meet the 2-simplex being
// the columns of the 3-simplex; a column's planes are cut into pieces of about
// the same height, one workgroup each, which reads its piece with a halo of
// `gens` planes and (W - rho) / 2 >= gens cells on each side (cells outside
// the simplex, or outside the box, dead).  H finds the columns with the 2-D
// map (Theorem 1); the host lists the pieces, tallest first, in the kernel's
// arguments, so that a launch is a whole number of rounds over the chip.
//
// The planes stream through the workgroup along z, all generations at
// once: at step s generation g turns plane s - 2g of generation g - 1 into its
// own, from that plane, the one below and the one above, which generation
// g - 1 made in the step before.  So the generations of a step do not depend on
// each other, every WPG waves of the workgroup work on one of them, and a
// step needs one barrier.  A generation hands its plane to the next through
// LDS (two planes of W x W bits each); what it needs of the planes below are
// their in-plane 3x3 sums, which stay in registers.  Loading a plane (16
// cells per lane, a step or two ahead) and storing the finished one are spread
// over all threads.
//
// A cell is one bit: a lane holds a column of R words (32 cells along x), XW
// lanes side by side, a generation's lanes covering the W x W plane.  The
// count is bit-sliced, in three-input logic operations: a row's 3-sum is a
// full adder over the row and its copies shifted by one cell (the
// neighbouring words by DPP), three rows are added by one full adder per bit
// and kept as the four bits q + 2 (k + t) + 4 m, and three planes of those
// are added by eight more.  Each generation the outermost cells of the
// region go stale by one; the tile itself never sees them.
//
// Bound: the VALU at 16 generations (41 operations per 32 cells), HBM and the
// load latency at 2.  n = 1024, 16 generations: 336 us (the form before, whole
// 96^3 regions in LDS stepped one generation after another with one
// workgroup a CU: 1409); n = 301, 8: 22 us (215, 35 workgroups).  A 128 x 128
// plane and 16 waves are what the registers of a CU hold the sums of.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "smap_bits.hpp"
#include "smap_ca2.hpp"
#include "smap_ca2k.hpp"
#include "smap_decode.hpp"
#include "smap_steps.hpp"

namespace smap {

// XW words (32 cells) and 32 XW rows a plane, R rows per lane, WPG waves per
// generation.
template <int XW, int R, int WPG>
struct Ca3kShape {
    static constexpr int W = 32 * XW;
    static constexpr int YG = 64 * WPG / XW;          // lane rows of a generation
    static constexpr int GS = 16 / WPG;               // generations the workgroup holds
    static constexpr int CH = W * 2 * XW;             // 16-cell pieces of a plane
    // LDS words of one lane row: a stride that spreads the lane rows' reads over all banks
    static constexpr int GP = R * XW + (R * XW % (2 * XW) == 0 ? XW : 0);
    static constexpr int PL = YG * GP;                // LDS words of a plane
    static_assert(YG * R == W && 64 * WPG % XW == 0 && CH <= 1024 && (XW == 2 || XW == 4), "bad CA3K shape");
    static constexpr int threads(int gens)            // of a pass of `gens` generations
    {
        return 64 * WPG * gens > CH ? 64 * WPG * gens : CH;
    }
};

template <int XW, int R, int WPG, bool SAFE>
__device__ __forceinline__ void ca3k_tile(const Plan &P, const uint8_t *__restrict__ in, uint8_t *__restrict__ out,
                                          int32_t tx, int32_t ty, int32_t sub, int gens, int rz)
{
    using Sh = Ca3kShape<XW, R, WPG>;
    constexpr int W = Sh::W, GP = Sh::GP, PL = Sh::PL, YG = Sh::YG;
    __shared__ uint32_t buf[2][Sh::GS + 1][PL];       // [step parity][generation][plane]
    const int32_t n = P.n, rho = P.rho;
    const int32_t x0 = tx * rho, y0 = ty * rho, height = n - x0 - y0 + 1;
    if (sub * rz >= height) return;                    // uniform: BB piece outside the simplex
    // the column's planes in pieces of at most rz, as even as they come
    const int32_t pieces = (height + rz - 1) / rz, each = (height + pieces - 1) / pieces;
    const int32_t z0 = sub * each, z1 = min(z0 + each, height) - 1;
    if (z0 > z1) return;
    const int32_t halo = (W - rho) / 2;
    const int32_t xs = x0 - halo, ys = y0 - halo;     // the region's first cell
    // the first plane with no live cell in the region: its mask is empty, so
    // what it is made from does not matter, and none above it is made
    const int32_t ztop = n - max(xs, 0) - max(ys, 0) + 1;
    const int64_t p1 = n + 1, p2 = p1 * p1;
    const int64_t total = p2 * p1;
    const int tid = threadIdx.x;
    const int gen = __builtin_amdgcn_readfirstlane(tid / (64 * WPG)) + 1;   // the wave's generation

    // Loading: the thread's 16-cell piece of every plane.  A piece with no
    // simplex cell reads the buffer's first 16 bytes (from n = 15 on a 16-byte
    // access that starts at a simplex cell stays inside the buffer; below, the
    // byte-safe loads are used); one that starts left of the box is loaded
    // from x = 0 and its bits shifted.
    const int lr = tid / (2 * XW), lc = tid % (2 * XW);
    const int32_t ly = ys + lr, lx = xs + 16 * lc, lxa = max(lx, 0);
    const bool loads = tid < Sh::CH;
    const int32_t lz = loads && ly >= 0 && lx > -16 ? n - ly - lxa : -1;    // planes 0 .. lz hold a cell of the piece
    const uint32_t loff = (uint32_t)max(ly, 0) * (uint32_t)p1 + (uint32_t)lxa;
    const uint32_t lleft = ca2k_left_bits(lx), lup = (uint32_t)min(max(-lx, 0), 31);
    auto load = [&](int32_t z) {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        const bool has = z <= lz;
        if constexpr (SAFE) {
            if (has) {
                const int64_t rb = (int64_t)z * p2 + (int64_t)ly * p1;
                v.x = ld_masked(in + rb, lxa, ly + z, n, total - rb);
                v.y = ld_masked(in + rb, lxa + 4, ly + z, n, total - rb);
                v.z = ld_masked(in + rb, lxa + 8, ly + z, n, total - rb);
                v.w = ld_masked(in + rb, lxa + 12, ly + z, n, total - rb);
            }
        } else {
            v = *reinterpret_cast<const uint4 *>(in + (has ? (int64_t)z * p2 + loff : (int64_t)0));
        }
        return v;
    };
    const int lat = (lr / R) * GP + (lr % R) * XW + lc / 2;   // LDS word of the piece
    auto commit = [&](int32_t z, const uint4 &v, int slot) {
        const uint32_t w = (pack16(v.x, v.y, v.z, v.w) << lup) & ca2k_row_bits(lleft, n - z - ly - lx, ly);
        reinterpret_cast<uint16_t *>(&buf[slot][0][lat])[lc % 2] = (uint16_t)w;
    };

    // Storing: the thread's 16-cell piece of the tile.
    const int32_t sx = x0 + 16 * lc, sy = y0 + lr;
    const bool stores = lr < rho && 16 * lc < rho;
    const int sb = (halo + 16 * lc) & 31, sw = (halo + 16 * lc) >> 5;
    const int sat = ((halo + lr) / R) * GP + ((halo + lr) % R) * XW;
    auto store = [&](int32_t z, int slot) {
        const int32_t v = n - z - sy - sx + 1;         // simplex cells from sx on
        if (!stores || v <= 0) return;
        const uint32_t *pl = buf[slot][gens];
        const uint32_t w = __builtin_amdgcn_alignbit(pl[sat + min(sw + 1, XW - 1)], pl[sat + sw], sb);
        uint32_t w4[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w4[i] = unpack4(w >> (4 * i));
        uint8_t *row = out + (int64_t)z * p2 + (int64_t)sy * p1;
        if (v >= 16) {
            *reinterpret_cast<uint4 *>(row + sx) = make_uint4(w4[0], w4[1], w4[2], w4[3]);
        } else {
            st_tail(row + sx, w4[0], w4[1], w4[2], w4[3], v);
        }
    };

    // Stepping: the lane's R words of its generation's planes.
    const int gt = tid % (64 * WPG), xw = gt % XW, yg = gt / XW;
    const int32_t gx = xs + 32 * xw, gy = ys + yg * R;
    // cells with x >= 0; the halo being a multiple of R, a lane's rows are all
    // below y = 0 or none is
    const uint32_t left = gy >= 0 ? ca2k_left_bits(gx) : 0u;
    const int32_t last = n - gx - gy;                 // row r, plane z: cells 0 .. last - r - z are inside
    const int32_t za = max(0, z0 - (gens - gen)), zb = min(ztop, z1 + (gens - gen));   // the generation's planes
    const int up = yg > 0 ? (yg - 1) * GP + (R - 1) * XW + xw : xw;          // (the region's edge rows go stale)
    const int mid = yg * GP + xw;
    const int dn = yg < YG - 1 ? (yg + 1) * GP + xw : mid + (R - 1) * XW;
    auto hsum = [&](uint32_t c, uint32_t &s0, uint32_t &s1) {
        constexpr int kPrev = XW == 4 ? 0x90 : 0xA0, kNext = XW == 4 ? 0xF9 : 0xF5;   // quad_perm: x-1, x+1
        const uint32_t l = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, kPrev, 0xf, 0xf, true);
        const uint32_t r = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, kNext, 0xf, 0xf, true);
        const uint32_t L = __builtin_amdgcn_alignbit(c, l, 31);    // cell x-1
        const uint32_t Rt = __builtin_amdgcn_alignbit(r, c, 1);    // cell x+1
        s0 = xor3(L, c, Rt);
        s1 = maj3(L, c, Rt);
    };
    // Reads plane z + 1 of the generation below from slot `rd`, makes plane z
    // in slot `wr` (the two before the generation's first are made from less
    // and never read); Sp and Sc hold the sums of planes z - 1 and z, C plane
    // z; Sp is left with the sums of plane z + 1.
    auto advance = [&](int32_t z, Ca3kSum (&Sp)[R], Ca3kSum (&Sc)[R], uint32_t (&C)[R], int rd, int wr) {
        uint32_t w[R + 2];
        const uint32_t *pl = buf[rd][gen - 1];
        w[0] = pl[up];
#pragma unroll
        for (int r = 0; r < R; ++r) w[r + 1] = pl[mid + r * XW];
        w[R + 1] = pl[dn];
        uint32_t a0, a1, b0, b1;
        hsum(w[0], a0, a1);
        hsum(w[1], b0, b1);
        // cells of row r inside the simplex: the low last - z - r + 1 bits, cut
        // from those of row 0 as a 64-bit number
        const int32_t lz0 = last - z;
        const uint32_t klo = ca2k_row_bits(~0u, lz0, 0), khi = ca2k_row_bits(~0u, lz0 - 32, 0);
        uint32_t *po = buf[wr][gen];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint32_t c0, c1;
            hsum(w[r + 2], c0, c1);
            Ca3kSum S;
            S.q = xor3(a0, b0, c0);
            S.k = maj3(a0, b0, c0);
            S.t = xor3(a1, b1, c1);
            S.m = maj3(a1, b1, c1);
            po[mid + r * XW] = ca3k_rule(Sp[r], Sc[r], S, C[r], left, __builtin_amdgcn_alignbit(khi, klo, r));
            Sp[r] = S;
            C[r] = w[r + 1];
            a0 = b0; a1 = b1;
            b0 = c0; b1 = c1;
        }
    };

    Ca3kSum SA[R] = {}, SB[R] = {};
    uint32_t C[R] = {};
    const int32_t s0 = max(0, z0 - gens) & ~1;         // first step (even: the parity of a step is its slot's)
    const int32_t s1 = z1 + 2 * gens + 1;              // last: stores plane z1
    const int32_t zl = min(ztop, z1 + gens);          // last plane loaded
    constexpr int PF = R >= 8 ? 1 : 2;                 // steps that loads run ahead (the registers allow one at R = 8)
    uint4 next[PF];
#pragma unroll
    for (int h = 0; h < PF; ++h) next[h] = load(s0 + h);
    const bool steps = gen <= gens;
    for (int32_t s = s0; s <= s1; s += 2) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int32_t sc = s + h, z = sc - 2 * gen;
            if (steps && z + 1 >= max(0, za - 1) && z <= zb) {   // uniform
                if (h == 0) advance(z, SA, SB, C, 1, 0);
                else advance(z, SB, SA, C, 0, 1);
            }
            if (sc <= zl) {
                if (loads) commit(sc, next[h % PF], h);
                next[h % PF] = load(sc + PF);
            }
            const int32_t zo = sc - 1 - 2 * gens;
            if (zo >= z0 && zo <= z1) store(zo, 1 - h);
            lds_barrier();
        }
    }
}

template <int XW, int R, int WPG, bool SAFE>
__global__ __launch_bounds__(1024, R >= 4 ? 4 : 8) void k_ca3k(const Plan P, const uint8_t *__restrict__ in,
                                               uint8_t *__restrict__ out, int gens, int rz, const Ca3kUnits U)
{
    const uint32_t u = U.unit[blockIdx.x];
    ca3k_tile<XW, R, WPG, SAFE>(P, in, out, u & 1023u, u >> 10 & 1023u, u >> 20, gens, rz);
}

// The bounding box of columns and pieces.
template <int XW, int R, int WPG, bool SAFE>
__global__ __launch_bounds__(1024, R >= 4 ? 4 : 8) void k_ca3k_bb(const Plan P, const uint8_t *__restrict__ in,
                                                  uint8_t *__restrict__ out, int gens, int rz)
{
    int32_t t[4] = {0, 0, 0, 0};
    const WgId g = wg_id(P);
    decode_bb(P, g.x, g.y, 0, t);
    ca3k_tile<XW, R, WPG, SAFE>(P, in, out, t[0], t[1], (int32_t)g.z, gens, rz);
}

}  // namespace smap
