// smap_rows.hpp -- ACCUM, HASH and EDM on Delta_n^2 in line-aligned parts of
// rows.
//
// EDM as in smap_edm.hpp, ACCUM and HASH as in smap_point.hpp, whose k_point is
// the route of smaller boxes and of those whose rows start at lines.  The tile
// comes from the H decode or the BB grid.
//
// All three are bound by HBM writes, and those by whole 128-byte lines: a line
// that two workgroups write part by part, from different L2s, costs about
// twice once the box outgrows the caches (n = 16384, 537 MB: 5.2 TB/s where the
// rows happen to start on lines, 3.3 TB/s where they don't, a fill 6.9).  A row
// of the box starts at any element.  So the part of a row that a tile writes
// starts up to a line after the tile does, at a line's start, and ends as much
// later; the elements before a row's first whole line are its first tile's.
// Default tiles, k_point and this (us): n = 16384 EDM 129, 116, HASH 131, 114,
// ACCUM 240, 225; n = 16000 EDM 210, 119, HASH 245, 125, ACCUM 391, 255; n = 8000
// HASH 31.9, 27.9, ACCUM 77, 61.  (Aligned to 32 or 64 bytes only, EDM at n =
// 16384 took 136 and 127 us.)
//
// A lane owns 4 consecutive x_1 (one 16-byte store); in rows kAlign apart the
// parts start at the same offset from the tile, so the lane keeps what depends
// on x_1 alone (EDM: its points; HASH: the state after the first word) over its
// rows of one offset.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "smap_decode.hpp"
#include "smap_edm.hpp"
#include "smap_point.hpp"

namespace smap {

template <int RHO, int OP, int NT, int SUB, bool BB>
__global__ __launch_bounds__(NT) void k_rows(const Plan P, const uint32_t *in, uint32_t *out)
{
    constexpr int G = RHO / 4;                   // lanes per tile row
    constexpr int RPI = NT / G;                  // rows of the workgroup at once
    constexpr int RSUB = RHO / SUB;              // rows of the workgroup
    constexpr int kAlign = RHO < 32 ? RHO : 32;  // elements of a line (half a line at rho = 16)
    constexpr int NB = kAlign > RPI ? kAlign / RPI : 1;   // offsets a lane's rows start at
    static_assert(NT % G == 0 && RHO % SUB == 0 && RSUB % (NB * RPI) == 0 && NB * RPI % kAlign == 0 && RSUB <= NT,
                  "bad row shape");
    int32_t t[4] = {0, 0, 0, 0};
    uint32_t sub;
    const WgId g = wg_id_point<BB>(P);
    if (BB) {
        decode_bb(P, g.x, g.y, 0, t);
        sub = g.z;
    } else {
        if (!decode_h<2>(P, g.x / SUB, t)) return;
        sub = g.x % SUB;
    }
    const int32_t n = P.n;
    const int32_t x0 = t[0] * RHO, y0 = t[1] * RHO + (int32_t)sub * RSUB;
    if (x0 + y0 > n) return;                      // uniform: nothing inside the simplex
    const float *pts = reinterpret_cast<const float *>(in);
    __shared__ float4 rowpt[OP == OP_EDM ? RSUB : 1];     // EDM: the rows' points
    if constexpr (OP == OP_EDM) {
        if (threadIdx.x < RSUB) {
            const int64_t j = n - y0 - (int32_t)threadIdx.x;
            if (j >= 0) rowpt[threadIdx.x] = make_float4(pts[3 * j], pts[3 * j + 1], pts[3 * j + 2], 0.0f);
        }
        lds_barrier();
    }
    const int64_t pitch = P.stride[1];
    const int l = (int)(threadIdx.x % G);

    // The 4 columns i0 .. i0+3 (those below 0 belong to no element) in rows
    // ra, ra + NB RPI, ...  of the workgroup.
    auto walk = [&](int32_t i0, int ra) {
        float px[4], py[4], pz[4];
        uint32_t h1[4];
        if constexpr (OP == OP_EDM) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int64_t i = min(max(i0 + k, 0), n);
                px[k] = pts[3 * i]; py[k] = pts[3 * i + 1]; pz[k] = pts[3 * i + 2];
            }
        } else if constexpr (OP == OP_HASH) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int32_t x = i0 + k;
                h1[k] = hash32_state<0, 1>(0x811C9DC5u, &x);
            }
        }
        int64_t at = (int64_t)(y0 + ra) * pitch + i0;
#pragma unroll 2
        for (int r = ra; r < RSUB; r += NB * RPI, at += (int64_t)(NB * RPI) * pitch) {
            const int32_t y = y0 + r, v = n - y - i0 + 1;    // elements up to the hypotenuse, fewer each row
            if (v <= 0) break;
            const bool whole = v >= 4 && i0 >= 0;
            uint32_t d[4];
            if constexpr (OP == OP_EDM) {
                const float4 q = rowpt[r];
                float s[4];
                if (edm_tiny(edm_squares(px, py, pz, q.x, q.y, q.z, s))) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) d[k] = __float_as_uint(sqrtf(s[k]));
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) d[k] = __float_as_uint(sqrt_rounded(s[k]));
                }
            } else if constexpr (OP == OP_HASH) {
#pragma unroll
                for (int k = 0; k < 4; ++k) d[k] = hash32_fmix((h1[k] ^ (uint32_t)y) * 0x01000193u);
            } else {
                if (whole) {
                    const uint4 q = *reinterpret_cast<const uint4 *>(in + at);
                    d[0] = q.x; d[1] = q.y; d[2] = q.z; d[3] = q.w;
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) d[k] = k < v && i0 + k >= 0 ? in[at + k] : 0u;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) d[k] += 1u;
            }
            if (whole) {
                *reinterpret_cast<uint4 *>(out + at) = make_uint4(d[0], d[1], d[2], d[3]);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k < v && i0 + k >= 0) out[at + k] = d[k];
            }
        }
    };
#pragma unroll 1
    for (int b = 0; b < NB; ++b) {
        const int ra = (int)(threadIdx.x / G) + b * RPI;
        // elements from the tile's start to the next line's in row ra
        const uint32_t a = (uint32_t)(reinterpret_cast<uintptr_t>(out) >> 2) +
                           (uint32_t)(y0 + ra) * (uint32_t)pitch + (uint32_t)x0;
        const int32_t shift = (int32_t)((0u - a) & (uint32_t)(kAlign - 1));
        walk(x0 + shift + 4 * l, ra);
        if (x0 == 0 && 4 * l < shift) walk(shift - 4 * (l + 1), ra);   // before the row's first whole line
    }
}

}  // namespace smap
