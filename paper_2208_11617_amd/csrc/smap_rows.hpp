// smap_rows.hpp -- ACCUM, HASH and EDM on Delta_n^2 in line-aligned parts of
// rows.
//
// EDM (Section 5.1): element (x_1, x_2) holds the distance of points i = x_1
// and j = n - x_2 of a set of n+1 points in R^3 (x_1 + x_2 <= n is i <= j), in
// float32: three differences, a sum of squares, a correctly rounded square
// root.  ACCUM and HASH as in smap_point.hpp.  The tile comes from the H decode
// or the BB grid.
//
// All three are bound by HBM writes, and those by whole 128-byte lines: a line
// that two workgroups write part by part, from different L2s, costs about
// twice (n = 16384, 537 MB: 5.2 TB/s where the rows happen to start on lines,
// 3.3 TB/s where they don't, a fill 6.9).  A row of the box starts at any
// element.  So the part of a row that a tile writes starts up to a line after
// the tile does, at a line's start, and ends as much later; the elements before
// a row's first whole line are its first tile's.  At n = 16384: EDM 148 -> 117
// us, HASH 138 -> 115, ACCUM 247 -> 228; n = 8000: 52 -> 35, 49 -> 34,
// 93 -> 68.  (Aligned to 32 or 64 bytes only, EDM took 136 and 127 us; it also
// loaded its points for every row and used a root that scales its argument
// first, which by themselves were worth 10 us.)
//
// A lane owns 4 consecutive x_1 (one 16-byte store); in rows kAlign apart the
// parts start at the same offset from the tile, so the lane keeps what depends
// on x_1 alone (EDM: its points; HASH: the state after the first word) over its
// rows of one offset.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "smap_decode.hpp"
#include "smap_point.hpp"

namespace smap {

// sqrt(x) correctly rounded, for x = 0, x >= 2^-96, infinity or NaN.  The
// hardware's square root s is within one unit u in the last place.  Of s - u, s
// and s + u the nearest to the root is s - u where x < (s - u/2)^2 =
// s (s - u) + u^2/4 and s + u where x > s (s + u) + u^2/4; floats that near
// are whole multiples of u^2, as the products are, so x <= s (s - u) and
// x > s (s + u) say the same, and a fused multiply-add gives each difference's
// sign exactly (from 2^-96 on it cannot underflow).  For 0, infinity and NaN
// both comparisons fail and s is the answer.
__device__ __forceinline__ float sqrt_rounded(float x)
{
    const float s = __builtin_amdgcn_sqrtf(x);
    const float lo = __uint_as_float(__float_as_uint(s) - 1u), hi = __uint_as_float(__float_as_uint(s) + 1u);
    const float below = __builtin_fmaf(-lo, s, x), above = __builtin_fmaf(-hi, s, x);
    float r = below <= 0.0f ? lo : s;
    r = above > 0.0f ? hi : r;
    return r;
}

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
    const WgId g = wg_id(P);
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
                uint32_t tiny = ~0u;                     // least nonzero square, as bits minus one
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float dx = px[k] - q.x, dy = py[k] - q.y, dz = pz[k] - q.z;
                    s[k] = __builtin_fmaf(dz, dz, __builtin_fmaf(dx, dx, dy * dy));
                    tiny = min(tiny, __float_as_uint(s[k]) - 1u);
                }
                if (tiny < 0x0F7FFFFFu) {                // a square below 2^-96: the scaled root
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
