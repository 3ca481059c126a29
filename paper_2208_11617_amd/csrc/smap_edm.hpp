// smap_edm.hpp -- the Euclidean distances of one lane (EDM, Section 5.1): element
// (x_1, x_2) of Delta_n^2 holds the distance of points i = x_1 and j = n - x_2
// of a set of n+1 points in R^3 (x_1 + x_2 <= n is i <= j), in float32: three
// differences, a sum of squares, a correctly rounded square root.
#pragma once

#include <stdint.h>

#include "smap_bits.hpp"

namespace smap {

// The correctly rounded root of x = 0, x >= 2^-100, infinity or NaN from s, the
// root to within one unit u in the last place (Tuckerman's test: Agarwal,
// Cooley, Gustavson, Shearer, Slishman and Tuckerman, New scalar and vector
// elementary functions for the IBM System/370, IBM J. Res. Dev. 30(2), 1986).
// Of s - u, s and s + u the nearest to the root is s - u where x < (s - u/2)^2
// = s (s - u) + u^2/4 and s + u where x > s (s + u) + u^2/4; x and the products
// are whole multiples of u^2 (at a power of two, where s - u is half as far,
// of u^2/2), so x <= s (s - u) and x > s (s + u) say the same.  A fused
// multiply-add gives each difference's sign: from x = 2^-100 on s and its
// neighbours are multiples of 2^-74, so a difference that isn't 0 is at least
// 2^-148, which float32 holds.  For 0, infinity and NaN both comparisons fail
// and s is the answer.
SMAP_HD float root_rounded(float x, float s)
{
    const float lo = bits_float(float_bits(s) - 1u), hi = bits_float(float_bits(s) + 1u);
    const float below = __builtin_fmaf(-lo, s, x), above = __builtin_fmaf(-hi, s, x);
    float r = below <= 0.0f ? lo : s;
    r = above > 0.0f ? hi : r;
    return r;
}

#if defined(__HIPCC__)
// The hardware's root is within one unit there.
__device__ __forceinline__ float sqrt_rounded(float x) { return root_rounded(x, __builtin_amdgcn_sqrtf(x)); }

// The squares of the distances of 4 points to the point q; returns the least
// nonzero one, as bits minus one.
__device__ __forceinline__ uint32_t edm_squares(const float (&px)[4], const float (&py)[4], const float (&pz)[4],
                                                float qx, float qy, float qz, float (&s)[4])
{
    uint32_t tiny = ~0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float dx = px[k] - qx, dy = py[k] - qy, dz = pz[k] - qz;
        s[k] = __builtin_fmaf(dz, dz, __builtin_fmaf(dx, dx, dy * dy));
        tiny = min(tiny, __float_as_uint(s[k]) - 1u);
    }
    return tiny;
}
// Whether any of them is below 2^-100: the roots need the scaled sqrtf.
__device__ __forceinline__ bool edm_tiny(uint32_t tiny) { return tiny < ((127u - 100u) << 23) - 1u; }
#endif

}  // namespace smap
