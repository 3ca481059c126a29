// smap_edm.hpp -- the Euclidean distances of one lane (EDM, Section 5.1): element
// (x_1, x_2) of Delta_n^2 holds the distance of points i = x_1 and j = n - x_2
// of a set of n+1 points in R^3 (x_1 + x_2 <= n is i <= j), in float32: three
// differences, a sum of squares, a correctly rounded square root.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

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
// Whether any of them is below 2^-96: the roots need the scaled sqrtf.
__device__ __forceinline__ bool edm_tiny(uint32_t tiny) { return tiny < 0x0F7FFFFFu; }

}  // namespace smap
