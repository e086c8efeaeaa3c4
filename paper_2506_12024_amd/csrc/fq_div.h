// Binary32 division of many halves by one scale, and reductions over the 16 lanes of a DPP row.
#ifndef FQ_DIV_H
#define FQ_DIV_H

#include <hip/hip_runtime.h>

// w / s in three operations instead of the ten of a full division: y = RN(1 / s) is divided out once, RN(w y) is
// within 1.5 ulp of w / s, and one residual step, RN(q + RN(w - q s) y), rounds w / s with an error of less than
// 2^-22 ulp before the rounding (Markstein's correction, "Computation of elementary functions on the IBM RISC
// System/6000 processor", 1990).  The result is RN(w / s), the IEEE quotient, unless w / s lies that close to the
// middle between two floats.  What the quantizers take from it is round(RN(w / s) + z) for a half w and an integer
// z: that can differ only next to the numbers n / 2 and n / 2 +- 2^-i at which the sum's rounding turns over, and for the
// 11-bit w and 24-bit s all the pairs within 2^-18 ulp of such a middle (1956 of them) round like the division, as do all
// symmetric codes (92 10^6 up to powers of two) and random groups: tests/test_division_pins.py compiles this
// header for the host and goes through them.  For finite halves and scales of groups of halves
// (2^-32 .. 2^17) nothing under- or overflows on the way.  An infinite scale (a group that holds an infinity)
// has y = 0 and would make the residual 0 * infinity: it is left out of the residual, so that finite numerators
// divide to 0 and infinite ones to NaN.
struct Divisor {
    float s, y;
    __device__ __forceinline__ explicit Divisor(float d) : s(d == __builtin_inff() ? 0.0f : d), y(__fdiv_rn(1.0f, d)) {}
    __device__ __forceinline__ float of(float w) const
    {
        const float q0 = __fmul_rn(w, y);
        return __fmaf_rn(__fmaf_rn(-q0, s, w), y, q0);
    }
};

// v of the lane N places on in its row of 16 (cyclic): a vector instruction, no trip through LDS.
template <int N>
__device__ __forceinline__ float row_ror(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xF, 0xF, false));
}
template <int N>
__device__ __forceinline__ int row_ror(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xF, 0xF, false);
}
// minimum / maximum / sum over the 16 lanes of a row, result in all of them
__device__ __forceinline__ float row_min(float v)
{
    v = fminf(v, row_ror<8>(v));
    v = fminf(v, row_ror<4>(v));
    v = fminf(v, row_ror<2>(v));
    return fminf(v, row_ror<1>(v));
}
__device__ __forceinline__ float row_max(float v)
{
    v = fmaxf(v, row_ror<8>(v));
    v = fmaxf(v, row_ror<4>(v));
    v = fmaxf(v, row_ror<2>(v));
    return fmaxf(v, row_ror<1>(v));
}
__device__ __forceinline__ int row_sum(int v)
{
    v += row_ror<8>(v);
    v += row_ror<4>(v);
    v += row_ror<2>(v);
    return v + row_ror<1>(v);
}

#endif
