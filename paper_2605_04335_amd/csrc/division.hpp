// Division by a cell's diagonal, whose reciprocal is at hand or kept: three
// instructions in place of the ten of an IEEE division.  Finite operands of
// ordinary size (1 / d and the quotient normal numbers).
#pragma once

namespace ibm {

// 1 / d by Newton's method on the hardware reciprocal (off by at most 2^-24.3
// of it over four million samples): two steps square that to below 2^-90, and
// the last rounding is the result's.  The correctly rounded reciprocal, or its
// neighbour where 1 / d lies within 2^-35 units of halfway between the two.
__device__ __forceinline__ double recip(double d)
{
    double r = __builtin_amdgcn_rcp(d);
    r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
    return __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
}

// a / d with r = 1 / d rounded: the product is within two units, its remainder
// a - q d is exact, and adding r times it leaves the last rounding.  Off from
// the quotient by at most 1/2 + 2^-50 units: the correctly rounded quotient, or
// its neighbour where a / d lies that close to halfway.
__device__ __forceinline__ double quot(double a, double d, double r)
{
    const double q = a * r;
    return __builtin_fma(__builtin_fma(-q, d, a), r, q);
}

}  // namespace ibm
