// fp64.hpp -- FP64 reciprocal, quotient and square root from the hardware
// estimates: Newton's iteration for the reciprocal, the coupled iteration for
// the root and its reciprocal (Goldschmidt's), each ended by a correction with
// the exact FMA residual.
//
// The estimates (v_rcp_f64, v_rsq_f64) are good to 4.6e-8 and 5.3e-8
// (measured); after one more step on the residual the results are the correctly
// rounded ones.  Over 8 M arguments each in 2^+-40, 2^+-500 and 2^+-1000
// (quotients: divisors of these, quotients in 2^+-1000) all three equal the
// compiler's IEEE division and square root bit for bit, without its operand
// scaling, and v_div_fixup gives zero, infinite and NaN arguments their IEEE
// results.  Without the scaling they are not IEEE's at the ends of the range:
//   rcp64   subnormal results are not correctly rounded
//   div64   NaN for a divisor below 2^-1024 and for a quotient that overflows;
//           subnormal quotients are not correctly rounded
//   sqrt64  a subnormal argument's root is good to 1e-15
// so divisors that are not a density, a speed or a sum of WENO weights (a
// squared field, an estimator's denominator) take the compiler's division.
// Throughput per wave64 instruction on one SIMD (4 waves): 1/x 58 -> 36 cycles,
// sqrt 75 -> 48 cycles.
#pragma once

#include <hip/hip_runtime.h>

namespace mapk {

// 1/x to the last bit before the special cases.  The first step is a product,
// so that an estimate that overflowed (x below 2^-1024) stays infinite: as a
// sum it would be inf - inf
__device__ __forceinline__ double rcp_newton(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = r * __builtin_fma(-x, r, 2.0);
    return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

__device__ __forceinline__ double rcp64(double x)
{
    return __builtin_amdgcn_div_fixup(rcp_newton(x), x, 1.0);
}

__device__ __forceinline__ double div64(double a, double b)
{
    const double r = rcp_newton(b);
    const double q = a * r;
    return __builtin_amdgcn_div_fixup(__builtin_fma(__builtin_fma(-b, q, a), r, q), b, a);
}

// x >= 0 or NaN
__device__ __forceinline__ double sqrt64(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, r, g);
    h = __builtin_fma(h, r, h);
    g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
    return __builtin_amdgcn_div_fixup(g, 1.0, x);
}

// any x: NaN below zero, minus infinity included
__device__ __forceinline__ double sqrt64_any(double x)
{
    return x < 0.0 ? __builtin_nan("") : sqrt64(x);
}

}  // namespace mapk
