// physics.hpp -- device-side pointwise EGLM-MHD physics: pressure, fluxes,
// fast speeds and limiters (paper Sec. 2 and Sec. 3).  T = double for the
// FP64 path; T = float with MIXED = true for the FP32 path, where the
// pressure is recovered in FP64 from the FP32 conserved variables (the
// products of FP32 numbers are exact in FP64, so the cancellation in
// e - rho v^2/2 - B^2/2 at low plasma beta costs no precision).
#pragma once

#include <hip/hip_runtime.h>

#include "fp64.hpp"
#include "map_internal.hpp"

namespace mapk {

template <typename T>
struct Num;

template <>
struct Num<double> {
    static __device__ __forceinline__ double rcp(double x) { return rcp64(x); }
    static __device__ __forceinline__ double sqrt_(double x) { return sqrt64(x); }
    static __device__ __forceinline__ double div(double a, double b) { return div64(a, b); }
    static __device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
    static __device__ __forceinline__ double max_(double a, double b) { return __builtin_fmax(a, b); }
    static __device__ __forceinline__ double min_(double a, double b) { return __builtin_fmin(a, b); }
    // r, or NaN where a is NaN
    static __device__ __forceinline__ double nan_as(double a, double r)
    {
        return __hiloint2double(__builtin_isnan(a) ? 0x7ff80000 : __double2hiint(r), __double2loint(r));
    }
    // b where the mask m is 0, a where it is all ones
    static __device__ __forceinline__ double pick(unsigned m, double a, double b)
    {
        const unsigned lo = (m & (unsigned)__double2loint(a)) | (~m & (unsigned)__double2loint(b));
        const unsigned hi = (m & (unsigned)__double2hiint(a)) | (~m & (unsigned)__double2hiint(b));
        return __hiloint2double((int)hi, (int)lo);
    }
};

template <>
struct Num<float> {
    static __device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
    static __device__ __forceinline__ float sqrt_(float x) { return __builtin_amdgcn_sqrtf(x); }
    static __device__ __forceinline__ float div(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }
    static __device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
    static __device__ __forceinline__ float max_(float a, float b) { return __builtin_fmaxf(a, b); }
    static __device__ __forceinline__ float pick(unsigned m, float a, float b)
    {
        return __uint_as_float((m & __float_as_uint(a)) | (~m & __float_as_uint(b)));
    }
};

// conduction coefficient kappa = kappa0 T^(khalf/2) (Sec. 3.4): whole
// powers by repeated multiplication, then one square root for a half power
__device__ __forceinline__ double kappa_of(double kappa0, int khalf, double T)
{
    double q = 1.0;
    for (int i = 0; i < khalf / 2; i++)
        q = q * T;
    if (khalf & 1)
        q = q * sqrt64_any(T);
    return kappa0 * q;
}

// minmod(a,b) = sgn(a) max(0, min(|a|, sgn(a) b))  (eq. minmod), as the
// smaller of two positive values plus the larger of two negative ones (one of
// the two terms is zero): five FP64 instructions where the sign, its products
// and their selects took about fifteen, and two that keep a NaN in a, which
// the minima and maxima pass over (a NaN in b leaves a, as in the formula)
template <typename T>
__device__ __forceinline__ T lim_minmod(T a, T b)
{
    using N = Num<T>;
    const T r = N::max_(N::min_(a, b), T(0)) + N::min_(N::max_(a, b), T(0));
    return N::nan_as(a, r);
}

// in FP32 the same value is the median of (a, b, 0): the smaller magnitude
// when a and b share a sign, zero otherwise -- one v_med3_f32 instruction
template <>
__device__ __forceinline__ float lim_minmod<float>(float a, float b)
{
    return __builtin_amdgcn_fmed3f(a, b, 0.0f);
}

// slope / flux limiter, chosen at compile time (kernels are instantiated
// per limiter so that no per-call dispatch sits in the cell loop): minmod,
// van Leer (ab + |ab|)/(a + b), or the literal flux limiter of Sec. 3.1 in
// ratio-free form phi(a/b) b
template <int KIND, typename T>
__device__ __forceinline__ T limiter(T a, T b)
{
    if constexpr (KIND == MAP_MINMOD) {
        return lim_minmod(a, b);
    } else if constexpr (KIND == MAP_VANLEER) {
        T ab = a * b;
        return ab <= T(0) ? T(0) : Num<T>::div(ab + fabs(ab), a + b);
    } else {
        return fabs(a) <= fabs(b) ? a : b;
    }
}

// a0 b0 + a1 b1 + a2 b2.  I: the product that is rounded first, the others
// entering by FMAs (the compiler's own choice, I = -1, depends on which of the
// products another expression shares, and with it the last bits)
template <int I, typename T>
__device__ __forceinline__ T dot3(T a0, T b0, T a1, T b1, T a2, T b2)
{
    if constexpr (I < 0) {
        return a0 * b0 + a1 * b1 + a2 * b2;
    } else {
#pragma clang fp contract(off)
        using N = Num<T>;
        return N::fma_(a2, b2, I == 0 ? N::fma_(a1, b1, a0 * b0) : N::fma_(a0, b0, a1 * b1));
    }
}

template <typename T, bool MIXED>
struct Phys {
    T gamma, gm1;
    double gm1d;

    // p = (gamma - 1)(e - rho v^2/2 - B^2/2); ir = 1/rho, v = m ir.
    // MIXED: recovered in FP64 from the FP32 conserved variables, whose
    // products are exact in FP64, so the cancellation at low beta costs no
    // precision.
    __device__ __forceinline__ T pressure(const T u[NV], T ir, T vx, T vy, T vz, T me) const
    {
        if constexpr (MIXED) {
            double r = (double)ir;
            r = r * (2.0 - (double)u[RHO] * r);  // one Newton step on 1/rho
            double m2 = (double)u[MX] * (double)u[MX] + (double)u[MY] * (double)u[MY] +
                        (double)u[MZ] * (double)u[MZ];
            double b2 = (double)u[BX] * (double)u[BX] + (double)u[BY] * (double)u[BY] +
                        (double)u[BZ] * (double)u[BZ];
            return (T)(gm1d * (((double)u[EN] - 0.5 * m2 * r) - 0.5 * b2));
        } else {
            T ke = T(0.5) * (u[MX] * vx + u[MY] * vy + u[MZ] * vz);
            return gm1 * (u[EN] - ke - me);
        }
    }

    __device__ __forceinline__ bool admissible(const T u[NV]) const
    {
        if (!(u[RHO] > T(0)))
            return false;
        T ir = Num<T>::rcp(u[RHO]);
        T vx = u[MX] * ir, vy = u[MY] * ir, vz = u[MZ] * ir;
        T me = T(0.5) * (u[BX] * u[BX] + u[BY] * u[BY] + u[BZ] * u[BZ]);
        return pressure(u, ir, vx, vy, vz, me) > T(0);
    }

    // flux<D, false> with the contractions written out, so that every inlined
    // instance gives the same bits
    template <int D>
    __device__ __forceinline__ void flux_fma(const T u[NV], T ch2, T f[NV]) const
    {
#pragma clang fp contract(off)
        using N = Num<T>;
        const T ir = N::rcp(u[RHO]);
        const T v[3] = {u[MX] * ir, u[MY] * ir, u[MZ] * ir};
        const T B[3] = {u[BX], u[BY], u[BZ]};
        const T bb = dot3<D == 0 ? 0 : 1>(B[0], B[0], B[1], B[1], B[2], B[2]);
        T pr;
        if constexpr (MIXED) {
            using E = Num<double>;
            const double m[3] = {(double)u[MX], (double)u[MY], (double)u[MZ]};
            const double b[3] = {(double)u[BX], (double)u[BY], (double)u[BZ]};
            double r = (double)ir;
            r = r * E::fma_(-(double)u[RHO], r, 2.0);  // one Newton step on 1/rho
            const double m2 = dot3<1>(m[0], m[0], m[1], m[1], m[2], m[2]);
            const double b2 = dot3<1>(b[0], b[0], b[1], b[1], b[2], b[2]);
            pr = (T)(gm1d * E::fma_(-0.5, b2, E::fma_(-0.5 * m2, r, (double)u[EN])));
        } else {
            const T k2 = dot3<1>(u[MX], v[0], u[MY], v[1], u[MZ], v[2]);
            pr = gm1 * N::fma_(T(-0.5), bb, N::fma_(T(-0.5), k2, u[EN]));
        }
        const T pt = N::fma_(T(0.5), bb, pr);
        const T vb = dot3<1>(v[0], B[0], v[1], B[1], v[2], B[2]);
        f[RHO] = u[MX + D];
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const T m = N::fma_(u[MX + j], v[D], -(B[j] * B[D]));
            f[MX + j] = j == D ? m + pt : m;
            f[BX + j] = j == D ? u[PSI] : N::fma_(B[j], v[D], -(B[D] * v[j]));
        }
        f[EN] = N::fma_(u[EN] + pt, v[D], -(B[D] * vb));
        f[PSI] = ch2 * B[D];
    }

    // EGLM flux along D (MHD-1..MHD-5); returns |v_D| + c_f,D if SPEED
    template <int D, bool SPEED>
    __device__ __forceinline__ T flux(const T u[NV], T ch2, T f[NV]) const
    {
        T ir = Num<T>::rcp(u[RHO]);
        T v[3] = {u[MX] * ir, u[MY] * ir, u[MZ] * ir};
        const T B[3] = {u[BX], u[BY], u[BZ]};
        T bb = B[0] * B[0] + B[1] * B[1] + B[2] * B[2];
        T me = T(0.5) * bb;
        T pr = pressure(u, ir, v[0], v[1], v[2], me);
        T pt = pr + me;
        T vd = v[D], Bd = B[D];
        T vb = v[0] * B[0] + v[1] * B[1] + v[2] * B[2];
        f[RHO] = u[MX + D];
#pragma unroll
        for (int j = 0; j < 3; j++)
            f[MX + j] = u[MX + j] * vd - B[j] * Bd;
        f[MX + D] = f[MX + D] + pt;
#pragma unroll
        for (int j = 0; j < 3; j++)
            f[BX + j] = B[j] * vd - Bd * v[j];
        f[BX + D] = u[PSI];
        f[EN] = (u[EN] + pt) * vd - Bd * vb;
        f[PSI] = ch2 * Bd;
        if constexpr (SPEED) {
            T a2 = gamma * pr * ir;
            T b2 = bb * ir;
            T s = a2 + b2;
            T disc = s * s - T(4) * a2 * (Bd * Bd) * ir;
            disc = disc < T(0) ? T(0) : disc;
            T cf2 = T(0.5) * (s + Num<T>::sqrt_(disc));
            cf2 = cf2 < T(0) ? T(0) : cf2;
            return fabs(vd) + Num<T>::sqrt_(cf2);
        } else {
            return T(0);
        }
    }
};

// primitive quantities of one state, computed once and shared by the
// admissibility test, the flux and the fast speed of that state
template <typename T>
struct Prim {
    T ir, vx, vy, vz, bb, p;
};

template <typename T, bool MIXED>
__device__ __forceinline__ void prim_of(const Phys<T, MIXED> &ph, const T u[NV], Prim<T> &w)
{
    w.ir = Num<T>::rcp(u[RHO]);
    w.vx = u[MX] * w.ir;
    w.vy = u[MY] * w.ir;
    w.vz = u[MZ] * w.ir;
    w.bb = u[BX] * u[BX] + u[BY] * u[BY] + u[BZ] * u[BZ];
    w.p = ph.pressure(u, w.ir, w.vx, w.vy, w.vz, T(0.5) * w.bb);
}

template <typename T>
__device__ __forceinline__ bool admissible_w(const T u[NV], const Prim<T> &w)
{
    return u[RHO] > T(0) && w.p > T(0);
}

// EGLM flux along dimension d from a state and its primitives.  d may differ
// between lanes (a wave that serves faces of several orientations); with a
// constant d the selects fold away, so every caller forms the same
// arithmetic and a flux does not depend on which lane evaluated it.
// (VB: the form of v . B, see dot3)
template <int VB = -1, typename T>
__device__ __forceinline__ void flux_sel(const T u[NV], const Prim<T> &w, int d, T ch2, T f[NV])
{
    const T me = T(0.5) * w.bb;
    const T pt = w.p + me;
    const T vd = d == 0 ? w.vx : (d == 1 ? w.vy : w.vz);
    const T Bd = d == 0 ? u[BX] : (d == 1 ? u[BY] : u[BZ]);
    const T vb = dot3<VB>(w.vx, u[BX], w.vy, u[BY], w.vz, u[BZ]);
    f[RHO] = d == 0 ? u[MX] : (d == 1 ? u[MY] : u[MZ]);
    f[MX] = u[MX] * vd - u[BX] * Bd;
    f[MY] = u[MY] * vd - u[BY] * Bd;
    f[MZ] = u[MZ] * vd - u[BZ] * Bd;
    f[MX] = d == 0 ? f[MX] + pt : f[MX];
    f[MY] = d == 1 ? f[MY] + pt : f[MY];
    f[MZ] = d == 2 ? f[MZ] + pt : f[MZ];
    f[BX] = d == 0 ? u[PSI] : u[BX] * vd - Bd * w.vx;
    f[BY] = d == 1 ? u[PSI] : u[BY] * vd - Bd * w.vy;
    f[BZ] = d == 2 ? u[PSI] : u[BZ] * vd - Bd * w.vz;
    f[EN] = (u[EN] + pt) * vd - Bd * vb;
    f[PSI] = ch2 * Bd;
}

template <int D, typename T>
__device__ __forceinline__ void flux_w(const T u[NV], const Prim<T> &w, T ch2, T f[NV])
{
    flux_sel(u, w, D, ch2, f);
}

// fast magnetosonic speed c_f,d from a state and its primitives
template <typename T>
__device__ __forceinline__ T fast_sel(const T u[NV], const Prim<T> &w, int d, T gamma)
{
    const T a2 = gamma * w.p * w.ir;
    const T b2 = w.bb * w.ir;
    const T s = a2 + b2;
    const T Bd = d == 0 ? u[BX] : (d == 1 ? u[BY] : u[BZ]);
    // (comparisons, not maxima: a NaN stays one)
    T disc = s * s - T(4) * a2 * (Bd * Bd) * w.ir;
    disc = disc < T(0) ? T(0) : disc;
    T cf2 = T(0.5) * (s + Num<T>::sqrt_(disc));
    cf2 = cf2 < T(0) ? T(0) : cf2;
    return Num<T>::sqrt_(cf2);
}

// |v_d| + c_f,d from a state and its primitives (d as in flux_sel)
template <typename T>
__device__ __forceinline__ T speed_sel(const T u[NV], const Prim<T> &w, int d, T gamma)
{
    const T vd = d == 0 ? w.vx : (d == 1 ? w.vy : w.vz);
    return fabs(vd) + fast_sel(u, w, d, gamma);
}

template <int D, typename T>
__device__ __forceinline__ T speed_w(const T u[NV], const Prim<T> &w, T gamma)
{
    return speed_sel(u, w, D, gamma);
}

}  // namespace mapk
