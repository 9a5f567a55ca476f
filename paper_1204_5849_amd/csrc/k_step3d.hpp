// k_step3d.hpp -- the FP32 block update of 3-D leaf blocks, the three
// dimensions of a cell on three threads: the TVD-LF step (paper Sec. 3.2) or
// one stage of WENO with TVD Runge-Kutta 2 (Sec. 3.3), with the EGLM source
// terms (Sec. 2), uniform resistivity (Sec. 3.5) and exact psi damping.
//
// Schedule (gfx950): one block per workgroup of 15 waves, one workgroup per CU
// (LDS: LF 128.6 KB, WENO 122.2 KB, 8 KB more with resistivity), marching along
// z one plane per iteration.  Waves 0-3, 4-7 and 8-11 own the 16 x 16 columns
// for x, y and z; waves 12-14 own the ring of 64 cells just outside the
// interior for the same three dimensions.  A thread forms
// its cell's slope, half-step flux pair, face states and face flux along its
// own dimension only, so it keeps to 128 registers and each SIMD has four
// waves to issue from (an FP32 add, multiply or FMA issues every 2 cycles from
// two or more waves and every 4 from one).
//
// Per plane k, three barriers (WENO, whose face states need no exchange and
// whose face buffers alternate, two):
//   P1  slopes and the half-step flux difference along the own dimension into
//       LDS (WENO: the face states); EGLM sources and eta J (x, y)        B1
//   P2  u~ from the three differences, the two face states of the own
//       dimension; x and y publish the right state                        B2
//   P3  the face flux of the own dimension: x+1/2, y+1/2 (over the right
//       state it was formed from, whose only reader is that lane), z-1/2;
//       ring waves the faces -1/2; plane k+2 into LDS                     B3
//   P4  x threads update rho, m and B_x, y threads the other variables: the
//       z difference finishes plane k-1, the in-plane ones start plane k.
// Three planes of state stay in LDS, so that no thread carries neighbours in
// registers.
//
// What bounds it: issue on the three SIMDs that hold a ring wave, and the
// waits at the barriers (19328 leaves, LF: waves wait 0.50 of their time; LDS
// bank conflicts, 8 times more with a wave on four adjacent rows, take 0.03 of
// the LDS cycles).  Against one thread per column for all dimensions (two
// 4-wave workgroups per CU, 256 registers, 44 to 180 bytes of them in scratch),
// per map_step at the default step_shape 0: the Harris sheet's 4768 leaves, LF
// 1489 -> 1385 us, LF with HLLC 1686 -> 1442, WENO 4744 -> 3571, WENO with HLLC
// 5148 -> 3898 (both stages with the fill between); the blast's 1464 leaves,
// without resistivity and spills, 429 -> 418 (416 at the priorities of shape
// 1).  Every sum and contraction is the one-thread version's, so that the state
// and the FP64 time steps taken from it keep their bits: scaling the half-step
// differences and sources before they meet was 1 % faster, the face states of
// WENO from differences (u0 + d/2) 7 %, but both moved the time steps, by up to
// 1e-7.
// The waves of one role run their own loop; every wave passes the same
// barriers.  Ghost cells are read where the ghost descriptors point (Sec.
// 4.3), so U_out must not alias U_in (WENO stage 2 reads U_base at the cells
// it writes).  Each face flux is evaluated once and differences are formed
// explicitly, so a uniform state stays exactly uniform (WENO: as far as the
// products 3 u0 that weno_pair_fma rounds first are exact).
#pragma once

#include <type_traits>

#include "kernels.hpp"
#include "physics.hpp"
#include "step_common.hpp"
#include "sched.hpp"
#include "tile.hpp"

namespace mapk {

namespace {
constexpr int NTD = 15 * 64;               // threads
constexpr int XSD = PD * PD;               // plane of a padded tile
constexpr int PTD = XSD * PD;              // padded tile
constexpr int NCD = NB * NB;               // columns
constexpr int NRD = 4 * NB;                // ring cells of a plane
constexpr int NCELLD = NCD + NRD;          // cells with a predictor
constexpr int NOD = 4 * PD;                // outer ring cells and ring corners (load only)
constexpr int OPWD = NOD / 2;              // of them per x or y ring wave
constexpr int NLDD = NRD + NOD;            // cells loaded one by one
static_assert(NB == 16 && OPWD <= 64, "lane layout assumes 16^3 blocks");

// outer cell c of a plane: the outermost rows and columns, then the corners
// of the ring
__device__ __forceinline__ void outer_xy(int c, int &x, int &y)
{
    if (c < 2 * PD) {
        x = c % PD - NG;
        y = c < PD ? -NG : NB + 1;
    } else if (c < 2 * PD + 2 * (NB + 2)) {
        const int r = c - 2 * PD;
        x = r < NB + 2 ? -NG : NB + 1;
        y = r % (NB + 2) - 1;
    } else {
        const int r = c - 2 * PD - 2 * (NB + 2);
        x = (r & 1) ? NB : -1;
        y = (r & 2) ? NB : -1;
    }
}

// a value that is the same in every lane, moved to a scalar register
__device__ __forceinline__ float uni(float x)
{
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}
}  // namespace

template <typename T, bool RESIST, bool PREDICT>
struct Shared3d {
    T su[3][NV * XSD];                          // state of planes k-1, k, k+1 (by plane mod 3)
    // right face states along x and y, then fluxes, and the states' pressures
    // (WENO: by plane parity)
    T srf[PREDICT ? 1 : 2][2][NV * XSD];
    T spr[PREDICT ? 1 : 2][2][XSD];
    T sac[PREDICT ? 3 : 1][PREDICT ? NV * NCELLD : 1];  // half-step differences per dimension
    int sok[PREDICT ? 3 : 1][PREDICT ? NCELLD : 1];     // whether the face states are admissible
    T sfz[NV * NCD];                            // z face fluxes
    T sj[RESIST ? 5 * XSD : 1];                 // eta J and eta (J x B)
    size_t gld[5 * NLDD];                       // ring and outer cells: offset per plane region
};

// (SHAPE does not change it, but gives each kernel a copy of its own to
// inline: one shared by two kernels spilled 36 registers instead of 10)
template <typename T, bool MIXED, bool RESIST, int SCH, int LIM, int RS, int SHAPE>
struct March3d {
    static constexpr bool PREDICT = SCH == SCH_LF;
    using Sh = Shared3d<T, RESIST, PREDICT>;

    // flux of a face along D.  The contractions that the compiler chooses
    // differently for otherwise equal callers are written out: B . B, v . B and
    // the sum of the two psi fluxes ch2 B_D
    template <int D, bool RING>
    static __device__ __forceinline__ void face(const T L[NV], T pL, const T R[NV], T pR, T gam, T gm1,
                                                T ch, T ch2, T f[NV])
    {
        constexpr int BB = D == 0 && (RS == MAP_HLLC || !RING) ? 0 : 1;
        constexpr int VL = D == 1 && RS == MAP_HLLC ? 0 : 1;
        constexpr int VR = RS == MAP_HLLC && !PREDICT && !RING && D < 2 ? 1 - VL : VL;
        face_flux<RS, D, BB, VL, VR>(L, pL, R, pR, gam, gm1, ch, ch2, f);
        if constexpr (RS == MAP_RUSANOV) {
#pragma clang fp contract(off)
            const T bl = L[BX + D], br = R[BX + D];
            const T s = D == 2 ? Num<T>::fma_(bl, ch2, br * ch2) : Num<T>::fma_(br, ch2, bl * ch2);
            f[PSI] = Num<T>::fma_(T(0.5), s, -(T(0.5) * ch * (R[PSI] - L[PSI])));
        }
    }

    // one role of the march over one block: dimension D, interior columns or
    // the ring cells
    template <int D, bool RING>
    static __device__ __forceinline__ void run(const StepArgs &a, Sh &sh, const int slot, int t)
    {
        // opaque, so that no role's addresses are kept in registers across
        // the work items of another
        asm volatile("" : "+v"(t));
        constexpr int FC = NB * NB;
        constexpr int ST = D == 0 ? 1 : PD;  // in-plane stride of this dimension
        const int ln = t & 63;
        // interior column: the four rows of a wave lie four apart, so that
        // their 16 cells fall into different LDS banks (rows of 20 words)
        const int col = t & (NCD - 1);
        const int cx = col % NB, cy = (col >> 6) + 4 * ((col >> 4) & 3);
        const int sd = ln >> 4, rix = ln & 15;  // ring side and position
        const int qx = RING ? (sd == 0 ? -1 : (sd == 1 ? NB : rix)) : cx;
        const int qy = RING ? (sd == 2 ? -1 : (sd == 3 ? NB : rix)) : cy;
        const int q = (qy + NG) * PD + qx + NG;
        const int cell = RING ? NCD + ln : col;
        // whether the interior reads this cell's face state along D, and for
        // ring cells which one: at -1 the left state of the face -1/2
        const bool rface = !RING || (D < 2 && (sd >> 1) == D);
        const bool rlo = (sd & 1) == 0;

        Phys<T, MIXED> ph;
        ph.gamma = (T)a.gamma;
        ph.gm1 = (T)(a.gamma - 1.0);
        ph.gm1d = a.gamma - 1.0;
        const T gam = ph.gamma, gm1 = ph.gm1;
        const T *Uin = (const T *)a.Uin;
        T *fbuf = (T *)a.fbuf;
        auto put_flux = [&](size_t i, T f) {
            if constexpr (SCH == SCH_WENO2)
                fbuf[i] = T(0.5) * fbuf[i] + T(0.5) * f;
            else
                fbuf[i] = f;
        };
        const BlockRec br = a.blk[slot];
        const map_dt rec = a.dt[br.sim];
        const double *dxp = a.lvl_dx + ((size_t)br.sim * (MAXL + 1) + br.level) * 3;
        const T dt = uni((T)rec.dt), ch = uni((T)rec.ch), ch2 = uni((T)(rec.ch * rec.ch));
        const T rx = uni((T)(rec.dt / dxp[0])), ry = uni((T)(rec.dt / dxp[1])),
                rz = uni((T)(rec.dt / dxp[2]));
        const T ix = uni((T)(0.5 / dxp[0])), iy = uni((T)(0.5 / dxp[1])), iz = uni((T)(0.5 / dxp[2]));

        // who loads what: z interior threads their column (the z neighbours'
        // interiors or the block's own ghosts, uniform bases), the z ring
        // wave the ring cells, the x and y ring waves the outer cells
        constexpr bool COL = D == 2 && !RING;
        const bool ldr = RING && (D == 2 || ln < OPWD);
        const T *zb[COL ? 5 : 1] = {};
        int li = ln, oq = q;
        {
            const int zr[5] = {-2, -1, 0, NB, NB + 1};
            if constexpr (COL) {
#pragma unroll
                for (int r = 0; r < 5; r++)
                    zb[r] = Uin + cell_src<3>(a.desc, slot, 0, 0, zr[r]) - (NG * PD + NG);
            } else if constexpr (RING) {
                int ex = qx, ey = qy;
                if constexpr (D < 2) {
                    const int c = D * OPWD + (ln < OPWD ? ln : 0);
                    outer_xy(c, ex, ey);
                    oq = (ey + NG) * PD + ex + NG;
                    li = NRD + c;
                }
                if (ldr)
#pragma unroll
                    for (int r = 0; r < 5; r++)
                        sh.gld[r * NLDD + li] = cell_src<3>(a.desc, slot, ex, ey, zr[r]);
            }
        }
        auto load = [&](T(&dst)[NV], int k) {
            const T *p;
            if constexpr (COL)
                p = (k == -2 ? zb[0]
                             : (k == -1 ? zb[1] : (k < NB ? zb[2] + k * XSD : (k == NB ? zb[3] : zb[4])))) +
                    q;
            else
                p = Uin + (k < 0 ? sh.gld[(k + 2) * NLDD + li]
                                 : (k < NB ? sh.gld[2 * NLDD + li] + (size_t)k * XSD
                                           : sh.gld[(k - NB + 3) * NLDD + li]));
#pragma unroll
            for (int v = 0; v < NV; v++)
                dst[v] = p[v * PTD];
        };
        auto plane = [&](int k) { return &sh.su[(k + 3) % 3][0]; };
        auto put = [&](int k, const T(&u)[NV]) {
            T *s = plane(k);
#pragma unroll
            for (int v = 0; v < NV; v++)
                s[v * XSD + oq] = u[v];
        };

        // planes -2 (columns only), -1 and 0 in LDS, plane 1 in flight; the
        // last planes read are NB + 1 of the columns and NB of the ring
        constexpr int KL = COL ? NB + 1 : NB;
        T un[NV];
        if (COL || ldr) {
            T u2[NV], u1[NV], u0[NV];  // all in flight together
            if constexpr (COL)
                load(u2, -2);
            load(u1, -1);
            load(u0, 0);
            load(un, 1);
            if constexpr (COL)
                put(-2, u2);
            put(-1, u1);
            put(0, u0);
        }
        __syncthreads();

        // x: variables rho .. B_x, y: B_y .. psi
        constexpr int V0 = D == 0 ? 0 : 5, V1 = D == 0 ? 5 : NV;
        constexpr bool FIN = D < 2 && !RING;     // finalises
        T Wc[FIN ? NV : 1], fzp[FIN ? NV : 1];   // started plane, z flux below it
        T Lp[COL ? NV : 1], pLp = T(1);          // left state of the face below
        T ja[3] = {T(0), T(0), T(0)}, jb[3] = {T(0), T(0), T(0)};  // eta J of planes k-1, k-2
#pragma unroll
        for (int v = 0; v < NV; v++) {
            if constexpr (FIN) {
                Wc[v] = T(0);
                fzp[v] = T(0);
            }
            if constexpr (COL)
                Lp[v] = T(0);
        }
        T *ob = (T *)a.Uout + (size_t)slot * NV * PTD;

        for (int k = -1; k <= NB; ++k) {
            const bool kI = k >= 0 && k < NB;
            auto &srf = sh.srf[PREDICT ? 0 : k & 1];
            auto &spr = sh.spr[PREDICT ? 0 : k & 1];
            const T *const sc = plane(k), *const sm = plane(k - 1), *const sn = plane(k + 1);
            // the cells at work in this plane: rows -1 and NB only feed the
            // faces between planes (interior columns)
            const bool on = kI || !RING;

            // ---- P1
            T uc[NV], dl[NV], acc[NV];
            T L[NV], R[NV];
            bool ok = true;
            T src[3] = {T(0), T(0), T(0)};  // EGLM source terms: m (x threads), e (y)
            T jc[3] = {T(0), T(0), T(0)};
            if (on) {
                const T *const pa = D == 2 ? sm + q : sc + q - ST, *const pb = D == 2 ? sn + q : sc + q + ST;
                T a_[NV], b_[NV];
#pragma unroll
                for (int v = 0; v < NV; v++) {
                    uc[v] = sc[v * XSD + q];
                    a_[v] = pa[v * XSD];
                    b_[v] = pb[v * XSD];
                }
                if constexpr (PREDICT) {
                    // slopes (limiter1) and the half-step flux difference
#pragma unroll
                    for (int v = 0; v < NV; v++)
                        dl[v] = limiter<LIM>(uc[v] - a_[v], b_[v] - uc[v]);
                    T s1[NV], f1[NV], f2[NV];
                    Prim<T> w;
#pragma unroll
                    for (int v = 0; v < NV; v++)
                        s1[v] = uc[v] + T(0.5) * dl[v];
                    prim_of(ph, s1, w);
                    ok = admissible_w(s1, w);
                    flux_w<D>(s1, w, ch2, f1);
#pragma unroll
                    for (int v = 0; v < NV; v++)
                        s1[v] = uc[v] - T(0.5) * dl[v];
                    prim_of(ph, s1, w);
                    ok = ok && admissible_w(s1, w);
                    flux_w<D>(s1, w, ch2, f2);
#pragma unroll
                    for (int v = 0; v < NV; v++) {
                        acc[v] = f1[v] - f2[v];
                        sh.sac[D][v * NCELLD + cell] = acc[v];
                    }
                    sh.sok[D][cell] = ok;
                } else if (D == 2 ? !RING : (kI && rface)) {
#pragma unroll
                    for (int v = 0; v < NV; v++)
                        weno_pair_fma<RING || D == 0, RING>(a_[v], uc[v], b_[v], L[v], R[v]);
                }
                // EGLM sources from central differences of u^n
                if (FIN && kI && a.eglm) {
                    if constexpr (D == 0) {
                        const T *bx = sc + BX * XSD + q, *by = sc + BY * XSD + q;
                        T divb = (bx[1] - bx[-1]) * ix;
                        divb += (by[PD] - by[-PD]) * iy;
                        divb += (sn[BZ * XSD + q] - sm[BZ * XSD + q]) * iz;
#pragma unroll
                        for (int i = 0; i < 3; i++)
                            src[i] = divb * uc[BX + i];
                    } else {
                        const T *ps = sc + PSI * XSD + q;
                        T bgp = uc[BX] * ((ps[1] - ps[-1]) * ix);
                        bgp += uc[BY] * ((ps[PD] - ps[-PD]) * iy);
                        bgp += uc[BZ] * ((sn[PSI * XSD + q] - sm[PSI * XSD + q]) * iz);
                        src[0] = bgp;
                    }
                }
                // eta J and eta (J x B), by the y waves
                if constexpr (RESIST && D == 1) {
                    const T eta = uni((T)a.eta);
                    const T *bx = sc + BX * XSD + q, *by = sc + BY * XSD + q, *bz = sc + BZ * XSD + q;
                    const T dyBz = (bz[PD] - bz[-PD]) * iy;
                    const T dzBy = (sn[BY * XSD + q] - sm[BY * XSD + q]) * iz;
                    const T dzBx = (sn[BX * XSD + q] - sm[BX * XSD + q]) * iz;
                    const T dxBz = (bz[1] - bz[-1]) * ix;
                    const T dxBy = (by[1] - by[-1]) * ix;
                    const T dyBx = (bx[PD] - bx[-PD]) * iy;
                    const T jx = dyBz - dzBy, jy = dzBx - dxBz, jz = dxBy - dyBx;
                    sh.sj[0 * XSD + q] = eta * jx;
                    sh.sj[1 * XSD + q] = eta * jy;
                    sh.sj[2 * XSD + q] = eta * jz;
                    sh.sj[3 * XSD + q] = eta * (jz * uc[BY] - jy * uc[BZ]);
                    sh.sj[4 * XSD + q] = eta * (jx * uc[BZ] - jz * uc[BX]);
                    jc[0] = eta * jx;
                    jc[2] = eta * (jy * uc[BX] - jx * uc[BY]);
                }
            }
            if constexpr (PREDICT)
                __syncthreads();  // (B1)

            // ---- P2
            T pL = T(1), pR = T(1);
            if (D == 2 ? !RING : (kI && rface)) {
                T ut[NV];  // u~, or for WENO u: the state that replaces inadmissible ones
                if constexpr (PREDICT) {
                    constexpr int E0 = D == 0 ? 1 : 0, E1 = D == 2 ? 1 : 2;
                    const bool okc = ok && sh.sok[E0][cell] && sh.sok[E1][cell];
#pragma unroll
                    for (int v = 0; v < NV; v++) {
                        const T x = D == 0 ? acc[v] : sh.sac[0][v * NCELLD + cell];
                        const T y = D == 1 ? acc[v] : sh.sac[1][v * NCELLD + cell];
                        const T z = D == 2 ? acc[v] : sh.sac[2][v * NCELLD + cell];
                        ut[v] = uc[v] - Num<T>::fma_(T(0.5) * rz, z,
                                                     Num<T>::fma_(T(0.5) * ry, y, T(0.5) * rx * x));
                    }
                    if (!okc) {
#pragma unroll
                        for (int v = 0; v < NV; v++) {
                            dl[v] = T(0);
                            ut[v] = uc[v];
                        }
                        // once per cell: interior columns by z, ring cells by
                        // the dimension that uses them
                        if (D == 2 || RING)
                            atomicAdd(&a.cnt[0], 1ull);
                    }
#pragma unroll
                    for (int v = 0; v < NV; v++) {
                        L[v] = ut[v] + T(0.5) * dl[v];
                        R[v] = ut[v] - T(0.5) * dl[v];
                    }
                } else {
#pragma unroll
                    for (int v = 0; v < NV; v++)
                        ut[v] = uc[v];
                }
                Prim<T> w;
                if (!RING || rlo) {
                    prim_of(ph, L, w);
                    if (!admissible_w(L, w)) {
#pragma unroll
                        for (int v = 0; v < NV; v++)
                            L[v] = ut[v];
                        prim_of(ph, L, w);
                        if (D < 2 || k < NB)
                            atomicAdd(&a.cnt[1], 1ull);
                    }
                    pL = w.p;
                }
                if (!RING || !rlo) {
                    prim_of(ph, R, w);
                    if (!admissible_w(R, w)) {
#pragma unroll
                        for (int v = 0; v < NV; v++)
                            R[v] = ut[v];
                        prim_of(ph, R, w);
                        if (D < 2 || k >= 0)
                            atomicAdd(&a.cnt[1], 1ull);
                    }
                    pR = w.p;
                    if constexpr (D < 2) {
#pragma unroll
                        for (int v = 0; v < NV; v++)
                            srf[D][v * XSD + q] = R[v];
                        spr[D][q] = pR;
                    }
                }
            }
            __syncthreads();  // (B2)

            // ---- P3
            // plane k+2 over plane k-1, whose readers are behind the barrier
            if (k + 2 <= KL && (COL || ldr)) {
                put(k + 2, un);
                if (k + 3 <= KL)
                    load(un, k + 3);
            }
            // WENO stage 2: u of the cell finished in this plane
            T ub[FIN && SCH == SCH_WENO2 ? NV : 1];
            if constexpr (FIN && SCH == SCH_WENO2) {
                if (k >= 1) {
                    const T *b = (const T *)a.Ubase + (size_t)slot * NV * PTD + (k - 1 + NG) * XSD + q;
#pragma unroll
                    for (int v = V0; v < V1; v++)
                        ub[v] = b[v * PTD];
                }
            }
            T f[NV];
            if constexpr (D < 2) {
                if (kI && rface && (!RING || rlo)) {
#pragma unroll
                    for (int v = 0; v < NV; v++)
                        R[v] = srf[D][v * XSD + q + ST];
                    face<D, RING>(L, pL, R, spr[D][q + ST], gam, gm1, ch, ch2, f);
#pragma unroll
                    for (int v = 0; v < NV; v++)
                        srf[D][v * XSD + q + ST] = f[v];
                    // faces of the block shared with another level (reflux)
                    const int e = D == 0 ? qx : qy;
                    if (RING || e == NB - 1) {
                        const int fb = a.fbidx[(size_t)slot * 6 + 2 * D + (RING ? 0 : 1)];
                        if (fb >= 0) {
                            const int tt = (D == 0 ? qy : qx) + NB * k;
#pragma unroll
                            for (int v = 0; v < NV; v++)
                                put_flux(((size_t)fb * NV + v) * FC + tt, f[v]);
                        }
                    }
                }
            } else if constexpr (COL) {
                if (k >= 0) {
                    face<2, false>(Lp, pLp, R, pR, gam, gm1, ch, ch2, f);
#pragma unroll
                    for (int v = 0; v < NV; v++)
                        sh.sfz[v * NCD + col] = f[v];
                    if (k == 0 || k == NB) {
                        const int fb = a.fbidx[(size_t)slot * 6 + 4 + (k == NB ? 1 : 0)];
                        if (fb >= 0) {
#pragma unroll
                            for (int v = 0; v < NV; v++)
                                put_flux(((size_t)fb * NV + v) * FC + qx + NB * qy, f[v]);
                        }
                    }
                }
#pragma unroll
                for (int v = 0; v < NV; v++)
                    Lp[v] = L[v];
                pLp = pL;
            }
            // in-plane resistive terms x dt: B_x (x threads); B_y, B_z, e (y)
            T rin[3] = {T(0), T(0), T(0)};
            if constexpr (RESIST && FIN) {
                const T *J0 = sh.sj + q, *J1 = J0 + XSD, *J2 = J0 + 2 * XSD, *Q0 = J0 + 3 * XSD,
                        *Q1 = J0 + 4 * XSD;
                if (kI) {
                    if constexpr (D == 0) {
                        rin[0] = -((J2[PD] - J2[-PD]) * iy);
                    } else {
                        rin[0] = (J2[1] - J2[-1]) * ix;
                        rin[1] = (J0[PD] - J0[-PD]) * iy - (J1[1] - J1[-1]) * ix;
                        rin[2] = (Q0[1] - Q0[-1]) * ix + (Q1[PD] - Q1[-PD]) * iy;
                    }
                }
                if constexpr (D == 0)
                    jc[1] = J1[0];
            }
            __syncthreads();  // (B3)

            // ---- P4
            if constexpr (FIN) {
                if (k >= 0) {
                    T fz[NV];
#pragma unroll
                    for (int v = V0; v < V1; v++)
                        fz[v] = sh.sfz[v * NCD + col];
                    if (k >= 1) {
                        T o[NV];
#pragma unroll
                        for (int v = V0; v < V1; v++)
                            o[v] = Wc[v] - rz * (fz[v] - fzp[v]);
                        if constexpr (RESIST) {
                            // (eta J is rounded before the difference, on the
                            // x threads, which read it, as on the y threads,
                            // which formed it)
#pragma clang fp contract(off)
                            if constexpr (D == 0) {
                                o[BX] = Num<T>::fma_((jc[1] - jb[1]) * iz, dt, o[BX]);
                            } else {
                                o[BY] = Num<T>::fma_(-((jc[0] - jb[0]) * iz), dt, o[BY]);
                                o[EN] = Num<T>::fma_((jc[2] - jb[2]) * iz, dt, o[EN]);
                            }
                        }
#pragma unroll
                        for (int v = V0; v < V1; v++) {
                            if constexpr (SCH == SCH_WENO2)
                                o[v] = T(0.5) * (ub[v] + o[v]);
                            if (SCH != SCH_WENO1 && v == PSI)
                                o[v] = o[v] * uni((T)rec.damp);
                            ob[v * PTD + (k - 1 + NG) * XSD + q] = o[v];
                        }
                    }
                    if (kI) {
#pragma unroll
                        for (int v = V0; v < V1; v++) {
                            const T x1 = D == 0 ? f[v] : srf[0][v * XSD + q + 1];
                            const T y1 = D == 1 ? f[v] : srf[1][v * XSD + q + PD];
                            T d = rx * (x1 - srf[0][v * XSD + q]);
                            d += ry * (y1 - srf[1][v * XSD + q]);
                            Wc[v] = uc[v] - d;
                            fzp[v] = fz[v];
                        }
                        if constexpr (D == 0) {
                            Wc[MX] = Wc[MX] - dt * src[0];
                            Wc[MY] = Wc[MY] - dt * src[1];
                            Wc[MZ] = Wc[MZ] - dt * src[2];
                            if constexpr (RESIST)
                                Wc[BX] = Wc[BX] + dt * rin[0];
                        } else {
                            Wc[EN] = Wc[EN] - dt * src[0];
                            if constexpr (RESIST) {
                                Wc[BY] = Wc[BY] + dt * rin[0];
                                Wc[BZ] = Wc[BZ] + dt * rin[1];
                                Wc[EN] = Wc[EN] + dt * rin[2];
                            }
                        }
                    }
                }
                if constexpr (RESIST) {
#pragma unroll
                    for (int i = 0; i < 3; i++) {
                        jb[i] = ja[i];
                        ja[i] = jc[i];
                    }
                }
            }
        }
        __syncthreads();  // LDS reuse by the next work item
    }
};

}  // namespace mapk
