// k_step_mmc.hip -- the modified MacCormack block update (paper Sec. 3.1) on
// 2-D blocks: Lax-Friedrichs flux splitting f+- = (f +- alpha u)/2 with the
// global alpha (c_h on the GLM pair), predictor u~ from h = f+_i + f-_{i+1},
// and the flux-limited correction built from g+ and g-, all directions
// together (Sec. 3.7), followed by the same EGLM sources, resistive terms
// and psi damping as the LF update.  (3-D blocks: k_step_mmc3.hip.)
//
// One block at a time per workgroup of eight waves, a thread per cell of the
// padded 20 x 20 tile.  A thread reads its cell where the ghost descriptors
// point (a same-level neighbour's interior in U_in, or the block's own
// prolongated ghosts), so U_out must not alias U_in, keeps it and its fluxes
// of both dimensions in registers, and shares the split fluxes of one
// dimension at a time through LDS.  The next block's cells and records are
// requested during the corrector.
// Bound by FP64 issue on two waves per SIMD (LDS holds one FP64 block per CU)
// and the barriers between the phases: 135 -> 83 us for 2008 FP64 leaves
// (van Leer) against four waves with two cells a thread, which staged the
// tile as well and formed the split fluxes of x twice.
#include <type_traits>

#include "kernels.hpp"
#include "physics.hpp"
#include "sched.hpp"
#include "tile.hpp"

namespace mapk {

namespace {
constexpr int T2 = PD * PD;     // padded cells (400)
constexpr int EW2 = NB + 2;     // E region edge (18)
constexpr int E2 = EW2 * EW2;   // E region (324)
constexpr int F2 = (NB + 1) * NB;        // faces of one dimension (272)
constexpr int NT = 512;
static_assert(T2 <= NT, "a thread per padded cell");

// what the update of a block needs of its records
struct MmcHead {
    int slot, fb[4];
    double dt, ch, alpha, damp, dx[2];
};

__device__ __forceinline__ MmcHead mmc_head(const StepArgs &a, int item)
{
    MmcHead h;
    h.slot = a.leaves[item];
    const BlockRec br = a.blk[h.slot];
    const map_dt &rec = a.dt[br.sim];
    h.dt = rec.dt;
    h.ch = rec.ch;
    h.alpha = rec.alpha;
    h.damp = rec.damp;
    const double *dxp = a.lvl_dx + ((size_t)br.sim * (MAXL + 1) + br.level) * 3;
    h.dx[0] = dxp[0];
    h.dx[1] = dxp[1];
#pragma unroll
    for (int k = 0; k < 4; k++)
        h.fb[k] = a.fbidx[(size_t)h.slot * 6 + k];
    return h;
}
}  // namespace

template <typename T, bool MIXED, int LIM>
__global__ void __launch_bounds__(NT) k_step_mmc2(StepArgs a)
{
    __shared__ T sfp[NV * T2], sfm[NV * T2];  // f+, f- of u along one dimension
    __shared__ T stp[NV * E2], stm[NV * E2];  // f+, f- of u~
    __shared__ T sfh[NV * F2];                // face fluxes
    __shared__ T sb[2][4 * T2];               // B and psi of u, by item parity

    Phys<T, MIXED> ph;
    ph.gamma = (T)a.gamma;
    ph.gm1 = (T)(a.gamma - 1.0);
    ph.gm1d = a.gamma - 1.0;
    const T *Uin = (const T *)a.Uin;
    T *Uout = (T *)a.Uout;
    T *fbuf = (T *)a.fbuf;
    const int t = threadIdx.x;
    const int c = t < T2 ? t : T2 - 1;
    const int x = c % PD - NG, y = c / PD - NG;
    const bool cell = t < T2;
    // cells of E (interior and ring)
    const bool isE = cell && x >= -1 && x <= NB && y >= -1 && y <= NB;
    const bool xin = x >= 0 && x < NB, yin = y >= 0 && y < NB;
    const int e = (y + 1) * EW2 + x + 1;

    // neighbouring blocks on one XCD, so that the ghost cells read from
    // neighbours come from that XCD's L2
    int first, stride, end;
    xcd_range(a.nitems, first, stride, end);
    end = end < a.nleaves ? end : a.nleaves;
    if (first >= end)
        return;
    MmcHead hn = mmc_head(a, first);
    T un[NV];
    if (cell) {
        const T *p = Uin + cell_src<2>(a.desc, hn.slot, x, y, 0);
#pragma unroll
        for (int v = 0; v < NV; v++)
            un[v] = p[v * T2];
    }
    int par = 0;
    for (int item = first; item < end; item += stride, par ^= 1) {
        const MmcHead h = hn;
        T u[NV];
#pragma unroll
        for (int v = 0; v < NV; v++)
            u[v] = un[v];
        T dtdx[2], i2d[2];
        for (int d = 0; d < 2; d++) {
            dtdx[d] = (T)(h.dt / h.dx[d]);
            i2d[d] = (T)(0.5 / h.dx[d]);
        }
        const T dt = (T)h.dt, ch = (T)h.ch, ch2 = (T)(h.ch * h.ch), damp = (T)h.damp;
        const T alpha = (T)h.alpha;
        T *ob = Uout + (size_t)h.slot * NV * T2;
        T *ub = sb[par];

        auto al = [&](int v, int D) { return (v == BX + D || v == PSI) ? ch : alpha; };
        // split fluxes of a state w with the flux F along D into planes of
        // stride n at index i, contractions written out (the flux is hidden
        // from common-subexpression elimination: kept split fluxes would spill)
        auto publish = [&](auto dc, const T (&w)[NV], T (&F)[NV], T *fp, T *fm, int n, int i) {
#pragma clang fp contract(off)
            constexpr int D = decltype(dc)::value;
#pragma unroll
            for (int v = 0; v < PSI; v++) {
                asm volatile("" : "+v"(F[v]));
                fp[v * n + i] = T(0.5) * Num<T>::fma_(al(v, D), w[v], F[v]);
                fm[v * n + i] = T(0.5) * Num<T>::fma_(-al(v, D), w[v], F[v]);
            }
            const T q = ch * w[PSI];
            fp[PSI * n + i] = T(0.5) * Num<T>::fma_(w[BX + D], ch2, q);
            fm[PSI * n + i] = T(0.5) * Num<T>::fma_(w[BX + D], ch2, -q);
        };
        // the predictor term dt/dx_D (h_{i+1/2} - h_{i-1/2}) of the own cell
        auto pred = [&](auto dc, T (&term)[NV]) {
            constexpr int D = decltype(dc)::value;
            constexpr int s = D == 0 ? 1 : PD;
#pragma unroll
            for (int v = 0; v < NV; v++) {
                T hp = sfp[v * T2 + c] + sfm[v * T2 + c + s];
                T hm = sfp[v * T2 + c - s] + sfm[v * T2 + c];
                term[v] = dtdx[D] * (hp - hm);
            }
        };
        // the limited fluxes of the faces along D into sfh and, where a face
        // is shared with another level, the reflux buffer.  No variable needs
        // another, so the work is split by variable and face: 2448 items on
        // eight waves, where a thread per face left the faces past 256 to a
        // fifth wave (and one SIMD with twice the work)
        auto faces = [&](auto dc) {
            constexpr int D = decltype(dc)::value;
            constexpr int s = D == 0 ? 1 : PD, se = D == 0 ? 1 : EW2;
            int t0 = t;
            if constexpr (sizeof(T) == 8)  // the items' indices are not kept over blocks (spills)
                asm volatile("" : "+v"(t0));
#pragma unroll
            for (int j = 0; j < (NV * F2 + NT - 1) / NT; j++) {
                const int k = t0 + j * NT;
                if (k >= NV * F2)
                    break;
                const int v = k / F2, f = k - v * F2;
                const int fx = D == 0 ? f % (NB + 1) - 1 : f % NB;
                const int fy = D == 0 ? f / (NB + 1) : f / NB - 1;
                const int i = (fy + NG) * PD + fx + NG, ie = (fy + 1) * EW2 + fx + 1;
                const T *FP = sfp + v * T2, *FM = sfm + v * T2;
                const T *TP = stp + v * E2, *TM = stm + v * E2;
                T hh = FP[i] + FM[i + s];
                T gp_m = TP[ie] - FP[i - s];
                T gp_p = TP[ie + se] - FP[i];
                T gm_p = FM[i + s] - TM[ie];
                T gm_pp = FM[i + 2 * s] - TM[ie + se];
                const T fh = hh + T(0.5) * (limiter<LIM>(gp_m, gp_p) - limiter<LIM>(gm_pp, gm_p));
                sfh[k] = fh;
                const int cd = D == 0 ? fx : fy;
                if (cd == -1 || cd == NB - 1) {
                    const int fb = cd == -1 ? h.fb[2 * D] : h.fb[2 * D + 1];
                    if (fb >= 0)
                        fbuf[((size_t)fb * NV + v) * NB + (D == 0 ? fy : fx)] = fh;
                }
            }
        };
        // dt/dx_D times the difference of the own cell's faces
        auto diff = [&](auto dc, T (&div)[NV]) {
            constexpr int D = decltype(dc)::value;
            const int f = D == 0 ? y * (NB + 1) + x + 1 : (y + 1) * NB + x;
            constexpr int fs = D == 0 ? 1 : NB;
#pragma unroll
            for (int v = 0; v < NV; v++)
                div[v] = dtdx[D] * (sfh[v * F2 + f] - sfh[v * F2 + f - fs]);
        };
        constexpr std::integral_constant<int, 0> X{};
        constexpr std::integral_constant<int, 1> Y{};

        // ---- split fluxes of u; predictor on E: u~ = u - sum_d dt/dx_d (h_{i+1/2} - h_{i-1/2})
        T Fx[NV], Fy[NV];
        if (cell) {
            ph.template flux_fma<0>(u, ch2, Fx);
            ph.template flux_fma<1>(u, ch2, Fy);
            publish(X, u, Fx, sfp, sfm, T2, c);
#pragma unroll
            for (int k = 0; k < 3; k++)
                ub[k * T2 + c] = u[BX + k];
            ub[3 * T2 + c] = u[PSI];
        }
        __syncthreads();
        T tx[NV];
        if (isE)
            pred(X, tx);
        __syncthreads();
        if (cell)
            publish(Y, u, Fy, sfp, sfm, T2, c);
        // the next block's records
        const int nxt = item + stride < end ? item + stride : item;
        hn = mmc_head(a, nxt);
        __syncthreads();

        // ---- corrector, dimension y first (its split fluxes of u are in LDS)
        T ut[NV], Ft[NV];
        if (isE) {
            T ty[NV], Fty[NV];
            pred(Y, ty);
            {
                // (both terms rounded, whichever phase formed them)
#pragma clang fp contract(off)
#pragma unroll
                for (int v = 0; v < NV; v++)
                    ut[v] = u[v] - (tx[v] + ty[v]);
            }
            ph.template flux_fma<0>(ut, ch2, Ft);
            ph.template flux_fma<1>(ut, ch2, Fty);
            publish(Y, ut, Fty, stp, stm, E2, e);
        }
        if (cell) {
            const T *p = Uin + cell_src<2>(a.desc, hn.slot, x, y, 0);
#pragma unroll
            for (int v = 0; v < NV; v++)
                un[v] = p[v * T2];
        }
        __syncthreads();
        faces(Y);
        __syncthreads();
        T div[2][NV];
        if (xin && yin)
            diff(Y, div[1]);
        if (cell)
            publish(X, u, Fx, sfp, sfm, T2, c);
        if (isE)
            publish(X, ut, Ft, stp, stm, E2, e);
        __syncthreads();
        faces(X);
        __syncthreads();

        // ---- update, EGLM sources from u^n, psi damping
        if (cell && xin && yin) {
            diff(X, div[0]);
            T o[NV];
#pragma unroll
            for (int v = 0; v < NV; v++)
                o[v] = u[v] - (div[0][v] + div[1][v]);
            const T *bx = ub, *by = ub + T2, *bz = ub + 2 * T2, *ps = ub + 3 * T2;
            if (a.eglm) {
                T divb = (bx[c + 1] - bx[c - 1]) * i2d[0];
                divb += (by[c + PD] - by[c - PD]) * i2d[1];
                T bgp = u[BX] * ((ps[c + 1] - ps[c - 1]) * i2d[0]);
                bgp += u[BY] * ((ps[c + PD] - ps[c - PD]) * i2d[1]);
                o[MX] = o[MX] - dt * (divb * u[BX]);
                o[MY] = o[MY] - dt * (divb * u[BY]);
                o[MZ] = o[MZ] - dt * (divb * u[BZ]);
                o[EN] = o[EN] - dt * bgp;
            }
            // resistive terms -curl(eta J) and -div((eta J) x B) (Sec. 3.5)
            // from central differences of u^n; in 2-D the z derivatives vanish
            if (a.eta > 0.0) {
                const T eta = (T)a.eta;
                // eta J and the x, y rows of eta (J x B) at padded index i
                auto ej = [&](int i, T (&r)[5]) {
                    const T jx = (bz[i + PD] - bz[i - PD]) * i2d[1];
                    const T jy = -((bz[i + 1] - bz[i - 1]) * i2d[0]);
                    const T jz = (by[i + 1] - by[i - 1]) * i2d[0] - (bx[i + PD] - bx[i - PD]) * i2d[1];
                    r[0] = eta * jx;
                    r[1] = eta * jy;
                    r[2] = eta * jz;
                    r[3] = eta * (jz * by[i] - jy * bz[i]);
                    r[4] = eta * (jx * bz[i] - jz * bx[i]);
                };
                T xm[5], xp[5], ym[5], yp[5];
                ej(c - 1, xm);
                ej(c + 1, xp);
                ej(c - PD, ym);
                ej(c + PD, yp);
                o[BX] = o[BX] + dt * (-((yp[2] - ym[2]) * i2d[1]));
                o[BY] = o[BY] + dt * ((xp[2] - xm[2]) * i2d[0]);
                o[BZ] = o[BZ] + dt * ((yp[0] - ym[0]) * i2d[1] - (xp[1] - xm[1]) * i2d[0]);
                o[EN] = o[EN] + dt * ((xp[3] - xm[3]) * i2d[0] + (yp[4] - ym[4]) * i2d[1]);
            }
            o[PSI] = o[PSI] * damp;
#pragma unroll
            for (int v = 0; v < NV; v++)
                ob[v * T2 + c] = o[v];
        }
        // (the next block's first phase writes f+-, last read before the last
        // barrier, and the other B plane; its faces come three barriers later)
    }
}

template <typename T, bool MIXED, int LIM>
static void launch_mmc(const StepArgs &a, int g, hipStream_t s)
{
    hipLaunchKernelGGL((k_step_mmc2<T, MIXED, LIM>), dim3(g), dim3(NT), 0, s, a);
}

template <typename T, bool MIXED>
static void launch_mmc_lim(const StepArgs &a, int g, hipStream_t s)
{
    if (a.limiter == MAP_MINMOD)
        launch_mmc<T, MIXED, MAP_MINMOD>(a, g, s);
    else if (a.limiter == MAP_VANLEER)
        launch_mmc<T, MIXED, MAP_VANLEER>(a, g, s);
    else
        launch_mmc<T, MIXED, MAP_PAPER_PHI>(a, g, s);
}

hipError_t launch_step_mmc(int ndim, bool fp64, const StepArgs &a, double, int grid, hipStream_t s)
{
    if (ndim == 3)
        return launch_step_mmc3(fp64, a.eta > 0.0, a, grid, s);
    if (a.nitems <= 0)
        return hipSuccess;
    // as many workgroups as LDS lets run: each prefetches its next block
    const int want = grid > 0 ? grid : (fp64 ? 1 : 2) * a.ncu;
    const int g = want < a.nitems ? want : a.nitems;
    if (fp64)
        launch_mmc_lim<double, false>(a, g, s);
    else
        launch_mmc_lim<float, true>(a, g, s);
    return hipGetLastError();
}

}  // namespace mapk
