// k_regrid.hip -- device side of a regrid (paper Sec. 4.5): the error
// estimator per block, and the copy of surviving blocks onto a new tree.
#include "fp64.hpp"
#include "kernels.hpp"
#include "sched.hpp"
#include "tile.hpp"

#pragma clang fp contract(off)

namespace mapk {

namespace {
constexpr int NTE = 256;
constexpr int NTE3 = 448;  // 3-D estimator: seven waves, one lane per cell of a padded plane
}  // namespace

// a criterion's value from the variables it reads, in FP64
template <typename T>
__device__ __forceinline__ double est_form(const EstArgs &a, int i, const T (&r)[3])
{
    if (a.est.mode[i] == MAP_EST_BMAG) {
        const double bx = (double)r[0], by = (double)r[1], bz = (double)r[2];
        return sqrt64(bx * bx + by * by + bz * bz);
    }
    return (double)r[0];
}

// the variables criterion i reads of the cell at element offset o
template <int NDIM, typename T>
__device__ __forceinline__ void est_load(const EstArgs &a, int i, size_t o, T (&r)[3])
{
    constexpr int P = tile_cells<NDIM>();
    const T *p = (const T *)a.U + o;
    if (a.est.mode[i] == MAP_EST_BMAG) {
        r[0] = p[BX * P];
        r[1] = p[BY * P];
        r[2] = p[BZ * P];
    } else {
        r[0] = p[(size_t)a.est.var[i] * P];
    }
}

// the estimate of one cell from its value v and the sums over dimensions of
// the squared first and second differences
__device__ __forceinline__ double est_cell(const EstArgs &a, int i, double v, double s1, double s2,
                                           double scale)
{
    const double d1 = 0.5 * sqrt(3.0) * sqrt64(s1);
    const double d2 = sqrt64(s2);
    const double av = fabs(v) + a.est.eps[i];
    // (eps may be 0 and the value tiny: IEEE division, which gives infinity where
    // the quotient overflows)
    return (a.est.bias * d1 / av + (1.0 - a.est.bias) * d2 / (d1 + a.est.filt * av)) * scale;
}

// the largest `best` of the workgroup's threads
template <int NT>
__device__ __forceinline__ double est_max(double best, double (&red)[NT / 64])
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double o = __shfl_xor(best, off, 64);
        best = o > best ? o : best;
    }
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = best;
    __syncthreads();
    double r = red[0];
    for (int w = 1; w < NT / 64; w++)
        r = red[w] > r ? red[w] : r;
    return r;
}

// largest estimate over the interior and the first ghost ring of each block,
// maximum over the criteria; one workgroup per block.  2-D: each criterion's
// value is formed once per padded cell (ghosts read where the descriptors
// point) and staged in LDS; the stencil then runs on LDS.
template <typename T>
__global__ void __launch_bounds__(NTE) k_estimate2(EstArgs a)
{
    constexpr int PT = tile_cells<2>(), E = NB + 2;
    __shared__ double sv[PT];
    __shared__ double red[NTE / 64];
    for (int slot = blockIdx.x; slot < a.nslots; slot += gridDim.x) {
        const int level = a.blk[slot].level;
        const double scale = pow(a.est.ratio, a.est.xi * (level - 1));
        double best = 0.0;
        for (int i = 0; i < a.est.ncrit; i++) {
            for (int c = threadIdx.x; c < PT; c += NTE) {
                T r[3];
                est_load<2, T>(a, i, cell_src<2>(a.desc, slot, c % PD - NG, c / PD - NG, 0), r);
                sv[c] = est_form(a, i, r);
            }
            __syncthreads();
            for (int e = threadIdx.x; e < E * E; e += NTE) {
                const int c = lin<2>(e % E - 1, e / E - 1, 0);
                const double v = sv[c];
                double s1 = 0.0, s2 = 0.0;
#pragma unroll
                for (int d = 0; d < 2; d++) {
                    const int st = d == 0 ? 1 : PD;
                    const double vp = sv[c + st], vm = sv[c - st];
                    s1 += (vp - vm) * (vp - vm);
                    s2 += (vp - 2.0 * v + vm) * (vp - 2.0 * v + vm);
                }
                const double est = est_cell(a, i, v, s1, s2, scale);
                best = est > best ? est : best;
            }
            __syncthreads();  // sv is restaged for the next criterion / block
        }
        const double r = est_max<NTE>(best, red);
        if (threadIdx.x == 0)
            a.err[slot] = r;
        __syncthreads();
    }
}

// 3-D: a march along z with a window of four planes in LDS for all criteria
// at once (NC of them).  Each lane loads the cells of one in-plane position
// through five source offsets formed once per block (below, inside and above
// it), one plane ahead, so a block is read once and the cells cost no index
// arithmetic; one barrier per plane, and 4.4 GB fetched for a 6.3 GB state
// (two criteria; it was 6.9).  2656 -> 1475 us for 22016 FP32 blocks, 722 ->
// 406 for 5440 FP64 ones and 117 -> 74 for 1000 FP32 ones.  Bound by the
// march: a plane's loads, FP64 criteria and barrier for 256 cells.
template <typename T, int NC>
__global__ void __launch_bounds__(NTE3) k_estimate3(EstArgs a)
{
    constexpr int XS = PD * PD, E = NB + 2;
    __shared__ double sv[4][NC][XS];
    __shared__ double red[NTE3 / 64];
    const int t = threadIdx.x;
    const bool cell = t < XS, est = t < E * E;
    const int px = t % PD - NG, py = t / PD - NG;
    const int c = (t / E + 1) * PD + t % E + 1;  // the cell this lane estimates
    int first, stride, end;
    xcd_range(a.nslots, first, stride, end);  // neighbouring blocks share lines in L2
    for (int slot = first; slot < end; slot += stride) {
        const int level = a.blk[slot].level;
        const double scale = pow(a.est.ratio, a.est.xi * (level - 1));
        size_t o[5] = {};
        if (cell) {
            const int zr[5] = {-2, -1, 0, NB, NB + 1};
#pragma unroll
            for (int r = 0; r < 5; r++)
                o[r] = cell_src<3>(a.desc, slot, px, py, zr[r]);
        }
        T raw[NC][3];
        auto load = [&](int z) {
            if (!cell)
                return;
            const size_t at = z == -2 ? o[0]
                                      : (z == -1 ? o[1]
                                                 : (z < NB ? o[2] + (size_t)z * XS : (z == NB ? o[3] : o[4])));
#pragma unroll
            for (int i = 0; i < NC; i++)
                est_load<3, T>(a, i, at, raw[i]);
        };
        double best = 0.0;
        load(-2);
        for (int z = -2; z <= NB + 1; z++) {
            if (cell) {
#pragma unroll
                for (int i = 0; i < NC; i++)
                    sv[z & 3][i][t] = est_form(a, i, raw[i]);
            }
            if (z <= NB)
                load(z + 1);
            __syncthreads();
            // plane z-1 from z-2, z-1 and z; plane z+1 goes into a fourth slot
            if (z >= 0 && est) {
#pragma unroll
                for (int i = 0; i < NC; i++) {
                    const double *q = sv[(z - 1) & 3][i];
                    const double v = q[c];
                    double s1 = 0.0, s2 = 0.0;
#pragma unroll
                    for (int d = 0; d < 3; d++) {
                        const double vp = d == 0 ? q[c + 1] : (d == 1 ? q[c + PD] : sv[z & 3][i][c]);
                        const double vm = d == 0 ? q[c - 1] : (d == 1 ? q[c - PD] : sv[(z - 2) & 3][i][c]);
                        s1 += (vp - vm) * (vp - vm);
                        s2 += (vp - 2.0 * v + vm) * (vp - 2.0 * v + vm);
                    }
                    const double e = est_cell(a, i, v, s1, s2, scale);
                    best = e > best ? e : best;
                }
            }
        }
        const double r = est_max<NTE3>(best, red);
        if (t == 0)
            a.err[slot] = r;
        __syncthreads();
    }
}

// padded tiles of the blocks present in both trees, 16 bytes per thread
__global__ void __launch_bounds__(NTE) k_remap_copy(RemapArgs a)
{
    const size_t n16 = a.tile_bytes / 16;
    for (int slot = blockIdx.x; slot < a.nslots; slot += gridDim.x) {
        const int src = a.map[slot];
        if (src < 0)
            continue;
        const uint4 *s = (const uint4 *)((const char *)a.Usrc + (size_t)src * a.tile_bytes);
        uint4 *d = (uint4 *)((char *)a.Udst + (size_t)slot * a.tile_bytes);
        for (size_t i = threadIdx.x; i < n16; i += NTE)
            d[i] = s[i];
    }
}

template <typename T>
static void launch_estimate3(const EstArgs &a, hipStream_t s)
{
    if (a.est.ncrit == 1)
        hipLaunchKernelGGL((k_estimate3<T, 1>), dim3(a.nslots), dim3(NTE3), 0, s, a);
    else if (a.est.ncrit == 2)
        hipLaunchKernelGGL((k_estimate3<T, 2>), dim3(a.nslots), dim3(NTE3), 0, s, a);
    else if (a.est.ncrit == 3)
        hipLaunchKernelGGL((k_estimate3<T, 3>), dim3(a.nslots), dim3(NTE3), 0, s, a);
    else
        hipLaunchKernelGGL((k_estimate3<T, 4>), dim3(a.nslots), dim3(NTE3), 0, s, a);
}

hipError_t launch_estimate(int ndim, bool fp64, const EstArgs &a, hipStream_t s)
{
    if (a.nslots <= 0)
        return hipSuccess;
    if (ndim == 3)
        fp64 ? launch_estimate3<double>(a, s) : launch_estimate3<float>(a, s);
    else if (fp64)
        hipLaunchKernelGGL(k_estimate2<double>, dim3(a.nslots), dim3(NTE), 0, s, a);
    else
        hipLaunchKernelGGL(k_estimate2<float>, dim3(a.nslots), dim3(NTE), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_remap_copy(const RemapArgs &a, hipStream_t s)
{
    if (a.nslots <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_remap_copy, dim3(a.nslots), dim3(NTE), 0, s, a);
    return hipGetLastError();
}

}  // namespace mapk
