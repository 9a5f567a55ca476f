// sched.hpp -- how the workgroups of a launch walk a Morton-ordered work list.
#pragma once

#include <hip/hip_runtime.h>

namespace mapk {

// Work items of a grid of G workgroups, mapped so that the workgroups that
// run on one XCD (workgroups are dealt to the 8 XCDs round robin) walk one
// contiguous range of the Morton-ordered list: neighbouring blocks then meet
// in that XCD's L2.  Workgroup b, the (b / 8)-th on XCD b % 8, processes the
// items first, first + stride, ... below end.  Every item is covered exactly
// once for any G >= 1.
__device__ __forceinline__ void xcd_range(int nitems, int &first, int &stride, int &end)
{
    const int G = gridDim.x, b = blockIdx.x;
    const int x = b & 7, l = b >> 3;
    const int full = G >> 3, rem = G & 7;
    const int cnt = full + (x < rem ? 1 : 0);             // workgroups on this XCD
    const int before = x * full + (x < rem ? x : rem);    // on the XCDs before it
    const long long lo = (long long)nitems * before / G;
    const long long hi = (long long)nitems * (before + cnt) / G;
    first = (int)lo + l;
    stride = cnt;
    end = (int)hi;
}

// Blocks marched by one workgroup each, split so that the last round of an
// XCD is not nearly empty: of the XCD's blocks (consecutive ones, as above)
// those that fill whole rounds of its `slots` resident workgroups are whole
// items, and the rest are cut into 2^lseg march segments each, the most that
// are resident at once (and at most 2^lmax).
struct Marches {
    int lo, full, lseg, n;  // first block, whole blocks, segments of the others, items
};

__host__ __device__ inline Marches marches_of(int lo, int nblocks, int slots, int lmax)
{
    const int rest = nblocks % slots;
    int l = 0;
    while (rest > 0 && l < lmax && rest << (l + 1) <= slots)
        l++;
    return {lo, nblocks - rest, l, nblocks - rest + (rest << l)};
}

// this XCD's items; the calling workgroup takes first, first + stride, .. < n
__device__ __forceinline__ Marches xcd_marches(int nblocks, int slots, int lmax, int &first, int &stride)
{
    int lo, hi;
    xcd_range(nblocks, lo, stride, hi);
    first = blockIdx.x >> 3;
    return marches_of(lo - first, hi - (lo - first), slots, lmax);
}

// item j: its block, and its segment among 2^lseg
__device__ __forceinline__ int march_item(const Marches &m, int j, int &seg, int &lseg)
{
    const int k = j - m.full;
    seg = k < 0 ? 0 : k & ((1 << m.lseg) - 1);
    lseg = k < 0 ? 0 : m.lseg;
    return m.lo + (k < 0 ? j : m.full + (k >> m.lseg));
}

// workgroups for one item each
inline int marches_grid(int nblocks, int slots, int lmax)
{
    const int a = marches_of(0, nblocks / 8, slots, lmax).n, b = marches_of(0, (nblocks + 7) / 8, slots, lmax).n;
    return 8 * (a > b ? a : b);
}

}  // namespace mapk
