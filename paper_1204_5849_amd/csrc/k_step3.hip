// k_step3.hip -- launches of the 3-D block update: the FP32 LF step is
// instantiated in k_step3_lf32.hip, every other instance here.
#include "k_step3.hpp"

namespace mapk {

template <typename T, bool MIXED, bool RESIST, int RS>
static hipError_t launch3_weno(int sch, const StepArgs &a, int grid, hipStream_t s)
{
    if (sch == SCH_WENO1)
        return launch3<T, MIXED, RESIST, SCH_WENO1, MAP_MINMOD, RS>(a, grid, s);
    return launch3<T, MIXED, RESIST, SCH_WENO2, MAP_MINMOD, RS>(a, grid, s);
}

template <bool RESIST, int RS>
static hipError_t launch3_lf64(const StepArgs &a, int grid, hipStream_t s)
{
    if (a.limiter == MAP_MINMOD)
        return launch3<double, false, RESIST, SCH_LF, MAP_MINMOD, RS>(a, grid, s);
    if (a.limiter == MAP_VANLEER)
        return launch3<double, false, RESIST, SCH_LF, MAP_VANLEER, RS>(a, grid, s);
    return launch3<double, false, RESIST, SCH_LF, MAP_PAPER_PHI, RS>(a, grid, s);
}

template <bool RESIST, int RS>
static hipError_t launch3_any(bool fp64, int sch, const StepArgs &a, int grid, hipStream_t s)
{
    if (!fp64)
        return launch3_weno<float, true, RESIST, RS>(sch, a, grid, s);
    if (sch == SCH_LF)
        return launch3_lf64<RESIST, RS>(a, grid, s);
    return launch3_weno<double, false, RESIST, RS>(sch, a, grid, s);
}

hipError_t launch_step3(bool fp64, bool resist, int sch, const StepArgs &a, int grid, hipStream_t s)
{
    if (a.nitems <= 0)
        return hipSuccess;
    if (!fp64 && sch == SCH_LF)
        return launch_step3_lf32(resist, a, grid, s);
    if (a.riemann == MAP_HLLC)
        return resist ? launch3_any<true, MAP_HLLC>(fp64, sch, a, grid, s)
                      : launch3_any<false, MAP_HLLC>(fp64, sch, a, grid, s);
    return resist ? launch3_any<true, MAP_RUSANOV>(fp64, sch, a, grid, s)
                  : launch3_any<false, MAP_RUSANOV>(fp64, sch, a, grid, s);
}

}  // namespace mapk
