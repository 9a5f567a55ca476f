// k_step3_lf32.hip -- the FP32 instances of the 3-D TVD-LF step (one per limiter
// and face flux, with and without resistivity).  They run faster without
// LLVM's loop strength reduction, whose per-variable address registers spill
// at 128 registers per lane; the others stay in k_step3.hip with the defaults
// (see the build script).
#include "k_step3.hpp"

namespace mapk {

template <bool RESIST, int RS>
static hipError_t launch3_lf32(const StepArgs &a, int grid, hipStream_t s)
{
    if (a.limiter == MAP_MINMOD)
        return launch3<float, true, RESIST, SCH_LF, MAP_MINMOD, RS>(a, grid, s);
    if (a.limiter == MAP_VANLEER)
        return launch3<float, true, RESIST, SCH_LF, MAP_VANLEER, RS>(a, grid, s);
    return launch3<float, true, RESIST, SCH_LF, MAP_PAPER_PHI, RS>(a, grid, s);
}

hipError_t launch_step3_lf32(bool resist, const StepArgs &a, int grid, hipStream_t s)
{
    if (a.nitems <= 0)
        return hipSuccess;
    if (a.riemann == MAP_HLLC)
        return resist ? launch3_lf32<true, MAP_HLLC>(a, grid, s) : launch3_lf32<false, MAP_HLLC>(a, grid, s);
    return resist ? launch3_lf32<true, MAP_RUSANOV>(a, grid, s)
                  : launch3_lf32<false, MAP_RUSANOV>(a, grid, s);
}

}  // namespace mapk
