// rt_sweep_f64_par.hip -- the fused sweep instantiated for double arithmetic,
// the DELO-parabolic pairs streamed.
#include "rt_sweep_kernel.h"

namespace rt {

hipError_t launch_sweep_f64_par(int L, int W, bool pf, const SweepArgs &a, int nblocks, int ns_max,
                              hipStream_t s) {
    return sweep::launch_any<double, kCoefParabolic>(L, W, pf, a, nblocks, ns_max, s);
}

}  // namespace rt
