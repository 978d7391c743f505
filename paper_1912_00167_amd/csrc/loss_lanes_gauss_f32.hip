// Register-resident loss kernels: diagonal-Gaussian policies, fp32 buffer.
#include "loss_lanes.h"

namespace impact {

void launch_lanes_gauss_f32(const LanesLaunch &l, const LossArgs &a, const LanesShape &g, hipStream_t s)
{
    launch_lanes_typed<IMPACT_DIAG_GAUSSIAN, float>(l, a, g, s);
}

}  // namespace impact
