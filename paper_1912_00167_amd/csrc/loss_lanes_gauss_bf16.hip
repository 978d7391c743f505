// Register-resident loss kernels: diagonal-Gaussian policies, bf16 buffer.
#include "loss_lanes.h"

namespace impact {

void launch_lanes_gauss_bf16(const LanesLaunch &l, const LossArgs &a, const LanesShape &g, hipStream_t s)
{
    launch_lanes_typed<IMPACT_DIAG_GAUSSIAN, bf16_t>(l, a, g, s);
}

}  // namespace impact
