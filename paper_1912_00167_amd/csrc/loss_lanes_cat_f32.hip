// Register-resident loss kernels: categorical policies, fp32 buffer.
#include "loss_lanes.h"

namespace impact {

void launch_lanes_cat_f32(const LanesLaunch &l, const LossArgs &a, const LanesShape &g, hipStream_t s)
{
    launch_lanes_typed<IMPACT_CATEGORICAL, float>(l, a, g, s);
}

}  // namespace impact
