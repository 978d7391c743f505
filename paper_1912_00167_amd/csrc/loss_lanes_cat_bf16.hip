// Register-resident loss kernels: categorical policies, bf16 buffer.
#include "loss_lanes.h"

namespace impact {

void launch_lanes_cat_bf16(const LanesLaunch &l, const LossArgs &a, const LanesShape &g, hipStream_t s)
{
    launch_lanes_typed<IMPACT_CATEGORICAL, bf16_t>(l, a, g, s);
}

}  // namespace impact
