// lb_flow_f32_q5.hip -- instantiates the flowing kernel (lb_flow.h) for
// FP32 populations on D2Q5: single-grid, graph and batched launches.
#include "lb_flow.h"

namespace lbw {
LBW_FLOW_UNIT(float, 5, f32_q5)
LBW_FLOW_PATCH_UNIT(float, f32)
}  // namespace lbw
