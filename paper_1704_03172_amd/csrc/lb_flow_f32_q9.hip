// lb_flow_f32_q9.hip -- instantiates the flowing kernel (lb_flow.h) for
// FP32 populations on D2Q9: single-grid, graph and batched launches.
#include "lb_flow.h"

namespace lbw {
LBW_FLOW_UNIT(float, 9, f32_q9)
}  // namespace lbw
