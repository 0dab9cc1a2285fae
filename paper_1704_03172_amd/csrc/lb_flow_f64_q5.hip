// lb_flow_f64_q5.hip -- instantiates the flowing kernel (lb_flow.h) for
// FP64 populations on D2Q5: single-grid, graph and batched launches.
#include "lb_flow.h"

namespace lbw {
LBW_FLOW_UNIT(double, 5, f64_q5)
LBW_FLOW_PATCH_UNIT(double, f64)
}  // namespace lbw
