// lb_flow_f16_q5.hip -- instantiates the flowing kernel (lb_flow.h) for
// FP16-stored populations on D2Q5: single-grid, graph and batched launches.
#include "lb_flow.h"

namespace lbw {
LBW_FLOW_UNIT(_Float16, 5, f16_q5)
LBW_FLOW_PATCH_UNIT(_Float16, f16)
}  // namespace lbw
