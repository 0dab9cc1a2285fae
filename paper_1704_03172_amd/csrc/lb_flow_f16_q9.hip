// lb_flow_f16_q9.hip -- instantiates the flowing kernel (lb_flow.h) for
// FP16-stored populations on D2Q9: single-grid, graph and batched launches.
#include "lb_flow.h"

namespace lbw {
LBW_FLOW_UNIT(_Float16, 9, f16_q9)
}  // namespace lbw
