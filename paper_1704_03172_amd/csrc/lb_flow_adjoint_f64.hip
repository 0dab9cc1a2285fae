// lb_flow_adjoint_f64.hip -- the backward flowing kernel (lb_flow_adjoint.h)
// in FP64.
#include "lb_flow_adjoint.h"

namespace lbw {
LBW_FLOW_ADJOINT_UNIT(double, 5, f64_q5)
LBW_FLOW_ADJOINT_UNIT(double, 9, f64_q9)
}  // namespace lbw
