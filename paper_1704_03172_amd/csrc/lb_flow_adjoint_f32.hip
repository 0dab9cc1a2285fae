// lb_flow_adjoint_f32.hip -- the backward flowing kernel (lb_flow_adjoint.h)
// with 32-bit lambda and rho (FP32 and half storage).
#include "lb_flow_adjoint.h"

namespace lbw {
LBW_FLOW_ADJOINT_UNIT(float, 5, f32_q5)
LBW_FLOW_ADJOINT_UNIT(float, 9, f32_q9)
}  // namespace lbw
