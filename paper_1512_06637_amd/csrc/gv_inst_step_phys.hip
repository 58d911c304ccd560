// Per-step kernel of the basket form: physics-limited.
#include "gv_inst.h"

namespace gv {

StepKernel step_kernel_phys(int kind, bool work, bool fp32) {
  constexpr int E = kElementary, C = kComposites;
  if (kind == C) return fp32 ? k_bt_step<true, true, C, false, 3> : k_bt_step<false, true, C, false, 3>;
  if (work) return fp32 ? k_bt_step<true, true, E, true, 3> : k_bt_step<false, true, E, true, 3>;
  return fp32 ? k_bt_step<true, true, E, false, 3> : k_bt_step<false, true, E, false, 3>;
}

}  // namespace gv
