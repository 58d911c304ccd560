// Per-step kernel of the basket form: navigation.
#include "gv_inst.h"

namespace gv {

StepKernel step_kernel(int kind, bool work, bool fp32, bool phys, bool waves3) {
  constexpr int B = kBoxTube, E = kElementary, C = kComposites;
  if (phys) return step_kernel_phys(kind, work, fp32);
  if (kind == C) return fp32 ? k_bt_step<true, false, C, false, 4> : k_bt_step<false, false, C, false, 4>;
  if (work) return fp32 ? k_bt_step<true, false, E, true, 4> : k_bt_step<false, false, E, true, 4>;
  if (kind == B && !waves3) return fp32 ? k_bt_step<true, false, B, false, 4> : k_bt_step<false, false, B, false, 4>;
  if (waves3) return fp32 ? k_bt_step<true, false, E, false, 3> : k_bt_step<false, false, E, false, 3>;
  return fp32 ? k_bt_step<true, false, E, false, 4> : k_bt_step<false, false, E, false, 4>;
}

}  // namespace gv
