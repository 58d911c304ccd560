// Per-step kernel of the basket form: physics-limited.
#include "gv_inst.h"

namespace gv {

StepKernel step_kernel_phys(bool has_bool, bool work, bool fp32) {
  if (has_bool) return fp32 ? k_bt_step<true, true, true, false, 3> : k_bt_step<false, true, true, false, 3>;
  if (work) return fp32 ? k_bt_step<true, true, false, true, 3> : k_bt_step<false, true, false, true, 3>;
  return fp32 ? k_bt_step<true, true, false, false, 3> : k_bt_step<false, true, false, false, 3>;
}

}  // namespace gv
