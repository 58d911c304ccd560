// Per-step kernel of the basket form: navigation.
#include "gv_inst.h"

namespace gv {

StepKernel step_kernel(bool has_bool, bool work, bool fp32, bool phys, bool waves3) {
  if (phys) return step_kernel_phys(has_bool, work, fp32);
  if (has_bool) return fp32 ? k_bt_step<true, false, true, false, 4> : k_bt_step<false, false, true, false, 4>;
  if (work) return fp32 ? k_bt_step<true, false, false, true, 4> : k_bt_step<false, false, false, true, 4>;
  if (waves3) return fp32 ? k_bt_step<true, false, false, false, 3> : k_bt_step<false, false, false, false, 3>;
  return fp32 ? k_bt_step<true, false, false, false, 4> : k_bt_step<false, false, false, false, 4>;
}

}  // namespace gv
