// ComputeStep with each lane in its own volume, and the serving round.
#include "gv_inst.h"

namespace gv {

StepNavKernel step_nav_kernel(bool has_bool, bool fp32) {
  if (has_bool) return fp32 ? k_step_nav<true, true> : k_step_nav<false, true>;
  return fp32 ? k_step_nav<true, false> : k_step_nav<false, false>;
}

ServeKernel serve_kernel(bool has_bool) { return has_bool ? k_serve<true> : k_serve<false>; }

}  // namespace gv
