// ComputeStep with each lane in its own volume, and the serving round.
#include "gv_inst.h"

namespace gv {

template <bool F32>
static StepNavKernel step_nav_kernel_for(int kind, bool group) {
  if (kind == kBoxTube) return group ? k_step_nav<F32, kBoxTube, true> : k_step_nav<F32, kBoxTube, false>;
  if (kind == kElementary) return group ? k_step_nav<F32, kElementary, true> : k_step_nav<F32, kElementary, false>;
  return k_step_nav<F32, kComposites, false>;
}

StepNavKernel step_nav_kernel(int kind, bool fp32, bool group) {
  return fp32 ? step_nav_kernel_for<true>(kind, group) : step_nav_kernel_for<false>(kind, group);
}

ServeKernel serve_kernel(int kind) {
  return kind == kBoxTube ? k_serve<kBoxTube> : kind == kElementary ? k_serve<kElementary> : k_serve<kComposites>;
}

}  // namespace gv
