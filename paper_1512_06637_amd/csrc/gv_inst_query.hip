// ComputeStep with each lane in its own volume, and the serving round.
#include "gv_inst.h"

namespace gv {

StepNavKernel step_nav_kernel(int kind, bool fp32) {
  if (kind == kBoxTube) return fp32 ? k_step_nav<true, kBoxTube> : k_step_nav<false, kBoxTube>;
  if (kind == kElementary) return fp32 ? k_step_nav<true, kElementary> : k_step_nav<false, kElementary>;
  return fp32 ? k_step_nav<true, kComposites> : k_step_nav<false, kComposites>;
}

ServeKernel serve_kernel(int kind) {
  return kind == kBoxTube ? k_serve<kBoxTube> : kind == kElementary ? k_serve<kElementary> : k_serve<kComposites>;
}

}  // namespace gv
