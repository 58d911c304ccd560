// Lane transport: navigation in FP64, and the choice among all instances.
#include "gv_inst.h"

namespace gv {

LaneKernel lane_kernel(bool has_bool, bool fp32, bool phys, int waves, bool stage, bool cls) {
  if (has_bool) return lane_kernel_bool(fp32, phys);
  if (phys) return fp32 ? lane_kernel_phys32(waves, stage, cls) : lane_kernel_phys64(waves, stage, cls);
  return fp32 ? lane_kernel_nav32(waves, stage, cls) : lane_kernel_for<false, false>(waves, stage, cls);
}

}  // namespace gv
