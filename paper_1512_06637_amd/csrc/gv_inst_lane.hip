// Lane transport of geometries of boxes and full tubes, and the choice among all instances.
#include "gv_inst.h"

namespace gv {

LaneKernel lane_kernel(int kind, bool fp32, bool phys, int waves, bool stage, bool cls) {
  if (kind == kComposites) return lane_kernel_composites(fp32, phys);
  if (kind == kBoxTube && cls && waves == (phys ? 3 : 4)) {
    if (phys) return fp32 ? k_lane_transport<true, true, kBoxTube, 3, 8, true> : k_lane_transport<false, true, kBoxTube, 3, 8, true>;
    return fp32 ? k_lane_transport<true, false, kBoxTube, 4, 8, true> : k_lane_transport<false, false, kBoxTube, 4, 8, true>;
  }
  if (phys) return fp32 ? lane_kernel_phys32(waves, stage, cls) : lane_kernel_phys64(waves, stage, cls);
  return fp32 ? lane_kernel_nav32(waves, stage, cls) : lane_kernel_nav64(waves, stage, cls);
}

}  // namespace gv
