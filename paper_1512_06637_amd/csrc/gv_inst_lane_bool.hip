// Lane transport of geometries holding composites.
#include "gv_inst.h"

namespace gv {

LaneKernel lane_kernel_bool(bool fp32, bool phys) {
  return fp32 ? (phys ? k_lane_transport<true, true, true, 3, 0> : k_lane_transport<true, false, true, 3, 0>)
              : (phys ? k_lane_transport<false, true, true, 3, 0> : k_lane_transport<false, false, true, 3, 0>);
}

}  // namespace gv
