// Lane transport of geometries holding composites.
#include "gv_inst.h"

namespace gv {

LaneKernel lane_kernel_composites(bool fp32, bool phys) {
  constexpr int K = kComposites;
  return fp32 ? (phys ? k_lane_transport<true, true, K, 2, 0, true> : k_lane_transport<true, false, K, 2, 0, true>)
              : (phys ? k_lane_transport<false, true, K, 2, 0, true> : k_lane_transport<false, false, K, 2, 0, true>);
}

}  // namespace gv
