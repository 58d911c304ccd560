// Lane transport of geometries holding composites: 2 waves per SIMD (no spills
// beyond 12 bytes; 262,144 tracks of the detector with a composite in one kind of
// module 0.85 ms at 2, 1.22 at 3 and 1.43 at 4), outputs staged (0.91 without).
#include "gv_inst.h"

namespace gv {

LaneKernel lane_kernel_composites(bool fp32, bool phys) {
  constexpr int K = kComposites;
  return fp32 ? (phys ? k_lane_transport<true, true, K, 2, 8, true> : k_lane_transport<true, false, K, 2, 8, true>)
              : (phys ? k_lane_transport<false, true, K, 2, 8, true> : k_lane_transport<false, false, K, 2, 8, true>);
}

}  // namespace gv
