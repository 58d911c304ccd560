// Lane transport of elementary solids: physics-limited with FP32 screens.
#include "gv_inst.h"

namespace gv {

LaneKernel lane_kernel_phys32(int waves, bool stage, bool cls) {
  return lane_kernel_for<true, true>(waves, stage, cls);
}

}  // namespace gv
