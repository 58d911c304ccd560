// Lane transport of elementary solids: physics-limited, FP64.
#include "gv_inst.h"

namespace gv {

LaneKernel lane_kernel_phys64(int waves, bool stage, bool cls) {
  return lane_kernel_for<false, true>(waves, stage, cls);
}

}  // namespace gv
