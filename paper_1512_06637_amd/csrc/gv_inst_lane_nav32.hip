// Lane transport of elementary solids: navigation with FP32 screens.
#include "gv_inst.h"

namespace gv {

LaneKernel lane_kernel_nav32(int waves, bool stage, bool cls) {
  return lane_kernel_for<true, false>(waves, stage, cls);
}

}  // namespace gv
