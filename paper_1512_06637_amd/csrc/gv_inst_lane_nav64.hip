// Lane transport of elementary solids: navigation in FP64.
#include "gv_inst.h"

namespace gv {

LaneKernel lane_kernel_nav64(int waves, bool stage, bool cls) {
  return lane_kernel_for<false, false>(waves, stage, cls);
}

}  // namespace gv
