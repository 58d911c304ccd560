// The large navigation kernels are instantiated in source files of their own
// (gv_inst_*.hip), so that the library builds in parallel; these functions
// hand their entry points to the host side in gv_abi.hip.
#pragma once
#include "gv_baskets.h"
#include "gv_lane.h"
#include "gv_serve_kernel.h"

namespace gv {

using StepKernel = void (*)(DevGeom, int, int, int, const int*, const int*, TRec*, const int*, int*, uint32_t*, int*,
                            TCtl, int32_t*, double*, int32_t*, uint32_t*, const int*, double*, int*, int64_t,
                            PhysArgs, int8_t*, int8_t*);
using LaneKernel = void (*)(LaneArgs);
using StepNavKernel = void (*)(DevGeom, int64_t, const double*, const double*, const double*, const double*,
                               const double*, const double*, const int32_t*, const double*, double*, int32_t*,
                               uint32_t*);
using ServeKernel = void (*)(DevGeom, const SDesc*, int, int64_t, const char*, char*);

// The per-step kernel of the basket form: the geometry's solids (SolidKind; the
// kernels for elementary solids serve boxes and tubes too), the work-counting
// instance while counters are asked for (geometries without composites), FP32
// screens or not, physics-limited or not, and the register budget of the
// navigation step (3 or 4 waves per SIMD).
StepKernel step_kernel(int kind, bool work, bool fp32, bool phys, bool waves3);
StepKernel step_kernel_phys(int kind, bool work, bool fp32);

// The lane-transport instance: the geometry's solids, FP32 screens or not,
// physics-limited or not, the register budget (3 or 4 waves per SIMD), output
// staging and per-class scheduling (which always stages).  Boxes and full tubes
// have instances of their own for the default shapes (per-class scheduling, 4
// waves for navigation and 3 for physics) and share the elementary solids'
// otherwise; geometries with composites run one shape per precision and physics.
LaneKernel lane_kernel(int kind, bool fp32, bool phys, int waves, bool stage, bool cls);
LaneKernel lane_kernel_nav64(int waves, bool stage, bool cls);
LaneKernel lane_kernel_nav32(int waves, bool stage, bool cls);
LaneKernel lane_kernel_phys64(int waves, bool stage, bool cls);
LaneKernel lane_kernel_phys32(int waves, bool stage, bool cls);
LaneKernel lane_kernel_composites(bool fp32, bool phys);

// ComputeStep of a basket (group: regrouped by volume), and the serving round.
StepNavKernel step_nav_kernel(int kind, bool fp32, bool group);
ServeKernel serve_kernel(int kind);

// The launch shapes of one precision and kind of transport (elementary solids).
template <bool F32, bool PHYS>
LaneKernel lane_kernel_for(int waves, bool stage, bool cls) {
  constexpr int K = kElementary;
  if (cls) return waves == 3 ? k_lane_transport<F32, PHYS, K, 3, 8, true> : k_lane_transport<F32, PHYS, K, 4, 8, true>;
  if (waves == 3) return stage ? k_lane_transport<F32, PHYS, K, 3, 8> : k_lane_transport<F32, PHYS, K, 3, 0>;
  return stage ? k_lane_transport<F32, PHYS, K, 4, 8> : k_lane_transport<F32, PHYS, K, 4, 0>;
}

}  // namespace gv
