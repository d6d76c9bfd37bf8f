// Dataflow schedule: the reverse sweep's kernels.
#include "msl_flow_launch.hpp"

namespace msl {

hipError_t launch_flow_rev(const Ctx& c, const FlowArgs& a, hipStream_t st) { return flow_launch<KIND_REV_MID>(c, a, st); }
hipError_t flow_occupancy_rev(int nz, int ny, int& per_cu, int& grid) {
  return flow_occupancy<KIND_REV_MID>(nz, ny, per_cu, grid);
}

}  // namespace msl
