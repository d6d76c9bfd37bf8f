// Dataflow schedule: the reverse sweep's kernels.
#include "msl_flow_launch.hpp"

namespace msl {
template hipError_t flow_launch<FLOW_REV>(const Ctx& c, const FlowArgs& a, hipStream_t st);
template hipError_t flow_occupancy<FLOW_REV>(int nz, int ny, int& per_cu, int& grid);
}  // namespace msl
