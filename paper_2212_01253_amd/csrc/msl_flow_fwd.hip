// Dataflow schedule: the forward sweep's and the recompute's kernels.
#include "msl_flow_launch.hpp"

namespace msl {
template hipError_t flow_launch<FLOW_FWD>(const Ctx& c, const FlowArgs& a, hipStream_t st);
template hipError_t flow_occupancy<FLOW_FWD>(int nz, int ny, int& per_cu, int& grid);
}  // namespace msl
