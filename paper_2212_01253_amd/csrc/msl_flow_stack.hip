// Dataflow schedule: the forward sweep's kernels without a slice pack.
#include "msl_flow_launch.hpp"

namespace msl {
template hipError_t flow_launch<FLOW_STACK>(const Ctx& c, const FlowArgs& a, hipStream_t st);
template hipError_t flow_occupancy<FLOW_STACK>(int nz, int ny, int& per_cu, int& grid);
}  // namespace msl
