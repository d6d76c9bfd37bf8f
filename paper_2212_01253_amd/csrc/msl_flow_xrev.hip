// Dataflow schedule: the exact propagator's reverse kernels.
#include "msl_flow_launch.hpp"

namespace msl {
template hipError_t flow_launch<FLOW_XREV>(const Ctx& c, const FlowArgs& a, hipStream_t st);
template hipError_t flow_occupancy<FLOW_XREV>(int nz, int ny, int& per_cu, int& grid);
}  // namespace msl
