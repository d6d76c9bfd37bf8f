// Dataflow schedule: the exact propagator's forward kernels.
#include "msl_flow_launch.hpp"

namespace msl {
template hipError_t flow_launch<FLOW_XFWD>(const Ctx& c, const FlowArgs& a, hipStream_t st);
template hipError_t flow_occupancy<FLOW_XFWD>(int nz, int ny, int& per_cu, int& grid);
}  // namespace msl
