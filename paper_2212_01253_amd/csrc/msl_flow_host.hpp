// Host side of the dataflow schedule (msl_flow.hip).
#pragma once
#include "msl_passes.hpp"

namespace msl {
struct FlowArgs {
  PhaseSpec ph;
  int p0, n;              // passes p0 .. p0 + n - 1 of the phase, all of the kernel's kind
  float2* x;              // exchange fields, [4][ny][nz], all kUnset at the start but X[rot]
  int rot;                // pass i reads X[(rot + i) % 4]
  unsigned* err;          // error word of the call's launches on these fields
  unsigned* status;       // status word of the workspace
  unsigned spin_limit;
  int nap;                // pauses before the first look at a pass's input
};

constexpr int kFlowMinPasses = 4;   // a launch of fewer passes is not worth its two ends

// Whether the dataflow schedule serves an ny x nz grid on the current device.
bool flow_serves(int ny, int nz);
// All elements of the exchange fields to kUnset.
hipError_t launch_flow_init(float2* x, int64_t m, hipStream_t st);
// The launch; kind: KIND_FWD_MID or KIND_REV_MID.
hipError_t launch_flow(const Ctx& c, FlowArgs a, int kind, hipStream_t st);
// The reverse sweep's part (msl_flow_rev.hip).
hipError_t launch_flow_rev(const Ctx& c, const FlowArgs& a, hipStream_t st);
hipError_t flow_occupancy_rev(int nz, int ny, int& per_cu, int& grid);
}  // namespace msl
