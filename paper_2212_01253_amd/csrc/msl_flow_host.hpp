// Host side of the dataflow schedule (msl_flow.hip).
#pragma once
#include "msl_passes.hpp"

namespace msl {
constexpr uint32_t kUnset = 0xffb5a3c7u;  // real part of an element not yet stored (a quiet NaN)

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

// What the passes of a launch are: the paraxial middle passes of the forward sweep and the recompute with
// the transmission from the slice pack or (FLOW_STACK) from the caller's stacks, those of the reverse
// sweep, and the two passes per slice of the exact propagator, forward and reverse (from the stacks).
enum FlowKind : int { FLOW_FWD = 0, FLOW_REV = 1, FLOW_STACK = 2, FLOW_XFWD = 3, FLOW_XREV = 4, FLOW_KINDS = 5 };

// Whether pass pd is one that a launch of the kind takes.
inline bool flow_takes(int kind, const PassDesc& pd) {
  const bool rev = kind == FLOW_REV || kind == FLOW_XREV;
  const int lay = kind == FLOW_STACK ? (int)LAY_R : (int)LAY_T;
  if (pd.src_lay != lay || pd.dst_lay != lay || pd.src != pd.dst || (pd.conj != 0) != (rev && pd.pre != PRE_IFFT_N))
    return false;
  const int mid = rev ? MID_T_ADJ : MID_T_FWD;
  if (kind < FLOW_XFWD) return pd.pre == PRE_PROP && pd.mid == mid && pd.post == POST_PROP;
  if (pd.axis == COL) return pd.pre == PRE_NONE && pd.mid == MID_NONE && pd.post == POST_PROP2D;
  return pd.pre == PRE_IFFT_N && pd.mid == mid && pd.post == POST_FFT;
}

// Whether the dataflow schedule serves the kind on an ny x nz grid on the current device.
bool flow_serves(int kind, int ny, int nz);
// All elements of the exchange fields to kUnset.
hipError_t launch_flow_init(float2* x, int64_t m, hipStream_t st);
// The launch.
hipError_t launch_flow(int kind, const Ctx& c, FlowArgs a, hipStream_t st);

// One kind's kernels (each kind in a translation unit of its own): the launch, and how many workgroups
// one compute unit holds of the grid's kernel and how many the launch has.
template <int K>
hipError_t flow_launch(const Ctx& c, const FlowArgs& a, hipStream_t st);
template <int K>
hipError_t flow_occupancy(int nz, int ny, int& per_cu, int& grid);
}  // namespace msl
