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

// Points per lane of the dataflow kernels (default_points_per_lane of the per-pass launches, so that
// both compute the same bits).
constexpr int flow_pts(int n) { return n >= 512 ? 8 : 4; }

// Threads per workgroup: one wavefront, or two where both axes have lines of a wavefront each and one
// of them 512 points (FlowEnds).  One-wavefront workgroups touch the 128-byte tiles of the exchange
// field in 16-byte pieces there, and 512 lines of 512 points then wait for the memory pipes: 12.2 k
// cycles a pass of 512x512 against 10.9 k in pairs of lines; at 256x256 the pairs' barriers
// cost more than the pieces (6.8 k cycles against 5.8 k).  Four lines: 13.9 k.
constexpr int flow_threads(int nz, int ny) {
  return (nz == 512 || ny == 512) && nz >= 256 && ny >= 256 ? 128 : 64;
}

// Lines per workgroup of an n-point axis, and workgroups of a row and of a column pass.
constexpr int flow_lines(int nz, int ny, int n) { return flow_threads(nz, ny) / (n / flow_pts(n)); }
constexpr int flow_row_units(int nz, int ny) { return ny / flow_lines(nz, ny, nz); }
constexpr int flow_col_units(int nz, int ny) { return nz / flow_lines(nz, ny, ny); }

// Whether a pass returns its share of the exchange field of two passes before to unset ahead of its output
// instead of after it (msl_flow.hpp): where the axes have different numbers of workgroups, so that
// some sit out every second pass.
constexpr bool flow_resets_early(int nz, int ny) { return flow_row_units(nz, ny) != flow_col_units(nz, ny); }

// Whether launches of `grid` workgroups, `per_cu` of which one compute unit holds, may run on a
// device of `cus` compute units.  Every workgroup of a launch has to be resident for its passes to end.
// Kernels of other kinds end by themselves and only delay that; launches of this schedule on other
// streams wait like this one, and they may be of any kind and grid (an adjoint runs two kinds side by
// side), so what has to fit is any mix of as many as there are hardware queues.  A compute unit holds any
// kFlowPerCu workgroups together, since it holds that many of each (none takes more than
// 1 / kFlowPerCu of a resource: two wavefronts per SIMD by the launch bounds, 16 KiB of LDS).
constexpr int kFlowPerCu = 4;
constexpr bool flow_admits(int queues, int cus, int per_cu, int grid) {
  return per_cu >= kFlowPerCu && (int64_t)queues * grid <= (int64_t)cus * kFlowPerCu;
}

// The fewest passes that are worth a launch's two ends: 4, but 6 in calls of fewer than 16 slice passes, which
// also pay for the fill of the exchange fields and the call's error kernel.  Forward of 64x64, 256x256 and
// 512x512 with 4 middle passes 34.5, 39.0 and 59.4 us against 34.0, 39.0 and 55.7 one launch each, with 7 37, 48 and 71
// against 46, 49 and 73; gradient of 8 slices of 256x256, a checkpoint every 4, 169 against 159, of 64 slices
// 911 against 990.
constexpr int flow_min_passes(int n_slices, bool exact) { return (exact ? 2 : 1) * n_slices < 16 ? 6 : 4; }

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
// The outputs of a call: n floats each, nullptr where there is none.
struct FlowOuts {
  float* p[4];
  int64_t n[4];
};
// End of a call that ran dataflow launches: its outputs to NaN if one of them gave up (err: their two error
// words).
hipError_t launch_flow_fold(const unsigned* err, const FlowOuts& o, hipStream_t st);
// The launch.
hipError_t launch_flow(int kind, const Ctx& c, FlowArgs a, hipStream_t st);

// One kind's kernels (each kind in a translation unit of its own): the launch, and how many workgroups
// one compute unit holds of the grid's kernel and how many the launch has.
template <int K>
hipError_t flow_launch(const Ctx& c, const FlowArgs& a, hipStream_t st);
template <int K>
hipError_t flow_occupancy(int nz, int ny, int& per_cu, int& grid);
}  // namespace msl
