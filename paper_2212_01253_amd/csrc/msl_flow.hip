// Dataflow schedule: the host side.
#include <cstdlib>
#include <mutex>

#include "msl_flow_host.hpp"

namespace msl {
namespace {

__global__ void __launch_bounds__(256) k_flow_init(float4* x, int64_t n4) {
  const float q = __uint_as_float(kUnset);
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256)
    x[i] = make_float4(q, q, q, q);
}

// What a launch that gave up has poisoned by itself is only what depends on it: slices done before it and
// lines done beside it would stay finite.  One launch per call, not per phase (1.5 us of a 64x64x128
// forward's 273, 6 us of a 128x64x97 gradient's 680).
__global__ void __launch_bounds__(256) k_flow_fold(const unsigned* err, FlowOuts o) {
  if ((err[0] | err[1]) == 0u) return;
  const float q = __builtin_nanf("");
  for (int k = 0; k < 4; ++k)
    if (o.p[k])
      for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < o.n[k]; i += (int64_t)gridDim.x * 256) o.p[k][i] = q;
}

int log2_of(int n) { return __builtin_ctz((unsigned)n); }

// Pauses (256 cycles each) before the first look at a pass's input: the more a pass exchanges, the
// longer its stores take to land, and looking too early only slows them.  Cycles per pass by pauses:
// 64x64 4412 with none, 4574 with one; 128x128 5509, 5429, 5652 (0, 1, 2); 256x256 6675, 6014, 5781,
// 5943 (0..3); 512x512 11110 with none, 10924 with four.
int flow_nap(int64_t m) { return m <= 8192 ? 0 : (m <= 32768 ? 1 : (m <= 131072 ? 2 : 4)); }

}  // namespace

// (flow_admits)  Streams of one priority share GPU_MAX_HW_QUEUES hardware queues (4 unless set), each of which
// runs one kernel at a time; flow_kind sees to the priority.  Other processes' launches are not seen.
bool flow_serves(int kind, int ny, int nz) {
  struct Fits {
    signed char known[FLOW_KINDS][11][11];   // 0: not asked yet, 1: fits, -1: does not
  };
  static std::mutex mu;
  static Fits fits[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
  std::lock_guard<std::mutex> lock(mu);
  signed char& k = fits[dev].known[kind][log2_of(ny)][log2_of(nz)];
  if (k == 0) {
    int cus = 0, per_cu = 0, grid = 0;
    const char* q = std::getenv("GPU_MAX_HW_QUEUES");
    const int queues = q && std::atoi(q) > 4 ? std::atoi(q) : 4;
    hipError_t e = hipErrorNotSupported;
    switch (kind) {
      case FLOW_FWD: e = flow_occupancy<FLOW_FWD>(nz, ny, per_cu, grid); break;
      case FLOW_REV: e = flow_occupancy<FLOW_REV>(nz, ny, per_cu, grid); break;
      case FLOW_STACK: e = flow_occupancy<FLOW_STACK>(nz, ny, per_cu, grid); break;
      case FLOW_XFWD: e = flow_occupancy<FLOW_XFWD>(nz, ny, per_cu, grid); break;
      case FLOW_XREV: e = flow_occupancy<FLOW_XREV>(nz, ny, per_cu, grid); break;
      default: break;
    }
    // (masks of the whole process, which neither the device's nor the stream's attributes show)
    const bool masked = std::getenv("HSA_CU_MASK") || std::getenv("ROC_GLOBAL_CU_MASK");
    const bool ok = e == hipSuccess && !masked &&
                    hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
                    flow_admits(queues, cus, per_cu, grid);
    if (!ok) (void)hipGetLastError();
    k = ok ? 1 : -1;
  }
  return k > 0;
}

hipError_t launch_flow_init(float2* x, int64_t m, hipStream_t st) {
  const int64_t n4 = 4 * m / 2, nb = (n4 + 255) / 256;
  hipLaunchKernelGGL(k_flow_init, dim3((unsigned)(nb < 2048 ? nb : 2048)), dim3(256), 0, st,
                     reinterpret_cast<float4*>(x), n4);
  return hipGetLastError();
}

hipError_t launch_flow_fold(const unsigned* err, const FlowOuts& o, hipStream_t st) {
  hipLaunchKernelGGL(k_flow_fold, dim3(128), dim3(256), 0, st, err, o);
  return hipGetLastError();
}

hipError_t launch_flow(int kind, const Ctx& c, FlowArgs a, hipStream_t st) {
  a.nap = flow_nap(c.m);
  switch (kind) {
    case FLOW_FWD: return flow_launch<FLOW_FWD>(c, a, st);
    case FLOW_REV: return flow_launch<FLOW_REV>(c, a, st);
    case FLOW_STACK: return flow_launch<FLOW_STACK>(c, a, st);
    case FLOW_XFWD: return flow_launch<FLOW_XFWD>(c, a, st);
    case FLOW_XREV: return flow_launch<FLOW_XREV>(c, a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace msl
