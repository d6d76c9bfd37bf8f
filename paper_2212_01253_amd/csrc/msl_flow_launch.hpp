// Kernel choice of the dataflow schedule for one pass kind (included by one
// translation unit per kind, so that they compile side by side).
#pragma once

#include "msl_flow.hpp"

namespace msl {

// Points per lane of the dataflow kernels (default_points_per_lane of the per-pass launches, so that
// both compute the same bits).
template <int N>
constexpr int flow_pts() { return N >= 512 ? 8 : 4; }

// Threads per workgroup: one wavefront, or two where both axes have lines of a wavefront each and one
// of them 512 points (FlowEnds).  One-wavefront workgroups touch the 128-byte tiles of the exchange
// field in 16-byte pieces there, and 512 lines of 512 points then wait for the memory pipes: 12.2 k
// cycles a pass of 512x512 against 10.9 k in pairs of lines; at 256x256 the pairs' barriers
// cost more than the pieces (6.8 k cycles against 5.8 k).  Four lines: 13.9 k.
constexpr int flow_threads(int nz, int ny) {
  return (nz == 512 || ny == 512) && nz >= 256 && ny >= 256 ? 128 : 64;
}

template <int NZ, int NY>
constexpr int flow_grid() {
  constexpr int T = flow_threads(NZ, NY), GZ = T / (NZ / flow_pts<NZ>()), GY = T / (NY / flow_pts<NY>());
  return NY / GZ > NZ / GY ? NY / GZ : NZ / GY;
}

// Calls f.template operator()<NZ, NY>() for the grid; false: no kernel for it.
template <class F>
bool flow_dispatch(int nz, int ny, F&& f) {
  auto with_z = [&](auto z) {
    constexpr int NZ = decltype(z)::value;
    switch (ny) {
      case 16: f(z, std::integral_constant<int, 16>{}); return true;
      case 32: f(z, std::integral_constant<int, 32>{}); return true;
      case 64: f(z, std::integral_constant<int, 64>{}); return true;
      case 128: f(z, std::integral_constant<int, 128>{}); return true;
      case 256: f(z, std::integral_constant<int, 256>{}); return true;
      case 512: f(z, std::integral_constant<int, 512>{}); return true;
      default: return false;
    }
    (void)NZ;
  };
  switch (nz) {
    case 16: return with_z(std::integral_constant<int, 16>{});
    case 32: return with_z(std::integral_constant<int, 32>{});
    case 64: return with_z(std::integral_constant<int, 64>{});
    case 128: return with_z(std::integral_constant<int, 128>{});
    case 256: return with_z(std::integral_constant<int, 256>{});
    case 512: return with_z(std::integral_constant<int, 512>{});
    default: return false;
  }
}

template <int K>
hipError_t flow_launch(const Ctx& c, const FlowArgs& a, hipStream_t st) {
  hipError_t e = hipErrorNotSupported;
  flow_dispatch(c.nz, c.ny, [&](auto z, auto y) {
    constexpr int NZ = decltype(z)::value, NY = decltype(y)::value, T = flow_threads(NZ, NY);
    hipLaunchKernelGGL((k_flow<NZ, NY, flow_pts<NZ>(), flow_pts<NY>(), K, T>), dim3(flow_grid<NZ, NY>()), dim3(T), 0,
                       st, c, a);
    e = hipGetLastError();
  });
  return e;
}

// How many workgroups of the grid's kernel one compute unit holds, and the kernel's grid.
template <int K>
hipError_t flow_occupancy(int nz, int ny, int& per_cu, int& grid) {
  hipError_t e = hipErrorNotSupported;
  flow_dispatch(nz, ny, [&](auto z, auto y) {
    constexpr int NZ = decltype(z)::value, NY = decltype(y)::value, T = flow_threads(NZ, NY);
    grid = flow_grid<NZ, NY>();
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_flow<NZ, NY, flow_pts<NZ>(), flow_pts<NY>(), K, T>, T,
                                                     0);
  });
  return e;
}

}  // namespace msl
