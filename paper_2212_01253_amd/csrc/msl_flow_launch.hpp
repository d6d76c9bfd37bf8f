// Kernel choice of the dataflow schedule for one pass kind (included by one
// translation unit per kind, so that they compile side by side).
#pragma once

#include "msl_flow.hpp"

namespace msl {

template <int NZ, int NY>
constexpr int flow_grid() {
  return flow_row_units(NZ, NY) > flow_col_units(NZ, NY) ? flow_row_units(NZ, NY) : flow_col_units(NZ, NY);
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
    hipLaunchKernelGGL((k_flow<NZ, NY, flow_pts(NZ), flow_pts(NY), K, T>), dim3(flow_grid<NZ, NY>()), dim3(T), 0,
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
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_flow<NZ, NY, flow_pts(NZ), flow_pts(NY), K, T>, T,
                                                     0);
  });
  return e;
}

}  // namespace msl
