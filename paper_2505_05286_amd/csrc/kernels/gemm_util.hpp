// Launch helpers shared by the GEMM translation units.
#pragma once

#include <hip/hip_ext.h>

#include "common.hpp"
#include "kernels.hpp"

namespace hxf {

// Workgroup i of nb renumbered so that consecutive numbers (tiles sharing a weight slice)
// land on one XCD and its L2: workgroups are dealt to the eight XCDs in turn.
__device__ __forceinline__ int xcd_remap(int i, int nb) {
  const int xcd = i & 7, local = i >> 3;
  const int per = nb >> 3, rem = nb & 7;
  return (xcd < rem) ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
}

// Launch; with events, the kernel itself records its start (e0) and end (e1).
template <typename K, typename... Args>
hipError_t launch_ev(K kernel, dim3 grid, dim3 block, hipStream_t st, hipEvent_t e0, hipEvent_t e1, Args... args) {
  if (e0 || e1) hipExtLaunchKernelGGL(kernel, grid, block, 0, st, e0, e1, 0, args...);
  else hipLaunchKernelGGL(kernel, grid, block, 0, st, args...);
  return hipGetLastError();
}

}  // namespace hxf
