// Lane and workgroup exchange of the fused stage kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "device_mhd.h"

namespace amrvac {
namespace {

// Workgroup barrier that orders LDS accesses only.  Every exchange between
// the threads of a workgroup in this kernel goes through LDS, so global loads
// in flight (the z-plane prefetch, the halo staging) stay in flight across it
// instead of being drained as a full fence would.
// (The compiler-level memory clobbers keep LDS accesses on their side; the
// wait makes this wave's LDS writes complete before it arrives.)
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt, expcnt untouched
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The value of the next lane of this lane's 16-lane row (a DPP row shift;
// the last lane of a row gets 0).
__device__ __forceinline__ float row_next(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x101, 0xF, 0xF, true));
}
__device__ __forceinline__ double row_next(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x101, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x101, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
// The value of the previous lane of the row; the first lane of a row gets
// first.
__device__ __forceinline__ float row_prev(float v, float first) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(first), __float_as_int(v), 0x111, 0xF, 0xF, false));
}
__device__ __forceinline__ double row_prev(double v, double first) {
  const long long b = __double_as_longlong(v), f = __double_as_longlong(first);
  const int lo = __builtin_amdgcn_update_dpp((int)f, (int)b, 0x111, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(f >> 32), (int)(b >> 32), 0x111, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
// The values of lanes l and l + 32 (l = lane % 32), in every lane.
__device__ __forceinline__ void both_halves(float v, float& lower, float& upper) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(v), __float_as_int(v), false, false);
  lower = __int_as_float(r[0]);
  upper = __int_as_float(r[1]);
}
__device__ __forceinline__ void both_halves(double v, double& lower, double& upper) {
  const long long b = __double_as_longlong(v);
  const auto lo = __builtin_amdgcn_permlane32_swap((int)b, (int)b, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((int)(b >> 32), (int)(b >> 32), false, false);
  lower = __longlong_as_double(((long long)(int)hi[0] << 32) | (long long)(unsigned)lo[0]);
  upper = __longlong_as_double(((long long)(int)hi[1] << 32) | (long long)(unsigned)lo[1]);
}

// The variable that takes q's place when x and y are exchanged (swap 1).
__device__ __forceinline__ int swap_xy(int q, int swap) {
  return (q == 1 || q == I_BX) ? q + swap : ((q == 2 || q == I_BY) ? q - swap : q);
}

}  // namespace
}  // namespace amrvac
