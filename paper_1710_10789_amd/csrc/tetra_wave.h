// Wave and workgroup helpers of the spline kernels (gfx950). Internal header.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tetra {

// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniform(float v) { return __int_as_float(uniform(__float_as_int(v))); }
__device__ __forceinline__ double uniform(double v) {
  return __hiloint2double(uniform(__double2hiint(v)), uniform(__double2loint(v)));
}

// Reduction over the wave by row shifts within 16 lanes and two broadcasts; every lane gets the result.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_f32(float v) {
  const int x = __float_as_int(v);
  return __int_as_float(__builtin_amdgcn_update_dpp(x, x, CTRL, ROWS, 0xf, false));  // lanes without a source: their own
}
template <typename F>
__device__ __forceinline__ float wave_reduce(float v, F&& f) {
  v = f(v, dpp_f32<0x111, 0xf>(v));  // row_shr:1, 2, 4, 8
  v = f(v, dpp_f32<0x112, 0xf>(v));
  v = f(v, dpp_f32<0x114, 0xf>(v));
  v = f(v, dpp_f32<0x118, 0xf>(v));
  v = f(v, dpp_f32<0x142, 0xa>(v));  // row_bcast:15 into rows 1 and 3
  v = f(v, dpp_f32<0x143, 0xc>(v));  // row_bcast:31 into rows 2 and 3
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_min(float v) {
  return wave_reduce(v, [](float a, float b) { return fminf(a, b); });
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float wave_sum(float v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// f(i) for i < n over the workgroup's lanes. The trip count is uniform, and the lane index opaque in every
// call, so that nothing derived from it stays live (or spilled) between the loops of a unit.
template <typename F>
__device__ __forceinline__ void for_lanes(int n, F&& f, bool reverse = false) {
  const int nt = blockDim.x;
  int tid = threadIdx.x;
  if (reverse) tid = nt - 1 - tid;
  asm volatile("" : "+v"(tid));
  for (int i0 = 0; i0 < n; i0 += nt)
    if (i0 + tid < n) f(i0 + tid);
}

// A lane's share of a 64-lane inclusive running sum, by row shifts within 16 lanes and two broadcasts.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp64(uint64_t v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xf, true);
  return (uint64_t)(uint32_t)lo | ((uint64_t)(uint32_t)hi << 32);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_of(double v) {
  return __longlong_as_double((long long)dpp64<CTRL, ROWS>((uint64_t)__double_as_longlong(v)));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ long long dpp_of(long long v) {
  return (long long)dpp64<CTRL, ROWS>((uint64_t)v);
}
template <typename T>
__device__ __forceinline__ T wave_scan(T v) {
  v += dpp_of<0x111, 0xf>(v);  // row_shr:1, 2, 4, 8
  v += dpp_of<0x112, 0xf>(v);
  v += dpp_of<0x114, 0xf>(v);
  v += dpp_of<0x118, 0xf>(v);
  v += dpp_of<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp_of<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ double last_lane(double v) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                          __builtin_amdgcn_readlane(__double2loint(v), 63));
}
__device__ __forceinline__ long long last_lane(long long v) {
  return __double_as_longlong(last_lane(__longlong_as_double(v)));
}

}  // namespace tetra
