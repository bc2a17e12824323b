// Lane exchanges of FP64 values within a wavefront of 64 without the LDS pipe:
// row operations (16 lanes) and the gfx950 row swaps.
#pragma once
#include <hip/hip_runtime.h>

namespace mgl {

constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppRor4 = 0x124, kDppRor8 = 0x128, kDppHalfMirror = 0x141;

template <int CTRL>
__device__ __forceinline__ double lane_dpp(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double lane_pair(unsigned lo, unsigned hi) {
  return __longlong_as_double(((long long)hi << 32) | lo);
}
// v + the value of the lane 16 (32) away, in both
__device__ __forceinline__ double lane_add16(double v) {
  const long long b = __double_as_longlong(v);
  const auto l = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
  const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return lane_pair(l[0], h[0]) + lane_pair(l[1], h[1]);
}
__device__ __forceinline__ double lane_add32(double v) {
  const long long b = __double_as_longlong(v);
  const auto l = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
  const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return lane_pair(l[0], h[0]) + lane_pair(l[1], h[1]);
}
// v of one lane, in every lane (a scalar)
__device__ __forceinline__ double lane_get(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// sum over the wavefront, in every lane (a fixed order)
__device__ __forceinline__ double wave_sum(double v) {
  v += lane_dpp<kDppXor1>(v);
  v += lane_dpp<kDppXor2>(v);
  v += lane_dpp<kDppHalfMirror>(v);
  v += lane_dpp<kDppRor8>(v);
  return lane_add32(lane_add16(v));
}

}  // namespace mgl
