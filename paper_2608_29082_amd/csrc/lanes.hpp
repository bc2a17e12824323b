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

// An unevaluated sum hi + lo of two doubles: sums of products kept this way round once, at the end, to
// about twice the FP64 precision, so they do not depend on the order of their terms (the same bits from
// sweeps that walk rows, tiles or columns).
struct Sum2 {
  double hi, lo;
};
// The sum, rounded.  hi is the plain FP64 sum of the terms; once it is infinite or NaN its error term lo is
// NaN, and hi alone is the result.
__device__ __forceinline__ double sum2_value(Sum2 s) { return __builtin_isfinite(s.lo) ? s.hi + s.lo : s.hi; }
// s + v (Knuth's two-sum; the error of hi goes to lo)
__device__ __forceinline__ Sum2 sum2_add(Sum2 s, double v) {
  const double h = s.hi + v, t = h - s.hi;
  return Sum2{h, s.lo + ((s.hi - (h - t)) + (v - t))};
}
__device__ __forceinline__ Sum2 sum2_add(Sum2 a, Sum2 b) {
  Sum2 s = sum2_add(a, b.hi);
  s.lo += b.lo;
  return s;
}
template <int CTRL>
__device__ __forceinline__ Sum2 lane_dpp(Sum2 v) {
  return Sum2{lane_dpp<CTRL>(v.hi), lane_dpp<CTRL>(v.lo)};
}
// the pair of values 16 (32) lanes apart, as (one, other) in both lanes
__device__ __forceinline__ Sum2 lane_sum16(Sum2 v) {
  const long long h = __double_as_longlong(v.hi), l = __double_as_longlong(v.lo);
  const auto a = __builtin_amdgcn_permlane16_swap((unsigned)h, (unsigned)h, false, false);
  const auto b = __builtin_amdgcn_permlane16_swap((unsigned)(h >> 32), (unsigned)(h >> 32), false, false);
  const auto c = __builtin_amdgcn_permlane16_swap((unsigned)l, (unsigned)l, false, false);
  const auto d = __builtin_amdgcn_permlane16_swap((unsigned)(l >> 32), (unsigned)(l >> 32), false, false);
  return sum2_add(Sum2{lane_pair(a[0], b[0]), lane_pair(c[0], d[0])}, Sum2{lane_pair(a[1], b[1]), lane_pair(c[1], d[1])});
}
__device__ __forceinline__ Sum2 lane_sum32(Sum2 v) {
  const long long h = __double_as_longlong(v.hi), l = __double_as_longlong(v.lo);
  const auto a = __builtin_amdgcn_permlane32_swap((unsigned)h, (unsigned)h, false, false);
  const auto b = __builtin_amdgcn_permlane32_swap((unsigned)(h >> 32), (unsigned)(h >> 32), false, false);
  const auto c = __builtin_amdgcn_permlane32_swap((unsigned)l, (unsigned)l, false, false);
  const auto d = __builtin_amdgcn_permlane32_swap((unsigned)(l >> 32), (unsigned)(l >> 32), false, false);
  return sum2_add(Sum2{lane_pair(a[0], b[0]), lane_pair(c[0], d[0])}, Sum2{lane_pair(a[1], b[1]), lane_pair(c[1], d[1])});
}
__device__ __forceinline__ Sum2 wave_sum(Sum2 v) {
  v = sum2_add(v, lane_dpp<kDppXor1>(v));
  v = sum2_add(v, lane_dpp<kDppXor2>(v));
  v = sum2_add(v, lane_dpp<kDppHalfMirror>(v));
  v = sum2_add(v, lane_dpp<kDppRor8>(v));
  return lane_sum32(lane_sum16(v));
}

}  // namespace mgl
