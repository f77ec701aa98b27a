// Lane broadcasts of binary64 values within a wavefront of four rows of 16
// lanes (no LDS), and fast reciprocals: the parts of the kernels that factor a
// 16 x 16 block in registers.
#pragma once

#include <hip/hip_runtime.h>

namespace rrf {
namespace {

// Lane J of the own row of 16 lanes (DPP row_newbcast).
template <int J>
__device__ __forceinline__ double row_lane(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)u, 0x150 + J, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), 0x150 + J, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// The value of the lane's column in lane row Q, in every lane row: the halves
// of the value share the swaps (wavefront halves, then odd and even rows,
// then the wavefront halves again).
template <int Q>
__device__ __forceinline__ double row_of(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const auto a = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)(u >> 32), false, false);
  const unsigned y = (Q & 2) ? a[1] : a[0];     // lane rows lo, lo, hi, hi of Q's half
  const auto b = __builtin_amdgcn_permlane16_swap(y, y, false, false);
  const unsigned z = (Q & 1) ? b[1] : b[0];     // row Q: lo, lo, hi, hi
  const auto c = __builtin_amdgcn_permlane32_swap(z, z, false, false);
  return __longlong_as_double((long long)(((unsigned long long)c[1] << 32) | c[0]));
}
// Lane L's value, uniform.
template <int L>
__device__ __forceinline__ double lane_value(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)u, L);
  const int hi = __builtin_amdgcn_readlane((int)(u >> 32), L);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// 1 / sqrt(v) and 1 / v to about an ulp for normal v: the hardware estimate
// (at least 2^-14 relative) and two Newton steps (relative error e to 0.6 e^3
// and e^2).
__device__ __forceinline__ double fast_rsqrt(double v) {
  double y = __builtin_amdgcn_rsq(v);
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const double e = fma(-(v * y), y, 1.0);
    y = fma(y * e, fma(0.375, e, 0.5), y);
  }
  return y;
}
__device__ __forceinline__ double fast_rcp(double v) {
  double y = __builtin_amdgcn_rcp(v);
#pragma unroll
  for (int it = 0; it < 2; ++it) y = fma(fma(-v, y, 1.0), y, y);
  return y;
}

}  // namespace
}  // namespace rrf
