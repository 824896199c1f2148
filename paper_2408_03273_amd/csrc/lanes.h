// Sums across the lanes of a wave (device code).
#pragma once
#include <hip/hip_runtime.h>

namespace mpe {

// x of the lower and y of the upper half wave, each summed over both halves
__device__ __forceinline__ double fold32(double x, double y) {
  const unsigned long long a = __double_as_longlong(x), b = __double_as_longlong(y);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)(a & 0xffffffffu), (unsigned)(b & 0xffffffffu), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
  return __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
         __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}

// x of the even and y of the odd rows of 16 lanes, each summed over a row pair
__device__ __forceinline__ double fold16(double x, double y) {
  const unsigned long long a = __double_as_longlong(x), b = __double_as_longlong(y);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)(a & 0xffffffffu), (unsigned)(b & 0xffffffffu), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
  return __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
         __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}

// sum over the 16 lanes of a row, in every lane (rotations by 8, 4, 2, 1)
template <int CTRL>
__device__ __forceinline__ double row_rotate(double v) {
  const unsigned long long b = __double_as_longlong(v);
  const int lo = (int)(unsigned)(b & 0xffffffffu), hi = (int)(unsigned)(b >> 32);
  const unsigned l2 = (unsigned)__builtin_amdgcn_update_dpp(0, lo, CTRL, 0xf, 0xf, true);
  const unsigned h2 = (unsigned)__builtin_amdgcn_update_dpp(0, hi, CTRL, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)h2 << 32) | l2));
}

__device__ __forceinline__ double row_sum(double v) {
  v += row_rotate<0x128>(v);
  v += row_rotate<0x124>(v);
  v += row_rotate<0x122>(v);
  v += row_rotate<0x121>(v);
  return v;
}

}  // namespace mpe
