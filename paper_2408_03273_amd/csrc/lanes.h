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

}  // namespace mpe
