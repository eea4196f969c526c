// Small FP64 linear algebra inside one wavefront: a column per lane, another
// lane's entry by a cross-lane move.
#pragma once

#include <cstdint>
#include <type_traits>
#include <utility>

#include <hip/hip_runtime.h>

namespace tk {

// x of lane N of this lane's row of 16 (one 64-bit move)
template <int N>
__device__ __forceinline__ double row_bcast(double x) {
  return __builtin_amdgcn_mov_dpp(x, 0x150 + N, 0xf, 0xf, true);
}

// x of lane l (l wave-uniform)
__device__ __forceinline__ double lane_value(double x, int l) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)(unsigned)(v & 0xffffffffLL), l);
  const int hi = __builtin_amdgcn_readlane((int)(v >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Calls f(integral constant 0 .. N-1).
template <int... I, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

}  // namespace tk
