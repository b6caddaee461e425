// All-reduces inside groups of up to 16 lanes with DPP moves, and the choice of such a group for a token's experts.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace moe {

// Exchange with the partner lane of all-reduce stage `ST` inside a group of up to 16 lanes: neighbours, pairs, then the
// mirror image inside 8 and inside 16 (whose halves hold one value each by then).  DPP moves, no LDS round trip.
template <int ST> __device__ __forceinline__ unsigned dpp_partner(unsigned v) {
  constexpr int ctrl = ST == 0 ? 0xB1 : ST == 1 ? 0x4E : ST == 2 ? 0x141 : 0x140;
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, true);
}
template <int ST> __device__ __forceinline__ unsigned long long dpp_partner(unsigned long long v) {
  return ((unsigned long long)dpp_partner<ST>((unsigned)(v >> 32)) << 32) | dpp_partner<ST>((unsigned)v);
}
template <int ST> __device__ __forceinline__ float dpp_partner(float v) {
  return __uint_as_float(dpp_partner<ST>(__float_as_uint(v)));
}
// op over the G lanes of a group; every lane of the wave must be active
template <int G, typename T, typename Op> __device__ __forceinline__ T group_reduce(T v, Op op) {
  static_assert(G <= 16, "a group lies inside one DPP row");
  if constexpr (G >= 2) v = op(v, dpp_partner<0>(v));
  if constexpr (G >= 4) v = op(v, dpp_partner<1>(v));
  if constexpr (G >= 8) v = op(v, dpp_partner<2>(v));
  if constexpr (G >= 16) v = op(v, dpp_partner<3>(v));
  return v;
}
template <int G> __device__ __forceinline__ float group_sum(float v) { return group_reduce<G>(v, [](float a, float b) { return a + b; }); }
template <int G> __device__ __forceinline__ float group_max(float v) { return group_reduce<G>(v, [](float a, float b) { return fmaxf(a, b); }); }

// lanes per token G = min(16, pow2 >= E) (so G >= k: one slot per lane); experts beyond 16 go VPL per lane
template <typename F> int with_group(int E, F f) {
  if (E <= 1) return f(std::integral_constant<int, 1>(), std::integral_constant<int, 1>());
  if (E <= 2) return f(std::integral_constant<int, 2>(), std::integral_constant<int, 1>());
  if (E <= 4) return f(std::integral_constant<int, 4>(), std::integral_constant<int, 1>());
  if (E <= 8) return f(std::integral_constant<int, 8>(), std::integral_constant<int, 1>());
  if (E <= 16) return f(std::integral_constant<int, 16>(), std::integral_constant<int, 1>());
  if (E <= 32) return f(std::integral_constant<int, 16>(), std::integral_constant<int, 2>());
  if (E <= 64) return f(std::integral_constant<int, 16>(), std::integral_constant<int, 4>());
  if (E <= 128) return f(std::integral_constant<int, 16>(), std::integral_constant<int, 8>());
  return f(std::integral_constant<int, 16>(), std::integral_constant<int, 16>());
}

}  // namespace moe
