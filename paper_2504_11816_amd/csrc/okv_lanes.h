// Exchanges and reductions inside a wavefront of 64 lanes (device code, gfx950).
#pragma once

#include <hip/hip_runtime.h>

namespace okv {

// Values of other lanes of a wavefront without the round trip through LDS that a shuffle is (some 50 ns, one after the other in
// every chain below).  The swaps exchange the odd rows of 16 lanes (the upper half of the wavefront) of one register with the even rows
// (the lower half) of another: of two copies of a value one then holds lane & ~16 (& ~32) of it in every lane, the other lane | 16 (| 32).
// Written as assembly: the compiler's builtin returned the first register twice.
// us, shuffles -> these: a layer of 32 sequences x 768 keys x 32 heads (d = 128) 61.2 -> 59.9, 16 ragged sequences of 32 heads with
// their joining launch 35.5 -> 33.5, a step of 4 layers of two long sequences of 32 / 8 heads 57 -> 55.5.
template <int X>
__device__ __forceinline__ void split_lanes(const float v, float &a, float &b) {
  static_assert(X == 16 || X == 32, "");
  a = v, b = v;
  if constexpr (X == 16) asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  else asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
template <int X>
__device__ __forceinline__ float max_with_lane_xor(const float v) {
  float a, b;
  split_lanes<X>(v, a, b);
  return fmaxf(a, b);
}
template <int X>
__device__ __forceinline__ float sum_with_lane_xor(const float v) {
  float a, b;
  split_lanes<X>(v, a, b);
  return a + b;
}
// the value CTRL lanes further in the row of 16 (row_ror: CTRL - 0x120)
template <int CTRL>
__device__ __forceinline__ float row_turned(const float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
// Over all 64 lanes, which all take part, in the order of a butterfly from lane ^ 32 to lane ^ 1 (a value that repeats every 2 n lanes is
// the same n lanes further as in lane ^ n)
__device__ __forceinline__ float wave_max(float v) {
  v = max_with_lane_xor<16>(max_with_lane_xor<32>(v));
  v = fmaxf(v, row_turned<0x128>(v));
  v = fmaxf(v, row_turned<0x124>(v));
  v = fmaxf(v, row_turned<0x122>(v));
  return fmaxf(v, row_turned<0x121>(v));
}
__device__ __forceinline__ float row_sum(float v) {      // over the lane's row of 16
  v += row_turned<0x128>(v);
  v += row_turned<0x124>(v);
  v += row_turned<0x122>(v);
  return v + row_turned<0x121>(v);
}
__device__ __forceinline__ float wave_sum(float v) { return row_sum(sum_with_lane_xor<16>(sum_with_lane_xor<32>(v))); }

}  // namespace okv
