// Sums and maxima over the 64 lanes of a wavefront without LDS: exchanges
// inside 16 lanes are DPP modifiers, those across 16 and 32 lanes the gfx950
// row swaps, so a step costs a few cycles instead of an LDS permute's round
// trip (two per float64 step).  Every step adds a lane and its mirror image,
// so all lanes end with the same bits, in a fixed order.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sd {

// DPP controls: lane ^ 1, lane ^ 2, 7 - lane (of 8), 15 - lane (of 16), lane ^ 8
// (a rotation of 16 by 8).
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140, kDppRor8 = 0x128;

template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = dpp32<CTRL>((uint32_t)u), hi = dpp32<CTRL>((uint32_t)(u >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, dpp32<CTRL>(__builtin_bit_cast(uint32_t, v)));
}

// Row swaps of a pair (a, b).  swap32: a = {a.lanes 0-31, b.lanes 0-31},
// b = {a.lanes 32-63, b.lanes 32-63}; swap16: the same with the even and odd
// 16-lane rows.  a + b afterwards is a reduce-scatter step: the lower lanes
// hold a's total over the pair of lanes, the upper ones b's.
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void swap16(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
template <bool ROW32>
__device__ __forceinline__ void swap_pair(double& a, double& b) {
  const uint64_t ua = __builtin_bit_cast(uint64_t, a), ub = __builtin_bit_cast(uint64_t, b);
  uint32_t al = (uint32_t)ua, ah = (uint32_t)(ua >> 32), bl = (uint32_t)ub, bh = (uint32_t)(ub >> 32);
  if constexpr (ROW32) {
    swap32(al, bl);
    swap32(ah, bh);
  } else {
    swap16(al, bl);
    swap16(ah, bh);
  }
  a = __builtin_bit_cast(double, ((uint64_t)ah << 32) | al);
  b = __builtin_bit_cast(double, ((uint64_t)bh << 32) | bl);
}
template <bool ROW32>
__device__ __forceinline__ double swap_add(double a, double b) {
  swap_pair<ROW32>(a, b);
  return a + b;
}
template <bool ROW32>
__device__ __forceinline__ double swap_max(double v) {
  double w = v;
  swap_pair<ROW32>(v, w);
  return fmax(v, w);
}

// Sum over each aligned group of n lanes (a power of two from 4 to 64, the same
// in the whole wavefront), in every lane of it.
__device__ __forceinline__ double group_sum(double v, int n) {
  v += dpp<kDppXor1>(v);
  v += dpp<kDppXor2>(v);
  if (n >= 8) v += dpp<kDppHalfMirror>(v);
  if (n >= 16) v += dpp<kDppMirror>(v);
  if (n >= 32) v = swap_add<false>(v, v);
  if (n >= 64) v = swap_add<true>(v, v);
  return v;
}
__device__ __forceinline__ double wave_sum(double v) { return group_sum(v, 64); }

// Maximum over each such group.
__device__ __forceinline__ double group_max(double v, int n) {
  v = fmax(v, dpp<kDppXor1>(v));
  v = fmax(v, dpp<kDppXor2>(v));
  if (n >= 8) v = fmax(v, dpp<kDppHalfMirror>(v));
  if (n >= 16) v = fmax(v, dpp<kDppMirror>(v));
  if (n >= 32) v = swap_max<false>(v);
  if (n >= 64) v = swap_max<true>(v);
  return v;
}

}  // namespace sd
