// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) and the draws built on it.
//
// A round maps counter (c0,c1,c2,c3) and key (k0,k1) to
//   (hi(M1 c2) ^ c1 ^ k0, lo(M1 c2), hi(M0 c0) ^ c3 ^ k1, lo(M0 c0)),
// M0 = 0xD2511F53, M1 = 0xCD9E8D57, and the key is bumped by the Weyl
// constants (0x9E3779B9, 0xBB67AE85) between rounds.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sd {

enum : uint32_t {
  TAG_INIT = 1,
  TAG_DRAFT = 2,
  TAG_COIN = 3,
  TAG_USAMPLE = 4,
  TAG_RESID = 5,
  TAG_TARGET = 6
};

// a ^ b ^ c in one instruction (truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                        uint64_t seed) {
  uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    // one 32x32 -> 64-bit product per multiplier (a single v_mad_u64_u32)
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
    const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
    // (the first round's n0 is the same for every counter c0: left to the scalar unit)
    const uint32_t n0 = r == 0 ? hi1 ^ c1 ^ k0 : xor3(hi1, c1, k0), n2 = xor3(hi0, c3, k1);
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return make_uint4(c0, c1, c2, c3);
}

__device__ __forceinline__ uint32_t pick(const uint4& w, int i) {
  return i == 0 ? w.x : i == 1 ? w.y : i == 2 ? w.z : w.w;
}

// 24-bit uniform in (0, 1), exact in float64.
__device__ __forceinline__ double uniform64(uint32_t w) {
  return ((double)(w >> 8) + 0.5) * 0x1p-24;
}

// -2 ln u for the 24-bit uniform u = (m + 0.5) 2^-24 of word w, in float32
// without losing the small-radius tail.  v = fl(u) is exact for u < 1/2; e = u -
// v (0 or 2^-25 either way) is exact by the two subtractions, and ln u = ln v +
// e/v, where e/v = e (1 + s + s^2) with s = 1 - v: e is not 0 only for v in
// [1/2, 1], where that is within 2^-27 of it.  v is a normal number below or at
// 1, so the hardware logarithm (base 2, about 1 ulp) needs no scaling.  Its product
// with ln 2 is compensated in the standard way: the constant in two floats (ln 2
// rounded, and what the rounding left), the product's own rounding error from a
// fused multiply-add (Dekker's product; Numer. Math. 18 (1971)).
__device__ __forceinline__ float neg2log_u24(uint32_t w) {
  constexpr float kHi = -2.0f * 0x1.62e42ep-1f, kLo = -2.0f * 0x1.efa39ep-25f;  // -2 ln 2
  const float m = (float)(w >> 8) * 0x1p-24f;
  const float v = m + 0x1p-25f;
  const float e = -2.0f * ((m - v) + 0x1p-25f), s = 1.0f - v;
  const float y = __builtin_amdgcn_logf(v);
  const float h = y * kHi;
  const float l = __fmaf_rn(y, kLo, __fmaf_rn(y, kHi, -h)) + __fmaf_rn(e, __fmaf_rn(s, s, s), e);
  return __fmaf_rn(y, kHi, l);
}

// Box-Muller on (w0, w1) and (w2, w3): radius sqrt(-2 ln u_a), angle 2 pi u_b.
// The hardware sine and cosine take their argument in revolutions, so they
// evaluate sin(2 pi u_b), cos(2 pi u_b) directly on u_b in (0, 1); the radius
// uses the hardware square root (about 1 ulp; the argument is a normal
// float32 of at most 2 ln 2^25, so no range scaling is needed).
__device__ __forceinline__ float4 normals4(uint4 w) {
  const float ra = __builtin_amdgcn_sqrtf(neg2log_u24(w.x));
  const float rc = __builtin_amdgcn_sqrtf(neg2log_u24(w.z));
  const float ub = __fmaf_rn((float)(w.y >> 8), 0x1p-24f, 0x1p-25f);
  const float ud = __fmaf_rn((float)(w.w >> 8), 0x1p-24f, 0x1p-25f);
  return make_float4(ra * __builtin_amdgcn_cosf(ub), ra * __builtin_amdgcn_sinf(ub),
                     rc * __builtin_amdgcn_cosf(ud), rc * __builtin_amdgcn_sinf(ud));
}

// q + sigma xi of four coordinates (group g) of a plain Euler-Maruyama step:
// the TARGET stream's slot 1 of the chain's round n.
__device__ __forceinline__ float4 em_state(float4 q, float sigma, uint32_t g, uint32_t chain, uint32_t n,
                                           uint64_t seed) {
  const float4 z = normals4(philox(g, chain, n, (TAG_TARGET << 24) | 1u, seed));
  return make_float4(q.x + sigma * z.x, q.y + sigma * z.y, q.z + sigma * z.z, q.w + sigma * z.w);
}

__device__ __forceinline__ float get4(const float4& v, int i) {
  return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
}

}  // namespace sd
