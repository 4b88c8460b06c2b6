// Four-coordinate row access and the Free-Drafter recursion, shared by the
// standalone draft kernel and the sampler's fused advance kernel.
#pragma once

#include "common.hpp"
#include "philox.hpp"

namespace sd {

__device__ __forceinline__ void load4(const float* p, int cnt, bool vec, float (&v)[4]) {
  if (vec) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = c < cnt ? p[c] : 0.0f;
  }
}

// stream: a non-temporal store of an aligned vector (see stream_rows).
__device__ __forceinline__ void store4(float* p, int cnt, bool vec, const float (&v)[4],
                                      bool stream = false) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  if (vec && stream) {
    const f32x4 t = {v[0], v[1], v[2], v[3]};
    __builtin_nontemporal_store(t, reinterpret_cast<f32x4*>(p));
  } else if (vec) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (c < cnt) p[c] = v[c];
  }
}

// Per-step (c1, c2, sigma, 1/c2): from the target's float32 table when given,
// else evaluated from the schedule in float64 and rounded.
__device__ __forceinline__ float4 step_coef(const Sched& sc, const float4* __restrict__ coef, int n) {
  if (coef) return coef[n];
  const double c2 = sched_c2(sc, n);
  return make_float4((float)sched_c1(sc, n), (float)c2, (float)sched_sigma(sc, n), (float)(1.0 / c2));
}

// The Free Drafter's mean m^p = c1_n yhat + c2s sv with c2s = c2_n / c2_c and
// sv = c2_c S_c, in one fixed sequence of float32 operations (the product,
// then one fused multiply-add), so that every kernel that needs m^p recomputes
// the same bits as the draft that produced yhat.
__device__ __forceinline__ float draft_mean(float c1, float y, float c2s, float sv) {
  return __fmaf_rn(c1, y, c2s * sv);
}

// The next block's per-step coefficients (c1, c2 * scale, sigma, -) for a
// workgroup: entry i - 1 belongs to step n = k + i - 1 of draft row i.  One
// thread per step evaluates them (or reads the table), once per workgroup
// instead of once per thread and step: in float64 they cost as much as a
// step's normals.  The caller's barrier comes before draft_rows.  (1024 blocks
// of 8 x 3072, the schedule evaluated here: 47.6 -> 37.1 us, with the normals
// of four rows drawn at a time; both written blocks streamed, 51.9 -> 43.8 us
// a call, 5.5 TB/s.)
__device__ __forceinline__ void draft_coefs(const Sched& sc, const float4* __restrict__ coef, int k, int kb,
                                            float scale, float4* lds) {
  for (int i = threadIdx.x; i < kb; i += blockDim.x) {
    const float4 cf = step_coef(sc, coef, k + i);
    lds[i] = make_float4(cf.x, cf.y * scale, cf.z, 0.0f);
  }
}

// Draft rows 1..K of one chain for coordinates e0..e0+3 (group g), starting
// at yhat_0 = yv (already stored as row 0 by the caller) with the kb valid
// drafts whose coefficients are in lds (Sec. 3.3):
//   m^p_{i-1} = c1_n yhat_{i-1} + c2_n S_c,  yhat_i = m^p_{i-1} + sigma_n xi_i,
// where c2_n S_c = (c2_n * scale) * sv; rows past K_b repeat the last draft
// and mean so that every row the target call reads is finite.  mb may be
// null (the sampler recomputes m^p where it needs it, see draft_mean).
// stream: the rows are written with non-temporal stores (stream_rows).
// Four rows' normals are drawn at a time: they do not depend on the state, so
// their chains of 32-bit multiplies overlap.
__device__ __forceinline__ void draft_rows(const float4* lds, int K, int kb, uint32_t chain, uint32_t rnd,
                                           uint64_t seed, int g, float (&yv)[4], const float (&sv)[4],
                                           float* xb, int64_t xr, float* mb, int64_t mr, int cnt, bool vec,
                                           bool stream) {
  float m[4] = {0.f, 0.f, 0.f, 0.f};
  constexpr int U = 4;
  for (int i0 = 1; i0 <= kb; i0 += U) {
    float4 z[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      z[u] = normals4(philox((uint32_t)g, chain, rnd, (TAG_DRAFT << 24) | (uint32_t)(i0 + u), seed));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u;
      if (i > kb) break;
      const float4 cf = lds[i - 1];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        m[c] = draft_mean(cf.x, yv[c], cf.y, sv[c]);
        yv[c] = m[c] + cf.z * get4(z[u], c);
      }
      if (mb) store4(mb + (int64_t)(i - 1) * mr, cnt, vec, m, stream);
      store4(xb + (int64_t)i * xr, cnt, vec, yv, stream);
    }
  }
  for (int i = kb + 1; i <= K; ++i) {
    if (mb) store4(mb + (int64_t)(i - 1) * mr, cnt, vec, m, stream);
    store4(xb + (int64_t)i * xr, cnt, vec, yv, stream);
  }
}

// The draft row of a block of one (K = 1), whose coefficients each thread evaluates:
// shared through LDS they cost the barrier and save nothing (60000 blocks of 1 x 16:
// 40.0 -> 31.4 us a call, 35.0 with the coefficients of every row on each thread).
__device__ __forceinline__ void draft_single(float4 cf, float scale, uint32_t chain, uint32_t rnd, uint64_t seed,
                                             int g, const float (&yv)[4], const float (&sv)[4], float* x1,
                                             float* mb, int cnt, bool vec, bool stream) {
  const float4 z = normals4(philox((uint32_t)g, chain, rnd, (TAG_DRAFT << 24) | 1u, seed));
  const float c2 = cf.y * scale;
  float m[4], y[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    m[c] = draft_mean(cf.x, yv[c], c2, sv[c]);
    y[c] = m[c] + cf.z * get4(z, c);
  }
  if (mb) store4(mb, cnt, vec, m, stream);
  store4(x1, cnt, vec, y, stream);
}

// Draft rows of few chains, by a workgroup of four wavefronts over the same 64
// groups of coordinates (g, one per lane): a launch of fewer wavefronts than
// SIMDs takes as long as one thread's serial draws, so each wavefront draws the
// normals of every fourth row into zs, all four walk the recursion, and each
// stores the rows it drew.  The first barrier also orders the callers' reads of
// the chain's rows before these stores, and publishes their coefs (draft_coefs).
// Same arithmetic as draft_rows.
constexpr int kSpreadRows = 16;
__device__ __forceinline__ void draft_rows_spread(const float4* coefs, float4 (*zs)[64], int K, int kb,
                                                  uint32_t chain, uint32_t rnd, uint64_t seed, int g,
                                                  float (&yv)[4], const float (&sv)[4], float* xb, int64_t xr,
                                                  float* mb, int64_t mr, int cnt, bool vec, bool stream) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  float m[4] = {0.f, 0.f, 0.f, 0.f};
  for (int i0 = 1; i0 <= kb; i0 += kSpreadRows) {
    if (i0 > 1) __syncthreads();  // the previous rows' normals are consumed
#pragma unroll
    for (int u = 0; u < kSpreadRows / 4; u += 2) {
      if (i0 + w + 4 * u > kb) break;
      // (two rows at a time, the second perhaps past the block: their chains overlap)
      const float4 za = normals4(philox((uint32_t)g, chain, rnd, (TAG_DRAFT << 24) | (uint32_t)(i0 + w + 4 * u), seed));
      const float4 zb = normals4(philox((uint32_t)g, chain, rnd, (TAG_DRAFT << 24) | (uint32_t)(i0 + w + 4 * u + 4), seed));
      zs[w + 4 * u][lane] = za;
      zs[w + 4 * u + 4][lane] = zb;
    }
    __syncthreads();
    for (int i = i0; i <= min(kb, i0 + kSpreadRows - 1); ++i) {
      const float4 z = zs[i - i0][lane], cf = coefs[i - 1];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        m[c] = draft_mean(cf.x, yv[c], cf.y, sv[c]);
        yv[c] = m[c] + cf.z * get4(z, c);
      }
      if (((i - 1) & 3) != w) continue;
      if (mb) store4(mb + (int64_t)(i - 1) * mr, cnt, vec, m, stream);
      store4(xb + (int64_t)i * xr, cnt, vec, yv, stream);
    }
  }
  for (int i = kb + 1; i <= K; ++i) {
    if (((i - 1) & 3) != w) continue;
    if (mb) store4(mb + (int64_t)(i - 1) * mr, cnt, vec, m, stream);
    store4(xb + (int64_t)i * xr, cnt, vec, yv, stream);
  }
}

// Whether a draft of B blocks of K rows in d coordinates is spread: at one
// wavefront per 64 groups it would leave SIMDs (1024 on the chip) without any.
// (advance 8 x 8 x 3072, 96 wavefronts: 7.5 -> 6.0 us; draft 300 x 20 x 64: 24.7
// -> 9.9 a call with the coefficients of draft_coefs; at 256 x 8 x 784, 1024
// wavefronts, 11.7 us either way.)
inline bool spread_rows(int B, int K, int d) {
  return K > 1 && (int64_t)B * (((d + 3) / 4 + 63) / 64) <= 1024;
}

}  // namespace sd
