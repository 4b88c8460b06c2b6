// Free Drafter (Sec. 3.3), chain initialisation and per-round bookkeeping.
//
// The draft recursion is sequential in the draft step i but independent across
// the d coordinates, so each thread owns four consecutive coordinates of one
// chain and walks i = 1..K_b keeping yhat in registers: the state is read once
// and every draft row and draft mean is written once (HBM-bound, no reuse).
#include "common.hpp"
#include "philox.hpp"
#include "rows.hpp"

namespace sd {
namespace {

constexpr int kThreads = 256;

__global__ __launch_bounds__(kThreads) void init_chains_kernel(int d, uint64_t seed, float* y,
                                                               bool vec) {
  const int b = blockIdx.y;
  const int g = blockIdx.x * kThreads + threadIdx.x;
  const int e0 = 4 * g;
  if (e0 >= d) return;
  const float4 z = normals4(philox((uint32_t)g, (uint32_t)b, 0u, TAG_INIT << 24, seed));
  const float v[4] = {z.x, z.y, z.z, z.w};
  const int cnt = min(4, d - e0);
  store4(y + (int64_t)b * d + e0, cnt, vec && cnt == 4, v);
}

// A new run's state in one launch: Y_0 into y and into row 0 of the chain's x
// block, and the bookkeeping of every chain (its first workgroup) and of the
// run (the first workgroup of all): a launch each took 2 us apiece.
__global__ __launch_bounds__(kThreads) void sampler_init_kernel(
    Sched sc, int B, int K, int d, uint64_t seed, float* __restrict__ y, float* __restrict__ x,
    bool vec, int32_t* __restrict__ k2, uint32_t* __restrict__ rnd2, int32_t* __restrict__ crow2,
    int32_t* __restrict__ cstep2, int32_t* __restrict__ hist, int64_t* __restrict__ steps,
    int32_t* __restrict__ ties, int32_t* __restrict__ tau, int32_t* __restrict__ step,
    double* __restrict__ sigma, int32_t* __restrict__ act, int32_t* __restrict__ nan) {
  const int b = blockIdx.y, K1 = K + 1, t = threadIdx.x;
  if (blockIdx.x == 0) {
    if (t < 2) {
      k2[t * B + b] = 0;
      rnd2[t * B + b] = 0u;
      crow2[t * B + b] = 0;
      cstep2[t * B + b] = 0;
    }
    if (t == 2) {
      steps[b] = 0;
      ties[b] = 0;
      tau[b] = 0;
    }
    if (b == 0 && t < 4) act[t] = t % 2 == 0 ? 1 : 0;  // [group][round parity]: round 0 is active
    if (b == 0 && t == 4) *nan = 0;
    if (t >= 64 && t < 64 + SD_MAX_BLOCK + 2) hist[(int64_t)b * (SD_MAX_BLOCK + 2) + t - 64] = 0;
    if (t >= 64 && t < 64 + K1) {
      const int j = t - 64;
      step[(int64_t)b * K1 + j] = min(j, sc.N - 1);
      sigma[(int64_t)b * K1 + j] = sched_sigma(sc, min(j, sc.N));
    }
  }
  const int g = blockIdx.x * kThreads + t;
  const int e0 = 4 * g;
  if (e0 >= d) return;
  const float4 z = normals4(philox((uint32_t)g, (uint32_t)b, 0u, TAG_INIT << 24, seed));
  const float v[4] = {z.x, z.y, z.z, z.w};
  const int cnt = min(4, d - e0);
  store4(y + (int64_t)b * d + e0, cnt, vec && cnt == 4, v);
  store4(x + (int64_t)b * K1 * d + e0, cnt, vec && cnt == 4, v);
}

// Draft block of one chain, four coordinates per thread.  The cached target
// score enters only as c2_n S_c.  With CACHE_FROM_MEANS the score is not
// stored: it is the score behind the target mean m^q_c = c1_c x_c + c2_c S_c
// of row crow of the previous round (step cstep), so
//   c2_n S_c = (c2_n / c2_c) (m^q_c - c1_c x_c),
// read from the same x / mq buffers before this chain's rows are overwritten
// (each thread reads and then writes only its own coordinates).  SINGLE: blocks of
// one row (draft_single).
template <bool CACHE_FROM_MEANS, bool SPREAD, bool SINGLE = false>
__global__ __launch_bounds__(kThreads) void draft_kernel(
    Sched sc, const float4* __restrict__ coef, int K, int d, const float* __restrict__ y,
    const float* __restrict__ cs,
    const int32_t* __restrict__ crow, const int32_t* __restrict__ cstep,
    const float* __restrict__ mqprev, int64_t qc, int64_t qr, const int32_t* __restrict__ kk,
    const uint32_t* __restrict__ rnd, uint64_t seed, float* __restrict__ x, int64_t xc,
    int64_t xr, float* __restrict__ mp, int64_t mc, int64_t mr, float* __restrict__ svout,
    bool vec_ok, bool stream, const int* gate, int chain0) {
  if (gate && *gate == 0) return;
  __shared__ float4 cfs[SD_MAX_BLOCK];
  __shared__ float4 zs[SPREAD ? kSpreadRows : 1][64];
  const int b = blockIdx.y;
  const int k = kk[b];
  if (k >= sc.N) return;
  const int kb = min(K, sc.N - k);
  const uint32_t r = rnd[b];
  const float4 cc = CACHE_FROM_MEANS ? step_coef(sc, coef, cstep[b]) : make_float4(0.f, 0.f, 0.f, 1.0f);
  if constexpr (!SINGLE) {
    draft_coefs(sc, coef, k, kb, cc.w, cfs);
    if (!SPREAD) __syncthreads();
  }
  // SPREAD: the four wavefronts share 64 groups (draft_rows_spread); what is
  // written once, the first one writes
  const bool first = !SPREAD || threadIdx.x < 64;
  const int g = SPREAD ? blockIdx.x * 64 + (threadIdx.x & 63) : blockIdx.x * kThreads + threadIdx.x;
  const int e0 = 4 * g;
  if (!SPREAD && e0 >= d) return;
  const int cnt = max(0, min(4, d - e0));
  const bool vec = vec_ok && cnt == 4;
  float yv[4], sv[4];
  float* xb = x + (int64_t)b * xc + e0;
  float* mb = mp ? mp + (int64_t)b * mc + e0 : nullptr;
  load4(y + (int64_t)b * d + e0, cnt, vec, yv);
  if (CACHE_FROM_MEANS) {
    const int cr = crow[b];
    float xcv[4], qcv[4];
    load4(xb + (int64_t)cr * xr, cnt, vec, xcv);
    load4(mqprev + (int64_t)b * qc + (int64_t)cr * qr + e0, cnt, vec, qcv);
#pragma unroll
    for (int c = 0; c < 4; ++c) sv[c] = qcv[c] - cc.x * xcv[c];  // c2_c S_c
    if (svout && first) store4(svout + (int64_t)b * d + e0, cnt, vec, sv);
  } else {
    load4(cs + (int64_t)b * d + e0, cnt, vec, sv);
  }
  if constexpr (SPREAD) {
    float y0[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) y0[c] = yv[c];
    draft_rows_spread(cfs, zs, K, kb, (uint32_t)(chain0 + b), r, seed, g, yv, sv, xb, xr, mb, mr, cnt, vec, stream);
    if (first) store4(xb, cnt, vec, y0, stream);
  } else if constexpr (SINGLE) {
    store4(xb, cnt, vec, yv, stream);
    draft_single(step_coef(sc, coef, k), cc.w, (uint32_t)(chain0 + b), r, seed, g, yv, sv, xb + xr, mb,
                 cnt, vec, stream);
  } else {
    store4(xb, cnt, vec, yv, stream);
    draft_rows(cfs, K, kb, (uint32_t)(chain0 + b), r, seed, g, yv, sv, xb, xr, mb, mr, cnt, vec, stream);
  }
}

__global__ void fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ __launch_bounds__(kThreads) void chains_active_kernel(int B, int split, int N,
                                                                const int32_t* __restrict__ k,
                                                                int* f0, int* f1) {
  __shared__ int any[2];
  if (threadIdx.x < 2) any[threadIdx.x] = 0;
  __syncthreads();
  int a0 = 0, a1 = 0;
  for (int b = threadIdx.x; b < B; b += kThreads) {
    const int on = k[b] < N ? 1 : 0;
    if (b < split)
      a0 |= on;
    else
      a1 |= on;
  }
  if (a0) atomicOr(&any[0], 1);
  if (a1) atomicOr(&any[1], 1);
  __syncthreads();
  if (threadIdx.x == 0) {
    *f0 = any[0];
    *f1 = any[1];
  }
}

// Totals over the chains, one workgroup each: stats[c] for c <= SD_MAX_BLOCK + 1
// the rounds with tau = c, then steps advanced and tied coins.
__global__ __launch_bounds__(kThreads) void sampler_totals_kernel(int B, const int32_t* __restrict__ hist,
                                                                  const int64_t* __restrict__ steps,
                                                                  const int32_t* __restrict__ ties,
                                                                  int64_t* __restrict__ stats) {
  constexpr int H = SD_MAX_BLOCK + 2;
  const int c = blockIdx.x;
  int64_t v = 0;
#pragma unroll 4
  for (int b = threadIdx.x; b < B; b += kThreads)
    v += c < H ? (int64_t)hist[(int64_t)b * H + c] : c == H ? steps[b] : (int64_t)ties[b];
  __shared__ long long red[kThreads / 64];
  long long t = v;
  for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < kThreads / 64; ++i) t += red[i];
    stats[c] = t;
  }
}

// The totals, the non-finite flag and the groups' gates into mapped host
// words, then the tag that the host polls.
__global__ __launch_bounds__(128) void sampler_publish_kernel(const int64_t* __restrict__ stats,
                                                              const int32_t* __restrict__ nan,
                                                              const int32_t* __restrict__ act, int parity,
                                                              int64_t* host, int64_t tag) {
  const int t = threadIdx.x;
  if (t < kStatNan) host[t] = stats[t];
  if (t == kStatNan) host[t] = *nan;
  if (t == kStatGate || t == kStatGate + 1) host[t] = act[2 * (t - kStatGate) + parity];
  __threadfence_system();
  __syncthreads();
  if (t == 0) __atomic_store_n(host + kStatTag, tag, __ATOMIC_RELEASE);
}

__global__ void philox_words_kernel(uint64_t seed, int n, const uint32_t* ctr, uint32_t* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint4 w = philox(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3], seed);
  out[4 * i] = w.x;
  out[4 * i + 1] = w.y;
  out[4 * i + 2] = w.z;
  out[4 * i + 3] = w.w;
}

__global__ void philox_normals_kernel(uint64_t seed, uint32_t chain, uint32_t rnd, uint32_t c3,
                                      int d, float* out) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  const int e0 = 4 * g;
  if (e0 >= d) return;
  const float4 z = normals4(philox((uint32_t)g, chain, rnd, c3, seed));
  for (int c = 0; c < min(4, d - e0); ++c) out[e0 + c] = get4(z, c);
}

}  // namespace

hipError_t init_chains_launch(int B, int d, uint64_t seed, float* y, hipStream_t s) {
  const int ng = (d + 3) / 4;
  return launch_timed("init_chains", init_chains_kernel, dim3((ng + kThreads - 1) / kThreads, B), dim3(kThreads), s,
                      d, seed, y, d % 4 == 0 && aligned16(y));
}

hipError_t sampler_init_launch(const Sched& sc, int B, int K, int d, uint64_t seed, float* y, float* x,
                               int32_t* k2, uint32_t* rnd2, int32_t* crow2, int32_t* cstep2,
                               int32_t* hist, int64_t* steps, int32_t* ties, int32_t* tau,
                               int32_t* step, double* sigma, int32_t* act, int32_t* nan, hipStream_t s) {
  const int ng = (d + 3) / 4;
  return launch_timed("init_chains", sampler_init_kernel, dim3((ng + kThreads - 1) / kThreads, B), dim3(kThreads), s,
                      sc, B, K, d, seed, y, x, d % 4 == 0 && aligned16(y) && aligned16(x), k2, rnd2, crow2, cstep2,
                      hist, steps, ties, tau, step, sigma, act, nan);
}

hipError_t sampler_finish_launch(int B, const int32_t* hist, const int64_t* steps, const int32_t* ties,
                                 const int32_t* nan, const int32_t* act, int parity, int64_t* stats,
                                 int64_t* host, int64_t tag, hipStream_t s) {
  sampler_totals_kernel<<<SD_MAX_BLOCK + 4, kThreads, 0, s>>>(B, hist, steps, ties, stats);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  sampler_publish_kernel<<<1, 128, 0, s>>>(stats, nan, act, parity, host, tag);
  return hipGetLastError();
}

static bool draft_vec(int d, sd_stride xs, sd_stride mps, const float* y, const float* x,
                      const float* mp) {
  return (d % 4 == 0) && (xs.chain % 4 == 0) && (xs.row % 4 == 0) && (mps.chain % 4 == 0) &&
         (mps.row % 4 == 0) && aligned16(y) && aligned16(x) && aligned16(mp);
}

hipError_t draft_launch(const Sched& sc, int B, int K, int d, const float* y, const float* cs,
                        const int32_t* k, const uint32_t* rnd, uint64_t seed, float* x,
                        sd_stride xs, float* mp, sd_stride mps, hipStream_t s, const int* gate) {
  const int ng = (d + 3) / 4;
  const bool spread = spread_rows(B, K, d);
  const int per = spread ? 64 : kThreads;  // groups of a workgroup
  dim3 grid((ng + per - 1) / per, B);
  const bool vec = draft_vec(d, xs, mps, y, x, mp) && aligned16(cs);
  // (both blocks are written: together they decide what the cache can hold)
  const bool stream = stream_rows((int64_t)B * (2 * K + 1) * d * 4);
  const auto kernel = spread   ? draft_kernel<false, true>
                      : K == 1 ? draft_kernel<false, false, true>
                               : draft_kernel<false, false>;
  return timed("draft_block", s, [&] {
    kernel<<<grid, kThreads, 0, s>>>(sc, nullptr, K, d, y, cs, nullptr, nullptr, nullptr, 0, 0, k, rnd, seed,
                                     x, xs.chain, xs.row, mp, mps.chain, mps.row, nullptr, vec, stream, gate, 0);
  });
}

hipError_t draft_cached_launch(const Sched& sc, const float4* coef, int B, int K, int d,
                               const float* y,
                               const int32_t* crow, const int32_t* cstep, const float* mqprev,
                               sd_stride mqs, const int32_t* k, const uint32_t* rnd,
                               uint64_t seed, float* x, sd_stride xs, float* sv,
                               hipStream_t s, const int* gate, int chain0, int64_t stream_bytes) {
  const int ng = (d + 3) / 4;
  const bool spread = spread_rows(B, K, d);
  const int per = spread ? 64 : kThreads;  // groups of a workgroup
  dim3 grid((ng + per - 1) / per, B);
  const bool vec = draft_vec(d, xs, sd_stride{d, d}, y, x, sv) && aligned16(mqprev) &&
                   mqs.chain % 4 == 0 && mqs.row % 4 == 0;
  const bool stream = stream_rows(stream_bytes > 0 ? stream_bytes : (int64_t)B * (K + 1) * d * 4);
  const auto kernel = spread ? draft_kernel<true, true> : draft_kernel<true, false>;
  return timed("draft_block", s, [&] {
    kernel<<<grid, kThreads, 0, s>>>(sc, coef, K, d, y, nullptr, crow, cstep, mqprev, mqs.chain, mqs.row, k, rnd,
                                     seed, x, xs.chain, xs.row, nullptr, 0, 0, sv, vec, stream, gate, chain0);
  });
}

hipError_t fill_i32_launch(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t nb = (n + 255) / 256;
  fill_i32_kernel<<<(unsigned)nb, 256, 0, s>>>(p, n, v);
  return hipGetLastError();
}

hipError_t chains_active_launch(int B, int split, int N, const int32_t* k, int* f0, int* f1,
                                hipStream_t s) {
  chains_active_kernel<<<1, kThreads, 0, s>>>(B, split, N, k, f0, f1);
  return hipGetLastError();
}

hipError_t philox_words_launch(uint64_t seed, int n, const uint32_t* ctr, uint32_t* out,
                               hipStream_t s) {
  if (n <= 0) return hipSuccess;
  philox_words_kernel<<<(n + 255) / 256, 256, 0, s>>>(seed, n, ctr, out);
  return hipGetLastError();
}

hipError_t philox_normals_launch(uint64_t seed, uint32_t chain, uint32_t rnd, uint32_t tag,
                                 uint32_t slot, int d, float* out, hipStream_t s) {
  const int ng = (d + 3) / 4;
  philox_normals_kernel<<<(ng + 255) / 256, 256, 0, s>>>(seed, chain, rnd, (tag << 24) | slot,
                                                         d, out);
  return hipGetLastError();
}

}  // namespace sd
