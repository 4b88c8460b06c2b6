// Verification of drafted blocks: log density ratios (App. A.2) reduced over
// d, then the block (Alg. 6) or token (Alg. 2) acceptance scan and the U draw
// of Alg. 7.
//
// logratio_kernel: one workgroup per (chain, draft row).  The three float32
// rows (draft, draft mean, target mean) are streamed once with 16-byte
// non-temporal loads; differences and products are formed in float64 and
// accumulated in float64, then reduced across the wavefront with shuffles and
// across the four wavefronts through LDS.  Pure HBM streaming: 12 B per element.
//
// scan_kernel: one wavefront per chain, lane j-1 owns draft step j (K <= 64).
// Every lane replays the prefix recursion log alpha_j = min(0, log alpha_{j-1}
// + ell_j) in the same order as the definition, evaluates its h_j, draws its
// coin, and a ballot gives tau.  U is found by inverting Psi_alpha on all 64
// lanes at once (usample_exact): a grid over the law's bulk, then a window
// around the cubic inverse interpolant, usually two passes.
//
// Both scans take the temperature as w2 = omega^2 (the tempered
// verifications of the appendix divide every ell_j by omega^2), and the
// sampler's scan can hand the reflection residual (Alg. 4) to the next kernel
// instead of the Decomposition residual, skipping the U draw.
#include "common.hpp"
#include "dmath.hpp"
#include "philox.hpp"
#include "wavered.hpp"

namespace sd {
namespace {

constexpr int kThreads = 256;
typedef float f4v __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kThreads) void logratio_kernel(
    int K, int d, const float* __restrict__ yd, int64_t yc, int64_t yr,
    const float* __restrict__ mp, int64_t pc, int64_t pr, const float* __restrict__ mq,
    int64_t qc, int64_t qr, const double* __restrict__ sigma, const int32_t* __restrict__ kb,
    double* __restrict__ dn, double* __restrict__ lr, bool vec, const int* gate) {
  if (gate && *gate == 0) return;
  const int row = blockIdx.x;
  const int b = row / K, j = row - b * K;
  if (j >= kb[b]) {
    if (threadIdx.x == 0) {
      dn[row] = 0.0;
      lr[row] = 0.0;
    }
    return;
  }
  const float* py = yd + (int64_t)b * yc + (int64_t)j * yr;
  const float* pp = mp + (int64_t)b * pc + (int64_t)j * pr;
  const float* pq = mq + (int64_t)b * qc + (int64_t)j * qr;
  double s2 = 0.0, sz = 0.0;
  if (vec) {
    const f4v* vy = reinterpret_cast<const f4v*>(py);
    const f4v* vp = reinterpret_cast<const f4v*>(pp);
    const f4v* vq = reinterpret_cast<const f4v*>(pq);
    const int n4 = d >> 2;
#pragma unroll 4
    for (int i = threadIdx.x; i < n4; i += kThreads) {
      const f4v a = __builtin_nontemporal_load(vy + i);
      const f4v p = __builtin_nontemporal_load(vp + i);
      const f4v q = __builtin_nontemporal_load(vq + i);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double dd = (double)p[c] - (double)q[c];
        const double zz = (double)a[c] - (double)p[c];
        s2 = fma(dd, dd, s2);
        sz = fma(zz, dd, sz);
      }
    }
  } else {
    for (int i = threadIdx.x; i < d; i += kThreads) {
      const double dd = (double)pp[i] - (double)pq[i];
      const double zz = (double)py[i] - (double)pp[i];
      s2 = fma(dd, dd, s2);
      sz = fma(zz, dd, sz);
    }
  }
  s2 = wave_sum(s2);
  sz = wave_sum(sz);
  __shared__ double red[2][kThreads / 64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) {
    red[0][w] = s2;
    red[1][w] = sz;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t2 = 0.0, tz = 0.0;
    for (int i = 0; i < kThreads / 64; ++i) {
      t2 += red[0][i];
      tz += red[1][i];
    }
    const double s = sigma[(int64_t)b * (K + 1) + j];
    const double inv = 1.0 / (s * s);
    dn[row] = sqrt(t2 * inv);
    lr[row] = -tz * inv - 0.5 * t2 * inv;
  }
}

// log Psi_alpha(x) given the log normaliser Lstar = log(alpha Phi(u*) - Phi(u* - v)).
__device__ __forceinline__ double log_cdf(double x, double la, double v, double us,
                                          double Lstar) {
  if (x >= us) return 0.0;
  return log_excess(x, la, v) - Lstar;
}

// The value of lane i (wavefront-uniform), by a scalar lane read.
__device__ __forceinline__ double lane_value(double v, int i) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, i);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), i);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// 1/d to about an ulp (no finite value where d is zero or infinite).
__device__ __forceinline__ double recip(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  return fma(fma(-d, r, 1.0), r, r);
}

// x at g from four points (x_q, g_q): the cubic interpolant, and in *err the
// larger distance to the quadratics through the first and the last three.
__device__ __forceinline__ double cubic_at(const double (&px)[4], const double (&pg)[4], double g,
                                           double* err) {
  const double r01 = recip(pg[0] - pg[1]), r02 = recip(pg[0] - pg[2]), r03 = recip(pg[0] - pg[3]);
  const double r12 = recip(pg[1] - pg[2]), r13 = recip(pg[1] - pg[3]), r23 = recip(pg[2] - pg[3]);
  const double d0 = g - pg[0], d1 = g - pg[1], d2 = g - pg[2], d3 = g - pg[3];
  const double x3 = px[0] * (d1 * d2 * d3) * (r01 * r02 * r03) - px[1] * (d0 * d2 * d3) * (r01 * r12 * r13) +
                    px[2] * (d0 * d1 * d3) * (r02 * r12 * r23) - px[3] * (d0 * d1 * d2) * (r03 * r13 * r23);
  const double q0 = px[0] * (d1 * d2) * (r01 * r02) - px[1] * (d0 * d2) * (r01 * r12) +
                    px[2] * (d0 * d1) * (r02 * r12);
  const double q1 = px[1] * (d2 * d3) * (r12 * r13) - px[2] * (d1 * d3) * (r12 * r23) +
                    px[3] * (d1 * d2) * (r13 * r23);
  *err = fmax(fabs(x3 - q0), fabs(x3 - q1));
  return x3;
}

// Inverse of Psi_alpha at u (log u given), with all 64 lanes of the wavefront.
// In the coordinate g = sqrt(-log Psi) the inverse is nearly linear: next to
// u*, where 1 - Psi vanishes quadratically, and far in the left tail.  Pass 1
// evaluates a uniform grid of 63 points over the bulk of the law (and the
// normaliser on lane 63): down from min(u*, 6.5) (Psi there is 1 within the
// coin's resolution) to where Psi is below the smallest uniform, 2^-25 (the
// Gaussian tail below m = max(0, -u*) reaches e^-22 at sqrt(m^2 + 44) - m).
// Pass 2 puts 64 points into a window around the cubic inverse interpolant of
// the four points about the crossing, eight times as wide as its distance to
// the quadratics.  A pass is accepted when the crossing lies inside its points
// and cubic and quadratics agree to 1e-13 (relative): two passes for 97 % of
// u uniform, log alpha in [-6, 0], v in [1e-3, 300] (a doubling pass and a
// multisection on log Psi took four or five).  Otherwise the window shrinks
// again about the new interpolant, or the bracket is cut into 65, until the
// bracket is 1e-8 (relative) wide and a linear interpolation of log Psi closes
// it (next to u* only, where the density vanishes).
__device__ double usample_exact(double logu, double la, double v, int lane) {
  const double us = la / v + 0.5 * v;
  const double gt = sqrt(-logu);
  const double top = fmin(us, 6.5), m = fmax(0.0, -us);
  const double span = sqrt(fma(m, m, 44.0)) - m + fmax(top, 0.0);
  double x = lane < 63 ? top - span * ((double)(62 - lane) / 62.0) : us;
  double fx = log_excess(x, la, v);
  const double Lstar = lane_value(fx, 63);
  fx = x >= us ? 0.0 : fmin(fx - Lstar, 0.0);
  int cnt = __popcll(__ballot(lane < 63 && fx < logu));
  double lo, flo, hi = us, fhi = 0.0;
  if (cnt == 0) {
    // below the grid (a uniform at its smallest values): double the distance
    hi = lane_value(x, 0);
    fhi = lane_value(fx, 0);
    const double xd = us - ldexp(us - hi, lane + 1);
    const double fd = fmin(log_excess(xd, la, v) - Lstar, 0.0);
    const uint64_t below = __ballot(fd < logu) | (1ull << 63);
    const int p = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)below) - 1);
    lo = lane_value(xd, p);
    flo = lane_value(fd, p);
    if (p > 0) {
      hi = lane_value(xd, p - 1);
      fhi = lane_value(fd, p - 1);
    }
  } else {
    cnt = __builtin_amdgcn_readfirstlane(cnt);
    lo = lane_value(x, cnt - 1);
    flo = lane_value(fx, cnt - 1);
    if (cnt < 63) {
      hi = lane_value(x, cnt);
      fhi = lane_value(fx, cnt);
    }
  }
  bool centred = cnt > 0 && cnt < 63;  // the last points hold the crossing
  int top_lane = 62;                   // their last lane
  for (int it = 0; it < 64; ++it) {
    double blo = lo, bhi = hi;
    if (centred) {
      const int e0 = min(max(cnt - 2, 0), top_lane - 3);
      const double gx = sqrt(-fx);  // every lane's, before the reads: one square root
      double px[4], pg[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        px[q] = lane_value(x, e0 + q);
        pg[q] = lane_value(gx, e0 + q);
      }
      double err;
      const double xc = cubic_at(px, pg, gt, &err);
      if (it > 0 && err <= 1e-13 * fmax(1.0, fabs(xc)) && xc >= lo && xc <= hi) return xc;
      const double w = fmax(8.0 * err, 1e-7 * span);
      if (isfinite(xc) && isfinite(w) && xc - w < hi && xc + w > lo) {
        blo = fmax(lo, xc - w);
        bhi = fmin(hi, xc + w);
      }
    }
    const double mid = 0.5 * (lo + hi);
    if (!(mid > lo && mid < hi) || hi - lo <= 1e-8 * fmin(span, fmax(1.0, fabs(lo)))) break;
    x = blo + (bhi - blo) * ((double)lane / 63.0);
    fx = x >= us ? 0.0 : fmin(log_excess(x, la, v) - Lstar, 0.0);
    cnt = __builtin_amdgcn_readfirstlane(__popcll(__ballot(fx < logu)));
    if (cnt > 0) {
      lo = lane_value(x, cnt - 1);
      flo = lane_value(fx, cnt - 1);
    }
    if (cnt < 64) {
      hi = lane_value(x, cnt);
      fhi = lane_value(fx, cnt);
    }
    centred = cnt > 0 && cnt < 64;
    top_lane = 63;
  }
  const double t = fhi > flo ? (logu - flo) / (fhi - flo) : 0.5;
  return lo + (hi - lo) * fmin(fmax(t, 0.0), 1.0);
}

// The capped doubling/bisection of the paper's experiments (3 + 4 steps).
__device__ double usample_paper(double u, double logu, double la, double v) {
  const double us = la / v + 0.5 * v;
  const double Lstar = log_excess(us, la, v);
  double hi = us, lo = us - 1.0;
  for (int n = 0; n < 3 && log_cdf(lo, la, v, us, Lstar) > logu; ++n) lo = hi - 2.0 * (hi - lo);
  double mid = 0.5 * (lo + hi);
  for (int n = 0; n < 4; ++n) {
    const double lc = log_cdf(mid, la, v, us, Lstar);
    if (fabs(exp(lc) - u) <= 1e-6) break;
    if (lc < logu)
      lo = mid;
    else
      hi = mid;
    mid = 0.5 * (lo + hi);
  }
  return mid;
}

// The acceptance decision of one chain (one wavefront; lane j-1 holds ell_j
// and ||Delta_j|| of draft step j, kb valid steps): prefix recursion, h_j,
// coins, tau, alpha_res and, when tau <= kb and need_u, the U draw of Alg. 7.
// Temperature omega (w2 = omega^2): the tempered verifications of the
// appendix use ell_j / omega^2 wherever ell_j enters the acceptance, and the
// untempered ||Delta||; w2 = 1 is the exact method.
struct Decision {
  int tau;
  double la_res, U;
  uint64_t coins;
  uint64_t ties;  // steps whose coin lies within kTieWindow of its threshold
};

// A coin within this distance of its threshold (|eta_j - h_j|, or alpha_j for
// token verification) is a tie: rounding in another implementation may flip
// it, so such decisions are counted.
constexpr double kTieWindow = 1e-6;

// The uniforms of one chain's decision, drawn ahead of its log-ratios: the
// coin of this lane's draft step and the U draw's uniform (with its log).
struct Draws {
  double eta, u, logu;
};

__device__ __forceinline__ Draws draw_uniforms(uint32_t b, uint32_t r, uint64_t seed, int lane) {
  const uint4 w = philox((uint32_t)(lane >> 2), b, r, TAG_COIN << 24, seed);
  const uint4 wu = philox(0u, b, r, TAG_USAMPLE << 24, seed);
  const double u = uniform64(wu.x);
  return Draws{uniform64(pick(w, lane & 3)), u, log(u)};
}

__device__ Decision decide(int mode, int umode, int kb, double ell_raw, double vn, const Draws& dr,
                           int lane, double w2, bool need_u) {
  const bool valid = lane < kb;
  const double ell = ell_raw / w2;
  // prefix recursion, replayed per lane in the definition's order
  double acc = 0.0, la = 0.0;
  for (int i = 0; i < kb; ++i) {
    acc = fmin(0.0, acc + lane_value(ell, i));
    if (i == lane) la = acc;
  }
  const double vnext = __shfl_down(vn, 1);
  double h;
  if (mode == SD_BLOCK) {
    h = block_h(la, vnext);
    if (lane + 1 >= kb) h = exp(la);
  } else {
    h = exp(fmin(0.0, ell));
  }
  const uint64_t cm = __ballot(valid && dr.eta < h);
  const uint64_t tm = __ballot(valid && fabs(dr.eta - h) <= kTieWindow);
  const uint64_t vmask = kb >= 64 ? ~0ull : ((1ull << kb) - 1ull);
  int t;
  if (mode == SD_BLOCK) {
    t = cm ? (64 - __clzll((long long)cm)) + 1 : 1;
  } else {
    const uint64_t rej = ~cm & vmask;
    t = rej ? __ffsll((unsigned long long)rej) : kb + 1;
  }
  t = __builtin_amdgcn_readfirstlane(t);
  const double la_res = (mode == SD_BLOCK && t >= 2) ? lane_value(la, t - 2) : 0.0;
  double U = NAN;
  if (t <= kb && need_u) {
    const double v = lane_value(vn, t - 1);  // > 0: a rejection never lands on a zero offset
    if (umode == SD_USAMPLE_PAPER) {
      double up = 0.0;
      if (lane == 0) up = usample_paper(dr.u, dr.logu, la_res, v);
      U = lane_value(up, 0);
    } else {
      U = usample_exact(dr.logu, la_res, v, lane);
    }
  }
  return Decision{t, la_res, U, cm, tm};
}

__global__ __launch_bounds__(kThreads) void scan_kernel(
    int B, int K, int mode, int umode, const double* __restrict__ dn,
    const double* __restrict__ lr, const int32_t* __restrict__ kbv,
    const uint32_t* __restrict__ rnd, uint64_t seed, double w2, int32_t* __restrict__ tau,
    double* __restrict__ lar, double* __restrict__ ures, uint64_t* __restrict__ coins,
    int* nanflag, const int* gate) {
  if (gate && *gate == 0) return;
  const int lane = threadIdx.x & 63;
  const int b = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (b >= B) return;  // whole wavefront
  const int kb = min(kbv[b], K);
  if (kb <= 0) {
    if (lane == 0) {
      tau[b] = 0;
      lar[b] = 0.0;
      ures[b] = NAN;
      if (coins) coins[b] = 0ull;
    }
    return;
  }
  const bool valid = lane < kb;
  const double ell = valid ? lr[(int64_t)b * K + lane] : 0.0;
  const double vn = valid ? dn[(int64_t)b * K + lane] : 0.0;
  const Draws dr = draw_uniforms((uint32_t)b, rnd[b], seed, lane);
  if (nanflag && __ballot(valid && !(isfinite(ell) && isfinite(vn))) != 0ull && lane == 0)
    atomicOr(nanflag, 1);
  const Decision D = decide(mode, umode, kb, ell, vn, dr, lane, w2, true);
  if (lane == 0) {
    tau[b] = D.tau;
    lar[b] = D.la_res;
    ures[b] = D.U;
    if (coins) coins[b] = D.coins;
  }
}

// The sampler's verification: sums the partials of the fused target call
// (fixed tile order) into ||Delta_j||, ell_j and, for the residual,
// e.G = sum_i (m^p - m^q)_i G_i / (sigma ||Delta||) of every row, decides, and
// hands the next kernel what it needs to form the residual elementwise:
//   rmode 1: y = m^q + sigma G + rcoef (m^p - m^q),  rcoef = (U - e.G)/||Delta||
//   rmode 2: y = m^q_{K_b} + sigma xi'  (full accept, target draw)
//   rmode 3: y = yhat_{K_b}             (full accept that reaches step N)
//   rmode 4: y = yhat_tau - rcoef (m^p - m^q),  rcoef = 1 + 2 D.W / D.D
//            (reflection residual, Alg. 4: m^q + sigma (I - 2 e e^T) Z with
//            D = m^p - m^q = sigma Delta and W = yhat_tau - m^p = sigma Z,
//            whose two sums are the log-ratio partials of row tau - 1)
// The round's decision record (tau, coins, log alpha_res, U) is kept per chain,
// and the coins within kTieWindow of their thresholds are added to ties[b].
// One workgroup per chain sums the partials with all four wavefronts; the
// first one then decides.  The kernel's time is one chain's latency: pixel3072
// (1024 chains in two groups) 23.8 -> 16.7 us per launch, 8 chains of the same
// size 20.5 -> 10.2, against one wavefront per chain with the earlier U draw.
// The workgroup after the last chain clears the next round's active flag and
// stores the gate (whether any chain was still active after the previous
// round) tagged with that round's index, (pub_round << 1) | flag, into
// host_prev, a word of mapped host memory that the host polls, so that
// neither a device-to-host copy nor an event is queued per round.
__global__ __launch_bounds__(kThreads) void scan_fused_kernel(
    int B, int K, int d, int N, int mode, int umode, const double* __restrict__ lrp, int nct,
    const double* __restrict__ sigma, const int32_t* __restrict__ kcur,
    const uint32_t* __restrict__ rcur, uint64_t seed, double w2, bool reflect,
    int32_t* __restrict__ tau, int32_t* __restrict__ rmode,
    float* __restrict__ rcoef, float* __restrict__ rsig, uint64_t* __restrict__ coins,
    double* __restrict__ lar, double* __restrict__ ures, int32_t* __restrict__ ties,
    int* nanflag, int* act_next, int* host_prev, int pub_round, const int* gate, int chain0) {
  if ((int)blockIdx.x == B) {  // the extra workgroup: no chain waits for its system-scope store
    if (threadIdx.x == 0) {
      *act_next = 0;
      if (host_prev) {
        __atomic_store_n(host_prev, (pub_round << 1) | (gate ? *gate : 1), __ATOMIC_RELAXED);
        __threadfence_system();
      }
    }
    return;
  }
  // every input of the chain is requested before the first one is used (the
  // gate among them): one trip to memory instead of a chain of them
  const int lane = threadIdx.x & 63;
  const int b = blockIdx.x, K1 = K + 1;
  const int k = kcur[b];
  const uint32_t r = rcur[b];
  // sigma of rows 0..K_b (lane j holds row j); the residual's sigma is taken
  // from these lanes below instead of a second load
  double sgl = lane <= K ? sigma[(int64_t)b * K1 + lane] : 1.0;
  const int live = gate ? *gate : 1;
  // Sum the column-tile partials of each draft row: row j is spread over lpr
  // of the 256 lanes (256 / K rounded down to a power of two, at most 64),
  // each lane takes every lpr-th tile with four independent accumulators
  // (loads in flight together), and the lanes of a row combine in a fixed xor
  // tree; then lane j of the first wavefront reads row j's totals.  Fixed
  // order throughout, so the sums are deterministic.
  int kp = 4;
  while (kp < K) kp <<= 1;
  const int lpr = kThreads / kp, j = threadIdx.x / lpr, sub = threadIdx.x % lpr;
  double a2[4] = {0.0, 0.0, 0.0, 0.0}, az[4] = {0.0, 0.0, 0.0, 0.0}, ag[4] = {0.0, 0.0, 0.0, 0.0};
  const double* pl = lrp + ((int64_t)b * K1 + min(j, K - 1)) * nct * 3;
  double q[4][3];
  auto request = [&](int ct) {  // four tiles' partials (a missing one repeats the last)
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 3; ++e) q[u][e] = pl[3 * min(ct + u * lpr, nct - 1) + e];
  };
  auto add = [&](int ct) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool in = j < K && ct + u * lpr < nct;
      a2[u] += in ? q[u][0] : 0.0;
      az[u] += in ? q[u][1] : 0.0;
      ag[u] += in ? q[u][2] : 0.0;
    }
  };
  request(sub);
  // the chain's uniforms while the partials are on their way
  Draws dr{};
  if (threadIdx.x < 64) dr = draw_uniforms((uint32_t)(chain0 + b), r, seed, lane);
  add(sub);
  for (int ct = sub + 4 * lpr; ct - sub < nct; ct += 4 * lpr) {
    request(ct);
    add(ct);
  }
  if (live == 0) return;
  const int kb = k < N ? min(K, N - k) : 0;
  if (kb <= 0) {
    if (threadIdx.x == 0) {
      tau[b] = 0;
      rmode[b] = 0;
    }
    return;
  }
  double s2 = (a2[0] + a2[1]) + (a2[2] + a2[3]);
  double sz = (az[0] + az[1]) + (az[2] + az[3]);
  double sgd = (ag[0] + ag[1]) + (ag[2] + ag[3]);
  s2 = group_sum(s2, lpr);
  sz = group_sum(sz, lpr);
  sgd = group_sum(sgd, lpr);
  __shared__ double sums[SD_MAX_BLOCK][3];
  if (sub == 0 && j < K) {
    sums[j][0] = s2;
    sums[j][1] = sz;
    sums[j][2] = sgd;
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;  // one wavefront decides
  const bool valid = lane < kb;
  s2 = valid ? sums[lane][0] : 0.0;
  sz = valid ? sums[lane][1] : 0.0;
  sgd = valid ? sums[lane][2] : 0.0;
  if (lane > kb) sgl = 1.0;
  const double sg = valid ? sgl : 1.0;
  const double inv = 1.0 / (sg * sg);
  const double vn = valid ? sqrt(s2 * inv) : 0.0;
  const double ell = valid ? -sz * inv - 0.5 * s2 * inv : 0.0;
  if (__ballot(valid && !(isfinite(ell) && isfinite(vn))) != 0ull && lane == 0) atomicOr(nanflag, 1);
  const Decision D = decide(mode, umode, kb, ell, vn, dr, lane, w2, !reflect);
  const int t = D.tau;
  int rm;
  float cf = 0.f, sgo = 0.f;
  // (row 64 of a full accept with K_b = 64 is in no lane)
  const double st = t <= kb || kb < 64 ? lane_value(sgl, t <= kb ? t - 1 : kb)
                                       : sigma[(int64_t)b * K1 + kb];
  const double s2t = lane_value(s2, t <= kb ? t - 1 : 0), szt = lane_value(sz, t <= kb ? t - 1 : 0);
  if (t <= kb && reflect) {
    // D.D > 0: a rejection never lands on a zero offset (kept as a guard)
    rm = 4;
    cf = s2t > 0.0 ? (float)(1.0 + 2.0 * szt / s2t) : 1.0f;
  } else if (t <= kb) {
    const double v = lane_value(vn, t - 1);
    const double eG = lane_value(sgd, t - 1) / (st * v);
    rm = 1;
    cf = (float)((D.U - eG) / v);
    sgo = (float)st;
  } else if (kb + 1 <= N - k) {
    rm = 2;
    sgo = (float)st;
  } else {
    rm = 3;
  }
  if (lane == 0) {
    tau[b] = t;
    rmode[b] = rm;
    rcoef[b] = cf;
    rsig[b] = sgo;
    coins[b] = D.coins;
    lar[b] = D.la_res;
    ures[b] = D.U;
    ties[b] += __popcll(D.ties);
  }
}

}  // namespace

hipError_t verify_launch(int B, int K, int d, int mode, const float* yd, sd_stride ys,
                         const float* mp, sd_stride mps, const float* mq, sd_stride mqs,
                         const double* sigma, const int32_t* kb, const uint32_t* rnd,
                         uint64_t seed, int umode, double w2, int32_t* tau, double* lar,
                         double* ures, double* dn, double* lr, uint64_t* coins, int* nanflag,
                         hipStream_t s, const int* gate) {
  const bool vec = (d % 4 == 0) && ys.chain % 4 == 0 && ys.row % 4 == 0 && mps.chain % 4 == 0 &&
                   mps.row % 4 == 0 && mqs.chain % 4 == 0 && mqs.row % 4 == 0 &&
                   aligned16(yd) && aligned16(mp) && aligned16(mq);
  const int64_t rows = (int64_t)B * K;
  hipError_t e = timed("logratio_reduce", s, [&] {
    logratio_kernel<<<(unsigned)rows, kThreads, 0, s>>>(K, d, yd, ys.chain, ys.row, mp,
                                                        mps.chain, mps.row, mq, mqs.chain,
                                                        mqs.row, sigma, kb, dn, lr, vec, gate);
  });
  if (e != hipSuccess) return e;
  const int per = kThreads / 64;
  return timed("block_scan", s, [&] {
    scan_kernel<<<(B + per - 1) / per, kThreads, 0, s>>>(B, K, mode, umode, dn, lr, kb, rnd, seed,
                                                        w2, tau, lar, ures, coins, nanflag, gate);
  });
}

hipError_t scan_fused_launch(int B, int K, int d, int N, int mode, int umode, const double* lrp,
                             int nct, const double* sigma, const int32_t* kcur,
                             const uint32_t* rcur, uint64_t seed, double w2, bool reflect,
                             int32_t* tau, int32_t* rmode, float* rcoef, float* rsig,
                             uint64_t* coins, double* lar, double* ures, int32_t* ties,
                             int* nanflag, int* act_next, int* host_prev, int pub_round,
                             hipStream_t s, const int* gate, int chain0) {
  return launch_timed("scan_fused", scan_fused_kernel, dim3(B + 1), dim3(kThreads), s,
                      B, K, d, N, mode, umode, lrp, nct, sigma, kcur, rcur, seed, w2, reflect, tau,
                      rmode, rcoef, rsig, coins, lar, ures, ties, nanflag, act_next, host_prev,
                      pub_round, gate, chain0);
}

}  // namespace sd
