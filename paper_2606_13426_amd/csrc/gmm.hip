// Closed-form Gaussian-mixture target: m^q_n(x) = c1_n x + c2_n s(x) for many
// rows (eq. target-distribution; the B(K+1) states of a round "in parallel").
//
// For a row x at step n with signal level a and s2_m = a^2 var_m + 1 - a^2,
//   logit_m = log w_m - (d/2) log s2_m - (||x||^2 - 2 a x.mu_m + a^2 ||mu_m||^2) / (2 s2_m)
//   r = softmax(logit),  P_m = r_m a / s2_m,  rho = sum_m r_m / s2_m,
//   score = P mu - rho x,   m^q = c1 x + c2 score.
// The two contractions are GEMMs on the matrix cores:
//   gmm_logits:  S = X mu^T   (rows x d by d x M), split over d, with ||x||^2;
//   gmm_softmax: sums the split partials in a fixed order and forms P, rho (float64 logits);
//   gmm_mean:    O = P mu     (rows x M by M x d) with the EM epilogue fused.
// Both GEMMs are "A times B-transposed" over row-major operands whose
// contraction index is contiguous (mu^T is stored at target creation), on the
// bf16 matrix cores through exact three-term operand splits (gemm_split.hpp:
// float32-accurate products, mu and mu^T pre-split at target creation, rows
// padded to 16 bytes).  Rows that were not 16-byte aligned, d or M no multiple
// of 64 and K + 1 < 4 used to take element-wise loads and float32 matrix
// instructions: 777 rows of 4107 x 100 components logits 27.8 -> 16.7 us, mean
// 26.7 -> 19.2; a round's 2304 rows of 784 x 100 logits 15.5 -> 10.5, mean
// 21.4 -> 15.0.  The partial logits and P have rows of Mp = M rounded up to 64
// components (P is zero past M), so every shape takes the same kernels.
#include <type_traits>

#include "common.hpp"
#include "gemm_split.hpp"
#include "philox.hpp"
#include "rows.hpp"
#include "rowsum.hpp"
#include "wavered.hpp"

namespace sd {
namespace {

constexpr int kThreads = 256;
constexpr int TILE = 64;
constexpr int KC = 64;
constexpr int LDW = TILE + 4;  // LDS row stride in floats (16-byte aligned rows)

using split::f4u;
using split::ld4u;

// Columns col .. col + 3 of a row of d floats, zero past it.  EDGE 0: all exist
// (d a whole number of tiles).  EDGE 1 (d >= 4): one 16-byte load that ends at
// the row's end at the latest, its values shifted into place (no branch, so
// loads stay in flight together).  EDGE 2 (d < 4): element by element.
template <int EDGE>
__device__ __forceinline__ float4 load_quad(const float* row, int col, int d) {
  if constexpr (EDGE == 0) {
    return ld4u(row + col);
  } else if constexpr (EDGE == 1) {
    const int at = min(col, d - 4), s = col - at;
    const float4 v = ld4u(row + at);
    return make_float4(s == 0 ? v.x : s == 1 ? v.y : s == 2 ? v.z : s == 3 ? v.w : 0.f,
                       s == 0 ? v.y : s == 1 ? v.z : s == 2 ? v.w : 0.f,
                       s == 0 ? v.z : s == 1 ? v.w : 0.f, s == 0 ? v.w : 0.f);
  } else {
    float f[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float v = row[min(col + c, d - 1)];
      f[c] = col + c < d ? v : 0.f;
    }
    return make_float4(f[0], f[1], f[2], f[3]);
  }
}
inline int edge_of(int d) { return d % 64 == 0 ? 0 : d >= 4 ? 1 : 2; }

template <bool STREAM>
__device__ __forceinline__ void store_quad(float* p, int cnt, float4 v) {
  if (cnt >= 4) {
    const f4u t = {v.x, v.y, v.z, v.w};
    if constexpr (STREAM)
      __builtin_nontemporal_store(t, reinterpret_cast<f4u*>(p));
    else
      *reinterpret_cast<f4u*>(p) = t;
  } else {
    if (cnt > 0) p[0] = v.x;
    if (cnt > 1) p[1] = v.y;
    if (cnt > 2) p[2] = v.z;
  }
}

__device__ __forceinline__ float comp(const float4& v, int c) {
  return c == 0 ? v.x : c == 1 ? v.y : c == 2 ? v.z : v.w;
}

// The logits GEMM: X rows split in registers, mu from its pre-split planes,
// float64 ||x||^2 from the unsplit values.  The tile is kSplitRows = 128 rows
// of X (two 16-row blocks per wavefront, each B fragment read from LDS serving
// both) by 64 components: half the LDS traffic and B loads per output of a
// 64-row tile, at two wavefronts per SIMD (the 32 accumulators and 32 A values
// per lane need the registers).
constexpr int kSplitRB = 2, kSplitRows = 64 * kSplitRB;

template <bool RAGGED, split::Sum SUM>
__global__ __launch_bounds__(kThreads, 2) void gmm_logits_split_kernel(
    int R, int M, int Mp, int d, int dp, const float* __restrict__ X, int64_t ldx,
    const uint16_t* __restrict__ musplit, int ksplit, float* __restrict__ part,
    double* __restrict__ xsq, const int* gate) {
  __shared__ uint16_t lds[split::kLdsBytes / 2];
  // grid (splits, row tiles, column tiles): the split index varies fastest so
  // that neighbouring workgroups stream neighbouring pieces of the same rows
  const int nsplit = gridDim.x, nrt = gridDim.y;
  const int lin = xcd_tile(nsplit * nrt * gridDim.z);
  const int s = lin % nsplit, rt = (lin / nsplit) % nrt, ct = lin / (nsplit * nrt);
  const int r0 = rt * kSplitRows, c0 = ct * TILE;
  const int kbeg = s * ksplit, kend = min(RAGGED ? d / KC * KC : d, kbeg + ksplit);
  const split::ARows<kSplitRB> arows = split::a_rows<kSplitRB>(X, ldx, R, r0);
  const split::BRows brows = split::b_rows(musplit, (int64_t)M * dp, dp, M, c0);
  split::Acc acc[kSplitRB];
  double sq[kSplitRB];
#pragma unroll
  for (int r = 0; r < kSplitRB; ++r) {
    split::zero(acc[r]);
    sq[r] = 0.0;
  }
  const bool want_sq = ct == 0;
  if (!RAGGED || kbeg < kend) {
    split::AChunk ra[kSplitRB];
    split::BChunk rb;
    split::load_b(brows, kbeg, rb);
    split::load_a<kSplitRB>(arows, kbeg, ra);
    if (gate && *gate == 0) return;
    if (want_sq)
      split::tile_run<true, kSplitRB, SUM>(lds, arows, brows, kbeg, kend, ra, rb, acc, sq);
    else
      split::tile_run<false, kSplitRB, SUM>(lds, arows, brows, kbeg, kend, ra, rb, acc, sq);
  } else if (gate && *gate == 0) {
    return;
  }
  if (RAGGED && s == nsplit - 1) split::tile_tail<true, kSplitRB, SUM>(lds, arows, brows, kend, d, acc, sq);
  float* ps = part + (int64_t)s * R * Mp;
#pragma unroll
  for (int r = 0; r < kSplitRB; ++r) {
    const int row = r0 + split::out_row<kSplitRB>(r);
    if (row >= R) continue;
#pragma unroll
    for (int b = 0; b < 4; ++b)  // (columns past M are not read; the chain's M is whole)
      if (SUM == split::CHAIN || c0 + split::out_col(b) < M)
        *reinterpret_cast<split::f32x4*>(&ps[(int64_t)row * Mp + c0 + split::out_col(b)]) = acc[r].c[b];
  }
  if (want_sq) {
    // the four lanes of a row are l % 16 + 16 q
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int r = 0; r < kSplitRB; ++r) {
      double t = sq[r];
      t += __shfl_xor(t, 16);
      t += __shfl_xor(t, 32);
      const int row = r0 + 16 * (kSplitRB * w + r) + lane;
      if (lane < 16 && row < R) xsq[(int64_t)s * R + row] = t;
    }
  }
}

// Softmax over a row's components.  With the per-(step, component) table
// ls[n][m] = (log s2, 1/s2):
//   logit_m = log w_m - (d/2) log s2 - (||x||^2 - 2 a x.mu_m + a^2 ||mu_m||^2) / (2 s2)
// in float64, then one maximum, one exp per component, and the sums of
// e_m and e_m / s2_m (rho is their ratio).
//
// The kernel is a chain of dependent latencies (step -> tables -> reductions).
// SPREAD, for few rows, spreads a row as wide as it goes: a wavefront takes 64
// components; lane 16 q + l first sums the split partials s = q, q + 4, .. of
// the components 4 l .. 4 l + 3 of its wavefront (all in flight together), and
// a reduce-scatter over q leaves each lane one component.  Otherwise, where
// the wavefronts' own instructions are the limit, a lane keeps all splits of
// four components and a wavefront takes 256 of a row, or PACK rows of up to 256 /
// PACK.  NW wavefronts hold a row; every input that does not hang on the step is
// requested at the start; the row's lanes sum ||x||^2, a split each.  The maximum
// is a float64 one: rounded to float32 it would be off by more than the
// exponential's range from logits of about 2e9 on (a row far from the data at a
// late step), and infinite from 3e38 on.
// Per launch (rocprofv3), against one kernel of four components per lane with
// LDS-permute reductions and the splits summed serially: 64 rows x 64
// components of 24 splits 12.3 -> 4.7 us, 72 rows 11.9 -> 4.7, 777 rows x 100
// 8.8 -> 5.7, 2304 x 1024 (66 MB of partials) 18.5 -> 18.0.
template <int NW, bool SPREAD, int PACK, class TP>
__global__ __launch_bounds__(NW > 4 ? 64 * NW : kThreads) void gmm_softmax_kernel(
    int R, int M, int Mp, int ldp, int d, int S, const float* __restrict__ part, const double* __restrict__ xsq,
    const int32_t* __restrict__ step, const double* __restrict__ sig, const double2* __restrict__ ls,
    const double* __restrict__ logw, const double* __restrict__ musq, const float4* __restrict__ coef,
    TP* __restrict__ P, float* __restrict__ rowc, const int* gate) {
  static_assert(PACK == 1 || (NW == 1 && !SPREAD), "rows share a wavefront that holds whole rows");
  constexpr int kT = NW > 4 ? 64 * NW : kThreads, RPW = PACK * kT / (64 * NW);
  constexpr int NC = SPREAD ? 1 : 4, DS = SPREAD ? 4 : 1;  // components per lane, split stride
  constexpr int LR = 64 / PACK;                            // lanes of a wavefront that hold a row
  const int lane = threadIdx.x & (LR - 1), w = (threadIdx.x >> 6) % NW;
  const int row = blockIdx.x * RPW + (int)(threadIdx.x / (LR * NW));
  const bool on = row < R;
  const int rr = on ? row : R - 1;  // lanes of a missing row follow the last one (no stores)
  const int live = gate ? *gate : 1;
  const int n = step[rr];
  const int q = SPREAD ? lane >> 4 : 0, l = SPREAD ? lane & 15 : lane;
  // the quad summed, and the first component kept (SPREAD: lane bits 5 and 4
  // select it after the reduce-scatter)
  const int m0 = (SPREAD ? 64 : 256) * w + 4 * l, m = m0 + q;
  double lw[NC], mq2[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int mc = min(m + c, M - 1);
    lw[c] = logw[mc];
    mq2[c] = musq[mc];
  }
  // (at most 64 splits: one lane each, or PACK)
  double xs = 0.0;
#pragma unroll
  for (int u = 0; u < PACK; ++u) {
    const int sp = lane + u * LR;
    const double xl = xsq[(int64_t)min(sp, S - 1) * R + rr];
    xs += sp < S ? xl : 0.0;
  }
  double dot[4] = {0.0, 0.0, 0.0, 0.0};
  if (m0 < M) {
    const float* pr = part + (int64_t)rr * Mp + m0;
    // a batch of splits' loads together (a missing one repeats the last)
    auto sum = [&](auto batch) {
      constexpr int U = decltype(batch)::value;
      for (int s0 = 0; s0 < S; s0 += U * DS) {
        split::f32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          v[u] = *reinterpret_cast<const split::f32x4*>(pr + (int64_t)min(s0 + q + u * DS, S - 1) * R * Mp);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool in = s0 + q + u * DS < S;
#pragma unroll
          for (int c = 0; c < 4; ++c) dot[c] += in ? (double)v[u][c] : 0.0;
        }
      }
    };
    if (S <= 2 * DS)
      sum(std::integral_constant<int, 2>{});
    else
      sum(std::integral_constant<int, 8>{});
  }
  const double a = sig[n];
  double2 t[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) t[c] = ls[(int64_t)n * M + min(m + c, M - 1)];
  const float4 cf = coef[n];
  if (live == 0) return;
  xs = group_sum(xs, LR);
  if constexpr (SPREAD) {
    const double d02 = swap_add<true>(dot[0], dot[2]), d13 = swap_add<true>(dot[1], dot[3]);
    dot[0] = swap_add<false>(d02, d13);
  }
  double lg[NC];
  double mx = -INFINITY;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    lg[c] = lw[c] - 0.5 * (double)d * t[c].x - 0.5 * (xs - 2.0 * a * dot[c] + a * a * mq2[c]) * t[c].y;
    if (m + c < M) mx = fmax(mx, lg[c]);
  }
  __shared__ double redm[kT / 64];
  __shared__ double2 reds[kT / 64];
  mx = group_max(mx, LR);
  const int w0 = (int)(threadIdx.x >> 6) - w;  // the row's first wavefront
  if constexpr (NW > 1) {
    if (lane == 0) redm[w0 + w] = mx;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NW; ++i) mx = fmax(mx, redm[w0 + i]);
  }
  float e[NC];
  double sum = 0.0, sis = 0.0;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    e[c] = m + c < M ? __expf((float)(lg[c] - mx)) : 0.0f;
    sum += (double)e[c];
    sis += (double)e[c] * t[c].y;
  }
  sum = group_sum(sum, LR);
  sis = group_sum(sis, LR);
  if constexpr (NW > 1) {
    if (lane == 0) reds[w0 + w] = make_double2(sum, sis);
    __syncthreads();
    sum = reds[w0].x;
    sis = reds[w0].y;
#pragma unroll
    for (int i = 1; i < NW; ++i) {
      sum += reds[w0 + i].x;
      sis += reds[w0 + i].y;
    }
  }
  const double inv = 1.0 / sum;
  if (on && m < ldp) {  // (the weights past M are zero)
    TP o[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const float pm = (float)((double)e[c] * inv * a * t[c].y);
      if constexpr (sizeof(TP) == 2)
        o[c] = __builtin_bit_cast(uint16_t, (__bf16)pm);
      else
        o[c] = pm;
    }
    TP* pp = P + (int64_t)row * ldp + m;
    if constexpr (NC == 4) {
      struct alignas(4 * sizeof(TP)) Quad { TP v[4]; };
      *reinterpret_cast<Quad*>(pp) = Quad{{o[0], o[1], o[2], o[3]}};
    } else {
      *pp = o[0];
    }
  }
  if (on && w == 0 && lane < 3)
    rowc[3 * (int64_t)row + lane] = lane == 0 ? cf.x : lane == 1 ? cf.y : (float)(sis * inv);
}

// O = P mu with the EM epilogue: P split in registers, mu^T from its pre-split
// planes.  A lane's accumulators are four consecutive columns of one row, so x
// comes in and the means go out in 16-byte pieces, 64 bytes of 16 rows per
// instruction.  EM: the plain Euler-Maruyama step (EmStep), whose noise as a
// kernel of its own was a fourth of a small step's launches and one more pass
// over the rows (64 rows of 3072, a step: 16.7 -> 13.7 us, with the logits' splits).
template <int EDGE, split::Sum SUM, bool EM>
__global__ __launch_bounds__(kThreads) void gmm_mean_split_kernel(
    int R, int Mp, int Mk, int d, const float* __restrict__ P, const uint16_t* __restrict__ muTs,
    const float* __restrict__ X, int64_t ldx, const float* __restrict__ rowc,
    float* __restrict__ mq, int64_t ldq, float* __restrict__ score, int64_t lds_,
    const int* gate, EmStep em) {
  __shared__ uint16_t lds[split::kLdsBytes / 2];
  const int r0 = blockIdx.x * TILE, c0 = blockIdx.y * TILE;
  const split::ARows<1> arows = split::a_rows<1>(P, Mp, R, r0);
  const split::BRows brows = split::b_rows(muTs, (int64_t)d * Mk, Mk, d, c0);
  split::AChunk sa[1];
  split::BChunk sb;
  split::load_b(brows, 0, sb);
  split::load_a<1>(arows, 0, sa);
  // the epilogue's inputs, whose latency then overlaps the contraction
  const int row = r0 + split::out_row<1>(0), rr = min(row, R - 1);
  const float c1 = rowc[3 * (int64_t)rr], c2 = rowc[3 * (int64_t)rr + 1], rho = rowc[3 * (int64_t)rr + 2];
  float4 xv[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    xv[b] = load_quad<EDGE>(X + (int64_t)rr * ldx, c0 + split::out_col(b), d);
  }
  if (gate && *gate == 0) return;
  split::Acc acc[1];
  split::zero(acc[0]);
  double unused[1] = {0.0};
  split::tile_run<false, 1, SUM>(lds, arows, brows, 0, Mp, sa, sb, acc, unused);
  if (row >= R) return;
  if (EM && blockIdx.y == 0 && split::out_col(0) == 0) em.step[row] = em.n + 1;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int col = c0 + split::out_col(b), cnt = EDGE == 0 ? 4 : d - col;
    const float4 x = xv[b];
    const split::f32x4 o = acc[0].c[b];
    const float4 sc = make_float4(o[0] - rho * x.x, o[1] - rho * x.y, o[2] - rho * x.z, o[3] - rho * x.w);
    float4 q = make_float4(c1 * x.x + c2 * sc.x, c1 * x.y + c2 * sc.y, c1 * x.z + c2 * sc.z, c1 * x.w + c2 * sc.w);
    if constexpr (EM) q = em_state(q, em.sigma, (uint32_t)(col >> 2), (uint32_t)row, (uint32_t)em.n, em.seed);
    store_quad<false>(mq + (int64_t)row * ldq + col, cnt, q);
    if (!EM && score) store_quad<false>(score + (int64_t)row * lds_ + col, cnt, sc);
  }
}

// The sampler's second GEMM: O = P mu with the EM epilogue, plus the partial
// log-ratio sums of verification while the tile is on chip.  Rows are
// (chain b, row j) of a [B][K+1][d] block: x row j is draft yhat_{k+j} (row 0
// the state); the draft mean m^p_{k+j} is recomputed from x row j and the
// chain's cache row SV[b] = c2_c S_c exactly as the draft formed it
// (draft_mean, with c2_{k+j} / c2_c from the step tables and the cache step
// cstep[b]).  For j < K and the tile's 64 columns the kernel accumulates, in
// float64 from the float32 values,
//   sum (m^p - m^q)^2   and   sum (yhat_{j+1} - m^p)(m^p - m^q),
// i.e. ||Delta_{j+1}||^2 sigma^2 and Z.Delta sigma^2 (App. A.2), and
// sum (m^p - m^q) G with the residual's G (Alg. 5), into
// lrp[row][column tile][3]; the scan sums the tiles in a fixed order.
// Epilogue layout: the contraction's output is staged in LDS and thread t
// owns columns 4 (t % 16) .. + 3 of the four consecutive tile rows 4 (t / 16)
// .. + 3, so a wavefront's access to one row index is four rows x 256
// contiguous bytes, the next draft of a row is the x of the thread's next one
// (one extra load for the last), and the rows meet at most two chains (two
// cache-row loads: four rows from a multiple of four on, for every K + 1 >= 2);
// the per-row sums are reduced over the 16 lanes of a row (rowsum.hpp).
// Columns past d read x, the cache and their products as zero and add nothing.
// m^q is stored non-temporally: of a chain's K + 1 rows the round reads back two
// (the residual's mean and the next cache row).  Products on the bf16 matrix cores as in gmm_mean_split_kernel.
template <int EDGE, split::Sum SUM>
__global__ __launch_bounds__(kThreads) void gmm_mean_lr_kernel(
    int R, int Mp, int Mk, int d, int K1, const float* __restrict__ P,
    const uint16_t* __restrict__ muTs, const float* __restrict__ X,
    const float* __restrict__ rowc, const float* __restrict__ SV,
    const int32_t* __restrict__ cstep, const float4* __restrict__ coef, float* __restrict__ mq,
    double* __restrict__ lrp, const uint32_t* __restrict__ rnd, uint64_t seed, const int* gate,
    int chain0) {
  if (gate && *gate == 0) return;
  // the operand planes, then the staged output and G
  __shared__ __align__(16) float sm[2 * TILE * LDW];
  static_assert(split::kLdsBytes <= (int)sizeof(sm), "the operand planes and the epilogue share the LDS");
  float *const stage = sm, *const gz = sm + TILE * LDW;
  __shared__ float rc[3 * TILE];
  __shared__ float cscale[TILE];  // 1 / c2 at each chain's cache step
  // grid (column tiles, row tiles): the column tile varies fastest so that
  // neighbouring workgroups stream neighbouring pieces of the same rows
  const int nct = gridDim.x;
  const int lin = xcd_tile(nct * gridDim.y);
  const int ct = lin % nct, rt = lin / nct;
  const int r0 = rt * TILE, c0 = ct * TILE;
  const int B = R / K1;
  const int cg = threadIdx.x & 15, rg = threadIdx.x >> 4;
  const int col = c0 + 4 * cg, cnt = EDGE == 0 ? 4 : d - col;
  const int b_first = r0 / K1;
  const int nchain = min((min(r0 + TILE, R) - 1) / K1 - b_first + 1, TILE);
  // the contraction's first operand chunk, then every global load of the
  // epilogue, whose latency then overlaps the contraction
  const split::ARows<1> arows = split::a_rows<1>(P, Mp, R, r0);
  const split::BRows brows = split::b_rows(muTs, (int64_t)d * Mk, Mk, d, c0);
  split::AChunk sa[1];
  split::BChunk sb;
  split::load_b(brows, 0, sb);
  split::load_a<1>(arows, 0, sa);
  // small per-row and per-chain inputs next (the epilogue's coefficients and
  // the rounds of the residual's G), so that their waits exclude the bulk
  // (unconditional loads from clamped indices, unused where out of range)
  const float rcv = rowc[min(3 * (int64_t)r0 + threadIdx.x, 3 * (int64_t)R - 1)];
  constexpr int kGItems = 3;  // ceil(16 x chains / 256): at most 33 chains meet a tile
  uint32_t rn[kGItems];
#pragma unroll
  for (int u = 0; u < kGItems; ++u)
    rn[u] = rnd[min(b_first + (int)((threadIdx.x + kThreads * u) >> 4), B - 1)];
  // (the table lookup that depends on the step follows the bulk loads, and is
  // used after the contraction: its wait for the step covers none of them)
  const int csi = cstep[min(b_first + (int)threadIdx.x, B - 1)];
  // keep that issue order: the scheduler must not hoist the bulk loads above
  __builtin_amdgcn_sched_barrier(0);
  const int lrb = 4 * rg;
  const int bl = (r0 + lrb) / K1, bh = (r0 + lrb + 3) / K1;
  float4 xv[5], svl, svh;  // x of the four rows and of the one after, cache rows of their chains
#pragma unroll
  for (int i = 0; i < 5; ++i) xv[i] = load_quad<EDGE>(X + (int64_t)min(r0 + lrb + i, R - 1) * d, col, d);
  svl = load_quad<EDGE>(SV + (int64_t)min(bl, B - 1) * d, col, d);
  svh = load_quad<EDGE>(SV + (int64_t)min(bh, B - 1) * d, col, d);
  const float csw = coef[csi].w;  // 1 / c2 at the chain's cache step
  split::Acc acc[1];
  split::zero(acc[0]);
  double unused[1] = {0.0};
  split::tile_run<false, 1, SUM>(reinterpret_cast<uint16_t*>(sm), arows, brows, 0, Mp, sa, sb, acc, unused);
  __syncthreads();  // every wavefront is done with the operand planes
#pragma unroll
  for (int b = 0; b < 4; ++b)
    *reinterpret_cast<split::f32x4*>(&stage[split::out_row<1>(0) * LDW + split::out_col(b)]) = acc[0].c[b];
  if (threadIdx.x < 3 * TILE) rc[threadIdx.x] = r0 + (int)threadIdx.x / 3 < R ? rcv : 0.f;
  if (threadIdx.x < TILE) cscale[threadIdx.x] = csw;
  // G of the residual (RESID stream of each chain's current round) depends
  // only on the chain and the coordinate: drawn once per chain of the tile
  // (item e: chain e / 16, coordinates 4 (e % 16) ..)
#pragma unroll
  for (int u = 0; u < kGItems; ++u) {
    const int e = threadIdx.x + kThreads * u;
    if (e < nchain * 16)
      *reinterpret_cast<float4*>(&gz[(e >> 4) * LDW + 4 * (e & 15)]) =
          normals4(philox((uint32_t)((c0 >> 2) + (e & 15)), (uint32_t)(chain0 + b_first + (e >> 4)), rn[u],
                          TAG_RESID << 24, seed));
  }
  __syncthreads();
  double s2[4], sz[4], sgd[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int lr = lrb + i, row = r0 + lr;
    const int b = row / K1, j = row - b * K1;
    const float c1 = rc[3 * lr], c2 = rc[3 * lr + 1], rho = rc[3 * lr + 2];
    float4 ov = *reinterpret_cast<const float4*>(&stage[lr * LDW + 4 * cg]);
    if (EDGE != 0)
      ov = make_float4(cnt > 0 ? ov.x : 0.f, cnt > 1 ? ov.y : 0.f, cnt > 2 ? ov.z : 0.f, cnt > 3 ? ov.w : 0.f);
    const float4 x = xv[i], y = xv[i + 1];
    const float4 sv = b == bl ? svl : svh;
    const float4 qv = make_float4(c1 * x.x + c2 * (ov.x - rho * x.x),
                                  c1 * x.y + c2 * (ov.y - rho * x.y),
                                  c1 * x.z + c2 * (ov.z - rho * x.z),
                                  c1 * x.w + c2 * (ov.w - rho * x.w));
    if (row < R) store_quad<true>(mq + (int64_t)row * d + col, cnt, qv);
    // every row is computed and kept only when it is a draft row of the block
    // (a select, no branch; the chain index of rows past R stays inside gz and
    // cscale)
    const bool keep = row < R && j < K1 - 1;
    const int bi = min(b - b_first, TILE - 1);
    const float4 gv = *reinterpret_cast<const float4*>(&gz[bi * LDW + 4 * cg]);
    const float c2s = c2 * cscale[bi];
    double a2 = 0.0, az = 0.0, ag = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float pe = draft_mean(c1, comp(x, e), c2s, comp(sv, e));  // m^p
      const double dd = (double)pe - (double)comp(qv, e);
      const double zz = (double)comp(y, e) - (double)pe;
      a2 = fma(dd, dd, a2);
      az = fma(zz, dd, az);
      ag = fma((double)comp(gv, e), dd, ag);
    }
    s2[i] = keep ? a2 : 0.0;
    sz[i] = keep ? az : 0.0;
    sgd[i] = keep ? ag : 0.0;
  }
  // every lane of the group takes part (rows past R and empty columns add zeros)
  const double t2 = reduce_rows16<4>(s2, cg), tz = reduce_rows16<4>(sz, cg),
               tg = reduce_rows16<4>(sgd, cg);
  const int row = r0 + lrb + row_of<4>(cg);
  if ((cg & 3) == 0 && row < R) {
    double* o = lrp + ((int64_t)row * nct + ct) * 3;
    o[0] = t2;
    o[1] = tz;
    o[2] = tg;
  }
}

// The bf16 operand planes of components mb .. me - 1, mu [me - mb][d]: NP = 3 the
// exact split, NP = 1 its rounding.  A [NP][M][dp] as it is, T [NP][d][Mk]
// transposed through LDS; both zero in the padding of their rows (T's is written
// with the last component's).
template <int NP>
__global__ __launch_bounds__(kThreads) void operands_kernel(int M, int Mk, int d, int dp, int mb, int me,
                                                            const float* __restrict__ mu,
                                                            uint16_t* __restrict__ A, uint16_t* __restrict__ T) {
  __shared__ uint16_t tile[NP][32][34];
  const int i0 = blockIdx.x * 32, m0 = mb + blockIdx.y * 32, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const int m = m0 + ty + 8 * h, i = i0 + tx;
    float v = m < me && i < d ? mu[(int64_t)(m - mb) * d + i] : 0.0f;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const __bf16 b = (__bf16)v;
      v -= (float)b;
      const uint16_t u = __builtin_bit_cast(uint16_t, b);
      tile[p][ty + 8 * h][tx] = u;
      if (m < me && i < dp) A[((int64_t)p * M + m) * dp + i] = u;
    }
  }
  __syncthreads();
  const int mt = me == M ? Mk : me;
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const int i = i0 + ty + 8 * h, m = m0 + tx;
    if (i < d && m < mt)
#pragma unroll
      for (int p = 0; p < NP; ++p) T[((int64_t)p * d + i) * Mk + m] = tile[p][tx][ty + 8 * h];
  }
}

struct Plan {
  int rows;  // the rows the plan is for (the whole batch's, for a part of one)
  int S, ksplit;
  size_t off_part, off_xsq, off_p, off_rowc, total;
};

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Split of the logits GEMM over d: the number of k-chunks per split and the
// number of splits (at most 64: a lane of the softmax each) minimise the time of
// the critical path, (rounds of workgroups over 512 slots, two per compute unit)
// x (chunks per workgroup) x 2.4 us a chunk (twice that where no row of X but the
// first is 16-byte aligned), plus that of the partials, written and read at 2.7
// TB/s.  Both rates come from two shapes: one and two chunks a workgroup at 2304
// rows of 784 (two: logits 12.7 -> 11.4, softmax 6.8 -> 5.2 us) and two and three
// at 777 rows of 4107 (two is better: 16.0 + 6.1 against 19.1 + 4.6 us).  The
// alignment is judged by d, which is what the workspace query knows: rows of a
// longer stride, or from an odd address, are priced as those of d are.
// measure: the workspace by which calls on the fixed scratch are accepted, rows
// of M components and splits chosen by the critical path among at most 32.
// Buffers for R rows; the split is chosen for plan_rows rows (0: R).
Plan make_plan(const Target& t, int R, int plan_rows = 0, bool measure = false) {
  Plan p{};
  const size_t M = measure ? t.M : t.Mp;
  // (tiles of kSplitRows rows, two workgroups per compute unit)
  const int Rp = plan_rows > 0 ? plan_rows : R;
  const int tiles = ((Rp + kSplitRows - 1) / kSplitRows) * ((t.M + TILE - 1) / TILE);
  const int nchunks = (t.d + KC - 1) / KC;
  constexpr int kSlots = 512;
  const int max_splits = measure ? 32 : 64;
  const double chunk_us = t.d % 4 ? 4.8 : 2.4;
  const double split_us = measure ? 0.0 : 8.0 * Rp * t.Mp / 2.7e6;
  double best_cost = 1e30;
  int best_per = nchunks;
  for (int S = 1; S <= max_splits && S <= nchunks; ++S) {
    const int per = (nchunks + S - 1) / S;
    const int splits = (nchunks + per - 1) / per;
    const double cost = chunk_us * (((tiles * splits + kSlots - 1) / kSlots) * per) + split_us * splits;
    if (cost < best_cost) {
      best_cost = cost;
      best_per = per;
    }
  }
  p.rows = Rp;
  p.ksplit = best_per * KC;
  p.S = (t.d + p.ksplit - 1) / p.ksplit;
  size_t off = 0;
  p.off_part = off;
  off = align256(off + sizeof(float) * (size_t)p.S * R * M);
  p.off_xsq = off;
  off = align256(off + sizeof(double) * (size_t)p.S * R);
  p.off_p = off;
  off = align256(off + sizeof(float) * (size_t)R * M);
  p.off_rowc = off;
  off = align256(off + sizeof(float) * 3 * (size_t)R);
  p.total = off;
  return p;
}

hipError_t logits_launch(const Target& t, const Plan& p, int R, const float* x, int64_t ldx,
                         float* part, double* xsq, hipStream_t s, const int* gate) {
  return launch_timed("gmm_logits", t.d % KC      ? gmm_logits_split_kernel<true, split::APART>
                                    : t.M % TILE ? gmm_logits_split_kernel<false, split::APART>
                                                 : gmm_logits_split_kernel<false, split::CHAIN>,
                      dim3(p.S, (R + kSplitRows - 1) / kSplitRows, t.Mp / TILE), dim3(kThreads), s, R, t.M, t.Mp,
                      t.d, t.dp, x, ldx, t.mu_split, p.ksplit, part, xsq, gate);
}

}  // namespace

hipError_t operands_launch(const Target& t, int planes, const float* mu, int m0, int n, uint16_t* A, uint16_t* T,
                           hipStream_t s) {
  const int m1 = m0 + n;
  const dim3 grid((t.dp + 31) / 32, ((m1 == t.M ? t.Mk : m1) - m0 + 31) / 32);
  (planes == 3 ? operands_kernel<3> : operands_kernel<1>)<<<grid, kThreads, 0, s>>>(t.M, t.Mk, t.d, t.dp, m0, m1, mu,
                                                                                    A, T);
  return hipGetLastError();
}

size_t target_ws_bytes(const Target& t, int rows, int plan_rows) {
  return t.prec == SD_BF16 ? target_ws_bytes_bf16(t, rows, plan_rows)
                           : make_plan(t, rows, plan_rows).total;
}

size_t target_ws_bytes_unpadded(const Target& t, int rows) {
  return t.prec == SD_BF16 ? target_ws_bytes_unpadded_bf16(t, rows) : make_plan(t, rows, 0, true).total;
}

hipError_t gmm_softmax_launch(const Target& t, int R, int plan_rows, int S, const float* part, const double* xsq,
                              const int32_t* step, void* P, bool p_bf16, float* rowc,
                              hipStream_t s, const int* gate) {
  auto launch = [&](auto nw, auto spread, auto pack) {
    constexpr int NW = decltype(nw)::value, PACK = decltype(pack)::value;
    constexpr bool SP = decltype(spread)::value;
    constexpr int kT = NW > 4 ? 64 * NW : kThreads, RPW = PACK * kT / (64 * NW);
    auto go = [&](auto kernel, auto* p) {
      return launch_timed("gmm_softmax", kernel, dim3((R + RPW - 1) / RPW), dim3(kT), s, R, t.M, t.Mp, p_bf16 ? t.Mk : t.Mp,
                          t.d, S, part, xsq, step, t.sig, t.ls, t.logw, t.musq, t.coef, p, rowc, gate);
    };
    if (p_bf16) return go(gmm_softmax_kernel<NW, SP, PACK, uint16_t>, static_cast<uint16_t*>(P));
    return go(gmm_softmax_kernel<NW, SP, PACK, float>, static_cast<float*>(P));
  };
  // Spread rows while their wavefronts are fewer than four per SIMD (a latency);
  // from there on four components per lane, four or two rows in a wavefront where
  // they fit one (us spread / here, by HIP events):
  //   M = 4    16384 rows 11.9 / 8.3    65536 rows 31.1 / 17.2
  //   M = 64    9216 rows  7.0 / 6.2    16384 rows 11.9 / 7.9   65536 rows 30.8 / 16.0
  //   M = 100   2048 rows  6.3 / 4.9    16384 rows 18.7 / 10.7
  //   M = 256   1024 rows  5.1 / 5.4     2048 rows  8.0 / 5.9    4352 rows 30.1 / 26.3 (bf16)
  //   M = 1000   128 rows  4.1 / 4.0      384 rows  7.6 / 4.4    2304 rows 29.7 / 18.0 (bf16, M = 1024)
  // Rows of up to 64 components, a wavefront each, stay spread up to ten per SIMD: a
  // launch may be half of the plan (chain groups), and beside the other half's kernels
  // the wider launch is the better one (a run of 1024 x 9 x 3072, M = 64, in two
  // groups 27.06 / 27.22 ms).
  // plan_rows, not R, decides, so that a part of a batch sums as the whole does.
  const int64_t waves = (int64_t)plan_rows * ((t.M + 63) / 64);
  const std::true_type sp{};
  const std::false_type wide{};
  constexpr std::integral_constant<int, 1> k1{};
  constexpr std::integral_constant<int, 2> k2{};
  constexpr std::integral_constant<int, 4> k4{};
  constexpr std::integral_constant<int, 8> k8{};
  constexpr std::integral_constant<int, 16> k16{};
  if (waves >= (t.M <= 64 ? 10240 : 4096)) {
    if (t.M <= 64) return launch(k1, wide, k4);
    if (t.M <= 128) return launch(k1, wide, k2);
    if (t.M <= 256) return launch(k1, wide, k1);
    if (t.M <= 512) return launch(k2, wide, k1);
    return launch(k4, wide, k1);
  }
  if (t.M <= 64) return launch(k1, sp, k1);
  if (t.M <= 128) return launch(k2, sp, k1);
  if (t.M <= 256) return launch(k4, sp, k1);
  if (t.M <= 512) return launch(k8, sp, k1);
  return launch(k16, sp, k1);
}

hipError_t target_mean_launch(const Target& t, int R, const float* x, int64_t ldx,
                              const int32_t* step, float* mq, int64_t ldq, float* score,
                              int64_t lds, void* ws, hipStream_t s, const int* gate,
                              int plan_rows, const EmStep* em) {
  if (t.prec == SD_BF16)
    return target_mean_bf16_launch(t, R, x, ldx, step, mq, ldq, score, lds, ws, s, gate,
                                   plan_rows, em);
  const Plan p = make_plan(t, R, plan_rows);
  char* base = static_cast<char*>(ws);
  float* part = reinterpret_cast<float*>(base + p.off_part);
  double* xsq = reinterpret_cast<double*>(base + p.off_xsq);
  float* P = reinterpret_cast<float*>(base + p.off_p);
  float* rowc = reinterpret_cast<float*>(base + p.off_rowc);
  hipError_t e = logits_launch(t, p, R, x, ldx, part, xsq, s, gate);
  if (e != hipSuccess) return e;
  e = gmm_softmax_launch(t, R, p.rows, p.S, part, xsq, step, P, false, rowc, s, gate);
  if (e != hipSuccess) return e;
  dim3 g2((R + TILE - 1) / TILE, (t.d + TILE - 1) / TILE);
  const int edge = edge_of(t.d);
  auto go = [&](auto noise) {
    constexpr bool EM = decltype(noise)::value;
    // (whole chunks of components keep the chain of six at any d, as they had it: the
    // sums apart gain nothing over 64 terms and more; 49 rows of 10 x 512 25.8 -> 23.5
    // us a call, 128 of 784 x 1024 48.0 -> 42.9)
    const auto pick = [&](auto sum) {
      constexpr split::Sum S = decltype(sum)::value;
      return edge == 2   ? gmm_mean_split_kernel<2, S, EM>
             : edge == 1 ? gmm_mean_split_kernel<1, S, EM>
                         : gmm_mean_split_kernel<0, S, EM>;
    };
    return launch_timed(EM ? "em_step" : "gmm_mean",
                        t.M % TILE ? pick(std::integral_constant<split::Sum, split::APART_ALL>{})
                                   : pick(std::integral_constant<split::Sum, split::CHAIN>{}),
                        g2, dim3(kThreads), s, R, t.Mp, t.Mk, t.d, P, t.muT_split, x, ldx, rowc, mq, ldq, score,
                        lds, gate, em ? *em : EmStep{});
  };
  return em ? go(std::true_type{}) : go(std::false_type{});
}

hipError_t target_mean_lr_launch(const Target& t, int R, int K1, const float* x,
                                 const int32_t* step, float* mq, const float* sv,
                                 const int32_t* cstep, double* lrp, const uint32_t* rnd,
                                 uint64_t seed, void* ws, hipStream_t s, const int* gate,
                                 int plan_rows, int chain0) {
  if (t.prec == SD_BF16)
    return target_mean_lr_bf16_launch(t, R, K1, x, step, mq, sv, cstep, lrp, rnd, seed, ws, s,
                                      gate, plan_rows, chain0);
  const Plan p = make_plan(t, R, plan_rows);
  char* base = static_cast<char*>(ws);
  float* part = reinterpret_cast<float*>(base + p.off_part);
  double* xsq = reinterpret_cast<double*>(base + p.off_xsq);
  float* P = reinterpret_cast<float*>(base + p.off_p);
  float* rowc = reinterpret_cast<float*>(base + p.off_rowc);
  hipError_t e = logits_launch(t, p, R, x, t.d, part, xsq, s, gate);
  if (e != hipSuccess) return e;
  e = gmm_softmax_launch(t, R, p.rows, p.S, part, xsq, step, P, false, rowc, s, gate);
  if (e != hipSuccess) return e;
  dim3 g2((t.d + TILE - 1) / TILE, (R + TILE - 1) / TILE);
  const int edge = edge_of(t.d);
  return launch_timed("gmm_mean_lr",
                      edge == 2   ? gmm_mean_lr_kernel<2, split::APART_ALL>
                      : edge == 1 ? gmm_mean_lr_kernel<1, split::APART_ALL>
                      : t.M % TILE ? gmm_mean_lr_kernel<0, split::APART_ALL>
                                   : gmm_mean_lr_kernel<0, split::CHAIN>,
                      g2, dim3(kThreads), s, R, t.Mp, t.Mk, t.d, K1, P,
                      t.muT_split, x, rowc, sv, cstep, t.coef, mq, lrp, rnd, seed, gate, chain0);
}

int lr_tiles(const Target& t, int K1) {
  return t.prec == SD_BF16 ? lr_tiles_bf16(t, K1) : (t.d + TILE - 1) / TILE;
}

}  // namespace sd
