// Float32 contractions on the bf16 matrix cores (gfx950).
//
// Each float32 value is split exactly into three bf16 terms, v = hi + mid + lo
// (hi = bf16(v), mid = bf16(v - hi), lo = bf16(v - hi - mid), rounding to
// nearest even; both residuals are exact in float32, and the 24-bit mantissa
// fits the three 8-bit ones).  A product a.b is formed from the six terms
//   lo.hi + hi.lo + mid.mid + mid.hi + hi.mid + hi.hi
// (smallest first) on v_mfma_f32_16x16x32_bf16, whose bf16 x bf16 products are
// exact in its float32 accumulator.  The three dropped terms (mid.lo, lo.mid,
// lo.lo) are below 2^-23 |a||b| together, the size of one float32 rounding, so
// the result is float32-accurate at 6/16 of the float32 instruction's
// matrix-core time.  (Where that rounding shows, two of the three are kept: Sum.)
//
// Tile: 64 RB rows of A x 64 rows of B (the output's columns) per workgroup
// of four wavefronts; wavefront w owns RB blocks of 16 rows (rows 16 (RB w +
// r) .. + 15, r < RB) and all four 16-column blocks, so each B fragment read
// from LDS feeds RB row blocks.  A (float32) goes from memory straight into
// its wavefront's registers, lane l holding row 16 (RB w + r) + l % 16 and
// k = 8 (l / 16) .. + 7 of each 32-wide step, and is split there.  B comes
// pre-split (three bf16 planes in memory, row-major) and is staged through
// LDS, 64 k per chunk, three planes of 64 x 72 (row stride 144 bytes: the 16
// rows of one 16-lane read pass fall in distinct banks).
// B is the matrix instruction's first operand, so that a lane's four
// accumulators of output block c are four CONSECUTIVE columns 16 c + 4 (l / 16)
// .. + 3 of row l % 16 of its row block: 16-byte stores and epilogue accesses.
//
// Any shape: rows of A and B past the matrix repeat its last row (their outputs
// are not stored, or masked); A's rows may lie at any 4-byte address (16-byte
// loads need no more), and only the chunk that crosses the row's end loads
// element by element, reading zero past it.  B's rows start at multiples of 8
// elements; past a row's end it reads whatever finite values follow (the last
// plane has a chunk of slack), which meet A's zeros.
#pragma once

#include "common.hpp"

namespace sd {
namespace split {

constexpr int TILE = 64, KC = 64;
constexpr int LDH = KC + 8;  // LDS row stride in bf16 elements
constexpr int kPlaneElems = TILE * LDH;
constexpr int kLdsBytes = 3 * kPlaneElems * 2;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct Acc {
  f32x4 c[4];
};

__device__ __forceinline__ void zero(Acc& a) {
#pragma unroll
  for (int b = 0; b < 4; ++b) a.c[b] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// The three bf16 terms of eight float32 values.
__device__ __forceinline__ void split8(const float4& u, const float4& v, bf16x8& hi, bf16x8& mid,
                                       bf16x8& lo) {
  const float x[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const __bf16 h = (__bf16)x[i];
    const float r = x[i] - (float)h;
    const __bf16 m = (__bf16)r;
    hi[i] = h;
    mid[i] = m;
    lo[i] = (__bf16)(r - (float)m);
  }
}

// Four floats at any 4-byte address.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ float4 ld4u(const float* p) {
  const f4u v = *reinterpret_cast<const f4u*>(p);
  return make_float4(v[0], v[1], v[2], v[3]);
}

// B chunk in registers: plane p, rows t / 8 + 32 h (h < 2), k = 8 (t % 8) .. + 7.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
struct BChunk {
  u32x4 v[3][2];
};

// The thread's piece of the 64 rows row0.. (nrows exist) of the three planes
// (each `plane` elements, leading dimension ld): pointers at k = 0.
struct BRows {
  const uint16_t* p[3];
  int64_t hstep;  // to the row 32 further down
};
__device__ __forceinline__ BRows b_rows(const uint16_t* planes, int64_t plane, int64_t ld, int nrows, int row0) {
  const int t = threadIdx.x, last = nrows - 1;
  const int64_t r = min(row0 + (t >> 3), last), r2 = min(row0 + (t >> 3) + 32, last);
  const uint16_t* q = planes + r * ld + 8 * (t & 7);
  return BRows{{q, q + plane, q + 2 * plane}, (r2 - r) * ld};
}

__device__ __forceinline__ void load_b(const BRows& b, int k0, BChunk& c) {
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int h = 0; h < 2; ++h) c.v[p][h] = *reinterpret_cast<const u32x4*>(b.p[p] + h * b.hstep + k0);
}

__device__ __forceinline__ void store_b(uint16_t* lds, const BChunk& c) {
  const int t = threadIdx.x;
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      *reinterpret_cast<u32x4*>(&lds[p * kPlaneElems + ((t >> 3) + 32 * h) * LDH + 8 * (t & 7)]) = c.v[p][h];
}

// A chunk of this lane's row: k = 32 s + 8 (l / 16) .. + 7 for s < 2.
struct AChunk {
  float4 v[2][2];
};

// This lane's rows of A (nrows of them exist, leading dimension ld): pointers
// at k = 8 (l / 16).
template <int RB>
struct ARows {
  const float* p[RB];
};
template <int RB>
__device__ __forceinline__ ARows<RB> a_rows(const float* A, int64_t ld, int nrows, int r0) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  ARows<RB> a;
#pragma unroll
  for (int r = 0; r < RB; ++r)
    a.p[r] = A + (int64_t)min(r0 + 16 * (RB * w + r) + (lane & 15), nrows - 1) * ld + 8 * (lane >> 4);
  return a;
}

// The chunk at k0 (whole inside the rows).
template <int RB>
__device__ __forceinline__ void load_a(const ARows<RB>& rows, int k0, AChunk (&a)[RB]) {
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int q = 0; q < 2; ++q) a[r].v[s][q] = ld4u(rows.p[r] + k0 + 32 * s + 4 * q);
}

// The chunk at k0 of rows of len < k0 + 64 elements, zero past them (loads from
// the row's start where an element does not exist: no branch).
template <int RB>
__device__ __forceinline__ void load_a_tail(const ARows<RB>& rows, int k0, int len, AChunk (&a)[RB]) {
  const int back = 8 * ((threadIdx.x & 63) >> 4);  // the row's start lies `back` elements before p
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        float f[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int k = k0 + 32 * s + 4 * q + c;
          const bool in = k + back < len;
          const float v = rows.p[r][in ? k : -back];
          f[c] = in ? v : 0.0f;
        }
        a[r].v[s][q] = make_float4(f[0], f[1], f[2], f[3]);
      }
}

// float64 sum of squares of the lane's A values of a chunk.
__device__ __forceinline__ double squares(const AChunk& a) {
  double t = 0.0;
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float4 v = a.v[s][q];
      t += (double)v.x * v.x + (double)v.y * v.y + (double)v.z * v.z + (double)v.w * v.w;
    }
  return t;
}

__device__ __forceinline__ bf16x8 frag(const uint16_t* p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p));
}

// The chunk's 2 steps x 4 column blocks x RB row blocks of products:
//   CHAIN      the six terms one after another on the running sum;
//   APART      the five small ones of a step summed from zero and added to the
//              leading product's sum once: two roundings of the running sum per
//              step instead of six;
//   APART_ALL  the same with mid.lo and lo.mid (what is left out is below 2^-32).
// In a contraction of few terms six roundings show beside the one or two of a
// float32 instruction (error of a score against 64 bits, 2 x 191 components:
// 8.1e-7 there, 4.7e-7 apart; 4 x 20: 5.6e-7, 4.5e-7), so APART serves the logits
// where d or M is no multiple of 64.  Where one component has all of a row's weight
// its mean GEMM is a single product, and dropping two terms of it adds to its one
// rounding: score errors of up to 1.008 times a float32 instruction's over 70
// ragged shapes (448 x 1 component, 2168 x 88), 1.000 with all of them, hence
// APART_ALL for the mean GEMMs that once took float32 instructions (M no multiple
// of 64; in the sampler's, d too).  The others keep the chain they had: the extra
// registers take a wavefront per SIMD (a sampler call of 1024 x 3072 846 us against
// 816).
enum Sum { CHAIN, APART, APART_ALL };
template <int RB, Sum SUM>
__device__ __forceinline__ void mma_chunk(const uint16_t* lds, const AChunk (&a)[RB], Acc (&acc)[RB]) {
  const int lane = threadIdx.x & 63;
  const uint16_t* pb = lds + (lane & 15) * LDH + 8 * (lane >> 4);
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    bf16x8 ah[RB], am[RB], al[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) split8(a[r].v[s][0], a[r].v[s][1], ah[r], am[r], al[r]);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint16_t* q = pb + 16 * b * LDH + 32 * s;
      const bf16x8 bh = frag(q), bm = frag(q + kPlaneElems), bl = frag(q + 2 * kPlaneElems);
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        f32x4 c = acc[r].c[b];
        if constexpr (SUM != CHAIN) c = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (SUM == APART_ALL) {
          c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bm, al[r], c, 0, 0, 0);
          c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bl, am[r], c, 0, 0, 0);
        }
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh, al[r], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bl, ah[r], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bm, am[r], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh, am[r], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bm, ah[r], c, 0, 0, 0);
        if constexpr (SUM != CHAIN)
          acc[r].c[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh, ah[r], acc[r].c[b], 0, 0, 0) + c;
        else
          acc[r].c[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh, ah[r], c, 0, 0, 0);
      }
    }
  }
}

// Accumulate the tile over the chunks of k in [kbeg, kend) (at least one, all
// inside A's rows), starting from the first chunk already loaded into ra, rb (so
// a caller can issue other loads after them: the first wait then excludes those),
// the B planes staged through `lds` (kLdsBytes); with SQ also this lane's float64
// squares of A.  Later chunks are loaded when they are due, not a chunk ahead: a
// prefetch register set would cost the occupancy that hides those loads behind
// the other workgroups' matrix work.  The caller's first use of lds afterwards
// must follow a barrier.
template <bool SQ, int RB, Sum SUM>
__device__ __forceinline__ void tile_run(uint16_t* lds, const ARows<RB>& arows, const BRows& brows,
                                         int kbeg, int kend, AChunk (&ra)[RB], BChunk& rb, Acc (&acc)[RB],
                                         double (&sq)[RB]) {
  store_b(lds, rb);
  __syncthreads();
  if constexpr (SQ) {
#pragma unroll
    for (int r = 0; r < RB; ++r) sq[r] += squares(ra[r]);
  }
  mma_chunk<RB, SUM>(lds, ra, acc);
  for (int k0 = kbeg + KC; k0 < kend; k0 += KC) {
    load_b(brows, k0, rb);
    load_a<RB>(arows, k0, ra);
    __syncthreads();  // every wavefront is done with the previous chunk
    store_b(lds, rb);
    __syncthreads();
    if constexpr (SQ) {
#pragma unroll
      for (int r = 0; r < RB; ++r) sq[r] += squares(ra[r]);
    }
    mma_chunk<RB, SUM>(lds, ra, acc);
  }
}

// The last, partial chunk at k0 of rows of len elements.
template <bool SQ, int RB, Sum SUM>
__device__ __forceinline__ void tile_tail(uint16_t* lds, const ARows<RB>& arows, const BRows& brows, int k0,
                                          int len, Acc (&acc)[RB], double (&sq)[RB]) {
  AChunk ra[RB];
  BChunk rb;
  load_b(brows, k0, rb);
  load_a_tail<RB>(arows, k0, len, ra);
  __syncthreads();
  store_b(lds, rb);
  __syncthreads();
  if constexpr (SQ) {
#pragma unroll
    for (int r = 0; r < RB; ++r) sq[r] += squares(ra[r]);
  }
  mma_chunk<RB, SUM>(lds, ra, acc);
}

// Row (inside the tile) of row block r's accumulators of this lane, and the
// first of their four columns in block b.
template <int RB>
__device__ __forceinline__ int out_row(int r) {
  return 16 * (RB * (threadIdx.x >> 6) + r) + (threadIdx.x & 15);
}
__device__ __forceinline__ int out_col(int b) { return 16 * b + 4 * ((threadIdx.x >> 4) & 3); }

}  // namespace split
}  // namespace sd
