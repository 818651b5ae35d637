// Two-part fp16 split and three-part bf16 split of FP32 values and the
// fragment-blocked operand planes of the split products (k_xgemm.hip,
// k_xgemm3.hip, and the batched kernel's in k_batch.hip).
//
// A row (or column) of an operand is first scaled by a power of two that
// brings its largest component into [2^13, 2^14); the product's epilogue
// takes the scales out again, so both steps are exact.  The scaled value x
// is split as x = h + l + r, h = fp16(x), l = fp16(x - h), both rounded to
// nearest even: h holds 11 significand bits, x - h is exact in FP32, and l
// holds the next 11 with its sign, so |r| <= 2^-23 |x|; below 2^-15 of the
// row's largest, where l is an fp16 subnormal of spacing 2^-24, |r| <= 2^-25
// in the scaled range (2^-38 of the row's largest).
//
// Planes of a d x d complex matrix as the row operand of a product (row r,
// k = column): unit (rb, kb, g, s) of 1 KB holds rows 32 rb .. 32 rb + 31,
// k = 16 kb .. 16 kb + 15 of group g (re, im) and part s (h, l); lane u of
// the unit holds row 32 rb + u % 32, k = 16 kb + 8 (u / 32) .. + 7 as one
// 16-byte vector (the MFMA fragment of that lane).  Unit (rb, kb, g, s)
// starts at vector (((rb * d / 16 + kb) * 2 + g) * 2 + s) * 64.
#pragma once

#include "qst_device.h"
#include "qst_plan.h"

namespace qst {

constexpr int kX6UnitVecs = 64;                // 16-byte vectors per 1 KB unit
constexpr int kX6BlockVecs = 4 * kX6UnitVecs;  // the four units of one (row block, K panel)

typedef _Float16 h16x8 __attribute__((ext_vector_type(8)));

// Exponent e of the power-of-two scale for a largest component m: m 2^e in
// [2^top, 2^(top + 1)); 0 for m = 0 and for a non-finite m (whose row holds
// an infinity or NaN and comes out as NaN at any scale).  |e| <= 126, so
// that 2^e and 2^-e are both normal.
__device__ __forceinline__ int x6_scale_exp(float m, int top) {
  if (!(m > 0.f) || m > 3.402823466e38f) return 0;
  const int e = top + 1 - __builtin_amdgcn_frexp_expf(m);
  return e > 126 ? 126 : (e < -126 ? -126 : e);
}
__device__ __forceinline__ bool x6_finite(float m) { return m <= 3.402823466e38f; }
__device__ __forceinline__ float x6_pow2(int e) { return __builtin_amdgcn_ldexpf(1.0f, e); }
// top of the scaled range: sums of two components of a row stay below 2^15
constexpr int kX6Top = 13;
// An operand is dense where at least three quarters of the entries of every
// piece of a row (column) have a component not below 2^-bits of the row's
// (column's) largest.  Two dense operands then have at least half of the
// terms of every sum of their product with both factors that large, and
// FP32 accumulation, which rounds at every one of them, loses more than the
// split does per term: sqrt(d / 4) roundings of the partial sums against
// about four of the terms.  12 bits are the most that leaves such terms above
// 2^-24 of the largest product (and an entry all its 22 bits); at d = 128 to
// 512, where d / 4 is not many, 8, which is what a heavy last column needs.  Least
// fraction of any piece within 2^-12 at N = 10 and 11: Gaussian T 0.97, the
// absolute map's T 0.91 (its diagonal is 2^5 above the rest), G' 0.94 for
// three Pauli bases, 0.98 for Gaussian T; within 2^-8 those fall to 0.94,
// 0.41, 0.32 and 0.91.
// Besides, at least an eighth of the indices of the contraction (columns of T
// for T T^dagger; columns of G' and rows of T for G' T) have their largest
// component within 2^-4 of the largest of all: else a few terms carry every
// sum, and FP32 rounds it little where they come last (the last column of T
// 2^7 above the rest, N = 10: 7.6e-8 against 1.5e-7).
constexpr float kX6Near = 1.f / 16.f;
__device__ __forceinline__ bool x6_sparse(const X6Gate& g) {
  // all four loads in flight together: they miss the caches in every kernel
  const int b0 = *g.bad[0], b1 = *g.bad[1], n0 = *g.near[0], n1 = *g.near[1];
  return (b0 | b1 | int(n0 < g.least) | int(n1 < g.least)) != 0;
}
constexpr int x6_dense_bits(int n) { return n >= 10 ? 12 : 8; }
constexpr float x6_dense_low(int n) { return float(1 << (kX6Top - x6_dense_bits(n))); }

// H + L = the split of sc * x, eight values.
__device__ __forceinline__ void split2(const float (&x)[8], float sc, u16x8& H, u16x8& L) {
  h16x8 h, l;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float v = x[i] * sc;
    h[i] = (_Float16)v;
    l[i] = (_Float16)(v - (float)h[i]);
  }
  H = __builtin_bit_cast(u16x8, h);
  L = __builtin_bit_cast(u16x8, l);
}

// One lane's slot of a unit block: 8 values (re, im) scaled by sc, two
// parts each.  out points at the unit block's first unit plus the lane.
// Returns how many of the 8 values have a scaled component not below low.
__device__ __forceinline__ int write_unit_block(u16x8* out, const float (&re)[8], const float (&im)[8], float sc,
                                                float low = 0.f) {
  split2(re, sc, out[0 * kX6UnitVecs], out[1 * kX6UnitVecs]);
  split2(im, sc, out[2 * kX6UnitVecs], out[3 * kX6UnitVecs]);
  int n = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) n += int(fmaxf(fabsf(re[e]), fabsf(im[e])) * sc >= low);
  return n;
}

// Three-part bf16 split: x = h + m + l exactly for every finite FP32 x above
// 2^-110: h = bf16(x), m = bf16(x - h), l = bf16(x - h - m), each rounded to
// nearest even; x - h and x - h - m are exact in FP32, and the three parts
// carry 3 x 8 significand bits and FP32's exponent range.  Planes as above,
// three units (h, m, l) per group; groups re, im, re + im and, with NG = 4,
// re - im.
__device__ __forceinline__ uint32_t bf16x2_rne(float a, float b) {
  typedef __bf16 bf2v_t __attribute__((ext_vector_type(2)));
  const bf2v_t v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ void split3(const float (&x)[8], u16x8& H, u16x8& M, u16x8& L) {
  u32x4 h, m, l;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = bf16x2_rne(x[2 * i], x[2 * i + 1]);
    float r0 = x[2 * i] - bf16_lo(h[i]), r1 = x[2 * i + 1] - bf16_hi(h[i]);
    m[i] = bf16x2_rne(r0, r1);
    r0 -= bf16_lo(m[i]);
    r1 -= bf16_hi(m[i]);
    l[i] = bf16x2_rne(r0, r1);
  }
  H = __builtin_bit_cast(u16x8, h);
  M = __builtin_bit_cast(u16x8, m);
  L = __builtin_bit_cast(u16x8, l);
}

// One lane's slot of a three-part unit block.
template <int NG>
__device__ __forceinline__ void write_unit_block3(u16x8* out, const float (&re)[8], const float (&im)[8]) {
  float g2[8];
  split3(re, out[0 * kX6UnitVecs], out[1 * kX6UnitVecs], out[2 * kX6UnitVecs]);
  split3(im, out[3 * kX6UnitVecs], out[4 * kX6UnitVecs], out[5 * kX6UnitVecs]);
#pragma unroll
  for (int e = 0; e < 8; ++e) g2[e] = re[e] + im[e];
  split3(g2, out[6 * kX6UnitVecs], out[7 * kX6UnitVecs], out[8 * kX6UnitVecs]);
  if constexpr (NG == 4) {
#pragma unroll
    for (int e = 0; e < 8; ++e) g2[e] = re[e] - im[e];
    split3(g2, out[9 * kX6UnitVecs], out[10 * kX6UnitVecs], out[11 * kX6UnitVecs]);
  }
}

}  // namespace qst
