// Two-part fp16 split of FP32 values and the fragment-blocked operand
// planes of the split products (written by the split kernel of k_xgemm.hip
// and, in the combined likelihood-and-gradient call, by the last adjoint
// POVM stage).
//
// A row (or column) of an operand is first scaled by a power of two that
// brings its largest component into [2^13, 2^14); the product's epilogue
// takes the scales out again, so both steps are exact.  The scaled value x
// is split as x = h + l + r, h = fp16(x), l = fp16(x - h), both rounded to
// nearest even: h holds 11 significand bits, x - h is exact in FP32, and l
// holds the next 11 with its sign, so |r| <= 2^-23 |x| (2^-25 at most
// otherwise: entries below 2^-15 of the row's largest, where l is an fp16
// subnormal of spacing 2^-24).
//
// Planes of a d x d complex matrix as the row operand of a product (row r,
// k = column): unit (rb, kb, g, s) of 1 KB holds rows 32 rb .. 32 rb + 31,
// k = 16 kb .. 16 kb + 15 of group g (re, im) and part s (h, l); lane u of
// the unit holds row 32 rb + u % 32, k = 16 kb + 8 (u / 32) .. + 7 as one
// 16-byte vector (the MFMA fragment of that lane).  Unit (rb, kb, g, s)
// starts at vector (((rb * d / 16 + kb) * 2 + g) * 2 + s) * 64.
#pragma once

#include "qst_device.h"

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
__device__ __forceinline__ float x6_pow2(int e) { return __builtin_amdgcn_ldexpf(1.0f, e); }
// top of the scaled range: sums of two components of a row stay below 2^15
constexpr int kX6Top = 13;

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
__device__ __forceinline__ void write_unit_block(u16x8* out, const float (&re)[8], const float (&im)[8], float sc) {
  split2(re, sc, out[0 * kX6UnitVecs], out[1 * kX6UnitVecs]);
  split2(im, sc, out[2 * kX6UnitVecs], out[3 * kX6UnitVecs]);
}

}  // namespace qst
