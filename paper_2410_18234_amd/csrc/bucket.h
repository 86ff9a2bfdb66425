// Fixed tables and per-token arithmetic of the bucketed quadrature (bucket.hip).
//
// Every positive fp32 ratio w = p / q lies in one bucket: its binary exponent e
// (its octave) and the kBqSub equal parts of [2^e, 2^(e+1)).  Inside part j
//   w = 2^e (c_j + d t),  c_j = 1 + (j + 1/2) / kBqSub,  d = 1 / (2 kBqSub),  t in [-1, 1),
// and on the nodes a_k = 2^(k/2) every term exp(-a_k w) depends on k and e only through
// s = k + 2 e:  exp(-2^(s/2) (c_j + d t)) = sum_n G[s][j][n] t^n, a polynomial of degree
// kBqDeg (Chebyshev interpolation).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bucket_tables.h"

namespace mdss {
namespace {

__constant__ BqTables kBq = kBqTab;
__constant__ BqFragments kBqFrag = bq_make_fragments();

static_assert(kBqSub == 32, "the bit fields below and above take five mantissa bits");

// A token in fp32, for p, q and p / q inside [2^-96, 2^96]: the bucket of the rounded quotient
// w0, and t / 64 of the quotient itself: the remainder p - w0 q (one fma) corrects w0's mantissa,
// so t is off by fp32 rounding of a number in [-1, 1], 2^-24 (r: below 1e-9; t may leave [-1, 1]
// by 2^-17 for a quotient next to a part's edge).  w0 is a positive normal exactly when p and q are
// positive (0 for p = 0, infinite or NaN for q = 0).
struct BqTok {
  float w, t;
  uint32_t at;  // w0's exponent and part: kBqSub times the biased exponent, plus the part
};
__device__ __forceinline__ BqTok bq_tok(float p, float q) {
  const float y = __builtin_amdgcn_rcpf(q);
  BqTok k;
  k.w = p * y;
  const uint32_t bits = __float_as_uint(k.w);
  const float rest = fmaf(-k.w, q, p) * y;
  const float x = __uint_as_float((bits & 0x3FFFFu) | 0x3F800000u);  // [1, 1 + 1/32)
  const float up = __uint_as_float((uint32_t)(254 << 23) - (bits & 0x7F800000u));  // 2^-e, e the exponent of w0
  k.t = fmaf(rest, up, x - (1.0f + 0.5f / kBqSub));
  k.at = bits >> 18;
  return k;
}
constexpr float kBqTUnit = 0.5f / kBqSub;  // the unit of BqTok::t
// The same for any two positive fp32 numbers, from their mantissas and exponents; `at` as an
// integer (kBqSub times the biased exponent may be negative or past the fp32 range).
struct BqWideTok {
  float t;
  int at;
};
__device__ __forceinline__ BqWideTok bq_wide_tok(float p, float q) {
  const BqTok k = bq_tok(__builtin_amdgcn_frexp_mantf(p), __builtin_amdgcn_frexp_mantf(q));
  return {k.t, (int)k.at + kBqSub * (__builtin_amdgcn_frexp_expf(p) - __builtin_amdgcn_frexp_expf(q))};
}
__device__ __forceinline__ bool bq_positive(float w) { return __builtin_amdgcn_classf(w, 0x100); }
// nearest integer (halves up)
__device__ __forceinline__ int bq_round(float x) {
  int n;
  __asm__("v_cvt_rpi_i32_f32 %0, %1" : "=v"(n) : "v"(x));
  return n;
}

// 2^(s / 2)
__device__ __forceinline__ double bq_half_pow(int s) { return ldexp((s & 1) ? 1.41421356237309504880 : 1.0, s >> 1); }

}  // namespace
}  // namespace mdss
