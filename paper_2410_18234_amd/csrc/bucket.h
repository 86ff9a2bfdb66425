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

namespace mdss {
namespace {

constexpr int kBqSub = 32;               // parts of an octave
constexpr int kBqDeg = 3;                // degree of a part's polynomial
constexpr int kBqLen = kBqDeg + 1;       // its coefficients
constexpr int kBqOct = kBqSub * kBqLen;  // values per octave
constexpr int kBqNearLo = -12;           // s <= -13 (a_k w <= 2^-5.5): five terms of the power series
constexpr int kBqNearHi = 9;             // s >= 10 (a_k w >= 32): the term is dropped
constexpr int kBqNear = kBqNearHi - kBqNearLo + 1;
constexpr int kBqFar = 5;                // power series terms

constexpr int kBqCols = kBqNear + kBqFar;  // contractions of an octave's sums: near nodes, then power sums

struct BqTables {
  // [s - kBqNearLo][j * kBqLen + n]: G; then for i < kBqFar the coefficient of t^n in (c_j + d t)^i
  double g[kBqCols][kBqOct];
};

// e^-x for x in [0, 46] from the series of e^-(x / 64), squared six times
constexpr double bq_expm(double x) {
  const double y = -x / 64.0;
  double s = 1.0, term = 1.0;
  for (int i = 1; i < 22; ++i) {
    term *= y / i;
    s += term;
  }
  for (int i = 0; i < 6; ++i) s *= s;
  return s;
}

constexpr BqTables bq_make_tables() {
  BqTables o{};
  // Chebyshev nodes cos((2 i + 1) pi / 8), and the Lagrange basis in powers of t
  constexpr double x[kBqLen] = {0.92387953251128675613, 0.38268343236508977173, -0.38268343236508977173,
                                -0.92387953251128675613};
  double basis[kBqLen][kBqLen] = {};  // basis[i][n]
  for (int i = 0; i < kBqLen; ++i) {
    double poly[kBqLen] = {1.0, 0.0, 0.0, 0.0};
    double den = 1.0;
    int deg = 0;
    for (int m = 0; m < kBqLen; ++m) {
      if (m == i) continue;
      den *= x[i] - x[m];
      ++deg;
      for (int n = deg; n >= 1; --n) poly[n] = poly[n - 1] - x[m] * poly[n];
      poly[0] = -x[m] * poly[0];
    }
    for (int n = 0; n < kBqLen; ++n) basis[i][n] = poly[n] / den;
  }
  double z = 0.015625;  // 2^(kBqNearLo / 2)
  double zo = z * 1.41421356237309504880;
  for (int s = 0; s < kBqNear; ++s) {
    const double zs = (s & 1) ? zo : z;
    for (int j = 0; j < kBqSub; ++j) {
      for (int i = 0; i < kBqLen; ++i) {
        const double v = bq_expm(zs * (1.0 + (j + 0.5 + 0.5 * x[i]) / kBqSub));
        for (int n = 0; n < kBqLen; ++n) o.g[s][j * kBqLen + n] += v * basis[i][n];
      }
    }
    if (s & 1) {
      z *= 2.0;
      zo *= 2.0;
    }
  }
  for (int j = 0; j < kBqSub; ++j) {
    const double c = 1.0 + (j + 0.5) / kBqSub, d = 0.5 / kBqSub;
    for (int i = 0; i < kBqFar; ++i) {
      for (int n = 0; n <= i && n < kBqLen; ++n) {
        double v = 1.0;
        for (int m = 0; m < n; ++m) v = v * (i - m) / (m + 1) * d;  // C(i, n) d^n
        for (int m = 0; m < i - n; ++m) v *= c;
        o.g[kBqNear + i][j * kBqLen + n] = v;
      }
    }
  }
  return o;
}

constexpr BqTables kBqTab = bq_make_tables();
__constant__ BqTables kBq = kBqTab;

// The same in the order a wave's v_mfma_f64_16x16x4_f64 reads its B operand: columns 16 ct .. (past the last they
// repeat it), values 4 t .., lane by lane.
struct BqFragments {
  double g[2][kBqOct / 4][64];
};
constexpr BqFragments bq_make_fragments() {
  BqFragments o{};
  for (int ct = 0; ct < 2; ++ct)
    for (int t = 0; t < kBqOct / 4; ++t)
      for (int lane = 0; lane < 64; ++lane) {
        const int col = ct * 16 + lane % 16;
        o.g[ct][t][lane] = kBqTab.g[col < kBqCols ? col : kBqCols - 1][4 * t + lane / 16];
      }
  return o;
}
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
