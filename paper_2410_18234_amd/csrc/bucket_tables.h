// Fixed tables of the bucketed quadrature (bucket.h states what they stand for), computed from their series at
// compile time; host code only.
#pragma once

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

}  // namespace
}  // namespace mdss
