// Induced distribution r by a bucketed exponential-sum quadrature, gfx950.
//
// Notation: p = target, q = draft, w = p / q.  With the classical weights the
// selected-token law (proof of Theorem 1, eq. Ind; for K = 2 the pair form
// eq. p_Ieq0) is, for q(y) > 0 and p(y) > 0,
//   K i.i.d. drafts:  r(y) = K p(y) sum_{x_2..x_K in supp q} prod_j q(x_j) / (w(y) + sum_j w(x_j)),
//   two draft laws:   r(y) = p(y) [ sum_x q2(x) / (w1(y) + w2(x)) + sum_x q1(x) / (w1(x) + w2(y)) ],
// plus the closed forms of the zero-weight tokens.  Every denominator D is a sum of
// positive weights and 1 / D = integral over t of exp(t - D e^t) dt, so with
// S(a) = sum_x q(x) exp(-a w(x)) the trapezoidal rule on t_k = k h turns the sums into
//   r(y) = p(y) sum_k c_k exp(-a_k w(y)),   c_k = K h a_k S(a_k)^(K-1),   a_k = e^(t_k)
// (two laws: c_k = h a_k S_other(a_k)).  Here h = ln(2) / 2, so a_k = 2^(k/2), and the rule
// is within 2 |Gamma(1 + 2 pi i / h)| = 9e-12 of 1 / D, whatever D.
//
// Buckets.  A token enters only through its bucket (octave e and part j of w, bucket.h) and
// its place t in it, because a part's exp(-a_k w) is a polynomial in t with coefficients
// G[k + 2e][j][n].  So the row is summed once into M[e][j][n] = sum q t^n, and
//   S(a_k) = sum over (e, j, n) of M[e][j][n] G[k + 2e][j][n],
// and the row of a query's bucket is the transposed contraction A[e][j][n] = sum_k c_k
// G[k + 2e][j][n]: r(y) = p(y) sum_n A[e][j][n] t^n.  Nodes with a_k w <= 2^-5.5 take five
// terms of the power series per octave instead (error 4e-11), terms with a_k w >= 32 are
// dropped (1.5e-13), the grid starts where a_k D is below 1e-10.  Interpolation is the
// largest error: at most 6e-9 relative per entry (measured over rows of 1 to 32000 tokens,
// in fp64), so r is within its fp32 rounding.
//
// Order and precision.  M is summed by integer LDS atomics: q t^n scaled by a power of two, the
// bucket's largest q into [2^29, 2^30), and rounded to an integer (n = 2 and 3 to 18 and 12 bits:
// their share of a term is below 0.005 and 0.0002).  Integer sums do not depend on the order, so r
// is the same bit for bit on every run.  Everything after is fp64; a part's polynomial is kept as
// a_0 in two fp32 numbers and a_1 .. a_3 in one each (below 0.02 of the value).
//
// Measured (256 x 32000, K = 2, with the residual sums): 52 us, against 75 us for three kernels
// that took nine exponentials a token on the way in (their fp32 sums left r 7.5e-8 off in the
// 2-norm; 2.4e-8 here, all of it r's own rounding).  At 60 us a step: reading p and q 12 us, (B)
// 12 us (three 64-bit LDS atomics a token, 13 cycles a wave each), (C) 6 us, (D) with the drain of
// r's stores 15 us.
//
// Forms.  Rows whose probabilities and ratios stay inside [2^-96, 2^20] and [2^-96, 2^96] and
// whose ratios span at most 64 octaves take the fp32 per-token arithmetic of bucket.h:
//   bq_row_kernel   one workgroup of 1024 threads a row, the row in registers from its first
//                   load to r: (A) the largest q of every bucket, (B) the integer sums, (C) S,
//                   c and the parts' polynomials, (D) r and Algorithm 1's residual sums;
//   bq_part_kernel, bq_merge_kernel, bq_eval_kernel   the same with (A) and (B) on chunks of a
//                   row, (C) per row from the chunks' sums, (D) on tiles: long rows, few rows,
//                   two laws.
// Every other row (and calls without room for the chunks' sums) is taken by bq_row_general,
// which streams the row for every pass, on mantissas and exponents, 64 octaves at a time.
#include "bucket.h"
#include "common.h"

#include <math.h>

#include <algorithm>

namespace mdss {

namespace {

constexpr int kBqThreads = 1024;
constexpr int kBqWaves = kBqThreads / 64;
constexpr int kBqStep = 4 * kBqThreads;  // tokens per streaming step (four a thread)
constexpr int kBqWin = 64;               // octaves held in LDS
constexpr int kBqWinRows = kBqWin * kBqSub;
constexpr int kBqMaxNodes = 1280;        // fp32 ratios span at most 554 octaves: 2 * 554 + 85 nodes
constexpr int kBqGPad = kBqOct + 1;      // LDS stride of a node's table row
constexpr double kBqStepH = 0.34657359027997265471;      // h = ln(2) / 2
// The MDSS_ROW_RANGE rule of the quadrature entry points: more than kBqRangeNodes nodes of step
// 1/2 between the points where the tails fall below 1e-8.
constexpr int kBqRangeNodes = 480;
constexpr double kBqLnEps = -18.420680743952367;         // ln 1e-8
constexpr double kBqLnLnInvEps = 2.9134941423228814;     // ln ln 1e8

struct BqArgs {
  const float *p, *q1, *q2;
  int64_t V;
  int K;
  int s_max;       // > 0: a row with more support tokens is flagged
  int range_flag;  // rows spanning more than 2^300 are flagged (the quadrature entry points)
  int set_status;  // row_status is set, not OR-ed into
  float* r;
  int32_t* row_status;
  double* rsum;    // [B][nsub][kResParts] residual sums (kRes)
  int64_t nsub;
};

__device__ __forceinline__ void bq_load_table(double* g, int tid) {
  for (int x = tid; x < kBqCols * kBqOct; x += kBqThreads) g[(x / kBqOct) * kBqGPad + x % kBqOct] = (&kBq.g[0][0])[x];
}

// r of one token from its laws' sums.
template <int L>
__device__ __forceinline__ float bq_out(float pp, const float (&qq)[L], double sum, int K, const double (&q0)[L],
                                        double zw) {
  const double quad = (double)pp * sum;
  if (L == 1) {
    const double qd = (double)qq[0];
    const double pos = (K == 2) ? ::fma(2.0 * qd, q0[0], quad) : quad;
    const double v = pp > 0.0f ? pos : qd * zw;
    return qq[0] > 0.0f ? (float)v : 0.0f;
  }
  // a zero-weight pole of the other draft adds q_i(y) Qj_0; a zero target splits it in half
  const double za = qq[0] > 0.0f ? (double)qq[0] * q0[L - 1] : 0.0, zc = qq[L - 1] > 0.0f ? (double)qq[L - 1] * q0[0] : 0.0;
  return (float)(pp > 0.0f ? quad + za + zc : 0.5 * (za + zc));
}

// ------------------------------------------------------------------ fp32 tokens
constexpr float kBqTiny = 0x1p-96f, kBqHuge = 0x1p96f, kBqLarge = 0x1p20f;
constexpr int kBqPer = 32;       // tokens a thread, at most
constexpr int kBqFastNodes = 256;
// Integer sums of a bucket over at most 2^15 tokens, v = q 2^F / 2^(e_q) in [0, 2^30), u = t / 64:
// v and v u (signed) in 64 bits each, v u^2 (below 2^18 a token) in the low 34 bits and v u^3
// (signed, below 2^12) above.
constexpr int kBqF = 29;
constexpr int kBqAcc = 3;
constexpr int kBqPack = 34;
static_assert(kBqPer * kBqThreads <= 1 << 15, "the packed sums");

template <int L>
struct BqFastStats {
  uint32_t mx = 0u, mn = 0xFFFFFFFFu;  // bits of p and q: largest; smallest non-zero, minus one
  bool bad = false;
  int nsup = 0;                        // wave-uniform
  uint32_t lo[L], hi[L];               // bits of the positive ratios: smallest minus one, largest
  double q0[L];
  __device__ __forceinline__ BqFastStats() {
#pragma unroll
    for (int l = 0; l < L; ++l) {
      lo[l] = 0xFFFFFFFFu;
      hi[l] = 0u;
      q0[l] = 0.0;
    }
  }
};

// What the workgroup knows of its tokens after (A), the same in every thread.
template <int L>
struct BqRange {
  bool bad, special;
  int nsup;
  int e0[L], e1[L];  // biased exponents of the ratios (e1 = 0: no token in the sums)
  double q0[L];
};

template <int L>
struct BqSumsShared {
  uint64_t acc[kBqWinRows * kBqAcc];  // one law's
  uint32_t qm[L][kBqWinRows];         // largest q of a bucket (bits), then the bits of its scale
};
template <int L, int W>
struct BqStatShared {
  double q0[L][W];
  uint32_t u[4 + 2 * L][W];
};

template <int L>
__device__ __forceinline__ void bq_fast_count(const float (&pv)[4], const float (&qv)[L][4], BqSumsShared<L>& sh,
                                              BqFastStats<L>& st, bool support) {
#pragma unroll
  for (int l = 0; l < L; ++l) {
    uint32_t w[4];
    bool zero = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t pu = __float_as_uint(pv[i]), qu = __float_as_uint(qv[l][i]);
      st.mx = max(st.mx, max(pu, qu));
      st.mn = min(st.mn, min(pu - 1u, qu - 1u));
      const bool some = qv[l][i] > 0.0f;
      w[i] = some ? __float_as_uint(pv[i] * __builtin_amdgcn_rcpf(qv[l][i])) : 0u;
      zero |= some && w[i] == 0u;
      st.lo[l] = min(st.lo[l], w[i] - 1u);
      st.hi[l] = max(st.hi[l], w[i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (w[i] != 0u) atomicMax(&sh.qm[l][(w[i] >> 18) & (kBqWinRows - 1)], __float_as_uint(qv[l][i]));
    if (support) {
#pragma unroll
      for (int i = 0; i < 4; ++i) st.nsup += (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(qv[l][i] > 0.0f));
    }
    if (__builtin_amdgcn_ballot_w64(zero) != 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) st.q0[l] += (qv[l][i] > 0.0f && pv[i] == 0.0f) ? (double)qv[l][i] : 0.0;
    }
    if (__builtin_amdgcn_ballot_w64(st.mx >= 0x7F800000u) != 0) {  // NaN, infinite, negative or -0 somewhere
#pragma unroll
      for (int i = 0; i < 4; ++i)
        st.bad |= __builtin_amdgcn_classf(pv[i], 0x21F) | __builtin_amdgcn_classf(qv[l][i], 0x21F);
    }
    // the running extremes are taken here, not put off to the end (with every token's ratio kept)
    __asm__ volatile("" : "+v"(st.mx), "+v"(st.mn), "+v"(st.lo[l]), "+v"(st.hi[l]));
  }
}

template <int CTRL>
__device__ __forceinline__ uint32_t bq_dpp(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
}
// Minimum / maximum over the 64 lanes (in every lane): quad permutations, row rotations, row swaps.
template <bool MAX>
__device__ __forceinline__ uint32_t bq_pick(uint32_t a, uint32_t b) {
  return MAX ? max(a, b) : min(a, b);
}
template <bool MAX>
__device__ __forceinline__ uint32_t bq_row16(uint32_t x) {  // over each 16-lane row
  x = bq_pick<MAX>(x, bq_dpp<0xB1>(x));
  x = bq_pick<MAX>(x, bq_dpp<0x4E>(x));
  x = bq_pick<MAX>(x, bq_dpp<0x124>(x));
  return bq_pick<MAX>(x, bq_dpp<0x128>(x));
}
template <bool MAX>
__device__ __forceinline__ uint32_t bq_wave(uint32_t x) {
  x = bq_row16<MAX>(x);
  auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = bq_pick<MAX>(r[0], r[1]);
  r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return bq_pick<MAX>(r[0], r[1]);
}

// The waves' statistics combined (one barrier): every wave reads them, a lane a wave.
template <int L, int W>
__device__ __forceinline__ BqRange<L> bq_combine(BqFastStats<L>& st, BqStatShared<L, W>& sh, int lane, int wid) {
  static_assert(W <= 16 && (W & (W - 1)) == 0, "a 16-lane row holds every wave");
  const bool bad = __builtin_amdgcn_ballot_w64(st.bad) != 0;
  const uint32_t mx = bq_wave<true>(st.mx), mn = bq_wave<false>(st.mn);
#pragma unroll
  for (int l = 0; l < L; ++l) {
    st.lo[l] = bq_wave<false>(st.lo[l]);
    st.hi[l] = bq_wave<true>(st.hi[l]);
    if (__builtin_amdgcn_ballot_w64(st.q0[l] != 0.0) != 0) st.q0[l] = wave_sum_dpp(st.q0[l]);
  }
  if (lane == 0) {
    sh.u[0][wid] = mx;
    sh.u[1][wid] = mn;
    sh.u[2][wid] = bad ? 1u : 0u;
    sh.u[3][wid] = (uint32_t)st.nsup;
#pragma unroll
    for (int l = 0; l < L; ++l) {
      sh.u[4 + 2 * l][wid] = st.lo[l];
      sh.u[5 + 2 * l][wid] = st.hi[l];
      sh.q0[l][wid] = st.q0[l];
    }
  }
  __syncthreads();
  const int w = lane & (W - 1);
  BqRange<L> o;
  const uint32_t amx = bq_row16<true>(sh.u[0][w]), amn = bq_row16<false>(sh.u[1][w]);
  o.bad = __builtin_amdgcn_readfirstlane(bq_row16<true>(sh.u[2][w])) != 0u;
  int n = 0;
#pragma unroll
  for (int i = 0; i < W; ++i) n += (int)sh.u[3][i];
  o.nsup = __builtin_amdgcn_readfirstlane(n);
  bool special = amx > __float_as_uint(kBqLarge) || amn < __float_as_uint(kBqTiny);
#pragma unroll
  for (int l = 0; l < L; ++l) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane(bq_row16<false>(sh.u[4 + 2 * l][w]));
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane(bq_row16<true>(sh.u[5 + 2 * l][w]));
    double q0 = 0.0;
#pragma unroll
    for (int i = 0; i < W; ++i) q0 += sh.q0[l][i];
    o.q0[l] = q0;
    const bool some = hi != 0u;
    special |= some && (lo < __float_as_uint(kBqTiny) || hi > __float_as_uint(kBqHuge));
    o.e0[l] = some ? (int)((lo + 1u) >> 23) : 0x7FFFFFF;
    o.e1[l] = some ? (int)(hi >> 23) : 0;
    special |= some && o.e1[l] - o.e0[l] >= kBqWin;
  }
  o.special = __builtin_amdgcn_readfirstlane(special ? 1 : 0) != 0;
  return o;
}

// largest q of each bucket -> 2^(kBqF - e_q)
template <int L>
__device__ __forceinline__ void bq_fast_scales(BqSumsShared<L>& sh, int tid, int threads) {
#pragma unroll
  for (int l = 0; l < L; ++l)
    for (int x = tid; x < kBqWinRows; x += threads) {
      const uint32_t ef = sh.qm[l][x] >> 23;  // 0 for an empty bucket, else >= 31
      sh.qm[l][x] = ef ? (uint32_t)(254 + kBqF - (int)ef) << 23 : 0u;
    }
}

// Law l's sums: every token's values first, then the atomics.
template <int L>
__device__ __forceinline__ void bq_fast_add(const float (&pv)[4], const float (&qv)[4], BqSumsShared<L>& sh, int l) {
  BqTok k[4];
  int at[4];
  float sc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    k[i] = bq_tok(pv[i], qv[i]);
    at[i] = (int)(k[i].at & (kBqWinRows - 1));
    sc[i] = __uint_as_float(sh.qm[l][at[i]]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float v0 = qv[i] * sc[i];
    const float v1 = v0 * k[i].t;
    const float v2 = v1 * k[i].t;
    uint32_t n0 = (uint32_t)bq_round(v0);
    int n1 = bq_round(v1), n2 = bq_round(v2), n3 = bq_round(v2 * k[i].t) << (kBqPack - 32);
    __asm__ volatile("" : "+v"(n0), "+v"(n1), "+v"(n2), "+v"(n3));  // not sunk into the branch
    if (bq_positive(k[i].w)) {
      unsigned long long* a = reinterpret_cast<unsigned long long*>(&sh.acc[at[i] * kBqAcc]);
      atomicAdd(a, (unsigned long long)n0);
      atomicAdd(a + 1, (unsigned long long)(long long)n1);
      atomicAdd(a + 2, ((unsigned long long)(uint32_t)n3 << 32) | (uint32_t)n2);
    }
  }
}

// M of a bucket: value n of its polynomial sums, from the integer sums.
template <int L>
__device__ __forceinline__ double bq_decode(const BqSumsShared<L>& sh, int l, int at, int n) {
  const uint32_t sc = sh.qm[l][at];
  const int64_t raw = (int64_t)sh.acc[at * kBqAcc + min(n, 2)];
  const int64_t v = n < 2 ? raw : (n == 2 ? raw & ((1ll << kBqPack) - 1) : raw >> kBqPack);
  const double x = ldexp((double)v, 6 * n + 127 - (int)(sc >> 23));
  return sc ? x : 0.0;
}

// ------------------------------------------------------------------ (C)
// The two contractions are small dense products in fp64 and run on the matrix cores, 16 octaves
// by 16 columns a wave: S as (octaves x 128 values) x (128 x 27), the parts' polynomials as
// (octaves x 27) x (27 x 128).  On the VALU they are bound by LDS reads of the table: 3.4 us and
// 4.5 us a row of 20 octaves, against 2.6 us and 1.8 us.
typedef double BqQuad __attribute__((ext_vector_type(4)));
// v_mfma_f64_16x16x4_f64: A row / B column lane % 16 at depth lane / 16; D column lane % 16,
// rows lane / 16 + 4 i.

// n[half][o 28 + column]: octave e0 + o's values (moment(e, x)) against the near nodes and the
// power sums, each half of the 128 values apart.
template <class Moment>
__device__ __forceinline__ void bq_contract(double (*n)[kBqWin * 28], const double* g0, int e0, int noct, int lane,
                                            int wid, Moment&& moment) {
  const int mr = lane & 15, mk = lane >> 4;
  for (int u = wid; u < (noct + 15) / 16 * 4; u += kBqWaves) {
    const int ot = u >> 2, ct = (u >> 1) & 1, half = u & 1;
    const int e = e0 + min(ot * 16 + mr, noct - 1);
    const double* g = g0 + min(ct * 16 + mr, kBqCols - 1) * kBqGPad;  // columns past the last repeat it
    BqQuad d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int t = 0; t < kBqOct / 8; ++t) {
      const int x = half * (kBqOct / 2) + 4 * t + mk;
      d = __builtin_amdgcn_mfma_f64_16x16x4f64(moment(e, x), g[x], d, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = ot * 16 + mk + 4 * i;
      if (o < noct && ct * 16 + mr < kBqCols) n[half][o * 28 + ct * 16 + mr] = d[i];
    }
  }
}

// S at the nodes k_lo .. k_lo + nk - 1 from the contractions of the octaves e0 .. e1: eight groups
// of threads share the octaves out; emit(i, S) by one thread a node.  Ends with a barrier.
template <class Emit>
__device__ __forceinline__ void bq_nodes(const double (*n2)[kBqWin * 28], double (*red)[128], int e0, int e1, int k_lo,
                                         int nk, int tid, Emit&& emit) {
  const int li = tid & 127, grp = tid >> 7;
  for (int i0 = 0; i0 < nk; i0 += 128) {
    const int k = k_lo + i0 + li;
    double s = 0.0;
    for (int e = e0 + grp; e <= e1; e += 8) {
      const int sx = k + 2 * (e - 127);
      if (sx > kBqNearHi) break;  // and for every octave above
      const double* n = &n2[0][(e - e0) * 28];
      const double* m = &n2[1][(e - e0) * 28];
      if (sx >= kBqNearLo) {
        s += n[sx - kBqNearLo] + m[sx - kBqNearLo];
      } else {
        const double z = -bq_half_pow(sx);
        double f = (n[kBqNear + 4] + m[kBqNear + 4]) * (1.0 / 24.0);
        f = ::fma(f, z, (n[kBqNear + 3] + m[kBqNear + 3]) * (1.0 / 6.0));
        f = ::fma(f, z, (n[kBqNear + 2] + m[kBqNear + 2]) * 0.5);
        f = ::fma(f, z, n[kBqNear + 1] + m[kBqNear + 1]);
        s += ::fma(f, z, n[kBqNear] + m[kBqNear]);
      }
    }
    red[grp][li] = s;
    __syncthreads();
    if (grp == 0 && i0 + li < nk) {
      double t = red[0][li];
#pragma unroll
      for (int x = 1; x < 8; ++x) t += red[x][li];
      emit(i0 + li, t);
    }
    __syncthreads();
  }
}

// c_k of K i.i.d. drafts (K >= 3 keeps the zero-weight mass in S), or with two laws h a_k S of one
// for the other's queries.
template <int L>
__device__ __forceinline__ double bq_coef(double S, int k, int K, double q0) {
  const double ha = kBqStepH * bq_half_pow(k);
  if (L == 2) return ha * S;
  const double sm = S + (K >= 3 ? q0 : 0.0);
  double sp = 1.0;
  for (int j = 1; j < K; ++j) sp *= sm;
  return (double)K * ha * sp;
}

// The far nodes' series at the octaves e0 .. e0 + noct - 1 in powers of w / 2^e:
// b[o kBqFar + i] = sum_k c_k (-2^(s/2))^i / i! over s <= kBqNearLo - 1.  Eight lanes a value.
__device__ __forceinline__ void bq_far(const double* c, double* b, int e0, int noct, int k_lo, int tid) {
  for (int x = tid; x < noct * kBqFar * 8; x += kBqThreads) {
    const int part = x & 7, i = (x >> 3) % kBqFar, o = (x >> 3) / kBqFar;
    const int e2 = 2 * (e0 + o - 127);
    const int k_far = kBqNearLo - 1 - e2;
    // downwards, so that a power below the fp64 range is followed only by smaller ones
    double s = 0.0, z = bq_half_pow(i * (kBqNearLo - 1 - part));
    const double down = 1.0 / (double)(1 << (4 * i));  // eight nodes back: 2^(-8 i / 2)
    for (int k = k_far - part; k >= k_lo; k -= 8) {
      s = ::fma(c[k - k_lo], z, s);
      z *= down;
    }
    s += __shfl_xor(s, 1, 64);
    s += __shfl_xor(s, 2, 64);
    s += __shfl_xor(s, 4, 64);
    const double f = i == 0 ? 1.0 : (i == 1 ? -1.0 : (i == 2 ? 0.5 : (i == 3 ? -1.0 / 6.0 : 1.0 / 24.0)));
    if (part == 0) b[o * kBqFar + i] = s * f;
  }
}

// The parts' polynomials of the octaves e0 .. e0 + noct - 1: emit(o, y, v), coefficient y % kBqLen
// of part y / kBqLen: the near nodes' c_k, then the series (whose columns are 0 where i < n).
template <class Emit>
__device__ __forceinline__ void bq_polynomials(const double* c0, const double* b, const double* g, int e0, int noct,
                                               int k_lo, int lane, int wid, Emit&& emit) {
  const int mr = lane & 15, mk = lane >> 4;
  for (int u = wid; u < (noct + 15) / 16 * (kBqOct / 16); u += kBqWaves) {
    const int ot = u / (kBqOct / 16), y = (u % (kBqOct / 16)) * 16 + mr;
    const int oa = min(ot * 16 + mr, noct - 1);
    const double* c = c0 + (kBqNearLo - 2 * (e0 + oa - 127) - k_lo);
    const double* f = b + oa * kBqFar;
    BqQuad d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < (kBqCols + 3) / 4; ++t) {
      const int s = 4 * t + mk;
      const double v = *(s < kBqNear ? c + s : f + min(s, kBqCols - 1) - kBqNear);
      d = __builtin_amdgcn_mfma_f64_16x16x4f64(s < kBqCols ? v : 0.0, g[min(s, kBqCols - 1) * kBqGPad + y], d, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = ot * 16 + mk + 4 * i;
      if (o < noct) emit(o, y, d[i]);
    }
  }
}

// First node of a row whose weights lie below 2^(e_hi - 126): a_(k_lo) D <= 2^-33.5.
__device__ __forceinline__ int bq_first_node(int e_hi, int K) {
  const int lgk = K <= 2 ? 1 : (K <= 4 ? 2 : 3);
  return -2 * (e_hi - 127 + 1 + lgk) - 67;
}

template <int L>
struct BqSolve {
  double g[kBqCols * kBqGPad];
  double n[2][kBqWin * 28];          // contractions of one law's octaves (halves of the sum)
  double c[L][kBqFastNodes];
  double b[L][kBqWin * kBqFar];
  double red[8][128];
  int over;
};

// From M to the parts' polynomials of the octaves e0 .. e1 of every law: r4[row] = (a_0 rounded
// to fp32, a_1, a_2, a_3), r1[row] = a_0's rest, row = kBqSub (e - e0) + part.  Returns false if
// a coefficient does not fit fp32.  begin(l): before a law's octaves; moment(l, e, x): M of octave
// e, value x.  (g is readable on entry; the rows are written after barriers past the last moment().)
template <int L, class Begin, class Moment>
__device__ __forceinline__ bool bq_solve(BqSolve<L>& sh, const BqRange<L>& rg, int K, float4* const (&r4)[L],
                                         float* const (&r1)[L], int tid, int lane, int wid, Begin&& begin,
                                         Moment&& moment) {
  int e_lo = rg.e0[0], e_hi = rg.e1[0];
  if (L == 2) {
    e_lo = min(e_lo, rg.e0[L - 1]);
    e_hi = max(e_hi, rg.e1[L - 1]);
  }
  const int k_lo = bq_first_node(e_hi, K);
  const int nk = kBqNearHi - 2 * (e_lo - 127) - k_lo + 1;
  if (nk > kBqFastNodes) return false;  // two laws far apart
  if (tid == 0) sh.over = 0;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    begin(l);
    bq_contract(sh.n, sh.g, rg.e0[l], rg.e1[l] - rg.e0[l] + 1, lane, wid, [&](int e, int x) { return moment(l, e, x); });
    __syncthreads();
    bq_nodes(sh.n, sh.red, rg.e0[l], rg.e1[l], k_lo, nk, tid,
             [&](int i, double S) { sh.c[L - 1 - l][i] = bq_coef<L>(S, k_lo + i, K, rg.q0[0]); });
  }
#pragma unroll
  for (int l = 0; l < L; ++l) bq_far(sh.c[l], sh.b[l], rg.e0[l], rg.e1[l] - rg.e0[l] + 1, k_lo, tid);
  __syncthreads();
  bool over = false;
#pragma unroll
  for (int l = 0; l < L; ++l)
    bq_polynomials(sh.c[l], sh.b[l], sh.g, rg.e0[l], rg.e1[l] - rg.e0[l] + 1, k_lo, lane, wid, [&](int o, int y, double v) {
      const int row = o * kBqSub + y / kBqLen, n = y % kBqLen;
      const float a = (float)v;
      reinterpret_cast<float*>(r4[l] + row)[n] = a;
      if (n == 0) {
        over |= !(fabsf(a) <= 0x1p100f);
        r1[l][row] = (float)(v - (double)a);
      }
    });
  if (over) sh.over = 1;
  __syncthreads();
  return sh.over == 0;
}

// ------------------------------------------------------------------ (D)
// r of four tokens (rows: the parts' polynomials, base: kBqSub e0 of the law).  A token's ratio
// has the bits it had in (A), so a positive one finds its row inside the table.
template <int L>
__device__ __forceinline__ void bq_fast_eval(const float (&pv)[4], const float (&qv)[L][4], bool rows,
                                             const float4* const (&r4)[L], const float* const (&r1)[L],
                                             const int (&base)[L], int K, const double (&q0)[L], double zw,
                                             float (&out)[4]) {
  bool closed = false;  // a zero-weight mass in the row: the closed forms are added in fp64
#pragma unroll
  for (int l = 0; l < L; ++l) closed |= q0[l] != 0.0;
  float hi[4], u[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) hi[i] = u[i] = 0.0f;
  if (rows) {
#pragma unroll
    for (int l = 0; l < L; ++l) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const BqTok k = bq_tok(pv[i], qv[l][i]);
        const bool pos = bq_positive(k.w);
        const int at = pos ? (int)k.at - base[l] : 0;
        const float4 a = r4[l][at];
        const float rest = r1[l][at];
        const float t = k.t * (1.0f / kBqTUnit);
        const float f = fmaf(fmaf(fmaf(a.w, t, a.z), t, a.y), t, rest);
        if (L == 1) {
          hi[i] = pos ? a.x : 0.0f;
          u[i] = pos ? f : 0.0f;
        } else if (l == 0) {
          hi[i] = pos ? a.x : 0.0f;
          u[i] = pos ? f : 0.0f;
        } else {  // the sum of the laws' leading values with its rounding error (two-sum) kept in u
          const float h = pos ? a.x : 0.0f;
          const float s = hi[i] + h, bb = s - hi[i];
          u[i] += (pos ? f : 0.0f) + ((hi[i] - (s - bb)) + (h - bb));
          hi[i] = s;
        }
      }
    }
  }
  if (!closed) {
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = fmaf(pv[i], hi[i], pv[i] * u[i]);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float qq[L];
#pragma unroll
      for (int l = 0; l < L; ++l) qq[l] = qv[l][i];
      out[i] = bq_out<L>(pv[i], qq, (double)hi[i] + (double)u[i], K, q0, zw);
    }
  }
}

// the wave's fp64 sum of max(0, p - r) over its 256 tokens (NaN where r is no probability)
__device__ __forceinline__ double bq_residual(const float (&pv)[4], const float (&out)[4]) {
  double local = 0.0;
  uint32_t top = 0u;  // r is not negative unless it is NaN (or -0 next to a -0 probability)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    top = max(top, __float_as_uint(out[i]) & 0x7FFFFFFFu);
    local += residual_of(pv[i], out[i]);
  }
  const double tot = wave_sum_dpp(local);
  return __builtin_amdgcn_ballot_w64(top >= 0x7F800000u) != 0 ? (double)NAN : tot;
}

__device__ __forceinline__ void bq_status(const BqArgs& a, int64_t b, int flags, int tid) {
  if (tid == 0 && a.row_status) {
    if (a.set_status)
      a.row_status[b] = flags;
    else if (flags)
      a.row_status[b] |= flags;
  }
}

// ------------------------------------------------------------------ any row
struct BqGeneralCommon {
  uint32_t qm[kBqWinRows];           // largest q of a bucket (bits), then its shift
  double g[kBqCols * kBqGPad];
  double n[2][kBqWin * 28];
  double b[kBqWin * kBqFar];
  double red[8][128];
  double sd[2][kBqWaves];
  int si[6][kBqWaves];
};
template <int L>
struct BqGeneral {
  union {
    uint64_t acc[kBqWinRows * kBqLen];  // integer sums of a bucket, one word each (any row length)
    double rows[kBqWinRows * kBqLen];   // the parts' polynomials
  };
  double c[L][kBqMaxNodes];
  BqGeneralCommon s;
};

// One row by streaming passes: any fp32 row, any weight range, kBqWin octaves of a law at a time (r of two
// laws: kBqWin / 2 of each).  raw: the workgroup's LDS.
template <int L, bool kRes>
__device__ __attribute__((noinline)) void bq_row_general(const BqArgs& a, int64_t b,
                                                         __attribute__((address_space(3))) char* raw) {
  BqGeneral<L>& sh = *reinterpret_cast<BqGeneral<L>*>((char*)raw);
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t V = a.V;
  const float* pb = a.p + b * V;
  const float* qb[L];
  qb[0] = a.q1 + b * V;
  if (L == 2) qb[L - 1] = a.q2 + b * V;
  float* rb = a.r + b * V;
  const int K = a.K;
  const int64_t nstep = (V + kBqStep - 1) / kBqStep;
  // f(first token of the wave's 256, x0's four, x1's four) over the row, two steps in flight
  auto stream2 = [&](const float* x0, const float* x1, auto&& f) {
    constexpr int kAhead = 2;
    float f0[kAhead][4], f1[kAhead][4];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int64_t at = min((int64_t)j * kBqStep + wid * 256, V);
      row_load4(x0, at, lane, V, f0[j]);
      row_load4(x1, at, lane, V, f1[j]);
    }
    for (int64_t s = 0; s < nstep; s += kAhead) {
#pragma unroll
      for (int j = 0; j < kAhead; ++j) {
        float c0[4], c1[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          c0[i] = f0[j][i];
          c1[i] = f1[j][i];
        }
        const int64_t nx = min((s + j + kAhead) * kBqStep + wid * 256, V);  // past the row: nothing is read
        row_load4(x0, nx, lane, V, f0[j]);
        row_load4(x1, nx, lane, V, f1[j]);
        const int64_t xw = (s + j) * kBqStep + wid * 256;
        if (xw < V) f(xw, c0, c1);
      }
    }
  };
  __syncthreads();  // the caller's LDS is done with
  bq_load_table(sh.s.g, tid);
  for (int x = tid; x < kBqMaxNodes; x += kBqThreads)
#pragma unroll
    for (int l = 0; l < L; ++l) sh.c[l][x] = 0.0;

  // statistics: checks, support, zero-weight masses, the octaves of each law
  int bad = 0, nsup = 0, lo[L], hi[L], e0[L], e1[L];
  double q0[L];
#pragma unroll
  for (int l = 0; l < L; ++l) {
    lo[l] = 0x7FFFFFFF;
    hi[l] = -0x7FFFFFFF;
    q0[l] = 0.0;
    stream2(pb, qb[l], [&](int64_t, const float (&pv)[4], const float (&qv)[4]) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bad |= __builtin_amdgcn_classf(pv[i], 0x21F) | __builtin_amdgcn_classf(qv[i], 0x21F);
        nsup += (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(qv[i] > 0.0f));
        if (qv[i] > 0.0f && pv[i] > 0.0f) {
          const int at = bq_wide_tok(pv[i], qv[i]).at;
          lo[l] = min(lo[l], at);
          hi[l] = max(hi[l], at);
        }
        q0[l] += (qv[i] > 0.0f && pv[i] == 0.0f) ? (double)qv[i] : 0.0;
      }
    });
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      lo[l] = min(lo[l], __shfl_xor(lo[l], off, 64));
      hi[l] = max(hi[l], __shfl_xor(hi[l], off, 64));
    }
    q0[l] = wave_sum_dpp(q0[l]);
  }
  const bool wave_bad = __builtin_amdgcn_ballot_w64(bad != 0) != 0;
  if (lane == 0) {
    sh.s.si[0][wid] = wave_bad ? 1 : 0;
    sh.s.si[1][wid] = nsup;
#pragma unroll
    for (int l = 0; l < L; ++l) {
      sh.s.si[2 + 2 * l][wid] = lo[l];
      sh.s.si[3 + 2 * l][wid] = hi[l];
      sh.s.sd[l][wid] = q0[l];
    }
  }
  __syncthreads();
  bad = nsup = 0;
  bool any = true;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    lo[l] = 0x7FFFFFFF;
    hi[l] = -0x7FFFFFFF;
    q0[l] = 0.0;
#pragma unroll
    for (int w = 0; w < kBqWaves; ++w) {
      lo[l] = min(lo[l], sh.s.si[2 + 2 * l][w]);
      hi[l] = max(hi[l], sh.s.si[3 + 2 * l][w]);
      q0[l] += sh.s.sd[l][w];
    }
    any &= hi[l] >= lo[l];
    e0[l] = __builtin_amdgcn_readfirstlane(lo[l] >> 5);  // kBqSub parts an octave
    e1[l] = __builtin_amdgcn_readfirstlane(hi[l] >> 5);
  }
#pragma unroll
  for (int w = 0; w < kBqWaves; ++w) {
    bad |= sh.s.si[0][w];
    nsup += sh.s.si[1][w];
  }
  int flags = bad ? kRowBadProb : ((a.s_max > 0 && nsup > a.s_max) ? kRowSupport : 0);
  any &= !flags;
  int k_lo = 0, nk = 0;
  if (any) {
    int e_lo = e0[0], e_hi = e1[0];
    if (L == 2) {
      e_lo = min(e_lo, e0[L - 1]);
      e_hi = max(e_hi, e1[L - 1]);
    }
    k_lo = bq_first_node(e_hi, K);
    nk = min(kBqNearHi - 2 * (e_lo - 127) - k_lo + 1, kBqMaxNodes);
    if (a.range_flag && e_hi - e_lo > 290) {
      // the rule's nodes at step 1/2 between the 1e-8 cuts of every denominator, at most kBqRangeNodes
      double dmin = 0.0, dmax = 0.0;
#pragma unroll
      for (int l = 0; l < L; ++l) {
        double wl = INFINITY, wh = 0.0;
        stream2(pb, qb[l], [&](int64_t, const float (&pv)[4], const float (&qv)[4]) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (pv[i] > 0.0f && qv[i] > 0.0f) {
              const double w = (double)pv[i] / (double)qv[i];
              wl = fmin(wl, w);
              wh = fmax(wh, w);
            }
        });
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
          wl = fmin(wl, __shfl_xor(wl, off, 64));
          wh = fmax(wh, __shfl_xor(wh, off, 64));
        }
        __syncthreads();
        if (lane == 0) {
          sh.s.sd[0][wid] = wl;
          sh.s.sd[1][wid] = wh;
        }
        __syncthreads();
        for (int w = 0; w < kBqWaves; ++w) {
          wl = fmin(wl, sh.s.sd[0][w]);
          wh = fmax(wh, sh.s.sd[1][w]);
        }
        dmin += wl;
        dmax += wh;
      }
      if (L == 1) {
        if (K == 2 || q0[0] == 0.0) dmin *= K;
        dmax *= K;
      }
      const int n_lo = (int)floor((kBqLnEps - log(dmax)) * 2.0), n_hi = (int)ceil((kBqLnLnInvEps - log(dmin)) * 2.0);
      if (n_hi - n_lo + 1 > kBqRangeNodes) flags = kRowRange;
    }
  }
  bq_status(a, b, flags, tid);
  const int64_t nparts = a.nsub * kResParts;
  if (flags) {
    for (int64_t x = tid; x < V; x += kBqThreads) rb[x] = NAN;
    if (kRes)
      for (int64_t x = tid; x < nparts; x += kBqThreads) a.rsum[b * nparts + x] = NAN;
    return;
  }

  if (any) {
    // (A), (B) and S, a law and a window at a time
#pragma unroll
    for (int l = 0; l < L; ++l) {
      double below = 0.0, above = INFINITY;  // draft mass of the windows so far, and past them
      // the tokens past a window have larger weights, so their share of S at any node is at most
      // above / below: windows are left out once that is below 2^-40
      for (int w0 = e0[l]; w0 <= e1[l] && above > below * 0x1p-40; w0 += kBqWin) {
        const int w1 = min(w0 + kBqWin - 1, e1[l]);
        double in_q = 0.0, up_q = 0.0;
        __syncthreads();
        for (int x = tid; x < kBqWinRows * kBqLen; x += kBqThreads) sh.acc[x] = 0;
        for (int x = tid; x < kBqWinRows; x += kBqThreads) sh.s.qm[x] = 0;
        __syncthreads();
        stream2(pb, qb[l], [&](int64_t, const float (&pv)[4], const float (&qv)[4]) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int at = bq_wide_tok(pv[i], qv[i]).at - w0 * kBqSub;
            if (pv[i] > 0.0f && qv[i] > 0.0f && at >= 0) {
              if (at < kBqWinRows) {
                atomicMax(&sh.s.qm[at], __float_as_uint(qv[i]));
                in_q += (double)qv[i];
              } else {
                up_q += (double)qv[i];
              }
            }
          }
        });
        in_q = wave_sum_dpp(in_q);
        up_q = wave_sum_dpp(up_q);
        if (lane == 0) {
          sh.s.sd[0][wid] = in_q;
          sh.s.sd[1][wid] = up_q;
        }
        __syncthreads();
        above = 0.0;
        for (int w = 0; w < kBqWaves; ++w) {
          below += sh.s.sd[0][w];
          above += sh.s.sd[1][w];
        }
        for (int x = tid; x < kBqWinRows; x += kBqThreads)
          sh.s.qm[x] = (uint32_t)(kBqF + 1 - __builtin_amdgcn_frexp_expf(__uint_as_float(sh.s.qm[x])));
        __syncthreads();
        stream2(pb, qb[l], [&](int64_t, const float (&pv)[4], const float (&qv)[4]) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const BqWideTok k = bq_wide_tok(pv[i], qv[i]);
            const uint32_t at = (uint32_t)(k.at - w0 * kBqSub);
            if (!(pv[i] > 0.0f && qv[i] > 0.0f && at < (uint32_t)kBqWinRows)) continue;
            float v = ldexpf(qv[i], (int)sh.s.qm[at]);
            unsigned long long* acc = reinterpret_cast<unsigned long long*>(&sh.acc[at * kBqLen]);
#pragma unroll
            for (int n = 0; n < kBqLen; ++n) {
              atomicAdd(acc + n, (unsigned long long)(long long)bq_round(v));
              v *= k.t;
            }
          }
        });
        __syncthreads();
        bq_contract(sh.s.n, sh.s.g, w0, w1 - w0 + 1, lane, wid, [&](int e, int x) {
          const int at = (e - w0) * kBqSub + x / kBqLen, n = x % kBqLen;
          return ldexp((double)(int64_t)sh.acc[at * kBqLen + n], 6 * n - (int)sh.s.qm[at]);
        });
        __syncthreads();
        bq_nodes(sh.s.n, sh.s.red, w0, w1, k_lo, nk, tid, [&](int i, double S) { sh.c[L - 1 - l][i] += S; });
      }
    }
#pragma unroll
    for (int l = 0; l < L; ++l)
      for (int i = tid; i < nk; i += kBqThreads) sh.c[l][i] = bq_coef<L>(sh.c[l][i], k_lo + i, K, q0[0]);
    __syncthreads();
  }

  // (D), a pair of windows (one of each law) at a time: a token's laws are summed in fp64 and rounded
  // once, in the pass of its own pair (window 0 of a law it has no positive ratio in)
  constexpr int kOct = kBqWin / L;  // octaves of a window: every law's polynomials lie in `rows`
  double zw = q0[0];  // K i.i.d. drafts: Q0^(K-1)
  for (int j = 2; j < K; ++j) zw *= q0[0];
  const auto windows = [&](int l) { return any ? (e1[l] - e0[l]) / kOct + 1 : 1; };
  const auto build = [&](int l, int win) {  // (the last pass over the rows ended with a barrier)
    if (!any) return;
    const int first = e0[l] + win * kOct, noct = min(kOct, e1[l] - first + 1);
    double* rows = sh.rows + l * kOct * kBqOct;
    bq_far(sh.c[l], sh.s.b, first, noct, k_lo, tid);
    __syncthreads();
    bq_polynomials(sh.c[l], sh.s.b, sh.s.g, first, noct, k_lo, lane, wid,
                   [&](int o, int y, double v) { rows[o * kBqOct + y] = v; });
    __syncthreads();
  };
  const bool one = windows(0) * windows(L - 1) == 1;
  for (int i = 0; i < windows(0); ++i) {
    build(0, i);
    for (int j = 0; j < (L == 2 ? windows(L - 1) : 1); ++j) {
      if (L == 2) build(L - 1, j);
      stream2(pb, qb[0], [&](int64_t xw, const float (&pv)[4], const float (&qv)[4]) {
        float oq[4], out[4];
        if (L == 2) row_load4(qb[L - 1], xw, lane, V, oq);
        bool mine[4];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          float qq[L];
          qq[0] = qv[n];
          if (L == 2) qq[L - 1] = oq[n];
          double f = 0.0;
          mine[n] = true;
#pragma unroll
          for (int l = 0; l < L; ++l) {
            const BqWideTok k = bq_wide_tok(pv[n], qq[l]);
            const bool pos = any && pv[n] > 0.0f && qq[l] > 0.0f;
            const int at = pos ? k.at - (e0[l] + (l == 0 ? i : j) * kOct) * kBqSub : 0;
            const bool in = (uint32_t)at < (uint32_t)(kOct * kBqSub);
            mine[n] &= pos ? in : (l == 0 ? i : j) == 0;
            if (pos && in) {
              const double* r = &sh.rows[l * kOct * kBqOct + at * kBqLen];
              const double t = (double)k.t * (1.0 / (double)kBqTUnit);
              f += ::fma(::fma(::fma(r[3], t, r[2]), t, r[1]), t, r[0]);
            }
          }
          out[n] = bq_out<L>(pv[n], qq, f, K, q0, zw);
        }
        if (one) {
          row_store4(rb, xw, lane, V, out);
        } else {
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const int64_t x = xw + 4 * lane + n;
            if (mine[n] && x < V) rb[x] = out[n];
          }
        }
      });
      __syncthreads();
    }
  }
  if (kRes)  // from the r each thread wrote itself
    stream2(pb, rb, [&](int64_t xw, const float (&pv)[4], const float (&rv)[4]) {
      const double tot = bq_residual(pv, rv);
      if (lane == 0) a.rsum[b * nparts + (xw >> 8)] = tot;
    });
  if (kRes)  // parts past the row
    for (int64_t x = (V + 255) / 256 + tid; x < nparts; x += kBqThreads) a.rsum[b * nparts + x] = 0.0;
}

// The tokens of one step as new values: the compiler then takes a token's ratio again in every
// pass instead of keeping 32 tokens' worth of it (which spills), and keeps the steps apart.
template <int L>
__device__ __forceinline__ void bq_step_tokens(const float (&pr)[4], const float (&qr)[L][4], float (&pc)[4],
                                               float (&qc)[L][4]) {
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    pc[i] = pr[i];
    __asm__ volatile("" : "+v"(pc[i]));
#pragma unroll
    for (int l = 0; l < L; ++l) {
      qc[l][i] = qr[l][i];
      __asm__ volatile("" : "+v"(qc[l][i]));
    }
  }
}

// ------------------------------------------------------------------ one workgroup a row
template <int L>
struct BqRowShared {
  union {
    BqSumsShared<L> sums;
    struct {
      float4 r4[L][kBqWinRows];
      float r1[L][kBqWinRows];
    } rows;
  };
  BqSolve<L> solve;
  BqStatShared<L, kBqWaves> stat;
};

// Rows of up to 1024 PER tokens: thread t holds PER tokens in registers.
template <int L, int PER, bool kRes>
__global__ __launch_bounds__(kBqThreads) void bq_row_kernel(BqArgs a) {
  constexpr int kRaw = sizeof(BqRowShared<L>) > sizeof(BqGeneral<L>) ? sizeof(BqRowShared<L>) : sizeof(BqGeneral<L>);
  __shared__ __align__(16) char raw[kRaw];
  BqRowShared<L>& sh = *reinterpret_cast<BqRowShared<L>*>(raw);
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t b = blockIdx.x, V = a.V;
  float* rb = a.r + b * V;
  constexpr int kSteps = PER / 4;
  float pr[kSteps][4], qr[kSteps][L][4];
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    const int64_t xw = min((int64_t)s * kBqStep + wid * 256, V);
    row_load4(a.p + b * V, xw, lane, V, pr[s]);
    row_load4(a.q1 + b * V, xw, lane, V, qr[s][0]);
    if (L == 2) row_load4(a.q2 + b * V, xw, lane, V, qr[s][L - 1]);
  }
  for (int x = tid; x < kBqWinRows * kBqAcc; x += kBqThreads) sh.sums.acc[x] = 0;
#pragma unroll
  for (int l = 0; l < L; ++l)
    for (int x = tid; x < kBqWinRows; x += kBqThreads) sh.sums.qm[l][x] = 0;
  bq_load_table(sh.solve.g, tid);
  __syncthreads();
  // (A)
  BqFastStats<L> st;
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    float pc[4], qc[L][4];
    bq_step_tokens<L>(pr[s], qr[s], pc, qc);
    bq_fast_count<L>(pc, qc, sh.sums, st, a.s_max > 0);
  }
  const BqRange<L> rg = bq_combine(st, sh.stat, lane, wid);
  if (!rg.bad && rg.special) {
    bq_row_general<L, kRes>(a, b, (__attribute__((address_space(3))) char*)raw);
    return;
  }
  const int flags = rg.bad ? kRowBadProb : ((a.s_max > 0 && rg.nsup > a.s_max) ? kRowSupport : 0);
  bool any = !flags;
#pragma unroll
  for (int l = 0; l < L; ++l) any &= rg.e1[l] > 0;
  if (any) {
    bq_fast_scales<L>(sh.sums, tid, kBqThreads);
    float4* r4[L];
    float* r1[L];
#pragma unroll
    for (int l = 0; l < L; ++l) {
      r4[l] = sh.rows.r4[l];
      r1[l] = sh.rows.r1[l];
    }
    const auto begin = [&](int l) {  // (B)
      if (l > 0)
        for (int x = tid; x < kBqWinRows * kBqAcc; x += kBqThreads) sh.sums.acc[x] = 0;
      __syncthreads();
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        float pc[4], qc[L][4];
        bq_step_tokens<L>(pr[s], qr[s], pc, qc);
        bq_fast_add<L>(pc, qc[l], sh.sums, l);
      }
      __syncthreads();
    };
    const auto moment = [&](int l, int e, int x) {
      return bq_decode<L>(sh.sums, l, (e & (kBqWin - 1)) * kBqSub + x / kBqLen, x % kBqLen);
    };
    if (!bq_solve<L>(sh.solve, rg, a.K, r4, r1, tid, lane, wid, begin, moment)) {  // (C)
      bq_row_general<L, kRes>(a, b, (__attribute__((address_space(3))) char*)raw);
      return;
    }
  }
  bq_status(a, b, flags, tid);
  // (D)
  double zw = rg.q0[0];  // K i.i.d. drafts: Q0^(K-1)
  for (int j = 2; j < a.K; ++j) zw *= rg.q0[0];
  const int64_t nparts = a.nsub * kResParts;
  const float4* r4[L];
  const float* r1[L];
  int base[L];
#pragma unroll
  for (int l = 0; l < L; ++l) {
    r4[l] = sh.rows.r4[l];
    r1[l] = sh.rows.r1[l];
    base[l] = rg.e0[l] * kBqSub;
  }
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    const int64_t xw = (int64_t)s * kBqStep + wid * 256;
    float out[4], pc[4], qc[L][4];
    bq_step_tokens<L>(pr[s], qr[s], pc, qc);
    bq_fast_eval<L>(pc, qc, any, r4, r1, base, a.K, rg.q0, zw, out);
    if (flags) {
#pragma unroll
      for (int i = 0; i < 4; ++i) out[i] = NAN;
    }
    if (xw < V) row_store4(rb, xw, lane, V, out);
    if (kRes) {
      const double tot = bq_residual(pc, out);
      if (lane == 0 && (xw >> 8) < nparts) a.rsum[b * nparts + (xw >> 8)] = tot;
    }
  }
}

// ------------------------------------------------------------------ chunks of rows
// Record of a chunk: header, then per law `win` octaves of M, octave e at e modulo win: value 0 of
// its parts in fp64, then values 1 .. 3 in fp32 (their share of a sum is below 0.1).
constexpr int kBqRecOct = kBqSub * (8 + 4 * kBqDeg);  // bytes of an octave
__device__ __forceinline__ double bq_rec_get(const char* oct, int y) {
  const int j = y / kBqLen, n = y % kBqLen;
  return n == 0 ? reinterpret_cast<const double*>(oct)[j]
                : (double)reinterpret_cast<const float*>(oct + 8 * kBqSub)[j * kBqDeg + n - 1];
}
__device__ __forceinline__ void bq_rec_put(char* oct, int y, double v) {
  const int j = y / kBqLen, n = y % kBqLen;
  if (n == 0)
    reinterpret_cast<double*>(oct)[j] = v;
  else
    reinterpret_cast<float*>(oct + 8 * kBqSub)[j * kBqDeg + n - 1] = (float)v;
}
struct alignas(64) BqRecHdr {
  int32_t bad, special, nsup, pad;
  int32_t e0[2], e1[2];
  double q0[2];
};
struct alignas(64) BqPlan {
  int32_t flags, done, any, pad;     // done: r (and the residual sums) are written already
  int32_t e0[2], e1[2];
  double q0[2];
};
constexpr int kBqRowBytes = kBqWinRows * (int)(sizeof(float4) + sizeof(float));  // a law's polynomials
struct BqWork {
  BqPlan* plan;   // [B]
  char* area;     // [B] areas of `room` bytes: the records, then (the merge is done with them) the polynomials
  int64_t room, slot;
  int C, win;
  int64_t chunk;  // tokens of a chunk (a multiple of 2048)
  __device__ __forceinline__ char* rec(int64_t b, int c) const { return area + b * room + c * slot; }
  __device__ __forceinline__ float4* r4(int64_t b, int l) const {
    return reinterpret_cast<float4*>(area + b * room + l * kBqRowBytes);
  }
  __device__ __forceinline__ float* r1(int64_t b, int l) const {
    return reinterpret_cast<float*>(r4(b, l) + kBqWinRows);
  }
};
constexpr int kBqMPad = kBqOct + 2;  // LDS stride of an octave of M
constexpr int kBqMergeHdr = 512;   // chunks of a row, at most
constexpr int kBqPartThreads = 512;  // two workgroups a CU: one loads while the other sums
constexpr int kBqPartStep = 4 * kBqPartThreads;

// A chunk tile by tile (512 PER tokens), law after law.
template <int L, int PER>
__global__ __launch_bounds__(kBqPartThreads, 4) void bq_part_kernel(BqArgs a, BqWork wk) {
  constexpr int kWaves = kBqPartThreads / 64, kSteps = PER / 4;
  __shared__ __align__(16) BqSumsShared<1> sums;
  __shared__ BqStatShared<1, kWaves> stat[2];
  const int64_t b = blockIdx.x / (unsigned)wk.C, V = a.V;
  const int ch = (int)(blockIdx.x % (unsigned)wk.C);
  const float* pb = a.p + b * V;
  const int64_t x0 = (int64_t)ch * wk.chunk, end = min(V, x0 + wk.chunk);  // a multiple of four if V is
  char* rec = wk.rec(b, ch);
  BqRecHdr h;
  h.bad = h.special = h.nsup = h.pad = 0;
  int par = 0;
#pragma unroll
  for (int l = 0; l < 2; ++l) {
    h.e0[l] = 0x7FFFFFF;
    h.e1[l] = 0;
    h.q0[l] = 0.0;
  }
  for (int64_t xt = x0; xt < end; xt += PER * kBqPartThreads) {
    int tid = threadIdx.x;
    __asm__ volatile("" : "+v"(tid));  // nothing derived from it is kept across tiles
    const int lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    float pr[kSteps][4], qr[kSteps][L][4];
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      const int64_t xw = min(xt + (int64_t)s * kBqPartStep + wid * 256, end);
      row_load4(pb, xw, lane, end, pr[s]);
      row_load4(a.q1 + b * V, xw, lane, end, qr[s][0]);
      if (L == 2) row_load4(a.q2 + b * V, xw, lane, end, qr[s][L - 1]);
    }
#pragma unroll
    for (int l = 0; l < L; ++l) {
      for (int x = tid; x < kBqWinRows * kBqAcc; x += kBqPartThreads) sums.acc[x] = 0;
      for (int x = tid; x < kBqWinRows; x += kBqPartThreads) sums.qm[0][x] = 0;
      __syncthreads();
      BqFastStats<1> st;
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        if (xt + (int64_t)s * kBqPartStep >= end) break;  // uniform
        float pc[4], qc[1][4], qs[1][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) qs[0][i] = qr[s][l][i];
        bq_step_tokens<1>(pr[s], qs, pc, qc);
        bq_fast_count<1>(pc, qc, sums, st, a.s_max > 0);
      }
      const BqRange<1> rg = bq_combine(st, stat[par], lane, wid);
      par ^= 1;
      h.bad |= rg.bad;
      h.special |= rg.special;
      h.nsup += rg.nsup;
      h.q0[l] += rg.q0[0];
      if (rg.e1[0] > 0 && !rg.bad && !rg.special) {  // uniform
        const int e0 = min(h.e0[l], rg.e0[0]), e1 = max(h.e1[l], rg.e1[0]);
        if (e1 - e0 >= wk.win) {
          h.special = 1;
        } else {
          bq_fast_scales<1>(sums, tid, kBqPartThreads);
          __syncthreads();
#pragma unroll
          for (int s = 0; s < kSteps; ++s) {
            if (xt + (int64_t)s * kBqPartStep >= end) break;  // uniform
            float pc[4], qc[1][4], qs[1][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) qs[0][i] = qr[s][l][i];
            bq_step_tokens<1>(pr[s], qs, pc, qc);
            bq_fast_add<1>(pc, qc[0], sums, 0);
          }
          __syncthreads();
          // octaves new to the chunk are stored, the others added to
          char* out = rec + sizeof(BqRecHdr) + (int64_t)l * wk.win * kBqRecOct;
          for (int x = tid; x < (e1 - e0 + 1) * kBqOct; x += kBqPartThreads) {
            const int e = e0 + x / kBqOct, y = x % kBqOct;
            char* m = out + (e % wk.win) * kBqRecOct;
            const bool in = e >= rg.e0[0] && e <= rg.e1[0], old = e >= h.e0[l] && e <= h.e1[l];
            const double v = in ? bq_decode<1>(sums, 0, (e & (kBqWin - 1)) * kBqSub + y / kBqLen, y % kBqLen) : 0.0;
            if (!old)
              bq_rec_put(m, y, v);
            else if (in)
              bq_rec_put(m, y, bq_rec_get(m, y) + v);
          }
          h.e0[l] = e0;
          h.e1[l] = e1;
        }
      }
      __syncthreads();  // the sums are cleared next
    }
  }
  if (threadIdx.x == 0) *reinterpret_cast<BqRecHdr*>(rec) = h;
}

template <int L>
struct BqMergeShared {
  BqSolve<L> solve;
  double m[kBqWin * kBqMPad];  // one law's M
  int win[L][2][kBqMergeHdr];  // chunks' first and last octaves
};

// (C) of a row from its chunks' records, in chunk order; rows the records do not cover are taken
// whole by bq_row_general.
template <int L, bool kRes>
__global__ __launch_bounds__(kBqThreads) void bq_merge_kernel(BqArgs a, BqWork wk) {
  constexpr int kRaw = sizeof(BqMergeShared<L>) > sizeof(BqGeneral<L>) ? sizeof(BqMergeShared<L>) : sizeof(BqGeneral<L>);
  __shared__ __align__(16) char raw[kRaw];
  BqMergeShared<L>& ms = *reinterpret_cast<BqMergeShared<L>*>(raw);
  BqSolve<L>& sh = ms.solve;
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t b = blockIdx.x;
  bq_load_table(sh.g, tid);
  BqRange<L> rg;
  rg.bad = rg.special = false;
  rg.nsup = 0;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    rg.e0[l] = 0x7FFFFFF;
    rg.e1[l] = 0;
    rg.q0[l] = 0.0;
  }
  // every wave reads the headers, a lane a chunk (their octaves are kept in LDS by the first)
  for (int c0 = 0; c0 < wk.C; c0 += 64) {
    const int c = min(c0 + lane, wk.C - 1);
    const BqRecHdr h = *reinterpret_cast<const BqRecHdr*>(wk.rec(b, c));
    rg.bad |= __builtin_amdgcn_ballot_w64(h.bad != 0) != 0;
    rg.special |= __builtin_amdgcn_ballot_w64(h.special != 0) != 0;
    const bool mine = c0 + lane < wk.C;
    rg.nsup += __builtin_amdgcn_readfirstlane(wave_sum_int(mine ? h.nsup : 0));
#pragma unroll
    for (int l = 0; l < L; ++l) {
      rg.e0[l] = min(rg.e0[l], (int)bq_wave<false>((uint32_t)h.e0[l]));
      rg.e1[l] = max(rg.e1[l], (int)bq_wave<true>((uint32_t)h.e1[l]));
      if (__builtin_amdgcn_ballot_w64(h.q0[l] != 0.0) != 0) rg.q0[l] += wave_sum_dpp(mine ? h.q0[l] : 0.0);
      if (wid == 0 && mine) {
        ms.win[l][0][c] = h.e0[l];
        ms.win[l][1][c] = h.e1[l];
      }
    }
  }
  bool any = !rg.bad;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    rg.e0[l] = __builtin_amdgcn_readfirstlane(rg.e0[l]);
    rg.e1[l] = __builtin_amdgcn_readfirstlane(rg.e1[l]);
    any &= rg.e1[l] > 0;
    if (rg.e1[l] > 0) rg.special |= rg.e1[l] - rg.e0[l] >= kBqWin;
  }
  const int flags = rg.bad ? kRowBadProb : ((a.s_max > 0 && rg.nsup > a.s_max) ? kRowSupport : 0);
  any &= !flags;
  bool general = !rg.bad && rg.special;
  __syncthreads();
  if (any && !general) {
    float4* r4[L];
    float* r1[L];
#pragma unroll
    for (int l = 0; l < L; ++l) {
      r4[l] = wk.r4(b, l);
      r1[l] = wk.r1(b, l);
    }
    // a law's M: the chunks' records added in chunk order, eight loads in flight
    const auto begin = [&](int l) {
      const int noct = rg.e1[l] - rg.e0[l] + 1;
      // value 0 of every part, then the others, each element from eight records at a time
      const auto gather = [&](int per, auto&& at, auto&& put) {
        for (int x = tid; x < noct * per; x += kBqThreads) {
          const int o = x / per, e = rg.e0[l] + o;
          const char* from = wk.rec(b, 0) + sizeof(BqRecHdr) + ((int64_t)l * wk.win + e % wk.win) * kBqRecOct;
          double v = 0.0;
          for (int c0 = 0; c0 < wk.C; c0 += 8) {
            double t[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) t[i] = at(from + min(c0 + i, wk.C - 1) * wk.slot, x - o * per);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const int c = min(c0 + i, wk.C - 1);
              v += (c0 + i < wk.C && e >= ms.win[l][0][c] && e <= ms.win[l][1][c]) ? t[i] : 0.0;
            }
          }
          put(&ms.m[(e & (kBqWin - 1)) * kBqMPad], x - o * per, v);
        }
      };
      gather(
          kBqSub, [](const char* r, int j) { return reinterpret_cast<const double*>(r)[j]; },
          [](double* m, int j, double v) { m[j * kBqLen] = v; });
      gather(
          kBqSub * kBqDeg, [](const char* r, int j) { return (double)reinterpret_cast<const float*>(r + 8 * kBqSub)[j]; },
          [](double* m, int j, double v) { m[j / kBqDeg * kBqLen + j % kBqDeg + 1] = v; });
      __syncthreads();
    };
    general = !bq_solve<L>(sh, rg, a.K, r4, r1, tid, lane, wid, begin,
                           [&](int, int e, int x) { return ms.m[(e & (kBqWin - 1)) * kBqMPad + x]; });
  }
  if (general) {
    bq_row_general<L, kRes>(a, b, (__attribute__((address_space(3))) char*)raw);
  } else {
    bq_status(a, b, flags, tid);
  }
  if (tid == 0) {
    BqPlan pl;
    pl.flags = general ? 0 : flags;
    pl.done = general;
    pl.any = any;
    pl.pad = 0;
#pragma unroll
    for (int l = 0; l < 2; ++l) {
      pl.e0[l] = rg.e0[l < L ? l : 0];
      pl.e1[l] = rg.e1[l < L ? l : 0];
      pl.q0[l] = rg.q0[l < L ? l : 0];
    }
    wk.plan[b] = pl;
  }
}

constexpr int kBqEvalThreads = 256;
constexpr int kBqEvalTile = 4 * kBqEvalThreads;  // 1024 tokens, four a thread
constexpr int kBqEvalRows = 32 * kBqSub;         // a row's polynomials kept in LDS up to 32 octaves

// (D) on tiles of 1024 tokens: workgroup w takes the tiles [w per, (w + 1) per) of the B T
// (row, tile) pairs, row-major, the next tile's p and q in flight; a row's polynomials go to LDS
// (read from the workspace for wider rows).
template <int L, bool kRes>
__global__ __launch_bounds__(kBqEvalThreads) void bq_eval_kernel(BqArgs a, BqWork wk, int64_t T, int64_t G, int per) {
  __shared__ float4 s_r4[L][kBqEvalRows];
  __shared__ float s_r1[L][kBqEvalRows];
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t V = a.V, nparts = a.nsub * kResParts;
  const int64_t g0 = (int64_t)blockIdx.x * per, g1 = min(g0 + per, G);
  if (g0 >= g1) return;
  int64_t b = __builtin_amdgcn_readfirstlane((int)(g0 / T));
  int64_t t = g0 - b * T;
  float pv[4], qv[L][4];
  const auto load = [&]() {
    const int64_t xw = min(t * kBqEvalTile + wid * 256, V);
    row_load4(a.p + b * V, xw, lane, V, pv);
    row_load4(a.q1 + b * V, xw, lane, V, qv[0]);
    if (L == 2) row_load4(a.q2 + b * V, xw, lane, V, qv[L - 1]);
  };
  load();
  int64_t have = -1;
  BqPlan pl;
  double zw = 0.0, q0[L];
  int base[L];
  bool rows = false, lds = false;
  for (int64_t g = g0; g < g1; ++g) {
    float pc[4], qc[L][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      pc[i] = pv[i];
#pragma unroll
      for (int l = 0; l < L; ++l) qc[l][i] = qv[l][i];
    }
    const int64_t cb = b, xw = t * kBqEvalTile + wid * 256;
    if (cb != have) {  // uniform
      if (have >= 0) __syncthreads();  // every wave is done with the previous row's polynomials
      have = cb;
      pl = wk.plan[cb];
      zw = pl.q0[0];
      for (int j = 2; j < a.K; ++j) zw *= pl.q0[0];
      rows = pl.any && !pl.done && !pl.flags;
      lds = rows;
#pragma unroll
      for (int l = 0; l < L; ++l) {
        base[l] = pl.e0[l] * kBqSub;
        q0[l] = pl.q0[l];
        lds &= (pl.e1[l] - pl.e0[l] + 1) * kBqSub <= kBqEvalRows;
      }
      if (lds) {
#pragma unroll
        for (int l = 0; l < L; ++l)
          for (int x = tid; x < (pl.e1[l] - pl.e0[l] + 1) * kBqSub; x += kBqEvalThreads) {
            s_r4[l][x] = wk.r4(cb, l)[x];
            s_r1[l][x] = wk.r1(cb, l)[x];
          }
      }
      __syncthreads();
    }
    if (++t == T) {
      t = 0;
      ++b;
    }
    if (g + 1 < g1) load();
    if (pl.done) continue;  // uniform
    float out[4];
    const float4* r4[L];
    const float* r1[L];
    if (lds || !rows) {
#pragma unroll
      for (int l = 0; l < L; ++l) {
        r4[l] = s_r4[l];
        r1[l] = s_r1[l];
      }
      bq_fast_eval<L>(pc, qc, rows, r4, r1, base, a.K, q0, zw, out);
    } else {
#pragma unroll
      for (int l = 0; l < L; ++l) {
        r4[l] = wk.r4(cb, l);
        r1[l] = wk.r1(cb, l);
      }
      bq_fast_eval<L>(pc, qc, rows, r4, r1, base, a.K, q0, zw, out);
    }
    if (pl.flags) {
#pragma unroll
      for (int i = 0; i < 4; ++i) out[i] = NAN;
    }
    if (xw < V) row_store4(a.r + cb * V, xw, lane, V, out);
    if (kRes) {
      const double tot = bq_residual(pc, out);
      if (lane == 0 && (xw >> 8) < nparts) a.rsum[cb * nparts + (xw >> 8)] = tot;
    }
  }
}

// One workgroup a row, streaming: calls without room for the chunks' sums.
template <int L>
__global__ __launch_bounds__(kBqThreads) void bq_general_kernel(BqArgs a) {
  __shared__ __align__(16) char raw[sizeof(BqGeneral<L>)];
  bq_row_general<L, false>(a, blockIdx.x, (__attribute__((address_space(3))) char*)raw);
}

size_t bq_align(size_t x) { return (x + 255) & ~(size_t)255; }

// Workgroups of the evaluation: every resident slot of the device once (measured once per device).
unsigned bq_eval_grid(const void* kernel, int64_t tiles, int slot) {
  static int s_slots[64][2];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  int slots = s_slots[dev][slot];
  if (slots <= 0) {
    int cus = 0, occ = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, kBqEvalThreads, 0) != hipSuccess) occ = 0;
    slots = std::max(cus, 1) * std::max(occ, 1);
    s_slots[dev][slot] = slots;
  }
  const int64_t per = (tiles + slots - 1) / slots;
  return (unsigned)std::max<int64_t>(1, (tiles + per - 1) / per);
}

// The chunks of a call and its workspace; false if the workspace has no room for them.
bool bq_carve(void* base, size_t bytes, int64_t B, int64_t V, int L, BqWork* wk) {
  const size_t fixed = bq_align(sizeof(BqPlan) * B);
  if (base == nullptr || bytes <= fixed) return false;
  const int64_t room = (int64_t)((bytes - fixed) / (size_t)B) / 64 * 64;
  const int64_t hdr = (int64_t)sizeof(BqRecHdr), octave = (int64_t)L * kBqRecOct;
  // as many chunks as there are tiles (512 threads of 32 tokens, 16 with two laws; of 4096 tokens
  // when the rows do not fill the chip) but no more than leave each room for 32 octaves (18 rows of 118432,
  // four successive drafts: 39 octaves left room for seven chunks of three tiles, 229 us; now 207)
  const int64_t full = (L == 1 ? 32 : 16) * kBqPartThreads;
  const int64_t tile = B * ((V + full - 1) / full) >= 512 ? full : 8 * kBqPartThreads;
  int64_t C = std::min<int64_t>({(V + tile - 1) / tile, (1024 + B - 1) / B + (V + full - 1) / full,
                                 room / (hdr + 32 * octave), kBqMergeHdr});
  C = std::max<int64_t>(1, C);
  // chunks of several tiles hold whole ones: no more chunks than that takes (12 rows of 129864, three successive laws:
  // ten chunks of 7 / 4 tiles 175 us, eight of two tiles 172)
  const int64_t per = ((V + C - 1) / C + full - 1) / full;
  if (per > 1) C = (V + per * full - 1) / (per * full);
  wk->chunk = ((V + C - 1) / C + kBqPartStep - 1) / kBqPartStep * kBqPartStep;
  wk->C = (int)((V + wk->chunk - 1) / wk->chunk);
  wk->room = room;
  wk->slot = room / wk->C / 64 * 64;
  wk->win = (int)std::min<int64_t>(kBqWin, (wk->slot - hdr) / octave);
  wk->plan = static_cast<BqPlan*>(base);
  wk->area = static_cast<char*>(base) + fixed;
  return wk->win >= 8 && room >= (int64_t)L * kBqRowBytes;
}

template <int L, bool kRes>
void bq_launch_chunks(const BqArgs& a, const BqWork& wk, int64_t B, hipStream_t st) {
  const dim3 parts((unsigned)(B * wk.C));
  const int64_t per = wk.chunk / kBqPartThreads;
  if (per <= 8)
    hipLaunchKernelGGL((bq_part_kernel<L, 8>), parts, dim3(kBqPartThreads), 0, st, a, wk);
  else if (per <= 16 || L == 2)
    hipLaunchKernelGGL((bq_part_kernel<L, 16>), parts, dim3(kBqPartThreads), 0, st, a, wk);
  else
    hipLaunchKernelGGL((bq_part_kernel<1, 32>), parts, dim3(kBqPartThreads), 0, st, a, wk);
  hipLaunchKernelGGL((bq_merge_kernel<L, kRes>), dim3((unsigned)B), dim3(kBqThreads), 0, st, a, wk);
  const int64_t T = (a.V + kBqEvalTile - 1) / kBqEvalTile, G = B * T;
  const unsigned n = bq_eval_grid(reinterpret_cast<const void*>(&bq_eval_kernel<L, false>), G, L - 1);
  hipLaunchKernelGGL((bq_eval_kernel<L, kRes>), dim3(n), dim3(kBqEvalThreads), 0, st, a, wk, T, G,
                     (int)((G + n - 1) / n));
}

template <int L, bool kRes>
void bq_launch_rows(const BqArgs& a, int64_t B, hipStream_t st) {
  if (a.V <= 4 * kBqThreads)
    hipLaunchKernelGGL((bq_row_kernel<L, 4, kRes>), dim3((unsigned)B), dim3(kBqThreads), 0, st, a);
  else if (a.V <= 16 * kBqThreads || L == 2)
    hipLaunchKernelGGL((bq_row_kernel<L, 16, kRes>), dim3((unsigned)B), dim3(kBqThreads), 0, st, a);
  else
    hipLaunchKernelGGL((bq_row_kernel<1, 32, kRes>), dim3((unsigned)B), dim3(kBqThreads), 0, st, a);
}

}  // namespace

hipError_t launch_bucket(const float* p, const float* q1, const float* q2, int64_t B, int64_t V, int K, int s_max,
                         bool range_flag, float* r, int32_t* row_status, bool set_status, double* rsum,
                         void* workspace, size_t workspace_bytes, hipStream_t st) {
  const BqArgs a = {p, q1, q2, V, K, s_max, range_flag ? 1 : 0, set_status ? 1 : 0, r, row_status, rsum,
                    (V + kResSub - 1) / kResSub};
  const bool fits = V <= (q2 ? kBqPer / 2 : kBqPer) * kBqThreads;  // a workgroup's registers
  BqWork wk;
  if (!(fits && (B >= 128 || V <= kBqStep)) && bq_carve(workspace, workspace_bytes, B, V, q2 ? 2 : 1, &wk)) {
    if (q2 != nullptr)
      bq_launch_chunks<2, false>(a, wk, B, st);
    else if (rsum)
      bq_launch_chunks<1, true>(a, wk, B, st);
    else
      bq_launch_chunks<1, false>(a, wk, B, st);
  } else if (fits) {
    if (q2 != nullptr)
      bq_launch_rows<2, false>(a, B, st);
    else if (rsum)
      bq_launch_rows<1, true>(a, B, st);
    else
      bq_launch_rows<1, false>(a, B, st);
  } else if (q2 == nullptr) {
    hipLaunchKernelGGL((bq_general_kernel<1>), dim3((unsigned)B), dim3(kBqThreads), 0, st, a);
  } else {
    hipLaunchKernelGGL((bq_general_kernel<2>), dim3((unsigned)B), dim3(kBqThreads), 0, st, a);
  }
  return hipGetLastError();
}

}  // namespace mdss
