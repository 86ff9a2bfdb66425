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
// largest error: at most 7.1e-9 of an entry (a token at the edge of its octave's first part, paired with much smaller
// weights; 9e-10 with equal ones), so r is within its fp32 rounding.
//
// Order and precision.  M is summed by integer LDS atomics: v = q scaled by a power of two, the
// bucket's largest q into [2^29, 2^30), and v, v u, v u^2 and v u^3 with u = t / 64 rounded to integers.
// The four have the same unit, so each is off by at most 2^-31 of the bucket's largest q in units of its
// place in the polynomial: v u^2 and v u^3 are small numbers (18 and 12 bits) because they are small, not
// because they are rounded more coarsely; a token's fp32 values carried 2^-25 of themselves.  Integer sums do not
// depend on the order, so r is the same bit for bit on every run.  Everything after is fp64; a part's polynomial is
// kept as a_0 in two fp32 numbers and a_1 .. a_3 in one each (below 0.02 of the value: 1.2e-9 of it).
//
// Measured (256 x 32000, K = 2, bq_row_kernel): 43 us, with the residual sums 51, against 75 us for three kernels
// that took nine exponentials a token on the way in (their fp32 sums left r 7.5e-8 off in the 2-norm; 2.4e-8 here, all
// of it r's own rounding).  By the counters, of a CU's busy cycles: VALU issue 57 %, LDS active 38 %, six tenths of that
// bank conflicts of the tokens' atomics; 102 MB of the 98 MB that p, q and r take.
//
// Forms.  Rows whose probabilities and ratios stay inside [2^-96, 2^20] and [2^-96, 2^96] and
// whose ratios span at most 64 octaves take the fp32 per-token arithmetic of bucket.h:
//   bq_row_kernel   one workgroup of 1024 threads a row, the row in registers from its first
//                   load to r: (A) the largest q of every bucket, (B) the integer sums, (C) S,
//                   c and the parts' polynomials, (D) r and Algorithm 1's residual sums;
//   bq_part_kernel, bq_merge_kernel, bq_eval_kernel   the same with (A) and (B) on chunks of a
//                   row, (C) per row from the chunks' sums, (D) on tiles: long rows, few rows,
//                   two laws.
// Other rows (wide tokens: mantissas and exponents, 64 octaves of the sums at a time) are taken in the same places by the
// chunks; their polynomials carry an exponent an octave.  bq_row_general, which streams a row for every pass, is left
// rows of more than about 277 octaves, and of more polynomials than a small workspace holds.
#include "bucket.h"
#include "common.h"

#include <math.h>

#include <algorithm>
#include <atomic>

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
constexpr int kBqRowNodes = 640;                   // nodes of a row whose S is held in LDS, outside bq_row_general
constexpr int kBqRowOct = (kBqRowNodes - 80) / 2;  // at most its octaves
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

// The first word of bucket `at` (octave, part) in the sums.  An octave takes the room of 33 buckets, so that the same part of 16
// octaves, which the contraction's lanes read, lies in different banks (bq_part_kernel, 256 x 128256: 109 us without it,
// 107 with it).
constexpr int kBqAccWords = kBqWin * (kBqSub + 1) * kBqAcc;
__device__ __forceinline__ int bq_place(int at) { return kBqAcc * (at + (at >> 5)); }

template <int L>
struct BqSumsShared {
  uint64_t acc[kBqAccWords];          // one law's (bq_place)
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

// v = q scaled, t: the token's values added to its bucket's sums (if mine).
template <int N>
__device__ __forceinline__ void bq_pack_add(uint64_t* acc, const int (&at)[N], const float (&v0)[N], const float (&t)[N],
                                            const bool (&mine)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float v1 = v0[i] * t[i];
    const float v2 = v1 * t[i];
    uint32_t n0 = (uint32_t)bq_round(v0[i]);
    int n1 = bq_round(v1), n2 = bq_round(v2), n3 = bq_round(v2 * t[i]) << (kBqPack - 32);
    __asm__ volatile("" : "+v"(n0), "+v"(n1), "+v"(n2), "+v"(n3));  // not sunk into the branch
    if (mine[i]) {
      unsigned long long* a = reinterpret_cast<unsigned long long*>(&acc[bq_place(at[i])]);
      atomicAdd(a, (unsigned long long)n0);
      atomicAdd(a + 1, (unsigned long long)(long long)n1);
      atomicAdd(a + 2, ((unsigned long long)(uint32_t)n3 << 32) | (uint32_t)n2);
    }
  }
}

// Law l's sums: every token's values first, then the atomics.
template <int L>
__device__ __forceinline__ void bq_fast_add(const float (&pv)[4], const float (&qv)[4], BqSumsShared<L>& sh, int l) {
  BqTok k[4];
  int at[4];
  float sc[4], t[4];
  bool mine[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    k[i] = bq_tok(pv[i], qv[i]);
    at[i] = (int)(k[i].at & (kBqWinRows - 1));
    sc[i] = __uint_as_float(sh.qm[l][at[i]]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    sc[i] *= qv[i];
    t[i] = k[i].t;
    mine[i] = bq_positive(k[i].w);
  }
  bq_pack_add(sh.acc, at, sc, t, mine);
}

// M of a bucket: value n of its polynomial sums, from the integer sums of a token's v = q 2^shift.
__device__ __forceinline__ double bq_decode(const uint64_t* acc, int n, int shift) {
  const int64_t raw = (int64_t)acc[min(n, 2)];
  const int64_t v = n < 2 ? raw : (n == 2 ? raw & ((1ll << kBqPack) - 1) : raw >> kBqPack);
  return ldexp((double)v, 6 * n - shift);
}
template <int L>
__device__ __forceinline__ double bq_fast_moment(const BqSumsShared<L>& sh, int l, int e, int x) {
  const int at = (e & (kBqWin - 1)) * kBqSub + x / kBqLen;
  return bq_decode(&sh.acc[bq_place(at)], x % kBqLen, (int)(sh.qm[l][at] >> 23) - 127);  // an empty bucket's sums are 0
}

// ------------------------------------------------------------------ (C)
// The two contractions are small dense products in fp64 and run on the matrix cores, 16 octaves
// by 16 columns a wave: S as (octaves x 128 values) x (128 x 27), the parts' polynomials as
// (octaves x 27) x (27 x 128).  On the VALU they are bound by LDS reads of the table: 3.4 us and
// 4.5 us a row of 20 octaves, against 2.6 us and 1.8 us.
typedef double BqQuad __attribute__((ext_vector_type(4)));
// v_mfma_f64_16x16x4_f64: A row / B column lane % 16 at depth lane / 16; D column lane % 16,
// rows lane / 16 + 4 i.

// n[o 28 + column]: octave e0 + o's values (moment(e, x)) against the near nodes and the power sums.  The waves share
// the 128 values out (as many shares an octave tile as there are waves), each for both column tiles, so that a value is
// read and decoded once; g(ct, t): the lane's operand of columns 16 ct .. and values 4 t .. (bq_table, bq_fragments).
// n: room for 8 W octaves.  Begins and ends with a barrier.
template <int W, class G, class Moment>
__device__ __forceinline__ void bq_contract(double* n, int e0, int noct, int tid, int lane, int wid, G&& g, Moment&& moment) {
  const int tiles = noct <= 16 ? 1 : (noct <= 32 ? 2 : 4), shares = W / tiles, stride = tiles * 16 * 28;
  const int share = wid % shares, ot = wid / shares, mr = lane & 15, mk = lane >> 4;
  const int e = e0 + min(ot * 16 + mr, noct - 1);
  BqQuad d0 = {0.0, 0.0, 0.0, 0.0}, d1 = d0;
  __syncthreads();
  const int steps = kBqOct / 4 / shares;  // 2 at least
  for (int t0 = share * steps; t0 < (share + 1) * steps; t0 += 2) {
    double g0[2], g1[2], m[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      g0[t] = g(0, t0 + t);
      g1[t] = g(1, t0 + t);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) m[t] = moment(e, 4 * (t0 + t) + mk);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      d0 = __builtin_amdgcn_mfma_f64_16x16x4f64(m[t], g0[t], d0, 0, 0, 0);
      d1 = __builtin_amdgcn_mfma_f64_16x16x4f64(m[t], g1[t], d1, 0, 0, 0);
    }
  }
  // half the shares are stored, the other half added to them
  const bool add = share >= shares / 2;
  double* to = n + (add ? share - shares / 2 : share) * stride;
#pragma unroll
  for (int turn = 0; turn < 2; ++turn) {
    if (add == (turn == 1)) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int o = ot * 16 + mk + 4 * i;
        if (o < noct) {
          to[o * 28 + mr] = d0[i] + (add ? to[o * 28 + mr] : 0.0);
          if (16 + mr < kBqCols) to[o * 28 + 16 + mr] = d1[i] + (add ? to[o * 28 + 16 + mr] : 0.0);
        }
      }
    }
    __syncthreads();
  }
  if (shares > 2) {
    for (int x = tid; x < noct * 28; x += 64 * W) {
      double v = n[x];
      for (int i = 1; i < shares / 2; ++i) v += n[i * stride + x];
      n[x] = v;
    }
    __syncthreads();
  }
}
// the operand from the table in LDS
__device__ __forceinline__ auto bq_table(const double* g, int lane) {
  return [=](int ct, int t) { return g[min(ct * 16 + (lane & 15), kBqCols - 1) * kBqGPad + 4 * t + (lane >> 4)]; };
}
// and from memory (the second-level cache)
__device__ __forceinline__ auto bq_fragments(int lane) {
  return [=](int ct, int t) { return kBqFrag.g[ct][t][lane]; };
}

// The five power series terms of a far node: p(i) = sum of q (w / 2^e)^i over the tokens, z = -a 2^e.
template <class P>
__device__ __forceinline__ double bq_series(double z, P&& p) {
  double f = p(4) * (1.0 / 24.0);
  f = ::fma(f, z, p(3) * (1.0 / 6.0));
  f = ::fma(f, z, p(2) * 0.5);
  f = ::fma(f, z, p(1));
  return ::fma(f, z, p(0));
}

// S at the nodes k_lo .. k_lo + nk - 1 from the contractions n of the octaves e0 .. e1: groups of `width` of
// the 64 W threads share the octaves out; emit(i, S) by one thread a node, the same for the same i.  Ends with
// a barrier.  red: 64 W values.
template <int W, class Emit>
__device__ __forceinline__ void bq_nodes(const double* n, double* red, int width, int e0, int e1, int k_lo, int nk, int tid,
                                         Emit&& emit) {
  const int groups = 64 * W / width, li = tid & (width - 1), grp = tid / width;
  for (int i0 = 0; i0 < nk; i0 += width) {
    const int k = k_lo + i0 + li;
    double s = 0.0;
    for (int e = e0 + grp; e <= e1; e += groups) {
      const int sx = k + 2 * (e - 127);
      if (sx > kBqNearHi) break;  // and for every octave above
      const int at = (e - e0) * 28;
      if (sx >= kBqNearLo)
        s += n[at + sx - kBqNearLo];
      else
        s += bq_series(-bq_half_pow(sx), [&](int i) { return n[at + kBqNear + i]; });
    }
    red[grp * width + li] = s;
    __syncthreads();
    if (grp == 0 && i0 + li < nk) {
      double t = red[li];
#pragma unroll 4
      for (int x = 1; x < groups; ++x) t += red[x * width + li];
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
    // downwards, so that a power below the fp64 range is followed only by smaller ones; past 128 / i nodes they are
    // below 2^-64 and add nothing to the first series term (the sum of the c_k)
    double s = 0.0, z = bq_half_pow(i * (kBqNearLo - 1 - part));
    const double down = 1.0 / (double)(1 << (4 * i));  // eight nodes back: 2^(-8 i / 2)
    const int k_end = i == 0 ? k_lo : max(k_lo, k_far - 128 / i);
    for (int k = k_far - part; k >= k_end; k -= 8) {
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
  double n[2 * kBqWin * 28];         // contractions of one law's octaves
  double c[L][kBqRowNodes];
  double b[2 * kBqWin * kBqFar];     // of each of two laws, or of one law's 128 octaves
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
  if (nk > kBqRowNodes) return false;  // two laws far apart
  if (tid == 0) sh.over = 0;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    begin(l);
    bq_contract<kBqWaves>(sh.n, rg.e0[l], rg.e1[l] - rg.e0[l] + 1, tid, lane, wid, bq_table(sh.g, lane),
                          [&](int e, int x) { return moment(l, e, x); });
    bq_nodes<kBqWaves>(sh.n, sh.red[0], 128, rg.e0[l], rg.e1[l], k_lo, nk, tid,
                       [&](int i, double S) { sh.c[L - 1 - l][i] = bq_coef<L>(S, k_lo + i, K, rg.q0[0]); });
  }
#pragma unroll
  for (int l = 0; l < L; ++l) bq_far(sh.c[l], sh.b + l * kBqWin * kBqFar, rg.e0[l], rg.e1[l] - rg.e0[l] + 1, k_lo, tid);
  __syncthreads();
  bool over = false;
#pragma unroll
  for (int l = 0; l < L; ++l)
    bq_polynomials(sh.c[l], sh.b + l * kBqWin * kBqFar, sh.g, rg.e0[l], rg.e1[l] - rg.e0[l] + 1, k_lo, lane, wid, [&](int o, int y, double v) {
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
      float4 p4[4];
      float rest[4], place[4];
      bool some[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const BqTok k = bq_tok(pv[i], qv[l][i]);
        some[i] = bq_positive(k.w);
        const int at = some[i] ? (int)k.at - base[l] : 0;
        p4[i] = r4[l][at];
        rest[i] = r1[l][at];
        place[i] = k.t * (1.0f / kBqTUnit);
      }
      __builtin_amdgcn_sched_barrier(0);  // the four tokens' reads are in flight together
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool pos = some[i];
        const float4 a = p4[i];
        const float t = place[i];
        const float f = fmaf(fmaf(fmaf(a.w, t, a.z), t, a.y), t, rest[i]);
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
  double n[2 * kBqWin * 28];
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

// Arguments of the out-of-line forms, in LDS behind the kernel's own: nothing of the caller's registers is kept for a call
// or across one, which the ordinary row would pay for in spills (256 x 32000: 56 -> 60 us).
struct BqCall {
  BqArgs a;
  int64_t b;
  int left;  // the row is left to bq_row_general
};
typedef __attribute__((address_space(3))) char BqLds;
template <class T>
__device__ __forceinline__ T bq_uniform(T x) {
  static_assert(sizeof(T) % 4 == 0, "whole words");
  uint32_t w[sizeof(T) / 4];
  __builtin_memcpy(w, &x, sizeof(T));
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 4; ++i) w[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)w[i]);
  __builtin_memcpy(&x, w, sizeof(T));
  return x;
}
template <class T>
__device__ __forceinline__ T* bq_global(T* x) {  // device memory, also when the pointer comes from LDS
  return (T*)(__attribute__((address_space(1))) T*)x;
}
// Ends with a barrier.
__device__ __forceinline__ void bq_set_call(BqLds* at, const BqArgs& a, int64_t b, int tid) {
  __syncthreads();
  if (tid == 0) {
    BqCall& c = *reinterpret_cast<BqCall*>((char*)at);
    c.a = a;
    c.b = b;
    c.left = 0;
  }
  __syncthreads();
}
__device__ __forceinline__ BqArgs bq_get_call(BqLds* at, int64_t& b) {
  const BqCall& c = *reinterpret_cast<const BqCall*>((char*)at);
  BqArgs a = bq_uniform(c.a);
  b = bq_uniform(c.b);
  a.p = bq_global(a.p);
  a.q1 = bq_global(a.q1);
  a.q2 = bq_global(a.q2);
  a.r = bq_global(a.r);
  a.row_status = bq_global(a.row_status);
  a.rsum = bq_global(a.rsum);
  return a;
}

// One row by streaming passes: any fp32 row, any weight range, kBqWin octaves of a law at a time (r of two
// laws: kBqWin / 2 of each).  raw: the workgroup's LDS; call: its arguments.
template <int L, bool kRes>
__device__ __attribute__((noinline)) void bq_row_general(BqLds* raw, BqLds* call) {
  int64_t b;
  const BqArgs a = bq_get_call(call, b);
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
        bq_contract<kBqWaves>(sh.s.n, w0, w1 - w0 + 1, tid, lane, wid, bq_table(sh.s.g, lane), [&](int e, int x) {
          const int at = (e - w0) * kBqSub + x / kBqLen, n = x % kBqLen;
          return ldexp((double)(int64_t)sh.acc[at * kBqLen + n], 6 * n - (int)sh.s.qm[at]);
        });
        bq_nodes<kBqWaves>(sh.s.n, sh.s.red[0], 128, w0, w1, k_lo, nk, tid,
                           [&](int i, double S) { sh.c[L - 1 - l][i] += S; });
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

// ------------------------------------------------------------------ wide tokens held in registers
// Tokens of any positive fp32 p and q, a window of kBqWin octaves at a time.  `each(f)` calls f(p's four, q's four)
// for every step of the thread's tokens.

// The octaves e0 .. e1 (biased exponents, as integers; e1 < e0: none) and the zero-weight mass of a law over the
// workgroup, in every thread.  Begins with a barrier.
template <int W, int L, class Each>
__device__ __forceinline__ void bq_wide_range(Each&& each, BqStatShared<L, W>& st, int lane, int wid, int& e0, int& e1,
                                              double& q0) {
  constexpr int kBias = 1 << 20;  // makes places unsigned
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
  double z = 0.0;
  each([&](const float (&pv)[4], const float (&qv)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool some = qv[i] > 0.0f, pos = some && pv[i] > 0.0f;
      const uint32_t at = (uint32_t)(bq_wide_tok(pv[i], qv[i]).at + kBias);
      lo = min(lo, pos ? at : 0xFFFFFFFFu);
      hi = max(hi, pos ? at : 0u);
      z += some && !pos ? (double)qv[i] : 0.0;
    }
  });
  lo = bq_wave<false>(lo);
  hi = bq_wave<true>(hi);
  z = wave_sum_dpp(z);
  __syncthreads();
  if (lane == 0) {
    st.u[0][wid] = lo;
    st.u[1][wid] = hi;
    st.q0[0][wid] = z;
  }
  __syncthreads();
  lo = 0xFFFFFFFFu;
  hi = 0u;
  q0 = 0.0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    lo = min(lo, st.u[0][w]);
    hi = max(hi, st.u[1][w]);
    q0 += st.q0[0][w];
  }
  const bool some = hi != 0u;
  e0 = __builtin_amdgcn_readfirstlane(some ? ((int)lo - kBias) >> 5 : 0x7FFFFFF);  // kBqSub parts an octave
  e1 = __builtin_amdgcn_readfirstlane(some ? ((int)hi - kBias) >> 5 : -0x7FFFFFF);
}

// The draft mass of a law's windows so far and past them, from the lowest ratios on.  The tokens past a window have
// larger weights, so their share of S at any node is at most above / below: the rest is left out once that is
// below 2^-40.
struct BqMass {
  double below = 0.0, above = INFINITY;
  __device__ __forceinline__ bool more() const { return above > below * 0x1p-40; }
};

// The sums of the octaves w0 .. w0 + kBqWin - 1 of a law whose last octave is e1, as bq_fast_add's but with the
// scales' shifts in qm and octave w0 first.  Begins with a barrier; bq_contract sets one after it.
template <int W, int L, class Each>
__device__ __forceinline__ void bq_wide_sums(Each&& each, BqSumsShared<L>& sh, double (*mass)[W], BqMass& m, int w0, int e1,
                                             int tid, int lane, int wid) {
  const bool last = w0 + kBqWin - 1 >= e1;  // uniform
  __syncthreads();
  for (int x = tid; x < kBqAccWords; x += 64 * W) sh.acc[x] = 0;
  for (int x = tid; x < kBqWinRows; x += 64 * W) sh.qm[0][x] = 0;
  __syncthreads();
  float in_q = 0.0f, up_q = 0.0f;  // compared in magnitude only
  each([&](const float (&pv)[4], const float (&qv)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int at = bq_wide_tok(pv[i], qv[i]).at - w0 * kBqSub;
      if (pv[i] > 0.0f && qv[i] > 0.0f && at >= 0) {
        if (at < kBqWinRows) {
          atomicMax(&sh.qm[0][at], __float_as_uint(qv[i]));
          in_q += qv[i];
        } else {
          up_q += qv[i];
        }
      }
    }
  });
  if (!last) {
    const double in_w = wave_sum_dpp((double)in_q), up_w = wave_sum_dpp((double)up_q);
    if (lane == 0) {
      mass[0][wid] = in_w;
      mass[1][wid] = up_w;
    }
  }
  __syncthreads();
  if (!last) {
    m.above = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      m.below += mass[0][w];
      m.above += mass[1][w];
    }
  }
  // largest q of each bucket -> the shift that takes it into [2^kBqF, 2^(kBqF + 1))
  for (int x = tid; x < kBqWinRows; x += 64 * W)
    sh.qm[0][x] = (uint32_t)(kBqF + 1 - __builtin_amdgcn_frexp_expf(__uint_as_float(sh.qm[0][x])));
  __syncthreads();
  each([&](const float (&pv)[4], const float (&qv)[4]) {
    int at[4];
    float v0[4], t[4];
    bool mine[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const BqWideTok k = bq_wide_tok(pv[i], qv[i]);
      const uint32_t x = (uint32_t)(k.at - w0 * kBqSub);
      mine[i] = pv[i] > 0.0f && qv[i] > 0.0f && x < (uint32_t)kBqWinRows;
      at[i] = (int)(x & (uint32_t)(kBqWinRows - 1));
      v0[i] = ldexpf(qv[i], (int)sh.qm[0][at[i]]);
      t[i] = k.t;
    }
    bq_pack_add(sh.acc, at, v0, t, mine);
  });
}

// A binary exponent next to that of an octave's polynomials: c and the far series at the octave e0 + o bound their
// values (exp(-a w) is at least e^-2 on the nodes taken) within a factor of about 2^6.
__device__ __forceinline__ int bq_exponent(const double* c, const double* b, int e0, int o, int k_lo) {
  double s = b[o * kBqFar];
  for (int x = kBqNearLo; x <= 0; ++x) s += c[x - 2 * (e0 + o - 127) - k_lo];
  return s > 0.0 ? __builtin_amdgcn_frexp_exp(s) : 0;
}

// A law's polynomials with an exponent an octave: octaves e0 .. e0 + noct - 1, n of them from `first` on in LDS (s4, s1);
// kMem: all of them in memory (g4, g1).  ex: exponents, of every octave with kMem, else of those in LDS.
template <int L>
struct BqWideRows {
  const float4 *g4[L], *s4[L];
  const float *g1[L], *s1[L];
  const int* ex[L];
  int e0[L], noct[L], first[L], n;
};

// r of N tokens; mine (without kMem): the LDS polynomials are the token's (the first ones for a law it has no positive
// ratio in).
template <int L, bool kMem, int N>
__device__ __forceinline__ void bq_wide_eval(const float (&pv)[N], const float (&qv)[L][N], bool rows,
                                             const BqWideRows<L>& w, int K, const double (&q0)[L], double zw,
                                             float (&out)[N], bool (&mine)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) mine[i] = true;
  double f[N];
#pragma unroll
  for (int i = 0; i < N; ++i) f[i] = 0.0;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    float4 a[N];
    float rest[N], t[N];
    int at[N], e[N];
    bool pos[N], out_of[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const BqWideTok k = bq_wide_tok(pv[i], qv[l][i]);
      pos[i] = rows && pv[i] > 0.0f && qv[l][i] > 0.0f;
      at[i] = min(max(k.at - w.e0[l] * kBqSub, 0), w.noct[l] * kBqSub - 1);
      t[i] = k.t * (1.0f / kBqTUnit);
      const int near = at[i] - w.first[l] * kBqSub;
      const bool in = (uint32_t)near < (uint32_t)(w.n * kBqSub);
      mine[i] &= pos[i] ? in : w.first[l] == 0;
      out_of[i] = pos[i] && !in;
      a[i] = w.s4[l][in ? near : 0];
      rest[i] = w.s1[l][in ? near : 0];
      e[i] = w.ex[l][kMem ? at[i] >> 5 : (in ? near >> 5 : 0)];
    }
    __builtin_amdgcn_sched_barrier(0);  // LDS reads first, then those from memory, each kind in flight together
    bool some = false;
#pragma unroll
    for (int i = 0; i < N; ++i) some |= out_of[i];
    if (kMem && __builtin_amdgcn_ballot_w64(some) != 0) {
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (out_of[i]) {
          a[i] = w.g4[l][at[i]];
          rest[i] = w.g1[l][at[i]];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float u = fmaf(fmaf(fmaf(a[i].w, t[i], a[i].z), t[i], a[i].y), t[i], rest[i]);
      if (pos[i]) f[i] += ldexp((double)a[i].x + (double)u, e[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    float qq[L];
#pragma unroll
    for (int l = 0; l < L; ++l) qq[l] = qv[l][i];
    out[i] = bq_out<L>(pv[i], qq, f[i], K, q0, zw);
  }
}

// ------------------------------------------------------------------ one workgroup a row
template <int L>
struct BqRowShared {
  union {
    BqSumsShared<L> sums;
    struct {
      float4 r4[2 * kBqWinRows];  // a window of each of two laws, or 128 octaves of one law
      float r1[2 * kBqWinRows];
    } rows;
  };
  BqSolve<L> solve;
  BqStatShared<L, kBqWaves> stat;
  int ex[2 * kBqWin];
};

// A row of wide tokens (no flags), held in registers from one more load: the laws' windows one after the other into S,
// then r, 128 octaves of polynomials at a time (two laws: pairs of windows of 64); a token's r takes the place of its
// first draft probability.  A row of too many nodes is left, with nothing written.  256 x 32000, the whole call: a draft at
// temperature 0.3 (95 octaves, most mass in the first window) 96 us, a target at 0.3 (both windows) 114, against 166 and 205
// when bq_row_general streamed such rows up to eight times, and 118 and 112 with fp32 tiles of nine exponentials a token.
// not_tail_called: the compiler else takes the call for one that it might make a tail call, and saves 48 registers a lane in
// scratch around it (110 and 124 us).  bq_row_general keeps its saves: without them bq_merge_kernel spills 18 registers
// instead of 2, and calls of few rows, which never reach it, take 0.7 us longer (8 x 128256: 26.7 against 27.5).
template <int L, int PER, bool kRes>
__device__ __attribute__((noinline, not_tail_called)) void bq_row_wide(BqLds* raw, BqLds* call) {
  constexpr int kSteps = PER / 4;
  static_assert(PER <= 32, "a bit a token");
  BqRowShared<L>& sh = *reinterpret_cast<BqRowShared<L>*>((char*)raw);
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  int64_t b;
  const BqArgs a = bq_get_call(call, b);
  const int64_t V = a.V, nparts = a.nsub * kResParts;
  const float *pb = a.p + b * V, *q1 = a.q1 + b * V, *q2 = L == 2 ? a.q2 + b * V : nullptr;
  float pr[kSteps][4], qr[kSteps][L][4];
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    const int64_t xw = min((int64_t)s * kBqStep + wid * 256, V);
    row_load4(pb, xw, lane, V, pr[s]);
    row_load4(q1, xw, lane, V, qr[s][0]);
    if (L == 2) row_load4(q2, xw, lane, V, qr[s][L - 1]);
  }
  BqSolve<L>& so = sh.solve;
  int e0[L], e1[L];
  double q0[L];
  bool any = true;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    const auto each = [&](auto&& f) {
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        float pc[4], qc[L][4];
        bq_step_tokens<L>(pr[s], qr[s], pc, qc);
        f(pc, qc[l]);
      }
    };
    bq_wide_range(each, sh.stat, lane, wid, e0[l], e1[l], q0[l]);
    any &= e1[l] >= e0[l];
  }
  int k_lo = 0, nk = 0;
  if (any) {
    int e_lo = e0[0], e_hi = e1[0];
    if (L == 2) {
      e_lo = min(e_lo, e0[L - 1]);
      e_hi = max(e_hi, e1[L - 1]);
    }
    k_lo = bq_first_node(e_hi, a.K);
    nk = kBqNearHi - 2 * (e_lo - 127) - k_lo + 1;
    if (nk > kBqRowNodes) {
      if (tid == 0) reinterpret_cast<BqCall*>((char*)call)->left = 1;
      return;
    }
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const auto each = [&](auto&& f) {
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
          float pc[4], qc[L][4];
          bq_step_tokens<L>(pr[s], qr[s], pc, qc);
          f(pc, qc[l]);
        }
      };
      BqMass mass;
      for (int w0 = e0[l]; w0 <= e1[l] && mass.more(); w0 += kBqWin) {
        const int w1 = min(w0 + kBqWin - 1, e1[l]);
        bq_wide_sums<kBqWaves>(each, sh.sums, reinterpret_cast<double(*)[kBqWaves]>(so.red[0]), mass, w0, e1[l], tid, lane, wid);
        bq_contract<kBqWaves>(so.n, w0, w1 - w0 + 1, tid, lane, wid, bq_table(so.g, lane), [&](int e, int x) {
          const int at = (e - w0) * kBqSub + x / kBqLen;
          return bq_decode(&sh.sums.acc[bq_place(at)], x % kBqLen, (int)sh.sums.qm[0][at]);
        });
        bq_nodes<kBqWaves>(so.n, so.red[0], 128, w0, w1, k_lo, nk, tid, [&](int i, double S) {
          double& c = so.c[L - 1 - l][i];
          c = w0 == e0[l] ? S : c + S;
        });
      }
    }
#pragma unroll
    for (int l = 0; l < L; ++l)
      for (int i = tid; i < nk; i += kBqThreads) so.c[l][i] = bq_coef<L>(so.c[l][i], k_lo + i, a.K, q0[0]);
    __syncthreads();
  }
  double zw = q0[0];  // K i.i.d. drafts: Q0^(K-1)
  for (int j = 2; j < a.K; ++j) zw *= q0[0];
  BqWideRows<L> w;
  constexpr int kOct = 2 * kBqWin / L;  // octaves of a law's polynomials in LDS
  w.n = kOct;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    w.e0[l] = any ? e0[l] : 0;
    w.noct[l] = any ? e1[l] - e0[l] + 1 : 1;
    w.s4[l] = sh.rows.r4 + l * kBqWinRows;
    w.s1[l] = sh.rows.r1 + l * kBqWinRows;
    w.ex[l] = sh.ex + l * kBqWin;
  }
  const auto build = [&](int l, int win) {  // the polynomials of a law's window (the last pass ended with a barrier)
    w.first[l] = win * kOct;
    if (!any) return;
    const int first = e0[l] + win * kOct, noct = min(kOct, e1[l] - first + 1);
    bq_far(so.c[l], so.b + l * kBqWin * kBqFar, first, noct, k_lo, tid);
    __syncthreads();
    for (int o = tid; o < noct; o += kBqThreads) sh.ex[l * kBqWin + o] = bq_exponent(so.c[l], so.b + l * kBqWin * kBqFar, first, o, k_lo);
    __syncthreads();
    bq_polynomials(so.c[l], so.b + l * kBqWin * kBqFar, so.g, first, noct, k_lo, lane, wid, [&](int o, int y, double v) {
      const int row = o * kBqSub + y / kBqLen, n = y % kBqLen;
      v = ldexp(v, -sh.ex[l * kBqWin + o]);
      const float x = (float)v;
      reinterpret_cast<float*>(sh.rows.r4 + l * kBqWinRows + row)[n] = x;
      if (n == 0) sh.rows.r1[l * kBqWinRows + row] = (float)(v - (double)x);
    });
    __syncthreads();
  };
  uint32_t done = 0u;  // bit 4 s + i: the token has its r
  constexpr int kBatch = 1;  // tokens at a time: the registers hold the row
  for (int i = 0; i * kOct < w.noct[0]; ++i) {
    build(0, i);
    for (int j = 0; j * kOct < (L == 2 ? w.noct[L - 1] : 1); ++j) {
      if (L == 2) build(L - 1, j);
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        float pc[4], qc[L][4];
        bq_step_tokens<L>(pr[s], qr[s], pc, qc);
#pragma unroll
        for (int x = 0; x < 4; x += kBatch) {
          float p1[kBatch], q1[L][kBatch], out[kBatch];
          bool mine[kBatch];
#pragma unroll
          for (int y = 0; y < kBatch; ++y) {
            p1[y] = pc[x + y];
#pragma unroll
            for (int l = 0; l < L; ++l) q1[l][y] = qc[l][x + y];
          }
          bq_wide_eval<L, false, kBatch>(p1, q1, any, w, a.K, q0, zw, out, mine);
#pragma unroll
          for (int y = 0; y < kBatch; ++y) {
            const uint32_t bit = 1u << (4 * s + x + y);
            const bool now = mine[y] && !(done & bit);
            qr[s][0][x + y] = now ? out[y] : qr[s][0][x + y];
            done |= now ? bit : 0u;
          }
        }
      }
      __syncthreads();
    }
  }
  bq_status(a, b, 0, tid);
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    const int64_t xw = (int64_t)s * kBqStep + wid * 256;
    float pc[4], out[L][4];
    bq_step_tokens<L>(pr[s], qr[s], pc, out);
    if (xw < V) row_store4(a.r + b * V, xw, lane, V, out[0]);
    if (kRes) {
      const double tot = bq_residual(pc, out[0]);
      if (lane == 0 && (xw >> 8) < nparts) a.rsum[b * nparts + (xw >> 8)] = tot;
    }
  }
}

// Rows of up to 1024 PER tokens: thread t holds PER tokens in registers.
template <int L, int PER, bool kRes>
__global__ __launch_bounds__(kBqThreads) void bq_row_kernel(BqArgs a) {
  constexpr int kRaw = sizeof(BqRowShared<L>) > sizeof(BqGeneral<L>) ? sizeof(BqRowShared<L>) : sizeof(BqGeneral<L>);
  __shared__ __align__(16) char raw[kRaw + sizeof(BqCall)];
  BqLds *const lds = (BqLds*)raw, *const call = lds + kRaw;
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
  for (int x = tid; x < kBqAccWords; x += kBqThreads) sh.sums.acc[x] = 0;
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
  const int flags = rg.bad ? kRowBadProb : ((a.s_max > 0 && rg.nsup > a.s_max) ? kRowSupport : 0);
  if (!flags && rg.special) {
    bq_set_call(call, a, b, tid);
    bq_row_wide<L, PER, kRes>(lds, call);
    __syncthreads();
    if (reinterpret_cast<const BqCall*>((char*)call)->left) bq_row_general<L, kRes>(lds, call);
    return;
  }
  bool any = !flags;
#pragma unroll
  for (int l = 0; l < L; ++l) any &= rg.e1[l] > 0;
  if (any) {
    bq_fast_scales<L>(sh.sums, tid, kBqThreads);
    float4* r4[L];
    float* r1[L];
#pragma unroll
    for (int l = 0; l < L; ++l) {
      r4[l] = sh.rows.r4 + l * kBqWinRows;
      r1[l] = sh.rows.r1 + l * kBqWinRows;
    }
    const auto begin = [&](int l) {  // (B)
      if (l > 0)
        for (int x = tid; x < kBqAccWords; x += kBqThreads) sh.sums.acc[x] = 0;
      __syncthreads();
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        float pc[4], qc[L][4];
        bq_step_tokens<L>(pr[s], qr[s], pc, qc);
        bq_fast_add<L>(pc, qc[l], sh.sums, l);
      }
    };
    const auto moment = [&](int l, int e, int x) { return bq_fast_moment<L>(sh.sums, l, e, x); };
    if (!bq_solve<L>(sh.solve, rg, a.K, r4, r1, tid, lane, wid, begin, moment)) {  // (C)
      bq_set_call(call, a, b, tid);
      bq_row_general<L, kRes>(lds, call);
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
    r4[l] = sh.rows.r4 + l * kBqWinRows;
    r1[l] = sh.rows.r1 + l * kBqWinRows;
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
// A chunk's record: what one law's sums add to S at any node, in fp64: S at the nodes where some octave of the chunk is
// near or past (22 and two an octave more), and the five power sums of the far nodes below.  About 0.5 kB for
// ordinary rows; the room is there for kBqRecNodes nodes (278 octaves), so that no chunk of probabilities up to 1 is too
// wide.  A chunk contracts its own sums.  Records of the octaves' moments left the contraction to the merge, one
// workgroup a row, and took 20 kB in fp32 for 32 octaves, past which the row was streamed by one workgroup: drafts at
// temperature 0.5, 8 x 128256: 321 us, now 37; two laws, 8 x 32000: 45, now 30; 512 x 128256: parts 197 and merge 42, now 202 and 19.
constexpr int kBqRecNodes = 576;
constexpr int kBqRecLaw = 8 + kBqRecNodes;  // doubles of a law: power sums, then S
struct alignas(64) BqRecHdr {
  int32_t bad, wide, lost, nsup;     // wide: bq_wide_tok tokens; lost: more octaves than a record holds
  int32_t e0, e1;                    // octaves (e1 < e0: none)
  double q0;
};
struct alignas(64) BqPlan {
  int32_t flags, done, any, wide;    // done: r (and the residual sums) are written already
  int32_t e0[2], e1[2];
  double q0[2];
};
constexpr int kBqOctRows = kBqSub * (int)(sizeof(float4) + sizeof(float)) + (int)sizeof(int);  // an octave's polynomials
__host__ __device__ inline int64_t bq_law_rows(int noct) { return ((int64_t)noct * kBqOctRows + 63) / 64 * 64; }
struct BqWork {
  BqPlan* plan;   // [B]
  char* area;     // [B] areas of `room` bytes: the records, then (the merge is done with them) the polynomials
  int64_t room;
  int C;
  int64_t chunk;  // tokens of a chunk (a multiple of 2048)
  static constexpr int64_t kSlot = (int64_t)sizeof(BqRecHdr) + kBqRecLaw * (int64_t)sizeof(double);  // of a chunk and law
  template <int L>
  __device__ __forceinline__ char* rec(int64_t b, int c, int l) const { return area + b * room + (c * L + l) * kSlot; }
  static __device__ __forceinline__ double* sums(char* rec) { return reinterpret_cast<double*>(rec + sizeof(BqRecHdr)); }
};
constexpr int kBqMergeHdr = 1024;    // chunks of a row, at most
constexpr int kBqPartThreads = 512;  // two workgroups a CU: one loads while the other sums
constexpr int kBqPartWaves = kBqPartThreads / 64;
constexpr int kBqPartStep = 4 * kBqPartThreads;

struct BqPartShared {
  BqSumsShared<1> sums;
  double n[kBqWin * 28];
  double red[kBqPartThreads];
  double mass[2][kBqPartWaves];
  double power[kBqFar];
  BqStatShared<1, kBqPartWaves> stat;
};

// The sums of the octaves w0 .. w1 added to a record of the octaves e0 .. e1 (the first ones are stored).
template <class Moment>
__device__ __forceinline__ void bq_record(BqPartShared& sh, double* rec, int e0, int e1, int w0, int w1, int tid, int lane,
                                          int wid, Moment&& moment) {
  const bool first = w0 == e0;
  const int noct = w1 - w0 + 1;
  bq_contract<kBqPartWaves>(sh.n, w0, noct, tid, lane, wid, bq_fragments(lane), moment);
  if (wid == kBqPartWaves - 1) {  // power sums in units of 2^w1 and 2^e1, a lane an octave
#pragma unroll 1
    for (int i = 0; i < kBqFar; ++i) {
      const double v = lane < noct ? ldexp(sh.n[lane * 28 + kBqNear + i], i * (w0 + lane - w1)) : 0.0;
      const double tot = wave_sum_dpp(v);
      if (lane == 0) {
        const double up = ldexp(tot, i * (w1 - e1));
        sh.power[i] = tot;
        rec[i] = first ? up : rec[i] + up;
      }
    }
  }
  const auto emit = [&](int i, double S) { rec[8 + i] = first ? S : rec[8 + i] + S; };
  const int nk = kBqNear + 2 * (w1 - w0), below = 2 * (e1 - w1);  // nodes where the whole window is far
  bq_nodes<kBqPartWaves>(sh.n, sh.red, nk <= 64 ? 64 : 128, w0, w1, kBqNearLo - 2 * (w1 - 127), nk, tid,
                         [&](int i, double S) { emit(below + i, S); });
  for (int i = tid; i < below; i += kBqPartThreads)
    emit(i, bq_series(-bq_half_pow(kBqNearLo - below + i), [&](int x) { return sh.power[x]; }));
}

// One law of a chunk (512 PER tokens at most, in registers).  The workgroups of a chunk's two laws lie 8 apart, on the same
// XCD, so that the second one's p comes from its cache.  (Both laws in one workgroup: half the tokens a chunk, twice
// the contractions; 256 x 32000: 66 us, now 53.)
template <int PER>
__global__ __launch_bounds__(kBqPartThreads, 4) void bq_part_kernel(BqArgs a, BqWork wk, int laws, unsigned units) {
  constexpr int kSteps = PER / 4;
  __shared__ __align__(16) BqPartShared sh;
  const int l = laws == 2 ? (int)(blockIdx.x >> 3) & 1 : 0;
  const unsigned unit = laws == 2 ? (blockIdx.x >> 4 << 3) | (blockIdx.x & 7u) : blockIdx.x;
  if (unit >= units) return;
  const int64_t b = unit / (unsigned)wk.C, V = a.V;
  const int ch = (int)(unit % (unsigned)wk.C);
  const float* pb = a.p + b * V;
  const float* qb = (l == 0 ? a.q1 : a.q2) + b * V;
  const int64_t x0 = (int64_t)ch * wk.chunk, end = min(V, x0 + wk.chunk);
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  char* rec = laws == 2 ? wk.rec<2>(b, ch, l) : wk.rec<1>(b, ch, 0);
  float pr[kSteps][4], qr[kSteps][1][4];
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    const int64_t xw = min(x0 + (int64_t)s * kBqPartStep + wid * 256, end);
    row_load4(pb, xw, lane, end, pr[s]);
    row_load4(qb, xw, lane, end, qr[s][0]);
  }
  const auto each = [&](auto&& f) {
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      if (x0 + (int64_t)s * kBqPartStep >= end) break;  // uniform
      float pc[4], qc[1][4];
      bq_step_tokens<1>(pr[s], qr[s], pc, qc);
      f(pc, qc[0]);
    }
  };
  for (int x = tid; x < kBqAccWords; x += kBqPartThreads) sh.sums.acc[x] = 0;
  for (int x = tid; x < kBqWinRows; x += kBqPartThreads) sh.sums.qm[0][x] = 0;
  __syncthreads();
  BqFastStats<1> st;
  each([&](const float (&pv)[4], const float (&qv)[4]) {
    float q1[1][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) q1[0][i] = qv[i];
    bq_fast_count<1>(pv, q1, sh.sums, st, a.s_max > 0);
  });
  const BqRange<1> rg = bq_combine(st, sh.stat, lane, wid);
  int e0 = rg.e0[0], e1 = rg.e1[0] > 0 ? rg.e1[0] : -0x7FFFFFF;
  double q0 = rg.q0[0];
  const bool wide = !rg.bad && rg.special;  // uniform, as the other conditions
  if (wide) bq_wide_range(each, sh.stat, lane, wid, e0, e1, q0);
  const bool lost = e1 >= e0 && kBqNear + 2 * (e1 - e0) > kBqRecNodes;
  if (tid == 0) {
    BqRecHdr h;
    h.bad = rg.bad;
    h.wide = wide;
    h.lost = lost;
    h.nsup = rg.nsup;
    h.e0 = e0;
    h.e1 = e1;
    h.q0 = q0;
    *reinterpret_cast<BqRecHdr*>(rec) = h;
  }
  if (rg.bad || lost) return;
  BqMass mass;
  for (int w0 = e0; w0 <= e1 && mass.more(); w0 += kBqWin) {  // an ordinary chunk has one window
    const int w1 = min(w0 + kBqWin - 1, e1);
    if (wide) {
      bq_wide_sums<kBqPartWaves>(each, sh.sums, sh.mass, mass, w0, e1, tid, lane, wid);
    } else {
      bq_fast_scales<1>(sh.sums, tid, kBqPartThreads);
      __syncthreads();
      each([&](const float (&pv)[4], const float (&qv)[4]) { bq_fast_add<1>(pv, qv, sh.sums, 0); });
    }
    // the octaves' places in the sums and the scales' form differ
    const int at0 = wide ? w0 : 0, drop = wide ? 0 : 23, less = wide ? 0 : 127;
    bq_record(sh, BqWork::sums(rec), e0, e1, w0, w1, tid, lane, wid, [&](int e, int x) {
      const int at = ((e - at0) & (kBqWin - 1)) * kBqSub + x / kBqLen;
      return bq_decode(&sh.sums.acc[bq_place(at)], x % kBqLen, (int)(sh.sums.qm[0][at] >> drop) - less);
    });
  }
}

// Octaves of a row's polynomials kept in LDS by the evaluation.  Rows of more take bq_wide_eval with their middle ones
// there (and the exponents in place of the last three) and the others in memory: 256 x 128256, drafts at temperature 0.5,
// 40 to 50 octaves, the whole call: 310 us with all of them read from memory by bq_fast_eval, 219 so.
constexpr int kBqEvalOct = 32, kBqEvalWide = 29;
static_assert((kBqEvalOct - kBqEvalWide) * kBqSub * sizeof(float4) >= kBqRowOct * sizeof(int), "room for the exponents");
template <int L>
struct BqMergeShared {
  double g[kBqCols * kBqGPad];
  double c[L][kBqRowNodes];
  double b[kBqRowOct * kBqFar];
  double red[8][128];
  int ex[kBqRowOct];
  int win[L][2][kBqMergeHdr];  // chunks' first and last octaves
  int over;
};

// (C) of a row from its chunks' records, added in chunk order; rows the records do not cover are taken whole by
// bq_row_general.
template <int L, bool kRes>
__global__ __launch_bounds__(kBqThreads) void bq_merge_kernel(BqArgs a, BqWork wk) {
  constexpr int kRaw = sizeof(BqMergeShared<L>) > sizeof(BqGeneral<L>) ? sizeof(BqMergeShared<L>) : sizeof(BqGeneral<L>);
  __shared__ __align__(16) char raw[kRaw + sizeof(BqCall)];
  BqLds *const lds = (BqLds*)raw, *const call = lds + kRaw;
  BqMergeShared<L>& sh = *reinterpret_cast<BqMergeShared<L>*>(raw);
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t b = blockIdx.x;
  bq_load_table(sh.g, tid);
  if (tid == 0) sh.over = 0;
  bool bad = false, wide = false, lost = false, any = true;
  int nsup = 0, e0[L], e1[L];
  double q0[L];
#pragma unroll
  for (int l = 0; l < L; ++l) {
    e0[l] = 0x7FFFFFF;
    e1[l] = -0x7FFFFFF;
    q0[l] = 0.0;
  }
  // every wave reads the headers, a lane a chunk (their octaves are kept in LDS by the first)
  for (int c0 = 0; c0 < wk.C; c0 += 64) {
    const int c = min(c0 + lane, wk.C - 1);
    const bool mine = c0 + lane < wk.C;
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const BqRecHdr h = *reinterpret_cast<const BqRecHdr*>(wk.rec<L>(b, c, l));
      bad |= __builtin_amdgcn_ballot_w64(h.bad != 0) != 0;
      wide |= __builtin_amdgcn_ballot_w64(h.wide != 0) != 0;
      lost |= __builtin_amdgcn_ballot_w64(h.lost != 0) != 0;
      if (L == 1) nsup += __builtin_amdgcn_readfirstlane(wave_sum_int(mine ? h.nsup : 0));
      constexpr int kBias = 0x8000000;  // unsigned
      e0[l] = min(e0[l], (int)bq_wave<false>((uint32_t)(h.e0 + kBias)) - kBias);
      e1[l] = max(e1[l], (int)bq_wave<true>((uint32_t)(h.e1 + kBias)) - kBias);
      if (__builtin_amdgcn_ballot_w64(h.q0 != 0.0) != 0) q0[l] += wave_sum_dpp(mine ? h.q0 : 0.0);
      if (wid == 0 && mine) {
        sh.win[l][0][c] = h.e0;
        sh.win[l][1][c] = h.e1;
      }
    }
  }
  int64_t bytes = 0;
  int noct[L];
#pragma unroll
  for (int l = 0; l < L; ++l) {
    e0[l] = __builtin_amdgcn_readfirstlane(e0[l]);
    e1[l] = __builtin_amdgcn_readfirstlane(e1[l]);
    any &= e1[l] >= e0[l];
    noct[l] = e1[l] - e0[l] + 1;
    wide |= e1[l] >= e0[l] && noct[l] > kBqEvalOct;  // uniform
  }
  const int flags = bad ? kRowBadProb : ((a.s_max > 0 && nsup > a.s_max) ? kRowSupport : 0);
  any &= !flags;
  bool general = !bad && lost;
  int k_lo = 0, nk = 0;
  if (any && !general) {
    int e_lo = e0[0], e_hi = e1[0];
    if (L == 2) {
      e_lo = min(e_lo, e0[L - 1]);
      e_hi = max(e_hi, e1[L - 1]);
    }
    k_lo = bq_first_node(e_hi, a.K);
    nk = kBqNearHi - 2 * (e_lo - 127) - k_lo + 1;
#pragma unroll
    for (int l = 0; l < L; ++l) bytes += bq_law_rows(noct[l]);
    general = nk > kBqRowNodes || bytes > wk.room;
  }
  __syncthreads();
  if (any && !general) {
    const int li = tid & 127, grp = tid >> 7;
#pragma unroll
    for (int l = 0; l < L; ++l)
      for (int i0 = 0; i0 < nk; i0 += 128) {
        const int k = k_lo + i0 + li;
        double s = 0.0;
        for (int c = grp; c < wk.C; c += 8) {
          const int f0 = sh.win[l][0][c], f1 = sh.win[l][1][c];
          if (f1 < f0) continue;  // uniform in a wave
          const double* rec = BqWork::sums(wk.rec<L>(b, c, l));
          const int sx = k + 2 * (f1 - 127), i = sx - kBqNearLo;
          if (i < 0)
            s += bq_series(-bq_half_pow(sx), [&](int x) { return rec[x]; });
          else if (i < kBqNear + 2 * (f1 - f0))
            s += rec[8 + i];
        }
        sh.red[grp][li] = s;
        __syncthreads();
        if (grp == 0 && i0 + li < nk) {
          double t = sh.red[0][li];
#pragma unroll
          for (int x = 1; x < 8; ++x) t += sh.red[x][li];
          sh.c[L - 1 - l][i0 + li] = bq_coef<L>(t, k, a.K, q0[0]);
        }
        __syncthreads();
      }
    // the records are done with: the polynomials take their place
    bool over = false;
    char* rows = wk.area + b * wk.room;
#pragma unroll
    for (int l = 0; l < L; ++l) {
      bq_far(sh.c[l], sh.b, e0[l], noct[l], k_lo, tid);
      __syncthreads();
      if (wide) {
        for (int o = tid; o < noct[l]; o += kBqThreads) sh.ex[o] = bq_exponent(sh.c[l], sh.b, e0[l], o, k_lo);
        __syncthreads();
      }
      float4* r4 = reinterpret_cast<float4*>(rows);
      float* r1 = reinterpret_cast<float*>(r4 + noct[l] * kBqSub);
      int* ex = reinterpret_cast<int*>(r1 + noct[l] * kBqSub);
      rows += bq_law_rows(noct[l]);
      bq_polynomials(sh.c[l], sh.b, sh.g, e0[l], noct[l], k_lo, lane, wid, [&](int o, int y, double v) {
        const int row = o * kBqSub + y / kBqLen, n = y % kBqLen;
        if (wide) v = ldexp(v, -sh.ex[o]);
        const float f = (float)v;
        reinterpret_cast<float*>(r4 + row)[n] = f;
        if (n == 0) {
          over |= !(fabsf(f) <= 0x1p100f);
          r1[row] = (float)(v - (double)f);
        }
      });
      if (wide)
        for (int o = tid; o < noct[l]; o += kBqThreads) ex[o] = sh.ex[o];
      if (L == 2) __syncthreads();  // b and the exponents are written again
    }
    if (over) sh.over = 1;
    __syncthreads();
    general = sh.over != 0;
  }
  if (general) {
    bq_set_call(call, a, b, tid);
    bq_row_general<L, kRes>(lds, call);
  } else {
    bq_status(a, b, flags, tid);
  }
  if (tid == 0) {
    BqPlan pl;
    pl.flags = general ? 0 : flags;
    pl.done = general;
    pl.any = any;
    pl.wide = wide;
#pragma unroll
    for (int l = 0; l < 2; ++l) {
      pl.e0[l] = any ? e0[l < L ? l : 0] : 0;
      pl.e1[l] = any ? e1[l < L ? l : 0] : 0;
      pl.q0[l] = q0[l < L ? l : 0];
    }
    wk.plan[b] = pl;
  }
}

constexpr int kBqEvalThreads = 256;
constexpr int kBqEvalTile = 4 * kBqEvalThreads;  // 1024 tokens, four a thread

// (D) on tiles of 1024 tokens: workgroup w takes the tiles [w per, (w + 1) per) of the B T
// (row, tile) pairs, row-major, the next tile's p and q in flight; a row's polynomials go to LDS, a wide row's as
// far as they fit.
template <int L, bool kRes>
__global__ __launch_bounds__(kBqEvalThreads) void bq_eval_kernel(BqArgs a, BqWork wk, int64_t T, int64_t G, int per) {
  __shared__ float4 s_r4[L][kBqEvalOct * kBqSub];
  __shared__ float s_r1[L][kBqEvalOct * kBqSub];
  const auto s_ex = [&](int l) { return reinterpret_cast<int*>(&s_r4[l][kBqEvalWide * kBqSub]); };
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t V = a.V, nparts = a.nsub * kResParts;
  const int64_t g0 = (int64_t)blockIdx.x * per, g1_ = min(g0 + per, G);
  if (g0 >= g1_) return;
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
  BqWideRows<L> w;
  w.n = kBqEvalWide;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    w.s4[l] = s_r4[l];
    w.s1[l] = s_r1[l];
    w.ex[l] = s_ex(l);
  }
  bool rows = false;
  for (int64_t g = g0; g < g1_; ++g) {
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
      const int in_lds = pl.wide ? kBqEvalWide : kBqEvalOct;
      const char* at = wk.area + cb * wk.room;
#pragma unroll
      for (int l = 0; l < L; ++l) {
        w.e0[l] = pl.e0[l];
        w.noct[l] = pl.e1[l] - pl.e0[l] + 1;
        base[l] = pl.e0[l] * kBqSub;
        q0[l] = pl.q0[l];
        w.first[l] = max(0, (w.noct[l] - in_lds) / 2);
        w.g4[l] = reinterpret_cast<const float4*>(at);
        w.g1[l] = reinterpret_cast<const float*>(w.g4[l] + w.noct[l] * kBqSub);
        at += bq_law_rows(w.noct[l]);
      }
      if (rows) {
#pragma unroll
        for (int l = 0; l < L; ++l) {
          for (int x = tid; x < min(w.noct[l], in_lds) * kBqSub; x += kBqEvalThreads) {
            s_r4[l][x] = w.g4[l][w.first[l] * kBqSub + x];
            s_r1[l][x] = w.g1[l][w.first[l] * kBqSub + x];
          }
          if (pl.wide) {
            const int* ex = reinterpret_cast<const int*>(w.g1[l] + w.noct[l] * kBqSub);
            for (int x = tid; x < w.noct[l]; x += kBqEvalThreads) s_ex(l)[x] = ex[x];
          }
        }
      }
      __syncthreads();
    }
    if (++t == T) {
      t = 0;
      ++b;
    }
    if (g + 1 < g1_) load();
    if (pl.done) continue;  // uniform
    float out[4];
    if (rows && pl.wide) {
      bool mine[4];
      bq_wide_eval<L, true, 4>(pc, qc, rows, w, a.K, q0, zw, out, mine);
    } else {
      bq_fast_eval<L>(pc, qc, rows, w.s4, w.s1, base, a.K, q0, zw, out);
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

size_t bq_align(size_t x) { return (x + 255) & ~(size_t)255; }

// Workgroups of the evaluation: every resident slot of the device once (looked up once per device; threads that look it up
// at the same time store the same value).
unsigned bq_eval_grid(const void* kernel, int64_t tiles, int slot) {
  static std::atomic<int> s_slots[64][2];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  int slots = s_slots[dev][slot].load(std::memory_order_relaxed);
  if (slots <= 0) {
    int cus = 0, occ = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, kBqEvalThreads, 0) != hipSuccess) occ = 0;
    slots = std::max(cus, 1) * std::max(occ, 1);
    s_slots[dev][slot].store(slots, std::memory_order_relaxed);
  }
  const int64_t per = (tiles + slots - 1) / slots;
  return (unsigned)std::max<int64_t>(1, (tiles + per - 1) / per);
}

// The chunks of a call and its workspace; false if the workspace has no room for them.
bool bq_carve(void* base, size_t bytes, int64_t B, int64_t V, int L, BqWork* wk) {
  const size_t fixed = bq_align(sizeof(BqPlan) * B);
  if (base == nullptr || bytes <= fixed) return false;
  const int64_t room = (int64_t)((bytes - fixed) / (size_t)B) / 64 * 64;
  // as many chunks as there are tiles (512 threads of 32 tokens; of 4096 tokens when the rows do not fill the chip)
  const int64_t full = 32 * kBqPartThreads;
  const int64_t least = (V + full - 1) / full;
  const int64_t tile = B * L * least >= 512 ? full : 8 * kBqPartThreads;
  const int64_t C = std::min<int64_t>(
      {(V + tile - 1) / tile, (1024 + B - 1) / B + least, room / (L * BqWork::kSlot), kBqMergeHdr});
  if (C < least) return false;
  wk->chunk = ((V + C - 1) / C + kBqPartStep - 1) / kBqPartStep * kBqPartStep;
  wk->C = (int)((V + wk->chunk - 1) / wk->chunk);
  wk->room = room;
  wk->plan = static_cast<BqPlan*>(base);
  wk->area = static_cast<char*>(base) + fixed;
  return true;
}

template <int L, bool kRes>
void bq_launch_chunks(const BqArgs& a, const BqWork& wk, int64_t B, hipStream_t st) {
  const unsigned units = (unsigned)(B * wk.C);
  const dim3 parts(L == 2 ? (units + 7) / 8 * 16 : units);
  const int64_t per = wk.chunk / kBqPartThreads;
  if (per <= 8)
    hipLaunchKernelGGL(bq_part_kernel<8>, parts, dim3(kBqPartThreads), 0, st, a, wk, L, units);
  else if (per <= 16)
    hipLaunchKernelGGL(bq_part_kernel<16>, parts, dim3(kBqPartThreads), 0, st, a, wk, L, units);
  else
    hipLaunchKernelGGL(bq_part_kernel<32>, parts, dim3(kBqPartThreads), 0, st, a, wk, L, units);
  hipLaunchKernelGGL((bq_merge_kernel<L, kRes>), dim3((unsigned)B), dim3(kBqThreads), 0, st, a, wk);
  const int64_t T = (a.V + kBqEvalTile - 1) / kBqEvalTile, G = B * T;
  const unsigned n = bq_eval_grid(reinterpret_cast<const void*>(&bq_eval_kernel<L, false>), G, L - 1);
  hipLaunchKernelGGL((bq_eval_kernel<L, kRes>), dim3(n), dim3(kBqEvalThreads), 0, st, a, wk, T, G,
                     (int)((G + n - 1) / n));
}

template <bool kRes>
void bq_launch_rows(const BqArgs& a, int64_t B, hipStream_t st) {
  if (a.V <= 4 * kBqThreads)
    hipLaunchKernelGGL((bq_row_kernel<1, 4, kRes>), dim3((unsigned)B), dim3(kBqThreads), 0, st, a);
  else if (a.V <= 16 * kBqThreads)
    hipLaunchKernelGGL((bq_row_kernel<1, 16, kRes>), dim3((unsigned)B), dim3(kBqThreads), 0, st, a);
  else
    hipLaunchKernelGGL((bq_row_kernel<1, 32, kRes>), dim3((unsigned)B), dim3(kBqThreads), 0, st, a);
}

}  // namespace

hipError_t launch_bucket(const float* p, const float* q1, const float* q2, int64_t B, int64_t V, int K, int s_max,
                         bool range_flag, float* r, int32_t* row_status, bool set_status, double* rsum,
                         void* workspace, size_t workspace_bytes, hipStream_t st) {
  const BqArgs a = {p, q1, q2, V, K, s_max, range_flag ? 1 : 0, set_status ? 1 : 0, r, row_status, rsum,
                    (V + kResSub - 1) / kResSub};
  // A row in one workgroup's registers: two laws up to 4096 tokens (past that chunks are as fast or faster, also where a
  // law's share of the registers would do: 128 x 4600 46 us against 36, 256 x 16000 59.4 against 59.6, 512 x 8192 99 against 74).
  const bool fits = V <= (q2 ? 4 : kBqPer) * kBqThreads;
  // One law in registers from B = 128 on, or 4096 tokens at most: rows of 32768 36 us against 40 in chunks at B = 96, 37 against 32
  // at 64; shorter ones win by a few us at any B (12000 tokens 23 against 24 to 40), but wide rows of few positions
  // want the chunks' workgroups.  The two forms round differently (below r's fp32 rounding), so r's last bits may
  // differ between a row alone and in a batch.
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
      hipLaunchKernelGGL((bq_row_kernel<2, 4, false>), dim3((unsigned)B), dim3(kBqThreads), 0, st, a);
    else if (rsum)
      bq_launch_rows<true>(a, B, st);
    else
      bq_launch_rows<false>(a, B, st);
  } else {
    return hipErrorInvalidValue;  // no room for the chunks' records: the workspace is smaller than its query says
  }
  return hipGetLastError();
}

}  // namespace mdss
