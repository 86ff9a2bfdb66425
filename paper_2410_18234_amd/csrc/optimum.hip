// Optimal acceptance diagnostics, gfx950.
//
// Theorem 3 (K = 2 drafts from q): P* = min over token sets S of
// P(S) + Q(S^c)^2 + 2 Q(S) Q(S^c) = Qt^2 + min_S (P(S) - Q(S)^2), with P, Q
// the target / draft masses and Qt the draft mass of the row; Remark 2's
// K-draft form (conjectured for K > 2) replaces the power 2 by K.  By strict
// convexity of x^K a minimising S is {w < threshold} for w = p / q, so the
// minimum over all 2^V sets equals the minimum over the V + 1 prefixes of the
// tokens ordered by w ascending (the ratio rounded to fp32; q = 0 last; ties by
// lower id): f(P, Q) = P + Qt^K - Q^K at the prefix's masses.
//
// Only the neighbourhood of the minimum is ranked.  Inside a bin of ratios
// [w_lo, w_hi) that starts at (P0, Q0) and holds the masses dP, dQ,
//   f >= f(P0, Q0) + min over x in [0, dQ] of (w_lo x - ((Q0 + x)^K - Q0^K)),
// and the minimised function is concave in x, so its minimum is at an end.  Bins
// whose bound lies above the smallest f at a bin's end hold no minimiser.  A row's
// masses are summed into 16 bins an octave, the bins that remain (a few, next
// to the minimum) into up to 256 parts each, and the tokens of the parts that remain
// (tens) are ranked one against the other.
// Masses are 64-bit integers in units of 2^-61 (tokens above 2^-38 enter exactly),
// summed by LDS atomics, so the sums do not depend on the order.  Rows whose
// masses lie outside [2^-6, 2] or that leave too many candidates (w nearly
// constant near the minimum) are ranked whole (rank.h), from the masses ranked
// after each entry: P_k = Pt - (p mass after), Q_k = Qt - (q mass after).
//
// Notation: p = target, q = draft.
#include "rank.h"

namespace mdss {

namespace {

__device__ __forceinline__ double ipow(double x, int K) {
  double y = 1.0;
  for (int i = 0; i < K; ++i) y *= x;
  return y;
}

struct OptSpec {
  struct Args {
    const float *p, *q;
    double* pstar;
    int32_t* kstar;
    int32_t* row_status;
    int K;
  };
  struct Row {
    const float *in0, *in1, *in2;
    double* pstar;
    int32_t* kstar;
    int32_t* row_status;
    int64_t b;
    double Pt, Qt;
    int K;
  };
  struct State {
    double best = __longlong_as_double(0x7ff0000000000000ll);  // +inf
    uint32_t k = 0xffffffffu;                                   // prefix length attaining it
  };
  static __device__ __forceinline__ Row row(const Args& a, int64_t b, int64_t V) {
    Row r;
    r.in0 = a.p + b * V;
    r.in1 = a.q + b * V;
    r.in2 = r.in1;
    r.pstar = a.pstar;
    r.kstar = a.kstar;
    r.row_status = a.row_status;
    r.b = b;
    r.Pt = r.Qt = 0.0;
    r.K = a.K;
    return r;
  }
  // w = p / q ascending; q = 0 (and a ratio above the fp32 range) rank last
  static __device__ __forceinline__ uint32_t word(float p, float q, float) {
    const float w = q > 0.0f ? (float)((double)p / (double)q) : __int_as_float(0x7f800000);
    return __float_as_uint(w + 0.0f);
  }
  static __device__ __forceinline__ void set_totals(Row& r, double pt, double qt) {
    r.Pt = pt;
    r.Qt = qt;
  }
  static __device__ __forceinline__ void masses(const Row&, uint32_t, float p, float q, float, double* m1,
                                                double* m2) {
    *m1 = (double)p;
    *m2 = (double)q;
  }
  static __device__ __forceinline__ void visit(const Row& r, State& st, uint32_t rank, int, float, float, float,
                                               double s1, double s2) {
    const double f = (r.Pt - s1) + ipow(r.Qt, r.K) - ipow(r.Qt - s2, r.K);
    const uint32_t k = rank + 1u;
    if (f < st.best || (f == st.best && k < st.k)) {
      st.best = f;
      st.k = k;
    }
  }
  static __device__ __forceinline__ void flag(const Row& r, int64_t, int flags) {
    if (threadIdx.x == 0) {
      r.pstar[r.b] = __longlong_as_double(0x7ff8000000000000ll);
      if (r.kstar) r.kstar[r.b] = -1;
      if (r.row_status) r.row_status[r.b] |= flags;
    }
  }
  static __device__ __forceinline__ void finish(const Row& r, State& st, double, double, double* red) {
    // block minimum of (value, prefix length), smaller length on equal values
    double v = st.best;
    uint32_t k = st.k;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const double ov = __shfl_xor(v, off, 64);
      const uint32_t ok = __shfl_xor(k, off, 64);
      if (ov < v || (ov == v && ok < k)) {
        v = ov;
        k = ok;
      }
    }
    __shared__ uint32_t redk[kRankWaves];
    if ((threadIdx.x & 63) == 0) {
      red[threadIdx.x >> 6] = v;
      redk[threadIdx.x >> 6] = k;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      double bv = ipow(r.Qt, r.K);  // the empty prefix
      uint32_t bk = 0;
      for (int w = 0; w < kRankWaves; ++w)
        if (red[w] < bv || (red[w] == bv && redk[w] < bk)) {
          bv = red[w];
          bk = redk[w];
        }
      r.pstar[r.b] = bv;
      if (r.kstar) r.kstar[r.b] = (int32_t)bk;
    }
  }
};

constexpr int kOptStep = 4 * kRankThreads;
constexpr int kOptHold = 8;         // steps held in registers: rows of up to 32768 tokens
constexpr int kOptShift = 19;       // word >> kOptShift: 16 bins an octave
constexpr int kOptBins = 4096;      // the last one used, 4080, holds the infinite ratios (q = 0)
constexpr int kOptInfBin = 0x7f800000 >> kOptShift;
constexpr int kOptMaxCand = 128;    // bins taken to the second level (kOptBins / 32 parts)
constexpr int kOptList = 1024;      // tokens ranked at the end, one a thread
constexpr double kOptUnit = 0x1p-61;

struct OptShared {
  unsigned long long P[kOptBins], Q[kOptBins];
  uint8_t slot[kOptBins];           // of a bin in the second level, 0xFF: none
  uint8_t take[kOptBins];           // a part's tokens are ranked
  unsigned long long cP[kOptMaxCand], cQ[kOptMaxCand];  // masses before a candidate bin
  uint32_t cbin[kOptMaxCand];
  unsigned long long key[kOptList], eP[kOptList], eQ[kOptList];
  int part[kOptList];
  unsigned long long wP[kRankWaves], wQ[kRankWaves], wk[kRankWaves];
  double wf[kRankWaves];
  float ws[2][kRankWaves];
  uint32_t wm[kRankWaves];
  int wi[kRankWaves];
  int n;
};

// ranks w ascending; the correctly rounded quotient is the fp64 quotient rounded to fp32
__device__ __forceinline__ uint32_t opt_word(float p, float q) {
  const float w = q > 0.0f ? p / q : __int_as_float(0x7f800000);
  return __float_as_uint(w + 0.0f);
}
// x in [0, 2] in units of 2^-61, rounded to nearest
__device__ __forceinline__ unsigned long long opt_fixed(float x) {
  const float y = x * 0x1p29f;
  const uint32_t hi = (uint32_t)y;
  const uint32_t lo = (uint32_t)rintf((y - (float)hi) * 0x1p32f);  // the rest of a float: below 2^32 - 255
  return (unsigned long long)hi << 32 | lo;
}
__device__ __forceinline__ unsigned long long opt_shfl_up(unsigned long long v, int off) {
  return (unsigned long long)__shfl_up((long long)v, off, 64);
}
// x + its predecessors' over the wave
__device__ __forceinline__ unsigned long long opt_wave_scan(unsigned long long v, int lane) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned long long o = opt_shfl_up(v, off);
    if (lane >= off) v += o;
  }
  return v;
}
// block minimum of v, in every thread
__device__ __forceinline__ double opt_block_min(double v, double* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kRankWaves; ++w) v = fmin(v, red[w]);
  return v;
}

// P* and k* of one row by a workgroup; false, with nothing written, if the row is to be ranked whole.  Bound by
// the reads of p and q and, on chip, by two 64-bit LDS atomics and the division of every token.  kHold: the row
// stays in registers; longer rows are read once per pass.  256 x 32000, K = 2: 73 us and 5 for the launch that
// ranks the rows left over (none here), against 640 for ranking every row whole.
template <bool kHold>
__device__ __forceinline__ bool opt_row(const OptSpec::Args& args, int64_t b, int64_t V, OptShared& sh) {
  const float* pb = args.p + b * V;
  const float* qb = args.q + b * V;
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  float hp[kHold ? kOptHold : 1][4], hq[kHold ? kOptHold : 1][4];
  if (kHold) {
#pragma unroll
    for (int s = 0; s < kOptHold; ++s) {
      const int64_t xw = min((int64_t)s * kOptStep + wid * 256, V);
      row_load4(pb, xw, lane, V, hp[kHold ? s : 0]);
      row_load4(qb, xw, lane, V, hq[kHold ? s : 0]);
    }
  }
  // f(first token of the wave's 256, p's four, q's four); tokens from V on read as 0 and so have q = 0
  const auto each = [&](auto&& f) {
    if (kHold) {
#pragma unroll
      for (int s = 0; s < kOptHold; ++s) {
        const int64_t xw = (int64_t)s * kOptStep + wid * 256;
        if (xw >= V) continue;  // uniform
        float pc[4], qc[4];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // as new values: 32 tokens' ratios kept from pass to pass would spill
          pc[i] = hp[kHold ? s : 0][i];
          qc[i] = hq[kHold ? s : 0][i];
          __asm__ volatile("" : "+v"(pc[i]), "+v"(qc[i]));
        }
        f(xw, pc, qc);
      }
    } else {
      constexpr int kBatch = 4;
      for (int64_t x0 = wid * 256; x0 < V; x0 += kBatch * kOptStep) {
        float pv[kBatch][4], qv[kBatch][4];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
          row_load4(pb, min(x0 + j * kOptStep, V), lane, V, pv[j]);
          row_load4(qb, min(x0 + j * kOptStep, V), lane, V, qv[j]);
        }
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
          if (x0 + j * kOptStep < V) f(x0 + j * kOptStep, pv[j], qv[j]);
      }
    }
  };
  const auto clear = [&]() {
    for (int x = tid; x < kOptBins; x += kRankThreads) sh.P[x] = sh.Q[x] = 0ull;
    __syncthreads();
  };

  // level 1: the masses of every bin; validity and the rough totals
  for (int x = tid; x < kOptBins; x += kRankThreads) {
    sh.slot[x] = 0xFF;
    sh.take[x] = 0;
  }
  if (tid == 0) sh.n = 0;
  clear();
  bool bad = false;
  uint32_t mx = 0u;
  float tp = 0.0f, tq = 0.0f;
  each([&](int64_t, const float (&pv)[4], const float (&qv)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bad |= __builtin_amdgcn_classf(pv[i], 0x21F) | __builtin_amdgcn_classf(qv[i], 0x21F);
      mx = max(mx, max(__float_as_uint(pv[i]) & 0x7FFFFFFFu, __float_as_uint(qv[i]) & 0x7FFFFFFFu));
      tp += pv[i];
      tq += qv[i];
      const uint32_t bin = opt_word(pv[i], qv[i]) >> kOptShift;
      if (qv[i] > 0.0f) {  // (masses of tokens past 2 are not used)
        atomicAdd(&sh.P[bin & (kOptBins - 1)], opt_fixed(pv[i]));
        atomicAdd(&sh.Q[bin & (kOptBins - 1)], opt_fixed(qv[i]));
      }
    }
  });
  bad = __builtin_amdgcn_ballot_w64(bad) != 0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    tp += __shfl_xor(tp, off, 64);
    tq += __shfl_xor(tq, off, 64);
    mx = max(mx, (uint32_t)__shfl_xor((int)mx, off, 64));
  }
  if (lane == 0) {
    sh.wi[wid] = bad ? 1 : 0;
    sh.wm[wid] = mx;
    sh.ws[0][wid] = tp;
    sh.ws[1][wid] = tq;
  }
  __syncthreads();
  int any = 0;
  tp = tq = 0.0f;
#pragma unroll
  for (int w = 0; w < kRankWaves; ++w) {
    any |= sh.wi[w];
    mx = max(mx, sh.wm[w]);
    tp += sh.ws[0][w];
    tq += sh.ws[1][w];
  }
  if (any) {
    OptSpec::flag(OptSpec::row(args, b, V), V, kRowBadProb);
    return true;
  }
  if (mx > 0x40000000u || !(fmaxf(tp, tq) <= 2.0f) || !(fminf(tp, tq) >= 0x1p-6f)) return false;

  // masses before the thread's bins 4 t .. 4 t + 3: over the wave here (sP, sQ in its last lane with them)
  unsigned long long P0, Q0, sP, sQ;
  const auto prefix = [&]() {
    unsigned long long dP = 0ull, dQ = 0ull;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      dP += sh.P[4 * tid + j];
      dQ += sh.Q[4 * tid + j];
    }
    sP = opt_wave_scan(dP, lane);
    sQ = opt_wave_scan(dQ, lane);
    P0 = sP - dP;
    Q0 = sQ - dQ;
  };
  prefix();
  if (lane == 63) {
    sh.wP[wid] = sP;
    sh.wQ[wid] = sQ;
  }
  __syncthreads();
  unsigned long long Qall = 0;
#pragma unroll
  for (int w = 0; w < kRankWaves; ++w) {
    P0 += w < wid ? sh.wP[w] : 0ull;
    Q0 += w < wid ? sh.wQ[w] : 0ull;
    Qall += sh.wQ[w];
  }
  const int K = args.K;
  const double QtK = ipow((double)Qall * kOptUnit, K);
  const auto value = [&](unsigned long long p, unsigned long long q) {
    return (double)p * kOptUnit + QtK - ipow((double)q * kOptUnit, K);
  };
  // Rounding: of the masses (at most 2^-62 a token, 2^23 tokens: 2e-12, times the slope K Q^(K-1)) and of f;
  // the ratios' rounding is in w_lo.
  const double margin = 1e-9 * (1.0 + QtK);
  double best = QtK;  // the smallest f at a bin's end
  // g(bin, masses before it, f at its start, may it hold a minimiser) for the thread's bins of ratios from
  // lo_bits(bin) on; mine: the thread's bins count
  const auto find = [&](bool mine, auto&& lo_bits, auto&& g) {
    unsigned long long p = P0, q = Q0;
#pragma unroll 1
    for (int j = 0; j < 4; ++j) {
      p += sh.P[4 * tid + j];
      q += sh.Q[4 * tid + j];
      if (mine) best = fmin(best, value(p, q));
    }
    best = opt_block_min(best, sh.wf);
    p = P0;
    q = Q0;
    double f0 = value(p, q);
#pragma unroll 1
    for (int j = 0; j < 4; ++j) {
      const int at = 4 * tid + j;
      const unsigned long long dp = sh.P[at], dq = sh.Q[at];
      const double f1 = value(p + dp, q + dq);
      const double lo = (double)__uint_as_float(lo_bits(at)) * (1.0 - 0x1p-22);
      const double at_end = f1 - ((double)dp * kOptUnit - lo * ((double)dq * kOptUnit));
      g(at, p, q, mine && (dp | dq) != 0ull && fmin(f0, at_end) <= best + margin);
      p += dp;
      q += dq;
      f0 = f1;
    }
  };
  find(
      true, [](int bin) { return (uint32_t)bin << kOptShift; },
      [&](int bin, unsigned long long p, unsigned long long q, bool remains) {
        if (!remains || bin >= kOptInfBin) return;
        const int c = atomicAdd(&sh.n, 1);
        if (c < kOptMaxCand) {
          sh.slot[bin] = (uint8_t)c;
          sh.cbin[c] = (uint32_t)bin;
          sh.cP[c] = p;
          sh.cQ[c] = q;
        }
      });
  __syncthreads();
  const int cands = sh.n;
  if (cands > kOptMaxCand) return false;

  // level 2: the candidate bins in 2^lg parts each
  const int lg = cands <= 16 ? 8 : (cands <= 32 ? 7 : (cands <= 64 ? 6 : 5));
  const int low = kOptShift - lg;
  const auto part_of = [&](uint32_t word) {  // -1 outside the candidate bins
    const uint32_t c = sh.slot[(word >> kOptShift) & (kOptBins - 1)];
    return c == 0xFFu ? -1 : (int)(c << lg | ((word >> low) & ((1u << lg) - 1u)));
  };
  clear();  // (its barrier: every thread has read sh.n and the bins)
  if (tid == 0) sh.n = 0;
  each([&](int64_t, const float (&pv)[4], const float (&qv)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int at = part_of(opt_word(pv[i], qv[i]));
      if (at >= 0) {
        atomicAdd(&sh.P[at], opt_fixed(pv[i]));
        atomicAdd(&sh.Q[at], opt_fixed(qv[i]));
      }
    }
  });
  __syncthreads();
  prefix();
  {
    // a candidate's parts lie in one wave: from its first part's masses to the candidate's
    const int first = lane & ~((1 << (lg - 2)) - 1), c = (4 * tid) >> lg;
    const bool mine = c < cands;
    P0 += (mine ? sh.cP[c] : 0ull) - (unsigned long long)__shfl((long long)P0, first, 64);
    Q0 += (mine ? sh.cQ[c] : 0ull) - (unsigned long long)__shfl((long long)Q0, first, 64);
    const uint32_t bin = mine ? sh.cbin[c] : 0u;
    find(
        mine, [&](int at) { return (bin << kOptShift) | ((uint32_t)(at & ((1 << lg) - 1)) << low); },
        [&](int at, unsigned long long p, unsigned long long q, bool remains) {
          sh.P[at] = p;
          sh.Q[at] = q;
          if (remains) sh.take[at] = 1;
        });
  }
  __syncthreads();
  // the tokens of the parts that remain
  each([&](int64_t xw, const float (&pv)[4], const float (&qv)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t word = opt_word(pv[i], qv[i]);
      const int at = part_of(word);
      if (at >= 0 && sh.take[at]) {
        const int e = atomicAdd(&sh.n, 1);
        if (e < kOptList) {
          sh.key[e] = (unsigned long long)word << 32 | (uint32_t)(xw + 4 * lane + i);
          sh.eP[e] = opt_fixed(pv[i]);
          sh.eQ[e] = opt_fixed(qv[i]);
          sh.part[e] = at;
        }
      }
    }
  });
  __syncthreads();
  const int n = sh.n;
  if (n > kOptList) return false;
  double fv = QtK;  // the empty prefix
  unsigned long long fk = 0ull;
  if (tid < n) {
    const unsigned long long key = sh.key[tid];
    const int at = sh.part[tid];
    unsigned long long mp = sh.P[at], mq = sh.Q[at];
    for (int j = 0; j < n; ++j) {
      const bool before = sh.part[j] == at && sh.key[j] <= key;
      mp += before ? sh.eP[j] : 0ull;
      mq += before ? sh.eQ[j] : 0ull;
    }
    const double v = value(mp, mq);
    if (v < fv) {
      fv = v;
      fk = key + 1ull;  // 0: the empty prefix
    }
  }
  const auto better = [](double v, unsigned long long k, double w, unsigned long long l) {
    return v < w || (v == w && k < l);
  };
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const double ov = __shfl_xor(fv, off, 64);
    const unsigned long long ok = (unsigned long long)__shfl_xor((long long)fk, off, 64);
    if (better(ov, ok, fv, fk)) {
      fv = ov;
      fk = ok;
    }
  }
  __syncthreads();  // (sh.wf was last read before the barriers above)
  if (lane == 0) {
    sh.wf[wid] = fv;
    sh.wk[wid] = fk;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kRankWaves; ++w) {
    if (better(sh.wf[w], sh.wk[w], fv, fk)) {
      fv = sh.wf[w];
      fk = sh.wk[w];
    }
  }
  if (tid == 0) args.pstar[b] = fv;
  if (args.kstar == nullptr) return true;
  int k = 0;  // tokens up to the prefix's last
  if (fk != 0ull) {  // uniform
    each([&](int64_t xw, const float (&pv)[4], const float (&qv)[4]) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t x = xw + 4 * lane + i;
        const unsigned long long key = (unsigned long long)opt_word(pv[i], qv[i]) << 32 | (uint32_t)x;
        k += key < fk && x < V ? 1 : 0;
      }
    });
  }
  k = wave_sum_int(k);
  if (lane == 0) sh.wi[wid] = k;
  __syncthreads();
  if (tid == 0) {
    int t = 0;
#pragma unroll
    for (int w = 0; w < kRankWaves; ++w) t += sh.wi[w];
    args.kstar[b] = t;
  }
  return true;
}

// later[b V]: the row is left to rank_scan_kernel.
template <bool kHold>
__global__ __launch_bounds__(kRankThreads) void optimum_kernel(OptSpec::Args args, int64_t V,
                                                               uint32_t* __restrict__ later) {
  __shared__ OptShared sh;
  const bool done = opt_row<kHold>(args, blockIdx.x, V, sh);
  if (threadIdx.x == 0) later[blockIdx.x * V] = done ? 0u : 1u;
}

// sum over the row of min(p, r), fp64, in a fixed order; NaN if the row is bad
constexpr int kAccThreads = 1024;
__global__ __launch_bounds__(kAccThreads) void acceptance_kernel(const float* __restrict__ p,
                                                                 const float* __restrict__ r, int64_t V,
                                                                 double* __restrict__ out,
                                                                 int32_t* __restrict__ row_status) {
  __shared__ double red[kAccThreads / 64];
  __shared__ int bad_w[kAccThreads / 64];
  const int64_t b = blockIdx.x;
  const float* pb = p + b * V;
  const float* rb = r + b * V;
  double acc = 0.0;
  int bad = 0;
  constexpr int kU = 4;
  for (int64_t i0 = threadIdx.x; i0 < V; i0 += kU * kAccThreads) {
    float pv[kU], rv[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int64_t i = i0 + (int64_t)u * kAccThreads;
      pv[u] = i < V ? pb[i] : 0.0f;
      rv[u] = i < V ? rb[i] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      bad |= (bad_prob(pv[u]) || bad_prob(rv[u])) ? 1 : 0;
      acc += fmin((double)pv[u], (double)rv[u]);
    }
  }
  acc = wave_sum(acc);
  bad = __ballot(bad) != 0ull;
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = acc;
    bad_w[threadIdx.x >> 6] = bad;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int any = 0;
    double t = 0.0;
    for (int w = 0; w < kAccThreads / 64; ++w) {
      any |= bad_w[w];
      t += red[w];
    }
    out[b] = any ? __longlong_as_double(0x7ff8000000000000ll) : t;
    if (any && row_status) row_status[b] |= kRowBadProb;
  }
}

}  // namespace

size_t workspace_bytes_optimum(int64_t B, int64_t V) { return rank_workspace_bytes(B, V); }

hipError_t launch_optimum(const float* p, const float* q, int64_t B, int64_t V, int K, double* pstar, int32_t* kstar,
                          int32_t* row_status, void* workspace, hipStream_t st) {
  OptSpec::Args args = {p, q, pstar, kstar, row_status, K};
  const RankPlanes planes = carve_rank_planes(workspace, B, V);
  uint32_t* later = planes.bins.word;  // a row's first word: read before the ranking writes there
  if (V <= kOptHold * kOptStep)
    hipLaunchKernelGGL(optimum_kernel<true>, dim3((unsigned)B), dim3(kRankThreads), 0, st, args, V, later);
  else
    hipLaunchKernelGGL(optimum_kernel<false>, dim3((unsigned)B), dim3(kRankThreads), 0, st, args, V, later);
  hipLaunchKernelGGL(rank_scan_kernel<OptSpec>, dim3((unsigned)B), dim3(kRankThreads), 0, st, args, V, planes, later);
  return hipGetLastError();
}

hipError_t launch_acceptance(const float* p, const float* r, int64_t B, int64_t V, double* out, int32_t* row_status,
                             hipStream_t st) {
  hipLaunchKernelGGL(acceptance_kernel, dim3((unsigned)B), dim3(kAccThreads), 0, st, p, r, V, out, row_status);
  return hipGetLastError();
}

}  // namespace mdss
