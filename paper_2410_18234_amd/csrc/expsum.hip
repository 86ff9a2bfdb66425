// Top-s quadrature: r of K i.i.d. drafts from a truncated draft, taken directly over each row's
// support by the trapezoidal rule at step 1/2 (es_topk_kernel below), the allocation-free call's
// fixed scratch, and the entry points of the quadrature calls (whose form for whole rows is bucket.hip).
//
// Notation: p = target, q = draft, w = p / q.  Every denominator D of the selected-token law is a
// sum of positive weights, and 1 / D = integral over t of exp(t - D e^t) dt, so with
// S(a) = sum_x q(x) exp(-a w(x)) the K-draft law is the integral of exp(t) exp(-e^t w(y))
// S(e^t)^(K-1) dt, times K p(y).  The rule at step h differs from 1 / D by at most
// 2 sum_{m>=1} |Gamma(1 + 2 pi i m / h)| / D, 4.8e-8 for h = 1/2, independently of D.  A row's grid
// is cut where the left tail (t < t_lo: relative D e^t_lo) and the right tail (t > t_hi: relative
// exp(-D e^t_hi)) are below 1e-8 for every denominator of the row.
#include "common.h"
#include "draw.h"
#include "mdss.h"

#include <float.h>
#include <math.h>

#include <algorithm>
#include <mutex>

namespace mdss {

namespace {

constexpr int kEsMaxNodes = 480;                        // nodes of a row (weights spanning <= 2^300)
constexpr double kEsStep = 0.5;                         // h
constexpr double kEsLnEps = -18.420680743952367;        // ln 1e-8: left-tail cut
constexpr double kEsLnLnInvEps = 2.9134941423228814;    // ln ln 1e8: right-tail cut
constexpr double kEsLog2e = 1.4426950408889634;

// A row's plan.
struct EsPlan {
  int32_t flags;  // row status bits; a flagged row gets r = NaN
  int32_t k_lo;   // first node of the row's grid
  int32_t nk;     // nodes of the row's grid (0: no quadrature term)
};

__device__ __forceinline__ double wave_min64(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ double wave_max64(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

__device__ inline void es_scale_f32(float wlo, float whi, int& tau, int& range) {
  int e_lo, e_hi;
  frexpf(wlo, &e_lo);
  frexpf(whi, &e_hi);
  tau = -((e_lo + e_hi) >> 1);
  range = e_hi - e_lo;
}

__device__ __forceinline__ float es_decay(float beta, float w) { return __builtin_amdgcn_exp2f(-beta * w); }
template <typename Real>
__device__ __forceinline__ Real es_ratio(float p, float q);
template <>
__device__ __forceinline__ float es_ratio<float>(float p, float q) {
  // reciprocal and product: within 2 ulp of p / q, the same value in every kernel
  return p * __builtin_amdgcn_rcpf(q);
}
// The same ratio for a draft probability below the fp32 normal range, whose
// reciprocal would overflow: q is scaled up by 2^64 first (p / q itself is
// often far inside the range: a draft at a low temperature puts its tail there).
// The kernels take it only in waves that hold such a q (a uniform branch).
__device__ __forceinline__ float es_ratio_small_q(float p, float q) {
  return (p * __builtin_amdgcn_rcpf(q * 0x1p64f)) * 0x1p64f;
}
// positive fp32 denormal (class bit 7; bits 0-9: signalling NaN, quiet NaN, -inf, -normal,
// -denormal, -0, +0, +denormal, +normal, +inf)
__device__ __forceinline__ bool es_denormal(float q) { return __builtin_amdgcn_classf(q, 0x80); }
template <>
__device__ __forceinline__ double es_ratio<double>(float p, float q) {
  return (double)p / (double)q;
}

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

// Sum of 16 per-lane values over the wave, scattered, in a fixed order and without LDS traffic.
// Values are split by lane bit 2 and bit 3 within 16-lane rows through DPP rotations (a rotation
// by 4 or 8 always flips that bit and keeps the others below bit 4, so every lane is paired
// once), by bits 4 and 5 through the row and half swaps of gfx950; the two bits left over are summed
// (quad permutations).  Lane l ends with the total of value 8 b2 + 4 b3 + 2 b4 + b5 (b_i = bit i
// of l); es_scatter_node and es_scatter_writer name that value and one lane holding it.
constexpr int kEsBlock = 16;
template <int HALF, int N, int CTRL>
__device__ __forceinline__ void rs_dpp(float (&v)[N], bool up) {
#pragma unroll
  for (int i = 0; i < HALF; ++i) {
    const float send = up ? v[i] : v[i + HALF];
    const float keep = up ? v[i + HALF] : v[i];
    v[i] = keep + dpp<CTRL>(send);
  }
}
template <int HALF, int N, bool ROW>
__device__ __forceinline__ void rs_swap(float (&v)[N]) {
#pragma unroll
  for (int i = 0; i < HALF; ++i) {
    const auto r = ROW ? __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + HALF]), false, false)
                       : __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + HALF]), false, false);
    v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
}
__device__ __forceinline__ float wave_reduce_scatter_f32(float (&v)[kEsBlock], int lane) {
  rs_dpp<8, kEsBlock, 0x124>(v, (lane & 4) != 0);  // row_ror:4
  rs_dpp<4, kEsBlock, 0x128>(v, (lane & 8) != 0);  // row_ror:8
  rs_swap<2, kEsBlock, true>(v);
  rs_swap<1, kEsBlock, false>(v);
  float x = v[0];
  x += dpp<0xB1>(x);  // quad_perm [1,0,3,2]
  x += dpp<0x4E>(x);  // quad_perm [2,3,0,1]
  return x;
}
__device__ __forceinline__ int es_scatter_node(int lane) {
  const int b2 = (lane >> 2) & 1, b3 = (lane >> 3) & 1, b4 = (lane >> 4) & 1, b5 = (lane >> 5) & 1;
  return 8 * b2 + 4 * b3 + 2 * b4 + b5;
}
__device__ __forceinline__ bool es_scatter_writer(int lane) { return (lane & 3) == 0; }

// Minimum / maximum of a float over the 64 lanes of a wave, in every lane
// (quad permutations, row rotations by 4 and 8, then the gfx950 row and half
// swaps; all lanes must be active).
template <bool MAX>
__device__ __forceinline__ float es_pick(float a, float b) {
  return MAX ? fmaxf(a, b) : fminf(a, b);
}
template <bool MAX>
__device__ __forceinline__ float es_wave_ext(float x) {
  x = es_pick<MAX>(x, dpp<0xB1>(x));   // quad_perm [1,0,3,2]
  x = es_pick<MAX>(x, dpp<0x4E>(x));   // quad_perm [2,3,0,1]
  x = es_pick<MAX>(x, dpp<0x124>(x));  // row_ror:4
  x = es_pick<MAX>(x, dpp<0x128>(x));  // row_ror:8
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = es_pick<MAX>(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return es_pick<MAX>(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// Node rates of rows taken in fp32: log2(e) a_k = log2(e) e^(k/2) as an fp32 mantissa
// in [1, 2) and a binary exponent, for every node such a row may have (a row whose grid leaves
// the table is taken in fp64).  Built at compile time: e^(1/2) from its series, then
// successive products and quotients (relative error below 1e-13 over the range), rounded once
// to fp32.
constexpr int kEsNodeLo = -192, kEsNodeHi = 192;
struct EsRateTab {
  float mant[kEsNodeHi - kEsNodeLo];
  int expo[kEsNodeHi - kEsNodeLo];
};
constexpr EsRateTab es_make_rate_tab() {
  EsRateTab t{};
  double eh = 1.0, term = 1.0;
  for (int i = 1; i < 24; ++i) {
    term *= 0.5 / i;
    eh += term;
  }
  for (int dir = 0; dir < 2; ++dir) {
    double v = kEsLog2e;
    for (int k = 0; dir == 0 ? k < kEsNodeHi : k >= kEsNodeLo; k += dir == 0 ? 1 : -1) {
      double x = v;
      int n = 0;
      while (x >= 2.0) {
        x *= 0.5;
        ++n;
      }
      while (x < 1.0) {
        x *= 2.0;
        --n;
      }
      t.mant[k - kEsNodeLo] = (float)x;
      t.expo[k - kEsNodeLo] = n;
      v = dir == 0 ? v * eh : v / eh;
    }
  }
  return t;
}
__constant__ EsRateTab kEsRates = es_make_rate_tab();

// log2(e) a_k 2^-tau in fp32: an integer add to the exponent field (normal: the row's weights span at most
// 2^kTkMaxRange and tau centres them).
__device__ __forceinline__ float es_rate_f32(int k, int tau) {
  const int i = min(max(k - kEsNodeLo, 0), kEsNodeHi - kEsNodeLo - 1);
  return __int_as_float(__float_as_int(kEsRates.mant[i]) + ((kEsRates.expo[i] - tau) << 23));
}

// Workgroup barrier that orders LDS only: global loads issued before it stay in flight.
__device__ __forceinline__ void es_lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// kEsBlock nodes of E entries a lane: sums of q exp(-a_k w), added to the wave's sums (nodes at or above lim are not
// written).
template <int E>
__device__ __forceinline__ void es_run_block(const float (&w)[E], const float (&qq)[E], const float* __restrict__ rate,
                                             int lane, float* __restrict__ red, int lim) {
  float rt[kEsBlock], acc[kEsBlock];
#pragma unroll
  for (int i = 0; i < kEsBlock; ++i) {
    rt[i] = rate[i];
    acc[i] = 0.0f;
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
#pragma unroll
    for (int i = 0; i < kEsBlock; ++i) acc[i] = fmaf(qq[e], es_decay(rt[i], w[e]), acc[i]);
  }
  const float tot = wave_reduce_scatter_f32(acc, lane);
  const int node = es_scatter_node(lane);
  if (es_scatter_writer(lane) && node < lim) red[node] += tot;
}

// The row's plan from its statistics: the grid's node range (the left-tail and right-tail cuts of
// the quadrature), or MDSS_ROW_RANGE.
__device__ EsPlan es_make_plan(double wmin, double wmax, double q0, int npos, int K) {
  EsPlan pl = {0, 0, 0};
  if (npos > 0) {
    // K = 2 takes the zero-weight tokens in closed form; K >= 3 keeps them in S (denominator w(y) alone)
    const double dmin = (K == 2 || q0 == 0.0) ? K * wmin : wmin, dmax = K * wmax;
    pl.k_lo = (int)floor((kEsLnEps - log(dmax)) / kEsStep);
    pl.nk = (int)ceil((kEsLnLnInvEps - log(dmin)) / kEsStep) - pl.k_lo + 1;
    if (pl.nk > kEsMaxNodes) {  // only rows with probabilities far above 1 get here
      pl.flags = kRowRange;
      pl.nk = 0;
    }
  }
  return pl;
}

}  // namespace

// Per row and law about 74 kB and 4 kB per 4096 tokens: the plan, the chunks' sums and the parts'
// polynomials of bucket.hip (which takes as many chunks as fit), and the size callers already hold
// buffers of and the allocation-free call accepts.
size_t workspace_bytes_expsum(int64_t B, int64_t V, int L) {
  const auto align256 = [](size_t x) { return (x + 255) / 256 * 256; };
  const size_t T1 = (size_t)((V + 4095) / 4096), rows = (size_t)B * L;
  return align256(64 * rows * T1) + align256(4032 * rows * T1) + align256(128 * (size_t)B) + align256(30720 * rows) +
         align256(43648 * rows);
}

// q2 == nullptr: K i.i.d. drafts from q1; else two draft laws (K = 2).
hipError_t launch_induced_expsum(const float* p, const float* q1, const float* q2, int64_t B, int64_t V, int K,
                                 float* r, int32_t* row_status, void* workspace, hipStream_t st, double* rsum) {
  return launch_bucket(p, q1, q2, B, V, K, 0, true, r, row_status, rsum != nullptr, rsum, workspace,
                       workspace_bytes_expsum(B, V, q2 ? 2 : 1), st);
}

// Successive pairwise reduction (Remark 4) with every stage law by the quadrature.
hipError_t launch_induced_successive_expsum(const float* p, const float* q, int64_t B, int64_t V, int K,
                                            float* r_stages, int32_t* row_status, void* workspace, hipStream_t st) {
  hipError_t e = launch_induced_expsum(p, q, nullptr, B, V, 2, r_stages, row_status, workspace, st);
  const int64_t plane = B * V;
  for (int j = 1; j < K - 1 && e == hipSuccess; ++j)
    e = launch_induced_expsum(p, r_stages + (j - 1) * plane, q, B, V, 2, r_stages + j * plane, row_status,
                              workspace, st);
  return e;
}

// ------------------------------------------------------------------ top-s rows
// K i.i.d. drafts from a draft truncated to at most s_max tokens (a top-s draft):
// one workgroup of 1024 threads per row streams p and q once (twice when one wave
// meets more than kTkSeg support tokens), writes r = 0 (the support's entries are
// written again at the end), keeps the support (index, p, q, w) in LDS and takes the
// trapezoidal rule directly over it:
//   S_k = sum over the support of q(x) exp(-a_k w(x))      (p(x) > 0),
//   r(y) = p(y) sum_k c_k exp(-a_k w(y)),  c_k = K h a_k (S_k [+ Q0 for K >= 3])^(K-1),
// every (node, token) term exactly (no windows, expansions or polynomial tables),
// plus the zero-weight closed forms.  fp32 terms with a power-of-two
// scale (w' = w 2^tau, rates a_k 2^-tau), fp64 sums of the per-lane partials; a
// row whose weights leave the fp32 normal range, span more than 2^kTkMaxRange or
// need nodes outside the rate table is taken in fp64.
namespace {

constexpr int kTkThreads = 1024;
constexpr int kTkWaves = kTkThreads / 64;
constexpr int kTkCap = MDSS_K3_MAX_SUPPORT;   // support entries held in LDS
constexpr int kTkPer = 4;                     // tokens per thread per streaming step
constexpr int kTkStep = kTkThreads * kTkPer;  // 4096 tokens per step
constexpr int kTkSeg = kTkCap / kTkWaves;     // support tokens of one wave's stream segment
constexpr int kTkLdsParts = 1024;             // residual parts kept in LDS: rows of up to 262144 tokens
constexpr int kTkAhead = 2;                   // streaming steps in flight (64 KB of p and q per workgroup)
constexpr int kTkE = 4;                       // support entries per lane in the node sums
constexpr int kTkGroup = 64 * kTkE;           // entries of one wave group
constexpr int kTkMaxRange = 100;              // binary exponent span of the weights kept in fp32
static_assert(kTkCap % kTkGroup == 0 && kTkCap / kTkGroup <= kTkWaves, "groups of 256 entries, one a wave at most");
static_assert(kTkPer * kTkWaves == 64, "one (slot, wave) count per lane");

// Inclusive scan of an int over the wave: row_shr steps inside each 16-lane row (DPP,
// lanes before a row's start read 0), then the row totals carried by readlane.
__device__ __forceinline__ int tk_scan_int(int v, int lane) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);  // row_shr:8
  const int t0 = __builtin_amdgcn_readlane(v, 15), t1 = __builtin_amdgcn_readlane(v, 31),
            t2 = __builtin_amdgcn_readlane(v, 47);
  const int row = lane >> 4;
  return v + (row == 0 ? 0 : (row == 1 ? t0 : (row == 2 ? t0 + t1 : t0 + t1 + t2)));
}

// A streaming step's p and q, thread t holding the four consecutive tokens x0 + 4t ..
// x0 + 4t + 3 (one 16-byte load each); 0 past the row.
__device__ __forceinline__ void tk_load4(const float* __restrict__ pb, const float* __restrict__ qb, int64_t V,
                                         int64_t x0, int tid, float (&pv)[kTkPer], float (&qv)[kTkPer]) {
  static_assert(kTkPer == 4, "one float4 a thread and step");
  const int64_t x = x0 + 4 * tid;
  if (x + 3 < V) {
    const f32x4u a = *reinterpret_cast<const f32x4u*>(pb + x), c = *reinterpret_cast<const f32x4u*>(qb + x);
    pv[0] = a.x; pv[1] = a.y; pv[2] = a.z; pv[3] = a.w;
    qv[0] = c.x; qv[1] = c.y; qv[2] = c.z; qv[3] = c.w;
  } else {
#pragma unroll
    for (int i = 0; i < kTkPer; ++i) {
      pv[i] = (x + i < V) ? pb[x + i] : 0.0f;
      qv[i] = (x + i < V) ? qb[x + i] : 0.0f;
    }
  }
}

// The token-order pass's step: thread t holding tokens x0 + 1024 i + t (0 past the row's
// end); a whole step without bounds checks.
__device__ __forceinline__ void tk_load(const float* __restrict__ pb, const float* __restrict__ qb, int64_t V,
                                        int64_t x0, int tid, float (&pv)[kTkPer], float (&qv)[kTkPer]) {
  const float* ps = pb + x0 + tid;
  const float* qs = qb + x0 + tid;
  if (x0 + kTkStep <= V) {  // uniform
#pragma unroll
    for (int i = 0; i < kTkPer; ++i) {
      pv[i] = ps[i * kTkThreads];
      qv[i] = qs[i * kTkThreads];
    }
  } else {
    const int rest = (int)(V - x0) - tid;
#pragma unroll
    for (int i = 0; i < kTkPer; ++i) {
      pv[i] = (i * kTkThreads < rest) ? ps[i * kTkThreads] : 0.0f;
      qv[i] = (i * kTkThreads < rest) ? qs[i * kTkThreads] : 0.0f;
    }
  }
}

// kRes: also the residual sums of Algorithm 1 with proposal r (the summed form), one fp64
// sum per 256-token part (rsum[b][part], four parts per 1024-token sub-tile): while the
// row streams, each wave writes the sum of p over its part; once r is written, each
// support token's correction max(0, p - r) - p is added to its part's sum.  row_status is
// set, not OR-ed into.
// kDraw (with kRes): the step in one launch; once r and the sums are complete, wave 0
// takes the row's selection and Algorithm 1 from them (draw_from_sums, the code of
// the summed form's draw), with the drafts, uniforms and outputs of dr.
struct TkDraw {
  const float* u;
  uint64_t seed, offset;
  SelArgs sel;
  int32_t* out_token;
  uint8_t* accepted;
  double* residual_mass;
};
template <bool kRes, bool kDraw>
__global__ __launch_bounds__(kTkThreads) void es_topk_kernel(const float* __restrict__ p, const float* __restrict__ q,
                                                             int64_t V, int K, int s_max, float* __restrict__ r,
                                                             int32_t* __restrict__ row_status,
                                                             double* __restrict__ rsum, int64_t nsub, TkDraw dr) {
  static_assert(kTkStep == 4 * kResSub && kResSub / kResParts == 256 && kTkThreads / 4 == 256,
                "a wave's 256 tokens of a step are one part of the residual sums");
  static_assert(kRes || !kDraw, "the fused draw takes the residual sums");
  __shared__ int s_idx[kTkCap];
  __shared__ float s_p[kTkCap];
  __shared__ float s_q[kTkCap];
  __shared__ float s_w[kTkCap];                    // the weight (unscaled, then w 2^tau in fp32)
  __shared__ float s_part[kTkWaves][kEsMaxNodes];  // per wave: its entries' share of S_k at its nodes
  __shared__ float s_rate[kEsMaxNodes + 16];       // fp32: log2(e) a_k 2^-tau (16 spare entries: 0)
  __shared__ float s_cf[kEsMaxNodes + 16];         // fp32: c_k 2^-tau (0 on the spare entries)
  __shared__ double s_c64[kEsMaxNodes];            // fp64: c_k
  __shared__ int s_cnt[2][64];
  __shared__ int s_flag[kTkWaves];
  __shared__ float s_f[kTkWaves][2];
  __shared__ double s_d[kTkWaves];
  __shared__ double s_e[kTkWaves][2];
  __shared__ int s_n[kTkWaves];
  __shared__ EsPlan s_plan;
  // while streaming: wave w's support tokens (index, p, q) at [w kTkSeg, (w + 1) kTkSeg);
  // once the list is joined, kRes keeps each entry's residual correction here (fp64)
  __shared__ __align__(16) uint32_t s_seg[3 * kTkCap];
  int* const s_sidx = reinterpret_cast<int*>(s_seg);
  float* const s_sp = reinterpret_cast<float*>(s_seg + kTkCap);
  float* const s_sq = reinterpret_cast<float*>(s_seg + 2 * kTkCap);
  double* const s_dres = reinterpret_cast<double*>(s_seg);
  __shared__ int s_wn[kTkWaves];
  // kRes: the parts' sums of a row of up to kTkLdsParts parts are kept here and written
  // out once at the end; longer rows keep them in rsum itself
  __shared__ double s_parts[kRes ? kTkLdsParts : 1];
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t b = blockIdx.x;
  const float* pb = p + b * V;
  const float* qb = q + b * V;
  float* rb = r + b * V;
  if (kRes && tid == 0 && row_status) row_status[b] = 0;  // thread 0 adds the flags below
  const int64_t nparts = nsub * kResParts;
  const bool lds_parts = kRes && nparts <= kTkLdsParts;  // uniform
  double* const parts = lds_parts ? s_parts : rsum + b * nparts;
  // the fused draw, by wave 0 once every thread's r and sums are written (after a barrier)
  const auto draw = [&](const double* sb) {
    if (wid != 0) return;
    draw_from_sums<true, kResParts, kResSub>(pb, rb, sb, nsub, nullptr, dr.u, dr.seed, dr.offset, b, V, lane, dr.out_token,
                                             dr.accepted, dr.residual_mass, row_status, dr.sel);
  };

  // (1) stream the row, kTkAhead steps in flight, thread t on the four consecutive tokens
  //     x0 + 4t .. x0 + 4t + 3 of each step (wave w on the 256 tokens x0 + 256w ..): r = 0,
  //     the probability checks, each wave's support tokens appended to its own LDS segment
  //     (no barrier a step), and for kRes each wave's fp64 sum of p over its 256 tokens:
  //     part (x0 >> 8) + w of the residual sums' layout
  float pf[kTkAhead][kTkPer], qf[kTkAhead][kTkPer];  // the next kTkAhead steps, in flight
#pragma unroll
  for (int j = 0; j < kTkAhead; ++j) tk_load4(pb, qb, V, (int64_t)j * kTkStep, tid, pf[j], qf[j]);
  int bad = 0, wn = 0;  // wn: this wave's support tokens so far (uniform)
  const int64_t nstep = (V + kTkStep - 1) / kTkStep;
  for (int64_t st = 0; st < nstep; ++st) {
    const int64_t x0 = st * kTkStep;
    float pc[kTkPer], qc[kTkPer];
#pragma unroll
    for (int i = 0; i < kTkPer; ++i) {
      pc[i] = pf[0][i];
      qc[i] = qf[0][i];
#pragma unroll
      for (int j = 0; j + 1 < kTkAhead; ++j) {
        pf[j][i] = pf[j + 1][i];
        qf[j][i] = qf[j + 1][i];
      }
    }
    if (st + kTkAhead < nstep)
      tk_load4(pb, qb, V, x0 + kTkAhead * kTkStep, tid, pf[kTkAhead - 1], qf[kTkAhead - 1]);
    const int64_t x = x0 + 4 * tid;
    // r = 0 over the whole step in full lines (a masked store would leave partial lines);
    // the support's values overwrite these after the sums, past workgroup barriers
    if (x + 3 < V) {
      const f32x4u zero = {0.0f, 0.0f, 0.0f, 0.0f};
      *reinterpret_cast<f32x4u*>(rb + x) = zero;
    } else {
#pragma unroll
      for (int i = 0; i < kTkPer; ++i)
        if (x + i < V) rb[x + i] = 0.0f;
    }
    if (kRes) {
      double loc = 0.0;
#pragma unroll
      for (int i = 0; i < kTkPer; ++i) loc += (double)pc[i];  // p = 0 past the row's end
      const double tot = wave_sum_dpp(loc);
      const int64_t part = (x0 >> 8) + wid;
      if (lane == 0 && part < nparts) parts[part] = tot;
    }
#pragma unroll
    for (int i = 0; i < kTkPer; ++i) {
      // NaN, -inf, a negative normal or denormal, +inf (-0 is a zero probability)
      bad |= __builtin_amdgcn_classf(pc[i], 0x21F) | __builtin_amdgcn_classf(qc[i], 0x21F);
      const bool sup = qc[i] > 0.0f;  // 0 past the row's end
      const uint64_t mask = __builtin_amdgcn_ballot_w64(sup);
      const int pos = wn + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
      if (sup && pos < kTkSeg) {
        const int at = wid * kTkSeg + pos;
        s_sidx[at] = (int)x + i;  // rows < 2^31 tokens
        s_sp[at] = pc[i];
        s_sq[at] = qc[i];
      }
      wn += (int)__builtin_popcountll(mask);
    }
  }
  const bool wave_bad = __builtin_amdgcn_ballot_w64(bad != 0) != 0;  // every lane votes
  if (lane == 0) {
    s_flag[wid] = wave_bad ? 1 : 0;
    s_wn[wid] = wn;
  }
  __syncthreads();  // the segments are complete (and a flagged row's NaN below follows its zeros)
  int flags = 0, n = 0, wmax_n = 0, base = 0;
#pragma unroll
  for (int i = 0; i < kTkWaves; ++i) {
    flags |= s_flag[i];
    base += (i < wid) ? s_wn[i] : 0;
    n += s_wn[i];
    wmax_n = max(wmax_n, s_wn[i]);
  }
  flags = flags ? kRowBadProb : (n > s_max ? kRowSupport : 0);
  if (!flags) {  // uniform; here n <= s_max <= kTkCap
    if (wmax_n <= kTkSeg) {
      // (1b) the list: the segments in wave order (each in its tokens' stream order)
      for (int j = lane; j < wn; j += 64) {
        s_idx[base + j] = s_sidx[wid * kTkSeg + j];
        s_p[base + j] = s_sp[wid * kTkSeg + j];
        s_q[base + j] = s_sq[wid * kTkSeg + j];
      }
    } else {
      // (1c) a wave met more than kTkSeg support tokens: the row once more, its support
      //      compacted in token order (token x0 + 1024 i + thread; counts per (slot i,
      //      wave), one scan a step)
#pragma unroll
      for (int j = 0; j < kTkAhead; ++j) tk_load(pb, qb, V, (int64_t)j * kTkStep, tid, pf[j], qf[j]);
      int running = 0;
      for (int64_t st = 0; st < nstep; ++st) {
        const int par = (int)(st & 1);
        const int64_t x0 = st * kTkStep;
        float pc[kTkPer], qc[kTkPer];
#pragma unroll
        for (int i = 0; i < kTkPer; ++i) {
          pc[i] = pf[0][i];
          qc[i] = qf[0][i];
#pragma unroll
          for (int j = 0; j + 1 < kTkAhead; ++j) {
            pf[j][i] = pf[j + 1][i];
            qf[j][i] = qf[j + 1][i];
          }
        }
        if (st + kTkAhead < nstep)
          tk_load(pb, qb, V, x0 + kTkAhead * kTkStep, tid, pf[kTkAhead - 1], qf[kTkAhead - 1]);
        uint64_t mask[kTkPer];
#pragma unroll
        for (int i = 0; i < kTkPer; ++i) {
          mask[i] = __builtin_amdgcn_ballot_w64(qc[i] > 0.0f);
          if (lane == 0) s_cnt[par][i * kTkWaves + wid] = (int)__builtin_popcountll(mask[i]);
        }
        es_lds_barrier();  // (s_cnt by step parity: a step's counts are read before the next barrier)
        const int c = s_cnt[par][lane];
        const int incl = tk_scan_int(c, lane);
        const int ex = incl - c;
        const int xs = (int)x0 + tid;
#pragma unroll
        for (int i = 0; i < kTkPer; ++i) {
          const int pos = running + __builtin_amdgcn_readlane(ex, i * kTkWaves + wid) +
                          (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask[i] >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)mask[i], 0u));
          if (qc[i] > 0.0f && pos < kTkCap) {
            s_idx[pos] = xs + i * kTkThreads;
            s_p[pos] = pc[i];
            s_q[pos] = qc[i];
          }
        }
        running += __builtin_amdgcn_readlane(incl, 63);  // the same in every wave
      }
    }
  }
  __syncthreads();  // the list is complete
  const int nl = min(n, kTkCap);  // entries in LDS (n itself when the row is not flagged)

  // (2) weights and the row's statistics (entry e = thread + 1024 j)
  float wlo = INFINITY, whi = 0.0f;
  double q0 = 0.0;
  int npos = 0;
  for (int e = tid; e < nl; e += kTkThreads) {
    const float pp = s_p[e], qq = s_q[e];
    float w = 0.0f;
    if (pp > 0.0f) {
      w = es_denormal(qq) ? es_ratio_small_q(pp, qq) : es_ratio<float>(pp, qq);
      wlo = fminf(wlo, w);
      whi = fmaxf(whi, w);
      ++npos;
    } else {
      q0 += (double)qq;
    }
    s_w[e] = w;
  }
  wlo = es_wave_ext<false>(wlo);
  whi = es_wave_ext<true>(whi);
  q0 = wave_sum(q0);
  npos = wave_sum_int(npos);
  if (lane == 0) {
    s_f[wid][0] = wlo;
    s_f[wid][1] = whi;
    s_d[wid] = q0;
    s_n[wid] = npos;
  }
  __syncthreads();
  float wmin = s_f[0][0], wmax = s_f[0][1];
  q0 = s_d[0];
  npos = s_n[0];
#pragma unroll
  for (int i = 1; i < kTkWaves; ++i) {
    wmin = fminf(wmin, s_f[i][0]);
    wmax = fmaxf(wmax, s_f[i][1]);
    q0 += s_d[i];
    npos += s_n[i];
  }
  // weights outside the fp32 normal range (a ratio that overflowed or a denormal one):
  // the row's range again in fp64, and the fp64 form below
  const bool wide = !flags && npos > 0 && (!(wmin >= __FLT_MIN__) || !(wmax <= __FLT_MAX__));
  double wmin64 = (double)wmin, wmax64 = (double)wmax;
  if (wide) {  // uniform
    double lo = INFINITY, hi = 0.0;
    for (int e = tid; e < nl; e += kTkThreads) {
      const float pp = s_p[e], qq = s_q[e];
      if (pp > 0.0f) {
        const double w = es_ratio<double>(pp, qq);
        lo = fmin(lo, w);
        hi = fmax(hi, w);
      }
    }
    lo = wave_min64(lo);
    hi = wave_max64(hi);
    if (lane == 0) {
      s_e[wid][0] = lo;
      s_e[wid][1] = hi;
    }
    __syncthreads();
    wmin64 = s_e[0][0];
    wmax64 = s_e[0][1];
#pragma unroll
    for (int i = 1; i < kTkWaves; ++i) {
      wmin64 = fmin(wmin64, s_e[i][0]);
      wmax64 = fmax(wmax64, s_e[i][1]);
    }
  }
  // the row's grid, by wave 0 alone: its
  // fp64 logarithms in every one of the sixteen waves would cost each SIMD four times over
  if (wid == 0) {
    const EsPlan pw = es_make_plan(wmin64, wmax64, q0, npos, K);
    if (lane == 0) s_plan = pw;
  }
  __syncthreads();
  const EsPlan pl = s_plan;
  if (!flags) flags = pl.flags;
  if (flags) {  // NaN over the whole row
    if (tid == 0 && row_status) row_status[b] |= flags;
    for (int64_t x = tid; x < V; x += kTkThreads) rb[x] = NAN;
    if (kRes)
      for (int64_t t = tid; t < nparts; t += kTkThreads) rsum[b * nparts + t] = NAN;
  } else {
    const int k_lo = pl.k_lo, nk = pl.nk;
    // fp32 unless a weight is not an fp32 normal (an overflowed or denormal ratio), the
    // weights span more than 2^kTkMaxRange, or a node lies outside the rate table
    bool fp64 = wide;
    int tau = 0, range = 0;
    if (nk > 0 && !fp64) {
      es_scale_f32(wmin, wmax, tau, range);
      fp64 = range > kTkMaxRange || k_lo < kEsNodeLo || k_lo + nk > kEsNodeHi;
    }
    double zw = q0;  // K i.i.d. drafts: Q0^(K-1)
    for (int j = 2; j < K; ++j) zw *= q0;
    if (nk > 0 && !fp64) {
      // (3) fp32: S_k.  Entries in groups of 256 (four a lane); with G groups (a power of
      //     two), wave w takes group w % G and the node blocks of 16 congruent to w / G
      //     modulo 16 / G; each block summed across the wave (reduce-scatter)
      for (int e = tid; e < nl; e += kTkThreads) s_w[e] = ldexpf(s_w[e], tau);
      for (int k = tid; k < nk + 16; k += kTkThreads)  // past the grid: rate 0 (a term of 1, times c = 0)
        s_rate[k] = k < nk ? es_rate_f32(k_lo + k, tau) : 0.0f;
      for (int k = lane; k < nk; k += 64) s_part[wid][k] = 0.0f;
      __syncthreads();
      int G = 1;
      while (G * kTkGroup < nl) G *= 2;  // <= kTkWaves
      const int gi = wid % G, bs = kTkWaves / G;
      float w[kTkE], qq[kTkE];
  #pragma unroll
      for (int e = 0; e < kTkE; ++e) {
        const int x = gi * kTkGroup + e * 64 + lane;  // < kTkCap
        const bool in = x < nl && s_p[x] > 0.0f;
        w[e] = in ? s_w[x] : 0.0f;
        qq[e] = in ? s_q[x] : 0.0f;
      }
      for (int blk = wid / G; blk * 16 < nk; blk += bs)
        es_run_block(w, qq, s_rate + blk * 16, lane, s_part[wid] + blk * 16, min(16, nk - blk * 16));
      __syncthreads();
      // (4) c_k 2^-tau from the fp64 sum of the waves' shares (a wave adds 0 at nodes it does not take)
      for (int k = tid; k < nk; k += kTkThreads) {
        double S = 0.0;
  #pragma unroll
        for (int i = 0; i < kTkWaves; ++i) S += (double)s_part[i][k];  // 0 from the waves that did not take node k
        const double sm = S + (K >= 3 ? q0 : 0.0);
        double sp = 1.0;
        for (int j = 1; j < K; ++j) sp *= sm;
        s_cf[k] = (float)ldexp((double)K * kEsStep * exp((double)(k_lo + k) * kEsStep) * sp, -tau);
      }
      for (int k = nk + tid; k < nk + 16; k += kTkThreads) s_cf[k] = 0.0f;
      __syncthreads();
      // (5) r at the support: every node, blocks of 16 in fp32, the blocks summed in fp64
      for (int e = tid; e < nl; e += kTkThreads) {
        const float pp = s_p[e], qq1 = s_q[e];
        double v;
        if (pp > 0.0f) {
          const float we = s_w[e];
          double acc = 0.0;
          for (int k0 = 0; k0 < nk; k0 += 16) {
            float a = 0.0f;
  #pragma unroll
            for (int i = 0; i < 16; ++i) a = fmaf(s_cf[k0 + i], es_decay(s_rate[k0 + i], we), a);
            acc += (double)a;
          }
          const double quad = ldexp((double)pp * acc, tau);
          v = (K == 2) ? fma(2.0 * (double)qq1, q0, quad) : quad;
        } else {
          v = (double)qq1 * zw;
        }
        rb[s_idx[e]] = (float)v;
        if (kRes) s_dres[e] = residual_of(pp, (float)v) - (double)pp;
      }
    } else if (nk > 0) {
      // (3') fp64: S_k per node (wave w takes the nodes congruent to w), lanes over the entries
      for (int kk = wid; kk < nk; kk += kTkWaves) {
        const double a = exp((double)(k_lo + kk) * kEsStep);
        double acc = 0.0;
        for (int e = lane; e < nl; e += 64) {
          const float pp = s_p[e], qq1 = s_q[e];
          if (pp > 0.0f) acc += (double)qq1 * exp(-a * es_ratio<double>(pp, qq1));
        }
        acc = wave_sum(acc);
        if (lane == 0) {
          const double sm = acc + (K >= 3 ? q0 : 0.0);
          double sp = 1.0;
          for (int j = 1; j < K; ++j) sp *= sm;
          s_c64[kk] = (double)K * kEsStep * a * sp;
        }
      }
      __syncthreads();
      for (int e = tid; e < nl; e += kTkThreads) {
        const float pp = s_p[e], qq1 = s_q[e];
        double v;
        if (pp > 0.0f) {
          const double w = es_ratio<double>(pp, qq1);
          double acc = 0.0;
          for (int kk = 0; kk < nk; ++kk) acc += s_c64[kk] * exp(-exp((double)(k_lo + kk) * kEsStep) * w);
          const double quad = (double)pp * acc;
          v = (K == 2) ? fma(2.0 * (double)qq1, q0, quad) : quad;
        } else {
          v = (double)qq1 * zw;
        }
        rb[s_idx[e]] = (float)v;
        if (kRes) s_dres[e] = residual_of(pp, (float)v) - (double)pp;
      }
    } else {
      // no positive weight: zero-weight tokens only
      for (int e = tid; e < nl; e += kTkThreads) {
        const float v = (float)((double)s_q[e] * zw);
        rb[s_idx[e]] = v;
        if (kRes) s_dres[e] = residual_of(s_p[e], v) - (double)s_p[e];
      }
    }
    if (kRes) {
      // (6) the residual sums: the support entries of one 256-token part are consecutive in
      //     the list (a wave's segment holds its parts in stream order; the token-order list
      //     is sorted); the first entry of each run adds the run's corrections, in list order,
      //     to its part's sum of p
      __syncthreads();  // every correction is in LDS, every part's sum of p written
      for (int e = tid; e < nl; e += kTkThreads) {
        const int key = s_idx[e] >> 8;
        if (e > 0 && (s_idx[e - 1] >> 8) == key) continue;  // not the first entry of its run
        double corr = 0.0;
        for (int f = e; f < nl && (s_idx[f] >> 8) == key; ++f) corr += s_dres[f];
        parts[key] += corr;
      }
      if (lds_parts) {
        __syncthreads();
        for (int64_t t = tid; t < nparts; t += kTkThreads) rsum[b * nparts + t] = s_parts[t];
      }
    }
  }
  if (kDraw) {
    __syncthreads();  // r and the residual sums are complete (a flagged row: NaN sums in rsum)
    draw(flags ? rsum + b * nparts : parts);
  }
}

}  // namespace

hipError_t launch_induced_topk_expsum(const float* p, const float* q, int64_t B, int64_t V, int K, int s_max,
                                      float* r, int32_t* row_status, hipStream_t st, double* rsum) {
  const int64_t nsub = (V + kResSub - 1) / kResSub;
  const TkDraw none = {nullptr, 0, 0, {nullptr, nullptr, nullptr, 0, nullptr, nullptr}, nullptr, nullptr, nullptr};
  if (rsum)
    hipLaunchKernelGGL((es_topk_kernel<true, false>), dim3((unsigned)B), dim3(kTkThreads), 0, st, p, q, V, K, s_max, r,
                       row_status, rsum, nsub, none);
  else
    hipLaunchKernelGGL((es_topk_kernel<false, false>), dim3((unsigned)B), dim3(kTkThreads), 0, st, p, q, V, K, s_max,
                       r, row_status, nullptr, nsub, none);
  return hipGetLastError();
}

hipError_t launch_step_topk_expsum(const float* p, const float* q, const int32_t* drafts, const float* u, uint64_t seed,
                                   uint64_t offset, int64_t B, int64_t V, int K, int s_max, float* r,
                                   int32_t* sel_index, int32_t* sel_token, int32_t* out_token, uint8_t* accepted,
                                   double* residual_mass, int32_t* row_status, double* rsum, hipStream_t st) {
  const int64_t nsub = (V + kResSub - 1) / kResSub;
  const TkDraw dr = {u, seed, offset, {q, nullptr, drafts, K, sel_index, sel_token}, out_token, accepted,
                     residual_mass};
  hipLaunchKernelGGL((es_topk_kernel<true, true>), dim3((unsigned)B), dim3(kTkThreads), 0, st, p, q, V, K, s_max, r,
                     row_status, rsum, nsub, dr);
  return hipGetLastError();
}

// ------------------------------------------------------------------ fixed scratch
// Workspace of the allocation-free variant of the K-draft quadrature: a fixed
// device array, one copy on every GPU the library runs on, held until the
// process ends.  In host code `scratch` names a host-side stand-in, never a
// device address: host code uses only the address hipGetSymbolAddress returns
// for the current device.  Every call on a GPU reuses that GPU's copy (calls
// that overlap on one GPU race on it); the kernels write every scratch entry
// they read, so nothing has to be cleared between calls.
static __device__ __align__(256) unsigned char scratch[MDSS_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kScratchDevices] = {};  // per device, set on the first call made on it
}  // namespace

// Device address of the scratch array on the calling thread's current device.
static hipError_t es_scratch_address(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (ptr == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_induced_expsum_noalloc(const float* p, const float* q, int64_t B, int64_t V, int K, float* r,
                                         int32_t* row_status, hipStream_t st) {
  if (workspace_bytes_expsum(B, V, 1) > (size_t)MDSS_NOALLOC_SCRATCH_BYTES) return hipErrorInvalidValue;
  void* ws = nullptr;
  const hipError_t e = es_scratch_address(&ws);
  if (e != hipSuccess) return e;
  return launch_induced_expsum(p, q, nullptr, B, V, K, r, row_status, ws, st);
}

}  // namespace mdss
