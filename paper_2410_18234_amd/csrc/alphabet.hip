// Truncated alphabet (Section 4, after the truncated linear program), gfx950.
//
// Omega_0 = the m tokens of largest target probability (ties by lower id).  The
// selection and Algorithm 1 run with the renormalised target
// p~ = p 1[Omega_0] / p(Omega_0); their output Z is kept with probability
// p_a = p(Omega_0), otherwise a token is drawn from the complement of Omega_0
// in proportion to p, which gives the target law p overall.
//
// Notation: p = target.
#include "common.h"

#include <math.h>

namespace mdss {

namespace {

constexpr int kAlphaThreads = 1024;
constexpr int kAlphaWaves = kAlphaThreads / 64;
constexpr int kAlphaStep = 4 * kAlphaThreads;  // tokens per streaming step (four a thread)
constexpr int kAlphaHold = 8;                  // steps a workgroup holds in registers: rows of up to 32768 tokens
constexpr int kAlphaBins = 4096;
constexpr int kAlphaList = 256;                // entries ranked against each other in LDS

// Sum of v over the workgroup, in every thread (wave tree, then the waves in order).
__device__ __forceinline__ double alpha_block_sum(double v, double* red) {
  v = wave_sum_dpp(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < kAlphaWaves; ++w) t += red[w];
  return t;
}

struct AlphaPick {
  int bin, before, count;  // the bin that holds rank k, the entries of the bins before it, its own
};
// The bin of rank k (from 0) of a histogram of nbins, in descending or ascending bin order; bin = -1
// if there are no more than k entries.  Ends with a barrier.
__device__ __forceinline__ AlphaPick alpha_pick(const uint32_t* hist, int nbins, bool descending, int k, int* red,
                                                AlphaPick* out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t c[4], sum = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int at = 4 * tid + j;
    c[j] = at < nbins ? hist[descending ? nbins - 1 - at : at] : 0u;
    sum += c[j];
  }
  const int incl = wave_inclusive_scan_int((int)sum, lane);
  if (lane == 63) red[wave] = incl;
  if (tid == 0) *out = {-1, 0, 0};
  __syncthreads();
  int before = incl - (int)sum;
#pragma unroll
  for (int w = 0; w < kAlphaWaves; ++w) before += w < wave ? red[w] : 0;
  if (before <= k && k < before + (int)sum) {
    for (int j = 0; j < 4; ++j) {
      if (k < before + (int)c[j]) {
        const int at = 4 * tid + j;
        *out = {descending ? nbins - 1 - at : at, before, (int)c[j]};
        break;
      }
      before += (int)c[j];
    }
  }
  __syncthreads();
  return *out;
}

// p~ and p(Omega_0), one workgroup a row.  The last token of Omega_0 (the m-th in descending p, ascending
// id) is found by narrowing: a histogram of the positive entries' top 11 bits (eight bins an octave), and
// only where its bin holds more than kAlphaList entries the next 10 and the last 10 bits; what is left is
// ranked entry against entry.  More than kAlphaList equal entries are cut by two histograms of their ids.
// Bound by reading p and writing p~ (kHold: a row of up to 32768 tokens is read once and stays in
// registers; longer ones are read four times).  256 x 32000, m = 40: 25 us, of which the row's load and p~'s store are
// 13; the whole alphabet step, 290 us when this kernel and the one below made strided passes over the row
// with a block scan every 1024 tokens (seven here, two there), takes 94.
template <bool kHold>
__global__ __launch_bounds__(kAlphaThreads) void alphabet_truncate_kernel(const float* __restrict__ p, int64_t V,
                                                                          int m, float* __restrict__ pt,
                                                                          double* __restrict__ mass0,
                                                                          int32_t* __restrict__ row_status) {
  __shared__ uint32_t hist[kAlphaBins];
  __shared__ uint64_t list[kAlphaList];
  __shared__ uint32_t rank[kAlphaList];
  __shared__ int ired[kAlphaWaves], bred[kAlphaWaves];
  __shared__ double dred[kAlphaWaves];
  __shared__ AlphaPick picked;
  __shared__ uint64_t s_last;
  __shared__ uint32_t s_n;
  const int64_t b = blockIdx.x;
  const float* pb = p + b * V;
  float* ptb = pt + b * V;
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  float held[kHold ? kAlphaHold : 1][4];
  if (kHold) {
#pragma unroll
    for (int s = 0; s < kAlphaHold; ++s)
      row_load4(pb, min((int64_t)s * kAlphaStep + wid * 256, V), lane, V, held[kHold ? s : 0]);
  }
  // f(first token of the wave's 256, four values) over the row; tokens from V on read as 0
  const auto each = [&](auto&& f) {
    if (kHold) {
#pragma unroll
      for (int s = 0; s < kAlphaHold; ++s) {
        const int64_t xw = (int64_t)s * kAlphaStep + wid * 256;
        if (xw < V) f(xw, held[kHold ? s : 0]);
      }
    } else {
      constexpr int kBatch = 4;
      for (int64_t x0 = wid * 256; x0 < V; x0 += kBatch * kAlphaStep) {
        float v[kBatch][4];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) row_load4(pb, min(x0 + j * kAlphaStep, V), lane, V, v[j]);
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
          if (x0 + j * kAlphaStep < V) f(x0 + j * kAlphaStep, v[j]);
      }
    }
  };
  const auto token = [&](int64_t xw, int i) { return (uint32_t)(xw + 4 * lane + i); };
  const auto clear = [&]() {
    for (int x = tid; x < kAlphaBins; x += kAlphaThreads) hist[x] = 0u;
    __syncthreads();
  };

  clear();
  bool bad = false;
  each([&](int64_t, const float (&v)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bad |= __builtin_amdgcn_classf(v[i], 0x21F);
      if (v[i] > 0.0f) atomicAdd(&hist[__float_as_uint(v[i]) >> 20], 1u);
    }
  });
  bad = __builtin_amdgcn_ballot_w64(bad) != 0;
  if (lane == 0) bred[wid] = bad ? 1 : 0;
  __syncthreads();
  int any = 0;
#pragma unroll
  for (int w = 0; w < kAlphaWaves; ++w) any |= bred[w];
  if (any) {
    const float nan[4] = {NAN, NAN, NAN, NAN};
    each([&](int64_t xw, const float (&)[4]) { row_store4(ptb, xw, lane, V, nan); });
    if (tid == 0) {
      mass0[b] = __longlong_as_double(0x7ff8000000000000ll);
      if (row_status) row_status[b] |= kRowBadProb;
    }
    return;
  }
  // Omega_0 = the positive entries with bits > t_bits, or bits == t_bits and id <= t_id (entries of
  // p = 0 that it may also hold have p~ = 0 and no mass)
  uint32_t t_bits = 0u, t_id = 0u;
  AlphaPick k = alpha_pick(hist, 2048, true, (int)min((int64_t)m, V) - 1, ired, &picked);
  if (k.bin >= 0) {
    int need = (int)min((int64_t)m, V) - 1 - k.before;  // rank among the entries of the bin
    uint32_t prefix = (uint32_t)k.bin;
    int shift = 20;
    while (k.count > kAlphaList && shift > 0) {  // uniform
      clear();
      each([&](int64_t, const float (&v)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t bits = __float_as_uint(v[i]);
          if (v[i] > 0.0f && bits >> shift == prefix) atomicAdd(&hist[(bits >> (shift - 10)) & 1023u], 1u);
        }
      });
      __syncthreads();
      k = alpha_pick(hist, 1024, true, need, ired, &picked);
      need -= k.before;
      prefix = prefix << 10 | (uint32_t)k.bin;
      shift -= 10;
    }
    if (k.count <= kAlphaList) {
      if (tid == 0) s_n = 0u;
      if (tid < kAlphaList) rank[tid] = 0u;
      __syncthreads();
      each([&](int64_t xw, const float (&v)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t bits = __float_as_uint(v[i]);
          if (v[i] > 0.0f && bits >> shift == prefix)
            list[atomicAdd(&s_n, 1u)] = (uint64_t)~bits << 32 | token(xw, i);  // ascending: descending p, ascending id
        }
      });
      __syncthreads();
      // each entry's rank, a quarter of the others by each of four threads
      const int n = k.count, mine = tid & (kAlphaList - 1), part = tid / kAlphaList, per = (n + 3) / 4;
      if (mine < n) {
        const uint64_t key = list[mine];
        uint32_t below = 0;
        for (int j = part * per; j < min(n, (part + 1) * per); ++j) below += list[j] < key ? 1u : 0u;
        atomicAdd(&rank[mine], below);
      }
      __syncthreads();
      if (tid < n && rank[tid] == (uint32_t)need) s_last = list[tid];
      __syncthreads();
      t_bits = ~(uint32_t)(s_last >> 32);
      t_id = (uint32_t)s_last;
    } else {  // many equal entries: the one of rank `need` by id
      t_bits = prefix;
      for (int digit = 0; digit < 2; ++digit) {
        clear();
        each([&](int64_t xw, const float (&v)[4]) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t x = token(xw, i);
            if (__float_as_uint(v[i]) == prefix && (digit == 0 || x >> 12 == t_id))
              atomicAdd(&hist[digit == 0 ? x >> 12 : x & 4095u], 1u);
          }
        });
        __syncthreads();
        k = alpha_pick(hist, kAlphaBins, false, need, ired, &picked);
        need -= k.before;
        t_id = t_id << 12 | (uint32_t)k.bin;
      }
    }
  }
  const auto inside = [&](float v, uint32_t x) {
    const uint32_t bits = __float_as_uint(v);
    return v > 0.0f && (bits > t_bits || (bits == t_bits && x <= t_id));
  };
  double mass = 0.0;
  each([&](int64_t xw, const float (&v)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (inside(v[i], token(xw, i))) mass += (double)v[i];
  });
  const double M = alpha_block_sum(mass, dred);
  each([&](int64_t xw, const float (&v)[4]) {
    float out[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      out[i] = 0.0f;
      if (inside(v[i], token(xw, i)) && M > 0.0) out[i] = (float)((double)v[i] / M);
    }
    row_store4(ptb, xw, lane, V, out);
  });
  if (tid == 0) mass0[b] = M;
}

// Post-processing: keep Z iff u_keep < p_a, else the smallest id j outside
// Omega_0 (p~ = 0) with C_j > u_draw Z_c, C the complement's running p mass.
// One workgroup a row reads p and p~ once, all of a wave's loads first (rows of up to 32768 tokens), with the
// complement's sum of every unit of 256 c tokens in LDS (c = 1 up to 2^18 tokens, so at most 1024
// units); one wave then finds the unit and reads it again for the token.  15 us at 256 x 32000, m = 40.
constexpr int kPostUnits = 1024;
__global__ __launch_bounds__(kAlphaThreads) void alphabet_post_kernel(
    const float* __restrict__ p, const float* __restrict__ pt, const double* __restrict__ mass0,
    const int32_t* __restrict__ token, const float* __restrict__ u2, uint64_t seed, uint64_t offset, int64_t V,
    int32_t* __restrict__ out_token, uint8_t* __restrict__ kept) {
  __shared__ double sums[kPostUnits];
  const int64_t b = blockIdx.x;
  const int32_t z = token[b];
  float uk, ud;
  if (u2) {
    uk = u2[b * 2];
    ud = u2[b * 2 + 1];
  } else {
    const uint64_t pos = offset + (uint64_t)b;
    uint32_t c[4] = {(uint32_t)pos, (uint32_t)(pos >> 32), 0u, 1u};
    philox4x32_10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    uk = (float)(c[0] >> 8) * 5.9604644775390625e-8f;  // 2^-24
    ud = (float)(c[1] >> 8) * 5.9604644775390625e-8f;
  }
  const double pa = mass0[b];
  if (z < 0 || !((double)uk >= pa)) {  // an invalid Z is passed on; NaN p_a keeps Z
    if (threadIdx.x == 0) {
      out_token[b] = z;
      kept[b] = z >= 0 ? 1 : 0;
    }
    return;
  }
  const float* pb = p + b * V;
  const float* ptb = pt + b * V;
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = (int)((V + kPostUnits * 256 - 1) / (kPostUnits * 256));  // tiles of 256 tokens a unit
  const int units = (int)((V + 256 * c - 1) / (256 * c));
  // the wave's tiles: those of the units wid, wid + 16, ..; kBatch tiles' loads in flight
  constexpr int kBatch = 8;
  const int tiles = (units - wid + kAlphaWaves - 1) / kAlphaWaves * c;  // not positive without a unit
  double unit_sum = 0.0;
  for (int t0 = 0; t0 < tiles; t0 += kBatch) {
    float pv[kBatch][4], mv[kBatch][4];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int t = min(t0 + j, tiles - 1);
      const int64_t xw = min(((int64_t)(t / c * kAlphaWaves + wid) * c + t % c) * 256, V);
      row_load4(pb, xw, lane, V, pv[j]);
      row_load4(ptb, xw, lane, V, mv[j]);
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int t = t0 + j;
      if (t >= tiles) break;  // uniform
      double local = 0.0;
#pragma unroll
      for (int i = 0; i < 4; ++i) local += !(mv[j][i] > 0.0f) ? (double)pv[j][i] : 0.0;
      unit_sum += wave_sum_dpp(local);
      if (t % c == c - 1) {
        if (lane == 0) sums[t / c * kAlphaWaves + wid] = unit_sum;
        unit_sum = 0.0;
      }
    }
  }
  __syncthreads();
  if (wid != 0) return;
  // lane l takes the units [16 l, 16 l + 16)
  constexpr int kPer = kPostUnits / 64;
  double lane_sum = 0.0;
  for (int s = lane * kPer; s < min(units, (lane + 1) * kPer); ++s) lane_sum += sums[s];
  const double incl = wave_inclusive_scan_dpp(lane_sum, lane);
  const double Zc = __shfl(incl, 63, 64);
  double run = __shfl_up(incl, 1, 64);
  if (lane == 0) run = 0.0;
  const double t = (double)ud * Zc;
  int my = -1;
  double my_base = 0.0;
  for (int s = lane * kPer; s < min(units, (lane + 1) * kPer); ++s) {
    const double prev = run;
    run += sums[s];
    if (run > t) {
      my = s;
      my_base = prev;
      break;
    }
  }
  const unsigned long long hit = __builtin_amdgcn_ballot_w64(my >= 0);
  int found = -1;
  if (Zc > 0.0 && hit) {
    const int src = __ffsll((long long)hit) - 1;
    const int64_t first = (int64_t)__shfl(my, src, 64) * c * 256;
    double base = __shfl(my_base, src, 64);
    int last = -1;  // the unit's last token with mass, should the sums' rounding leave t at its end
    for (int j = 0; j < c && found < 0; ++j) {
      const int64_t x0 = first + 256 * j + 4 * lane;  // four consecutive tokens a lane
      double v[4], local = 0.0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = (x0 + i < V && !(ptb[x0 + i] > 0.0f)) ? (double)pb[x0 + i] : 0.0;
        local += v[i];
      }
      const double li = wave_inclusive_scan_dpp(local, lane);
      double C = base + __shfl_up(li, 1, 64);
      if (lane == 0) C = base;
      int at = -1;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        C += v[i];
        if (v[i] > 0.0) last = (int)(x0 + i);
        if (at < 0 && v[i] > 0.0 && C > t) at = (int)(x0 + i);
      }
      const unsigned long long h = __builtin_amdgcn_ballot_w64(at >= 0);
      if (h) found = __shfl(at, __ffsll((long long)h) - 1, 64);
      base += __shfl(li, 63, 64);
    }
    if (found < 0) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) last = max(last, __shfl_xor(last, off, 64));
      found = last;
    }
  }
  if (lane == 0) {  // without a mass outside Omega_0 the token stays
    out_token[b] = found >= 0 ? found : z;
    kept[b] = found >= 0 ? 0 : 1;
  }
}

}  // namespace

hipError_t launch_alphabet_truncate(const float* p, int64_t B, int64_t V, int m, float* pt, double* mass0,
                                    int32_t* row_status, hipStream_t st) {
  if (V <= kAlphaHold * kAlphaStep)
    hipLaunchKernelGGL(alphabet_truncate_kernel<true>, dim3((unsigned)B), dim3(kAlphaThreads), 0, st, p, V, m, pt, mass0,
                       row_status);
  else
    hipLaunchKernelGGL(alphabet_truncate_kernel<false>, dim3((unsigned)B), dim3(kAlphaThreads), 0, st, p, V, m, pt,
                       mass0, row_status);
  return hipGetLastError();
}

hipError_t launch_alphabet_post(const float* p, const float* pt, const double* mass0, const int32_t* token,
                                const float* u2, uint64_t seed, uint64_t offset, int64_t B, int64_t V,
                                int32_t* out_token, uint8_t* kept, hipStream_t st) {
  hipLaunchKernelGGL(alphabet_post_kernel, dim3((unsigned)B), dim3(kAlphaThreads), 0, st, p, pt, mass0, token, u2,
                     seed, offset, V, out_token, kept);
  return hipGetLastError();
}

}  // namespace mdss
