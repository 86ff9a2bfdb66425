// Truncated linear program for two drafts (Algorithm 2 with the fixed weights
// of eq. heur and the selected-token distribution of eq. p_Ieq; the sort-free
// variant eq. heur2 / p_Ieq3; the same construction for drafts from two
// different distributions, non-identical appendix), gfx950.
//
// Notation: p = target, q1 / q2 = distributions of the first / second draft
// (q2 = q1 for identical drafts).  Tokens are ranked by the key p - q1 q2
// (fp64, rounded once to fp32; larger first, ties by lower id).  Omega_1 =
// the first s ranked tokens; every pair that touches Omega_2 has a fixed
// winner, only the pairs inside Omega_1 are decided by the linear program.
//
// Per row:
//   rank kernel (one workgroup of 1024 threads):
//     SORTED tail (rows that tlp_sort_kernel below leaves): one stable scatter of the row into 256 bins by the top 8
//       bits of the rank word, each group of bins then sorted in LDS, and one
//       reverse scan over the ranked order: r(k) = q1 q2 + q2(k) S1(k) +
//       q1(k) S2(k) with S_i(k) the q_i mass ranked after k;
//     HALF tail: top-s selection only, then r(k) = q1 q2 + (q2 (A - q1) + q1
//       (B - q2)) / 2 with A, B the Omega_2 masses.
//   LP kernel (one wave): the Omega_1 program maximises sum_k min(p_k, c_k +
//     f_k), where c_k is the fixed part of token k's probability and f_k the
//     share it receives of the Omega_1 pairs' masses m_xy (both drafting
//     orders).  It is solved exactly as a maximum flow: start with every pair
//     credited to its earlier-ranked token, then move mass along shortest
//     augmenting paths (Edmonds-Karp) from tokens above their target mass to
//     tokens below it.  The resulting shares give the selection table w.
#include "rank.h"

#include <math.h>

namespace mdss {

namespace {

constexpr int kMaxS = 16;       // largest s accepted by the library
constexpr int kLpMaxIter = 4096;  // augmentations before a row is flagged (bound for s = 16: (s+2)(s(s-1)+2s) = 4608)
constexpr int kTailSorted = 0;
constexpr int kTailHalf = 1;

struct alignas(16) TlpHdr {
  int32_t s_eff;       // min(s, V)
  int32_t flags;       // row status bits found by the rank kernel
  int32_t pad0, pad1;
  double a_tail;       // q1 mass of Omega_2
  double b_tail;       // q2 mass of Omega_2
  double tail_accept;  // sum over Omega_2 of min(p, r)
  double pad2;
};

// Rank word: ascending order of the word = descending key, so a stable
// ascending sort of (word, id) in id order gives the ranking.
__device__ __forceinline__ uint32_t rank_word(float p, float a, float b) {
  const float key = (float)((double)p - (double)a * (double)b) + 0.0f;  // -0 -> +0
  const uint32_t u = __float_as_uint(key);
  const uint32_t asc = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ~asc;
}

__device__ __forceinline__ void flag_row(int64_t b, int64_t V, int s, float* rb, int32_t* omega1, TlpHdr* hdr,
                         int32_t* row_status, int flags) {
  for (int64_t i = threadIdx.x; i < V; i += kRankThreads) rb[i] = __int_as_float(0x7fc00000);
  if (threadIdx.x < s) omega1[b * s + threadIdx.x] = -1;
  if (threadIdx.x == 0) {
    TlpHdr h = {};
    h.flags = flags;
    hdr[b] = h;
    if (row_status) row_status[b] |= flags;
  }
}

// ---------------------------------------------------------------- SORTED tail
// The ranking of Algorithm 2 on the rank scan: values (p, q1, q2); the scan
// masses are (q1, q2) of the Omega_2 entries; an Omega_1 entry (rank < s) is
// recorded in omega1, every Omega_2 entry k gets r(k) = q1 q2 + q2 S1 + q1 S2.
struct TlpSpec {
  struct Args {
    const float *p, *q1, *q2;
    float* r;
    int32_t* omega1;
    TlpHdr* hdr;
    int32_t* row_status;
    int s;
  };
  struct Row {
    const float *in0, *in1, *in2;
    float* rb;
    int32_t* omega1;
    TlpHdr* hdr;
    int32_t* row_status;
    int64_t b, V;
    int s;
  };
  struct State {
    double acc = 0.0;  // sum over Omega_2 of min(p, r)
  };
  static __device__ __forceinline__ Row row(const Args& a, int64_t b, int64_t V);
  static __device__ __forceinline__ uint32_t word(float p, float q1, float q2) { return rank_word(p, q1, q2); }
  static __device__ __forceinline__ void set_totals(Row&, double, double) {}
  static __device__ __forceinline__ void masses(const Row& r, uint32_t rank, float, float q1, float q2, double* m1,
                                                double* m2) {
    const bool om1 = rank < (uint32_t)r.s;
    *m1 = om1 ? 0.0 : (double)q1;
    *m2 = om1 ? 0.0 : (double)q2;
  }
  static __device__ __forceinline__ void visit(const Row& r, State& st, uint32_t rank, int id, float p, float q1,
                                               float q2, double s1, double s2) {
    if (rank < (uint32_t)r.s) {
      r.omega1[r.b * r.s + rank] = id;
      return;
    }
    const double av = (double)q1, bv = (double)q2;
    const double rv = av * bv + bv * s1 + av * s2;
    r.rb[id] = (float)rv;
    st.acc += fmin((double)p, rv);
  }
  static __device__ __forceinline__ void flag(const Row& r, int64_t V, int flags) {
    flag_row(r.b, V, r.s, r.rb, r.omega1, r.hdr, r.row_status, flags);
  }
  static __device__ __forceinline__ void finish(const Row& r, State& st, double c1, double c2, double* red) {
    const int se = (int)min((int64_t)r.s, r.V);
    if ((int)threadIdx.x >= se && (int)threadIdx.x < r.s) r.omega1[r.b * r.s + threadIdx.x] = -1;
    const double acc = block_sum(st.acc, red);
    if (threadIdx.x == 0) {
      TlpHdr h = {};
      h.s_eff = se;
      h.a_tail = c1;
      h.b_tail = c2;
      h.tail_accept = acc;
      r.hdr[r.b] = h;
    }
  }
};

__device__ __forceinline__ TlpSpec::Row TlpSpec::row(const Args& a, int64_t b, int64_t V) {
  Row r;
  r.in0 = a.p + b * V;
  r.in1 = a.q1 + b * V;
  r.in2 = a.q2 + b * V;
  r.rb = a.r + b * V;
  r.omega1 = a.omega1;
  r.hdr = a.hdr;
  r.row_status = a.row_status;
  r.b = b;
  r.V = V;
  r.s = a.s;
  return r;
}

// ------------------------------------------------- SORTED tail, by cells
// The same plan without moving a row's entries through memory.  A token's word is kept in a workspace plane; its
// rank comes back by token, for rows of up to 32768 tokens through LDS into registers (kHold), for
// longer ones through a second plane.
//   Ranks.  A histogram of the words' top bits (kHold: 2048 bins, four an octave of the key; else 4096) splits
//     the ranking into groups of whole bins of at most kGroupMax tokens.  Inside a bin a token goes to the cell
//     floor(its low bits' share of the bin x the bin's tokens): about one token a cell; the tokens
//     of a cell are compared with each other.
//   Scan.  From the last ranks down, at most kScanGroup at a time, q1 and q2 are written to LDS in rank order,
//     scanned, and replaced by r, which the tokens' threads read back and store in token order.
// Rows with a bin of more tokens than a group, or a cell of more than kSortCell (equal keys), are left
// to rank_scan_kernel, and so are rows of more than kSortMaxV tokens: every group reads the whole row again, and Zipf rows
// past it have bins of more tokens than a group.  One law, this plan against rank_scan_kernel alone: 8 x 131072 778 us
// against 1474 (Zipf 803, 1499), 32 x 200000 1880 against 2654 (Zipf 3068, 3012: given up and ranked there), 8 x 262144
// 2606 against 2971 (Zipf 3302, 3256), 8 x 400000 6304 against 4523.
// Bound by LDS gathers and by the reads of the row (once for the words, once a scan group).  256 x 32000, two
// laws: 133 us (words 21, four groups' ranks 14 each, two groups' scans 23 each); the whole call takes 169 us
// against 484 with rank_scan_kernel alone.
constexpr int kSortStep = 4 * kRankThreads;
constexpr int kSortCopies = 8;
constexpr int kSortHold = 8;  // steps held in registers
constexpr int kSortCell = 64;
constexpr int kScanGroup = 16384;
constexpr int64_t kSortMaxV = 1 << 17;

template <bool kHold>
struct SortShared {
  static constexpr int kGroupMax = kHold ? 8704 : 12288;  // what the LDS has room for
  static constexpr int kSortShift = kHold ? 21 : 20;
  static constexpr int kSortBins = 1 << (32 - kSortShift);
  union {
    struct {
      uint64_t key[kGroupMax];       // word, id
      uint32_t cell[kGroupMax / 2];  // two cells' 16-bit counts, then places, then ends
      uint16_t rank[kHold ? kSortHold * kSortStep : 1];
    } a;
    uint32_t hist[kSortBins][kSortCopies];  // a copy for every kSortCopies-th lane: equal bins in a wave
    union {
      float2 q;
      double r;
    } slot[kScanGroup];
  };
  uint32_t start[kSortBins + 1];
  double sa[kRankWaves], sb[kRankWaves];
  uint32_t red[kRankWaves];
  uint32_t over, count;
};

// sum of v over the threads before this one (one barrier)
__device__ __forceinline__ uint32_t sort_block_exclusive(uint32_t v, uint32_t* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t incl = (uint32_t)wave_inclusive_scan_int((int)v, lane);
  if (lane == 63) red[wave] = incl;
  __syncthreads();
  uint32_t off = 0;
#pragma unroll
  for (int w = 0; w < kRankWaves; ++w) off += w < wave ? red[w] : 0u;
  return off + incl - v;
}

// f(the wave's first token, the values of N arrays at the thread's four) over a row, kBatch steps' loads in
// flight; arrays as floats (bits of words and ranks pass unchanged), 0 from V on.
template <int kBatch, int N, class F>
__device__ __forceinline__ void sort_each(const float* const (&x)[N], int64_t V, int lane, int wid, F&& f) {
  for (int64_t x0 = wid * 256; x0 < V; x0 += kBatch * kSortStep) {
    float v[kBatch][N][4];
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
#pragma unroll
      for (int k = 0; k < N; ++k) row_load4(x[k], min(x0 + j * kSortStep, V), lane, V, v[j][k]);
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      if (x0 + j * kSortStep < V) f((int)x0 + j * kSortStep, v[j]);
  }
}

template <bool kHold>
__device__ __forceinline__ bool sort_row(const TlpSpec::Args& args, int64_t b, int64_t V, float* words, float* ranks,
                                         SortShared<kHold>& sh) {
  constexpr int kGroupMax = SortShared<kHold>::kGroupMax;
  constexpr int kSortShift = SortShared<kHold>::kSortShift, kSortBins = SortShared<kHold>::kSortBins;
  constexpr int kSteps = kHold ? kSortHold : 1;
  const TlpSpec::Row row = TlpSpec::row(args, b, V);
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = (int)V;
  uint32_t held[kSteps][4];  // kHold, scan: ranks, then r
  uint32_t todo = ~0u;       // kHold: bit 4 s + i, the token's r is not known yet
  static_assert(kSortHold * 4 <= 32, "a bit a token");
  const auto token = [&](int xw, int i) { return xw + 4 * lane + i; };
  // kHold: a step's place, as new values: addresses and token numbers are not kept from pass to pass (they
  // would spill)
  struct Place {
    int xw, lane;
    __device__ __forceinline__ int token(int i) const { return xw + 4 * lane + i; }
  };
  const auto place = [&](int s) {
    __builtin_amdgcn_sched_barrier(0);
    Place at = {wid, lane};
    __asm__ volatile("" : "+s"(at.xw), "+v"(at.lane));
    at.xw = s * kSortStep + at.xw * 256;
#pragma unroll
    for (int i = 0; i < 4; ++i) __asm__ volatile("" : "+v"(held[s][i]));
    return at;
  };
  const auto load = [&](const float* x, const Place& at, float (&v)[4]) {
    row_load4(x, min((int64_t)at.xw, V), at.lane, V, v);
  };

  for (int x = tid; x < kSortBins * kSortCopies; x += kRankThreads) (&sh.hist[0][0])[x] = 0u;
  if (tid == 0) sh.over = 0u;
  __syncthreads();
  bool bad = false;
  const float* const pqq[3] = {row.in0, row.in1, row.in2};
  sort_each<2>(pqq, V, lane, wid, [&](int xw, const float (&v)[3][4]) {
    float w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int k = 0; k < 3; ++k) bad |= __builtin_amdgcn_classf(v[k][i], 0x21F);
      const uint32_t word = rank_word(v[0][i], v[1][i], v[2][i]);
      if (token(xw, i) < n) atomicAdd(&sh.hist[word >> kSortShift][lane % kSortCopies], 1u);
      w[i] = __uint_as_float(word);
    }
    row_store4(words, xw, lane, V, w);
  });
  bad = __builtin_amdgcn_ballot_w64(bad) != 0;
  if (lane == 0) sh.red[wid] = bad ? 1u : 0u;
  __syncthreads();
  uint32_t any = 0u;
#pragma unroll
  for (int w = 0; w < kRankWaves; ++w) any |= sh.red[w];
  if (any) {
    TlpSpec::flag(row, V, kRowBadProb);
    return true;
  }
  __syncthreads();
  {  // starts of the bins
    constexpr int kPer = kSortBins / kRankThreads;
    uint32_t c[kPer], sum = 0u;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      c[j] = 0u;
#pragma unroll
      for (int k = 0; k < kSortCopies; ++k) c[j] += sh.hist[kPer * tid + j][k];
      if (c[j] > (uint32_t)kGroupMax) sh.over = 1u;
      sum += c[j];
    }
    uint32_t at = sort_block_exclusive(sum, sh.red);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      sh.start[kPer * tid + j] = at;
      at += c[j];
    }
    if (tid == kRankThreads - 1) sh.start[kSortBins] = at;
  }
  __syncthreads();
  if (sh.over) return false;  // uniform

  // ranks, a group of bins at a time
  for (int c0 = 0; c0 < kSortBins;) {
    const uint32_t g0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.start[c0]);
    if (g0 == (uint32_t)n) break;
    int lo = c0 + 1, hi = kSortBins;  // the last c with start[c] - g0 <= kGroupMax
    while (lo < hi) {
      const int mid = (lo + hi + 1) / 2;
      if (sh.start[mid] - g0 <= (uint32_t)kGroupMax)
        lo = mid;
      else
        hi = mid - 1;
    }
    const int c1 = __builtin_amdgcn_readfirstlane(lo);
    const int G = (int)(sh.start[c1] - g0);
    for (int x = tid; x < kGroupMax / 2; x += kRankThreads) sh.a.cell[x] = 0u;
    if (tid == 0) sh.count = 0u;
    __syncthreads();
    // the group's tokens in any order: the words [w0, w0 + span); one atomic a wave and batch of 16 tokens a lane
    const uint32_t w0 = (uint32_t)c0 << kSortShift, span = (c1 < kSortBins ? (uint32_t)c1 << kSortShift : ~0u) - w0;
    constexpr int kBatch = 4;
    const auto put = [&](const uint32_t (&w)[kBatch][4], auto&& token_of) {
      uint32_t in_wave = 0u;
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          in_wave += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(w[j][i] - w0 < span));
      uint32_t at = 0u;
      if (lane == 0) at = atomicAdd(&sh.count, in_wave);
      at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool mine = w[j][i] - w0 < span;
          const uint64_t m = __builtin_amdgcn_ballot_w64(mine);
          const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
          if (mine) sh.a.key[at + below] = (uint64_t)w[j][i] << 32 | (uint32_t)token_of(j, i);
          at += (uint32_t)__builtin_popcountll(m);
        }
    };
    for (int64_t x0 = wid * 256; x0 < V; x0 += kBatch * kSortStep) {
      uint32_t w[kBatch][4];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        float v[4];
        row_load4(words, min(x0 + j * kSortStep, V), lane, V, v);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          // no finite key has the word 2^32 - 1
          w[j][i] = token((int)x0 + j * kSortStep, i) < n ? __float_as_uint(v[i]) : ~0u;
      }
      put(w, [&](int j, int i) { return token((int)x0 + j * kSortStep, i); });
    }
    __syncthreads();
    constexpr int kMine = (kGroupMax + kRankThreads - 1) / kRankThreads;
    uint64_t key[kMine];
    uint32_t cell[kMine];
#pragma unroll
    for (int j = 0; j < kMine; ++j) {
      const int g = tid + j * kRankThreads;
      key[j] = sh.a.key[min(g, kGroupMax - 1)];
      if (g >= G) continue;
      const uint32_t w = (uint32_t)(key[j] >> 32), c = w >> kSortShift;
      const uint32_t first = sh.start[c], size = sh.start[c + 1] - first;
      cell[j] = first - g0 + __umulhi(w << (32 - kSortShift), size);
      atomicAdd(&sh.a.cell[cell[j] >> 1], 1u << (16 * (cell[j] & 1u)));
    }
    __syncthreads();
    {
      constexpr int kCells = kGroupMax / 2, kPer = (kCells + kRankThreads - 1) / kRankThreads;
      uint32_t c[kPer], sum = 0u, most = 0u;
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const int x = kPer * tid + j;
        c[j] = x < kCells ? sh.a.cell[x] : 0u;
        sum += (c[j] & 0xFFFFu) + (c[j] >> 16);
        most = max(most, max(c[j] & 0xFFFFu, c[j] >> 16));
      }
      if (most > (uint32_t)kSortCell) sh.over = 1u;
      uint32_t at = sort_block_exclusive(sum, sh.red);
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const uint32_t l = c[j] & 0xFFFFu;
        if (kPer * tid + j < kCells) sh.a.cell[kPer * tid + j] = at | (at + l) << 16;
        at += l + (c[j] >> 16);
      }
    }
    __syncthreads();
    if (sh.over) return false;  // uniform
#pragma unroll
    for (int j = 0; j < kMine; ++j) {
      if (tid + j * kRankThreads >= G) continue;
      const uint32_t sf = 16 * (cell[j] & 1u);
      sh.a.key[(atomicAdd(&sh.a.cell[cell[j] >> 1], 1u << sf) >> sf) & 0xFFFFu] = key[j];
    }
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < kMine; ++j) {  // a cell's end is now the next one's start
      if (tid + j * kRankThreads >= G) continue;
      const uint32_t two = sh.a.cell[cell[j] >> 1], one = cell[j] >= 2u ? sh.a.cell[(cell[j] >> 1) - 1] : 0u;
      const uint32_t k0 = cell[j] & 1u ? two & 0xFFFFu : one >> 16, k1 = cell[j] & 1u ? two >> 16 : two & 0xFFFFu;
      uint32_t rank = k0;
      if (k1 - k0 > 1u)
#pragma unroll 1
        for (uint32_t k = k0; k < k1; ++k) rank += sh.a.key[k] < key[j] ? 1u : 0u;
      if constexpr (kHold)
        sh.a.rank[(uint32_t)key[j]] = (uint16_t)(g0 + rank);
      else
        ranks[(uint32_t)key[j]] = __uint_as_float(g0 + rank);
    }
    __syncthreads();
    c0 = c1;
  }
  if constexpr (kHold) {
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int x = token(s * kSortStep + wid * 256, i);
        held[s][i] = x < n ? sh.a.rank[x] : ~0u;
      }
    }
    __syncthreads();
  }

  // scan, the last ranks first
  double c1 = 0.0, c2 = 0.0, acc = 0.0;
  for (int g1 = n; g1 > 0;) {
    const int g0 = max(0, g1 - kScanGroup), G = g1 - g0;
    const auto put = [&](uint32_t rank, float av, float bv) {
      if (rank - (uint32_t)g0 < (uint32_t)G) sh.slot[rank - g0].q = make_float2(av, bv);
    };
    if constexpr (kHold) {
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        const Place at = place(s);
        float av[4], bv[4];
        load(row.in1, at, av);
        load(row.in2, at, bv);
#pragma unroll
        for (int i = 0; i < 4; ++i) put((todo >> (4 * s + i)) & 1u ? held[s][i] : ~0u, av[i], bv[i]);
      }
    } else {
      const float* const rqq[3] = {ranks, row.in1, row.in2};
      sort_each<2>(rqq, V, lane, wid, [&](int xw, const float (&v)[3][4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) put(token(xw, i) < n ? __float_as_uint(v[0][i]) : ~0u, v[1][i], v[2][i]);
      });
    }
    __syncthreads();
    const int E = (G + kRankThreads - 1) / kRankThreads | 1;  // odd: the threads' slots lie in different banks
    const int e0 = min(G, tid * E), e1 = min(G, e0 + E);
    const int om1 = row.s - g0;  // slots below it are in Omega_1
    double l1 = 0.0, l2 = 0.0;
#pragma unroll 4
    for (int g = e0; g < e1; ++g) {
      const float2 q = sh.slot[g].q;
      l1 += g < om1 ? 0.0 : (double)q.x;
      l2 += g < om1 ? 0.0 : (double)q.y;
    }
    double x1, x2, t1, t2;
    block_exclusive_suffix2(l1, l2, &x1, &x2, &t1, &t2, sh.sa, sh.sb);
    double s1 = c1 + x1, s2 = c2 + x2;  // masses ranked after the entry
#pragma unroll 4
    for (int g = e1 - 1; g >= e0; --g) {
      const float2 q = sh.slot[g].q;
      const double av = (double)q.x, bv = (double)q.y;
      sh.slot[g].r = av * bv + bv * s1 + av * s2;
      s1 += g < om1 ? 0.0 : av;
      s2 += g < om1 ? 0.0 : bv;
    }
    c1 += t1;
    c2 += t2;
    __syncthreads();
    // r of a token of the group
    const auto get = [&](uint32_t rank, int x, float pv, float& r) {
      if (rank - (uint32_t)g0 >= (uint32_t)G) return;
      const double rv = sh.slot[rank - g0].r;
      if ((int)rank < row.s)
        row.omega1[b * row.s + rank] = x;  // its r comes with the linear program
      else
        acc += fmin((double)pv, rv);
      r = (float)rv;
    };
    if constexpr (kHold) {
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        const Place at = place(s);
        float pv[4];
        load(row.in0, at, pv);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t rank = (todo >> (4 * s + i)) & 1u ? held[s][i] : ~0u;
          float r = __uint_as_float(held[s][i]);
          get(rank, at.token(i), pv[i], r);
          held[s][i] = __float_as_uint(r);
          todo &= ~((rank - (uint32_t)g0 < (uint32_t)G ? 1u : 0u) << (4 * s + i));
        }
      }
    } else {
      const float* const rp[2] = {ranks, row.in0};
      sort_each<2>(rp, V, lane, wid, [&](int xw, const float (&v)[2][4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int x = token(xw, i);
          const uint32_t rank = x < n ? __float_as_uint(v[0][i]) : ~0u;
          float r = 0.0f;
          get(rank, x, v[1][i], r);
          if (rank - (uint32_t)g0 < (uint32_t)G) row.rb[x] = r;
        }
      });
    }
    __syncthreads();
    g1 = g0;
  }
  if constexpr (kHold) {
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      const Place at = place(s);
      const float r[4] = {__uint_as_float(held[s][0]), __uint_as_float(held[s][1]), __uint_as_float(held[s][2]),
                          __uint_as_float(held[s][3])};
      if (at.xw < n) row_store4(row.rb, at.xw, at.lane, V, r);
    }
  }
  TlpSpec::State state;
  state.acc = acc;
  TlpSpec::finish(row, state, c1, c2, sh.sa);
  return true;
}

// later[b V]: the row is left to rank_scan_kernel.
template <bool kHold>
__global__ __launch_bounds__(kRankThreads) void tlp_sort_kernel(TlpSpec::Args args, int64_t V, float* words,
                                                                float* ranks, uint32_t* later) {
  __shared__ SortShared<kHold> sh;
  const int64_t b = blockIdx.x;
  const bool done = sort_row<kHold>(args, b, V, words + b * V, ranks + b * V, sh);
  if (threadIdx.x == 0) later[b * V] = done ? 0u : 1u;
}

// ------------------------------------------------------------------ HALF tail
// Composite rank: (rank word, id); the smallest composites are the first ranked.
__device__ __forceinline__ uint64_t composite(float p, float a, float b, int id) {
  return ((uint64_t)rank_word(p, a, b) << 32) | (uint32_t)id;
}

constexpr int kHalfList = 512;

// One workgroup a row, which it reads twice.  Pass 1: every thread's first-ranked token and its draft masses.  The s-th
// smallest of the threads' composites bounds Omega_1, so only the s threads at or below the bound look at their
// tokens again: those at or below it are candidates (about s; ranked one against the other), and
// their masses leave the thread's sums, so that the Omega_2 masses are sums of Omega_2 tokens alone.
// Pass 2: r and the acceptance.  More than kHalfList candidates (rows in an order of their keys): one pass a
// rank instead.  Bound by the two reads, with only as many CUs busy as there are rows.
// 96 x 50257, s = 8: 56 us; the whole call takes 104 us against 180 with three strided passes and a sorted list of
// 16 a thread.
template <bool kTwo>
__global__ __launch_bounds__(kRankThreads) void tlp_rank_half_kernel(
    const float* __restrict__ p, const float* __restrict__ q1, const float* __restrict__ q2, int64_t V, int s,
    float* __restrict__ r, int32_t* __restrict__ omega1, TlpHdr* __restrict__ hdr,
    int32_t* __restrict__ row_status) {
  __shared__ uint64_t top[kRankWaves * kMaxS];
  __shared__ uint64_t key[kHalfList], sorted[kHalfList];
  __shared__ float2 mass[kHalfList], sorted_mass[kHalfList];
  __shared__ double sa[kRankWaves];
  __shared__ uint64_t s_bound;
  __shared__ int red[kRankWaves];
  __shared__ int s_n;
  const int64_t b = blockIdx.x;
  const float* pb = p + b * V;
  const float* ab = q1 + b * V;
  const float* bb = (kTwo ? q2 : q1) + b * V;
  float* rb = r + b * V;
  const int n = (int)V;
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int se = min(s, n);
  const auto token = [&](int xw, int i) { return xw + 4 * lane + i; };
  // f(the wave's first token, p, q1, q2 of the thread's four)
  const auto each = [&](auto&& f) {
    if constexpr (kTwo) {
      const float* const x[3] = {pb, ab, bb};
      sort_each<2>(x, V, lane, wid, [&](int xw, const float (&v)[3][4]) { f(xw, v[0], v[1], v[2]); });
    } else {
      const float* const x[2] = {pb, ab};
      sort_each<4>(x, V, lane, wid, [&](int xw, const float (&v)[2][4]) { f(xw, v[0], v[1], v[1]); });
    }
  };
  if (tid == 0) s_n = 0;
  bool bad = false;
  uint32_t w_min = ~0u;  // no finite key has this word
  int id_min = -1;
  double A = 0.0, Bm = 0.0;
  each([&](int xw, const float (&pv)[4], const float (&av)[4], const float (&bv)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bad |= __builtin_amdgcn_classf(pv[i], 0x21F) | __builtin_amdgcn_classf(av[i], 0x21F);
      if (kTwo) bad |= __builtin_amdgcn_classf(bv[i], 0x21F);
      const uint32_t w = token(xw, i) < n ? rank_word(pv[i], av[i], bv[i]) : ~0u;
      if (w < w_min) {  // a thread's tokens come in the order of their ids
        w_min = w;
        id_min = token(xw, i);
      }
      A += (double)av[i];
      if (kTwo) Bm += (double)bv[i];
    }
  });
  bad = __builtin_amdgcn_ballot_w64(bad) != 0;
  if (lane == 0) red[wid] = bad ? 1 : 0;
  // the wave's first kMaxS composites
  const uint64_t mine = (uint64_t)w_min << 32 | (uint32_t)id_min;
  int rank = 0;
#pragma unroll 8
  for (int l = 0; l < 64; ++l) {
    const uint64_t o = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)w_min, l) << 32 |
                       (uint32_t)__builtin_amdgcn_readlane(id_min, l);
    rank += o < mine || (o == mine && l < lane) ? 1 : 0;
  }
  if (rank < kMaxS) top[wid * kMaxS + rank] = mine;
  __syncthreads();
  int any = 0;
#pragma unroll
  for (int w = 0; w < kRankWaves; ++w) any |= red[w];
  if (any) {
    flag_row(b, V, s, rb, omega1, hdr, row_status, kRowBadProb);
    return;
  }
  if (tid < kRankWaves * kMaxS) {
    const uint64_t k = top[tid];
    int at = 0;
#pragma unroll 8
    for (int j = 0; j < kRankWaves * kMaxS; ++j) at += top[j] < k || (top[j] == k && j < tid) ? 1 : 0;
    if (at == s - 1) s_bound = k;
  }
  __syncthreads();
  const uint64_t bound = s_bound;
  const bool owner = w_min != ~0u && mine <= bound;
  if (owner) {
    A = Bm = 0.0;
    for (int xw = wid * 256; xw < n; xw += kSortStep) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int x = token(xw, i);
        if (x >= n) continue;
        const float av = ab[x], bv = bb[x];
        const uint64_t c = composite(pb[x], av, bv, x);
        if (c <= bound) {
          const int e = atomicAdd(&s_n, 1);
          if (e < kHalfList) {
            key[e] = c;
            mass[e] = make_float2(av, bv);
          }
        } else {
          A += (double)av;
          if (kTwo) Bm += (double)bv;
        }
      }
    }
  }
  __syncthreads();
  const int cands = s_n;
  uint64_t last;  // Omega_1: the composites up to it
  if (cands <= kHalfList) {
    if (tid < cands) {
      const uint64_t k = key[tid];
      int at = 0;
      for (int j = 0; j < cands; ++j) at += key[j] < k ? 1 : 0;
      sorted[at] = k;
      sorted_mass[at] = mass[tid];
    }
    __syncthreads();
    A = block_sum(A, sa);
    if (kTwo) Bm = block_sum(Bm, sa);
    for (int t = se; t < cands; ++t) {
      A += (double)sorted_mass[t].x;
      if (kTwo) Bm += (double)sorted_mass[t].y;
    }
    last = sorted[se - 1];
    if (tid < s) omega1[b * s + tid] = tid < se ? (int32_t)(uint32_t)sorted[tid] : -1;
  } else {
    last = 0;
    for (int t = 0; t < se; ++t) {  // the next composite in order
      uint64_t next = ~0ull;
      each([&](int xw, const float (&pv)[4], const float (&av)[4], const float (&bv)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint64_t c = token(xw, i) < n ? composite(pv[i], av[i], bv[i], token(xw, i)) : ~0ull;
          if (c < next && (t == 0 || c > last)) next = c;
        }
      });
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        const uint64_t o = __shfl_xor(next, off, 64);
        next = o < next ? o : next;
      }
      if (lane == 0) top[wid] = next;
      __syncthreads();
      last = top[0];
#pragma unroll
      for (int w = 1; w < kRankWaves; ++w) last = top[w] < last ? top[w] : last;
      __syncthreads();
      if (tid == 0) omega1[b * s + t] = (int32_t)(uint32_t)last;
    }
    if (tid >= se && tid < s) omega1[b * s + tid] = -1;
    A = Bm = 0.0;
    each([&](int xw, const float (&pv)[4], const float (&av)[4], const float (&bv)[4]) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (token(xw, i) < n && composite(pv[i], av[i], bv[i], token(xw, i)) > last) {
          A += (double)av[i];
          if (kTwo) Bm += (double)bv[i];
        }
    });
    A = block_sum(A, sa);
    if (kTwo) Bm = block_sum(Bm, sa);
  }
  if (!kTwo) Bm = A;
  // r(k) = q1 q2 + (q2 (A - q1) + q1 (B - q2)) / 2 = (q2 A + q1 B) / 2 on Omega_2 (Omega_1's comes with the
  // linear program)
  double acc = 0.0;
  const bool check = owner || cands > kHalfList;  // the thread may hold Omega_1 tokens
  each([&](int xw, const float (&pv)[4], const float (&av)[4], const float (&bv)[4]) {
    float out[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double rv = 0.5 * ((double)bv[i] * A + (double)av[i] * Bm);
      out[i] = (float)rv;
      double m = fmin((double)pv[i], rv);
      if (check && composite(pv[i], av[i], bv[i], token(xw, i)) <= last) m = 0.0;
      acc += m;
    }
    row_store4(rb, xw, lane, V, out);
  });
  acc = block_sum(acc, sa);
  if (tid == 0) {
    TlpHdr h = {};
    h.s_eff = se;
    h.a_tail = A;
    h.b_tail = Bm;
    h.tail_accept = acc;
    hdr[b] = h;
  }
}

// ------------------------------------------------------------------------ LP
__device__ __forceinline__ double pick(const double (&v)[kMaxS], int j) {
  double t = 0.0;
#pragma unroll
  for (int k = 0; k < kMaxS; ++k)
    if (k == j) t = v[k];
  return t;
}
__device__ __forceinline__ void add_at(double (&v)[kMaxS], int j, double d) {
#pragma unroll
  for (int k = 0; k < kMaxS; ++k)
    if (k == j) v[k] += d;
}

// One wave per row; lane x < s_eff holds Omega_1 token x.  Lane y keeps column
// y of the allocation: col[x] = share of pair {x, y} currently credited to x.
__global__ __launch_bounds__(64) void tlp_lp_kernel(const float* __restrict__ p, const float* __restrict__ q1,
                                                    const float* __restrict__ q2, int64_t V, int s,
                                                    const TlpHdr* __restrict__ hdr, const int32_t* __restrict__ omega1,
                                                    float* __restrict__ r, double* __restrict__ w,
                                                    double* __restrict__ accept, int32_t* __restrict__ row_status) {
  __shared__ double W[kMaxS][kMaxS];
  const int64_t b = blockIdx.x;
  const int lane = threadIdx.x;
  const TlpHdr h = hdr[b];
  double* wb = w + b * (int64_t)s * s;
  if (h.flags) {
    for (int i = lane; i < s * s; i += 64) wb[i] = __longlong_as_double(0x7ff8000000000000ll);
    if (lane == 0 && accept) accept[b] = __longlong_as_double(0x7ff8000000000000ll);
    return;
  }
  const int se = h.s_eff;
  const bool mine = lane < se;
  int id = 0;
  double px = 0.0, ax = 0.0, bx = 0.0;
  if (mine) {
    id = omega1[b * s + lane];
    px = (double)p[b * V + id];
    ax = (double)q1[b * V + id];
    bx = (double)q2[b * V + id];
  }
  const double c = ax * bx + bx * h.a_tail + ax * h.b_tail;
  double mc[kMaxS], col[kMaxS];
  double load = c;
#pragma unroll
  for (int v = 0; v < kMaxS; ++v) {
    const double av = __shfl(ax, v, 64), bv = __shfl(bx, v, 64);
    mc[v] = (mine && v < se && v != lane) ? av * bx + ax * bv : 0.0;  // m[v][lane] = m[lane][v]
    col[v] = v < lane ? mc[v] : 0.0;                                    // earlier-ranked token first
    if (v > lane) load += mc[v];
  }
  double ex = mine ? load - px : 0.0;
  bool capped = false;
  for (int iter = 0;; ++iter) {
    const uint64_t src = __ballot(mine && ex > 0.0);
    const uint64_t dst = __ballot(mine && ex < 0.0);
    if (!src || !dst) break;
    if (iter >= kLpMaxIter) {
      capped = true;
      break;
    }
    // breadth-first search from every surplus token over edges x -> y with col_y[x] > 0
    int parent = -1;
    uint64_t visited = src, frontier = src;
    int found = -1;
    while (frontier) {
      bool got = false;
      if (mine && !((visited >> lane) & 1ull)) {
#pragma unroll
        for (int v = 0; v < kMaxS; ++v)
          if (!got && ((frontier >> v) & 1ull) && col[v] > 0.0) {
            parent = v;
            got = true;
          }
      }
      const uint64_t nf = __ballot(got);
      visited |= nf;
      const uint64_t hit = nf & dst;
      if (hit) {
        found = __ffsll((long long)hit) - 1;
        break;
      }
      frontier = nf;
    }
    if (found < 0) break;
    double delta = -__shfl(ex, found, 64);
    int u = found;
    for (int step = 0; step < kMaxS; ++step) {
      const int v = __shfl(parent, u, 64);
      if (v < 0) break;
      delta = fmin(delta, __shfl(pick(col, v), u, 64));
      u = v;
    }
    const int source = u;
    delta = fmin(delta, __shfl(ex, source, 64));
    u = found;
    for (int step = 0; step < kMaxS; ++step) {
      const int v = __shfl(parent, u, 64);
      if (v < 0) break;
      if (lane == u) add_at(col, v, -delta);
      if (lane == v) add_at(col, u, delta);
      u = v;
    }
    if (lane == source) ex -= delta;
    if (lane == found) ex += delta;
  }
  // selection table: W[x][y] = Pr(Y = x | drafted pair {x, y}), either order
  if (mine) {
#pragma unroll
    for (int x = 0; x < kMaxS; ++x) {
      if (x < lane) {
        double wv = mc[x] > 0.0 ? col[x] / mc[x] : 1.0;
        wv = fmin(1.0, fmax(0.0, wv));
        W[x][lane] = wv;
        W[lane][x] = 1.0 - wv;
      }
    }
    W[lane][lane] = 1.0;
  }
  __syncthreads();
  for (int i = lane; i < s * s; i += 64) {
    const int x = i / s, y = i % s;
    wb[i] = (x < se && y < se) ? W[x][y] : 0.0;
  }
  double rv = c;
  if (mine) {
#pragma unroll
    for (int y = 0; y < kMaxS; ++y)
      if (y < se && y != lane) rv += mc[y] * W[lane][y];
    r[b * V + id] = (float)rv;
  }
  const double obj = wave_sum(mine ? fmin(px, rv) : 0.0);
  if (lane == 0) {
    if (accept) accept[b] = h.tail_accept + obj;
    if (capped && row_status) row_status[b] |= kRowLpLimit;
  }
}

// ------------------------------------------------------------------ selection
__global__ __launch_bounds__(256) void tlp_select_kernel(
    const float* __restrict__ p, const float* __restrict__ q1, const float* __restrict__ q2,
    const int32_t* __restrict__ drafts, const float* __restrict__ u, uint64_t seed, uint64_t offset, int64_t B,
    int64_t V, int s, int tail, const int32_t* __restrict__ omega1, const double* __restrict__ w,
    int32_t* __restrict__ sel_index, int32_t* __restrict__ sel_token, int32_t* __restrict__ row_status) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const int32_t x1 = drafts[b * 2], x2 = drafts[b * 2 + 1];
  int st = 0;
  if (omega1[b * s] < 0) {
    st = kRowBadProb;  // the plan flagged this row
  } else if (x1 < 0 || (int64_t)x1 >= V || x2 < 0 || (int64_t)x2 >= V) {
    st = kRowBadDraft;
  } else if (!(q1[b * V + x1] > 0.0f) || !(q2[b * V + x2] > 0.0f)) {
    st = kRowBadDraft;
  }
  if (st) {
    sel_index[b] = -1;
    sel_token[b] = -1;
    if (row_status) row_status[b] |= st;
    return;
  }
  float uu[3];
  position_uniforms(u, seed, offset, b, uu);
  int idx = 0;
  if (x1 != x2) {
    int i1 = -1, i2 = -1;
    for (int t = 0; t < s; ++t) {
      const int32_t o = omega1[b * s + t];
      if (o == x1) i1 = t;
      if (o == x2) i2 = t;
    }
    double f;
    if (i1 >= 0 && i2 >= 0) {
      const double* wb = w + b * (int64_t)s * s;
      f = i1 < i2 ? wb[i1 * s + i2] : 1.0 - wb[i2 * s + i1];
    } else if (i1 >= 0) {
      f = 1.0;
    } else if (i2 >= 0) {
      f = 0.0;
    } else if (tail == kTailHalf) {
      f = 0.5;
    } else {
      const uint32_t k1 = rank_word(p[b * V + x1], q1[b * V + x1], q2[b * V + x1]);
      const uint32_t k2 = rank_word(p[b * V + x2], q1[b * V + x2], q2[b * V + x2]);
      f = (k1 < k2 || (k1 == k2 && x1 < x2)) ? 1.0 : 0.0;
    }
    idx = (double)uu[0] < f ? 0 : 1;
  }
  sel_index[b] = idx;
  sel_token[b] = idx == 0 ? x1 : x2;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

size_t workspace_bytes_tlp(int64_t B, int64_t V, int tail) {
  size_t bytes = align256((size_t)B * sizeof(TlpHdr));
  if (tail == kTailSorted) bytes += rank_workspace_bytes(B, V);
  return bytes;
}

hipError_t launch_tlp(const float* p, const float* q1, const float* q2, int64_t B, int64_t V, int s, int tail,
                      float* r, int32_t* omega1, double* w, double* accept, int32_t* row_status, void* workspace,
                      hipStream_t st) {
  if (!q2) q2 = q1;
  char* base = static_cast<char*>(workspace);
  TlpHdr* hdr = reinterpret_cast<TlpHdr*>(base);
  base += align256((size_t)B * sizeof(TlpHdr));
  if (tail == kTailSorted) {
    TlpSpec::Args args = {p, q1, q2, r, omega1, hdr, row_status, s};
    const RankPlanes planes = carve_rank_planes(base, B, V);
    uint32_t* later = planes.bins.word;  // a row's first word: read before the ranking writes there
    const dim3 grid((unsigned)B), block(kRankThreads);
    if (V <= kSortHold * kSortStep)
      hipLaunchKernelGGL(tlp_sort_kernel<true>, grid, block, 0, st, args, V, planes.bins.v0, planes.bins.v1, later);
    else if (V <= kSortMaxV)
      hipLaunchKernelGGL(tlp_sort_kernel<false>, grid, block, 0, st, args, V, planes.bins.v0, planes.bins.v1, later);
    else
      later = nullptr;
    hipLaunchKernelGGL(rank_scan_kernel<TlpSpec>, grid, block, 0, st, args, V, planes, later);
  } else {
    if (q2 == q1)
      hipLaunchKernelGGL(tlp_rank_half_kernel<false>, dim3((unsigned)B), dim3(kRankThreads), 0, st, p, q1, q1, V, s, r,
                         omega1, hdr, row_status);
    else
      hipLaunchKernelGGL(tlp_rank_half_kernel<true>, dim3((unsigned)B), dim3(kRankThreads), 0, st, p, q1, q2, V, s, r,
                         omega1, hdr, row_status);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(tlp_lp_kernel, dim3((unsigned)B), dim3(64), 0, st, p, q1, q2, V, s, hdr, omega1, r, w, accept,
                     row_status);
  return hipGetLastError();
}

hipError_t launch_select_tlp(const float* p, const float* q1, const float* q2, const int32_t* drafts, const float* u,
                             uint64_t seed, uint64_t offset, int64_t B, int64_t V, int s, int tail,
                             const int32_t* omega1, const double* w, int32_t* sel_index, int32_t* sel_token,
                             int32_t* row_status, hipStream_t st) {
  if (!q2) q2 = q1;
  const unsigned blocks = (unsigned)((B + 255) / 256);
  hipLaunchKernelGGL(tlp_select_kernel, dim3(blocks), dim3(256), 0, st, p, q1, q2, drafts, u, seed, offset, B, V, s,
                     tail, omega1, w, sel_index, sel_token, row_status);
  return hipGetLastError();
}

}  // namespace mdss
