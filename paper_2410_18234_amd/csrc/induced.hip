// Entry points of the induced distribution without the quadrature calls' limits (any fp32 row, any
// weight range): K = 2 and K = 3 i.i.d. drafts, two draft laws, successive pairwise stages, all by
// the bucketed quadrature (bucket.hip), whose error (7.1e-9 of an entry at most) is below r's fp32 rounding.
//
// The O(n^2) pair sums this replaced (chunks of poles as rational functions, contracted on the bf16
// matrix cores) took 6.6 ms at 256 x 32000, 2.4e-8 to 5e-8 off in the 2-norm, against 44 us and
// 2.4e-8; the O(n^3) triple sums of K = 3 at 256 x 32000 with 1024 support tokens 6.9 ms against
// 40 us.
#include "common.h"

namespace mdss {

namespace {

// K = 2 keeps the 44 bytes a token that its callers hold buffers for, far more than the chunks' sums and polynomials
// need (workspace_bytes_expsum).
constexpr int64_t kPad = 128;

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace

size_t workspace_bytes(int64_t B, int64_t V, int K, int s_max) {
  (void)s_max;  // K = 3: a row takes the same room whatever its support
  if (K != 2) return workspace_bytes_expsum(B, V, 1);
  const size_t tokens = (size_t)B * (size_t)((V + kPad - 1) / kPad * kPad);
  return align256(32 * (size_t)B) + 3 * align256(4 * tokens) + align256(32 * tokens);
}

hipError_t launch_induced(const float* p, const float* q, int64_t B, int64_t V, int K, int s_max, float* r,
                          int32_t* row_status, void* workspace, hipStream_t st) {
  return launch_bucket(p, q, nullptr, B, V, K, K == 3 ? s_max : 0, false, r, row_status, false, nullptr, workspace,
                       workspace_bytes(B, V, K, s_max), st);
}

size_t workspace_bytes_pair(int64_t B, int64_t V) {
  return 2 * workspace_bytes(B, V, 2, 0) + 2 * align256(sizeof(double) * B * V);
}

hipError_t launch_induced_pair(const float* p, const float* q1, const float* q2, int64_t B, int64_t V, float* r,
                               int32_t* row_status, void* workspace, hipStream_t st) {
  return launch_bucket(p, q1, q2, B, V, 2, 0, false, r, row_status, false, nullptr, workspace,
                       workspace_bytes_pair(B, V), st);
}

// Successive pairwise reduction (Remark 4): r_1 = the K = 2 law of (q, q),
// r_j = the law of a pair drawn from (r_{j-1}, q), each stage read back in fp32.
hipError_t launch_induced_successive(const float* p, const float* q, int64_t B, int64_t V, int K, float* r_stages,
                                     int32_t* row_status, void* workspace, hipStream_t st) {
  hipError_t e = launch_induced(p, q, B, V, 2, 0, r_stages, row_status, workspace, st);
  const int64_t plane = B * V;
  for (int j = 1; j < K - 1 && e == hipSuccess; ++j)
    e = launch_induced_pair(p, r_stages + (j - 1) * plane, q, B, V, r_stages + j * plane, row_status, workspace, st);
  return e;
}

}  // namespace mdss
