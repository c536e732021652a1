// What the matrix-core score kernels (score_mfma.hip, score_tall.hip) share.
#pragma once
#include "common.hpp"

namespace obf {

// v_exp_f32, denormal results flush to 0
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

template <int AHEAD>
__device__ __forceinline__ double fold_row_lse_by(const double2* __restrict__ p, const size_t stride, const int n) {
  double M = -INFINITY, L = 0.0;
  for (int s0 = 0; s0 < n; s0 += AHEAD) {
    double2 v[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) v[i] = p[(size_t)min(s0 + i, n - 1) * stride];
    double m = M;
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) m = fmax(m, v[i].x);
    if (M != -INFINITY) L *= exp(M - m);
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) if (s0 + i < n && v[i].x != -INFINITY) L += v[i].y * exp(v[i].x - m);
    M = m;
  }
  return M + log(L);
}

// The log-sum-exp of a query row from the partials (max, sum-exp) that the n ranges of its head left, `stride` double2 apart: eight at a time, whose
// loads travel together (one by one they cost a memory latency each, which a head that is spread over many ranges feels), or the two at most that a
// head has where heads are many (second pass, 288 heads of 256 tokens, 160, 448 and 640 rows: 20.1, 41.7, 53.2 us by eight, 19.4, 40.1, 51.3 by two).
__device__ __forceinline__ double fold_row_lse(const double* __restrict__ part, const size_t stride, const int n) {
  return n <= 2 ? fold_row_lse_by<2>((const double2*)part, stride, n) : fold_row_lse_by<8>((const double2*)part, stride, n);
}

}  // namespace obf
