// What the matrix-core score kernels (score_mfma.hip, score_tall.hip) share.
#pragma once
#include "common.hpp"

namespace obf {

// v_exp_f32, denormal results flush to 0
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// The log-sum-exp of a query row from the partials (max, sum-exp) that the n ranges of its head left, `stride` double2 apart: eight at a time, whose
// loads travel together (one by one they cost a memory latency each, which a head that is spread over many ranges feels).
__device__ __forceinline__ double fold_row_lse(const double* __restrict__ part, const size_t stride, const int n) {
  const double2* p = (const double2*)part;
  double M = -INFINITY, L = 0.0;
  for (int s0 = 0; s0 < n; s0 += 8) {
    double2 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = p[(size_t)min(s0 + i, n - 1) * stride];
    double m = M;
#pragma unroll
    for (int i = 0; i < 8; ++i) m = fmax(m, v[i].x);
    if (M != -INFINITY) L *= exp(M - m);
#pragma unroll
    for (int i = 0; i < 8; ++i) if (s0 + i < n && v[i].x != -INFINITY) L += v[i].y * exp(v[i].x - m);
    M = m;
  }
  return M + log(L);
}

}  // namespace obf
