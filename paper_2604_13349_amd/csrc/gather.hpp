// Gather of the retained rows (the gather step of Alg. 2): K_out = K[idx], V_out = V[idx], bit copies in
// 16-byte pieces; rows past n_keep are zero-filled so the padded output is deterministic.
#pragma once
#include "common.hpp"

namespace obf {

constexpr int GA_UNROLL = 4;             // rows per thread

// workgroups of NT threads per head
template <int NT>
inline int ga_blocks(int max_budget, int row_bytes) {
  const int rows = GA_UNROLL * NT / (row_bytes / 16);
  return (max_budget + rows - 1) / rows;
}

// Workgroup `block` of the `blocks` of a head.  s_red: NT / 64 floats of LDS, for fro_part only.
template <int NT>
__device__ __forceinline__ void ga_rows(const uint4* __restrict__ K, const uint4* __restrict__ V, const int32_t* __restrict__ idx,
                                        const int32_t* __restrict__ n_keep, int kvs /*tokens per head in K, V*/, int row_vec /*uint4 per row*/,
                                        int max_budget, uint4* __restrict__ K_out, uint4* __restrict__ V_out,
                                        double* __restrict__ fro_part /*bf16 rows of 256 bytes only*/, int head, int block, int blocks, float* s_red) {
  const int rows_per_pass = NT / row_vec;
  const int r0 = block * rows_per_pass * GA_UNROLL + threadIdx.x / row_vec;
  const int c = threadIdx.x % row_vec;
  const int n = n_keep[head];
  // GA_UNROLL rows per thread, all loads issued before the first store
  int j[GA_UNROLL];
#pragma unroll
  for (int u = 0; u < GA_UNROLL; ++u) {
    const int r = r0 + u * rows_per_pass;
    j[u] = (r < n && r < max_budget) ? idx[(size_t)head * max_budget + r] : -1;
  }
  uint4 kv[GA_UNROLL], vv[GA_UNROLL];
#pragma unroll
  for (int u = 0; u < GA_UNROLL; ++u) {
    kv[u] = make_uint4(0, 0, 0, 0); vv[u] = make_uint4(0, 0, 0, 0);
    if (j[u] >= 0) {
      const size_t s = ((size_t)head * kvs + j[u]) * row_vec + c;
      if (K_out) kv[u] = K[s];
      if (V_out) vv[u] = V[s];
    }
  }
#pragma unroll
  for (int u = 0; u < GA_UNROLL; ++u) {
    const int r = r0 + u * rows_per_pass;
    if (r < max_budget) {
      const size_t o = ((size_t)head * max_budget + r) * row_vec + c;
      if (K_out) K_out[o] = kv[u];
      if (V_out) V_out[o] = vv[u];
    }
  }
  if (fro_part) {
    // sum of squares of this workgroup's V rows (zero for the padding), in a fixed order
    float sq = 0.f;
#pragma unroll
    for (int u = 0; u < GA_UNROLL; ++u) {
      const uint32_t w4[4] = {vv[u].x, vv[u].y, vv[u].z, vv[u].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float a = __uint_as_float(w4[i] << 16), b = __uint_as_float(w4[i] & 0xffff0000u);
        sq = fmaf(a, a, sq); sq = fmaf(b, b, sq);
      }
    }
    for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0)
      fro_part[(size_t)head * blocks + block] = ((double)s_red[0] + (double)s_red[1]) + ((double)s_red[2] + (double)s_red[3]);
  }
}

}  // namespace obf
