// Statistics of the deleted value rows of a head (see del_stats_mfma.hip, whose output format this shares) for the shapes that
// kernel does not take: fp32 caches and head_dim 64.  Values enter the matrix cores as single precision
// (v_mfma_f32_32x32x2_f32): products and sums are fp32.
//
// An operand of that instruction holds, in lane l, row l % 32 and k = l / 32; for V^T V the row is a column of V and k a token, so
// a lane's operand is V[t + l/32][32 b + l%32] - a coalesced load straight from memory, with no staging.  A workgroup takes a chunk
// of 1024 tokens, its eight waves every eighth pair of tokens for all tiles of the lower triangle, and the waves' accumulators meet
// in LDS at the end, tile by tile, in wave order.  Bound by the matrix instructions (ten per pair of tokens at head_dim 128, three at
// 64) and, for the few workgroups of a small call, by the latency of the loads, which run one batch ahead.
// Before, 16 x 16 threads kept 8 x 8 accumulators with a head_dim known only at run time (in scratch memory) and 256 threads shared a
// chunk: 1.37 ms for 2 heads x 512 tokens of fp32 at head_dim 64, most of a 1.92 ms call that takes 0.59 ms now.
#pragma once
#include "common.hpp"

namespace obf {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float dg_f32x16;

constexpr int DG_THREADS = 512;
constexpr int DG_WAVES = DG_THREADS / 64;
constexpr int DG_STEP = 2 * DG_WAVES;    // tokens per iteration of a workgroup

struct DgShared {
  double tred[DG_WAVES];
  uint32_t kept[kStatChunk / 32];                        // bitmap of the retained tokens of the chunk
  float wt[kStatChunk];                                  // score of a deleted token
  float red[DG_WAVES][1024];                             // one tile per wave; then the waves' column sums
};

// One chunk of one head (the whole workgroup).
template <typename T, int D>
__device__ __forceinline__ void dg_chunk(const T* __restrict__ V, const float* __restrict__ scores, const int32_t* __restrict__ idx, int N,
                                         int max_budget, int nstat, const HeadState* __restrict__ state,
                                         const int32_t* __restrict__ n_keep /*non-null: do not read the head states*/,
                                         float* __restrict__ gram_part, int scs, int kvs, int head, int chunk, DgShared& sh) {
  constexpr int DB = D / 32;                           // 32-column blocks
  constexpr int NT = DB * (DB + 1) / 2;                // tiles on and below the diagonal
  constexpr int U = 16 / DB;                           // iterations whose loads travel together (16 loads per lane)
  const int n = n_keep ? n_keep[head] : state[head].n_keep;
  if (n_keep ? !(n > 0 && n < N) : !state[head].active) return;
  auto& kept = sh.kept;
  auto& wt = sh.wt;
  auto& red = sh.red;
  auto& tred = sh.tred;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lh = lane >> 5;
  const int32_t* id = idx + (size_t)head * max_budget;
  const T* Vh = V + (size_t)head * kvs * D;
  const float* sc = scores + (size_t)head * scs;
  const int t0 = chunk * kStatChunk, rows = min(N - t0, kStatChunk);

  T pre[U][DB];
  auto fetch = [&](int r0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const T* p = Vh + (size_t)(t0 + min(r0 + u * DG_STEP + 2 * wave + lh, rows - 1)) * D + lr;   // clamped: masked below
#pragma unroll
      for (int b = 0; b < DB; ++b) pre[u][b] = p[b * 32];
    }
  };
  fetch(0);
  if (tid < kStatChunk / 32) kept[tid] = 0u;
  __syncthreads();
  for (int i = tid; i < n; i += DG_THREADS) {
    const int j = id[i] - t0;
    if (j >= 0 && j < rows) atomicOr(&kept[j >> 5], 1u << (j & 31));
  }
  for (int i = tid; i < kStatChunk; i += DG_THREADS) wt[i] = (i < rows) ? sc[t0 + i] : 0.f;
  __syncthreads();

  dg_f32x16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
  float u_sum[DB], s_sum[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b) { u_sum[b] = 0.f; s_sum[b] = 0.f; }
  for (int r0 = 0; r0 < rows; r0 += U * DG_STEP) {
    float v[U][DB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = r0 + u * DG_STEP + 2 * wave + lh;
      const bool del = r < rows && !((kept[(r >> 5) & (kStatChunk / 32 - 1)] >> (r & 31)) & 1u);
#pragma unroll
      for (int b = 0; b < DB; ++b) v[u][b] = del ? Elem<T>::load(&pre[u][b]) : 0.f;
    }
    fetch(r0 + U * DG_STEP);                             // past the end: the last row again, not used
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float w = wt[(r0 + u * DG_STEP + 2 * wave + lh) & (kStatChunk - 1)];
#pragma unroll
      for (int b = 0; b < DB; ++b) { u_sum[b] = fmaf(w, v[u][b], u_sum[b]); s_sum[b] += v[u][b]; }
#pragma unroll
      for (int rb = 0; rb < DB; ++rb)
#pragma unroll
        for (int cb = 0; cb <= rb; ++cb)
          acc[rb * (rb + 1) / 2 + cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[u][rb], v[u][cb], acc[rb * (rb + 1) / 2 + cb], 0, 0, 0);
    }
  }

  // entry i of lane l of a tile is G[32 rb + (i/4)*8 + (l/32)*4 + i%4][32 cb + l%32]
  float* out = gram_part + ((size_t)head * nstat + chunk) * gram_stride(D);
  double tr = 0.0;                                       // this thread's share of the trace (the squared norms)
#pragma unroll
  for (int rb = 0; rb < DB; ++rb) {
#pragma unroll
    for (int cb = 0; cb <= rb; ++cb) {
      const int t = rb * (rb + 1) / 2 + cb;
#pragma unroll
      for (int i = 0; i < 16; ++i) red[wave][i * 64 + lane] = acc[t][i];
      __syncthreads();
      for (int e = tid; e < 1024; e += DG_THREADS) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < DG_WAVES; ++w) s += red[w][e];
        const int i = e >> 6, row = (i >> 2) * 8 + ((e >> 5) & 1) * 4 + (i & 3), col = e & 31;
        out[(rb * 32 + row) * D + cb * 32 + col] = s;
        if (rb == cb && row == col) tr += (double)s;
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int b = 0; b < DB; ++b) {                         // red[w][(2 h + lh) * D + column]: weighted (h = 0) and plain sums of the wave's half lh
    red[wave][lh * D + b * 32 + lr] = u_sum[b];
    red[wave][(2 + lh) * D + b * 32 + lr] = s_sum[b];
  }
  for (int off = 32; off > 0; off >>= 1) tr += __shfl_xor(tr, off);
  if (lane == 0) tred[wave] = tr;
  __syncthreads();
  if (tid < 2 * D) {
    const int h = tid / D, c = tid - h * D;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < DG_WAVES; ++w) s += red[w][2 * h * D + c] + red[w][(2 * h + 1) * D + c];
    out[D * D + h * D + c] = s;
  }
  if (tid == 0) {
    double s = 0.0;
    for (int w = 0; w < DG_WAVES; ++w) s += tred[w];
    out[D * D + 2 * D] = (float)s;
  }
}

}  // namespace obf
