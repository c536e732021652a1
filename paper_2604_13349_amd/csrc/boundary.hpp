// Exact re-decision of the tokens at the selection threshold, shared by the standalone refinement kernel and by the
// fused select+refine kernel so that both take bit-identical decisions.
#pragma once
#include "f64_tile.hpp"

namespace obf {

// Exact (double) attention mass of each band token, sixteen tokens against sixteen query rows at a time on the double-precision matrix
// instructions: a wave takes every WAVES-th block of rows, leaves the block's sixteen column sums in LDS, and a thread per token adds
// the blocks in order - the order of the additions does not depend on the number of waves, and tokens with equal keys get equal masses.
// With a wave per token and the products as scalar double-precision multiply-adds this was 46k of the 103k cycles of a selection
// workgroup on 16384 tokens x 320 rows.  All threads call; `part` is LDS scratch; ends with a barrier.
constexpr int kRescoreBlocks = 32;       // row blocks per round of the scratch
struct RescoreScratch { double part[kRescoreBlocks][16]; };

template <typename T, int WAVES, int D>
__device__ __forceinline__ void rescore_band_d(const T* __restrict__ Kh, const T* __restrict__ Qh, const double* __restrict__ lse, int R,
                                               const int* band, int nband, double* band_score, RescoreScratch& rs) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double scale = 1.0 / sqrt((double)D);
  const int nblk = (R + 15) >> 4;
  for (int b0 = 0; b0 < nband; b0 += 16) {
    RowPart<T, D> kp;
    kp.load(Kh + (size_t)band[min(b0 + (lane & 15), nband - 1)] * D, lane);        // tokens past the band: the last one again, not written
    double sum = 0.0;
    for (int c0 = 0; c0 < nblk; c0 += kRescoreBlocks) {
      const int nc = min(kRescoreBlocks, nblk - c0);
      for (int c = wave; c < nc; c += WAVES) {
        const int r0 = (c0 + c) * 16;
        RowPart<T, D> qp;
        qp.load(Qh + (size_t)min(r0 + (lane & 15), R - 1) * D, lane);
        double l[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) { const int r = r0 + (lane >> 4) + 4 * i; l[i] = (r < R) ? lse[r] : 0.0; }
        // (the token's entries are converted again for every block: kept as doubles they would take D / 2 registers)
#pragma unroll
        for (int i = 0; i < RowPart<T, D>::NV; ++i) asm volatile("" : "+v"(kp.v[i].x), "+v"(kp.v[i].y), "+v"(kp.v[i].z), "+v"(kp.v[i].w));
        f64x4 x = {0.0, 0.0, 0.0, 0.0}, y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < D / 4; s += 2) {
          x = __builtin_amdgcn_mfma_f64_16x16x4f64(qp.at(s), kp.at(s), x, 0, 0, 0);
          y = __builtin_amdgcn_mfma_f64_16x16x4f64(qp.at(s + 1), kp.at(s + 1), y, 0, 0, 0);
          if ((s & 7) == 6) __builtin_amdgcn_sched_barrier(0);           // conversions stay near their use
        }
        x += y;
        double col = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) if (r0 + (lane >> 4) + 4 * i < R) col += exp(x[i] * scale - l[i]);
        col += __shfl_xor(col, 16);
        col += __shfl_xor(col, 32);
        if (lane < 16) rs.part[c][lane] = col;
      }
      __syncthreads();
      if (threadIdx.x < 16) for (int c = 0; c < nc; ++c) sum += rs.part[c][threadIdx.x];
      __syncthreads();
    }
    if (threadIdx.x < 16 && b0 + (int)threadIdx.x < nband) band_score[b0 + threadIdx.x] = sum;
  }
  __syncthreads();
}

template <typename T, int WAVES>
__device__ __forceinline__ void rescore_band(const T* __restrict__ Kh, const T* __restrict__ Qh, const double* __restrict__ lse, int d, int R,
                                             const int* band, int nband, double* band_score, RescoreScratch& rs) {
  if (d == 128) rescore_band_d<T, WAVES, 128>(Kh, Qh, lse, R, band, nband, band_score, rs);
  else rescore_band_d<T, WAVES, 64>(Kh, Qh, lse, R, band, nband, band_score, rs);
}

// Thread u < nband: is band token u among the nkb best (exact score descending, index ascending; band[] is ascending)?
__device__ __forceinline__ int band_keeps(const double* band_score, int nband, int nkb, int u) {
  const double mine = band_score[u];
  int rank = 0;
  for (int v = 0; v < nband; ++v) {
    const double o = band_score[v];
    rank += (o > mine) || (o == mine && v < u);
  }
  return rank < nkb;
}

}  // namespace obf
