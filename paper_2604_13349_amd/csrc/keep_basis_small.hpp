// Retained-span basis (Eq. 2) for heads with at most head_dim retained rows: the budget is below the
// head dimension, so the span always leaves a complement and Orthogonal BackFill (Sec. 4.4) is active.
//
// Per head one workgroup, everything in double precision.  Ordinary heads take a blocked factorisation (ks_chol_head below); heads whose
// rows are dependent or nearly so take the pivoted loop (ks_head; 16 x 32 threads):
//   C = A A^T, the n x n Gram matrix of the retained rows A (entries of A are exact in float; products and
//       sums are taken in double), kept in registers (thread (ty, tx) owns C[ty + 16a][tx + 32b]; a single-precision
//       copy in LDS serves the power iteration only);
//   sigma_max^2 = lambda_max(C) by power iteration (the rank rule's threshold);
//   pivoted Gram-Schmidt on the rows of A, which live in registers (thread (ty, tx) owns A[ty + 16a][tx*CW ..]):
//       the pivot is the row with the largest remaining squared norm, read off the diagonal of C; the
//       projection coefficients of all rows onto the new direction are row j of C over sqrt(C[j][j]), so a
//       step is one rank-1 update of C and one of A, both in registers (no inner products; the owners of row j publish
//       it, two barriers);
//   rows whose remaining norm is at or below sigma_max * max(n, d) * 2^-23 end the loop: r = number of steps.
// Row s of the basis is written as soon as it is final.
#pragma once
#include "common.hpp"
#include "wave_ops.hpp"

namespace obf {

constexpr int KS_THREADS = 512;
constexpr int KS_WAVES = KS_THREADS / 64;
constexpr double kRankEpsKs = 1.1920928955078125e-07;   // 2^-23, the rank rule's epsilon

__device__ __forceinline__ double ks_block_sum(double v, double* red /*[KS_WAVES]*/) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < KS_WAVES; ++i) s += red[i];
  return s;
}

template <typename T, int CW> struct RowLoad;
template <> struct RowLoad<uint16_t, 2> {
  static __device__ __forceinline__ void get(const uint16_t* p, double (&o)[2]) {
    const uint32_t w = *(const uint32_t*)p;
    o[0] = (double)__uint_as_float(w << 16); o[1] = (double)__uint_as_float(w & 0xffff0000u);
  }
};
template <> struct RowLoad<uint16_t, 4> {
  static __device__ __forceinline__ void get(const uint16_t* p, double (&o)[4]) {
    const uint2 q = *(const uint2*)p;
    const uint32_t w[2] = {q.x, q.y};
#pragma unroll
    for (int i = 0; i < 2; ++i) { o[2 * i] = (double)__uint_as_float(w[i] << 16); o[2 * i + 1] = (double)__uint_as_float(w[i] & 0xffff0000u); }
  }
};
template <> struct RowLoad<float, 4> {
  static __device__ __forceinline__ void get(const float* p, double (&o)[4]) {
    const float4 q = *(const float4*)p;
    o[0] = (double)q.x; o[1] = (double)q.y; o[2] = (double)q.z; o[3] = (double)q.w;
  }
};
template <> struct RowLoad<float, 2> {
  static __device__ __forceinline__ void get(const float* p, double (&o)[2]) {
    const float2 q = *(const float2*)p;
    o[0] = (double)q.x; o[1] = (double)q.y;
  }
};

constexpr int KS_LT = 17;                // row stride of an LDS tile in doubles: operand reads (16 rows, one column) without bank conflicts
constexpr int KS_TILE = 16 * KS_LT;

__host__ __device__ inline int ks_tile(int i, int j) { return i * (i + 1) / 2 + j; }

struct KsShared {
  double red[KS_WAVES];
  float xv[128], yp[4][128];         // power iteration: iterate, partial products
  double qrow[128];                  // row j of A at a step (unscaled)
  double crow[128];                  // row j of C at a step (before the loop: the diagonal of C)
  uint32_t wkey[2][2];
  int stop;                          // the blocked factorisation leaves the head to the pivoted loop
};

// One head.  TI = ceil(n / 16) rounded up to even, CW = d / 32.  Returns r.
// C is stored padded to NP = 16 TI rows and columns (zero beyond n), so that every index below is an immediate.
// Lt: the Gram matrix as ks_chol_head leaves it, 16 x 16 tiles on and below the diagonal (LDS, behind C).
template <typename T, int TI, int CW>
__device__ __forceinline__ int ks_head(const T* __restrict__ Vh, const int32_t* __restrict__ id, int n, float* __restrict__ bh,
                       double* C, const double* Lt, KsShared& sh) {
  constexpr int d = 32 * CW;
  constexpr int TJ = TI / 2;                                   // column blocks of 32 of a thread's C elements
  constexpr int NP = 16 * TI;
  const int tid = threadIdx.x, lane = tid & 63;
  const int ty = tid >> 5, tx = tid & 31;
  float* Cf = (float*)C;                                       // [NP][NP], single-precision copy for the power iteration

  // ---- Gram matrix: thread (ty, tx) takes C[ty + 16a][tx + 32b]
  double creg[TI][TJ];
  {
    const int tc = tx & 15;
#pragma unroll
    for (int a = 0; a < TI; ++a)
#pragma unroll
      for (int b = 0; b < TJ; ++b) {
        const int bt = 2 * b + (tx >> 4);                      // tile column
        const int o = (a >= bt) ? ks_tile(a, bt) * KS_TILE + ty * KS_LT + tc : ks_tile(bt, a) * KS_TILE + tc * KS_LT + ty;
        creg[a][b] = (ty + 16 * a < n && tx + 32 * b < n) ? Lt[o] : 0.0;
      }
    __syncthreads();                                           // the tiles are read (the copy may lie over them)
#pragma unroll
    for (int a = 0; a < TI; ++a)
#pragma unroll
      for (int b = 0; b < TJ; ++b) {
        const int i = ty + 16 * a, jj = tx + 32 * b;
        Cf[i * NP + jj] = (float)creg[a][b];
        if (i == jj) sh.crow[i] = creg[a][b];
      }
    __syncthreads();
  }

  // ---- sigma_max^2 = lambda_max(C): power iteration in single precision (the estimate only sets the rank rule's
  // threshold, where a percent is immaterial).  Each quarter of the workgroup (a wave pair) takes every fourth row of
  // C for all columns, the partial products meet in LDS.  The iterate is scaled by the first step's estimate only;
  // the last step takes the true ratio.
  if (tid < 128) sh.xv[tid] = (tid < n) ? (float)(1.0 / sqrt((double)n)) * (1.f + 0.01f * (float)(tid % 7)) : 0.f;
  __syncthreads();
  double lam = 0.0;
  float scale = 1.f;
  const int prow = tid & 127, ppart = tid >> 7;                // ppart is uniform over a wave
  const bool pact = prow < NP;
  const float* cp = Cf + ppart * NP + (pact ? prow : 0);       // C symmetric: column reads are row reads
  const float* xp = sh.xv + ppart;
  constexpr int kPowerIters = 12;
  for (int it = 0; it < kPowerIters; ++it) {
    float y0 = 0.f, y1 = 0.f;
#pragma unroll
    for (int u = 0; u < NP / 4; u += 2) {
      y0 = fmaf(cp[(4 * u) * NP], xp[4 * u], y0);
      y1 = fmaf(cp[(4 * u + 4) * NP], xp[4 * u + 4], y1);
    }
    sh.yp[ppart][prow] = pact ? y0 + y1 : 0.f;
    lds_barrier();
    float y = 0.f;
    if (tid < 128) y = (sh.yp[0][tid] + sh.yp[1][tid]) + (sh.yp[2][tid] + sh.yp[3][tid]);
    if (it == 0 || it == kPowerIters - 1) {
      const float x0 = (tid < 128) ? sh.xv[tid] : 0.f;
      const double n2 = ks_block_sum((double)y * y, sh.red);
      const double d2 = ks_block_sum((double)x0 * x0, sh.red);
      lam = sqrt(n2 / fmax(d2, 1e-300));
      if (!(lam > 0.0)) break;
      scale = (float)(1.0 / lam);
    }
    if (tid < 128) sh.xv[tid] = y * scale;
    lds_barrier();
  }
  const double thr = sqrt(lam) * (double)max(n, d) * kRankEpsKs;
  const double thr2 = thr * thr;                               // pivots are squared distances

  // ---- rows of A: thread (ty, tx) owns A[ty + 16a][tx*CW ..]
  double areg[TI][CW];
  {
    int rid[TI];
#pragma unroll
    for (int a = 0; a < TI; ++a) rid[a] = id[min(ty + 16 * a, n - 1)];
#pragma unroll
    for (int a = 0; a < TI; ++a) RowLoad<T, CW>::get(Vh + (size_t)rid[a] * d + tx * CW, areg[a]);
#pragma unroll
    for (int a = 0; a < TI; ++a)
      if (ty + 16 * a >= n) {
#pragma unroll
        for (int c = 0; c < CW; ++c) areg[a][c] = 0.0;
      }
  }

  // ---- pivoted Gram-Schmidt driven by C
  double dg = (tid < n) ? sh.crow[tid] : -1.0;                 // threads < n: remaining squared norm of row tid
  bool used = false;
  // Pivot search key: the high word of the (positive) double, low 7 bits replaced by 127 - row, so that the
  // maximum over the keys is the largest remaining norm (to 13 mantissa bits), lowest row first among equals.
  auto publish = [&](int buf) {
    if (tid < 128) {
      uint32_t key = (!used && dg > 0.0) ? ((((uint32_t)(((uint64_t)__double_as_longlong(dg)) >> 32)) & ~0x7Fu) | (uint32_t)(127 - tid)) : 0u;
      key = wave_max_u32(key);
      if (lane == 0) sh.wkey[buf][tid >> 6] = key;
    }
  };
  publish(0);
  __syncthreads();
  int r = 0;
  for (int s = 0; s < n; ++s) {
    const uint32_t key = max(sh.wkey[s & 1][0], sh.wkey[s & 1][1]);
    if (key == 0u) break;
    const int j = 127 - (int)(key & 0x7Fu);
    if (ty == (j & 15)) {                                      // row j of C and of A sit in these threads, register j / 16
      double* qr = sh.qrow + tx * CW;
      double* cr = sh.crow + tx;
#define KS_ROW(k) case k: if constexpr (k < TI) { \
        _Pragma("unroll") for (int c = 0; c < CW; ++c) qr[c] = areg[k][c]; \
        _Pragma("unroll") for (int b = 0; b < TJ; ++b) cr[32 * b] = creg[k][b]; } break;
      switch (j >> 4) { KS_ROW(0) KS_ROW(1) KS_ROW(2) KS_ROW(3) KS_ROW(4) KS_ROW(5) KS_ROW(6) KS_ROW(7) default: break; }
#undef KS_ROW
    }
    lds_barrier();
    const double xjj = sh.crow[j];
    if (!(xjj > thr2)) break;                                  // the largest remaining norm is at the rank threshold (uniform)
    const double inv = rsqrt(xjj);                             // 1 / remaining norm of row j
    double la[TI];
#pragma unroll
    for (int a = 0; a < TI; ++a) la[a] = sh.crow[ty + 16 * a] * inv;     // <row, new direction>
    {
      double q[CW];
#pragma unroll
      for (int c = 0; c < CW; ++c) q[c] = sh.qrow[tx * CW + c] * inv;    // the new direction
#pragma unroll
      for (int a = 0; a < TI; ++a)
#pragma unroll
        for (int c = 0; c < CW; ++c) areg[a][c] = fma(-la[a], q[c], areg[a][c]);
      if (ty == 0) {
        float* o = bh + (size_t)s * d + tx * CW;
        if constexpr (CW == 4) *(float4*)o = make_float4((float)q[0], (float)q[1], (float)q[2], (float)q[3]);
        else *(float2*)o = make_float2((float)q[0], (float)q[1]);
      }
    }
#pragma unroll
    for (int b = 0; b < TJ; ++b) {
      const double lbs = sh.crow[tx + 32 * b] * inv;
#pragma unroll
      for (int a = 0; a < TI; ++a) creg[a][b] = fma(-la[a], lbs, creg[a][b]);
    }
    if (tid < 128) {
      const double l = sh.crow[min(tid, NP - 1)] * inv;        // this thread's own row's coefficient
      if (tid == j) used = true;
      if (!used) dg -= l * l;
    }
    publish((s + 1) & 1);
    lds_barrier();
    r = s + 1;
  }
  __syncthreads();
  return r;
}

// ---- The ordinary head: well conditioned, n independent rows.  Q = L^-1 A with C = A A^T = L L^T factored in order, no pivot search, in
// blocks of 16 rows on the double-precision matrix instructions (v_mfma_f64_16x16x4_f64: operands row l % 16, k = l / 16; result entry r of
// lane l is row l/16 + 4 r, column l % 16 - which is also how it serves as the right operand of the next product, k-step by k-step).
//   C       tiles on and below the diagonal, one per wave at a time, from A staged as floats; then kept in LDS as 16 x 16 tiles;
//   panel k one row per lane: lanes 0 - 15 of waves 0 - 2 carry the diagonal block (each wave for itself), the other lanes the rows
//           below it and, in wave 0, an identity that becomes the inverse of the diagonal block's factor; sixteen pivots as unscaled
//           rank-one steps (a reciprocal each), the square roots at the end;
//   trail   C_ij -= L_ik L_jk^T, a tile per wave;
//   solve   wave w owns 16 columns of A in registers: Q_k = L_kk^-1 A_k, A_i -= L_ik Q_k.  Waves 3 - 7 do it beside the next panel,
//           waves 0 - 2 at the end (head_dim 64: waves 4 - 7 have all of it).
// Whether the rows really are independent by the rank rule is settled there too: waves 3 - 7 solve for the columns of the identity at the
// end, a block of sixteen at a time, and |L^-1|_F^2 = trace(C^-1) >= 1 / lambda_min(C).  A head passes when that times trace(C) is below
// 1e9: then every pivot in any order is at least 1e-9 of the trace, the rank threshold is (max(n, d) 2^-23)^2 lambda_max, 2.4e-10 of it at
// most (the computed factor is that of C + E, |E| <= n 2^-52 trace), and L^-1 A is as far from orthonormal as the pivoted loop's rows are
// (4e-9 at the limit, their rounding to single precision 2.5e-8).  An estimate from sign vectors instead of the identity takes as long
// (those waves have nothing else to do) and misses dependences whose coefficients are orthogonal to all of them.  Any other head takes
// the pivoted loop above, one row at a time.  Heads of n close to d are the ones that come near the limit: at 1e7 half of those of 127 rows
// and nine tenths of those of 128 were given up at the end (288 heads of 700 tokens, basis: 291 us at 127 and 448 at 128; 131 and 284 with
// 1e9; the pivoted loop alone 368 and 365).
// A head that will not pass is given up as early as that shows: after the first panel where two rows alone are too close (repeated
// values), one panel after a pivot that is too small, else at the end; the pivoted loop then starts from the Gram matrix formed here.
// Bound by the chain of pivots inside the panels.  288 heads, d = 128, 32 rows of 256 tokens and 96 of 2048: 22 and 96 us where all heads
// pass, 44 and 178 with the heads of one layer in 36 repeating value rows, 58 and 225 with all of them.  The pivoted loop for all
// heads, with its Gram matrix from scalar multiply-adds, took 59 and 239 (56 and 232 with repeated rows); both routes one after the other, each
// from its own Gram matrix, 67 and 289.
typedef __attribute__((__vector_size__(4 * sizeof(double)))) double ks_f64x4;
constexpr double kCholLimit = 1.0e9;     // largest trace(C) trace(C^-1) of a head that is settled here

__device__ __forceinline__ double ks_lane_f64(const double x, const int l) {
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// number t of a triangle walked by rows: (i, j), j <= i
__device__ __forceinline__ void ks_untri(const int t, int& i, int& j) {
  i = 0;
  while ((i + 1) * (i + 2) / 2 <= t) ++i;
  j = t - i * (i + 1) / 2;
}

// 16 x 16 product a b^T subtracted from acc; both operands 16 x 16 tiles in LDS
__device__ __forceinline__ ks_f64x4 ks_mul_bt(const double* a, const double* b, const int lane, ks_f64x4 acc) {
  const int o = (lane & 15) * KS_LT + (lane >> 4);
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[o + 4 * s], b[o + 4 * s], acc, 0, 0, 0);
  return acc;
}

// LDS of a head of n rows: the rows as they are stored (row stride ks_row_elems: 16 rows, 4 consecutive entries each, on different
// banks), then the tiles.
template <typename T> __host__ __device__ constexpr int ks_row_elems(int d) { return d + 16 / (int)sizeof(T); }
template <typename T> __host__ __device__ constexpr size_t ks_tiles_off(int nb, int d) { return (size_t)16 * nb * ks_row_elems<T>(d) * sizeof(T); }

__device__ __forceinline__ void ks_load4(const uint16_t* p, double (&o)[4]) {
  const uint2 q = *(const uint2*)p;
  o[0] = (double)__uint_as_float(q.x << 16); o[1] = (double)__uint_as_float(q.x & 0xffff0000u);
  o[2] = (double)__uint_as_float(q.y << 16); o[3] = (double)__uint_as_float(q.y & 0xffff0000u);
}
__device__ __forceinline__ void ks_load4(const float* p, double (&o)[4]) {
  const float4 q = *(const float4*)p;
  o[0] = (double)q.x; o[1] = (double)q.y; o[2] = (double)q.z; o[3] = (double)q.w;
}

// NBM: most 16-row blocks (n <= 16 NBM).  True when the head was settled: its n basis rows are in bh.  False: C is in the tiles, for ks_head.
// All threads call.
template <typename T, int D, int NBM>
__device__ __forceinline__ bool ks_chol_head(const T* __restrict__ Vh, const int32_t* __restrict__ id, const int n, float* __restrict__ bh,
                                             double* lds, KsShared& sh) {
  constexpr int GT = (NBM * (NBM + 1) / 2 + KS_WAVES - 1) / KS_WAVES;        // Gram tiles per wave
  constexpr int SLD = ks_row_elems<T>(D);
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int NB = (n + 15) >> 4;
  T* stg = (T*)lds;
  double* Lt = (double*)((char*)lds + ks_tiles_off<T>(NB, D));
  if (tid == 0) sh.stop = 0;
  {
    constexpr int EPP = 16 / (int)sizeof(T), PPR = D / EPP;
#pragma unroll 4
    for (int e = tid; e < 16 * NB * PPR; e += KS_THREADS) {
      const int i = e / PPR, pc = e - i * PPR;
      uint4 q = *(const uint4*)(Vh + (size_t)id[min(i, n - 1)] * D + pc * EPP);
      if (i >= n) q = make_uint4(0u, 0u, 0u, 0u);
      *(uint4*)(stg + i * SLD + pc * EPP) = q;
    }
  }
  __syncthreads();
  // C, and the diagonal to sh.crow (past n: infinite); this thread's share of the trace
  auto gram = [&]() -> double {
    double tr = 0.0;
#pragma unroll 1
    for (int q = 0; q < GT; ++q) {
      const int t = wave + KS_WAVES * q;
      if (t >= NB * (NB + 1) / 2) break;
      int i, j;
      ks_untri(t, i, j);
      ks_f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      const T* pa = stg + (16 * i + r16) * SLD + 4 * g;
      const T* pb = stg + (16 * j + r16) * SLD + 4 * g;
#pragma unroll 4
      for (int c = 0; c < D; c += 16) {
        double a[4], b[4];
        ks_load4(pa + c, a);
        ks_load4(pb + c, b);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[e], b[e], acc, 0, 0, 0);
      }
      double* o = Lt + ks_tile(i, j) * KS_TILE;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = g + 4 * r;
        double v = acc[r];
        if (i == j && row == r16) {
          const bool real = 16 * i + row < n;
          if (real) tr += v; else v = 1.0;                     // rows past n: an identity
          sh.crow[16 * i + row] = real ? v : INFINITY;
        }
        o[row * KS_LT + r16] = v;
      }
    }
    return tr;
  };
  const double trace = ks_block_sum(gram(), sh.red);           // (its barriers also publish the tiles)

  // Two rows alone bound the trace of the inverse from below, by (C_ii + C_jj) / (C_ii C_jj - C_ij^2), which is at the limit over trace(C)
  // where (C_ii - floor) (C_jj - floor) - floor^2 = C_ij^2: rows that repeat, or vanish, are seen beside the first panel.  c: C(i, j)
  const double floor = trace * (1.0 / kCholLimit);
  auto look_at_pairs = [&](const int i, const int j, const double (&c)[4]) {
    const double b = sh.crow[16 * j + r16] - floor;
    bool ok = true;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double a = sh.crow[16 * i + g + 4 * r] - floor;
      ok &= (i == j && g + 4 * r == r16) ? a > 0.0 : fma(a, b, -floor * floor) > c[r] * c[r];
    }
    if (!ok) sh.stop = 1;
  };
  auto tile_entries = [&](const int t, double (&c)[4]) {
    const double* o = Lt + t * KS_TILE + g * KS_LT + r16;
#pragma unroll
    for (int r = 0; r < 4; ++r) c[r] = o[4 * r * KS_LT];
  };

  // trailing tiles after panel k, a tile per wave
  auto trail = [&](const int k) {
    const int mt = (NB - 1 - k) * (NB - k) / 2;
    for (int t = wave; t < mt; t += KS_WAVES) {
      int i, j;
      ks_untri(t, i, j);
      i += k + 1; j += k + 1;
      double* o = Lt + ks_tile(i, j) * KS_TILE + g * KS_LT + r16;
      ks_f64x4 acc = {o[0], o[4 * KS_LT], o[8 * KS_LT], o[12 * KS_LT]};
      acc = ks_mul_bt(Lt + ks_tile(i, k) * KS_TILE, Lt + ks_tile(j, k) * KS_TILE, lane, acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) o[4 * r * KS_LT] = acc[r];
    }
  };
  double ss = 0.0;                                             // waves 3 - 7: squares of their columns of L^-1
  // The solve for 16 right-hand sides per wave: entry r of block i is row 16 i + g + 4 r.  cb: the columns of A, < 0: those of the
  // identity's block column k0, which is zero above row block k0
  auto solve = [&](const int cb, const int k0, auto&& before_step) {
    ks_f64x4 at[NBM];
#pragma unroll
    for (int i = 0; i < NBM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * i + g + 4 * r;
        if (cb >= 0) at[i][r] = (i < NB) ? (double)Elem<T>::load(stg + row * SLD + cb * 16 + r16) : 0.0;
        else at[i][r] = (i == k0 && row == 16 * i + r16) ? 1.0 : 0.0;
      }
    for (int k = k0; k < NB; ++k) {
      if (!before_step(k)) break;
      const int o = r16 * KS_LT + g;
      const double* iv = Lt + ks_tile(k, k) * KS_TILE + o;
      ks_f64x4 b = {0.0, 0.0, 0.0, 0.0}, q = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int i = 0; i < NBM; ++i) if (i == k) b = at[i];
#pragma unroll
      for (int s = 0; s < 4; ++s) q = __builtin_amdgcn_mfma_f64_16x16x4f64(iv[4 * s], b[s], q, 0, 0, 0);
#pragma unroll
      for (int i = 1; i < NBM; ++i)
        if (i > k && i < NB) {
          const double* l = Lt + ks_tile(i, k) * KS_TILE + o;
#pragma unroll
          for (int s = 0; s < 4; ++s) at[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(-l[4 * s], q[s], at[i], 0, 0, 0);
        }
      if (cb >= 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * k + g + 4 * r;
          if (row < n) bh[(size_t)row * D + cb * 16 + r16] = (float)q[r];
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) ss += (16 * k + g + 4 * r < n) ? q[r] * q[r] : 0.0;      // (rows past n: the padding's identity)
      }
    }
  };
  const int cblk = (D == 128) ? wave : wave - 4;               // this wave's columns of A
  // Three barriers per panel for every wave, whatever it does between them: rows read - panel written - trailing tiles written.  At the
  // second every wave learns whether a pair of rows, or a pivot of an earlier panel, fell below what the limit allows (1 / pivot is a
  // lower bound of the inverse's trace; the waves beside the panels look) and leaves if one did.
  bool stop = false;
  if (wave < 3) {
#pragma unroll 1
    for (int k = 0; k < NB; ++k) {
      // panel k, a row per lane
      double a[16];
      const bool diag = lane < 16, unit = wave == 0 && lane >= 16 && lane < 32;
      const int p = diag ? 16 * k + lane : 16 * (k + 1) + (wave == 0 ? lane - 32 : 32 + (wave - 1) * 48 + lane - 16);
      const bool have = !unit && p < 16 * NB;
      const bool used = wave == 0 || 16 * (k + 1) + 32 + (wave - 1) * 48 < 16 * NB;      // uniform
      double* prow = Lt + (have ? ks_tile(p >> 4, k) * KS_TILE + (p & 15) * KS_LT : 0);
      if (used) {
#pragma unroll
        for (int c = 0; c < 16; ++c) a[c] = have ? prow[c] : (unit && c == lane - 16) ? 1.0 : 0.0;
      }
      lds_barrier();                                           // the diagonal block is read by all three waves
      if (used) {
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          const double d = ks_lane_f64(a[c], c);
          double rc = __builtin_amdgcn_rcp(d);
          const double e = fma(-d, rc, 1.0);
          rc = fma(rc, fma(e, e, e), rc);
          rc = fma(fma(-d, rc, 1.0), rc, rc);
          const double t = -(a[c] * rc);
#pragma unroll
          for (int j = c + 1; j < 16; ++j) a[j] = fma(t, ks_lane_f64(a[c], j), a[j]);
        }
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          const double d = ks_lane_f64(a[c], c);               // the c-th pivot: lane c's own entry
          double y = __builtin_amdgcn_rsq(d);
          y = fma(fma(-d * y, y, 1.0), 0.5 * y, y);
          y = fma(fma(-d * y, y, 1.0), 0.5 * y, y);
          a[c] *= y;
        }
        if (have && !diag) {
#pragma unroll
          for (int c = 0; c < 16; ++c) prow[c] = a[c];
        }
        if (unit) {                                            // row i of L_kk^-T: column i of the inverse
          double* o = Lt + ks_tile(k, k) * KS_TILE + lane - 16;
#pragma unroll
          for (int c = 0; c < 16; ++c) o[c * KS_LT] = a[c];
        }
      }
      lds_barrier();
      stop = sh.stop != 0;                                     // uniform
      if (stop) break;
      trail(k);
      lds_barrier();
    }
    if (cblk >= 0 && !stop) solve(cblk, 0, [](int) { return true; });
  } else {
    // step k of the solve runs beside panel k + 1
    solve(cblk >= 0 ? cblk : 0, 0, [&](const int k) {
      if (k == 0) {
        double c[2][4];                                        // column block 0 changes in the panel: its tiles are fetched before
#pragma unroll
        for (int u = 0; u < 2; ++u) { const int i = wave - 3 + 5 * u; tile_entries(i < NB ? ks_tile(i, 0) : 0, c[u]); }
        lds_barrier();                                         // (the rows of panel 0 are read)
#pragma unroll
        for (int u = 0; u < 2; ++u) { const int i = wave - 3 + 5 * u; if (i < NB) look_at_pairs(i, 0, c[u]); }
#pragma unroll 1
        for (int t = wave - 3; t < NB * (NB - 1) / 2; t += 5) {
          int i, j;
          ks_untri(t, i, j);
          tile_entries(ks_tile(i + 1, j + 1), c[0]);
          look_at_pairs(i + 1, j + 1, c[0]);
        }
      }
      lds_barrier();
      stop = sh.stop != 0;
      if (stop) return false;
      trail(k);
      lds_barrier();
      if (k + 1 < NB) lds_barrier();
      const double d = Lt[ks_tile(k, k) * KS_TILE + r16 * (KS_LT + 1)];        // 1 / square root of a pivot
      if (16 * k + r16 < n && !(floor * d * d < 1.0)) sh.stop = 1;
      return true;
    });
    // block columns of the identity: wave w takes w - 3, and of the last three, which are the shortest, number 12 - w: eight steps at most
#pragma unroll 1
    for (int b = stop ? NB : wave - 3; b < NB; b = (b < 5 && 12 - wave > b) ? 12 - wave : NB) solve(-1, b, [](int) { return true; });
  }
  if (!stop) {
    const double inv_trace = ks_block_sum(ss, sh.red);
    if (trace * inv_trace < kCholLimit) return true;           // false also when a pivot was not positive
  }
  __syncthreads();
  (void)gram();                                                // for the pivoted loop: the factor lies where C was
  __syncthreads();
  return false;
}

// The workgroup of a head with n retained rows: its basis and its state.  D: head_dim; BIG: more than 96 rows.  lds: ks_smem bytes.
template <typename T, int D, bool BIG>
__device__ __forceinline__ void ks_workgroup(const T* __restrict__ V, const float* __restrict__ scores, const int32_t* __restrict__ idx, const int n,
                                             const int N, const int max_budget, const int rank, HeadState* __restrict__ state,
                                             float* __restrict__ basis, const int scs, const int kvs, const int head, double* Cs, KsShared& sh) {
  constexpr int d = D;
  const int n_del = N - n;
  const float* sc = scores + (size_t)head * scs;
  const int32_t* id = idx + (size_t)head * max_budget;
  const T* Vh = V + (size_t)head * kvs * d;
  const int tid = threadIdx.x;

  // demand sums of Eq. 6, in double, fixed summation order: this thread's shares, added up over the workgroup at the end
  double pk = 0.0, pt = 0.0;
  for (int i = tid; i < n; i += KS_THREADS) pk += (double)sc[id[i]];
  for (int i0 = tid; i0 < N; i0 += 8 * KS_THREADS) {           // eight loads in flight
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = (i0 + u * KS_THREADS < N) ? sc[i0 + u * KS_THREADS] : 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u) pt += (double)v[u];
  }

  int r_keep = 0, active = 0;
  if (rank > 0 && n > 0 && n_del > 0) {
    float* bh = basis + (size_t)head * d * d;
    bool done;
    if constexpr (BIG) {                                       // n > 96 implies d = 128
      done = ks_chol_head<T, 128, 8>(Vh, id, n, bh, Cs, sh);
    } else if constexpr (d == 128) {
      if (n <= 32) done = ks_chol_head<T, 128, 2>(Vh, id, n, bh, Cs, sh);
      else done = ks_chol_head<T, 128, 6>(Vh, id, n, bh, Cs, sh);
    } else {
      done = ks_chol_head<T, 64, 4>(Vh, id, n, bh, Cs, sh);
    }
    r_keep = n;
    if (!done) {
      const double* Lt = (const double*)((const char*)Cs + ks_tiles_off<T>((n + 15) >> 4, d));
      if constexpr (BIG) {
        r_keep = ks_head<T, 8, 4>(Vh, id, n, bh, Cs, Lt, sh);
      } else if constexpr (d == 128) {
        if (n <= 32) r_keep = ks_head<T, 2, 4>(Vh, id, n, bh, Cs, Lt, sh);
        else if (n <= 64) r_keep = ks_head<T, 4, 4>(Vh, id, n, bh, Cs, Lt, sh);
        else r_keep = ks_head<T, 6, 4>(Vh, id, n, bh, Cs, Lt, sh);
      } else {
        if (n <= 32) r_keep = ks_head<T, 2, 2>(Vh, id, n, bh, Cs, Lt, sh);
        else r_keep = ks_head<T, 4, 2>(Vh, id, n, bh, Cs, Lt, sh);
      }
    }
    active = (r_keep < d) ? 1 : 0;
  }
  const double a_keep = ks_block_sum(pk, sh.red);
  const double a_tot = ks_block_sum(pt, sh.red);
  double a_del = a_tot - a_keep;
  if (a_del < 0.0) a_del = 0.0;
  if (tid == 0) {
    HeadState s;
    s.a_keep = a_keep; s.a_del = a_del; s.n_keep = n; s.n_del = n_del; s.r_keep = r_keep; s.active = active;
    s.k_used = 0; s.pad = 0; s.rcr = 0.f; s.ivn = 0.f;
    state[head] = s;
  }
}

// dynamic LDS of a launch whose heads keep at most nmax rows: the rows and the tiles of the blocked factorisation, or the padded
// single-precision Gram matrix of the pivoted loop
template <typename T>
inline size_t ks_smem(size_t nmax, int d) {
  const size_t np = (nmax + 31) / 32 * 32, nb = (nmax + 15) / 16;
  return max(np * np * sizeof(float),
             ks_tiles_off<T>((int)nb, d) + nb * (nb + 1) / 2 * KS_TILE * sizeof(double));
}

}  // namespace obf
