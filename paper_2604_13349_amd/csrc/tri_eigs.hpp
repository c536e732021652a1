// Leading eigenpairs of a small symmetric matrix, for a workgroup of 512 threads: the direct route for
// the case "a few leading right singular vectors of the residual" (Sec. 4.4: k = pca_rank is small against the
// width of the complement), in place of a full Jacobi diagonalisation:
//   1. Householder tridiagonalisation T = H S H^T (m - 2 reflectors, one barrier each; fewer where T has low rank);
//   2. the k largest eigenvalues of the tridiagonal S by multisection on Sturm counts (every thread evaluates one
//      shift per round; three or four rounds shrink an eigenvalue's bracket below single-precision resolution);
//   3. their eigenvectors by inverse iteration on S - theta I (tridiagonal elimination with row exchanges, one lane
//      per eigenvector, two solves from a fixed pseudo-random start, three under one shift for eigenvalues that agree), eight at a time;
//   4. back-transformation through the reflectors (one wave per eigenvector) and a final Gram-Schmidt pass over the
//      k vectors (eigenvalues that agree to rounding give vectors that only span the right subspace together).
// All arithmetic is single precision; nothing here depends on convergence of an iteration.
#pragma once
#include "common.hpp"
#include "wave_ops.hpp"

namespace obf {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_te;

constexpr int TE_THREADS = 512;
constexpr int TE_WAVES = TE_THREADS / 64;
constexpr int TE_MAXK = 16;              // most eigenpairs
constexpr int TE_BATCH = 8;              // eigenvectors per pass of the inverse iteration and the back-transformation (one wave each)

// floats of LDS scratch tri_top_eigs needs for an m x m matrix and k eigenpairs
__host__ __device__ inline int tri_lane_stride(int k) { return k <= 4 ? 4 : 8; }
__host__ __device__ inline int tri_work_floats(int m, int k) {
  return 4 * m + 256 + TE_THREADS + 96 + 7 * tri_lane_stride(k) * m + (k > TE_BATCH ? k * m : 0);
}

// floats of LDS of the packed reflectors, and where entry i of reflector j lies: tri_refl_off(m, j) + i
__host__ __device__ inline int tri_refl_floats(int m) { return m * (m - 1) / 2; }
__device__ __forceinline__ int tri_refl_off(const int m, const int j) { return __mul24(j, m - 2) - (__mul24(j, j - 1) >> 1) - 1; }

// sum over the 64 lanes, the result in every lane: four in-row DPP steps, then the rows and the halves meet through
// lane swaps (no LDS traffic, a fixed order of additions)
__device__ __forceinline__ float te_wave_sum(float v) {
  v += __uint_as_float(OBF_DPP_MOV(__float_as_uint(v), 0xB1));
  v += __uint_as_float(OBF_DPP_MOV(__float_as_uint(v), 0x4E));
  v += __uint_as_float(OBF_DPP_MOV(__float_as_uint(v), 0x141));
  v += __uint_as_float(OBF_DPP_MOV(__float_as_uint(v), 0x140));
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// The sums over the wave of three values at once, uniform: two lane swaps leave a value in each 16-lane row (p in row 0, r in row 1,
// q in row 2), four in-row steps finish all of them together.
__device__ __forceinline__ void te_wave_sum3(const float p, const float q, const float r, float& sp, float& sq, float& sr) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(p), __float_as_uint(q), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(r), __float_as_uint(r), false, false);
  const float pq = __uint_as_float(a[0]) + __uint_as_float(a[1]), rr = __uint_as_float(b[0]) + __uint_as_float(b[1]);
  const auto c = __builtin_amdgcn_permlane16_swap(__float_as_uint(pq), __float_as_uint(rr), false, false);
  float v = __uint_as_float(c[0]) + __uint_as_float(c[1]);
  v += __uint_as_float(OBF_DPP_MOV(__float_as_uint(v), 0xB1));
  v += __uint_as_float(OBF_DPP_MOV(__float_as_uint(v), 0x4E));
  v += __uint_as_float(OBF_DPP_MOV(__float_as_uint(v), 0x141));
  v += __uint_as_float(OBF_DPP_MOV(__float_as_uint(v), 0x140));
  sp = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), 0));
  sr = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), 16));
  sq = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), 32));
}

// One wave: each of the kb vectors (entry t of vector i at z[t * KS + i], n entries) whose bit is set in `which` is made orthogonal to those before
// it whose eigenvalues follow one another by at most `close`.  Not inlined: its registers would count against the whole caller.
template <int KS>
__device__ __attribute__((noinline)) void te_separate(float* z, const float* th, const int n, const int kb, const float close, const uint64_t which) {
  const int lane = threadIdx.x & 63;
  const bool a = lane < n, b = lane + 64 < n;
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
  for (int i = 1; i < kb; ++i) {
    if (!((which >> i) & 1)) continue;
    float x0 = a ? z[lane * KS + i] : 0.f, x1 = b ? z[(lane + 64) * KS + i] : 0.f;
    for (int j = i - 1; j >= 0 && th[j] - th[j + 1] <= close; --j) {
      const float y0 = a ? z[lane * KS + j] : 0.f, y1 = b ? z[(lane + 64) * KS + j] : 0.f;
      const float xy = te_wave_sum(fmaf(x0, y0, x1 * y1)), yy = te_wave_sum(fmaf(y0, y0, y1 * y1));
      const float f = (yy > 0.f && yy < INFINITY) ? xy / yy : 0.f;
      x0 = fmaf(-f, y0, x0); x1 = fmaf(-f, y1, x1);
    }
    if (a) z[lane * KS + i] = x0;
    if (b) z[(lane + 64) * KS + i] = x1;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
  }
}

// Inverse iteration on the tridiagonal S - theta I for one eigenvector per lane.  Arrays of the factorisation live at
// f[(q * m + j) * KS] for q = 0 .. 4: the upper triangle's three diagonals (the first as its reciprocal), the
// multiplier and the row-exchange flag of step j (elimination with partial pivoting).  KS, the lane stride, is a
// compile-time constant.  The three passes are chains through one or two registers; what they read comes from LDS in batches of
// TE_AHEAD steps, so that the chain does not wait for it step by step.
constexpr int TE_AHEAD = 8;

template <int KS>
__device__ __forceinline__ void te_factor(const float* __restrict__ dv, const float* __restrict__ ev, const int m,
                                          const float theta, const float tiny, float* __restrict__ f) {
  float* i0 = f; float* a1 = f + m * KS; float* a2 = a1 + m * KS; float* mu = a2 + m * KS; float* sw = mu + m * KS;
  float r0 = dv[0] - theta, r1 = (m > 1) ? ev[0] : 0.f, r2 = 0.f;
  auto step = [&](const int j, float n0, const float d1, float n2) {
    float n1 = d1 - theta;
    const bool swap = fabsf(n0) > fabsf(r0);
    if (swap) { float t; t = r0; r0 = n0; n0 = t; t = r1; r1 = n1; n1 = t; t = r2; r2 = n2; n2 = t; }
    if (r0 == 0.f) r0 = tiny;
    float inv = __builtin_amdgcn_rcpf(r0);                      // one Newton step on the hardware reciprocal: the pivots only
    inv = fmaf(fmaf(-r0, inv, 1.f), inv, inv);                  // steer an iteration that converges whatever their last bit
    const float g = n0 * inv;
    i0[j * KS] = inv; a1[j * KS] = r1; a2[j * KS] = r2; mu[j * KS] = g; sw[j * KS] = swap ? 1.f : 0.f;
    r0 = fmaf(-g, r1, n1); r1 = fmaf(-g, r2, n2); r2 = 0.f;
  };
  int j0 = 0;
  for (; j0 + TE_AHEAD + 1 < m; j0 += TE_AHEAD) {
    float d[TE_AHEAD], e[TE_AHEAD + 1];
#pragma unroll
    for (int u = 0; u < TE_AHEAD; ++u) { d[u] = dv[j0 + u + 1]; e[u] = ev[j0 + u]; }
    e[TE_AHEAD] = ev[j0 + TE_AHEAD];
#pragma unroll
    for (int u = 0; u < TE_AHEAD; ++u) step(j0 + u, e[u], d[u], e[u + 1]);
  }
  for (; j0 + 1 < m; ++j0) step(j0, ev[j0], dv[j0 + 1], (j0 + 2 < m) ? ev[j0 + 1] : 0.f);
  i0[(m - 1) * KS] = 1.f / ((fabsf(r0) > 1e-3f * tiny) ? r0 : tiny);
  a1[(m - 1) * KS] = 0.f; a2[(m - 1) * KS] = 0.f;
}

// the row operations of the elimination applied to the right-hand side: scale * in -> out
template <int KS>
__device__ __forceinline__ void te_forward(const float* __restrict__ f, const int m, const float* __restrict__ in,
                                           float* __restrict__ out, const float scale) {
  const float* mu = f + 3 * m * KS; const float* sw = mu + m * KS;
  float carry = in[0] * scale;
  auto step = [&](const int j, const float x, const float g, const float s) {
    const float nx = x * scale;
    const bool swap = s != 0.f;
    const float bj = swap ? nx : carry, bn = swap ? carry : nx;
    out[j * KS] = bj;
    carry = fmaf(-g, bj, bn);
  };
  int j0 = 0;
  for (; j0 + TE_AHEAD < m; j0 += TE_AHEAD) {
    float x[TE_AHEAD], g[TE_AHEAD], s[TE_AHEAD];
#pragma unroll
    for (int u = 0; u < TE_AHEAD; ++u) { x[u] = in[(j0 + u + 1) * KS]; g[u] = mu[(j0 + u) * KS]; s[u] = sw[(j0 + u) * KS]; }
#pragma unroll
    for (int u = 0; u < TE_AHEAD; ++u) step(j0 + u, x[u], g[u], s[u]);
  }
  for (; j0 + 1 < m; ++j0) step(j0, in[(j0 + 1) * KS], mu[j0 * KS], sw[j0 * KS]);
  out[(m - 1) * KS] = carry;
}

// back substitution with the upper triangle: in -> out; returns the largest magnitude of the solution
template <int KS>
__device__ __forceinline__ float te_backward(const float* __restrict__ f, const int m, const float* __restrict__ in,
                                             float* __restrict__ out) {
  const float* i0 = f; const float* a1 = f + m * KS; const float* a2 = a1 + m * KS;
  float z1 = 0.f, z2 = 0.f, big = 0.f;
  auto step = [&](const int j, const float x, const float c1, const float c2, const float iv) {
    const float v = fmaf(-c1, z1, fmaf(-c2, z2, x)) * iv;
    out[j * KS] = v;
    z2 = z1; z1 = v;
    big = fmaxf(big, fabsf(v));
  };
  int j0 = m - 1;
  for (; j0 >= TE_AHEAD - 1; j0 -= TE_AHEAD) {
    float x[TE_AHEAD], c1[TE_AHEAD], c2[TE_AHEAD], iv[TE_AHEAD];
#pragma unroll
    for (int u = 0; u < TE_AHEAD; ++u) { x[u] = in[(j0 - u) * KS]; c1[u] = a1[(j0 - u) * KS]; c2[u] = a2[(j0 - u) * KS]; iv[u] = i0[(j0 - u) * KS]; }
#pragma unroll
    for (int u = 0; u < TE_AHEAD; ++u) step(j0 - u, x[u], c1[u], c2[u], iv[u]);
  }
  for (; j0 >= 0; --j0) step(j0, in[j0 * KS], a1[j0 * KS], a2[j0 * KS], i0[j0 * KS]);
  return big;
}

// Tridiagonalisation of the m x m symmetric matrix Tsrc (row stride ls), 32 (MB - 1) < m <= 32 MB: the diagonal to dv, the
// sub-diagonal to ev, reflector j (I - bet[j] v v^T), entries j + 1 .. m - 1, to Rf packed column behind column.  cbuf and ybuf [2][128] are LDS, 16-byte
// aligned.  All threads call; ends with a barrier.
//
// The matrix lives in registers as 32 x 32 tiles in the result layout of the matrix instructions (entry i of lane l: row
// (i/4)*8 + (l/32)*4 + i%4, column l%32); wave b < MB holds the tiles of row block b.  With x the column to be reduced, c the next
// one (both below the diagonal, before the step's update), v = x - alpha e and T v = T x - alpha c, a step is
//   every wave: |x| and its 32 entries of T x (a lane sums over its column of every tile, a reduce-scatter over the lanes of a
//               half-wave leaves each with one row) to LDS;                                     -- barrier --
//   every wave: p = beta (T x - alpha c), w = p - (beta/2 p.v) v, all entries, two per lane; the update T - v w^T - w v^T is one
//               v_mfma_f32_32x32x2_f32 per tile whose operands are lane swaps of v and w; the next x is c less its share of the
//               update; the tiles that hold the next c publish it.
// Repeating the vector work in every wave leaves one barrier and one LDS round trip per reflector (none of the waves' barriers once
// the trailing matrix fits one block); it is why only MB waves take part: two waves on a SIMD share its instruction issue, and two
// tiles on each of eight waves took as long (2900 cycles a step at m = 96) as the same work on the vector ALU with four barriers.
// Bound by the dependent chain of a step and, with two workgroups on a compute unit, by instruction issue: 2600 cycles at m = 128.
//
// A matrix of rank r is done early: after r + 1 steps the reflectors' columns span its range and what is left is rounding (a step more
// for each time that the columns run into an invariant subspace and start again, as clusters of eigenvalues make them; fewer where the
// eigenvalues fall below the rounding).  A column no longer than left_tol makes the waves look at all that is left, which is dropped
// when its Frobenius norm is no more than that either.  Returns the width of S: m, or one more than the reflectors so far.
// The residual Gram matrix P G P has the rank of the complement at most.  Back-fill of 288 heads with eigenvalues 1 - 1e-4 i, 2 directions, us, all columns and
// this way: complements 64, 32 and 20 wide 360 and 335, 407 and 317, 446 and 323; 96 wide, where the starts use up the rest of the
// columns, 334 and 355 (the last row block's loop is no longer unrolled for the columns before it).  0.546^i, 96 wide, 12 directions: 346 and 200.
template <int MB>
__device__ __forceinline__ int tri_reduce(const float* __restrict__ Tsrc, const int ls, float* Rf, const int m, const float left_tol,
                                          float* dv, float* ev, float* bet, float* cbuf, float* ybuf /*[256 + 7]*/) {
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr bool TWO = MB > 2;                                 // a lane holds two entries of a vector
  auto lane_val = [](const float x, const int l) -> float {
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), l));
  };
  if (tid < 128) cbuf[tid] = (m > 1 && tid < m) ? Tsrc[(size_t)ls + tid] : 0.f;    // column 1, read as row 1
  if (tid == 0) dv[0] = Tsrc[0];
  f32x16_te tile[MB];
  float xa = 0.f, xb = 0.f;                                    // entries lane and lane + 64 of x
  if (wave < MB) {
#pragma unroll
    for (int cb = 0; cb < MB; ++cb)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = wave * 32 + (i >> 2) * 8 + lh * 4 + (i & 3), c = cb * 32 + lr;
        tile[cb][i] = (r < m && c < m) ? Tsrc[(size_t)r * ls + c] : 0.f;
      }
    xa = (lane > 0 && lane < m) ? Tsrc[lane] : 0.f;            // column 0
    xb = (TWO && lane + 64 < m) ? Tsrc[lane + 64] : 0.f;
  }
  __syncthreads();
  // the row this lane is left with: entry 8 b4 + 4 b3 + 2 b2 + b1 of the tile's sixteen (b: the bits of the lane number)
  const bool l3 = (lane & 8) != 0, l2 = (lane & 4) != 0, l1 = (lane & 2) != 0;
  const int my_row = wave * 32 + ((lane >> 4) & 1) * 16 + ((lane >> 3) & 1) * 8 + lh * 4 + ((lane >> 2) & 1) * 2 + ((lane >> 1) & 1);
  float* lsum = ybuf + 256;                                    // [4] the waves' sums of squares, the width of S, [2] |x| by step parity
  auto step = [&](const int j, const int b0 /*block in which the trailing matrix starts*/, const bool alone) -> bool {      // was |x| at most left_tol (uniform)
    const int par = j & 1;
    const bool live = wave < MB && wave >= b0;                 // uniform over the wave
    float alpha = 0.f, beta = 0.f, head = 0.f, norm = 0.f;
    if (live) {
      const auto X0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(xa), __float_as_uint(xa), false, false);   // blocks 0 and 1 of x,
      const auto X1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(xb), __float_as_uint(xb), false, false);   // 2 and 3, in both half-waves
      const float ss = te_wave_sum(TWO ? fmaf(xa, xa, xb * xb) : xa * xa);
      head = lane_val((TWO && j + 1 >= 64) ? xb : xa, (j + 1) & 63);
      float s[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
      for (int cb = 0; cb < MB; ++cb)
        if (cb >= b0) {
          const float xc = __uint_as_float((cb == 0) ? X0[0] : (cb == 1) ? X0[1] : (cb == 2) ? X1[0] : X1[1]);
#pragma unroll
          for (int i = 0; i < 16; ++i) s[i] = fmaf(tile[cb][i], xc, s[i]);
        }
      // reduce-scatter over the 32 lanes of the half-wave: partners differ in bit 4, then in bits 3 - 0, 2 - 0, 1 and 0
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(s[i]), __float_as_uint(s[i + 8]), false, false);
        s[i] = __uint_as_float(q[0]) + __uint_as_float(q[1]);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float keep = l3 ? s[i + 4] : s[i], give = l3 ? s[i] : s[i + 4];
        s[i] = keep + __uint_as_float(OBF_DPP_MOV(__float_as_uint(give), 0x140));
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float keep = l2 ? s[i + 2] : s[i], give = l2 ? s[i] : s[i + 2];
        s[i] = keep + __uint_as_float(OBF_DPP_MOV(__float_as_uint(give), 0x141));
      }
      {
        const float keep = l1 ? s[1] : s[0], give = l1 ? s[0] : s[1];
        s[0] = keep + __uint_as_float(OBF_DPP_MOV(__float_as_uint(give), 0x4E));
      }
      s[0] += __uint_as_float(OBF_DPP_MOV(__float_as_uint(s[0]), 0xB1));
      ybuf[par * 128 + my_row] = s[0];                         // the same value from two lanes
      // Single-instruction square root and reciprocal (1 ulp): the reflector only has to be orthogonal to rounding.
      const float sigma = __builtin_amdgcn_sqrtf(ss);
      if (sigma > 0.f) {
        alpha = (head >= 0.f) ? -sigma : sigma;
        beta = __builtin_amdgcn_rcpf(sigma * (sigma + fabsf(head)));
      }
      norm = sigma;
      if (!alone && wave == MB - 1 && lane == 0) lsum[5 + par] = sigma;
    }
    if (alone) __builtin_amdgcn_wave_barrier(); else { lds_barrier(); norm = lsum[5 + par]; }
    if (live) {
      const float* yr = ybuf + par * 128;
      const float* cr = cbuf + par * 128;
      const float ya = yr[lane], yb = TWO ? yr[lane + 64] : 0.f, ca = cr[lane], cb_ = TWO ? cr[lane + 64] : 0.f;
      const bool ina = lane > j && lane < m, inb = TWO && lane + 64 > j && lane + 64 < m;
      const float v1 = head - alpha;
      const float va = (lane == j + 1) ? v1 : xa, vb = (lane + 64 == j + 1) ? v1 : xb;       // zero outside j < i < m
      const float pa = ina ? beta * fmaf(-alpha, ca, ya) : 0.f, pb = inb ? beta * fmaf(-alpha, cb_, yb) : 0.f;
      const float K = 0.5f * beta * te_wave_sum(TWO ? fmaf(pa, va, pb * vb) : pa * va);
      const float wa = fmaf(-K, va, pa), wb = fmaf(-K, vb, pb);
      // operands of the update: k = 0 in the lower half-wave, k = 1 in the upper; block b of a vector sits in half b % 2 of entry b / 2
      const bool hi = TWO && wave >= 2;
      const auto A = __builtin_amdgcn_permlane32_swap(__float_as_uint(hi ? vb : va), __float_as_uint(hi ? wb : wa), false, false);
      const auto B0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(wa), __float_as_uint(va), false, false);
      const auto B1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(wb), __float_as_uint(vb), false, false);
      const float a = -__uint_as_float((wave & 1) ? A[1] : A[0]);
#pragma unroll
      for (int cb = 0; cb < MB; ++cb)
        if (cb >= b0) {
          const uint32_t bo = (cb == 0) ? B0[0] : (cb == 1) ? B0[1] : (cb == 2) ? B1[0] : B1[1];
          tile[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, __uint_as_float(bo), tile[cb], 0, 0, 0);
        }
      // column j + 1 after the update: its diagonal entry is final, the rest is the next x
      const float w1 = lane_val((TWO && j + 1 >= 64) ? wb : wa, (j + 1) & 63);
      const float na = fmaf(-va, w1, fmaf(-wa, v1, ca)), nb = fmaf(-vb, w1, fmaf(-wb, v1, cb_));
      if (wave == MB - 1) {                                    // the wave that stays to the end keeps the books
        const int off = tri_refl_off(m, j);
        if (ina) Rf[off + lane] = va;
        if (inb) Rf[off + lane + 64] = vb;
        if (lane == 0) { bet[j] = beta; ev[j] = alpha; }
        if (lane == ((j + 1) & 63)) dv[j + 1] = (TWO && j + 1 >= 64) ? nb : na;
      }
      xa = (lane > j + 1 && lane < m) ? na : 0.f;
      xb = (TWO && lane + 64 > j + 1 && lane + 64 < m) ? nb : 0.f;
      const int cn = j + 2;                                    // the next raw column
#pragma unroll
      for (int cb = 0; cb < MB; ++cb)
        if (cb >= b0 && cb == (cn >> 5)) {
          if (lr == (cn & 31)) {
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4)
              *(float4*)&cbuf[(par ^ 1) * 128 + wave * 32 + i4 * 8 + lh * 4] =
                  make_float4(tile[cb][4 * i4], tile[cb][4 * i4 + 1], tile[cb][4 * i4 + 2], tile[cb][4 * i4 + 3]);
          }
        }
    }
    return __builtin_amdgcn_readfirstlane(norm <= left_tol ? 1 : 0) != 0;
  };
  // sum of squares of this wave's entries past row and column j, the last wave's with x
  auto left = [&](const int j, const int b0) -> float {
    float f = (wave == MB - 1) ? fmaf(xa, xa, xb * xb) : 0.f;
    int over = wave * 32 + lh * 4 - j;
    asm volatile("" : "+v"(over));                             // (the comparisons below, kept ahead of the loop, push the tiles to scratch)
#pragma unroll
    for (int cb = 0; cb < MB; ++cb)
      if (cb >= b0) {
        float g = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) g = (over > -((i >> 2) * 8 + (i & 3))) ? fmaf(tile[cb][i], tile[cb][i], g) : g;
        f += (cb * 32 + lr > j) ? g : 0.f;
      }
    return te_wave_sum(f);
  };
  const float left2 = left_tol * left_tol;
  bool done = false, look = false;
  int j = 0;
  for (; j + 2 < m && ((j + 1) >> 5) < MB - 1; ++j) {
    const int b0 = (j + 1) >> 5;
    if (look) {                                                // uniform
      if (wave >= b0 && wave < MB) { const float f = left(j, b0); if (lane == 0) lsum[wave] = f; }
      lds_barrier();
      float f = 0.f;
      for (int w = b0; w < MB; ++w) f += lsum[w];
      if (__builtin_amdgcn_readfirstlane(f <= left2 ? 1 : 0)) { done = true; break; }
    }
    look = step(j, b0, false);
  }
  lds_barrier();                                               // the other row blocks' last column is published
  if (wave == MB - 1) {
    if (!done) {
      for (; j + 2 < m; ++j) {
        if (look && __builtin_amdgcn_readfirstlane(left(j, MB - 1) <= left2 ? 1 : 0)) { done = true; break; }
        look = step(j, MB - 1, true);
      }
    }
    if (!done) {
      // the last 2 x 2 block: x is column m - 2, the published column is m - 1
      const float last = lane_val((TWO && m - 1 >= 64) ? xb : xa, (m - 1) & 63);
      __builtin_amdgcn_wave_barrier();
      if (m >= 2 && lane == 0) { ev[m - 2] = last; dv[m - 1] = cbuf[(m & 1) * 128 + m - 1]; }
    }
    if (lane == 0) *(int*)&lsum[4] = done ? j + 1 : m;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(*(const int*)&lsum[4]);
}

// The scratch of the direct route starts with these arrays; tri_work_floats(m, k) floats in all, in LDS and 16-byte aligned.
struct TriWork {
  float *cbuf, *dv, *ev, *e2, *bet;
  int* cnt;
  __device__ __forceinline__ TriWork(float* work, const int m) {
    cbuf = work;                      // [2][128] tridiagonalisation: the raw next column, by step parity
    dv = cbuf + 256;                  // diagonal of S
    ev = dv + m;                      // sub-diagonal of S: ev[j] = S[j+1][j]
    e2 = ev + m;
    bet = e2 + m;                     // reflector j is I - bet[j] v v^T, v in column j of Rf
    cnt = (int*)(bet + m);            // [TE_THREADS]
  }
};

// Step 1.  Tsrc: the m x m symmetric matrix (row stride ls; global or LDS, read once), m = 32 MB.  Rf: LDS, tri_refl_floats(m) floats, with
// `work` behind it (masked lanes read past it).  left_tol, the result: see tri_reduce.  Every thread of the workgroup must call.
template <int MB>
__device__ __forceinline__ int tri_start(const float* __restrict__ Tsrc, const int ls, float* Rf, const int m, const float left_tol, float* work) {
  const TriWork w(work, m);
  return tri_reduce<MB>(Tsrc, ls, Rf, m, left_tol, w.dv, w.ev, w.bet, w.cbuf, (float*)w.cnt);       // (the counts come later)
}

// Steps 2 to 4 on the n x n tridiagonal matrix of tri_start.  1 <= k0 <= TE_MAXK; KS = tri_lane_stride(k0).
// More than TE_BATCH eigenpairs are found in passes of TE_BATCH (the eigenvalues' multisection, the inverse iteration and
// the back-transformation each run once per pass on the same scratch).
// On return (after its own final barrier) *theta points at the k0 eigenvalues, largest first, and *W at the unit eigenvectors, W[i * m + t].
// Where S is narrower than k0 the eigenvalues past its width are zero and have no vectors.  Every thread of the workgroup must call.
template <int KS>
__device__ __forceinline__ void tri_top_eigs(const float* Rf, const int m, const int n, const int k0, float* work, const float** theta,
                                             const float** W) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const TriWork tw(work, m);
  float *dv = tw.dv, *ev = tw.ev, *e2 = tw.e2, *bet = tw.bet;
  int* cnt = tw.cnt;
  float* br_a = (float*)(cnt + TE_THREADS); // [16] brackets, then eigenvalues
  float* br_b = br_a + 16;
  float* th = br_b + 16;
  int* wc = (int*)(th + 16);          // [16] per-wave counts
  float* scal = (float*)(wc + 16);    // [32] lo, hi, ...
  float* lu = scal + 32;              // [5][m][KS] factors of S - theta I per eigenvector + [m][KS] second iteration vector; later W [k][m]
  float* zz = lu + 6 * m * KS;        // [m][KS] iteration vectors

  const int k = min(k0, n);
  if (wave == 0) {
    // Gershgorin interval of S and its squared sub-diagonal entries: lane l looks at rows l and l + 64
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int i = lane + 64 * h;
      if (i < n) {
        const float below = (i + 1 < n) ? ev[i] : 0.f, above = (i > 0) ? ev[i - 1] : 0.f;
        const float r = fabsf(above) + fabsf(below);
        lo = fminf(lo, dv[i] - r); hi = fmaxf(hi, dv[i] + r);
        e2[i] = fmaxf(below * below, 1e-36f);                    // never 0: see the Sturm recurrence
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      lo = fminf(lo, __shfl_xor(lo, off)); hi = fmaxf(hi, __shfl_xor(hi, off));
    }
    if (lane == 0) {
      const float span = hi - lo;
      scal[0] = lo - (1e-3f * span + 1e-30f);
      scal[1] = hi + (1e-3f * span + 1e-30f);
      scal[3] = 1.2e-7f * fmaxf(fabsf(lo), fabsf(hi));           // pivot perturbation of the inverse iteration
    }
  }
  __syncthreads();

  // ---- 2. eigenvalues: number of eigenvalues below x = number of negative terms of the Sturm recurrence
  // (a pivot that vanishes gives an infinite term and the next step forgets it: the count is right without a guard as long as no
  // off-diagonal entry is an exact zero; two dependent instructions per step, the rest is read ahead)
  auto sturm = [&](const float x) -> int {
    float q = dv[0] - x;
    int c = q < 0.f;
    int i = 1;
    for (; i + TE_AHEAD <= n; i += TE_AHEAD) {
      float d[TE_AHEAD], e[TE_AHEAD];
#pragma unroll
      for (int u = 0; u < TE_AHEAD; ++u) { d[u] = dv[i + u] - x; e[u] = e2[i + u - 1]; }
#pragma unroll
      for (int u = 0; u < TE_AHEAD; ++u) { q = fmaf(-e[u], __builtin_amdgcn_rcpf(q), d[u]); c += q < 0.f; }
    }
    for (; i < n; ++i) { q = fmaf(-e2[i - 1], __builtin_amdgcn_rcpf(q), dv[i] - x); c += q < 0.f; }
    return c;
  };
  {
    const float lo = scal[0], hi = scal[1];
    constexpr float step = 1.f / (float)(TE_THREADS + 1);
    cnt[tid] = sturm(lo + (hi - lo) * ((float)(tid + 1) * step));
    __syncthreads();
    if (tid < k) {                                             // eigenvalue tid from the top is number n - 1 - tid from below
      const int tgt = n - 1 - tid;
      int a = 0, b = TE_THREADS;                               // first shift whose count exceeds tgt
      while (a < b) { const int mid = (a + b) >> 1; if (cnt[mid] <= tgt) a = mid + 1; else b = mid; }
      br_a[tid] = (a > 0) ? lo + (hi - lo) * ((float)a * step) : lo;
      br_b[tid] = (a < TE_THREADS) ? lo + (hi - lo) * ((float)(a + 1) * step) : hi;
    }
    __syncthreads();
  }
  for (int g0 = 0; g0 < k; g0 += TE_BATCH) {                   // eigenvalues g0 .. g0 + kb - 1 (from the top)
    const int kb = min(TE_BATCH, k - g0);
    int kp = 1;
    while (kp < kb) kp <<= 1;
    const int S = TE_THREADS / kp;                             // shifts per eigenvalue and round (a multiple of 64)
    const int g = tid / S, s = tid - g * S;
    // round one left a bracket of 1/513 of the spectrum's extent; each further round divides it by S + 1: two rounds of
    // 257 reach 3e-8 of the extent, half a unit in the last place of the largest eigenvalue
    const int rounds = (2 * S >= TE_THREADS) ? 2 : 3;
    for (int round = 0; round < rounds; ++round) {
      bool below = false;
      float a = 0.f, b = 0.f;
      if (g < kb) {
        a = br_a[g0 + g]; b = br_b[g0 + g];
        below = sturm(a + (b - a) * ((float)(s + 1) / (float)(S + 1))) <= n - 1 - (g0 + g);
      }
      const int c = __popcll(__ballot(below));
      if (lane == 0) wc[wave] = c;
      __syncthreads();
      if (tid < kb) {
        const float a2 = br_a[g0 + tid], b2 = br_b[g0 + tid];
        int p = 0;
        for (int w = 0; w < S / 64; ++w) p += wc[tid * (S / 64) + w];
        // counts are monotone in the shift: the first p shifts are at or below the eigenvalue
        if (p > 0) br_a[g0 + tid] = a2 + (b2 - a2) * ((float)p / (float)(S + 1));
        if (p < S) br_b[g0 + tid] = a2 + (b2 - a2) * ((float)(p + 1) / (float)(S + 1));
      }
      __syncthreads();
    }
    if (tid < kb) th[g0 + tid] = 0.5f * (br_a[g0 + tid] + br_b[g0 + tid]);
    __syncthreads();
  }
  if (tid >= k && tid < k0) th[tid] = 0.f;

  // ---- 3. eigenvectors of S: inverse iteration, lane i of wave 0 owns eigenvector b0 + i; 4. back-transformation
  // w = H_0 H_1 ... z, one wave per eigenvector, lane l holds entries l and l + 64
  float* Wv = (k0 > TE_BATCH) ? zz + m * KS : lu;               // [k][m]; a single pass leaves it where the factors were
  for (int b0 = 0; b0 < k; b0 += TE_BATCH) {
    const int kb = min(TE_BATCH, k - b0);
    // start: a fixed right-hand side of the first back substitution, pseudo-random from vector to vector too (vectors of a multiple
    // eigenvalue are told apart by nothing else)
    for (int e = tid; e < n * KS; e += TE_THREADS) {
      uint32_t h = (uint32_t)(e / KS) * 2654435761u + (uint32_t)(b0 + e % KS + 1) * 2246822519u;
      h ^= h >> 15; h *= 2246822519u; h ^= h >> 13; h *= 3266489917u; h ^= h >> 16;
      lu[5 * m * KS + e] = (float)(int)h * (1.f / 4294967296.f);
    }
    __syncthreads();
    if (wave == 0) {
      float* za = zz + lane;
      float* zb = lu + 5 * m * KS + lane;                      // second vector buffer (behind the factors)
      // Eigenvalues that agree to 3e-6 of the largest share a shift just above them: with their own, each accurate to 1e-7, the vectors
      // of an exact multiple lean towards whichever of its shifts is nearest, and what tells them apart is lost.
      const float close = 25.f * scal[3];
      bool shared = false;
      float big = 0.f;
      if (lane < kb) {
        int top = b0 + lane;
        while (top > 0 && th[top - 1] - th[top] <= close) --top;
        shared = top < b0 + lane || (top + 1 < k && th[top] - th[top + 1] <= close);
        te_factor<KS>(dv, ev, n, shared ? th[top] + 0.5f * close : th[top], scal[3], lu + lane);
        // Two solves, the first one without its row operations (a random right-hand side is one as well as the other): theta is within
        // 1e-7 of the spectrum's extent of the eigenvalue, so a solve shrinks the rest of the vector by the gap over that, and two
        // leave nothing that single precision could tell.  Between them the iterate is only rescaled by its largest magnitude (the
        // squares of the last normalisation cannot overflow, and nothing else depends on the length).
        big = te_backward<KS>(lu + lane, n, zb, za);
      }
      // Those under one shift are made orthogonal between the solves, three here; rounding that this enlarges lies outside their subspace, where the
      // next solve shrinks it.  (With two solves and start vectors that differed little from each other, offsets of planted multiples among
      // small eigenvalues were off by up to 7e-2.)
      const uint64_t together = __ballot(shared);
      for (int left = together ? 2 : 1; left > 0; --left) {
        if (together) te_separate<KS>(zz, th + b0, n, kb, close, together);
        if (lane < kb) {
          te_forward<KS>(lu + lane, n, za, zb, (big > 0.f && big < INFINITY) ? 1.f / big : 1.f);
          big = te_backward<KS>(lu + lane, n, zb, za);
        }
      }
      if (lane < kb) {
        scal[8 + lane] = big;                                  // the waves of the back-transformation bring it to unit length
      }
    }
    __syncthreads();
    float w0 = 0.f, w1 = 0.f;
    if (wave < kb) {
      w0 = (lane < n) ? zz[lane * KS + wave] : 0.f;
      w1 = (lane + 64 < n) ? zz[(lane + 64) * KS + wave] : 0.f;
      {
        // unit length (scaled by the largest magnitude first, so that the squares cannot overflow); this also clears what
        // is left of the start vector in blocks that S decouples from this eigenvalue (an exactly zero sub-diagonal
        // entry), exact zeros in exact arithmetic: after two solves the square of 1e-7 over the relative gap to that block's
        // eigenvalues, 1e-14 where the gap is of the order of the spectrum's extent (a smaller gap leaves more than the bound
        // below, but less than the rounding of T itself does to such a vector)
        const float big = scal[8 + wave];
        const float sc = (big > 0.f && big < INFINITY) ? 1.f / big : 1.f;
        w0 *= sc; w1 *= sc;
        const float nn = te_wave_sum(fmaf(w0, w0, w1 * w1));
        const float rn = (nn > 0.f) ? rsqrtf(nn) : 0.f;
        w0 *= rn; w1 *= rn;
        if (fabsf(w0) < 1e-12f) w0 = 0.f;
        if (fabsf(w1) < 1e-12f) w1 = 0.f;
      }
      // Two reflectors at a time: (I - b2 v2 v2^T)(I - b1 v1 v1^T) w needs v1.w, v2.w and v1.v2, three sums that go through the wave
      // together; the next pair is fetched meanwhile.
      const int ia = lane < m ? lane : -1, ib = lane + 64 < m ? lane + 64 : -1;      // entries of this lane; -1: none
      int j = min(n - 2, m - 3);                               // the last reflector
      float p0 = 0.f, p1 = 0.f, q0 = 0.f, q1 = 0.f, bp = 0.f, bq = 0.f;
      auto fetch = [&](const int jj) {                         // reflectors jj and jj - 1
        const int a = max(jj, 0), b = max(jj - 1, 0), oa = tri_refl_off(m, a) + lane, ob = tri_refl_off(m, b) + lane;
        const float a0 = Rf[max(oa, 0)], a1 = Rf[oa + 64], b0 = Rf[max(ob, 0)], b1 = Rf[ob + 64];
        p0 = (ia > a) ? a0 : 0.f; p1 = (ib > a) ? a1 : 0.f; q0 = (ia > b) ? b0 : 0.f; q1 = (ib > b) ? b1 : 0.f;
        bp = bet[a]; bq = bet[b];
      };
      fetch(j);
      for (; j >= 1; j -= 2) {
        const float v0 = p0, v1 = p1, u0 = q0, u1 = q1, b1 = bp, b2 = bq;
        fetch(j - 2);
        float g1, g2, c;
        te_wave_sum3(fmaf(v0, w0, v1 * w1), fmaf(u0, w0, u1 * w1), fmaf(v0, u0, v1 * u1), g1, g2, c);
        const float s1 = b1 * g1, s2 = b2 * fmaf(-s1, c, g2);  // beta = 0: an identity reflector
        w0 = fmaf(-s2, u0, fmaf(-s1, v0, w0)); w1 = fmaf(-s2, u1, fmaf(-s1, v1, w1));
      }
      if (j == 0) {
        const float s = bp * te_wave_sum(fmaf(p0, w0, p1 * w1));
        w0 = fmaf(-s, p0, w0); w1 = fmaf(-s, p1, w1);
      }
    }
    __syncthreads();                                           // every wave has read its column of zz / lu is free
    if (wave < kb) {
      if (lane < m) Wv[(b0 + wave) * m + lane] = w0;
      if (lane + 64 < m) Wv[(b0 + wave) * m + lane + 64] = w1;
    }
    __syncthreads();
  }
  if (wave == 0) {                                             // Gram-Schmidt over the k vectors, in order
    for (int i = 0; i < k; ++i) {
      float x0 = (lane < m) ? Wv[i * m + lane] : 0.f, x1 = (lane + 64 < m) ? Wv[i * m + lane + 64] : 0.f;
      for (int j = 0; j < i; ++j) {
        const float y0 = (lane < m) ? Wv[j * m + lane] : 0.f, y1 = (lane + 64 < m) ? Wv[j * m + lane + 64] : 0.f;
        const float dt = te_wave_sum(fmaf(x0, y0, x1 * y1));
        x0 = fmaf(-dt, y0, x0); x1 = fmaf(-dt, y1, x1);
      }
      const float nn = te_wave_sum(fmaf(x0, x0, x1 * x1));
      const float rn = (nn > 0.f) ? rsqrtf(nn) : 0.f;
      if (lane < m) Wv[i * m + lane] = x0 * rn;
      if (lane + 64 < m) Wv[i * m + lane + 64] = x1 * rn;
    }
  }
  __syncthreads();
  *theta = th;
  *W = Wv;
}

}  // namespace obf
