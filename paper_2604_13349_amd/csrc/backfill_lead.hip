// Orthogonal BackFill (Sec. 4.4, Eq. 3-7) for the heads that want a few leading directions: everything after the statistics pass in
// one kernel, one workgroup per head.
//
//   1. G = V_del^T V_del is summed from its partials into registers (wave w holds columns 16 w .. 16 w + 15) and projected in place,
//      G <- P G P with P = I - Q^T Q: two left projections on the matrix cores with a transposition through LDS between them.
//   2. The leading eigenvectors of P G P, the top right singular vectors of R, by a block iteration on the matrix cores:
//      Chebyshev polynomials of P G P applied to a block of 8 or 16 vectors, a Rayleigh-Ritz step after each, until the residual has
//      reached the rounding of the matrix.  Its cost depends on the spectrum: three to five steps and ten to twenty products on the
//      caches that the benchmark draws; clusters wider than the block would take it too long and go to the direct route of tri_eigs.hpp
//      on the same matrix.
//   3. App. H's literal Gram subspace iteration, when asked for, on the same registers.
//   4. rbar, Delta, delta and Eq. 7.
//
// What bounds it is latency: chains of small products with a barrier each (1600 cycles, of which the matrix cores work 500 for eight columns, 800 for
// sixteen) and the small problems on one wave (6500 cycles a step for eight columns, 14000 for sixteen, a sweep of rotations 2000 and 4500 of them).
// At m = 96, k = 2 a workgroup alone on its compute unit takes 50 us: G 4, the projection 8, sixteen products 12, four small problems 12 with 5 around
// them, the rest loads and the tail; two that share one take 73, most of the difference in the projection (14), which fills the vector ALU, the matrix
// cores and LDS in turn, and so 288 heads on 256 compute units take 73 where 256 take 54.  With the middle parts in the block's free columns, a sweep
// for the early small problems and the parts by conversion instructions 288 such heads went from 80 us to 73.  The kernel took the place
// of a basis of the complement, the tridiagonalisation of its m x m matrix and inverse iteration (68 + 148 us for 288 heads of 256 tokens with 32
// kept, 2 directions; 73 now, the whole call 299 -> 128; twelve samples, four in flight, 2060 -> 857), and the offset's error against double
// precision fell from 8.6e-7 to 3.3e-7 (2000 tokens with 96 kept, 8 directions: 4.0e-6 to 5.0e-7).
//
// What it depends on: this kernel against those before it (us, 288 heads), and the whole call when it took their place
//   256 tokens, 32 kept    2, 8, 12, 16 directions   210 223 272 282 -> 73 96 129 166    299 312 360 369 -> 155 173 201 241
//   1024 tokens, 80 kept                             165 172 199 207 -> 101 125 154 193  331 338 365 373 -> 244 263 286 330
//   2000 tokens, 96 kept                             130 136 156 163 -> 105 128 149 187  366 371 390 395 -> 311 327 353 391
//   1024 tokens, 112 kept                             99 103 118 123 -> 94 93 93 93      316 320 336 340 -> 299 301 301 300
// A narrow complement costs as much as a wide one here, the kernels before it worked in its own coordinates: at 32 columns they are ahead from
// thirteen directions on, and where the direct route takes over after the first products (eigenvalues closer than the block can tell
// apart, 2 directions: complements 96, 64, 32 and 20 wide 308 300 267 275 -> 355 338 315 327).
#include "common.hpp"
#include "wave_ops.hpp"
#include "tri_eigs.hpp"
#include "ritz.hpp"
#include "backfill_emit.hpp"

namespace obf {

constexpr int LE_XTILE = 68;             // float4 of one wave's 16 x 16 tile of a block in LDS: four rows of 16, one apart for the banks
constexpr int LE_LDR = 132;              // floats between rows of a subspace basis in LDS
// The widths and limits of the block iteration.  Eight columns for up to four directions (a sweep of the small problem costs 2000 cycles
// against 5000, which the slower convergence does not make up), sixteen for more; up to twelve directions at a time (twelve together:
// the whole call takes 206 us for 288 heads of 256 tokens with 32 kept and 339 with 96 of 2000; as eight and four: 226 and 363), the thirteenth on in groups of eight.
constexpr int kBlockMaxRank = 12;        // most directions the block iteration is asked for at a time
constexpr int kThinWidth = 16;           // complements no wider than this are spanned by a block
constexpr int kGroups = 4;               // most times that it goes on with the rest of the matrix
// A wanted eigenvalue below this share of the first sends the head to the direct route: the residual, which is relative to the first, no longer
// tells whether its direction has settled, and the block's columns grow so differently that single precision loses some of them.  (Offsets of planted
// ladders against double precision, worst of 150 heads: 0.546^i, 12 directions 1e-3 by the block iteration, 9e-7 this way, 425 and 200 us;
// 0.38^i, 8 directions 3.5e-4 and 2e-6, 360 and 187 us.  The benchmark's caches have 0.1 at twelve directions and about 0.03 at sixteen.)
constexpr float kSteep = 1.f / 128;
constexpr float kLeftShare = 1.5e-6f;    // what the direct route may drop, relative to ||P G P||_F (whose rounding is about a tenth of that)
constexpr int kBlockRounds = 12;         // most Rayleigh-Ritz steps of it
constexpr int kBlockSteps = 24;          // highest polynomial degree between two of them
constexpr int kBlockReach = 80;          // products still to come beyond which a head takes the direct route (which takes as long as 100 to 180)

// Floats of dynamic LDS: the whole matrix or operands from Q, then (in the same place) the block's two copies, the partial Gram matrices and the
// subspace's rows, or the scratch of the direct route.  (All of it in 16-byte pieces: on a base off that alignment the iteration took twice as long.)
__host__ __device__ inline int lead_block_floats(int d) { return 2 * 3 * (d / 32) * 64 * 4 + 2 * (d / 16) * LE_XTILE * 4 + 2 * (d / 16) * 64 * 4 + 16 * LE_LDR + 16; }
__host__ __device__ inline int lead_direct_floats(int d, int kq) { return ((tri_refl_floats(d) + 3) & ~3) + tri_work_floats(d, kq); }
inline size_t lead_lds_floats(int d, int kq) {
  int n = lead_block_floats(d);
  n = n > lead_direct_floats(d, kq) ? n : lead_direct_floats(d, kq);
  n = n > 2 * 16 * LE_LDR ? n : 2 * 16 * LE_LDR;
  n = n > d * (d + 4) ? n : d * (d + 4);
  return (size_t)n;                      // (the operands of 32 rows of Q take 384 d bytes)
}

// orth of App. H's iteration for one wave: Gram-Schmidt over the kk <= KQ rows of Yb (ldr floats apart, D entries) in order, two passes
// each; a row left with at most 1e-5 of the first row's norm depends on the rows before it and is dropped.  The kept rows go to Ya;
// returns their number.  All rows are in registers, a pass takes the coefficients on all earlier rows at once (a dropped row is zero).
// Ya and Yb are places in the dynamic LDS.  Not inlined: see lead_direct.
template <int KQ, int D>
__device__ __attribute__((noinline)) int lead_orth(const int at_a, const int at_b, const int kk) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  float* Ya = sm + at_a;
  const float* Yb = sm + at_b;
  const int lane = threadIdx.x & 63;
  float x0[KQ], x1[KQ];
#pragma unroll
  for (int i = 0; i < KQ; ++i) {
    x0[i] = (i < kk) ? Yb[i * LE_LDR + lane] : 0.f;
    x1[i] = (D > 64 && i < kk) ? Yb[i * LE_LDR + lane + 64] : 0.f;
  }
  int nk = 0;
  float first = -1.f;
#pragma unroll
  for (int i = 0; i < KQ; ++i) {
    if (i < kk) {
#pragma unroll
      for (int pass = 0; pass < 2; ++pass) {
        float g[KQ + 2];
#pragma unroll
        for (int j = 0; j < i; j += 3) {
          const int j1 = (j + 1 < i) ? j + 1 : j, j2 = (j + 2 < i) ? j + 2 : j;
          te_wave_sum3(fmaf(x0[i], x0[j], x1[i] * x1[j]), fmaf(x0[i], x0[j1], x1[i] * x1[j1]), fmaf(x0[i], x0[j2], x1[i] * x1[j2]),
                       g[j], g[j + 1], g[j + 2]);
        }
#pragma unroll
        for (int j = 0; j < i; ++j) { x0[i] = fmaf(-g[j], x0[j], x0[i]); x1[i] = fmaf(-g[j], x1[j], x1[i]); }
      }
      const float nn = sqrtf(te_wave_sum(fmaf(x0[i], x0[i], x1[i] * x1[i])));
      if (first < 0.f) first = nn;
      const bool kept = first > 0.f && nn > 1e-5f * first;
      const float rn = kept ? 1.f / nn : 0.f;
      x0[i] = kept ? x0[i] * rn : 0.f; x1[i] = kept ? x1[i] * rn : 0.f;
      if (kept) {
        Ya[nk * LE_LDR + lane] = x0[i];
        if (D > 64) Ya[nk * LE_LDR + lane + 64] = x1[i];
        ++nk;
      }
    }
  }
  return nk;
}

// acc <- (I - Q^T Q) acc for the wave's sixteen columns: tile t of acc holds rows 16 t + 4 q + e of column 16 w + j.  Q is taken 32 rows at a
// time (rows past r as zeros), split into its parts once for all waves and left in LDS as operands of both products: Q acc, whose result
// comes out in the layout in which it is the operand of the update, and Q^T (Q acc).  Every thread must call.  In single precision on
// the matrix cores, with Q read by every wave, 32 rows took 10500 cycles instead of 8500 (r = 32, one workgroup on the CU: LDS reads,
// splits and matrix instructions take 3000 each and hardly overlap between waves in step).
template <int D>
struct QRows {                           // a thread's share of 32 rows of Q on its way to LDS: operands of either product
  static constexpr int NP = D / 32, COUNT = 2 * NP * 64, EACH = (COUNT + TE_THREADS - 1) / TE_THREADS;
  f32x4 ra[EACH], rb[EACH], ca[EACH], cb[EACH];
  __device__ __forceinline__ void fetch(const float* __restrict__ Qb, const int r, const int base) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < EACH; ++u) {
      const int f = u * TE_THREADS + tid, fq = (f >> 4) & 3, fj = f & 15, g = f >> 6;        // operand g of either kind
      if (COUNT % TE_THREADS == 0 || f < COUNT) {
        const int row = base + 16 * (g / NP) + fj;
        const float* qr = Qb + (size_t)min(row, r - 1) * D + 32 * (g % NP) + 4 * fq;
        ra[u] = *(const f32x4*)qr; rb[u] = *(const f32x4*)(qr + 16);
        if (row >= r) { ra[u] = f32x4{0.f, 0.f, 0.f, 0.f}; rb[u] = ra[u]; }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int k = base + 4 * fq + e;
          const float a = Qb[(size_t)min(k, r - 1) * D + 16 * g + fj], b = Qb[(size_t)min(k + 16, r - 1) * D + 16 * g + fj];
          ca[u][e] = (k < r) ? a : 0.f; cb[u][e] = (k + 16 < r) ? b : 0.f;
        }
      }
    }
  }
};

// next: the first 32 rows, fetched by the caller; left with them again when `again` is set
template <int D>
__device__ __forceinline__ void project_columns(f32x4 (&acc)[D / 16], const float* __restrict__ Qb, const int r, bf16x8* qs, const bool own,
                                                QRows<D>& next, const bool again) {
  constexpr int NT = D / 16, NP = D / 32, EACH = QRows<D>::EACH;
  const int tid = threadIdx.x, lane = tid & 63;
  bf16x8* rows = qs;                                           // [3][2][NP][64]: rows 16 a + j, columns 32 p + 4 q .. and 32 p + 16 + 4 q ..
  bf16x8* cols = qs + 3 * 2 * NP * 64;                         // [3][NT][64]: column 16 t + j, rows 4 q .. and 16 + 4 q ..
  for (int base = 0; base < r; base += 32) {
    __syncthreads();                                           // the rows before these are read
#pragma unroll
    for (int u = 0; u < EACH; ++u) {
      const int f = u * TE_THREADS + tid;
      if (2 * NP * 64 % TE_THREADS == 0 || f < 2 * NP * 64) {
        const Split8 x = split8(next.ra[u], next.rb[u]), y = split8(next.ca[u], next.cb[u]);
        rows[f] = x.hi; rows[2 * NP * 64 + f] = x.mid; rows[2 * 2 * NP * 64 + f] = x.lo;
        cols[f] = y.hi; cols[NT * 64 + f] = y.mid; cols[2 * NT * 64 + f] = y.lo;
      }
    }
    __syncthreads();
    if (base + 32 < r || again) next.fetch(Qb, r, base + 32 < r ? base + 32 : 0);
    if (!own) continue;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 s[2][3];
#pragma unroll
    for (int a = 0; a < 2; ++a) { s[a][0] = zero; s[a][1] = zero; s[a][2] = zero; }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const Split8 v = split8(acc[2 * p], acc[2 * p + 1]);
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const bf16x8* o = rows + (a * NP + p) * 64 + lane;
        const bf16x8 hi = o[0], mid = o[2 * NP * 64], lo = o[2 * 2 * NP * 64];
        s[a][0] = mfma32(hi, v.hi, s[a][0]);
        s[a][1] = mfma32(hi, v.mid, s[a][1]);
        s[a][2] = mfma32(hi, v.lo, s[a][2]);
        s[a][1] = mfma32(mid, v.hi, s[a][1]);
        s[a][2] = mfma32(mid, v.mid, s[a][2]);
        s[a][2] = mfma32(lo, v.hi, s[a][2]);
      }
    }
    __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);         // operands one step ahead of the products
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (p + 1 < NP) __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 12, 0);
    }
    const Split8 c = split8(zero - (s[0][0] + (s[0][1] + s[0][2])), zero - (s[1][0] + (s[1][1] + s[1][2])));   // -(Q acc), rows 4 q + e and 16 + 4 q + e
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const bf16x8* o = cols + t * 64 + lane;
      const bf16x8 hi = o[0], mid = o[NT * 64], lo = o[2 * NT * 64];
      f32x4 y0 = mfma32(hi, c.hi, acc[t]), y1 = mfma32(hi, c.mid, zero), y2 = mfma32(hi, c.lo, zero);
      y1 = mfma32(mid, c.hi, y1);
      y2 = mfma32(mid, c.mid, y2);
      y2 = mfma32(lo, c.hi, y2);
      acc[t] = y0 + (y1 + y2);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t + 2 < NT) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
    }
  }
}

// vec <- vec - Q^T (Q vec) for a vector of D entries in LDS; coef [128] and part [512] are scratch.  Every thread must call.  Eight rows of a
// wave, then sixteen entries of a column per thread, in flight at a time; the rows' sums go through the wave together.
template <int D>
__device__ __forceinline__ void project_vector(const float* __restrict__ Qb, const int r, float* vec, float* coef, float* part) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float u0 = vec[lane], u1 = (D > 64) ? vec[lane + 64] : 0.f;
  if (tid >= r && tid < 128) coef[tid] = 0.f;
#pragma unroll 1
  for (int k0 = wave; k0 < r; k0 += 8 * TE_WAVES) {
    float s[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {                              // rows past the last: the last one again, not stored
      const float* qr = Qb + (size_t)min(k0 + TE_WAVES * c, r - 1) * D + lane;
      s[c] = (D > 64) ? fmaf(qr[D > 64 ? 64 : 0], u1, qr[0] * u0) : qr[0] * u0;
    }
    // 16-lane row 2 a + b is left with the sums of rows 4 a + 2 b and 4 a + 2 b + 1
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(s[c]), __float_as_uint(s[c + 4]), false, false);
      s[c] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(s[c]), __float_as_uint(s[c + 2]), false, false);
      s[c] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
      s[c] += row_xor<1>(s[c]);
      s[c] += row_xor<2>(s[c]);
      s[c] += row_xor<7>(s[c]);
      s[c] += row_xor<15>(s[c]);
    }
    const int k = k0 + TE_WAVES * ((lane >> 5) * 4 + ((lane >> 4) & 1) * 2 + (lane & 1));
    if ((lane & 15) < 2 && k < r) coef[k] = (lane & 1) ? s[1] : s[0];
  }
  {
    const int g = tid >> 7, c = tid & (D - 1);
    float s = 0.f;
    bool synced = false;
#pragma unroll 1
    for (int k0 = g; k0 < r + g; k0 += 64) {                   // uniform: the same number of rounds for every thread
      float z[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) z[k] = Qb[(size_t)min(k0 + 4 * k, r - 1) * D + c];
      if (!synced) __syncthreads();
      synced = true;
#pragma unroll
      for (int k = 0; k < 16; ++k) s = fmaf(coef[k0 + 4 * k], z[k], s);
    }
    part[tid] = s;
  }
  __syncthreads();
  if (tid < D) vec[tid] -= (part[tid] + part[128 + tid]) + (part[256 + tid] + part[384 + tid]);
  __syncthreads();
}

// Where the block iteration's arrays lie in the dynamic LDS.
template <int D>
struct BlockLds {
  static constexpr int NT = D / 16;
  bf16x4* sbuf;                          // [2][3][NT / 2][64][2] the block in its three parts, two copies
  float4* xbuf;                          // [2][NT][LE_XTILE] the blocks X and Y for their transposition
  f32x4* gbuf;                           // [2][NT][64] partial X^T X and X^T Y
  float* rows;                           // [16][LE_LDR]
  float* lam;                            // [16]
  __device__ __forceinline__ BlockLds(float* sm) {
    sbuf = (bf16x4*)sm;
    xbuf = (float4*)(sbuf + 2 * 3 * NT * 64);
    gbuf = (f32x4*)(xbuf + 2 * NT * LE_XTILE);
    rows = (float*)(gbuf + 2 * NT * 64);
    lam = rows + 16 * LE_LDR;
  }
};

// a block in its three parts to LDS, each wave's sixteen rows
template <int D>
__device__ __forceinline__ void publish(bf16x4* b, const f32x4 x) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const Split s = split3(x);
  bf16x4* o = b + ((wave >> 1) * 64 + lane) * 2 + (wave & 1);
  o[0] = s.hi; o[D / 16 * 64] = s.mid; o[2 * (D / 16) * 64] = s.lo;
}

// y0 + y1 + y2 += a times rows 32 p .. of the block b
template <int D>
__device__ __forceinline__ void multiply(const Split8& a, const bf16x4* b, const int p, f32x4& y0, f32x4& y1, f32x4& y2) {
  const bf16x8* v = (const bf16x8*)b + (threadIdx.x & 63);
  const bf16x8 hi = v[p * 64], mid = v[(D / 32 + p) * 64], lo = v[(D / 16 + p) * 64];
  y0 = mfma32(a.hi, hi, y0);
  y1 = mfma32(a.hi, mid, y1);
  y2 = mfma32(a.hi, lo, y2);
  y1 = mfma32(a.mid, hi, y1);
  y2 = mfma32(a.mid, mid, y2);
  y2 = mfma32(a.lo, hi, y2);
}

// The same for a block of eight columns: the middle parts take the place of columns 8 - 15, so that four products do where six are needed
// for sixteen columns, and two reads of LDS, which each wave makes of the whole block, where three are.
template <int D>
__device__ __forceinline__ void publish_narrow(bf16x4* b, const f32x4 x) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const Split s = split3(x);
  bf16x4* o = b + ((wave >> 1) * 64 + lane) * 2 + (wave & 1);
  if ((lane & 15) < 8) { o[0] = s.hi; o[16] = s.mid; o[D / 16 * 64] = s.lo; }
}

// columns 0 - 7: y0 + y1 + y2 + y3, columns 8 - 15: y0 + y1 + y3, += their shares of a times rows 32 p .. (y2's columns 8 - 15 are not defined)
template <int D>
__device__ __forceinline__ void multiply_narrow(const Split8& a, const bf16x4* b, const int p, f32x4& y0, f32x4& y1, f32x4& y2, f32x4& y3) {
  const bf16x8* v = (const bf16x8*)b + (threadIdx.x & 63);
  const bf16x8 him = v[p * 64], lo = v[(D / 32 + p) * 64];
  y0 = mfma32(a.hi, him, y0);
  y1 = mfma32(a.mid, him, y1);
  y2 = mfma32(a.hi, lo, y2);
  y3 = mfma32(a.lo, him, y3);
}

// entry (row, j) of a start block, in [-1, 1), fixed
__device__ __forceinline__ float block_random(const int row, const int j, const int seed) {
  uint32_t h = (uint32_t)(row * 16 + j) * 2654435761u + (uint32_t)seed * 40503u + 12345u;
  h ^= h >> 15; h *= 2246822519u; h ^= h >> 13; h *= 3266489917u; h ^= h >> 16;
  return (float)(int)h * (1.f / 2147483648.f);
}

// The direct route on the D x D matrix Tg, in the workgroup's dynamic LDS: where in it the eigenvalues and the eigenvectors (D floats apart)
// lie.  A function of its own, not inlined: its register tiles otherwise push values of the block iteration's loops to scratch.
struct DirectResult { int theta, W; };
template <int D>
__device__ __attribute__((noinline)) DirectResult lead_direct(const float* Tg, int kq) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  float f = 0.f;                                               // ||P G P||_F
  for (int e = threadIdx.x; e < D * D / 4; e += TE_THREADS) {
    const f32x4 t = *(const f32x4*)(Tg + 4 * e);
    f += fmaf(t[0], t[0], t[1] * t[1]) + fmaf(t[2], t[2], t[3] * t[3]);
  }
  f = te_wave_sum(f);
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = f;
  __syncthreads();
  f = 0.f;
#pragma unroll
  for (int w = 0; w < TE_WAVES; ++w) f += sm[w];
  __syncthreads();
  const float left_tol = kLeftShare * sqrtf(f);
  float* work = sm + ((tri_refl_floats(D) + 3) & ~3);          // 16-byte aligned
  const float* th;
  const float* Wk;
  int md = D;
  asm volatile("" : "+s"(md));                                 // (loops unrolled for a width known to the compiler spill)
  const int n = tri_start<D / 32>(Tg, D, sm, md, left_tol, work);
  if (kq <= 4) tri_top_eigs<4>(sm, md, n, kq, work, &th, &Wk);
  else tri_top_eigs<8>(sm, md, n, kq, work, &th, &Wk);
  return DirectResult{(int)(th - sm), (int)(Wk - sm)};
}

// One wave's sixteen rows of the symmetric D x D matrix `from` to `to` (which may be the same), less X Y^T + (Y - X Lambda) X^T: kc <= 16
// eigenvectors X, LE_LDR floats apart, their images Y likewise and their Rayleigh quotients, at places in the dynamic LDS.  Each lane reads
// back only what it has written itself.  Not inlined: see lead_direct.
template <int D>
__device__ __attribute__((noinline)) void lead_deflate(const float* from, float* to, const int at_x, const int at_y, const int at_lam, const int kc) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const int lane = threadIdx.x & 63, q = lane >> 4, j = lane & 15, wave = threadIdx.x >> 6;
  const float* X = sm + at_x;
  const float* Y = sm + at_y;
  float xa[4], ya[4], th[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {                                // vector 4 s + q
    const int c = 4 * s + q;
    const bool in = c < kc;
    xa[s] = in ? X[c * LE_LDR + 16 * wave + j] : 0.f;
    ya[s] = in ? Y[c * LE_LDR + 16 * wave + j] : 0.f;
    th[s] = in ? sm[at_lam + c] : 0.f;
  }
  const size_t at = (size_t)(16 * wave + j) * D + 4 * q;
#pragma unroll 1
  for (int t = 0; t < D / 16; ++t) {
    f32x4 g = *(const f32x4*)(from + at + 16 * t);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int c = 4 * s + q;
      const float a = (c < kc) ? X[c * LE_LDR + 16 * t + j] : 0.f, b = (c < kc) ? Y[c * LE_LDR + 16 * t + j] : 0.f;
      g = __builtin_amdgcn_mfma_f32_16x16x4f32(-a, ya[s], g, 0, 0, 0);
      g = __builtin_amdgcn_mfma_f32_16x16x4f32(fmaf(th[s], a, -b), xa[s], g, 0, 0, 0);
    }
    *(f32x4*)(to + at + 16 * t) = g;
  }
}

// The exact directions of a head whose complement is only m <= kThinWidth wide, from G itself (D x D, of which a lane reads what it wrote): an orthonormal
// basis of the complement from m random vectors, projected and orthonormalised until nothing depended on the rest twice in a row
// (twice in all, as a rule), then one Rayleigh-Ritz step, which is the whole eigenproblem.  Leaves the m vectors in the block's rows and
// the Ritz values, descending and then zeros, in lam; ends with a barrier.  Not inlined: see lead_direct (the operands of the projection
// beside the matrix of the block iteration fill the registers).
template <int D>
__device__ __attribute__((noinline)) void lead_thin(const float* Q_, const float* G_, const int r_, const int m_) {
  constexpr int NT = D / 16;
  // (a function of its own sees neither that its arguments are the same in all lanes nor that the pointers are to global memory)
  typedef const __attribute__((address_space(1))) float* Global;
  typedef const __attribute__((address_space(1))) f32x4* Global4;
  auto same = [](const float* p) -> Global {
    const uint64_t u = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)u), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(u >> 32));
    return (Global)(((uint64_t)hi << 32) | lo);
  };
  const Global Qb = same(Q_), G = same(G_);
  const int r = __builtin_amdgcn_readfirstlane(r_), m = __builtin_amdgcn_readfirstlane(m_);
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const BlockLds<D> lds(sm);
  float4* s_rot = lds.xbuf + NT * LE_XTILE;                    // [64], where the block iteration has Y
  const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, j = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool own = wave < NT;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 x = zero, y = zero;
  // X <- X - Q^T (Q X): wave w takes rows 16 w .. of Q X (in place of the partial Gram matrices), then its rows of the update
  auto project = [&]() {
    bf16x4 *b = lds.sbuf, *bs = (bf16x4*)lds.gbuf;
    if (own) publish<D>(b, x);
    f32x4 qa[NT / 2][2], qc[NT / 2][2];
    const bool in = 16 * wave + j < r;
    int last = r - 1;
    asm volatile("" : "+s"(last));                           // (the rows' places, kept from one projection to the next, fill the registers)
    if (own) {
      const uint32_t at = (uint32_t)(min(16 * wave + j, last) * D + 4 * q);
#pragma unroll
      for (int p = 0; p < NT / 2; ++p) {
        qa[p][0] = *(Global4)(Qb + at + 32 * p); qa[p][1] = *(Global4)(Qb + at + 32 * p + 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int k = 32 * p + 4 * q + e;                    // rows past the last: Q X is zero there
          qc[p][0][e] = Qb[(uint32_t)(min(k, last) * D + 16 * wave + j)]; qc[p][1][e] = Qb[(uint32_t)(min(k + 16, last) * D + 16 * wave + j)];
        }
      }
    }
    lds_barrier();
    if (own) {
      f32x4 y0 = zero, y1 = zero, y2 = zero;
#pragma unroll
      for (int p = 0; p < NT / 2; ++p) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { if (!in) { qa[p][0][e] = 0.f; qa[p][1][e] = 0.f; } }
        multiply<D>(split8(qa[p][0], qa[p][1]), b, p, y0, y1, y2);
      }
      publish<D>(bs, y0 + (y1 + y2));
    }
    lds_barrier();
    if (own) {
      f32x4 y0 = zero, y1 = zero, y2 = zero;
#pragma unroll
      for (int p = 0; p < NT / 2; ++p) multiply<D>(split8(qc[p][0], qc[p][1]), bs, p, y0, y1, y2);
      x -= y0 + (y1 + y2);
    }
    lds_barrier();
  };
  // X <- X S; the Ritz values (basis_only: one, or zero where dropped) in lam
  auto small_problem = [&](const bool basis_only) {
    float4* xb = lds.xbuf + wave * LE_XTILE;
    if (own) {
      lds.gbuf[wave * 64 + lane] = mul_t(x, x, zero);
      lds.gbuf[(NT + wave) * 64 + lane] = basis_only ? mul_t(x, x, zero) : mul_t(y, x, mul_t(x, y, zero)) * 0.5f;
      xb[q * 17 + j] = make_float4(x[0], x[1], x[2], x[3]);
    }
    lds_barrier();
    if (wave == 0) {
      f32x4 M = lds.gbuf[lane], H = lds.gbuf[NT * 64 + lane];
#pragma unroll
      for (int w = 1; w < NT; ++w) { M += lds.gbuf[w * 64 + lane]; H += lds.gbuf[(NT + w) * 64 + lane]; }
      f32x4 S;
      float theta;
      int place;
      const int sweeps = basis_only ? 0 : 12;
      if (m <= 8) small_ritz<8>(M, H, 1e-6f, 3e-4f, sweeps, S, theta, place);
      else small_ritz<16>(M, H, 1e-6f, 3e-4f, sweeps, S, theta, place);
      s_rot[q * 16 + place] = make_float4(S[0], S[1], S[2], S[3]);
      if (q == 0) lds.lam[place] = theta;
    }
    lds_barrier();
    if (own) {
      const float4 s4 = s_rot[lane];
      const float* xs = (const float*)(xb + (j >> 2) * 17 + 4 * q) + (j & 3);
      f32x4 xt;
#pragma unroll
      for (int e = 0; e < 4; ++e) xt[e] = xs[4 * e];
      x = mul_t(xt, f32x4{s4.x, s4.y, s4.z, s4.w}, zero);
    }
  };
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = (j < m) ? block_random(16 * wave + 4 * q + e, j, -1) : 0.f;
  project();
  int whole_before = 0;
  for (int pass = 0; pass < 6 && whole_before < 2; ++pass) {
    small_problem(true);
    const bool all = lds.lam[m - 1] > 0.f;                     // uniform
    whole_before = all ? whole_before + 1 : 0;
    if (!all) {
#pragma unroll
      for (int e = 0; e < 4; ++e) if (j < m && !(lds.lam[j] > 0.f)) x[e] = block_random(16 * wave + 4 * q + e, j, pass);
    }
    project();
  }
  if (own) publish<D>(lds.sbuf, x);
  lds_barrier();
  if (own) {                                                   // Y = G X
    f32x4 y0 = zero, y1 = zero, y2 = zero;
    const Global g = G + (uint32_t)((16 * wave + j) * D + 4 * q);
#pragma unroll
    for (int p = 0; p < NT / 2; ++p) multiply<D>(split8(*(Global4)(g + 32 * p), *(Global4)(g + 32 * p + 16)), lds.sbuf, p, y0, y1, y2);
    y = y0 + (y1 + y2);
  }
  small_problem(false);
  if (own && j < m) *(f32x4*)&lds.rows[j * LE_LDR + 16 * wave + 4 * q] = x;
  __syncthreads();
}

// a value that every lane holds, moved to a scalar register
__device__ __forceinline__ float uniform(const float v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(v)));
}

// FAST selects the fast path of App. H: `iters` steps of C <- orth(C P G P) from a fixed orthonormal start; the exact directions are
// then only found when diagnostics are wanted, to report how far the fast path's Delta is from theirs.  (A kernel of its own: the calls
// to the orthogonalisation push six values of each of its products to scratch.  The compiler reports 37 to 41 registers that go to scratch
// somewhere in the plain kernels of head_dim 128, 116 in this one and 89 to 94 in the THIN ones; at head_dim 64 none, 90 to 94 and 13 to 16.)
// THIN: some heads may retain so many directions that their complement is no wider than a block (kThinWidth).  P G P is not formed for
// those (Q has more rows than there would be products): products with G are followed by a projection of the block, and the block's Ritz
// values give the trace; see lead_thin.  (288 heads of 1024 tokens, 112, 120 and 126 kept, whole call, 8 directions: 302, 316 and 313 us
// with that in here, where its operands pushed the matrix to scratch; 293, 305 and 303 as a function.)
// COLS: the columns of a block, 8 for at most four directions, 16 for more; 0: by what a head has to give, where some may have no more than four deleted
// rows (288 heads of 66 and 99 tokens, 64 and 96 kept, 8 directions: 66 and 85 us, 83 and 97 with sixteen columns).
template <typename T, int D, bool FAST, bool THIN, int COLS>
__global__ __launch_bounds__(TE_THREADS, 4) void k_bf_lead(int nstat, int rank, HeadState* __restrict__ state,
                                                          const float* __restrict__ basis, const float* __restrict__ gram_part,
                                                          float* __restrict__ mats, float* __restrict__ delta,
                                                          float* __restrict__ delta_out, obf_diag_t* __restrict__ diag,
                                                          T* __restrict__ V_out, int max_budget, const float* __restrict__ scores,
                                                          const int32_t* idx, int32_t* moved, int shift, int vflags, int scs, int iters) {
  constexpr int NT = D / 16;
  constexpr bool NARROW = COLS == 8;
  extern __shared__ __attribute__((aligned(16))) float sm[];
  __shared__ float uvec[128], svec[128], coef[128], part[TE_THREADS], dvec[2][16], dex[128];
  __shared__ double dred[TE_WAVES];
  __shared__ __attribute__((aligned(16))) float4 s_rot[64];
  __shared__ float s_th[16], red[TE_WAVES];
  __shared__ int s_k;
  __shared__ float s_val;
  const int head = blockIdx.x;
  HeadState st = state[head];
  int skipped = 1, k_used = 0;
  float rcr = 0.f, ivn = 0.f, pcr = 0.f, pc = 0.f, revr = 0.f, fast_err = -1.f;
  const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, j = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool own = wave < NT;                                  // uniform: the wave holds sixteen rows
  // The wave that solves the small problems: another one in workgroups that share a compute unit (a launch deals its first 256 to one each),
  // so that they do not wait for the same SIMD.
  const int solver = (blockIdx.x / kNumCU) % TE_WAVES;
  if (st.active) {
    const int r = st.r_keep, m = D - r;
    const float* Qb = basis + (size_t)head * D * D;            // [r][D] orthonormal rows
    const size_t pstride = gram_stride(D);
    const float* gp = gram_part + (size_t)head * nstat * pstride;
    QRows<D> next;
    const bool thin = THIN && m <= kThinWidth;                 // uniform
    if (r > 0 && !thin) next.fetch(Qb, r, 0);
    // ---- 1. G, u = sum_j A_j v_j, s = sum_j v_j, ||V_del||^2
    // only the 32 x 32 tiles on and below the diagonal of a partial are defined
    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    {
      // the 16 x 16 tiles (row, col) of those, five (D = 64: at most two) a wave, four partials' loads at a time; through LDS, mirrored
      constexpr int TILES = (D == 128) ? 40 : 12, EACH = (TILES + TE_WAVES - 1) / TE_WAVES;
      int place[EACH];
      f32x4 s[EACH];
#pragma unroll
      for (int u = 0; u < EACH; ++u) {
        // the tile rows hold 2, 2, 4, 4, 6, 6, 8, 8 tiles; pairs of them start at tile 0, 4, 12, 24
        const int n = min(wave + u * TE_WAVES, TILES - 1);
        const int b = n >= 24 ? 3 : n >= 12 ? 2 : n >= 4 ? 1 : 0, in = n - 2 * b * (b + 1), w = 2 * b + 2;
        const int row = 2 * b + (in >= w ? 1 : 0), col = in - (in >= w ? w : 0);
        place[u] = (16 * row + j) * D + 16 * col + 4 * q;
        s[u] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      int c = 0;
      for (; c + 4 <= nstat; c += 4) {
        f32x4 x[4][EACH];
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int u = 0; u < EACH; ++u) x[v][u] = *(const f32x4*)(gp + (c + v) * pstride + place[u]);
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int u = 0; u < EACH; ++u) s[u] += x[v][u];
      }
      for (; c < nstat; ++c) {
#pragma unroll
        for (int u = 0; u < EACH; ++u) s[u] += *(const f32x4*)(gp + c * pstride + place[u]);
      }
#pragma unroll
      for (int u = 0; u < EACH; ++u) {
        if (wave + u * TE_WAVES < TILES) {
          const int row = place[u] / D, col = place[u] & (D - 1);
          *(f32x4*)&sm[row * (D + 4) + col] = s[u];
          if ((row >> 5) > (col >> 5)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) sm[(col + e) * (D + 4) + row] = s[u][e];
          }
        }
      }
      __syncthreads();
      if (own) {
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = *(const f32x4*)&sm[(16 * wave + j) * (D + 4) + 16 * t + 4 * q];
      }
    }
    if (tid < D) {
      float s = 0.f, s2 = 0.f;
#pragma unroll 4
      for (int c = 0; c < nstat; ++c) { s += gp[c * pstride + D * D + tid]; s2 += gp[c * pstride + D * D + D + tid]; }
      uvec[tid] = s; svec[tid] = s2;
    }
    float vd2 = 0.f;
#pragma unroll 8
    for (int c = 0; c < nstat; ++c) vd2 += gp[c * pstride + D * D + 2 * D];
    __syncthreads();
    if (r > 0 && !thin) {
      bf16x8* qs = (bf16x8*)sm;
      project_columns<D>(acc, Qb, r, qs, own, next, true);     // P G, columns 16 w ..
      __syncthreads();
      if (own) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) sm[(16 * t + 4 * q + e) * (D + 4) + 16 * wave + j] = acc[t][e];
      }
      __syncthreads();
      if (own) {                                               // G P, columns 16 w ..: rows 16 w .. of P G
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = *(const f32x4*)&sm[(16 * wave + j) * (D + 4) + 16 * t + 4 * q];
      }
      project_columns<D>(acc, Qb, r, qs, own, next, false);
      __syncthreads();
    }
    if (r > 0) {
      if (diag) {
        // projection cosine (App. K.2): the column sum s of V_del against that of V_par, its part in the retained span
        float s2 = 0.f, p2 = 0.f;
        for (int c = 0; c < D; ++c) s2 = fmaf(svec[c], svec[c], s2);
        __syncthreads();
        project_vector<D>(Qb, r, svec, coef, part);
        for (int c = 0; c < D; ++c) p2 = fmaf(svec[c], svec[c], p2);
        pc = (s2 > 0.f) ? sqrtf(fmaxf(s2 - p2, 0.f) / s2) : 0.f;
      }
      project_vector<D>(Qb, r, uvec, coef, part);              // P u: the numerator of Eq. 4
    }
    {                                                          // trace(P G P) = ||R||_F^2, summed in double
      double tr = 0.0;
#pragma unroll
      for (int t = 0; t < NT; ++t)
        if (t == wave) {
#pragma unroll
          for (int e = 0; e < 4; ++e) if (4 * q + e == j) tr = (double)acc[t][e];
        }
      for (int o = 32; o > 0; o >>= 1) tr += __shfl_xor(tr, o);
      if (lane == 0) dred[wave] = tr;
    }
    __syncthreads();
    double tr = 0.0;
#pragma unroll
    for (int w = 0; w < NT; ++w) tr += dred[w];
    float res2 = uniform((float)tr);                           // (thin: ||V_del||_F^2 until the Ritz values are there)
    rcr = uniform(res2 / (vd2 + 1e-12f));
    pcr = uniform(fmaxf(vd2 - res2, 0.f) / (vd2 + 1e-12f));
    if (res2 > kRcrSkip * vd2 && res2 < INFINITY && m > 0) {   // (not negligible)
      // over the power of two that brings the trace to [1, 2): squares of the entries then stay in the range of single precision
      // whatever the values' own scale is
      const int ex = min(max((int)(__float_as_uint(res2) >> 23) - 127, -126), 126);
      const float down = __uint_as_float((uint32_t)(127 - ex) << 23);
      const double unit = (double)__uint_as_float((uint32_t)(127 + ex) << 23);
      Split8 mat[NT / 2];                                      // rows 16 w .. of P G P
#pragma unroll
      for (int p = 0; p < NT / 2; ++p) mat[p] = split8(acc[2 * p] * down, acc[2 * p + 1] * down);
      if (thin && own) {                                       // G, for lead_thin: each lane what it reads itself
        float* g = mats + (size_t)head * 3 * D * D + (16 * wave + j) * D + 4 * q;
#pragma unroll
        for (int t = 0; t < NT; ++t) *(f32x4*)(g + 16 * t) = acc[t] * down;
      }
      const float srel = (float)max(st.n_del, D) * (float)kRankEps;
      const float floor_rel = fmaxf(srel * srel, kEigFloor);
      const int kq = min(rank, m), kmax = min(kq, st.n_del);
      const int P = COLS ? COLS : kmax <= 4 ? 8 : 16;

      const BlockLds<D> lds(sm);
      bf16x4* sbuf = lds.sbuf;
      float4* xbuf = lds.xbuf;
      f32x4* gbuf = lds.gbuf;
      float *rows = lds.rows, *lam = lds.lam;
      int copy = 0;                                            // of the block, that the next product uses
      // (P G P) X for the block whose sixteen rows each wave holds; one barrier
      auto product = [&](const f32x4 x) -> f32x4 {
        bf16x4* b = sbuf + copy * (3 * NT * 64);
        copy ^= 1;
        if (own) { if (NARROW) publish_narrow<D>(b, x); else publish<D>(b, x); }
        lds_barrier();
        f32x4 y0 = {0.f, 0.f, 0.f, 0.f}, y1 = {0.f, 0.f, 0.f, 0.f}, y2 = {0.f, 0.f, 0.f, 0.f};
        if (NARROW) {
          f32x4 y3 = {0.f, 0.f, 0.f, 0.f};
          if (own) {
#pragma unroll
            for (int p = 0; p < NT / 2; ++p) multiply_narrow<D>(mat[p], b, p, y0, y1, y2, y3);
            __builtin_amdgcn_sched_group_barrier(0x100, NT > 4 ? 6 : 4, 0);    // reads ahead of the products
            __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
            if (NT > 4) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, NT > 4 ? 12 : 4, 0);
          }
          f32x4 y;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            y1[e] += y3[e];
            y[e] = y0[e] + ((row_xor<8>(y0[e]) + y1[e]) + (row_xor<8>(y1[e]) + y2[e]));
            y[e] = (j < 8) ? y[e] : 0.f;
          }
          return y;
        }
        if (own) {
#pragma unroll
          for (int p = 0; p < NT / 2; ++p) multiply<D>(mat[p], b, p, y0, y1, y2);
          __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);   // two groups of reads ahead of the products
          __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
          if (NT > 4) {
            __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 12, 0);
          } else {
            __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
          }
        }
        return y0 + (y1 + y2);
      };
      // Delta (times a_del + eps) from kk orthonormal rows, cs floats apart in Cb, into part: Eq. 5.  again: once more with what the
      // first pass missed, so that rows orthonormal to 1e-6 serve like exact ones
      auto offset = [&](const float* Cb, const int cs, const int kk, const bool again) {
        const float* vec = uvec;
        for (int pass = 0; pass < (again ? 2 : 1); ++pass) {
          for (int v = wave; v < kk; v += TE_WAVES) {
            float sc = vec[lane] * Cb[v * cs + lane];
            if (D > 64) sc = fmaf(vec[lane + 64], Cb[v * cs + lane + 64], sc);
            sc = te_wave_sum(sc);
            if (lane == 0) dvec[pass][v] = (pass == 0) ? sc : 2.f * dvec[0][v] - sc;
          }
          __syncthreads();
          if (tid < D) {
            float sd = 0.f;
            for (int i = 0; i < kk; ++i) sd = fmaf(dvec[pass][i], Cb[i * cs + tid], sd);
            part[tid] = sd;
          }
          __syncthreads();
          vec = part;
        }
      };
      // Per-token alternative (App. D): the subspace goes to the head's second scratch matrix for the kernel that forms the
      // per-slot directions
      auto export_basis = [&](const float* Cb, const int cs, const int kk) {
        if (!(vflags & VF_PER_TOKEN)) return;
        float* Cg = mats + ((size_t)head * 3 + 1) * D * D;
        for (int e = tid; e < kk * D; e += TE_THREADS) Cg[e] = Cb[(e / D) * cs + (e & (D - 1))];
      };

      // ---- 2. the exact directions
      if (!FAST || diag != nullptr) {
        bool direct = false, kept_matrix = false;
        float* Tg = mats + (size_t)head * 3 * D * D;           // P G P, once the registers' copy is about to change
        auto keep_matrix = [&]() {                             // (symmetric to rounding)
          if (own && !kept_matrix) {
            float* g = Tg + (16 * wave + j) * D + 4 * q;
#pragma unroll
            for (int p = 0; p < NT / 2; ++p) {
              *(f32x4*)(g + 32 * p) = f32x4{whole(mat[p], 0), whole(mat[p], 1), whole(mat[p], 2), whole(mat[p], 3)};
              *(f32x4*)(g + 32 * p + 16) = f32x4{whole(mat[p], 4), whole(mat[p], 5), whole(mat[p], 6), whole(mat[p], 7)};
            }
          }
          kept_matrix = true;
        };
        auto random_entry = [&](const int e, const int seed) -> float { return block_random(16 * wave + 4 * q + e, j, seed); };
        f32x4 x, y;
        int found = 0, group = 0;
        if (thin) {
          lead_thin<D>(Qb, Tg, r, m);
          float total = 0.f;
          for (int i = 0; i < m; ++i) total += lam[i];
          res2 = uniform(total) * (float)unit;
          rcr = uniform(res2 / (vd2 + 1e-12f));
          pcr = uniform(fmaxf(vd2 - res2, 0.f) / (vd2 + 1e-12f));
          if (res2 > kRcrSkip * vd2) {                         // (not negligible)
            for (int i = 0; i < kmax; ++i) if (lam[i] > lam[0] * floor_rel) ++found;
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = (j < P) ? random_entry(e, -1) : 0.f;
          float first = 0.f;                                     // the largest eigenvalue
          // Groups of directions: usually one.  More than kBlockMaxRank are found eight at a time, and directions far below the leading one of
          // their group wait for the next, which works on the matrix without those found.
          for (;;) {
            const int want = (kmax - found > kBlockMaxRank) ? 8 : kmax - found;
            x = product(x);
            x = product(x);
            y = product(x);
            const int full = min(min(P, m - found), st.n_del - found);              // most independent columns the block can have
            const bool loose = P == 16 && full == P;             // how the small problems are solved far from the end
            bool last = false, again = false;                    // again: the block as it is, its small problem solved to the end
            float rn_before = INFINITY;
            int kc = 0;                                          // directions of the group that can be resolved against its first
            for (int round = 0;; ++round) {
              // Rayleigh-Ritz: each wave's share of X^T X and X^T Y, one wave solves the small problem.  With eight columns a sweep does far from
              // the end, what it leaves goes with the next round; with sixteen that costs rounds, and two sweeps in the first and up to eight in the
              // others, to a looser tolerance, are faster (288 heads of 300 tokens, 16 kept, four strong directions, the kernel with 5, 6, 8 and 16
              // directions: 115, 129, 141, 227 us; with one sweep 137, 155, 165, 247; 144 calls of 5 to 16 directions 0.97 of the time), but
              // not where the matrix has fewer directions than that (40 tokens, 32 kept, 8 directions, fp32 at head_dim 64: 53, the other way 80).
              // That a residual has come down to the rounding of P G P is believed only of a problem that was solved to the end.
              const bool exact = last || again || (!loose && (group > 0 || rn_before < 1e-2f));       // uniform
              float4* xb = xbuf + wave * LE_XTILE;
              float4* yb = xbuf + (NT + wave) * LE_XTILE;
              const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
              if (own) {
                gbuf[wave * 64 + lane] = mul_t(x, x, zero);
                gbuf[(NT + wave) * 64 + lane] = mul_t(y, x, mul_t(x, y, zero)) * 0.5f;
                xb[q * 17 + j] = make_float4(x[0], x[1], x[2], x[3]);
                yb[q * 17 + j] = make_float4(y[0], y[1], y[2], y[3]);
              }
              lds_barrier();
              if (wave == solver) {
                f32x4 M = gbuf[lane], H = gbuf[NT * 64 + lane];
#pragma unroll
                for (int w = 1; w < NT; ++w) { M += gbuf[w * 64 + lane]; H += gbuf[(NT + w) * 64 + lane]; }
                f32x4 S;
                float theta;
                int place;
                const float tol = exact || !loose ? 3e-4f : 0.1f;
                const int sweeps = exact ? 8 : !loose ? 1 : round == 0 ? 2 : 8;
                if (P == 8) small_ritz<8>(M, H, 1e-5f, tol, sweeps, S, theta, place);
                else small_ritz<16>(M, H, 1e-5f, tol, sweeps, S, theta, place);
                s_rot[q * 16 + place] = make_float4(S[0], S[1], S[2], S[3]);
                if (q == 0) s_th[place] = theta;
              }
              lds_barrier();
              const float th1 = uniform(s_th[0]);
              if (group == 0) first = th1;
              const float least = first * floor_rel;
              kc = 0;
              for (int i = 0; i < want; ++i) if (s_th[i] > least) ++kc;
              if (kc > 0 && s_th[kc - 1] < kSteep * first) { direct = true; break; }       // uniform, as kc is
              if (own) {
                const float4 s4 = s_rot[lane];
                const f32x4 S = {s4.x, s4.y, s4.z, s4.w};
                f32x4 xt, yt;                                    // entry (16 w + j, 4 q + e) of the two blocks
                const float* xs = (const float*)(xb + (j >> 2) * 17 + 4 * q) + (j & 3);
                const float* ys = (const float*)(yb + (j >> 2) * 17 + 4 * q) + (j & 3);
#pragma unroll
                for (int e = 0; e < 4; ++e) { xt[e] = xs[4 * e]; yt[e] = ys[4 * e]; }
                x = mul_t(xt, S, zero);
                y = mul_t(yt, S, zero);
                const float th = s_th[j];
                float rr = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) { const float z = fmaf(-th, x[e], y[e]); rr = fmaf(z, z, rr); }
                rr = te_wave_sum(j < kc ? rr : 0.f);
                if (lane == 0) red[wave] = rr;
              }
              lds_barrier();
              if (kc == 0) break;                                // nothing (more) above the resolution of the matrix
              float rn = 0.f;
#pragma unroll
              for (int w = 0; w < NT; ++w) rn += red[w];
              rn = uniform(sqrtf(rn) / th1);                     // residual of the wanted directions, relative to the spectrum
              // done: at the rounding of the products; there by the polynomial's own estimate; or no longer falling, and then near enough for the
              // last wanted direction, or at the rounding that P G P brought along (of G, 1 / rcr times its own trace)
              const bool stuck = rn > 0.5f * rn_before;
              again = stuck && rn * th1 * rcr <= 3e-8f;
              if (rn <= 3e-7f || (last && rn <= 1e-6f) || (stuck && rn * th1 <= 1e-5f * s_th[kc - 1]) || (again && exact)) break;
              rn_before = rn;
              // columns that depended on the others make room for new ones (a steep spectrum hides all but its leading directions from
              // the first products), unless the matrix has no more directions
              if (!(s_th[full - 1] > 0.f)) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                  if (j < P && !(s_th[j] > 0.f)) { x[e] = random_entry(e, round); y[e] = 0.f; }
              }
              const float thk = uniform(s_th[kc - 1]), b = uniform(fmaxf(s_th[P - 1], 0.02f * thk)), ic = uniform(2.f / b);
              auto growth = [&](const float v) -> float {        // of a Chebyshev polynomial on [0, b], per degree, in log2
                const float a = fmaf(v, ic, -1.f);
                return a > 1.f ? __builtin_amdgcn_logf(a + __builtin_amdgcn_sqrtf(fmaf(a, a, -1.f))) : 0.f;
              };
              const float gk = growth(thk), g1 = growth(th1);
              const float need = ceilf(__builtin_amdgcn_logf(fmaxf(rn * 5e7f, 10.f)) / gk);
              if (!again && (!(need <= (float)kBlockReach) || round + 1 >= kBlockRounds)) { direct = true; break; }
              // caps: what single precision can tell apart after the columns have grown so differently (guards against the leading
              // one, then the wanted ones among themselves, less what still mixes them)
              const float c1 = __builtin_amdgcn_logf(round == 0 ? 1e3f : 3e6f) / g1;
              const float c2 = __builtin_amdgcn_logf(fmaxf(3.f / fmaxf(rn, 1e-7f), 2.f)) / fmaxf(g1 - gk, 1e-6f);
              const float cap = fmaxf(2.f, fminf(floorf(fminf(c1, c2)), (float)kBlockSteps));
              last = need <= cap;
              const int n = (int)fmaxf(2.f, fminf(need, cap));
              f32x4 xp = x;
              x = y * ic - x;
              for (int i = 1; i < n; ++i) {
                const f32x4 z = product(x) * (2.f * ic) - x * 2.f - xp;
                xp = x;
                x = z;
              }
              y = product(x);
            }
            if (direct || kc == 0) break;
            // the group's directions, their images and Rayleigh quotients
            float* images = (float*)gbuf;                        // [16][LE_LDR]
            if (own) {
              if (j < kc) {
                *(f32x4*)&rows[(found + j) * LE_LDR + 16 * wave + 4 * q] = x;
                *(f32x4*)&images[j * LE_LDR + 16 * wave + 4 * q] = y;
              }
              const float xy = sum_rows(fmaf(x[0], y[0], x[1] * y[1]) + fmaf(x[2], y[2], x[3] * y[3]));
              if (q == 0) coef[wave * 16 + j] = xy;
            }
            lds_barrier();
            if (tid < kc) {
              float th = 0.f;
#pragma unroll
              for (int w = 0; w < NT; ++w) th += coef[w * 16 + tid];
              lam[found + tid] = th;
            }
            if (found + kc >= kmax) { found += kc; break; }
            if (++group > kGroups) { direct = true; break; }
            // the rest of the matrix: G - X Y^T - (Y - X Lambda) X^T, through global memory (rarely taken);
            // the guards start the next group
            const bool deflated = kept_matrix;
            float* Td = Tg + (size_t)D * D;
            keep_matrix();
            __syncthreads();
            const size_t at = (size_t)(16 * wave + j) * D + 4 * q;
            if (own) {
              lead_deflate<D>(deflated ? Td : Tg, Td, (int)(rows - sm) + found * LE_LDR, (int)(images - sm), (int)(lam - sm) + found, kc);
#pragma unroll
              for (int p = 0; p < NT / 2; ++p) {                 // each lane what it wrote
                const float* g = Td + at + 32 * p;
                mat[p] = split8(*(const f32x4*)g, *(const f32x4*)(g + 16));
              }
            }
            {
              const int from = ((lane & 48) | min(j + kc, 15)) << 2;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const float v = __uint_as_float((uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)__float_as_uint(x[e])));
                x[e] = (j + kc < P) ? v : (j < P) ? random_entry(e, 100 + group) : 0.f;
              }
            }
            found += kc;
          }
        }
        __syncthreads();
        if (!direct) {
          k_used = found;
          double top = 0.0;
          for (int i = 0; i < found; ++i) top += (double)lam[i];
          revr = (found > 0) ? (float)(top * unit / ((double)res2 + 1e-12)) : 0.f;
          if (found > 0) {
            if (vflags & VF_PER_TOKEN) {
              if (wave == 0) (void)lead_orth<TE_MAXK, D>((int)(rows - sm), (int)(rows - sm), found);
              __syncthreads();
            }
            offset(rows, LE_LDR, found, true);
            if (!FAST) export_basis(rows, LE_LDR, found);
          }
        } else {
          keep_matrix();
          __syncthreads();
          const DirectResult dr = lead_direct<D>(Tg, kq);
          const float* th = sm + dr.theta;
          const float* Wk = sm + dr.W;
          if (tid == 0) {
            int rankR = 0;
            for (int i = 0; i < kmax; ++i) if (th[i] > th[0] * floor_rel) ++rankR;      // descending: the count is a prefix
            s_k = rankR;
            double top = 0.0;
            for (int i = 0; i < rankR; ++i) top += (double)th[i];
            s_val = (float)(top * unit / ((double)res2 + 1e-12));
          }
          __syncthreads();
          k_used = s_k;
          revr = (k_used > 0) ? s_val : 0.f;
          offset(Wk, D, k_used, true);
          if (!FAST) export_basis(Wk, D, k_used);
        }
        if (FAST && kept_matrix) {
          __syncthreads();                                     // (its writes by other waves)
          if (own) {
#pragma unroll
            for (int p = 0; p < NT / 2; ++p) {
              const float* g = &Tg[(16 * wave + j) * D + 32 * p + 4 * q];
              mat[p] = split8(*(const f32x4*)g, *(const f32x4*)(g + 16));
            }
          }
        }
      }
      // ---- 3. App. H's iteration
      if constexpr (FAST) {
        if (diag != nullptr && tid < D) dex[tid] = (k_used > 0) ? part[tid] : 0.f;       // the exact Delta, for the error report
        __syncthreads();                                       // the LDS of the above is free
        float* Ya = rows;                                      // the current rows
        float* Yb = (float*)gbuf;                              // their images (the partial Gram matrices are not used here)
        static_assert(2 * NT * 64 * 4 >= 15 * LE_LDR + D, "room for the images");
        // C_0: the first rows of the orthonormal cosine basis, C_0[i][c] = sqrt(2/D) cos(pi (i + 1/2)(c + 1/2) / D)
        for (int e = tid; e < 16 * D; e += TE_THREADS) {
          const int i = e / D, c = e & (D - 1);
          Ya[i * LE_LDR + c] = (i < kmax) ? sqrtf(2.f / (float)D) * cospif((float)((2 * i + 1) * (2 * c + 1)) / (float)(4 * D)) : 0.f;
        }
        int kk = kmax;
        __syncthreads();
        static_assert(!THIN, "the fast path projects the matrix");
        auto images = [&]() {                                  // Yb = Ya P G P
          f32x4 x = {0.f, 0.f, 0.f, 0.f};
          if (own) { const float4 v = *(const float4*)&Ya[j * LE_LDR + 16 * wave + 4 * q]; x = f32x4{v.x, v.y, v.z, v.w}; }
          if (j >= kk) x = f32x4{0.f, 0.f, 0.f, 0.f};
          const f32x4 y = product(x);
          if (own) *(float4*)&Yb[j * LE_LDR + 16 * wave + 4 * q] = make_float4(y[0], y[1], y[2], y[3]);
          __syncthreads();
        };
        for (int it = 0; it < iters && kk > 0; ++it) {         // uniform
          images();
          if (wave == solver) {
            const int nk = NARROW || (COLS == 0 && kk <= 4) ? lead_orth<4, D>((int)(Ya - sm), (int)(Yb - sm), kk) : lead_orth<TE_MAXK, D>((int)(Ya - sm), (int)(Yb - sm), kk);
            if (lane == 0) s_k = nk;
          }
          __syncthreads();
          kk = s_k;
          __syncthreads();
        }
        k_used = kk;
        revr = 0.f;
        if (k_used > 0) {
          images();                                            // explained share: sum_i c_i P G P c_i^T over the trace
          for (int v = wave; v < k_used; v += TE_WAVES) {
            float sc = Ya[v * LE_LDR + lane] * Yb[v * LE_LDR + lane];
            if (D > 64) sc = fmaf(Ya[v * LE_LDR + lane + 64], Yb[v * LE_LDR + lane + 64], sc);
            sc = te_wave_sum(sc);
            if (lane == 0) dvec[0][v] = sc;
          }
          __syncthreads();
          double top = 0.0;
          for (int i = 0; i < k_used; ++i) top += (double)dvec[0][i];
          revr = (float)(top * unit / ((double)res2 + 1e-12));
          __syncthreads();
          offset(Ya, LE_LDR, k_used, false);
          export_basis(Ya, LE_LDR, k_used);
        }
        if (diag != nullptr) {
          double num = 0.0, den = 0.0;
          for (int c = 0; c < D; ++c) {
            const double e = (k_used > 0 ? (double)part[c] : 0.0) - dex[c];
            num += e * e; den += (double)dex[c] * dex[c];
          }
          fast_err = (den > 0.0) ? (float)sqrt(num / den) : 0.f;
        }
      }
      // ---- 4. delta
      if (k_used > 0) {
        __syncthreads();
        if (tid < D) {
          const double alpha = (vflags & VF_NO_SCALING) ? 1.0 : st.a_del / (st.a_keep + kEps);          // Eq. 6
          uvec[tid] = (float)(alpha * ((double)part[tid] / (st.a_del + kEps)));
        }
        __syncthreads();
        if (r > 0) project_vector<D>(Qb, r, uvec, coef, part); // the rounding that leaked into the retained span
        if (wave == 0) {
          double s = (double)uvec[lane] * uvec[lane];
          if (D > 64) s += (double)uvec[lane + 64] * uvec[lane + 64];
          for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
          if (lane == 0) s_val = (float)sqrt(s);
        }
        __syncthreads();
        ivn = s_val;
        skipped = 0;
      }
    }
  }
  fn_emit<T, TE_THREADS>(head, D, rank, st, skipped, k_used, rcr, ivn, pcr, pc, revr, fast_err, uvec, state, delta, delta_out, diag, V_out,
                         max_budget, scores, idx, vflags, scs);
  if (shift > 0) {                                               // the lists of a token window: back to the head's own numbers, the -1 padding stays
    __syncthreads();
    int32_t* id = moved + (size_t)head * max_budget;
    for (int i = tid; i < max_budget; i += TE_THREADS) { const int32_t v = id[i]; if (v >= 0) id[i] = v + shift; }
  }
}

template <typename T, int D>
static obf_status_t run(const Dims& m, const Workspace& w, char* ws, const float* scores, const int32_t* idx, int32_t max_budget,
                        int32_t rank, void* V_out, float* delta_out, obf_diag_t* diag, hipStream_t st, int vflags, int iters,
                        IdxShift* shift) {
  static std::mutex attr_mu;
  static uint64_t attr_seen = 0;
  once_per_device(attr_mu, attr_seen, [] {
    const int most = (int)(sizeof(float) * lead_lds_floats(D, TE_MAXK));
    for (const void* k : {(const void*)k_bf_lead<T, D, false, false, 8>, (const void*)k_bf_lead<T, D, false, false, 16>, (const void*)k_bf_lead<T, D, false, false, 0>,
                          (const void*)k_bf_lead<T, D, false, true, 8>, (const void*)k_bf_lead<T, D, false, true, 16>, (const void*)k_bf_lead<T, D, false, true, 0>,
                          (const void*)k_bf_lead<T, D, true, false, 8>, (const void*)k_bf_lead<T, D, true, false, 16>, (const void*)k_bf_lead<T, D, true, false, 0>})
      (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, most);
  });
  const size_t lds = sizeof(float) * lead_lds_floats(D, rank);
  int32_t* moved = shift ? shift->idx : nullptr;
  const int by = shift ? shift->by : 0;
  if (shift) shift->done = true;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(m.heads), dim3(TE_THREADS), lds, st, w.nstat, rank, (HeadState*)(ws + w.head_state),
                       (const float*)(ws + w.basis), (const float*)(ws + w.gram_part), (float*)(ws + w.mats), (float*)(ws + w.delta),
                       delta_out, diag, (T*)V_out, max_budget, scores, idx, moved, by, vflags, m.scs, iters);
  };
  const bool thin = max_budget >= D - kThinWidth && !(vflags & VF_NO_PROJECTION);       // no head can be otherwise
  auto by_cols = [&](auto k8, auto k16, auto k0) { if (rank <= 4) go(k8); else if (m.N - max_budget > 4) go(k16); else go(k0); };
  if (iters > 0) by_cols(k_bf_lead<T, D, true, false, 8>, k_bf_lead<T, D, true, false, 16>, k_bf_lead<T, D, true, false, 0>);
  else if (thin) by_cols(k_bf_lead<T, D, false, true, 8>, k_bf_lead<T, D, false, true, 16>, k_bf_lead<T, D, false, true, 0>);
  else by_cols(k_bf_lead<T, D, false, false, 8>, k_bf_lead<T, D, false, false, 16>, k_bf_lead<T, D, false, false, 0>);
  return check_launch("backfill leading directions");
}

obf_status_t launch_backfill_lead(const Dims& m, const Workspace& w, char* ws, const float* scores, const int32_t* idx, int32_t max_budget,
                                  int32_t rank, void* V_out, float* delta_out, obf_diag_t* diag, hipStream_t st, int vflags, int iters,
                                  IdxShift* shift) {
  if (m.dtype == OBF_BF16)
    return m.d == 128 ? run<uint16_t, 128>(m, w, ws, scores, idx, max_budget, rank, V_out, delta_out, diag, st, vflags, iters, shift)
                      : run<uint16_t, 64>(m, w, ws, scores, idx, max_budget, rank, V_out, delta_out, diag, st, vflags, iters, shift);
  return m.d == 128 ? run<float, 128>(m, w, ws, scores, idx, max_budget, rank, V_out, delta_out, diag, st, vflags, iters, shift)
                    : run<float, 64>(m, w, ws, scores, idx, max_budget, rank, V_out, delta_out, diag, st, vflags, iters, shift);
}

}  // namespace obf
