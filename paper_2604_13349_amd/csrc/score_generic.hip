// Attention-mass scores (Eq. 1) for fp32 caches and head_dim 64: every logit, exponential and sum is carried in double.  Two passes
// over K because a column sum of softmax rows needs every row's normaliser first: pass A gives per-row log-sum-exp, pass B the column
// sums.
//
// The logits are products of the double-precision matrix instruction v_mfma_f64_16x16x4_f64 on 16 x 16 tiles (16 tokens against 16
// query rows; operand layout in f64_tile.hpp).
//   pass A: a wave keeps the operand of 16 query rows and walks the tiles of its chunk of tokens (tokens x rows: a lane owns one
//           query row and keeps its running maximum and sum);
//   pass B: a wave keeps the operand of 16 or 32 tokens and walks all query rows (rows x tokens: a lane owns one token).
// Bound by the double-precision matrix rate (64 multiply-adds per clock and compute unit: 43 us a pass at the first shape below) and
// the exponentials, which the same units compute: f64_exp.hpp's, of half the math library's instructions.  96 heads x 2048 tokens x
// 128 rows at head_dim 64, both: 153 us (170 with the library's exponential and a tile of tokens per wave).  With the products as scalar multiply-adds fed from
// LDS: 975 and 853 us; 2 heads x 512 tokens x 32 rows 224 and 215, now 12 and 6.
#include "f64_exp.hpp"
#include "f64_tile.hpp"

namespace obf {

constexpr int GS_THREADS = 256;
constexpr int GS_WAVES = GS_THREADS / 64;
constexpr int GS_T = 16;                 // tokens and query rows per tile
constexpr int GS_MIN_TILES = 2;          // shortest chunk of pass A, in tiles
constexpr int GS_TARGET_WAVES = 4096;    // waves of pass A that fill the chip (four per SIMD); fewer, longer chunks beyond
// A wave of pass B takes two tiles of tokens, which share the query operand's reads and conversions, where the compute unit with most
// workgroups then has at most a tenth more tokens to do (from this many query rows on: with fewer there is little to share).  Both passes, us,
// one tile - two a wave:
//   as many       96 heads x 1024 x 128 rows 88 - 84, x 2048 161 - 155; 64 x 2048 x 128 123 - 119; 40 x 4000 x 64 102 - 97; 8 x 16384 x 64 81 - 79
//   a tenth more  96 x 1500 x 128 124 - 125; 288 x 512 x 128 129 - 129
//   more          96 x 768 x 128 80 - 82; 288 x 256 x 128 73 - 76; 96 x 1300 x 128 110 - 117; 1280 x 130 x 128 167 - 180
constexpr int GS_WIDE_ROWS = 64;
constexpr int GS_FOLD = 1024;            // partials per head up to which pass B folds them itself (each of its workgroups reads them all;
                                         // a launch of its own costs 5 us)

// NT 16 x 16 tiles of dot products: `moving`, the operand a wave streams, gives the rows of the result, `fixed`, the one it keeps, the
// columns.  Two chains, so that an instruction does not wait for the one before it.
template <typename T, int D, int NT>
__device__ __forceinline__ void tile_products(f64x4 (&out)[NT], const double (&fixed)[NT][D / 4], const RowPart<T, D>& moving) {
  f64x4 a[NT], b[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) { a[t] = f64x4{0.0, 0.0, 0.0, 0.0}; b[t] = a[t]; }
#pragma unroll
  for (int s = 0; s < D / 4; s += 2) {
    const double x = moving.at(s), y = moving.at(s + 1);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      a[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, fixed[t][s], a[t], 0, 0, 0);
      b[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(y, fixed[t][s + 1], b[t], 0, 0, 0);
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) out[t] = a[t] + b[t];
}

// Pass A: partial (max, sum exp(logit - max)) per query row over one chunk of tokens.  Wave w of the grid's first dimension takes row
// block w % nrb and chunk w / nrb of head blockIdx.y.
template <typename T, int D>
__global__ __launch_bounds__(GS_THREADS, 2) void k_score_stats_f64(const T* __restrict__ K, const T* __restrict__ Q,
                                                                   double* __restrict__ stats_part, int N, int R, int nrb, int nchunk,
                                                                   int chunk_tokens, int kvs) {
  const int head = blockIdx.y, lane = threadIdx.x & 63;
  const int w = blockIdx.x * GS_WAVES + (threadIdx.x >> 6);
  const int chunk = w / nrb, row = (w - chunk * nrb) * GS_T + (lane & 15);
  __shared__ ExpTable etab;
  exp_table(etab, threadIdx.x);
  __syncthreads();
  if (chunk >= nchunk) return;                                // whole wave; no barrier follows
  const int t0 = chunk * chunk_tokens, t1 = min(N, t0 + chunk_tokens);
  const T* Kh = K + (size_t)head * kvs * D;
  const double scale = 1.0 / sqrt((double)D);
  double q[1][D / 4];
  {
    RowPart<T, D> p;
    p.load(Q + ((size_t)head * R + min(row, R - 1)) * D, lane);     // rows past R: the last one again, not written
#pragma unroll
    for (int s = 0; s < D / 4; ++s) q[0][s] = p.at(s);
  }
  double m = -INFINITY, l = 0.0;
  RowPart<T, D> cur, nxt;
  cur.load(Kh + (size_t)min(t0 + (lane & 15), N - 1) * D, lane);
  for (int tt = t0; tt < t1; tt += GS_T) {
    nxt.load(Kh + (size_t)min(tt + GS_T + (lane & 15), N - 1) * D, lane);      // clamped: masked below
    f64x4 dots[1];
    tile_products<T, D, 1>(dots, q, cur);
    const f64x4 acc = dots[0];
    double x[4];
    const bool full = tt + GS_T <= t1;                        // uniform; only a chunk's last tile may not be
    if (full) {
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = acc[i];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = (tt + (lane >> 4) + 4 * i < t1) ? acc[i] : -INFINITY;
    }
    const double mx = fmax(fmax(x[0], x[1]), fmax(x[2], x[3])) * scale;
    if (__ballot(mx > m)) {                                   // rare after the first tiles: the sum is rescaled only when a maximum moved
      const double mn = fmax(m, mx);
      if (mn > m) l *= exp(m - mn);
      m = mn;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = fma(x[i], scale, -m);
    exp_clamp(x);
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = exp_tab(x[i], etab);
    if (!full) {
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = (tt + (lane >> 4) + 4 * i < t1) ? x[i] : 0.0;
    }
    l += (x[0] + x[1]) + (x[2] + x[3]);
    cur = nxt;
  }
  // the four lanes of a row
#pragma unroll
  for (int off = 16; off < 64; off <<= 1) {
    const double m2 = __shfl_xor(m, off), l2 = __shfl_xor(l, off);
    const double M = fmax(m, m2);
    const double a = (m == -INFINITY) ? 0.0 : l * exp(m - M);
    const double b = (m2 == -INFINITY) ? 0.0 : l2 * exp(m2 - M);
    m = M; l = a + b;
  }
  if (lane < 16 && row < R) {
    double* o = stats_part + (((size_t)head * nchunk + chunk) * R + row) * 2;
    o[0] = m; o[1] = l;
  }
}

// log-sum-exp of one query row from its chunk partials (p: the first chunk's, `step` doubles between chunks)
__device__ __forceinline__ double fold_lse(const double* __restrict__ p, int nchunk, size_t step) {
  double M = -INFINITY;
  for (int c = 0; c < nchunk; ++c) M = fmax(M, p[c * step]);
  double L = 0.0;
  for (int c = 0; c < nchunk; ++c)
    if (p[c * step] != -INFINITY) L += p[c * step + 1] * exp(p[c * step] - M);
  return M + log(L);
}

// ... of every query row, where pass B does not do it itself
__global__ void k_score_lse(const double* __restrict__ stats_part, double* __restrict__ row_lse, int R, int nchunk,
                            int total_rows) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total_rows) return;
  const int head = i / R, row = i - head * R;
  row_lse[i] = fold_lse(stats_part + ((size_t)head * nchunk * R + row) * 2, nchunk, (size_t)R * 2);
}

// Pass B: scores[j] = sum_rows exp(logit - lse[row]).  A workgroup takes 64 NT tokens of a head, a wave 16 NT.  With stats_part the
// head's row normalisers are folded here first, by every workgroup alike; the first one writes them out.
template <typename T, int D, int NT>
__global__ __launch_bounds__(GS_THREADS, 2) void k_score_mass_f64(const T* __restrict__ K, const T* __restrict__ Q,
                                                                  const double* __restrict__ stats_part /*nullable*/, int nchunk,
                                                                  double* __restrict__ row_lse, float* __restrict__ scores, int N,
                                                                  int R, int kvs) {
  extern __shared__ double s_lse[];                           // [R rounded up to 16]
  __shared__ ExpTable etab;
  const int head = blockIdx.y, lane = threadIdx.x & 63;
  const int tok = (blockIdx.x * GS_WAVES + (threadIdx.x >> 6)) * NT * GS_T + (lane & 15);     // and the 16 behind
  const T* Qh = Q + (size_t)head * R * D;
  const double scale = 1.0 / sqrt((double)D);
  RowPart<T, D> kp[NT], cur, nxt;
#pragma unroll
  for (int t = 0; t < NT; ++t) kp[t].load(K + ((size_t)head * kvs + min(tok + t * GS_T, N - 1)) * D, lane);   // tokens past the end: the last one again, not written
  cur.load(Qh + (size_t)min(lane & 15, R - 1) * D, lane);
  for (int r = threadIdx.x; r < (R + GS_T - 1) / GS_T * GS_T; r += GS_THREADS) {
    double lse = INFINITY;                                    // rows past R add exp(-inf) = 0
    if (r < R) {
      if (stats_part) {
        lse = fold_lse(stats_part + ((size_t)head * nchunk * R + r) * 2, nchunk, (size_t)R * 2);
        if (blockIdx.x == 0) row_lse[(size_t)head * R + r] = lse;
      } else {
        lse = row_lse[(size_t)head * R + r];
      }
    }
    s_lse[r] = lse;
  }
  exp_table(etab, threadIdx.x);
  __syncthreads();
  double k[NT][D / 4], col[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    col[t] = 0.0;
#pragma unroll
    for (int s = 0; s < D / 4; ++s) k[t][s] = kp[t].at(s);
  }
  for (int r0 = 0; r0 < R; r0 += GS_T) {
    nxt.load(Qh + (size_t)min(r0 + GS_T + (lane & 15), R - 1) * D, lane);
    f64x4 acc[NT];
    tile_products<T, D, NT>(acc, k, cur);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      double x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = fma(acc[t][i], scale, -s_lse[r0 + (lane >> 4) + 4 * i]);
      exp_clamp(x);
      col[t] += (exp_tab(x[0], etab) + exp_tab(x[1], etab)) + (exp_tab(x[2], etab) + exp_tab(x[3], etab));
    }
    cur = nxt;
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    col[t] += __shfl_xor(col[t], 16);
    col[t] += __shfl_xor(col[t], 32);
    if (lane < 16 && tok + t * GS_T < N) scores[(size_t)head * N + tok + t * GS_T] = (float)col[t];
  }
}

template <typename T, int D>
static obf_status_t run(const Dims& m, const Workspace& w, char* ws, const void* K, const void* Q, float* scores,
                        double* row_lse, hipStream_t st) {
  double* stats_part = (double*)(ws + w.stats_part);
  // chunks of pass A: enough waves for the chip, within the slots the workspace has per query row
  const int nrb = (m.R + GS_T - 1) / GS_T, tiles = (m.N + GS_T - 1) / GS_T, slots = w.nchunk > w.nslot ? w.nchunk : w.nslot;
  const long units = (long)m.heads * nrb;
  int nchunk = (int)((GS_TARGET_WAVES + units - 1) / units);
  if (nchunk > slots) nchunk = slots;
  const int per = (tiles + nchunk - 1) / nchunk > GS_MIN_TILES ? (tiles + nchunk - 1) / nchunk : GS_MIN_TILES;
  nchunk = (tiles + per - 1) / per;
  { ProfScope prof_(ST_SCORE_STATS, st);
    hipLaunchKernelGGL((k_score_stats_f64<T, D>), dim3((unsigned)(((long)nrb * nchunk + GS_WAVES - 1) / GS_WAVES), m.heads), dim3(GS_THREADS), 0, st,
                       (const T*)K, (const T*)Q, stats_part, m.N, m.R, nrb, nchunk, per * GS_T, m.kvs); }
  if (check_launch("score stats (f64)") != OBF_OK) return OBF_ERR_HIP;
  const bool fold = (long)nchunk * m.R <= GS_FOLD;
  if (!fold) {
    const int total_rows = m.heads * m.R;
    ProfScope prof_(ST_SCORE_LSE, st);
    hipLaunchKernelGGL(k_score_lse, dim3((total_rows + 255) / 256), dim3(256), 0, st, stats_part, row_lse, m.R, nchunk, total_rows);
    if (check_launch("score lse") != OBF_OK) return OBF_ERR_HIP;
  }
  { ProfScope prof_(ST_SCORE_MASS, st);
    constexpr int WIDE = D == 64 ? 2 : 1;                     // (two operands of head_dim 128 fill the registers)
    auto go = [&](auto kernel, const int nt) {
      const int per_wg = GS_WAVES * GS_T * nt;
      hipLaunchKernelGGL(kernel, dim3((m.N + per_wg - 1) / per_wg, m.heads), dim3(GS_THREADS), sizeof(double) * nrb * GS_T, st, (const T*)K,
                         (const T*)Q, fold ? (const double*)stats_part : (const double*)nullptr, nchunk, row_lse, scores, m.N, m.R, m.kvs);
    };
    auto busiest = [&](const int nt) {                        // tiles of tokens of a wave of the compute unit with most of them
      const int per_wg = GS_WAVES * GS_T * nt;
      return (((long)m.heads * ((m.N + per_wg - 1) / per_wg) + kNumCU - 1) / kNumCU) * nt;
    };
    if (10 * busiest(2) <= 11 * busiest(1) && m.R >= GS_WIDE_ROWS) go(k_score_mass_f64<T, D, WIDE>, WIDE);
    else go(k_score_mass_f64<T, D, 1>, 1); }
  return check_launch("score mass (f64)");
}

obf_status_t launch_score_generic(const Dims& m, const Workspace& w, char* ws, const void* K, const void* Q,
                                  float* scores, double* row_lse, hipStream_t st) {
  // (bf16 caches of head_dim 128 are score_mfma.hip's)
  if (m.dtype == OBF_BF16) return run<uint16_t, 64>(m, w, ws, K, Q, scores, row_lse, st);
  if (m.d == 64) return run<float, 64>(m, w, ws, K, Q, scores, row_lse, st);
  return run<float, 128>(m, w, ws, K, Q, scores, row_lse, st);
}

}  // namespace obf
