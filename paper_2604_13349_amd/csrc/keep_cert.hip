// Fast decision "the retained values span all of R^d" (then Eq. 3's residual is identically zero and
// the head stays plain eviction) for heads with more retained rows than head_dim.  Heads it cannot certify go to the reference-precision
// basis kernel; the allowance for rounding below keeps it from certifying others.
//
//   G   = V_s^T V_s over a strided subset V_s of the retained rows (all rows up to 512), on the matrix
//         cores: products of bf16 values are exact in fp32, accumulation is fp32 (fp32 caches and head_dim
//         64: products and sums in fp32);
//   mu  = (max(n, d) 2^-23)^2 ||V_keep||_F^2;
//   S   = D^-1/2 G D^-1/2 with D = diag(G): G - mu I is positive definite iff S - mu D^-1 is;
//   if the LDL^T factorisation of S - mu D^-1 - eps I (eps: allowance for the fp32 error of G and of the
//   factorisation, relative to trace(S) = d) runs through with positive pivots, then
//   sigma_min(V_keep)^2 >= lambda_min(G) > (max(n, d) 2^-23)^2 sigma_max(V_keep)^2, i.e. every singular
//   value is above the rank rule's threshold: r = d.
#include "common.hpp"
#include "gram_stage.hpp"
#include "wave_ops.hpp"

namespace obf {

typedef gs_f32x16 f32x16;

constexpr int KC_THREADS = 256;
constexpr int KC_WAVES = KC_THREADS / 64;
constexpr int KC_D = GS_D;
constexpr int KC_TILE = GS_TILE;         // rows staged per iteration
constexpr int KC_MINROWS = 512;          // rows entering G: all up to 512, else about max(512, n/4) at a constant stride
// Allowance for the rounding of G and of the factorisation, relative to the trace of the scaled Gram matrix (= d).  An entry of S errs by at most as
// many 2^-24 as its sum and the factorisation's chain have roundings, and d times that bounds the matrix's error.  For bf16 values, whose products are
// exact, 1.6e-5 is ten times and more what the sums of up to 512 rows and n/4 from there err by with rounding errors of independent signs
// (the bound itself would be rows 2^-24, above it from 140 rows on).  In single precision (cert_allowance) it is the bound: sums in
// parts of KF_PART rows, d steps of the factorisation, and 32 for products, scaling and reciprocals.
constexpr float kCertErr = 1.6e-5f;
constexpr int KF_PART = 128;
__device__ __forceinline__ float cert_allowance(const int rows, const int d) {
  return fmaxf(kCertErr, (float)(KF_PART + (rows + KF_PART - 1) / KF_PART + d + 32) * 5.9604645e-8f);
}


// The lower triangle of G is ten 32x32 tiles (row block rb >= column block cb).  Each tile lives in one wave's
// registers from the Gram phase to the end of the factorisation: entry i of lane l is
// G[rb*32 + (i/4)*8 + (l/32)*4 + (i%4)][cb*32 + l%32].  No wave holds two tiles of the same column block, so the
// part of a step that the next pivot column waits for is at most one tile update per wave.
__device__ __forceinline__ void wave_tiles(int wave, int (&rb)[3], int (&cb)[3], int& nt) {
  if (wave == 0) { rb[0] = 0; cb[0] = 0; rb[1] = 1; cb[1] = 1; rb[2] = 3; cb[2] = 2; nt = 3; }
  else if (wave == 1) { rb[0] = 1; cb[0] = 0; rb[1] = 2; cb[1] = 1; rb[2] = 3; cb[2] = 3; nt = 3; }
  else if (wave == 2) { rb[0] = 2; cb[0] = 0; rb[1] = 3; cb[1] = 1; rb[2] = 0; cb[2] = 0; nt = 2; }
  else { rb[0] = 3; cb[0] = 0; rb[1] = 2; cb[1] = 2; rb[2] = 0; cb[2] = 0; nt = 2; }
}

// What a workgroup shares during the factorisation (its memory may have held something else before).
constexpr int CF_LD = 20;                // floats between rows of 16 columns: rows are whole 16-byte pieces, 8 of them on different banks
template <int D>
struct CertShared {
  __attribute__((aligned(16))) float panel[D][CF_LD];        // the columns that are factored next
  __attribute__((aligned(16))) float y[2][D][CF_LD], l[2][D][CF_LD];     // -L d and L of a panel, for the updates
  __attribute__((aligned(16))) float isd[D];
};

// value of lane K of each 16-lane row, in every lane of the row
template <int K>
__device__ __forceinline__ float cf_bcast(const float v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x150 + K, 0xF, 0xF, true));
}
template <int C, int J>
__device__ __forceinline__ void cf_eliminate(float (&a)[16], float (&b)[16], const float ma, const float mb) {
  if constexpr (J < 16) {
    const float e = cf_bcast<J>(b[C]);                         // entry (J, C) of the diagonal block
    b[J] = fmaf(e, mb, b[J]);
    a[J] = fmaf(e, ma, a[J]);
    cf_eliminate<C, J + 1>(a, b, ma, mb);
  }
}
// Columns C .. 15 of a panel: a is the lane's row, b row lane % 16 of the diagonal block.  Leaves L d in a, and 1 / d in rc.
template <int C>
__device__ __forceinline__ void cf_columns(float (&a)[16], float (&b)[16], float (&rc)[16], bool& positive) {
  if constexpr (C < 16) {
    const float d = cf_bcast<C>(b[C]);
    positive = positive && d > 0.f;
    rc[C] = __builtin_amdgcn_rcpf(d);
    cf_eliminate<C, C + 1>(a, b, -(a[C] * rc[C]), -(b[C] * rc[C]));
    cf_columns<C + 1>(a, b, rc, positive);
  }
}

// Factors G - mu I (scaled, less the allowance) for the Gram matrix G that the workgroup's waves hold in the tiles (trb, tcb) of g; *bad, zeroed by
// the kernel ahead of a barrier, is set where a pivot is not positive.
template <int D>
__device__ __forceinline__ void cert_factor(f32x16 (&g)[3], const int (&trb)[3], const int (&tcb)[3], const int nt, const float mu,
                                            CertShared<D>& sh, int* bad, const float allowance = kCertErr) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int lr = lane & 31, lh = lane >> 5;
  const bool has_diag = ((lr & 7) >> 2) == lh;
  const int di = (lr >> 3) * 4 + (lr & 3);
  // Symmetric diagonal scaling S = D^-1/2 G D^-1/2 (unit diagonal): G - mu I is positive definite iff S - mu D^-1 is,
  // and the scaled matrix no longer carries the spread of the channel magnitudes (a few outlier channels otherwise
  // own the trace, and with it the rounding allowance, while lambda_min sits in the small ones).
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    if (t < nt && trb[t] == tcb[t] && has_diag) {
      float v = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) if (i == di) v = g[t][i];
      sh.isd[tcb[t] * 32 + lr] = __builtin_amdgcn_rsqf(v);            // a zero column gives inf, then NaN pivots: not certified
    }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    if (t < nt) {
      const float sc_col = sh.isd[tcb[t] * 32 + lr];
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const float4 sr = *(const float4*)&sh.isd[trb[t] * 32 + i4 * 8 + lh * 4];
        g[t][4 * i4 + 0] *= sr.x * sc_col; g[t][4 * i4 + 1] *= sr.y * sc_col;
        g[t][4 * i4 + 2] *= sr.z * sc_col; g[t][4 * i4 + 3] *= sr.w * sc_col;
      }
      if (trb[t] == tcb[t] && has_diag) {
        const float shift = fmaf(mu, sc_col * sc_col, allowance * (float)D);   // mu / G_jj + allowance relative to trace(S) = d
#pragma unroll
        for (int i = 0; i < 16; ++i) if (i == di) g[t][i] -= shift;
      }
    }
  }

  // ---- LDL^T in panels of sixteen columns.  A panel passes through LDS to the waves that factor it, a row below the diagonal block per lane, so
  // two waves take the first three panels and one the rest.  Each of their 16-lane rows holds the diagonal block as well and eliminates it
  // again: its entries, which every lane needs, then come from the same 16 lanes by DPP.  (As scalars read from one copy: 1.5 us a panel.)  The tiles stay with their waves, which update those with the next panel's columns
  // first and publish these, the others beside the factorisation of the next panel: the chain from panel to panel is the factorisation
  // (1 us), one tile update (eight matrix instructions) and two barriers.  The waves that factor have the fewest tiles left then.
  // Entries above the diagonal and in finished columns are carried along and never read.
  // 288 heads of 205 rows, the whole kernel: 28 us; 34.6 with steps of four columns, two barriers and the same 4 x 4 block factored by every thread (one
  // barrier a step was slower).
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int part = D == 128 ? (wave == 2 ? 0 : wave == 3 ? 1 : 2) : (wave == 3 ? 0 : 2);      // which 64 rows below the diagonal block; 2: none
  auto publish = [&](int k) {                         // columns 16 k .. 16 k + 15
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      if (t < nt && tcb[t] == (k >> 1) && (lr >> 4) == (k & 1)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) sh.panel[trb[t] * 32 + (i >> 2) * 8 + lh * 4 + (i & 3)][lr & 15] = g[t][i];
      }
    }
  };
  // a tile less the product of panel k's columns: v_mfma_f32_32x32x2_f32, lane l with columns s + 8 (l / 32) of row l % 32 of either operand
  auto update = [&](int t, int k) {
    const float4* yp = (const float4*)&sh.y[k & 1][trb[t] * 32 + lr][8 * lh];
    const float4* lp = (const float4*)&sh.l[k & 1][tcb[t] * 32 + lr][8 * lh];
    const float4 y0 = yp[0], y1 = yp[1], l0 = lp[0], l1 = lp[1];
    g[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(y0.x, l0.x, g[t], 0, 0, 0);
    g[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(y0.y, l0.y, g[t], 0, 0, 0);
    g[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(y0.z, l0.z, g[t], 0, 0, 0);
    g[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(y0.w, l0.w, g[t], 0, 0, 0);
    g[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(y1.x, l1.x, g[t], 0, 0, 0);
    g[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(y1.y, l1.y, g[t], 0, 0, 0);
    g[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(y1.z, l1.z, g[t], 0, 0, 0);
    g[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(y1.w, l1.w, g[t], 0, 0, 0);
  };
  publish(0);
#pragma unroll 1
  for (int k = 0; k < D / 16; ++k) {
    lds_barrier();                                     // the panel is published
    if (k > 0) {
#pragma unroll
      for (int t = 0; t < 3; ++t)
        if (t < nt && tcb[t] > (k >> 1)) update(t, k - 1);
    }
    if (part == 0 || (part == 1 && 16 * (k + 1) + 64 < D)) {             // uniform
      const int p = 16 * (k + 1) + 64 * part + lane;
      const bool have = p < D;
      float a[16], b[16], rc[16];
      auto row_at = [&](const int r, float (&x)[16]) {
        const float4* pr = (const float4*)sh.panel[r];
#pragma unroll
        for (int c = 0; c < 4; ++c) { const float4 v = pr[c]; x[4 * c] = v.x; x[4 * c + 1] = v.y; x[4 * c + 2] = v.z; x[4 * c + 3] = v.w; }
      };
      row_at(16 * k + (lane & 15), b);
      row_at(have ? p : 16 * k, a);
      bool positive = true;
      cf_columns<0>(a, b, rc, positive);
      if (!positive) *bad = 1;
      if (have) {
        float4* yo = (float4*)sh.y[k & 1][p];
        float4* lo = (float4*)sh.l[k & 1][p];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          yo[c] = make_float4(-a[4 * c], -a[4 * c + 1], -a[4 * c + 2], -a[4 * c + 3]);
          lo[c] = make_float4(a[4 * c] * rc[4 * c], a[4 * c + 1] * rc[4 * c + 1], a[4 * c + 2] * rc[4 * c + 2], a[4 * c + 3] * rc[4 * c + 3]);
        }
      }
    }
    lds_barrier();                                     // it is factored
    if (k + 1 < D / 16) {
#pragma unroll
      for (int t = 0; t < 3; ++t)
        if (t < nt && tcb[t] == ((k + 1) >> 1)) update(t, k);
      publish(k + 1);
    }
  }
}

// Certified: r = d, OBF is the identity on this head; fills in the demand sums (Eq. 6) for the diagnostics.  pk: what the caller has
// already added of the retained tokens' scores, which go on from `first`.
__device__ __forceinline__ void cert_settle(double pk, const int first, const float* __restrict__ sc, const int32_t* __restrict__ id, const int n,
                                            const int N, const int want_sums, const int d, const int head, HeadState* __restrict__ state,
                                            int32_t* __restrict__ decided, double* red, double* red2) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool vec_scores = (N & 3) == 0 && ((uintptr_t)sc & 15) == 0;
  const int ns = want_sums ? n : 0, Ns = want_sums ? N : 0;          // extents of the two sums
  double ptot = 0.0;
  for (int i0 = first; i0 < ns; i0 += 8 * KC_THREADS) {      // further batches of index -> score loads
    int j[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) { const int i = i0 + u * KC_THREADS; j[u] = (i < ns) ? id[i] : -1; }
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = (j[u] >= 0) ? sc[j[u]] : 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u) pk += (double)v[u];
  }
  if (vec_scores) {
    const float4* sc4 = (const float4*)sc;
    const int n4 = Ns >> 2;
    for (int i0 = tid; i0 < n4; i0 += 8 * KC_THREADS) {
      float4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) { const int i = i0 + u * KC_THREADS; v[u] = (i < n4) ? sc4[i] : make_float4(0.f, 0.f, 0.f, 0.f); }
#pragma unroll
      for (int u = 0; u < 8; ++u) ptot += ((double)v[u].x + (double)v[u].y) + ((double)v[u].z + (double)v[u].w);
    }
  } else {
    for (int i = tid; i < Ns; i += KC_THREADS) ptot += (double)sc[i];
  }
  for (int off = 32; off > 0; off >>= 1) { pk += __shfl_xor(pk, off); ptot += __shfl_xor(ptot, off); }
  if (lane == 0) { red[wave] = pk; red2[wave] = ptot; }
  __syncthreads();
  if (tid == 0) {
    const double a_keep = ((red[0] + red[1]) + red[2]) + red[3];
    const double a_tot = ((red2[0] + red2[1]) + red2[2]) + red2[3];
    HeadState s;
    s.a_keep = a_keep; s.a_del = fmax(a_tot - a_keep, 0.0); s.n_keep = n; s.n_del = N - n; s.r_keep = d; s.active = 0;
    s.k_used = 0; s.pad = 0; s.rcr = 0.f; s.ivn = 0.f;
    state[head] = s;
    decided[head] = 1;
  }
}

template <bool via_idx>
__global__ __launch_bounds__(KC_THREADS, 2) void k_bf_keep_cert(const uint16_t* __restrict__ Vsrc /*via_idx ? V [heads][N][d] : gathered rows [heads][max_budget][d]*/,
                                                             const float* __restrict__ scores,
                                                             const int32_t* __restrict__ idx,
                                                             const int32_t* __restrict__ n_keep, int N, int max_budget,
                                                             int rank, HeadState* __restrict__ state,
                                                             int32_t* __restrict__ decided,
                                                             const double* __restrict__ fro_part /*optional: sums of squares of the retained rows, per gather block*/,
                                                             int fro_blocks, int scs, int kvs,
                                                             int want_sums /*0: the demand sums of a certified head (diagnostics only) are left at zero*/) {
  __shared__ __attribute__((aligned(16))) union { uint32_t stage[2][GS_STAGE_WORDS]; CertShared<KC_D> cert; } lds;
  auto& stage = lds.stage;
  __shared__ int bad;
  __shared__ double red[KC_THREADS / 64], red2[KC_THREADS / 64];
  const int head = blockIdx.x;
  const int n = n_keep[head];
  const int n_del = N - n;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform, kept in a scalar register
  const int lr = lane & 31, lh = lane >> 5;
  if (tid == 0) { decided[head] = 0; bad = 0; }
  if (!(rank > 0 && n > KC_D && n_del > 0)) return;
  const float* sc = scores + (size_t)head * scs;
  const int32_t* id = idx + (size_t)head * max_budget;
  const uint16_t* Vh = Vsrc + (size_t)head * (via_idx ? kvs : max_budget) * KC_D;
  auto row_of = [&](int r) -> size_t { return via_idx ? (size_t)id[r] : (size_t)r; };    // retained row r of the head
  const int cap = max(KC_MINROWS, n >> 2);
  const int stride = (n + cap - 1) / cap;
  const int rows = (n + stride - 1) / stride;
  int trb[3], tcb[3], nt;
  wave_tiles(wave, trb, tcb, nt);

  f32x16 acc[3];
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;

  // ---- Gram phase: rows staged 64 at a time through LDS (double buffered); the loads run two tiles ahead in
  // registers so that their latency is covered by the products of two tiles.  All waves run one instruction stream:
  // the operands of a wave's tiles are picked by LDS address (a wave with two tiles repeats its second product into an
  // accumulator nobody reads).
  const int pc = lane & 15;
  uint4 pre[2][4];
  auto fetch = [&](uint4 (&dst)[4], int r0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = min(r0 + gs_row<KC_WAVES>(wave, lane, q), rows - 1);      // clamped: rows past the end are zeroed in put
      dst[q] = *(const uint4*)(Vh + row_of(r * stride) * KC_D + pc * 8);
    }
  };
  auto put = [&](const uint4 (&src)[4], int buf, int r0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int rl = gs_row<KC_WAVES>(wave, lane, q);
      gs_put(stage[buf], rl, lane, src[q], r0 + rl < rows);
    }
  };
  const int oA0 = trb[0] * 32, oB0 = tcb[0] * 32, oA1 = trb[1] * 32, oB1 = tcb[1] * 32;
  const int oA2 = (nt > 2 ? trb[2] : trb[1]) * 32, oB2 = (nt > 2 ? tcb[2] : tcb[1]) * 32;
  auto compute = [&](const uint32_t* st) {
#pragma unroll
    for (int ks = 0; ks < KC_TILE / 16; ++ks) {
      GsFrag a0, b0, a1, b1, a2, b2;
      gs_frag(a0, st, ks, lane, oA0); gs_frag(b0, st, ks, lane, oB0);
      gs_frag(a1, st, ks, lane, oA1); gs_frag(b1, st, ks, lane, oB1);
      gs_frag(a2, st, ks, lane, oA2); gs_frag(b2, st, ks, lane, oB2);
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0.v, b0.v, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1.v, b1.v, acc[1], 0, 0, 0);
      acc[2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2.v, b2.v, acc[2], 0, 0, 0);
    }
  };
  // The demand sums of Eq. 6 (diagnostics of a certified head) need sum(scores[idx]) and sum(scores): their first
  // batch of loads is issued here and consumed after the factorisation, so that its latency is hidden.
  int ej[8];
  const int ns = want_sums ? n : 0;
#pragma unroll
  for (int u = 0; u < 8; ++u) { const int i = tid + u * KC_THREADS; ej[u] = (i < ns) ? id[i] : -1; }
  // tile j is staged in stage[j % 2]; the loads run two tiles ahead in registers
  fetch(pre[0], 0);
  fetch(pre[1], KC_TILE);
  put(pre[0], 0, 0);
  fetch(pre[0], 2 * KC_TILE);
  lds_barrier();
#pragma unroll 1
  for (int r0 = 0; r0 < rows; r0 += 2 * KC_TILE) {
    // even tile: in stage[0]; pre[1] holds tile r0+64, pre[0] holds tile r0+128
    compute(stage[0]);
    put(pre[1], 1, r0 + KC_TILE);
    fetch(pre[1], r0 + 3 * KC_TILE);
    lds_barrier();                      // LDS only: the loads just issued stay in flight across the barrier
    if (r0 + KC_TILE < rows) compute(stage[1]);
    put(pre[0], 0, r0 + 2 * KC_TILE);
    fetch(pre[0], r0 + 4 * KC_TILE);
    lds_barrier();
  }
  float ev[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) ev[u] = (ej[u] >= 0) ? sc[ej[u]] : 0.f;
  // ---- trace(G), ||V_keep||_F^2, shift
  // a lane holds a diagonal entry of a diagonal tile iff (lr % 8) / 4 == lh, at i = (lr / 8) * 4 + lr % 4
  const bool has_diag = ((lr & 7) >> 2) == lh;
  const int di = (lr >> 3) * 4 + (lr & 3);
  double part = 0.0;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    if (t < nt && trb[t] == tcb[t] && has_diag) {
      float v = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) if (i == di) v = acc[t][i];
      part += (double)v;
    }
  }
  for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
  if (lane == 0) red[wave] = part;
  __syncthreads();
  const double tr = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  double f2 = tr;
  if (stride > 1 && fro_part) {
    double p2 = 0.0;
    for (int b = tid; b < fro_blocks; b += KC_THREADS) p2 += fro_part[(size_t)head * fro_blocks + b];
    for (int off = 32; off > 0; off >>= 1) p2 += __shfl_xor(p2, off);
    if (lane == 0) red[wave] = p2;
    __syncthreads();
    f2 = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
  } else if (stride > 1) {
    double p2 = 0.0;
    const int sub = tid >> 4, piece = tid & 15;
    for (int r0 = sub; r0 < n; r0 += 8 * (KC_THREADS / 16)) {          // 8 independent row pieces in flight per lane
      uint4 q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int r = r0 + u * (KC_THREADS / 16);
        q[u] = (r < n) ? *(const uint4*)(Vh + row_of(r) * KC_D + piece * 8) : make_uint4(0u, 0u, 0u, 0u);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t w4[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float a = __uint_as_float(w4[i] << 16), b = __uint_as_float(w4[i] & 0xffff0000u);
          s = fmaf(a, a, s); s = fmaf(b, b, s);
        }
        p2 += (double)s;
      }
    }
    for (int off = 32; off > 0; off >>= 1) p2 += __shfl_xor(p2, off);
    if (lane == 0) red[wave] = p2;
    __syncthreads();
    f2 = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
  }
  const double thr_rel = (double)max(n, KC_D) * 1.1920928955078125e-07;
  cert_factor<KC_D>(acc, trb, tcb, nt, (float)(thr_rel * thr_rel * f2), lds.cert, &bad);
  __syncthreads();
  const bool ok = (bad == 0);
  if (!ok) return;

  double pk = 0.0;
#pragma unroll
  for (int u = 0; u < 8; ++u) pk += (double)ev[u];
  cert_settle(pk, tid + 8 * KC_THREADS, sc, id, n, N, want_sums, KC_D, head, state, decided, red, red2);
}

// The same for the other shapes (fp32 caches, head_dim 64): the Gram matrix by v_mfma_f32_32x32x2_f32 straight from the gathered rows - the
// operand's lane l holds row l / 32 of a pair and column l % 32, which is how rows lie in memory - a wave per tile or three, the next
// KF_PAIRS row pairs in flight, summed in parts of KF_PART rows so that the rounding does not grow with their number.  A column whose sum of squares leaves single precision's comfortable range is not certified.
// Bound by the latency of the loads and of the factorisation.  96 heads, 205 rows of 64 fp32 values: 18.5 us (19.2 with steps of four
// columns; sixteen pairs in flight change nothing), and 5 for the exact basis kernel, which then finds nothing to do (80 with every head in it).
constexpr int KF_PAIRS = 8;
constexpr float kCertMinSquare = 1e-30f, kCertMaxSquare = 1e30f;

template <typename T, int D>
__global__ __launch_bounds__(KC_THREADS, 2) void k_bf_keep_cert_rows(const T* __restrict__ Vsrc /*gathered rows [heads][max_budget][d]*/,
                                                                  const float* __restrict__ scores, const int32_t* __restrict__ idx,
                                                                  const int32_t* __restrict__ n_keep, int N, int max_budget, int rank,
                                                                  HeadState* __restrict__ state, int32_t* __restrict__ decided, int scs,
                                                                  int want_sums) {
  __shared__ CertShared<D> sh;
  __shared__ int bad;
  __shared__ double red[KC_WAVES], red2[KC_WAVES];
  const int head = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = n_keep[head];
  if (tid == 0) { decided[head] = 0; bad = 0; }
  if (!(rank > 0 && n > D && N - n > 0)) return;
  const int lr = lane & 31, lh = lane >> 5;
  const T* Vh = Vsrc + (size_t)head * max_budget * D;
  const int cap = max(KC_MINROWS, n >> 2);
  const int stride = (n + cap - 1) / cap;
  const int rows = (n + stride - 1) / stride;
  int trb[3] = {0, 0, 0}, tcb[3] = {0, 0, 0}, nt;
  if constexpr (D == 128) wave_tiles(wave, trb, tcb, nt);
  else { nt = wave < 3 ? 1 : 0; trb[0] = wave > 0 ? 1 : 0; tcb[0] = wave > 1 ? 1 : 0; }      // (0,0), (1,0), (1,1)
  constexpr int NT = D == 128 ? 3 : 1;
  f32x16 acc[3], sums[NT];                                     // of all parts, and of the present one
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
#pragma unroll
  for (int t = 0; t < NT; ++t) sums[t] = acc[t];
  if (nt > 0) {                                                // wave-uniform; no barrier inside
    float a[2][NT][KF_PAIRS], b[2][NT][KF_PAIRS];
    auto fetch = [&](const int buf, const int r0) {
#pragma unroll
      for (int p = 0; p < KF_PAIRS; ++p) {
        const int r = r0 + 2 * p + lh;
        const T* row = Vh + (size_t)min(r * stride, n - 1) * D + lr;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const float x = Elem<T>::load(row + trb[t] * 32), y = Elem<T>::load(row + tcb[t] * 32);
          a[buf][t][p] = r < rows ? x : 0.f;                   // rows past the subset add nothing, whatever they hold
          b[buf][t][p] = r < rows ? y : 0.f;
        }
      }
    };
    auto sum = [&](const int buf) {
#pragma unroll
      for (int p = 0; p < KF_PAIRS; ++p)
#pragma unroll
        for (int t = 0; t < NT; ++t) sums[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[buf][t][p], b[buf][t][p], sums[t], 0, 0, 0);
    };
    fetch(0, 0);
    for (int r0 = 0; r0 < rows; r0 += 4 * KF_PAIRS) {
      fetch(1, r0 + 2 * KF_PAIRS);
      sum(0);
      fetch(0, r0 + 4 * KF_PAIRS);
      sum(1);
      static_assert(KF_PART % (4 * KF_PAIRS) == 0, "a part is whole rounds");
      if ((r0 + 4 * KF_PAIRS) % KF_PART == 0 || r0 + 4 * KF_PAIRS >= rows) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int i = 0; i < 16; ++i) { acc[t][i] += sums[t][i]; sums[t][i] = 0.f; }
      }
    }
  }
  // ||V_keep||_F^2: the trace where every row is in G, else a sum over all rows
  const bool has_diag = ((lr & 7) >> 2) == lh;
  const int di = (lr >> 3) * 4 + (lr & 3);
  double part = 0.0;
  bool out = false;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    if (t < nt && trb[t] == tcb[t] && has_diag) {
      float v = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) if (i == di) v = acc[t][i];
      part += (double)v;
      out |= !(v > kCertMinSquare && v < kCertMaxSquare);
    }
  }
  if (stride > 1) {
    part = 0.0;
#pragma unroll 8
    for (int e = tid; e < n * D; e += KC_THREADS) { const float v = Elem<T>::load(Vh + e); part += (double)v * v; }
  }
  for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
  if (lane == 0) red[wave] = part;
  __syncthreads();                                             // (bad is zero from here)
  if (out) bad = 1;
  const double f2 = (red[0] + red[1]) + (red[2] + red[3]);
  const double thr_rel = (double)n * 1.1920928955078125e-07;   // n > D
  cert_factor<D>(acc, trb, tcb, nt, (float)(thr_rel * thr_rel * f2), sh, &bad, cert_allowance(rows, D));
  __syncthreads();
  if (bad) return;
  cert_settle(0.0, tid, scores + (size_t)head * scs, idx + (size_t)head * max_budget, n, N, want_sums, D, head, state, decided, red, red2);
}

// (no head retains more than head_dim rows under a smaller max_budget: nothing to certify)
bool keep_cert_supported(const Dims& m, int max_budget) { return max_budget > m.d; }

obf_status_t launch_keep_cert(const Dims& m, const void* Vsrc, int via_idx, const float* scores, const int32_t* idx,
                              const int32_t* n_keep, int32_t max_budget, int32_t rank, HeadState* state,
                              int32_t* decided, hipStream_t st, const double* fro_part, bool want_sums) {
  const int fro_blocks = (max_budget + kGatherRows - 1) / kGatherRows;
  { ProfScope prof_(ST_KEEP_CERT, st);
#define OBF_KC_ROWS(T, D) hipLaunchKernelGGL((k_bf_keep_cert_rows<T, D>), dim3(m.heads), dim3(KC_THREADS), 0, st, (const T*)Vsrc, scores, idx, \
                                             n_keep, m.N, max_budget, rank, state, decided, m.scs, want_sums ? 1 : 0)
    if (m.dtype == OBF_F32) { if (m.d == 128) OBF_KC_ROWS(float, 128); else OBF_KC_ROWS(float, 64); }
    else if (m.d == 64) OBF_KC_ROWS(uint16_t, 64);
#undef OBF_KC_ROWS
    else if (via_idx)
      hipLaunchKernelGGL(k_bf_keep_cert<true>, dim3(m.heads), dim3(KC_THREADS), 0, st, (const uint16_t*)Vsrc, scores, idx,
                         n_keep, m.N, max_budget, rank, state, decided, fro_part, fro_blocks, m.scs, m.kvs, want_sums ? 1 : 0);
    else
      hipLaunchKernelGGL(k_bf_keep_cert<false>, dim3(m.heads), dim3(KC_THREADS), 0, st, (const uint16_t*)Vsrc, scores, idx,
                         n_keep, m.N, max_budget, rank, state, decided, fro_part, fro_blocks, m.scs, m.kvs, want_sums ? 1 : 0); }
  return check_launch("backfill keep_cert");
}

}  // namespace obf
