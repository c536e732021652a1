// TopK_B (Sec. 4.3.2): the B largest scores of a head, ties to the lowest index, written as an
// ascending index list.  One workgroup per head; the N keys live in registers.  All comparisons are
// on an order-preserving integer image of the fp32 bit patterns, so the result is exact.
#include "boundary.hpp"

namespace obf {

constexpr int SEL_BATCH = 896;   // heads per launch when budgets differ per head (the budgets travel as a kernel argument: 3.5 KB of the 4 KB)

struct BudgetBatch { int32_t b[SEL_BATCH]; };

// larger float <=> larger key (total order on the bit patterns; -0 < +0)
__device__ __forceinline__ uint32_t order_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_to_float(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// exclusive prefix sums of (a, b) over the workgroup, in thread order
template <int SEL_WAVES>
__device__ __forceinline__ void block_exscan2(int a, int b, int& ea, int& eb, int& ta, int& tb, int* wsum /*[2*SEL_WAVES]*/) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int ia = a, ib = b;
  for (int off = 1; off < 64; off <<= 1) {
    const int xa = __shfl_up(ia, off), xb = __shfl_up(ib, off);
    if (lane >= off) { ia += xa; ib += xb; }
  }
  if (lane == 63) { wsum[wave] = ia; wsum[SEL_WAVES + wave] = ib; }
  __syncthreads();
  int pa = 0, pb = 0;
  ta = 0; tb = 0;
  for (int wv = 0; wv < SEL_WAVES; ++wv) {
    const int sa = wsum[wv], sb = wsum[SEL_WAVES + wv];
    if (wv < wave) { pa += sa; pb += sb; }
    ta += sa; tb += sb;
  }
  ea = pa + ia - a; eb = pb + ib - b;
  __syncthreads();
}

// Thread t owns the SEG consecutive tokens starting at t*SEG (keys stay in registers).  The key of rank B is found by counting: a
// histogram of the keys between the smallest and the largest one (SEL_BINS bins of equal width in the integer image, that is
// logarithmic in the score), a scan from the top for the bin that holds rank B, and again inside that bin until it is one key wide
// or its keys fit a list, whose entries then count the larger ones among themselves.  One histogram and a list of some tens of keys as a
// rule.  With a bisection on the key bits (a ballot and a population count per owned token and bit) and the scalar re-decision the whole
// kernel took 36, 113 and 158 us on 288, 320 and 288 heads of 8192, 16384 and 32768 tokens; it takes 25, 59 to 74 and 98.
// With REFINE the tokens whose score lies in the relative band around the threshold are re-decided in double from K, Q
// and the row log-sum-exp before the list is written (same decisions as select followed by the refinement kernel).
// Waves per SIMD: four, 128 registers a lane.  The fp32 kernel with REFINE keeps 45 of its values in scratch memory then, and six with 168 registers; with
// 256 threads three workgroups still share a compute unit (head_dim 64, 2048 tokens, 96, 288, 576 heads: four waves 11.2, 12.4, 17.2 us, three 9.3, 9.5,
// 11.7, two and no scratch 9.4, 9.5, 14.7).  bf16 has fewer to keep and gains nothing by them.
constexpr int SEL_BINS = 2048;
constexpr int SEL_LIST = 256;

template <int SEG, int SEL_THREADS, bool REFINE, typename ET>
__global__ __launch_bounds__(SEL_THREADS, REFINE && sizeof(ET) == 4 && SEL_THREADS == 256 ? 3 : 4) void k_select(const float* __restrict__ scores, int N, int head0,
                                                        int uniform_budget, BudgetBatch per_head, int use_per_head,
                                                        int max_budget, int32_t* __restrict__ idx,
                                                        int32_t* __restrict__ n_keep, const ET* __restrict__ K,
                                                        const ET* __restrict__ Q, const double* __restrict__ row_lse,
                                                        int d, int R, int scs, int kvs,
                                                        int32_t* __restrict__ sel_flags /*nullable; written with REFINE only*/) {
  constexpr int SEL_WAVES = SEL_THREADS / 64;
  __shared__ __attribute__((aligned(16))) int hist[SEL_BINS];
  __shared__ uint32_t list[SEL_LIST];
  __shared__ int band[REFINE ? kBandCap : 1], band_raw[REFINE ? kBandCap : 1];
  __shared__ double band_score[REFINE ? kBandCap : 1];
  __shared__ int keep_new[REFINE ? kBandCap : 1];
  __shared__ int s_changed, s_bin, s_above, s_nlist, s_nband, s_nkb;
  __shared__ uint32_t s_T;
  __shared__ uint32_t wmin[SEL_WAVES], wmax[SEL_WAVES];
  __shared__ int wsum[2 * SEL_WAVES];
  const int head = head0 + blockIdx.x;
  const float* sc = scores + (size_t)head * scs;
  int32_t* out = idx + (size_t)head * max_budget;
  int B = use_per_head ? per_head.b[blockIdx.x] : uniform_budget;
  if (B > N) B = N;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  if (B == 0 || B == N) {
    for (int i = tid; i < max_budget; i += SEL_THREADS) out[i] = (i < B) ? i : -1;
    if (tid == 0) { n_keep[head] = B; if (REFINE && sel_flags) sel_flags[head] = 0; }
    return;
  }
  const int base = tid * SEG;
  uint32_t key[SEG];
  int nvalid = min(SEG, max(0, N - base));                     // tokens of this thread inside the head
  if (nvalid == SEG && (((uintptr_t)(sc + base) & 15) == 0)) {
#pragma unroll
    for (int i = 0; i < SEG; i += 4) {
      const float4 v = *(const float4*)(sc + base + i);
      key[i] = order_key(v.x); key[i + 1] = order_key(v.y); key[i + 2] = order_key(v.z); key[i + 3] = order_key(v.w);
    }
  } else {
#pragma unroll
    for (int i = 0; i < SEG; ++i) key[i] = (i < nvalid) ? order_key(sc[base + i]) : 0u;
  }
  if (tid == 0) { s_nlist = 0; s_changed = 0; s_nband = 0; s_nkb = 0; }

  // the keys' range
  {
    uint32_t mn = 0xffffffffu, mx = 0u;
#pragma unroll
    for (int i = 0; i < SEG; ++i) if (i < nvalid) { mn = min(mn, key[i]); mx = max(mx, key[i]); }
    for (int off = 32; off > 0; off >>= 1) { mn = min(mn, (uint32_t)__shfl_xor((int)mn, off)); mx = max(mx, (uint32_t)__shfl_xor((int)mx, off)); }
    if (lane == 0) { wmin[wave] = mn; wmax[wave] = mx; }
  }
  __syncthreads();
  uint32_t lo_key = 0xffffffffu, hi_key = 0u;
  for (int w = 0; w < SEL_WAVES; ++w) { lo_key = min(lo_key, wmin[w]); hi_key = max(hi_key, wmax[w]); }
  int need = B;                                                // rank wanted among the keys of [lo_key, hi_key]
  int n_gt = 0;                                                // keys above hi_key; at the end: above T
  uint32_t T = lo_key;
  for (;;) {                                                   // uniform
    const uint32_t span = hi_key - lo_key;
    if (span == 0u) { T = lo_key; break; }
    const int shift = max(0, 32 - __clz((int)span) - 11);      // span >> shift < SEL_BINS = 2^11
    for (int i = tid; i < SEL_BINS; i += SEL_THREADS) hist[i] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SEG; ++i) {
      const uint32_t o = key[i] - lo_key;                      // keys below the range wrap to above the span
      if (i < nvalid && o <= span) atomicAdd(&hist[o >> shift], 1);
    }
    __syncthreads();
    // from the top: this thread's bins are hb - 1 .. hb - PER
    constexpr int PER = SEL_BINS / SEL_THREADS;
    const int hb = SEL_BINS - tid * PER;
    int c[PER], mine = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) { c[i] = hist[hb - 1 - i]; mine += c[i]; }
    int inc = mine;
    for (int off = 1; off < 64; off <<= 1) { const int x = __shfl_up(inc, off); if (lane >= off) inc += x; }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int before = inc - mine;
    for (int w = 0; w < wave; ++w) before += wsum[w];
    if (before < need && need <= before + mine) {
      int above = before;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        if (above < need && need <= above + c[i]) { s_bin = hb - 1 - i; s_above = above; }
        above += c[i];
      }
    }
    __syncthreads();
    const int bin = s_bin, above = s_above, inside = hist[bin];
    n_gt += above; need -= above;
    const uint64_t top = (uint64_t)lo_key + (((uint64_t)bin + 1u) << shift) - 1u;
    if (top < (uint64_t)hi_key) hi_key = (uint32_t)top;        // (the last bin may run past the largest key)
    lo_key += (uint32_t)bin << shift;
    if (shift == 0) { T = lo_key; break; }
    if (inside <= SEL_LIST) {
      const uint32_t w = hi_key - lo_key;
#pragma unroll
      for (int i = 0; i < SEG; ++i) if (i < nvalid && key[i] - lo_key <= w) list[atomicAdd(&s_nlist, 1)] = key[i];
      __syncthreads();
      for (int t = tid; t < inside; t += SEL_THREADS) {
        const uint32_t k = list[t];
        int gt = 0, ge = 0;
        for (int j = 0; j < inside; ++j) { gt += list[j] > k; ge += list[j] >= k; }
        if (gt < need && need <= ge) { s_T = k; s_above = gt; }                // the same from every copy of the key
      }
      __syncthreads();
      T = s_T;
      n_gt += s_above;
      break;
    }
    __syncthreads();                                           // hist is cleared again
  }
  // keys greater than T are all kept; of the keys equal to T the lowest indices fill the rest
  const int need_eq = B - n_gt;
  int cg = 0, ce = 0;
#pragma unroll
  for (int i = 0; i < SEG; ++i) { if (i < nvalid) { cg += (key[i] > T); ce += (key[i] == T); } }
  int eg, ee, tg, te;
  block_exscan2<SEL_WAVES>(cg, ce, eg, ee, tg, te, wsum);
  bool refined = false;
  int nband = 0;
  float lo = 0.f, hi = 0.f;
  if (REFINE) {
    // band around the threshold score, in the same float arithmetic as the standalone refinement
    const float tau = key_to_float(T);
    const float half = kBandRel * fabsf(tau);
    lo = tau - half; hi = tau + half;
    {
      int er = ee;                                      // running count of keys equal to T before this token
#pragma unroll
      for (int i = 0; i < SEG; ++i) {
        if (i < nvalid) {
          const uint32_t k = key[i];
          const float s = key_to_float(k);
          const bool kept = (k > T) || (k == T && er < need_eq);
          er += (k == T);
          if (s >= lo && s <= hi) {                     // few: collected as they come, put in index order below
            const int p = atomicAdd(&s_nband, 1);
            if (kept) atomicAdd(&s_nkb, 1);
            if (p < kBandCap) band_raw[p] = ((base + i) << 1) | (kept ? 1 : 0);
          }
        }
      }
    }
    __syncthreads();
    nband = s_nband;
    const int nkb = s_nkb;
    // a band that straddles the threshold but is too large to re-score keeps the single-precision order: say so
    if (sel_flags && tid == 0) sel_flags[head] = (nband > kBandCap && nkb > 0 && nkb < nband) ? OBF_SELECT_BAND_OVERFLOW : 0;
    if (nband > 1 && nband <= kBandCap && nkb > 0 && nkb < nband) {       // uniform
      for (int t = tid; t < nband; t += SEL_THREADS) {
        const int raw = band_raw[t];
        int rank = 0;
        for (int j = 0; j < nband; ++j) rank += band_raw[j] < raw;
        band[rank] = raw >> 1; keep_new[rank] = raw & 1;
      }
      __syncthreads();
      rescore_band<ET, SEL_WAVES>(K + (size_t)head * kvs * d, Q + (size_t)head * R * d, row_lse + (size_t)head * R, d, R,
                                 band, nband, band_score, *(RescoreScratch*)hist);
      int keep = 0, was = 0;
      if (tid < nband) { was = keep_new[tid]; keep = band_keeps(band_score, nband, nkb, tid); if (keep != was) s_changed = 1; }
      __syncthreads();
      if (tid < nband) keep_new[tid] = keep;
      __syncthreads();
      refined = s_changed != 0;
    }
  }
  if (!refined) {
#pragma unroll
    for (int i = 0; i < SEG; ++i) {
      if (i < nvalid) {
        const uint32_t k = key[i];
        if (k > T) { out[eg + min(ee, need_eq)] = base + i; ++eg; }
        else if (k == T) { if (ee < need_eq) out[eg + ee] = base + i; ++ee; }
      }
    }
  } else {
    // membership changed inside the band: recount positions from the final flags
    uint32_t flags = 0u;
    int cnt = 0;
    {
      int er = ee;
#pragma unroll
      for (int i = 0; i < SEG; ++i) {
        if (i < nvalid) {
          const uint32_t k = key[i];
          const float s = key_to_float(k);
          bool kept = (k > T) || (k == T && er < need_eq);
          er += (k == T);
          if (s >= lo && s <= hi) {
            int bp = 0;
            while (band[bp] != base + i) ++bp;          // it is one of the nband tokens listed
            kept = keep_new[bp] != 0;
          }
          if (kept) { flags |= 1u << i; ++cnt; }
        }
      }
    }
    int e0, e1, t0, t1;
    block_exscan2<SEL_WAVES>(cnt, 0, e0, e1, t0, t1, wsum);
#pragma unroll
    for (int i = 0; i < SEG; ++i) if (flags & (1u << i)) out[e0++] = base + i;
  }
  for (int i = B + tid; i < max_budget; i += SEL_THREADS) out[i] = -1;
  if (tid == 0) n_keep[head] = B;
}

template <int SEG, int SEL_THREADS, bool REFINE, typename T>
static obf_status_t launch_select_seg(const Dims& m, const float* scores, const int32_t* budgets_host, int32_t budget,
                                      int32_t max_budget, int32_t* idx, int32_t* n_keep, const void* K, const void* Q,
                                      const double* row_lse, hipStream_t st, int32_t* sel_flags) {
  BudgetBatch bb;
  if (!budgets_host) {
    { ProfScope prof_(ST_SELECT, st);
      hipLaunchKernelGGL((k_select<SEG, SEL_THREADS, REFINE, T>), dim3(m.heads), dim3(SEL_THREADS), 0, st, scores, m.N, 0,
                         budget, bb, 0, max_budget, idx, n_keep, (const T*)K, (const T*)Q, row_lse, m.d, m.R, m.scs, m.kvs, sel_flags); }
    return check_launch("select");
  }
  for (int h0 = 0; h0 < m.heads; h0 += SEL_BATCH) {
    const int nb = (m.heads - h0 < SEL_BATCH) ? (m.heads - h0) : SEL_BATCH;
    for (int i = 0; i < nb; ++i) bb.b[i] = budgets_host[h0 + i];
    { ProfScope prof_(ST_SELECT, st);
      hipLaunchKernelGGL((k_select<SEG, SEL_THREADS, REFINE, T>), dim3(nb), dim3(SEL_THREADS), 0, st, scores, m.N, h0, 0, bb,
                         1, max_budget, idx, n_keep, (const T*)K, (const T*)Q, row_lse, m.d, m.R, m.scs, m.kvs, sel_flags); }
    if (check_launch("select") != OBF_OK) return OBF_ERR_HIP;
  }
  return OBF_OK;
}

template <bool REFINE, typename T>
static obf_status_t dispatch_select(const Dims& m, const float* scores, const int32_t* budgets_host, int32_t budget,
                                    int32_t max_budget, int32_t* idx, int32_t* n_keep, const void* K, const void* Q,
                                    const double* row_lse, hipStream_t st, int32_t* sel_flags) {
  // a workgroup's time is its scans and barriers, which a larger one pays more for, and its keys in LDS atomics: 16 keys per thread up
  // to 8192 tokens, 32 above (288 heads x 8192: 26 us, 32 with (32, 256), 33 with (8, 1024); 320 x 16384: 59 us, 70 with (16, 1024);
  // 288 x 2048: 13 us, 13 with (4, 512), 20 with (2, 1024))
#define OBF_SEL(SEG, THR) launch_select_seg<SEG, THR, REFINE, T>(m, scores, budgets_host, budget, max_budget, idx, n_keep, K, Q, row_lse, st, sel_flags)
  if (m.N <= 4 * 256) return OBF_SEL(4, 256);
  if (m.N <= 8 * 256) return OBF_SEL(8, 256);
  if (m.N <= 16 * 256) return OBF_SEL(16, 256);
  if (m.N <= 16 * 512) return OBF_SEL(16, 512);
  if (m.N <= 32 * 512) return OBF_SEL(32, 512);
  return OBF_SEL(32, 1024);
#undef OBF_SEL
}

obf_status_t launch_select(const Dims& m, const float* scores, const int32_t* budgets_host, int32_t budget,
                           int32_t max_budget, int32_t* idx, int32_t* n_keep, hipStream_t st) {
  return dispatch_select<false, float>(m, scores, budgets_host, budget, max_budget, idx, n_keep, nullptr, nullptr, nullptr, st, nullptr);
}

obf_status_t launch_select_refine(const Dims& m, const float* scores, const int32_t* budgets_host, int32_t budget,
                                  int32_t max_budget, int32_t* idx, int32_t* n_keep, const void* K, const void* Q,
                                  const double* row_lse, hipStream_t st, int32_t* sel_flags) {
  if (m.dtype == OBF_BF16)
    return dispatch_select<true, uint16_t>(m, scores, budgets_host, budget, max_budget, idx, n_keep, K, Q, row_lse, st, sel_flags);
  return dispatch_select<true, float>(m, scores, budgets_host, budget, max_budget, idx, n_keep, K, Q, row_lse, st, sel_flags);
}

__global__ void k_diag_flags(obf_diag_t* __restrict__ diag, const int32_t* __restrict__ sel_flags, int heads) {
  const int h = blockIdx.x * blockDim.x + threadIdx.x;
  if (h < heads) diag[h].select_flags = sel_flags[h];
}

obf_status_t launch_diag_flags(obf_diag_t* diag, const int32_t* sel_flags, int heads, hipStream_t st) {
  if (!diag || !sel_flags || heads <= 0) return OBF_OK;
  hipLaunchKernelGGL(k_diag_flags, dim3((heads + 255) / 256), dim3(256), 0, st, diag, sel_flags, heads);
  return check_launch("diag flags");
}

}  // namespace obf
