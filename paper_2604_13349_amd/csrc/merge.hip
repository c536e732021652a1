// The cache-merging comparison system of App. E on an already selected and gathered head:
//   (ii)  route every deleted token j to the retained slot whose key has the highest cosine similarity with K_j
//         (the first maximum wins; a key of zero norm has cosine 0 with everything);
//   (iii) V*_t = V_t + sum over the deleted j routed to t of A_j / (A_t + eps) V_j; keys unchanged.
// Step (i) is the library's TopK_B.  The routing is a (tokens x slots x head_dim) contraction: bf16 caches with
// head_dim 128 run it on the matrix cores (exact bf16 products, fp32 accumulation), other shapes on the vector ALU in
// fp32.  The cosine of token j with slot t is <K_j, K_t> / (|K_j| |K_t|); 1 / |K_j| is the same for every slot, so the
// arg-max only needs <K_j, K_t> / |K_t| (sign and order preserved), and an all-zero K_j routes to slot 0.
#include "common.hpp"
#include "wave_ops.hpp"

namespace obf {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int MG_THREADS = 256;
constexpr int MG_D = 128;
constexpr int MG_KK = MG_D / 16;

union MgFrag { uint4 u; bf16x8 v; };

// 1 / |K_t| of every retained key (0 for a zero key), from the gathered keys, for the routing on the vector ALU: one wave per slot.
template <typename T>
__global__ __launch_bounds__(MG_THREADS) void k_mg_inv_norm(const T* __restrict__ K_out, const int32_t* __restrict__ n_keep,
                                                            int d, int max_budget, float* __restrict__ inv_norm) {
  const int head = blockIdx.y, lane = threadIdx.x & 63;
  const int slot = blockIdx.x * (MG_THREADS / 64) + (threadIdx.x >> 6);
  if (slot >= max_budget) return;
  float s = 0.f;
  if (slot < n_keep[head]) {
    const T* row = K_out + ((size_t)head * max_budget + slot) * d;
    for (int c = lane; c < d; c += 64) { const float x = Elem<T>::load(row + c); s = fmaf(x, x, s); }
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if (lane == 0) inv_norm[(size_t)head * max_budget + slot] = s > 0.f ? 1.0f / sqrtf(s) : 0.f;
}

// Routing on the matrix cores.  A workgroup owns 256 tokens, a wave two blocks of 32 whose keys stay in registers (lane l and lane
// l + 32 both hold token l % 32, the two halves of head_dim's 16-element MFMA steps); it walks the retained slots 32 at a time, staged
// in LDS once for the four waves (the next tile's rows travel meanwhile) together with their reciprocal norms: the 32 x 32 tile of dot
// products has, in entry i of lane l, slot s0 + (i/4)*8 + (l/32)*4 + i%4 against token l%32, so the running maximum is kept per lane
// over slots in ascending order and the two lanes of a token are combined at the end.  Retained tokens are written as -1 here.
// Bound by the vector work on the tiles (multiply, compare, two selects per entry) beside one pass over K.
// 56 us on 288 heads x 2048 tokens x 205 slots (59 with three waves per SIMD); 423 us with the slots' rows and norms read from memory by every wave, and two more
// launches (19 us) for the norms and the retained tokens.
constexpr int MG_TOK = 256;              // tokens per workgroup
constexpr int MG_LDB = MG_D * 2 + 16;    // LDS bytes per staged slot row: 16-byte reads of eight consecutive rows use different banks

__global__ __launch_bounds__(MG_THREADS, 4) void k_mg_route_mfma(const uint16_t* __restrict__ K, const uint16_t* __restrict__ K_out,
                                                                 const int32_t* __restrict__ idx, const int32_t* __restrict__ n_keep,
                                                                 int N, int kvs, int max_budget, int32_t* __restrict__ route) {
  __shared__ __attribute__((aligned(16))) uint8_t stage[2][32 * MG_LDB];
  __shared__ __attribute__((aligned(16))) float inv[2][32];
  __shared__ uint32_t kept[MG_TOK / 32];
  const int head = blockIdx.y, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 31, lh = lane >> 5;
  const int base = blockIdx.x * MG_TOK, tok = base + wave * 64 + lr;       // and tok + 32
  const int nk = min(n_keep[head], max_budget);
  int32_t* rt = route + (size_t)head * N;
  if (nk <= 0) { if (base + tid < N) rt[base + tid] = -1; return; }
  const uint16_t* Kh = K + (size_t)head * kvs * MG_D;
  const uint16_t* Ko = K_out + (size_t)head * max_budget * MG_D;
  const int32_t* id = idx + (size_t)head * max_budget;
  MgFrag tf[2][MG_KK];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const uint4* p = (const uint4*)(Kh + (size_t)min(tok + 32 * b, N - 1) * MG_D + lh * 8);
#pragma unroll
    for (int kk = 0; kk < MG_KK; ++kk) tf[b][kk].u = p[kk * 2];
  }
  // a thread moves 2 x 16 bytes of slot row tid / 8: columns c .. c + 7 and c + 64 .. c + 71, c = 8 spart; spart is numbered so that the
  // threads whose sparts differ in one bit are each other's mirror image of eight, or neighbours in four (single-instruction exchanges)
  const int srow = tid >> 3, spart = (tid & 7) ^ ((tid & 4) ? 3 : 0);
  uint4 pre[2];
  auto fetch = [&](const int s0) {
    const uint4* p = (const uint4*)(Ko + (size_t)min(s0 + srow, nk - 1) * MG_D + spart * 8);     // rows past the list: the last one again
    pre[0] = p[0]; pre[1] = p[8];
  };
  auto put = [&](const int s0, const int buf) {
    uint4* o = (uint4*)(stage[buf] + srow * MG_LDB + spart * 16);
    o[0] = pre[0]; o[8] = pre[1];
    // The squared norm is added as k_mg_inv_norm does, a lane per two columns c and c + 64 and a butterfly from the high bit down: routes
    // between nearly equal cosines depend on it.  Column 8 spart + i: the three high bits are the thread's, exchanged by halves.
    float q[8];
    {
      const uint32_t wa[4] = {pre[0].x, pre[0].y, pre[0].z, pre[0].w}, wb[4] = {pre[1].x, pre[1].y, pre[1].z, pre[1].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float a0 = __uint_as_float(wa[i] << 16), a1 = __uint_as_float(wa[i] & 0xffff0000u);
        const float b0 = __uint_as_float(wb[i] << 16), b1 = __uint_as_float(wb[i] & 0xffff0000u);
        q[2 * i] = fmaf(b0, b0, a0 * a0); q[2 * i + 1] = fmaf(b1, b1, a1 * a1);
      }
    }
    const bool p4 = (spart & 4) != 0, p2 = (spart & 2) != 0, p1 = (spart & 1) != 0;
#define OBF_MG_EXCH(x, ctrl) __uint_as_float(OBF_DPP_MOV(__float_as_uint(x), ctrl))      /* 0x141: spart ^ 4, 0x4E: ^ 2, 0xB1: ^ 1 */
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float keep = p4 ? q[i + 4] : q[i], give = p4 ? q[i] : q[i + 4];
      q[i] = keep + OBF_MG_EXCH(give, 0x141);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float keep = p2 ? q[i + 2] : q[i], give = p2 ? q[i] : q[i + 2];
      q[i] = keep + OBF_MG_EXCH(give, 0x4E);
    }
    float s;                                                   // column sum i = spart
    {
      const float keep = p1 ? q[1] : q[0], give = p1 ? q[0] : q[1];
      s = keep + OBF_MG_EXCH(give, 0xB1);
    }
    s += OBF_MG_EXCH(s, 0x141);
    s += OBF_MG_EXCH(s, 0x4E);
    s += OBF_MG_EXCH(s, 0xB1);
#undef OBF_MG_EXCH
    // 0 for a zero key; a slot past the list compares as not a number: never the maximum
    if (spart == 0) inv[buf][srow] = (s0 + srow >= nk) ? __uint_as_float(0x7fc00000u) : s > 0.f ? 1.0f / sqrtf(s) : 0.f;
  };
  fetch(0);
  if (tid < MG_TOK / 32) kept[tid] = 0u;
  put(0, 0);
  if (nk > 32) fetch(32);
  __syncthreads();
  for (int i = tid; i < nk; i += MG_THREADS) {                 // the retained tokens of the workgroup's range
    const unsigned j = (unsigned)(id[i] - base);
    if (j < (unsigned)MG_TOK) atomicOr(&kept[j >> 5], 1u << (j & 31));
  }
  float best[2] = {-INFINITY, -INFINITY};
  int bslot[2] = {0, 0};
  int buf = 0;
  for (int s0 = 0; s0 < nk; s0 += 32, buf ^= 1) {
    f32x16 acc[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[b][i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < MG_KK; ++kk) {
      MgFrag sf;
      sf.u = *(const uint4*)(stage[buf] + lr * MG_LDB + kk * 32 + lh * 16);
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sf.v, tf[0][kk].v, acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sf.v, tf[1][kk].v, acc[1], 0, 0, 0);
    }
    if (s0 + 32 < nk) {                                        // uniform
      put(s0 + 32, buf ^ 1);
      if (s0 + 64 < nk) fetch(s0 + 64);
    }
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const float4 iv = *(const float4*)&inv[buf][i4 * 8 + lh * 4];           // this lane's four consecutive slots of the group
      const float iw[4] = {iv.x, iv.y, iv.z, iv.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const float c = acc[b][i4 * 4 + e] * iw[e];
          if (c > best[b]) { best[b] = c; bslot[b] = s0 + i4 * 8 + lh * 4 + e; }    // strict: the first maximum wins
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const float ob = __shfl_xor(best[b], 32);
    const int os = __shfl_xor(bslot[b], 32);
    if (ob > best[b] || (ob == best[b] && os < bslot[b])) bslot[b] = os;
    const int t = tok + 32 * b;
    if (lh == 0 && t < N) rt[t] = ((kept[(t - base) >> 5] >> ((t - base) & 31)) & 1u) ? -1 : bslot[b];
  }
}

// Routing on the vector ALU (fp32 caches, head_dim 64): one thread per token, the retained keys staged through LDS
// 32 at a time; fp32 products and sums.
template <typename T>
__global__ __launch_bounds__(MG_THREADS) void k_mg_route_generic(const T* __restrict__ K, const T* __restrict__ K_out,
                                                                 const float* __restrict__ inv_norm,
                                                                 const int32_t* __restrict__ n_keep, int N, int d, int kvs,
                                                                 int max_budget, int32_t* __restrict__ route) {
  __shared__ float ks[32][129];
  const int head = blockIdx.y;
  const int tok = blockIdx.x * MG_THREADS + threadIdx.x;
  const int nk = n_keep[head];
  int32_t* rt = route + (size_t)head * N;
  if (nk <= 0) { if (tok < N) rt[tok] = -1; return; }
  const T* kr = K + ((size_t)head * kvs + min(tok, N - 1)) * d;
  const T* Ko = K_out + (size_t)head * max_budget * d;
  const float* inv = inv_norm + (size_t)head * max_budget;
  float best = -INFINITY;
  int bslot = 0;
  for (int s0 = 0; s0 < nk; s0 += 32) {
    __syncthreads();
    for (int e = threadIdx.x; e < 32 * d; e += MG_THREADS) {
      const int r = e / d, c = e % d;
      ks[r][c] = (s0 + r < nk) ? Elem<T>::load(Ko + (size_t)(s0 + r) * d + c) : 0.f;
    }
    __syncthreads();
    const int ns = min(32, nk - s0);
    for (int r = 0; r < ns; ++r) {
      float acc = 0.f;
      for (int c = 0; c < d; ++c) acc = fmaf(Elem<T>::load(kr + c), ks[r][c], acc);
      const float cs = acc * inv[s0 + r];
      if (cs > best) { best = cs; bslot = s0 + r; }
    }
  }
  if (tok < N) rt[tok] = bslot;
}

__global__ __launch_bounds__(MG_THREADS) void k_mg_fill(int32_t* __restrict__ p, size_t n, int32_t v) {
  const size_t i = (size_t)blockIdx.x * MG_THREADS + threadIdx.x;
  if (i < n) p[i] = v;
}

// retained tokens take no part in the routing
__global__ __launch_bounds__(MG_THREADS) void k_mg_unroute_kept(const int32_t* __restrict__ idx, const int32_t* __restrict__ n_keep,
                                                                int N, int max_budget, int32_t* __restrict__ route) {
  const int head = blockIdx.y;
  const int t = blockIdx.x * MG_THREADS + threadIdx.x;
  if (t < n_keep[head] && t < max_budget) route[(size_t)head * N + idx[(size_t)head * max_budget + t]] = -1;
}

// Deleted tokens sorted by slot, one workgroup per head: entries offs[slot] .. offs[slot + 1] of `order` list the tokens of a slot with
// their weights, in no particular order within it (the merge sorts its own, short, list).  The weight is worked out here, a thread per
// token: in the merge it would cost every slot's wave a double-precision division and two more reads in its chain.
struct MgEntry { int32_t tok; float w; };

// A_j / (A_t + eps), rounded once; the Per-token alternative weighs by A_j itself
__device__ __forceinline__ float mg_weight(float aj, float at, bool per_token) { return per_token ? aj : (float)((double)aj / ((double)at + kEps)); }

constexpr int MB_AHEAD = 4;              // tokens of a thread whose reads travel together
constexpr int MB_THREADS = 1024;
__global__ __launch_bounds__(MB_THREADS) void k_mg_bucket(const int32_t* __restrict__ route, const int32_t* __restrict__ n_keep,
                                                          const int32_t* __restrict__ idx, const float* __restrict__ scores, int N, int scs,
                                                          int max_budget, int per_token,
                                                          int32_t* __restrict__ order /*[heads][hstride]: N entries, then the offsets*/,
                                                          size_t hstride) {
  extern __shared__ int cnt[];                                 // [n_keep] counts, then running positions
  __shared__ int wsum[MB_THREADS / 64];
  const int head = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nk = min(n_keep[head], max_budget);
  if (nk <= 0) return;
  const int32_t* rt = route + (size_t)head * N;
  const int32_t* id = idx + (size_t)head * max_budget;
  const float* sc = scores + (size_t)head * scs;
  MgEntry* ord = (MgEntry*)(order + (size_t)head * hstride);   // hstride is even
  int32_t* offs = (int32_t*)(ord + N);                         // [n_keep + 1]
  for (int i = tid; i < nk; i += MB_THREADS) cnt[i] = 0;
  __syncthreads();
  for (int j = tid; j < N; j += MB_THREADS) { const int r = rt[j]; if (r >= 0) atomicAdd(&cnt[r], 1); }
  __syncthreads();
  int carry = 0;
  for (int i0 = 0; i0 < nk; i0 += MB_THREADS) {                // exclusive prefix sums, a stretch of MB_THREADS slots at a time
    const int i = i0 + tid, c = (i < nk) ? cnt[i] : 0;
    int inc = c;
    for (int off = 1; off < 64; off <<= 1) { const int x = __shfl_up(inc, off); if (lane >= off) inc += x; }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int before = carry, tot = 0;
    for (int w = 0; w < MB_THREADS / 64; ++w) { const int x = wsum[w]; if (w < wave) before += x; tot += x; }
    if (i < nk) { cnt[i] = before + inc - c; offs[i] = before + inc - c; }
    carry += tot;
    __syncthreads();
  }
  if (tid == 0) offs[nk] = carry;
  for (int j0 = tid; j0 < N; j0 += MB_AHEAD * MB_THREADS) {
    int r[MB_AHEAD];
    float aj[MB_AHEAD], at[MB_AHEAD];
#pragma unroll
    for (int u = 0; u < MB_AHEAD; ++u) {
      const int j = min(j0 + u * MB_THREADS, N - 1);
      r[u] = j == j0 + u * MB_THREADS ? rt[j] : -1;
      aj[u] = sc[j];
    }
#pragma unroll
    for (int u = 0; u < MB_AHEAD; ++u) at[u] = sc[id[max(r[u], 0)]];
#pragma unroll
    for (int u = 0; u < MB_AHEAD; ++u)
      if (r[u] >= 0) ord[atomicAdd(&cnt[r[u]], 1)] = MgEntry{j0 + u * MB_THREADS, mg_weight(aj[u], at[u], per_token != 0)};
  }
}

// The same per-slot sums serve the Per-token alternative of App. D (PER_TOKEN; the reading: the deleted tokens are shared
// out among the slots by the routing above, slot t's direction is B a_del / (a_keep + eps) times the projection of
// sum_{pi(j) = t} A_j v_j / (a_del + eps) onto the residual subspace C of Eq. 5 - C's rows lie in the complement of
// the retained span, so projecting the values is projecting their residuals; the mean over the slots is Eq. 6's delta).
// There the weights are the attention masses themselves, the sums are projected with the k_used rows of C that the
// back-fill kernel left in the head's scratch, and the result is added to the slot's value.
//
// Merge.  A wave per retained slot takes the slot's tokens in ascending order and adds their weighted value rows into a running
// sum in registers (a lane owns D / 64 columns): the order of the additions is fixed, so the result is the same on every run.  A list of
// up to MG_LIST tokens is put in order first (every entry counts the smaller ones); a longer one is not: the head's routes are scanned
// instead, which finds the slot's tokens in order.  Eight rows are in flight at a time, sixteen where the list is longer.  Slots that received nothing are left as the
// bit copies the gather wrote.  Bound by a wave's instructions per token and its chain offsets - list - rows (nine tokens a
// slot here; the offsets' read does not wait for n_keep, nor the store for the slot's own value), then by the pass over V: 55 us on 288
// heads x 2048 tokens x 205 slots, and 9 for the lists; 63 with sixteen loads for every list, 78 and 7 with the weights worked out here, 99 with eight rows ahead and every lane
// read waited for by itself, 157 with four slots per wave, 247 with each wave scanning all routes.
constexpr int MG_LIST = 256;
constexpr int MG_AHEAD = 16;

template <typename T, int CPL> struct LaneCols;                // CPL consecutive elements of a row
template <> struct LaneCols<uint16_t, 2> { typedef uint32_t type; static __device__ __forceinline__ void get(uint32_t v, float (&o)[2]) { o[0] = __uint_as_float(v << 16); o[1] = __uint_as_float(v & 0xffff0000u); } };
template <> struct LaneCols<uint16_t, 1> { typedef uint16_t type; static __device__ __forceinline__ void get(uint16_t v, float (&o)[1]) { o[0] = bf16_bits_to_float(v); } };
template <> struct LaneCols<float, 2> { typedef float2 type; static __device__ __forceinline__ void get(float2 v, float (&o)[2]) { o[0] = v.x; o[1] = v.y; } };
template <> struct LaneCols<float, 1> { typedef float type; static __device__ __forceinline__ void get(float v, float (&o)[1]) { o[0] = v; } };

template <typename T, int D, bool PER_TOKEN>
__global__ __launch_bounds__(MG_THREADS) void k_mg_merge(const T* __restrict__ V, const float* __restrict__ scores,
                                                         const int32_t* __restrict__ idx, const int32_t* __restrict__ n_keep,
                                                         const int32_t* __restrict__ route, const int32_t* __restrict__ order,
                                                         size_t hstride, int N, int kvs, int scs, int max_budget,
                                                         T* __restrict__ V_out,
                                                         const HeadState* __restrict__ state /*PER_TOKEN*/,
                                                         const float* __restrict__ mats /*PER_TOKEN: [heads][3][d*d], C in the second matrix*/,
                                                         int no_scaling) {
  constexpr int CPL = D / 64;
  typedef LaneCols<T, CPL> LC;
  __shared__ MgEntry list[MG_THREADS / 64][MG_LIST];
  __shared__ float cb[PER_TOKEN ? 16 : 1][MG_D];               // the rows of C
  const int head = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int slot = blockIdx.x * (MG_THREADS / 64) + wave;
  const MgEntry* ord = (const MgEntry*)(order + (size_t)head * hstride);
  const int32_t* offs = (const int32_t*)(ord + N);
  const int nk = min(n_keep[head], max_budget);
  const int at0 = min(slot, N);                                // the reads do not wait for n_keep; the workspace holds N + 1 offsets and more
  const int off = offs[at0], end = offs[at0 + 1];
  int kc = 0;
  float pt_scale = 0.f;
  if (PER_TOKEN) {
    const HeadState hs = state[head];
    if (!hs.active || hs.k_used <= 0) return;                  // no injection for this head (uniform over the workgroup)
    kc = min(hs.k_used, 16);
    const float* Cg = mats + ((size_t)head * 3 + 1) * D * D;
    for (int e = threadIdx.x; e < kc * D; e += MG_THREADS) cb[e / D][e % D] = Cg[e];
    pt_scale = (float)((double)hs.n_keep * (no_scaling ? 1.0 : hs.a_del / (hs.a_keep + kEps)) / (hs.a_del + kEps));
    __syncthreads();
  }
  if (slot >= nk) return;                                      // whole wave (no barrier below)
  const int len = end - off;
  if (len <= 0) return;
  const T* Vh = V + (size_t)head * kvs * D + lane * CPL;
  T* o = V_out + ((size_t)head * max_budget + slot) * D + lane * CPL;
  float old[CPL];                                              // the slot's own value, read beside the list
#pragma unroll
  for (int c = 0; c < CPL; ++c) old[c] = Elem<T>::load(o + c);
  float acc[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) acc[c] = 0.f;
  // the rows of the tokens that the first `n` lanes hold, added in lane order
  auto add_rows = [&](const int n, const int tok, const float w) {
    for (int i0 = 0; i0 < n; i0 += MG_AHEAD) {
      typename LC::type v[MG_AHEAD];
      auto load = [&](const int u) {
        const int j = __builtin_amdgcn_readlane(tok, min(i0 + u, n - 1));
        __builtin_memcpy(&v[u], Vh + (size_t)j * D, sizeof(v[u]));       // one load; V need only be aligned to its elements
      };
#pragma unroll
      for (int u = 0; u < MG_AHEAD / 2; ++u) load(u);
      if (i0 + MG_AHEAD / 2 < n) {                             // uniform; lists are short: the last row again costs as much as a new one
#pragma unroll
        for (int u = MG_AHEAD / 2; u < MG_AHEAD; ++u) load(u);
      }
#pragma unroll
      for (int u = 0; u < MG_AHEAD; ++u) {
        if (i0 + u < n) {
          const float wu = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(w), i0 + u));
          float x[CPL];
          LC::get(v[u], x);
#pragma unroll
          for (int c = 0; c < CPL; ++c) acc[c] = fmaf(wu, x[c], acc[c]);
        }
      }
    }
  };
  if (len <= MG_LIST) {
    const MgEntry* src = ord + off;
    MgEntry* dst = list[wave];
    for (int i0 = 0; i0 < len; i0 += 64) {
      const MgEntry mine = (i0 + lane < len) ? src[i0 + lane] : MgEntry{0x7fffffff, 0.f};
      int rank = 0;
      for (int q0 = 0; q0 < len; q0 += 64) {
        const int other = (q0 == i0) ? mine.tok : (q0 + lane < len) ? src[q0 + lane].tok : 0x7fffffff;
        const int n = min(64, len - q0);
        for (int q = 0; q < n; q += 8) {                       // lane reads ahead of their uses; past the end the entries are never smaller
          int k[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) k[u] = __builtin_amdgcn_readlane(other, q + u);
#pragma unroll
          for (int u = 0; u < 8; ++u) rank += (k[u] < mine.tok) ? 1 : 0;
        }
      }
      if (i0 + lane < len) dst[rank] = mine;
    }
    __builtin_amdgcn_wave_barrier();
    for (int i0 = 0; i0 < len; i0 += 64) { const MgEntry e = dst[min(i0 + lane, len - 1)]; add_rows(min(64, len - i0), e.tok, e.w); }
  } else {
    const int32_t* rt = route + (size_t)head * N;
    const float* sc = scores + (size_t)head * scs;
    const float at = PER_TOKEN ? 0.f : sc[idx[(size_t)head * max_budget + slot]];
    for (int base = 0; base < N; base += 64) {
      const int j = base + lane;
      uint64_t mask = __ballot(j < N && rt[min(j, N - 1)] == slot);
      const int n = __popcll(mask);
      int tok = 0;
      for (int i = 0; i < n; ++i) { const int b = __builtin_ctzll(mask); mask &= mask - 1; if (lane == i) tok = base + b; }
      if (n) add_rows(n, tok, lane < n ? mg_weight(sc[tok], at, PER_TOKEN) : 0.f);
    }
  }
  if (PER_TOKEN) {
    float dsum[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) dsum[c] = 0.f;
    for (int i = 0; i < kc; ++i) {                             // the sum's coefficient on every row of C, then the combination
      float g = 0.f;
#pragma unroll
      for (int c = 0; c < CPL; ++c) g = fmaf(acc[c], cb[i][lane * CPL + c], g);
      for (int of = 32; of > 0; of >>= 1) g += __shfl_xor(g, of);
#pragma unroll
      for (int c = 0; c < CPL; ++c) dsum[c] = fmaf(g, cb[i][lane * CPL + c], dsum[c]);
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c) Elem<T>::store(o + c, fmaf(pt_scale, dsum[c], old[c]));
  } else {
#pragma unroll
    for (int c = 0; c < CPL; ++c) Elem<T>::store(o + c, old[c] + acc[c]);
  }
}

// steps (ii) and (iii); per_token: the per-slot directions of App. D's Per-token alternative instead of the merge
static obf_status_t run_merge(const Dims& m, const Workspace& w, char* ws, const void* K, const void* V, const float* scores,
                              const int32_t* idx, const int32_t* n_keep, int32_t max_budget, const void* K_out,
                              void* V_out, int32_t* route_out, hipStream_t st, bool per_token, int no_scaling) {
  const HeadState* state = (const HeadState*)(ws + w.head_state);
  const float* mats = (const float*)(ws + w.mats);
  if (max_budget == 0) {                                         // nothing retained: nothing to route to
    if (route_out) {
      const size_t n = (size_t)m.heads * m.N;
      hipLaunchKernelGGL(k_mg_fill, dim3((unsigned)((n + MG_THREADS - 1) / MG_THREADS)), dim3(MG_THREADS), 0, st, route_out, n, -1);
      return check_launch("merge fill");
    }
    return OBF_OK;
  }
  float* inv_norm = (float*)(ws + w.inv_norm);
  int32_t* route = route_out ? route_out : (int32_t*)(ws + w.route);
  // the tokens by slot with their weights and the slots' offsets, 2 N + n_keep + 1 <= 3 N + 1 numbers a head (the merge's early read of the
  // offsets goes to 3 N + 2), lie where the statistics of the deleted values are during a back-fill (over 4 N a head): done with by now
  int32_t* order = (int32_t*)(ws + w.gram_part);
  const size_t hstride = (size_t)w.nstat * gram_stride(m.d);
  const bool bf = m.dtype == OBF_BF16;
  if (bf && m.d == MG_D) {
    hipLaunchKernelGGL(k_mg_route_mfma, dim3((m.N + MG_TOK - 1) / MG_TOK, m.heads), dim3(MG_THREADS), 0, st, (const uint16_t*)K,
                       (const uint16_t*)K_out, idx, n_keep, m.N, m.kvs, max_budget, route);
    if (check_launch("merge route") != OBF_OK) return OBF_ERR_HIP;
  } else {
    dim3 gn((max_budget + 3) / 4, m.heads), gr((m.N + MG_THREADS - 1) / MG_THREADS, m.heads);
    if (bf) {
      hipLaunchKernelGGL(k_mg_inv_norm<uint16_t>, gn, dim3(MG_THREADS), 0, st, (const uint16_t*)K_out, n_keep, m.d, max_budget, inv_norm);
      hipLaunchKernelGGL(k_mg_route_generic<uint16_t>, gr, dim3(MG_THREADS), 0, st, (const uint16_t*)K, (const uint16_t*)K_out, inv_norm,
                         n_keep, m.N, m.d, m.kvs, max_budget, route);
    } else {
      hipLaunchKernelGGL(k_mg_inv_norm<float>, gn, dim3(MG_THREADS), 0, st, (const float*)K_out, n_keep, m.d, max_budget, inv_norm);
      hipLaunchKernelGGL(k_mg_route_generic<float>, gr, dim3(MG_THREADS), 0, st, (const float*)K, (const float*)K_out, inv_norm, n_keep,
                         m.N, m.d, m.kvs, max_budget, route);
    }
    if (check_launch("merge route") != OBF_OK) return OBF_ERR_HIP;
    hipLaunchKernelGGL(k_mg_unroute_kept, dim3((max_budget + MG_THREADS - 1) / MG_THREADS, m.heads), dim3(MG_THREADS), 0, st, idx,
                       n_keep, m.N, max_budget, route);
    if (check_launch("merge unroute") != OBF_OK) return OBF_ERR_HIP;
  }
  static std::mutex attr_mu;
  static uint64_t attr_seen = 0;
  once_per_device(attr_mu, attr_seen, [] {
    (void)hipFuncSetAttribute((const void*)k_mg_bucket, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(int) * kMaxTokens);
  });
  hipLaunchKernelGGL(k_mg_bucket, dim3(m.heads), dim3(MB_THREADS), sizeof(int) * (size_t)(max_budget < m.N ? max_budget : m.N), st, route,
                     n_keep, idx, scores, m.N, m.scs, max_budget, per_token ? 1 : 0, order, hstride);
  if (check_launch("merge bucket") != OBF_OK) return OBF_ERR_HIP;
  dim3 gm((max_budget + MG_THREADS / 64 - 1) / (MG_THREADS / 64), m.heads);
#define OBF_MG_LAUNCH(T, D, PT) hipLaunchKernelGGL((k_mg_merge<T, D, PT>), gm, dim3(MG_THREADS), 0, st, (const T*)V, scores, idx, n_keep, \
                                                  route, order, hstride, m.N, m.kvs, m.scs, max_budget, (T*)V_out, state, mats, no_scaling)
  if (bf && m.d == 128) { if (per_token) OBF_MG_LAUNCH(uint16_t, 128, true); else OBF_MG_LAUNCH(uint16_t, 128, false); }
  else if (bf) { if (per_token) OBF_MG_LAUNCH(uint16_t, 64, true); else OBF_MG_LAUNCH(uint16_t, 64, false); }
  else if (m.d == 128) { if (per_token) OBF_MG_LAUNCH(float, 128, true); else OBF_MG_LAUNCH(float, 128, false); }
  else { if (per_token) OBF_MG_LAUNCH(float, 64, true); else OBF_MG_LAUNCH(float, 64, false); }
#undef OBF_MG_LAUNCH
  return check_launch("merge values");
}

obf_status_t launch_cache_merge(const Dims& m, const Workspace& w, char* ws, const void* K, const void* V, const float* scores,
                                const int32_t* idx, const int32_t* n_keep, int32_t max_budget, const void* K_out,
                                void* V_out, int32_t* route_out, hipStream_t st) {
  return run_merge(m, w, ws, K, V, scores, idx, n_keep, max_budget, K_out, V_out, route_out, st, false, 0);
}

obf_status_t launch_per_token_inject(const Dims& m, const Workspace& w, char* ws, const void* K, const void* V,
                                     const float* scores, const int32_t* idx, const int32_t* n_keep, int32_t max_budget,
                                     const void* K_out, void* V_out, int no_scaling, hipStream_t st) {
  if (m.d > MG_D) { set_error("per-token variant: head_dim above 128"); return OBF_ERR_UNSUPPORTED; }
  return run_merge(m, w, ws, K, V, scores, idx, n_keep, max_budget, K_out, V_out, nullptr, st, true, no_scaling);
}

}  // namespace obf
