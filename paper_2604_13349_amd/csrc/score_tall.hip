// Attention-mass scores (Eq. 1) on the matrix cores for groups of 192 and 256 query rows (bf16, head_dim 128): the two passes of score_mfma.hip -
// per-range (max, sum-exp) of every row, then the column sums of exp(logit - lse) - with a workgroup that carries all the rows of a group, so that
// K is streamed once per group and pass instead of once per 128 rows.
//
// Two workgroups of four waves share a compute unit.  K passes through LDS in steps of 64 tokens, a ring of four steps that
// global_load_lds fills (the loads of three steps in flight, no registers); the 16-byte pieces of a token lie permuted by its number, so that
// the operand reads (one piece of 32 tokens) use different banks.  A wave holds the Q operands of F blocks of 32 rows and, with H, half the work of
// one more, which it shares with its neighbour: of that block it takes the first tile of 32 tokens, the other wave the second.  All waves run
// one instruction stream, the operands are picked by LDS address.  The product of the next (block, tile) is issued beside the vector work of the
// present one; while a wave waits at a step's barrier the other workgroup's on the same SIMD goes on.
//
// Where there are thousands of tokens per workgroup: K from memory and the products beside each other, at a clock that falls with the power drawn (second
// pass, 288 heads of 32768 tokens: K once, 1.3 million cycles, the matrix pipe busy in 0.45 of them; 690 us at 1.9 GHz after a pause, 740 at 1.8 in a
// row of calls).  Else the loads, the waits at the steps and, with few heads, the fold of the partials.  Both passes, us, pairs of 128-row groups (192
// rows padded to them) and this:
//   256 rows  288 heads of 128, 2048, 8192 tokens 45 - 19, 113 - 98, 394 - 390    96 of 9000 147 - 133    8 of 2048 28 - 16
//   192 rows  288 heads of 2048, 4001 tokens 109 - 84, 200 - 156
// Carrying the first product of a step across its barrier was no faster, sums against a reference that moves only when outgrown neither
// (most tiles of a cache with outlier tokens outgrow it in some lane), 320 rows this way (160 operand registers a lane) slower.
// Errors against 64 bits, six draws of each of eleven shapes of 161 to 512 rows, with and without tokens of eight times the size: rms of scores 0.95 and of
// normalisers 0.83 of the pairs' (geometric means; 0.85 to 0.99 and 0.52 to 0.93), largest errors 0.98 and 0.91 (0.83 to 1.20 and 0.72 to 1.11).
#include "score_parts.hpp"
#include "wave_ops.hpp"

namespace obf {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

union TallFrag { uint4 u; bf16x8 v; };

constexpr int TA_THREADS = 256, TA_D = 128;
constexpr int TA_STEP = kScoreTallStep;  // tokens per step: two tiles of 32
constexpr int TA_RING = 4, TA_AHEAD = TA_RING - 1;
constexpr int TA_LOADS = TA_STEP / 16;   // 16-byte loads of a lane per step
constexpr int TA_BYTES = TA_STEP * TA_D * 2;

struct TallPart {
  int SH;        // steps per head; more than its tokens make where ranges end with their head, whose last range is then the shorter
  int T;         // steps per range
  long TT;       // heads * SH
  long kstride;  // elements between consecutive heads of K
};

// Four times 16 bytes per lane from base + off to LDS at `lds` + 16 lane and 4096 further each time, without registers between; complete when vmcnt says
// so.  (The builtin would have the compiler wait for the youngest of these loads before every read of LDS.)  m0 is left as it was: the compiler reserves
// it and would not be told by a clobber.
__device__ __forceinline__ void load_to_lds(const uint32_t lds, const uint32_t (&off)[4], const void* base) {
  uint32_t m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %6\n\t"
               "s_add_u32 m0, m0, 0x1000\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %6\n\t"
               "s_add_u32 m0, m0, 0x1000\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, %6\n\t"
               "s_add_u32 m0, m0, 0x1000\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %5, %6\n\ts_mov_b32 m0, %0"
               : "=&s"(m0) : "s"(lds), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base) : "memory", "scc");
}
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// The 64 tokens from Kt on (rows past `last` repeat it) to a step of the ring: token r's piece c goes to place c ^ (r % 16).  Keys off a 16-byte boundary
// go through registers.
__device__ __forceinline__ void fill_step(char* ring, const uint32_t lds, const uint16_t* Kt, const int last, const int wave, const int lane,
                                          const bool aligned) {
  const int r0 = wave * 4 + (lane >> 4);
  const uint32_t piece = (uint32_t)(((lane & 15) ^ r0) << 4);
  static_assert(TA_LOADS == 4, "loads of load_to_lds");
  uint32_t off[TA_LOADS];
#pragma unroll
  for (int i = 0; i < TA_LOADS; ++i) off[i] = (uint32_t)(min(i * 16 + r0, last) << 8) + piece;
  if (aligned) {
    load_to_lds(lds + wave * 1024, off, Kt);
  } else {
#pragma unroll
    for (int i = 0; i < TA_LOADS; ++i) *(uint4*)(ring + i * 4096 + wave * 1024 + lane * 16) = *(const uint4*)((const char*)Kt + off[i]);
  }
}

__device__ __forceinline__ void tall_q(TallFrag (&qf)[8], const uint16_t* __restrict__ Qh, const int row0, const int R, const int lane) {
  const uint4* p = (const uint4*)(Qh + (size_t)min(row0 + (lane & 31), R - 1) * TA_D) + (lane >> 5);
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) qf[kk].u = p[kk * 2];
}

// operands of a tile of 32 tokens
__device__ __forceinline__ void tall_k(TallFrag (&kf)[8], const char* tile, const int lane) {
  const int r = lane & 31, g = lane >> 5;
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) kf[kk].u = *(const uint4*)(tile + r * 256 + (((kk * 2 + g) ^ (r & 15)) << 4));
}

template <bool TOKENS_BY_ROWS>
__device__ __forceinline__ void tall_mfma(f32x16& acc, const TallFrag (&kf)[8], const TallFrag (&qf)[8]) {
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
  for (int kk = 0; kk < 8; ++kk)
    acc = TOKENS_BY_ROWS ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk].v, qf[kk].v, acc, 0, 0, 0)
                         : __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[kk].v, kf[kk].v, acc, 0, 0, 0);
}

// a matrix instruction of the next product, then vector work of the present one, eight times
__device__ __forceinline__ void tall_mix() {
#pragma unroll
  for (int i = 0; i < 8; ++i) { __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); __builtin_amdgcn_sched_group_barrier(0x402, 6, 0); }
}

__device__ __forceinline__ float tall_sum(const f32x16& acc, const float a2, const float ref) {
  float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll
  for (int i = 0; i < 16; i += 4) {
    s0 += fast_exp2(fmaf(acc[i], a2, -ref));
    s1 += fast_exp2(fmaf(acc[i + 1], a2, -ref));
    s2 += fast_exp2(fmaf(acc[i + 2], a2, -ref));
    s3 += fast_exp2(fmaf(acc[i + 3], a2, -ref));
  }
  return (s0 + s1) + (s2 + s3);
}

// First pass: the lane's row against 16 tokens; ref: the row's largest logit so far, in powers of two.
__device__ __forceinline__ void tall_stats(const f32x16& acc, const float a2, float& ref, double& l) {
  float mx = fmaxf(fmaxf(acc[0], acc[1]), acc[2]);
#pragma unroll
  for (int i = 3; i < 15; i += 2) mx = fmaxf(fmaxf(mx, acc[i]), acc[i + 1]);
  const float next = fmaxf(ref, fmaxf(mx, acc[15]) * a2);
  l = fma(l, (double)fast_exp2(ref - next), (double)tall_sum(acc, a2, next));          // (ref is -inf at first: a factor of 0)
  ref = next;
}

// The same for a tile of which only tokens below N count; tok: the lane's first.
__device__ __forceinline__ void tall_stats_ragged(const f32x16& acc, const float a2, float& ref, double& l, const int tok, const int N) {
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < 16; ++i) if (tok + (i >> 2) * 8 + (i & 3) < N) mx = fmaxf(mx, acc[i]);
  if (tok < N) {
    float next = fmaxf(ref, mx * a2);
    if (!(next > -INFINITY)) next = 0.f;
    float ts = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) if (tok + (i >> 2) * 8 + (i & 3) < N) ts += fast_exp2(fmaf(acc[i], a2, -next));
    l = fma(l, (double)fast_exp2(ref - next), (double)ts);
    ref = next;
  }
}

// Which range and row group a workgroup has: the RG workgroups that stream the same tokens get block indices 8 apart, so they run on one XCD.
struct TallPlace { int range, rg; };
__device__ __forceinline__ TallPlace tall_place(const int RG) {
  const int group = blockIdx.x / (8 * RG), in = blockIdx.x - group * (8 * RG);
  return TallPlace{group * 8 + (in & 7), in >> 3};
}

// Steps of the range that starts at gs, `pos` steps into a head.
__device__ __forceinline__ int tall_steps(const TallPart& pt, const long gs, const int pos, const int N) {
  const int n = (int)(min(pt.TT, gs + pt.T) - gs), own = (N + TA_STEP - 1) / TA_STEP;
  return own < pt.SH ? min(n, own - pos) : n;
}

// Pass A: leaves one partial (max, sum-exp) per query row and segment (the part of a head inside a range), as k_score_stats_mfma.
template <int F, int H>
__global__ __launch_bounds__(TA_THREADS, 2) void k_score_stats_tall(const uint16_t* __restrict__ K, const uint16_t* __restrict__ Q,
                                                                    double* __restrict__ stats_part, int N, int R, int RG, TallPart pt, int nslot,
                                                                    int aligned) {
  constexpr int ROWS = 128 * F + 64 * H, B = F + H, U = 2 * F + H;
  __shared__ struct { __attribute__((aligned(16))) char k[TA_RING * TA_BYTES]; double l[ROWS + 64 * H]; float m[ROWS + 64 * H]; } sm;
  const TallPlace at = tall_place(RG);
  const long gs = (long)at.range * pt.T;
  if (gs >= pt.TT) return;
  int head = (int)(gs / pt.SH), pos = (int)(gs - (long)head * pt.SH);
  const int n = tall_steps(pt, gs, pos, N);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = at.rg * ROWS;
  const float a2 = 1.4426950408889634f / sqrtf((float)TA_D);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)sm.k;
  int ih = head, ip = pos;                                     // what is loaded next
  auto feed = [&](const int b) {
    fill_step(sm.k + b * TA_BYTES, lds0 + b * TA_BYTES, K + (size_t)ih * pt.kstride + (size_t)ip * TA_STEP * TA_D, N - 1 - ip * TA_STEP, wave, lane, aligned != 0);
    if (++ip == pt.SH) { ip = 0; ++ih; }
  };
  for (int a = 0; a < TA_AHEAD; ++a) if (a < n) feed(a);
  int slot = at.range - (int)(((long)head * pt.SH) / pt.T);
  for (int s = 0; s < n;) {
    TallFrag qf[B][8];
    float ref[B];
    double l[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      tall_q(qf[b], Q + (size_t)head * R * TA_D, row0 + (b < F ? wave * F + b : 4 * F + (wave >> 1)) * 32, R, lane);
      ref[b] = -INFINITY; l[b] = 0.0;
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);                        // vmcnt(0): the loop below has no wait for them, which would wait for K as well
    const int e = min(n, s + pt.SH - pos);
    for (; s < e; ++s, ++pos) {
      if (s + TA_AHEAD <= n) wait_loads<(TA_AHEAD - 1) * TA_LOADS>(); else wait_loads<0>();
      lds_barrier();                                           // step s is there, step s - 1 has been read
      if (s + TA_AHEAD < n) feed((s + TA_AHEAD) & (TA_RING - 1));
      const int tok = pos * TA_STEP;
      const char* buf = sm.k + (s & (TA_RING - 1)) * TA_BYTES;
      TallFrag kf[2][8];
      f32x16 acc[2];
      tall_k(kf[0], buf, lane);
      tall_k(kf[1], buf + 32 * 256, lane);
      tall_mfma<true>(acc[0], kf[0], qf[0]);
      const bool whole = tok + TA_STEP <= N;                   // uniform
      auto units = [&](auto&& take) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (u + 1 < U) {
            if (H && u + 1 == 2 * F) tall_mfma<true>(acc[(u + 1) & 1], kf[0], qf[B - 1]);
            else tall_mfma<true>(acc[(u + 1) & 1], kf[(u + 1) / F], qf[(u + 1) % F]);
          }
          if (H && u == F - 1) tall_k(kf[0], buf + (wave & 1) * 32 * 256, lane);      // (its products have been issued)
          take(u, (H && u == 2 * F) ? F : u % F, (H && u == 2 * F) ? (wave & 1) : u / F);
          if (u + 1 < U) tall_mix();
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      if (whole) units([&](const int u, const int b, int) { tall_stats(acc[u & 1], a2, ref[b], l[b]); });
      else units([&](const int u, const int b, const int tile) { tall_stats_ragged(acc[u & 1], a2, ref[b], l[b], tok + tile * 32 + (lane >> 5) * 4, N); });
    }
    // the two lane halves (the same row, other tokens), then the two waves of a shared block
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const float mo = __shfl_xor(ref[b], 32);
      const double lo = __shfl_xor(l[b], 32);
      const float mn = fmaxf(ref[b], mo);
      double v = 0.0;
      if (ref[b] > -INFINITY) v = l[b] * (double)fast_exp2(ref[b] - mn);
      if (mo > -INFINITY) v += lo * (double)fast_exp2(mo - mn);
      const int row = (b < F ? (wave * F + b) * 32 : 128 * F + (wave & 1) * 64 + (wave >> 1) * 32) + lane;
      if (lane < 32) { sm.m[row] = mn; sm.l[row] = v; }
    }
    lds_barrier();
    for (int rl = threadIdx.x; rl < ROWS; rl += TA_THREADS) {
      const int row = row0 + rl;
      if (row < R) {
        float M = sm.m[rl];
        double L = sm.l[rl];
        if (H && rl >= 128 * F) {
          const float M2 = sm.m[rl + 64];
          const double L2 = sm.l[rl + 64];
          const float mn = fmaxf(M, M2);
          L = (M > -INFINITY ? L * exp2((double)M - (double)mn) : 0.0) + (M2 > -INFINITY ? L2 * exp2((double)M2 - (double)mn) : 0.0);
          M = mn;
        }
        double* o = stats_part + (((size_t)head * nslot + slot) * R + row) * 2;
        o[0] = (double)M * 0.6931471805599453; o[1] = L;      // log2 units -> natural log
      }
    }
    pos = 0; ++head; slot = 0;
  }
}

// Pass B: the same partition, walked backwards; folds its heads' partials first, as k_score_mass_mfma.
template <int F, int H>
__global__ __launch_bounds__(TA_THREADS, 2) void k_score_mass_tall(const uint16_t* __restrict__ K, const uint16_t* __restrict__ Q,
                                                                   const double* __restrict__ stats_part, double* __restrict__ row_lse,
                                                                   float* __restrict__ part, float* __restrict__ scores, int N, int R, int RG, size_t rg_stride, TallPart pt,
                                                                   TallPart sp /*the first pass's, in its units*/, int nslot, int aligned) {
  constexpr int ROWS = 128 * F + 64 * H, B = F + H, U = 2 * F + H;
  __shared__ struct { __attribute__((aligned(16))) char k[TA_RING * TA_BYTES]; __attribute__((aligned(16))) float b2[ROWS]; float ps[2][4][TA_STEP]; } sm;
  const TallPlace at = tall_place(RG);
  const long gs = (long)at.range * pt.T;
  if (gs >= pt.TT) return;
  const int n = tall_steps(pt, gs, (int)(gs % pt.SH), N);
  const long ge = gs + n;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = at.rg * ROWS;
  const float a2 = 1.4426950408889634f / sqrtf((float)TA_D);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)sm.k;
  int head = (int)((ge - 1) / pt.SH), pos = (int)(ge - 1 - (long)head * pt.SH);
  int ih = head, ip = pos;
  auto feed = [&](const int b) {
    fill_step(sm.k + b * TA_BYTES, lds0 + b * TA_BYTES, K + (size_t)ih * pt.kstride + (size_t)ip * TA_STEP * TA_D, N - 1 - ip * TA_STEP, wave, lane, aligned != 0);
    if (--ip < 0) { ip = pt.SH - 1; --ih; }
  };
  for (int a = 0; a < TA_AHEAD; ++a) if (a < n) feed(a);
  float* out = at.rg == RG - 1 ? scores : part + (size_t)at.rg * rg_stride;
  float* dst = nullptr;                                        // where the last step's sums go
  int dst_n = 0;
  auto flush = [&](const int p) {                              // the four waves' shares
    if ((int)threadIdx.x < dst_n)
      dst[threadIdx.x] = (sm.ps[p][0][threadIdx.x] + sm.ps[p][1][threadIdx.x]) + (sm.ps[p][2][threadIdx.x] + sm.ps[p][3][threadIdx.x]);
  };
  for (int s = 0; s < n;) {
    if (H) lds_barrier();                                      // the shared block's normalisers are read from LDS to the last step
    const long hs = (long)head * sp.SH;
    const int parts = (int)((hs + sp.SH - 1) / sp.T - hs / sp.T) + 1;
    for (int rl = threadIdx.x; rl < ROWS; rl += TA_THREADS) {
      const int row = row0 + rl;
      double lse = INFINITY;                                   // padded rows: exp2(-inf) = 0
      if (row < R) {
        lse = fold_row_lse(stats_part + ((size_t)head * nslot * R + row) * 2, (size_t)R, parts);
        if (gs <= (long)head * pt.SH) row_lse[(size_t)head * R + row] = lse;
      }
      sm.b2[rl] = (float)(lse * 1.4426950408889634);
    }
    TallFrag qf[B][8];
    float b2[F][16];
    lds_barrier();
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int rb = (b < F ? wave * F + b : 4 * F + (wave >> 1)) * 32;
      tall_q(qf[b], Q + (size_t)head * R * TA_D, row0 + rb, R, lane);
      if (b < F) {
#pragma unroll
        for (int i = 0; i < 4; ++i) *(float4*)&b2[b][4 * i] = *(const float4*)&sm.b2[rb + 8 * i + (lane >> 5) * 4];
      }
    }
    const float* b2h = &sm.b2[(4 * F + (wave >> 1)) * 32 + (lane >> 5) * 4];          // of the shared block
    __builtin_amdgcn_s_waitcnt(0x0070);                        // vmcnt(0) lgkmcnt(0), see k_score_stats_tall
    const int e = min(n, s + pos + 1);
    for (; s < e; ++s, --pos) {
      if (s + TA_AHEAD <= n) wait_loads<(TA_AHEAD - 1) * TA_LOADS>(); else wait_loads<0>();
      lds_barrier();
      flush((s + 1) & 1);
      if (s + TA_AHEAD < n) feed((s + TA_AHEAD) & (TA_RING - 1));
      const int tok = pos * TA_STEP;
      const char* buf = sm.k + (s & (TA_RING - 1)) * TA_BYTES;
      TallFrag kf[2][8];
      f32x16 acc[2];
      tall_k(kf[0], buf, lane);
      tall_k(kf[1], buf + 32 * 256, lane);
      tall_mfma<false>(acc[0], kf[0], qf[0]);
      float c[3][4];                                           // the two tiles' sums, and the shared block's
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) c[t][i] = 0.f;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u + 1 < U) {
          if (H && u + 1 == 2 * F) tall_mfma<false>(acc[(u + 1) & 1], kf[0], qf[B - 1]);
          else tall_mfma<false>(acc[(u + 1) & 1], kf[(u + 1) / F], qf[(u + 1) % F]);
        }
        if (H && u == F - 1) tall_k(kf[0], buf + (wave & 1) * 32 * 256, lane);
        const int t = u / F;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float4 b;
          if (t < 2) b = make_float4(b2[u % F][4 * i], b2[u % F][4 * i + 1], b2[u % F][4 * i + 2], b2[u % F][4 * i + 3]);
          else b = *(const float4*)(b2h + 8 * i);
          c[t][0] += fast_exp2(fmaf(acc[u & 1][4 * i], a2, -b.x));
          c[t][1] += fast_exp2(fmaf(acc[u & 1][4 * i + 1], a2, -b.y));
          c[t][2] += fast_exp2(fmaf(acc[u & 1][4 * i + 2], a2, -b.z));
          c[t][3] += fast_exp2(fmaf(acc[u & 1][4 * i + 3], a2, -b.w));
        }
        if (u + 1 < U) tall_mix();
        __builtin_amdgcn_sched_barrier(0);
      }
      float v0 = (c[0][0] + c[0][1]) + (c[0][2] + c[0][3]), v1 = (c[1][0] + c[1][1]) + (c[1][2] + c[1][3]);
      if (H) {
        const float vh = (c[2][0] + c[2][1]) + (c[2][2] + c[2][3]);
        if (wave & 1) v1 += vh; else v0 += vh;
      }
      // lanes below 32 are left with the first tile's sums over both row halves, the others with the second's
      const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v0), __float_as_uint(v1), false, false);
      sm.ps[s & 1][wave][lane] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
      dst = out + (size_t)head * N + tok;
      dst_n = min(TA_STEP, N - tok);
    }
    pos = pt.SH - 1; --head;
  }
  lds_barrier();
  flush((n - 1) & 1);
}

obf_status_t launch_score_tall(const Dims& m, const Workspace& w, double* stats_part, const void* K, const void* Q, float* part, float* scores,
                               double* row_lse, hipStream_t st) {
  const int RG = w.rgroups;
  const TallPart pt = {w.tiles_per_head, w.tiles_per_range, (long)m.heads * w.tiles_per_head, (long)m.kvs * TA_D};
  const TallPart sp = {w.stats_tiles_per_head, w.stats_tiles_per_range, (long)m.heads * w.stats_tiles_per_head, pt.kstride};
  const dim3 grid((unsigned)((w.nranges + 7) / 8 * 8 * RG));
  const int aligned = ((uintptr_t)K & 15) == 0;
  const size_t rg_stride = (size_t)m.heads * m.N;
  const bool two = w.tall_rows == 256;
  if (!w.narrow_stats) {
    ProfScope prof_(ST_SCORE_STATS, st);
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(TA_THREADS), 0, st, (const uint16_t*)K, (const uint16_t*)Q, stats_part, m.N, m.R, RG, pt, w.nslot, aligned);
    };
    if (two) go(k_score_stats_tall<2, 0>); else go(k_score_stats_tall<1, 1>);
  }
  if (check_launch("score stats (row groups of 192 or 256)") != OBF_OK) return OBF_ERR_HIP;
  { ProfScope prof_(ST_SCORE_MASS, st);
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(TA_THREADS), 0, st, (const uint16_t*)K, (const uint16_t*)Q, (const double*)stats_part, row_lse, part, scores, m.N, m.R,
                         RG, rg_stride, pt, sp, w.nslot, aligned);
    };
    if (two) go(k_score_mass_tall<2, 0>); else go(k_score_mass_tall<1, 1>); }
  return check_launch("score mass (row groups of 192 or 256)");
}

}  // namespace obf
