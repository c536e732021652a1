// Leading eigenpairs of a symmetric positive semi-definite D x D matrix of which each wave holds sixteen rows in registers:
// the building blocks of the block iteration in backfill_lead.hip.
//
// Everything small is a 16 x 16 matrix in the layout in which v_mfma_f32_16x16x4_f32 leaves its result: lane l = 16 q + j of a wave
// holds entries (4 q + e, j), e = 0 .. 3.  Used as operands, two such matrices S and T give S^T T in four instructions (the lane
// that owns column j of an operand supplies rows 4 q + e, for either operand), so no transposition is ever needed in here.
#pragma once
#include "common.hpp"
#include "wave_ops.hpp"

namespace obf {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;

// A single-precision value as the sum of three bf16 parts (what is left is at most 2^-27 of it): products of two such sums without the
// three terms below 2^-26, accumulated in single precision, err less than single-precision products do, and six bf16 matrix
// instructions take 96 cycles where the eight in single precision take 256.
struct Split { bf16x4 hi, mid, lo; };
__device__ __forceinline__ Split split3(const f32x4 v) {
  auto rest = [](const f32x4 x, const bf16x4 h) -> f32x4 {      // x - h, exact
    const uint2 u = __builtin_bit_cast(uint2, h);
    return f32x4{x[0] - __uint_as_float(u.x << 16), x[1] - __uint_as_float(u.x & 0xffff0000u),
                 x[2] - __uint_as_float(u.y << 16), x[3] - __uint_as_float(u.y & 0xffff0000u)};
  };
  const bf16x4 hi = __builtin_convertvector(v, bf16x4);        // to the nearest, one instruction for two
  const f32x4 r = rest(v, hi);
  const bf16x4 mid = __builtin_convertvector(r, bf16x4);
  return Split{hi, mid, __builtin_convertvector(rest(r, mid), bf16x4)};
}
__device__ __forceinline__ bf16x8 join(const bf16x4 a, const bf16x4 b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }

// An operand of v_mfma_f32_16x16x32_bf16 in three parts: lane 16 q + j holds rows 4 q .. 4 q + 3 of two 16-row tiles of column j, for
// either operand (any assignment of rows to the instruction's places does, as long as both operands share it).
struct Split8 { bf16x8 hi, mid, lo; };
__device__ __forceinline__ Split8 split8(const f32x4 a, const f32x4 b) {
  const Split x = split3(a), y = split3(b);
  return Split8{join(x.hi, y.hi), join(x.mid, y.mid), join(x.lo, y.lo)};
}
__device__ __forceinline__ float whole(const Split8& s, const int i) { return (float)s.hi[i] + ((float)s.mid[i] + (float)s.lo[i]); }
__device__ __forceinline__ f32x4 mfma32(const bf16x8 a, const bf16x8 b, const f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// One DPP move in which every lane has a source (no value to keep, so that the compiler may fold the move into the instruction that uses it).
template <int CTRL>
__device__ __forceinline__ float row_move(const float v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), CTRL, 0xF, 0xF, true));
}

// value of lane K of each 16-lane row, in every lane of the row
template <int K>
__device__ __forceinline__ float row_bcast(const float v) { return row_move<0x150 + K>(v); }

// value of lane j ^ X of the same 16-lane row
template <int X>
__device__ __forceinline__ float row_xor(const float v) {
  if constexpr (X == 1) return row_move<0xB1>(v);
  else if constexpr (X == 2) return row_move<0x4E>(v);
  else if constexpr (X == 3) return row_move<0x1B>(v);
  else if constexpr (X == 7) return row_move<0x141>(v);
  else if constexpr (X == 8) return row_move<0x128>(v);
  else if constexpr (X == 15) return row_move<0x140>(v);
  else if constexpr (X < 8) return row_xor<X ^ 7>(row_xor<7>(v));
  else if constexpr (X < 12) return row_xor<X ^ 8>(row_xor<8>(v));
  else return row_xor<X ^ 15>(row_xor<15>(v));
}

// the value that the 16-lane row R holds at the same place, in all four rows
template <int R>
__device__ __forceinline__ float from_row(const float v) {
  const uint32_t u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);     // rows 0, 0, 2, 2 and 1, 1, 3, 3
  const auto b = __builtin_amdgcn_permlane32_swap(a[R & 1], a[R & 1], false, false);
  return __uint_as_float(b[R >> 1]);
}

// sum over the four 16-lane rows, in all of them
__device__ __forceinline__ float sum_rows(const float v) {
  const uint32_t u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const uint32_t s = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(s, s, false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

__device__ __forceinline__ f32x4 mul_t(const f32x4 S, const f32x4 T, f32x4 acc) {      // acc + S^T T
#pragma unroll
  for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(S[e], T[e], acc, 0, 0, 0);
  return acc;
}

// One step of the column elimination of M (symmetric, unit diagonal): N collects the column operations, so that N^T M N = I at the end.
// A column whose pivot has fallen to `drop` depends on those before it and is dropped (zero in N).
template <int K, int P>
__device__ __forceinline__ void eliminate(f32x4& M, f32x4& N, float& sc, const int j, const float drop) {
  if constexpr (K < P) {
    const float row = from_row<(K >> 2)>(M[K & 3]);            // M[K][j]
    const float p = row_bcast<K>(row);
    const bool ok = p > drop;
    float ip = __builtin_amdgcn_rcpf(p);
    ip = fmaf(fmaf(-p, ip, 1.f), ip, ip);
    const float f = (ok && j > K) ? -row * ip : 0.f;
    if (j == K) sc = ok ? __builtin_amdgcn_rsqf(p) : 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      M[e] = fmaf(row_bcast<K>(M[e]), f, M[e]);
      N[e] = fmaf(row_bcast<K>(N[e]), f, N[e]);
    }
    eliminate<K + 1, P>(M, N, sc, j, drop);
  }
}

// One set of the one-sided Jacobi iteration: column j against column j ^ X, all pairs at once.  far: some pair's cosine exceeded tol.
template <int X>
__device__ __forceinline__ void rotate_set(f32x4& A, f32x4& S, float& n, bool& far, const int j, const float tol2) {
  constexpr int top = X >= 8 ? 8 : X >= 4 ? 4 : X >= 2 ? 2 : 1;
  const bool lo = (j & top) == 0;
  f32x4 a, s;
#pragma unroll
  for (int e = 0; e < 4; ++e) { a[e] = row_xor<X>(A[e]); s[e] = row_xor<X>(S[e]); }
  const float g = sum_rows(fmaf(A[0], a[0], A[1] * a[1]) + fmaf(A[2], a[2], A[3] * a[3]));
  const float np = row_xor<X>(n);
  far |= g * g > tol2 * (n * np);
  const float d = lo ? np - n : n - np;                        // second norm less first
  // cos 2 phi = |d| / h, sin 2 phi = 2 g / h, h^2 = d^2 + 4 g^2: one-ulp reciprocal roots do, the columns lose their unit length by as much
  // and get it back
  const float g2 = g + g, hh = fmaf(g2, g2, d * d);
  const bool turn = hh > 1e-36f;                               // (the reciprocal root of a denormal is infinite)
  const float rh = __builtin_amdgcn_rsqf(hh);
  const float c2 = turn ? fmaf(0.5f * fabsf(d), rh, 0.5f) : 1.f, rc = __builtin_amdgcn_rsqf(c2);
  const float c = c2 * rc, sg = turn ? (d < 0.f ? -g : g) * rh * rc : 0.f;        // sin phi, with the sign of g d
  const float sn = lo ? -sg : sg;
#pragma unroll
  for (int e = 0; e < 4; ++e) { A[e] = fmaf(sn, a[e], c * A[e]); S[e] = fmaf(sn, s[e], c * S[e]); }
  n = fmaxf(fmaf(sn * rc, g, n), 0.f);                         // n -+ t g, t = tan phi
}

// The columns in another order: each lane takes column `from` of its row.
__device__ __forceinline__ void reorder(f32x4& A, f32x4& S, float& n, const int from) {
  const int at = ((threadIdx.x & 48) | from) << 2;
  auto take = [&](const float v) -> float { return __uint_as_float((uint32_t)__builtin_amdgcn_ds_bpermute(at, (int)__float_as_uint(v))); };
#pragma unroll
  for (int e = 0; e < 4; ++e) { A[e] = take(A[e]); S[e] = take(S[e]); }
  n = take(n);
}

// A sweep: every pair of the P columns once.  For sixteen columns the exchanges that take one DPP move are those with j ^ 1, 2, 3, 7, 8 and
// 15; the other nine exchanges become such in two other orders of the columns, linear over GF(2): the unit vectors go to 4, 9, 8, 11,
// which turns 1, 2, 3 into 4, 9, 13 and 7, 8, 15 into 5, 11, 14, and then to 6, 10, 1, 2, which turns 1, 2, 3 into 6, 10, 12 (the second
// order's places are given in the first's).  Nothing depends on which column is where.
template <int P>
__device__ __forceinline__ void sweep(f32x4& A, f32x4& S, float& n, bool& far, const int j, const float tol2) {
  rotate_set<1>(A, S, n, far, j, tol2);
  rotate_set<2>(A, S, n, far, j, tol2);
  rotate_set<3>(A, S, n, far, j, tol2);
  rotate_set<7>(A, S, n, far, j, tol2);
  if constexpr (P == 8) {
    rotate_set<4>(A, S, n, far, j, tol2);
    rotate_set<5>(A, S, n, far, j, tol2);
    rotate_set<6>(A, S, n, far, j, tol2);
  } else {
    rotate_set<8>(A, S, n, far, j, tol2);
    rotate_set<15>(A, S, n, far, j, tol2);
    auto image = [&](const int e0, const int e1, const int e2, const int e3) -> int {
      return ((j & 1) ? e0 : 0) ^ ((j & 2) ? e1 : 0) ^ ((j & 4) ? e2 : 0) ^ ((j & 8) ? e3 : 0);
    };
    reorder(A, S, n, image(4, 9, 8, 11));
    rotate_set<1>(A, S, n, far, j, tol2);
    rotate_set<2>(A, S, n, far, j, tol2);
    rotate_set<3>(A, S, n, far, j, tol2);
    rotate_set<7>(A, S, n, far, j, tol2);
    rotate_set<8>(A, S, n, far, j, tol2);
    rotate_set<15>(A, S, n, far, j, tol2);
    reorder(A, S, n, image(11, 14, 6, 10));
    rotate_set<1>(A, S, n, far, j, tol2);
    rotate_set<2>(A, S, n, far, j, tol2);
    rotate_set<3>(A, S, n, far, j, tol2);
  }
}

// number of columns that come before column j in descending order of n (ties by index)
template <int K, int P>
__device__ __forceinline__ int rank_of(const float n, const int j) {
  if constexpr (K < P) {
    const float o = row_bcast<K>(n);
    return ((o > n || (o == n && K < j)) ? 1 : 0) + rank_of<K + 1, P>(n, j);
  } else return 0;
}

// One wave: the Ritz problem of a block X of P columns (P = 8 or 16; columns past P zero) from M = X^T X and H = X^T G X.  Leaves S with
// X S orthonormal and its columns the Ritz vectors (not yet in order), theta the Ritz value of the lane's column and `place` its rank in
// descending order.  The columns of H' = N^T H N are made orthogonal by plane rotations (H' V = U diag(theta) then); a sweep in
// which no pair's cosine exceeded tol is the last, `sweeps` at most.
template <int P>
__device__ __forceinline__ void small_ritz(f32x4 M, const f32x4 H, const float drop, const float tol, const int sweeps, f32x4& S,
                                           float& theta, int& place) {
  const int lane = threadIdx.x & 63, q = lane >> 4, j = lane & 15;
  const float own = (q != (j >> 2)) ? 0.f : (j & 2) ? ((j & 1) ? M[3] : M[2]) : ((j & 1) ? M[1] : M[0]);
  const float diag = sum_rows(own);                            // M[j][j]
  const float s = (diag > 0.f) ? __builtin_amdgcn_rsqf(diag) : 0.f;
  f32x4 N;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    M[e] *= s * __shfl(s, 4 * q + e);
    N[e] = (j == 4 * q + e) ? s : 0.f;
  }
  float sc = 0.f;
  eliminate<0, P>(M, N, sc, j, drop);
#pragma unroll
  for (int e = 0; e < 4; ++e) N[e] *= sc;
  f32x4 A = {0.f, 0.f, 0.f, 0.f};
  A = mul_t(H, N, A);
  A = mul_t(N, A, f32x4{0.f, 0.f, 0.f, 0.f});
  S = N;
  float n = 0.f;
  for (int w = 0; w < sweeps; ++w) {
    n = sum_rows(fmaf(A[0], A[0], A[1] * A[1]) + fmaf(A[2], A[2], A[3] * A[3]));
    bool far = false;
    sweep<P>(A, S, n, far, j, tol * tol);
    if (!__any(far)) break;
  }
  n = sum_rows(fmaf(A[0], A[0], A[1] * A[1]) + fmaf(A[2], A[2], A[3] * A[3]));
  theta = __builtin_amdgcn_sqrtf(n);
  place = (j < P) ? rank_of<0, P>(n, j) : j;
}

}  // namespace obf
