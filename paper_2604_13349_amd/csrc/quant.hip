// Post-hoc int8 / int4 codes for relay rows (the "+ int8" rows of App. E's comparison table).  The paper names no
// scheme; the one taken here reproduces its ratios: every row carries its own asymmetric code and two half-precision
// numbers, zero = fp16(min x), scale = fp16((max x - min x) / L), L = 2^bits - 1, q = clamp(rint((x - zero) / scale), 0, L).
// The integer decision is taken in single precision with individually rounded subtract, divide and round-to-even.
//
// Both directions are bound by memory: a lane handles 16 consecutive columns, so that a row of 128 is eight lanes and a wave moves
// eight rows (sixteen at head_dim 64); rows come and go in 16-byte pieces, the codes of a lane in one piece of 16 (int8) or 8 bytes.
// A lane of 16 columns also pays for the row's minimum, maximum, scale and zero once per 16 values.  366k rows of 128 bf16 values, int8:
// 25 us to codes and 29 back (5.4 and 4.9 TB/s; 97 and 108 us with a wave per row and a thread per value).
#include <hip/hip_fp16.h>
#include "common.hpp"

namespace obf {

constexpr int QT_THREADS = 256;
constexpr int QT_COLS = 16;              // columns per lane

// 16 consecutive elements (16-byte aligned) as floats, and back
__device__ __forceinline__ void load16(const uint16_t* __restrict__ p, float (&o)[QT_COLS]) {
  const uint4 v[2] = {((const uint4*)p)[0], ((const uint4*)p)[1]};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
    for (int k = 0; k < 4; ++k) { o[8 * i + 2 * k] = __uint_as_float(w[k] << 16); o[8 * i + 2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u); }
  }
}
__device__ __forceinline__ void load16(const float* __restrict__ p, float (&o)[QT_COLS]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) { const float4 v = ((const float4*)p)[i]; o[4 * i] = v.x; o[4 * i + 1] = v.y; o[4 * i + 2] = v.z; o[4 * i + 3] = v.w; }
}
__device__ __forceinline__ void store16(uint16_t* __restrict__ p, const float (&x)[QT_COLS]) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = (uint32_t)float_to_bf16_bits(x[8 * i + 2 * k]) | ((uint32_t)float_to_bf16_bits(x[8 * i + 2 * k + 1]) << 16);
    ((uint4*)p)[i] = make_uint4(w[0], w[1], w[2], w[3]);
  }
}
__device__ __forceinline__ void store16(float* __restrict__ p, const float (&x)[QT_COLS]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) ((float4*)p)[i] = make_float4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
}

template <typename T, int D, int BITS>
__global__ __launch_bounds__(QT_THREADS) void k_quant_rows(const T* __restrict__ X, long n_rows, uint8_t* __restrict__ codes,
                                                           uint16_t* __restrict__ scale, uint16_t* __restrict__ zero) {
  constexpr int LPR = D / QT_COLS;                             // lanes per row
  const long row = (long)blockIdx.x * (QT_THREADS / LPR) + threadIdx.x / LPR;
  const int part = threadIdx.x % LPR;
  if (row >= n_rows) return;                                   // all lanes of a row together
  float x[QT_COLS];
  load16(X + row * D + part * QT_COLS, x);
  float lo = x[0], hi = x[0];
#pragma unroll
  for (int i = 1; i < QT_COLS; ++i) { lo = fminf(lo, x[i]); hi = fmaxf(hi, x[i]); }
#pragma unroll
  for (int off = LPR / 2; off > 0; off >>= 1) { lo = fminf(lo, __shfl_xor(lo, off)); hi = fmaxf(hi, __shfl_xor(hi, off)); }
  constexpr float L = (float)((1 << BITS) - 1);
  const __half zh = __float2half_rn(lo), sh = __float2half_rn(__fdiv_rn(__fsub_rn(hi, lo), L));
  const float z = __half2float(zh), s = __half2float(sh);
  uint32_t q[QT_COLS];
  if (s > 0.f && s < INFINITY && fabsf(z) < INFINITY) {
    // The correctly rounded quotient from the row's reciprocal (Markstein): with r = RN(1/s), s of eleven significant bits, a quotient
    // within an ulp becomes the correctly rounded one by one residual step; the first step only brings it there.
    const float r = __frcp_rn(s);
#pragma unroll
    for (int i = 0; i < QT_COLS; ++i) {
      const float t = __fsub_rn(x[i], z);
      float y = __fmul_rn(t, r);
      y = __fmaf_rn(__fmaf_rn(-y, s, t), r, y);
      y = __fmaf_rn(__fmaf_rn(-y, s, t), r, y);
      q[i] = (uint32_t)fminf(fmaxf(rintf(y), 0.f), L);
    }
  } else {                                                     // a constant row, or values past the half-precision range
#pragma unroll
    for (int i = 0; i < QT_COLS; ++i)
      q[i] = (s > 0.f) ? (uint32_t)fminf(fmaxf(rintf(__fdiv_rn(__fsub_rn(x[i], z), s)), 0.f), L) : 0u;
  }
  uint32_t w[QT_COLS * BITS / 32];
#pragma unroll
  for (int k = 0; k < QT_COLS * BITS / 32; ++k) {              // little-endian: the even column of an int4 pair in the low half
    w[k] = 0u;
#pragma unroll
    for (int i = 0; i < 32 / BITS; ++i) w[k] |= q[k * (32 / BITS) + i] << (i * BITS);
  }
  uint8_t* o = codes + row * (D * BITS / 8) + part * (QT_COLS * BITS / 8);
  if constexpr (BITS == 8) *(uint4*)o = make_uint4(w[0], w[1], w[2], w[3]);
  else *(uint2*)o = make_uint2(w[0], w[1]);
  if (part == 0) { scale[row] = __half_as_ushort(sh); zero[row] = __half_as_ushort(zh); }
}

template <typename T, int D, int BITS>
__global__ __launch_bounds__(QT_THREADS) void k_dequant_rows(const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scale,
                                                             const uint16_t* __restrict__ zero, long n_rows, T* __restrict__ X) {
  constexpr int LPR = D / QT_COLS;
  const long row = (long)blockIdx.x * (QT_THREADS / LPR) + threadIdx.x / LPR;
  const int part = threadIdx.x % LPR;
  if (row >= n_rows) return;
  const uint8_t* c = codes + row * (D * BITS / 8) + part * (QT_COLS * BITS / 8);
  uint32_t w[QT_COLS * BITS / 32];
  if constexpr (BITS == 8) { const uint4 v = *(const uint4*)c; w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w; }
  else { const uint2 v = *(const uint2*)c; w[0] = v.x; w[1] = v.y; }
  const float s = __half2float(__ushort_as_half(scale[row])), z = __half2float(__ushort_as_half(zero[row]));
  float x[QT_COLS];
#pragma unroll
  for (int i = 0; i < QT_COLS; ++i) x[i] = fmaf(s, (float)((w[i * BITS / 32] >> (i * BITS % 32)) & ((1u << BITS) - 1u)), z);
  store16(X + row * D + part * QT_COLS, x);
}

// Pieces of 16 and 8 bytes need their arrays aligned so.  A caller's arrays usually are (rows of an allocation are); one that starts
// elsewhere takes the kernels below, a wave per row (codes: a thread per value) with element-sized accesses.
static bool qt_aligned(const void* X, const void* codes, int bits) { return ((uintptr_t)X & 15) == 0 && ((uintptr_t)codes & (bits == 8 ? 15 : 7)) == 0; }

// one wave per row; lane l owns columns l and l + 64
template <typename T>
__global__ __launch_bounds__(QT_THREADS) void k_quant_rows_any(const T* __restrict__ X, long n_rows, int d, int bits,
                                                               uint8_t* __restrict__ codes, uint16_t* __restrict__ scale,
                                                               uint16_t* __restrict__ zero) {
  const long row = (long)blockIdx.x * (QT_THREADS / 64) + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const int lane = threadIdx.x & 63;
  const T* x = X + row * d;
  const bool two = lane + 64 < d;
  const float a = Elem<T>::load(x + lane), b = two ? Elem<T>::load(x + lane + 64) : a;      // d is 64 or 128
  float lo = fminf(a, b), hi = fmaxf(a, b);
  for (int off = 32; off > 0; off >>= 1) { lo = fminf(lo, __shfl_xor(lo, off)); hi = fmaxf(hi, __shfl_xor(hi, off)); }
  const float L = (float)((1 << bits) - 1);
  const __half zh = __float2half_rn(lo), sh = __float2half_rn(__fdiv_rn(__fsub_rn(hi, lo), L));
  const float z = __half2float(zh), s = __half2float(sh);
  auto code = [&](float v) -> uint32_t {
    if (!(s > 0.f)) return 0u;
    const float q = rintf(__fdiv_rn(__fsub_rn(v, z), s));
    return (uint32_t)fminf(fmaxf(q, 0.f), L);
  };
  const uint32_t qa = code(a), qb = code(b);
  if (bits == 8) {
    codes[row * d + lane] = (uint8_t)qa;
    if (two) codes[row * d + lane + 64] = (uint8_t)qb;
  } else {
    // two codes per byte, the even column in the low half: lane pairs (2i, 2i + 1) meet
    const uint32_t na = __shfl_xor(qa, 1), nb = __shfl_xor(qb, 1);
    if ((lane & 1) == 0) {
      codes[row * (d / 2) + lane / 2] = (uint8_t)(qa | (na << 4));
      if (two) codes[row * (d / 2) + (lane + 64) / 2] = (uint8_t)(qb | (nb << 4));
    }
  }
  if (lane == 0) { scale[row] = __half_as_ushort(sh); zero[row] = __half_as_ushort(zh); }
}

template <typename T>
__global__ __launch_bounds__(QT_THREADS) void k_dequant_rows_any(const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scale,
                                                                 const uint16_t* __restrict__ zero, long n_rows, int d, int bits,
                                                                 T* __restrict__ X) {
  const long e = (long)blockIdx.x * QT_THREADS + threadIdx.x;
  if (e >= n_rows * d) return;
  const long row = e / d;
  const int c = (int)(e - row * d);
  const uint32_t q = (bits == 8) ? codes[e] : ((codes[row * (d / 2) + c / 2] >> ((c & 1) * 4)) & 15u);
  const float s = __half2float(__ushort_as_half(scale[row])), z = __half2float(__ushort_as_half(zero[row]));
  Elem<T>::store(X + e, fmaf(s, (float)q, z));
}

template <typename T, int D>
static void quant(const T* X, long n_rows, int bits, uint8_t* codes, uint16_t* scale, uint16_t* zero, hipStream_t st) {
  constexpr int rows = QT_THREADS * QT_COLS / D;
  const unsigned grid = (unsigned)((n_rows + rows - 1) / rows);
  if (!qt_aligned(X, codes, bits)) {
    const unsigned g1 = (unsigned)((n_rows + QT_THREADS / 64 - 1) / (QT_THREADS / 64));
    hipLaunchKernelGGL(k_quant_rows_any<T>, dim3(g1), dim3(QT_THREADS), 0, st, X, n_rows, D, bits, codes, scale, zero);
  } else if (bits == 8) hipLaunchKernelGGL((k_quant_rows<T, D, 8>), dim3(grid), dim3(QT_THREADS), 0, st, X, n_rows, codes, scale, zero);
  else hipLaunchKernelGGL((k_quant_rows<T, D, 4>), dim3(grid), dim3(QT_THREADS), 0, st, X, n_rows, codes, scale, zero);
}

template <typename T, int D>
static void dequant(const uint8_t* codes, const uint16_t* scale, const uint16_t* zero, long n_rows, int bits, T* X, hipStream_t st) {
  constexpr int rows = QT_THREADS * QT_COLS / D;
  const unsigned grid = (unsigned)((n_rows + rows - 1) / rows);
  if (!qt_aligned(X, codes, bits)) {
    const unsigned g1 = (unsigned)((n_rows * D + QT_THREADS - 1) / QT_THREADS);
    hipLaunchKernelGGL(k_dequant_rows_any<T>, dim3(g1), dim3(QT_THREADS), 0, st, codes, scale, zero, n_rows, D, bits, X);
  } else if (bits == 8) hipLaunchKernelGGL((k_dequant_rows<T, D, 8>), dim3(grid), dim3(QT_THREADS), 0, st, codes, scale, zero, n_rows, X);
  else hipLaunchKernelGGL((k_dequant_rows<T, D, 4>), dim3(grid), dim3(QT_THREADS), 0, st, codes, scale, zero, n_rows, X);
}

obf_status_t launch_quant_rows(const void* X, long n_rows, int d, int dtype, int bits, uint8_t* codes, uint16_t* scale,
                               uint16_t* zero, hipStream_t st) {
  if (n_rows == 0) return OBF_OK;
  if (dtype == OBF_BF16) {
    if (d == 128) quant<uint16_t, 128>((const uint16_t*)X, n_rows, bits, codes, scale, zero, st);
    else quant<uint16_t, 64>((const uint16_t*)X, n_rows, bits, codes, scale, zero, st);
  } else {
    if (d == 128) quant<float, 128>((const float*)X, n_rows, bits, codes, scale, zero, st);
    else quant<float, 64>((const float*)X, n_rows, bits, codes, scale, zero, st);
  }
  return check_launch("quantize rows");
}

obf_status_t launch_dequant_rows(const uint8_t* codes, const uint16_t* scale, const uint16_t* zero, long n_rows, int d, int dtype,
                                 int bits, void* X, hipStream_t st) {
  if (n_rows == 0) return OBF_OK;
  if (dtype == OBF_BF16) {
    if (d == 128) dequant<uint16_t, 128>(codes, scale, zero, n_rows, bits, (uint16_t*)X, st);
    else dequant<uint16_t, 64>(codes, scale, zero, n_rows, bits, (uint16_t*)X, st);
  } else {
    if (d == 128) dequant<float, 128>(codes, scale, zero, n_rows, bits, (float*)X, st);
    else dequant<float, 64>(codes, scale, zero, n_rows, bits, (float*)X, st);
  }
  return check_launch("dequantize rows");
}

}  // namespace obf
