// Operands of the double-precision matrix instruction v_mfma_f64_16x16x4_f64 straight from rows of K or Q in memory.  An operand holds, in
// lane l, row l % 16 and one k of four, picked by l / 16; which k that is does not matter as long as both operands agree, so lane l takes
// the head_dim entries (l/16) * d/4 ..  of its row: consecutive in memory, loaded in 16-byte pieces, converted to double as they are used.
// Entry i of lane l of the result is row l/16 + 4 i, column l % 16.
#pragma once
#include "common.hpp"

namespace obf {

typedef __attribute__((__vector_size__(4 * sizeof(double)))) double f64x4;

// the head_dim entries (lane / 16) * D/4 .. of one row, as they lie in memory
template <typename T, int D>
struct RowPart {
  static constexpr int NV = D / 4 * (int)sizeof(T) / 16;     // 16-byte pieces
  uint4 v[NV];
  __device__ __forceinline__ void load(const T* __restrict__ row, int lane) {
    const T* p = row + (lane >> 4) * (D / 4);
#pragma unroll
    for (int i = 0; i < NV; ++i) __builtin_memcpy(&v[i], p + i * (16 / (int)sizeof(T)), 16);     // one load; rows need only be aligned to their elements
  }
  __device__ __forceinline__ double at(int s) const {         // entry s; s is a compile-time constant after unrolling
    if constexpr (sizeof(T) == 2) {
      const uint4& q = v[s >> 3];
      const int k = s & 7;
      const uint32_t w = (k >> 1) == 0 ? q.x : (k >> 1) == 1 ? q.y : (k >> 1) == 2 ? q.z : q.w;
      return (double)__uint_as_float((k & 1) ? (w & 0xffff0000u) : (w << 16));
    } else {
      const uint4& q = v[s >> 2];
      const int k = s & 3;
      return (double)__uint_as_float(k == 0 ? q.x : k == 1 ? q.y : k == 2 ? q.z : q.w);
    }
  }
};

}  // namespace obf
