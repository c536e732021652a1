// The last phase of the back-fill, shared by the two kernels that can finish a head (backfill.hip, backfill_lead.hip).
#pragma once
#include "common.hpp"

namespace obf {

constexpr double kRankEps = 1.1920928955078125e-07;   // 2^-23, the rank rule's epsilon
constexpr float kRcrSkip = 1.0e-6f;                   // "||R||_F negligible": ||R||^2 <= 1e-6 ||V_del||^2
constexpr float kEigFloor = 1.0e-6f;                  // resolution of the fp32 residual Gram (relative)

// Outputs of one head, shared by the two kernels that can finish it: delta, the head state, the diagnostics, and Eq. 7 on
// the retained rows.  uvec (LDS) holds delta when the head is not skipped.  NT threads, all must call.
template <typename T, int NT>
__device__ __forceinline__ void fn_emit(const int head, const int d, const int rank, HeadState st, const int skipped,
                                        const int k_used, const float rcr, const float ivn, const float pcr, const float pc,
                                        const float revr, const float fast_err, const float* uvec,
                                        HeadState* __restrict__ state,
                                        float* __restrict__ delta, float* __restrict__ delta_out, obf_diag_t* __restrict__ diag,
                                        T* __restrict__ V_out, const int max_budget, const float* __restrict__ scores,
                                        const int32_t* __restrict__ idx, const int vflags, const int scs) {
  const int tid = threadIdx.x;
  if (tid < d) {
    const float v = skipped ? 0.f : uvec[tid];
    delta[(size_t)head * d + tid] = v;
    if (delta_out) delta_out[(size_t)head * d + tid] = v;
  }
  if (tid == 0) {
    st.active = skipped ? 0 : 1;
    st.k_used = k_used; st.rcr = rcr; st.ivn = ivn;
    state[head] = st;
    if (diag) {
      obf_diag_t dg;
      dg.n_keep = st.n_keep; dg.r_keep = st.r_keep; dg.k_used = k_used; dg.skipped = skipped;
      dg.a_keep = (float)st.a_keep; dg.a_del = (float)st.a_del; dg.rcr = rcr; dg.ivn = ivn;
      // a head whose retained span is all of R^d has its deleted values entirely inside it
      dg.pcr = (rank > 0 && st.n_keep > 0 && st.n_del > 0 && st.r_keep >= d) ? 1.f : pcr;
      dg.pc = pc; dg.revr = revr;
      dg.dr = (float)(st.a_del / (st.a_keep + kEps));
      dg.fast_err = fast_err;
      dg.select_flags = 0;                                     // the fused call fills it in afterwards
      diag[head] = dg;
    }
  }
  // Eq. 7: the one offset is added to every retained value row (rounded once to the storage type); under Attn-inject
  // (App. D) row t receives n_keep A_t / (a_keep + eps) times the offset instead
  if (!skipped && V_out) {
    const int total = st.n_keep * d;
    T* base = V_out + (size_t)head * max_budget * d;
    if (vflags & VF_ATTN_INJECT) {
      const float per_mass = (float)((double)st.n_keep / (st.a_keep + kEps));
      const float* sc = scores + (size_t)head * scs;
      const int32_t* id = idx + (size_t)head * max_budget;
      for (int e = tid; e < total; e += NT) {
        T* p = base + e;
        Elem<T>::store(p, fmaf(per_mass * sc[id[e / d]], uvec[e % d], Elem<T>::load(p)));
      }
    } else {
      // 16 bytes a thread and four of them in flight where the rows allow it (d elements are whole pieces): 96 rows of 256 bytes take
      // 5000 cycles, 12700 one element at a time
      constexpr int W = 16 / (int)sizeof(T);
      int e = 0;
      if (((uintptr_t)base & 15) == 0) {
        const int pieces = total / W;
        const float* u = uvec + (tid * W) % d;                 // NT pieces are whole rows: the same columns every time
        for (int p0 = tid; p0 < pieces; p0 += 4 * NT) {
          uint4 x[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) if (p0 + c * NT < pieces) x[c] = *(const uint4*)(base + (size_t)(p0 + c * NT) * W);
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            if (p0 + c * NT < pieces) {
              T v[W];
              __builtin_memcpy(v, &x[c], 16);
#pragma unroll
              for (int i = 0; i < W; ++i) Elem<T>::store(&v[i], Elem<T>::load(&v[i]) + u[i]);
              __builtin_memcpy(&x[c], v, 16);
              *(uint4*)(base + (size_t)(p0 + c * NT) * W) = x[c];
            }
          }
        }
        e = pieces * W;
      }
      for (e += tid; e < total; e += NT) {
        T* p = base + e;
        Elem<T>::store(p, Elem<T>::load(p) + uvec[e % d]);
      }
    }
  }
}

}  // namespace obf
