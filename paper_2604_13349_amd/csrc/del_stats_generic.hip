// The statistics of the deleted rows as a launch of their own (fp32 caches and head_dim 64).
#include "del_stats_generic.hpp"

namespace obf {

template <typename T, int D>
__global__ __launch_bounds__(DG_THREADS, 2) void k_bf_del_stats(const T* __restrict__ V, const float* __restrict__ scores,
                                                                const int32_t* __restrict__ idx, int N, int max_budget, int nstat,
                                                                const HeadState* __restrict__ state,
                                                                const int32_t* __restrict__ n_keep /*non-null: do not read the head states*/,
                                                                float* __restrict__ gram_part, int scs, int kvs) {
  __shared__ DgShared sh;
  dg_chunk<T, D>(V, scores, idx, N, max_budget, nstat, state, n_keep, gram_part, scs, kvs, blockIdx.y, blockIdx.x, sh);
}

template <typename T, int D>
static void launch(const Dims& m, const Workspace& w, const void* V, const float* scores, const int32_t* idx, int32_t max_budget,
                   const HeadState* state, const int32_t* n_keep, float* gram_part, hipStream_t st) {
  ProfScope prof_(ST_DEL_STATS, st);
  hipLaunchKernelGGL((k_bf_del_stats<T, D>), dim3(w.nstat, m.heads), dim3(DG_THREADS), 0, st, (const T*)V, scores, idx, m.N,
                     max_budget, w.nstat, state, n_keep, gram_part, m.scs, m.kvs);
}

obf_status_t launch_del_stats_generic(const Dims& m, const Workspace& w, const void* V, const float* scores, const int32_t* idx,
                                      int32_t max_budget, const HeadState* state, const int32_t* n_keep, float* gram_part,
                                      hipStream_t st) {
  // (bf16 caches of head_dim 128 are del_stats_mfma.hip's)
  if (m.dtype == OBF_BF16) launch<uint16_t, 64>(m, w, V, scores, idx, max_budget, state, n_keep, gram_part, st);
  else if (m.d == 64) launch<float, 64>(m, w, V, scores, idx, max_budget, state, n_keep, gram_part, st);
  else launch<float, 128>(m, w, V, scores, idx, max_budget, state, n_keep, gram_part, st);
  return check_launch("backfill del_stats");
}

}  // namespace obf
