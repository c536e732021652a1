// The bases as launches of their own (heads with more than head_dim rows are left untouched): calls with budgets above what basis_stats.hip takes.
#include "keep_basis_small.hpp"

namespace obf {

template <typename T, int D, bool BIG>
__global__ __launch_bounds__(KS_THREADS, BIG ? 2 : 4) void k_bf_keep_basis_small(const T* __restrict__ V, const float* __restrict__ scores,
                                                                    const int32_t* __restrict__ idx,
                                                                    const int32_t* __restrict__ n_keep, int N,
                                                                    int max_budget, int rank, HeadState* __restrict__ state,
                                                                    float* __restrict__ basis, int scs, int kvs) {
  const int head = blockIdx.x;
  const int n = n_keep[head];
  if (n > D) return;                         // heads of the general kernel
  if ((n > 96) != BIG) return;               // n > 96: larger LDS buffer and register budget, a launch of its own
  extern __shared__ double Cs[];             // the rows and C's tiles, or the single-precision copy of C
  __shared__ KsShared sh;
  ks_workgroup<T, D, BIG>(V, scores, idx, n, N, max_budget, rank, state, basis, scs, kvs, head, Cs, sh);
}

template <typename T, int D>
static obf_status_t run_small(const Dims& m, const void* V, const float* scores, const int32_t* idx,
                              const int32_t* n_keep, int32_t max_budget, int32_t rank, HeadState* state, float* basis,
                              hipStream_t st) {
  static std::mutex attr_mu;
  static uint64_t attr_seen = 0;
  once_per_device(attr_mu, attr_seen, [] {
    (void)hipFuncSetAttribute((const void*)k_bf_keep_basis_small<T, D, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)ks_smem<T>(min(96, D), D));
    (void)hipFuncSetAttribute((const void*)k_bf_keep_basis_small<T, D, D == 128>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)ks_smem<T>(D, D));
  });
  const size_t nmax = (size_t)min(max_budget, D);
  hipLaunchKernelGGL((k_bf_keep_basis_small<T, D, false>), dim3(m.heads), dim3(KS_THREADS), ks_smem<T>(min(nmax, (size_t)96), D), st,
                     (const T*)V, scores, idx, n_keep, m.N, max_budget, rank, state, basis, m.scs, m.kvs);
  if (check_launch("backfill keep_basis_small") != OBF_OK) return OBF_ERR_HIP;
  if (nmax > 96) {                                             // (head_dim 128)
    hipLaunchKernelGGL((k_bf_keep_basis_small<T, D, D == 128>), dim3(m.heads), dim3(KS_THREADS), ks_smem<T>(nmax, D), st,
                       (const T*)V, scores, idx, n_keep, m.N, max_budget, rank, state, basis, m.scs, m.kvs);
    if (check_launch("backfill keep_basis_small (wide)") != OBF_OK) return OBF_ERR_HIP;
  }
  return OBF_OK;
}

obf_status_t launch_keep_basis_small(const Dims& m, const void* V, const float* scores, const int32_t* idx,
                                     const int32_t* n_keep, int32_t max_budget, int32_t rank, HeadState* state,
                                     float* basis, hipStream_t st) {
  auto run = m.dtype == OBF_BF16 ? (m.d == 128 ? run_small<uint16_t, 128> : run_small<uint16_t, 64>)
                                 : (m.d == 128 ? run_small<float, 128> : run_small<float, 64>);
  return run(m, V, scores, idx, n_keep, max_budget, rank, state, basis, st);
}

}  // namespace obf
