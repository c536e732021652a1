// What the back-fill of a call with small budgets needs from the values, in one launch: the retained-span bases (a workgroup per head,
// keep_basis_small.hpp), the statistics of the deleted rows (a workgroup per chunk, del_stats_*.hpp) and the gathered rows themselves need
// nothing of each other when every budget is below head_dim: each head with deleted rows is then active whatever its basis is.  All of it is
// latency on few workgroups; the longest, the bases, come first in the grid.
// As three launches on two streams the bases ran beside the others too, but the fork and the join cost 7 and 11 us: 288 heads of 256 tokens, 32 kept,
// the whole call 154 -> 132 us; two fp32 heads of 512 tokens 92 -> 70; 12 short samples 1007 -> 936; 288 heads of 8192 tokens, 96 kept, 629 -> 611.
// Budgets above 96 rows stay apart: their basis kernel takes twice the registers, which would halve the waves of the statistics beside it.  fp32 at
// head_dim 128 has twice the registers here already (its statistics need them), and at 96 rows LDS for one workgroup to a compute unit; apart it is slower
// all the same: 2 heads of 300 tokens, 96 kept, 157 - 126 us, 288 of 4096 1079 - 1050, 640 of 1024 782 - 747, 288 of 8192 1931 - 1909.
#include "del_stats_generic.hpp"
#include "del_stats_mfma.hpp"
#include "gather.hpp"
#include "keep_basis_small.hpp"

namespace obf {

constexpr int BS_THREADS = KS_THREADS;
static_assert(BS_THREADS == DM_THREADS && BS_THREADS == DG_THREADS, "the parts of the grid share a workgroup size");
constexpr int BS_MAX_ROWS = 96;          // retained rows of the basis code without the wider registers

struct BsGather { const uint4 *K, *V; uint4 *K_out, *V_out; int blocks /*per head; 0: nothing is gathered*/; };

// grid: `heads` workgroups for the bases, then nstat per head for the statistics, then g.blocks per head for the gathered rows
template <typename T, int D>
__global__ __launch_bounds__(BS_THREADS, (D == 128 && sizeof(T) == 4) ? 2 : 4)
void k_bf_basis_stats(const T* __restrict__ V, const float* __restrict__ scores, const int32_t* __restrict__ idx, const int32_t* __restrict__ n_keep,
                      int N, int max_budget, int rank, int heads, int nstat, HeadState* __restrict__ state, float* __restrict__ basis,
                      float* __restrict__ gram_part, int scs, int kvs, BsGather g) {
  extern __shared__ __attribute__((aligned(16))) char bs_lds[];
  int b = blockIdx.x;
  if (b < heads) {
    KsShared& sh = *(KsShared*)bs_lds;
    ks_workgroup<T, D, false>(V, scores, idx, n_keep[b], N, max_budget, rank, state, basis, scs, kvs, b, (double*)(bs_lds + ((sizeof(KsShared) + 15) & ~15)), sh);
    return;
  }
  b -= heads;
  if (b < heads * nstat) {
    const int head = b / nstat, chunk = b - head * nstat;
    if constexpr (D == 128 && sizeof(T) == 2)
      dm_chunk(V, scores, idx, N, max_budget, nstat, state, n_keep, gram_part, scs, kvs, head, chunk, *(DmShared*)bs_lds);
    else
      dg_chunk<T, D>(V, scores, idx, N, max_budget, nstat, state, n_keep, gram_part, scs, kvs, head, chunk, *(DgShared*)bs_lds);
    return;
  }
  b -= heads * nstat;
  const int head = b / g.blocks;
  ga_rows<BS_THREADS>(g.K, g.V, idx, n_keep, kvs, D * (int)sizeof(T) / 16, max_budget, g.K_out, g.V_out, nullptr, head, b - head * g.blocks, g.blocks, nullptr);
}

bool basis_stats_supported(int32_t max_budget, int32_t rank, int d) {
  return rank > 0 && max_budget > 0 && max_budget < d && max_budget <= BS_MAX_ROWS;
}

template <typename T, int D>
static obf_status_t run(const Dims& m, const Workspace& w, char* ws, const void* K, const void* V, const float* scores, const int32_t* idx,
                        const int32_t* n_keep, int32_t max_budget, int32_t rank, void* K_out, void* V_out, hipStream_t st) {
  constexpr size_t kStats = (D == 128 && sizeof(T) == 2) ? sizeof(DmShared) : sizeof(DgShared);
  auto lds_of = [](size_t rows) { return max(kStats, ((sizeof(KsShared) + 15) & ~(size_t)15) + ks_smem<T>(rows, D)); };
  static std::mutex attr_mu;
  static uint64_t attr_seen = 0;
  once_per_device(attr_mu, attr_seen, [&] {
    (void)hipFuncSetAttribute((const void*)k_bf_basis_stats<T, D>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_of(min(BS_MAX_ROWS, D)));
  });
  BsGather g = {(const uint4*)K, (const uint4*)V, (uint4*)K_out, (uint4*)V_out, K_out ? ga_blocks<BS_THREADS>(max_budget, D * (int)sizeof(T)) : 0};
  const long blocks = (long)m.heads * (1 + w.nstat + g.blocks);
  ProfScope prof_(ST_BASIS_STATS, st);
  hipLaunchKernelGGL((k_bf_basis_stats<T, D>), dim3((unsigned)blocks), dim3(BS_THREADS), lds_of(max_budget), st, (const T*)V, scores, idx, n_keep, m.N,
                     max_budget, rank, m.heads, w.nstat, (HeadState*)(ws + w.head_state), (float*)(ws + w.basis), (float*)(ws + w.gram_part), m.scs,
                     m.kvs, g);
  return check_launch("backfill basis and statistics");
}

obf_status_t launch_basis_stats(const Dims& m, const Workspace& w, char* ws, const void* K, const void* V, const float* scores, const int32_t* idx,
                                const int32_t* n_keep, int32_t max_budget, int32_t rank, void* K_out, void* V_out, hipStream_t st) {
  auto go = m.dtype == OBF_BF16 ? (m.d == 128 ? run<uint16_t, 128> : run<uint16_t, 64>) : (m.d == 128 ? run<float, 128> : run<float, 64>);
  return go(m, w, ws, K, V, scores, idx, n_keep, max_budget, rank, K_out, V_out, st);
}

}  // namespace obf
