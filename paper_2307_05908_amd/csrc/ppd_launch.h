// Launchers of the two big kernel families.  Their template instances are compiled in separate
// translation units (ppd_inst.hip with -DPPD_INST=n) so that the library builds in parallel.
#pragma once
#include "ppd_kernels.h"

namespace ppd {

template <typename WT, bool PAIRED, int WR>
hipError_t launch_gemm_t(hipStream_t stream, const GemmArgs& a, int MA, int MB, dim3 grid, size_t lds);

// gemm_small_kernel, where it applies: fp32 weights, K <= GEMM_SMALL_K, and every output has a wave's turn of its own (up to
// GEMM_SMALL_ROWS outputs; of a head launch, one set per wave of its grid).  Measured over the rule (launches of one and k rows with
// the event pair around them, gemm_kernel / this one, us): 256 columns to 4096 outputs, k = 1 13.4 / 6.7, k = 8 38.1 / 10.6;
// 1024 columns to 1024 outputs 9.7 / 6.2 and 15.5 / 8.4, to 3072 15.5 / 9.3 and 40.0 / 20.5, to 4096 17.1 / 10.7 and 44.7 / 24.5, to 4096
// pairs 21.9 / 15.0 and 50.6 / 28.2; 64 rows of a prompt on the 1024-wide model of 8 layers 8.1 / 4.5 ms.
inline bool gemm_small_fits(const GemmArgs& a, int head_grid) {
  return a.K <= GEMM_SMALL_K && (a.topk > 0 ? (int64_t)a.ntot <= (int64_t)head_grid * GEMM_WAVES * 4 : a.ntot <= GEMM_SMALL_ROWS);
}
hipError_t launch_gemm_small(hipStream_t stream, const GemmArgs& a, int ngroups, bool paired, int head_grid);

template <int HD>
hipError_t launch_attn_t(hipStream_t stream, const AttnArgs& a, int mmax, dim3 grid, bool causal);
// attn_whole_kernel; mmax: the largest row count of the groups, pmax: the largest position any row may sit at
template <int HD>
hipError_t launch_attn_whole(hipStream_t stream, const AttnWholeArgs& w, int mmax, int ngroups, int pmax);

// Workgroups per group for a GEMM with `nsets` row sets (gemm_kernel): each workgroup has four waves and
// every wave takes ceil(nsets / waves) sets, so pick the count in [gmax/2, gmax] that wastes the fewest
// wave slots (ties: the larger grid).
inline int pick_grid(int nsets, int gmax) {
  int need = (nsets + GEMM_WAVES - 1) / GEMM_WAVES;
  if (need <= gmax) return need < 1 ? 1 : need;
  int best = gmax; double best_eff = 0.0;
  for (int g = gmax; g >= gmax / 2 && g >= 1; --g) {
    int nw = g * GEMM_WAVES, nit = (nsets + nw - 1) / nw;
    double eff = (double)nsets / ((double)nit * nw);
    if (eff > best_eff + 1e-9) { best_eff = eff; best = g; }
  }
  return best;
}

// LM-head launch of gemm_kernel (one row, four weight rows per wave): as many workgroups as a plain GEMM,
// more if a workgroup would otherwise produce over HEAD_MAX_ROWS logits
inline int head_grid_valu(int vocab, int gmax) {
  const int nsets = (vocab + 3) / 4;
  int g = pick_grid(nsets, gmax);
  const int sets_per_wg_cap = HEAD_MAX_ROWS / 4;               // per workgroup, all four waves together
  while (((nsets + g * GEMM_WAVES - 1) / (g * GEMM_WAVES)) * GEMM_WAVES > sets_per_wg_cap) ++g;
  return g;
}

// hipError_t of the last failing HIP call made outside any context (ppd_last_hip_error(NULL) reports it)
void set_global_hip_error(int e);

}  // namespace ppd
