// One slice of the kernel template instances, selected by -DPPD_INST=n (see build.py).
#include "ppd_launch.h"

namespace ppd {

#if PPD_INST == 7
template <int NB>
static hipError_t launch_gemm_small_t(hipStream_t stream, const GemmArgs& a, int mmax, bool paired, dim3 grid) {
#define GO(mt, lr) do { if (paired) hipLaunchKernelGGL((gemm_small_kernel<mt, NB, true, 1>), grid, dim3(GEMM_THREADS), 0, stream, a); \
    else hipLaunchKernelGGL((gemm_small_kernel<mt, NB, false, lr>), grid, dim3(GEMM_THREADS), 0, stream, a); } while (0)
  if (a.topk > 0) GO(1, 4);
  else if (mmax == 1) GO(1, 1);
  else if (mmax <= 4) GO(4, 1);
  else GO(8, 1);
#undef GO
  return hipGetLastError();
}

hipError_t launch_gemm_small(hipStream_t stream, const GemmArgs& a, int ngroups, bool paired, int head_grid) {
  int mmax = a.g[0].M;
  if (ngroups == 2 && a.g[1].M > mmax) mmax = a.g[1].M;
  if (!gemm_small_fits(a, head_grid) || mmax < 1 || ngroups < 1 || ngroups > 2 || mmax > (ngroups == 1 ? 65535 * MAXM : MAXM)) return hipErrorInvalidValue;
  if (a.topk > 0 && (ngroups != 1 || mmax != 1 || paired || head_grid > a.ntot)) return hipErrorInvalidValue;
  const dim3 grid(a.topk > 0 ? head_grid : (a.ntot + GEMM_WAVES - 1) / GEMM_WAVES, ngroups, (mmax + MAXM - 1) / MAXM);
  if (a.K <= 256) return launch_gemm_small_t<1>(stream, a, mmax, paired, grid);
  if (a.K <= 512) return launch_gemm_small_t<2>(stream, a, mmax, paired, grid);
  return launch_gemm_small_t<4>(stream, a, mmax, paired, grid);
}
#elif PPD_INST < 4 || PPD_INST == 6
// Whether one row's gains are requested with the row (bf16: rows of more than 5120 elements, the others are early_kernel's).  It puts the
// weights off, which pays where a wave streams several sets of rows.  Measured (early prediction over bf16 weights, last / first, us, RMSNorm and
// LayerNorm): 8192 elements 32000 logits 108.1 / 108.6 and 111.0 / 109.9, 12000 56.8 / 56.7 and 58.4 / 58.2, 5065 36.5 / 37.5 and 38.4 / 39.2, 1000
// 22.4 / 23.1 and 24.6 / 24.7; 7168 elements 32000 84.9 / 85.6 and 87.1 / 86.4, 1000 21.0 / 21.8 and 23.0 / 23.3; 6144 elements 32000 77.3 / 77.4
// and 78.6 / 78.6, 12000 43.9 / 44.8 and 45.5 / 45.8; 5128 elements 32000 71.5 / 71.4 and 72.7 / 73.0, 5065 28.9 / 29.4 and 30.8 / 31.2.
// fp32 weights: first everywhere (a plain token of a 3072-wide model 654 / 641 us, 1000 to 50000 logits within 1 %).
inline bool gains_first(const GemmArgs& a, unsigned grid) { return a.ntot > 2 * 4 * GEMM_WAVES * (int)grid; }
// MA rows in group 0; MB rows in group 1 (0: single-group launch).  Launch shapes in use:
// (1, 0) main token alone, (k, 0) the candidates alone, (1, k) both in one launch; bf16 weights: (1, 0).
template <typename WT, bool PAIRED, int WR>
hipError_t launch_gemm_t(hipStream_t stream, const GemmArgs& a, int MA, int MB, dim3 grid, size_t lds) {
#define GO(ma, mb) hipLaunchKernelGGL((gemm_kernel<WT, ma, mb, PAIRED, WR>), grid, dim3(GEMM_THREADS), lds, stream, a)
  if constexpr (sizeof(WT) == 2) {
    if (MA != 1 || MB != 0) return hipErrorInvalidValue;
    if (gains_first(a, grid.x)) GO(1, 0);
    else hipLaunchKernelGGL((gemm_kernel<WT, 1, 0, PAIRED, WR, false>), grid, dim3(GEMM_THREADS), lds, stream, a);
  } else if (MB == 0) {
    switch (MA) {
      case 1: GO(1, 0); break; case 2: GO(2, 0); break; case 3: GO(3, 0); break; case 4: GO(4, 0); break;
      case 5: GO(5, 0); break; case 6: GO(6, 0); break; case 7: GO(7, 0); break; case 8: GO(8, 0); break;
      default: return hipErrorInvalidValue;
    }
  } else {
    if (MA != 1) return hipErrorInvalidValue;
    switch (MB) {
      case 1: GO(1, 1); break; case 2: GO(1, 2); break; case 3: GO(1, 3); break; case 4: GO(1, 4); break;
      case 5: GO(1, 5); break; case 6: GO(1, 6); break; case 7: GO(1, 7); break; case 8: GO(1, 8); break;
      default: return hipErrorInvalidValue;
    }
  }
#undef GO
  return hipGetLastError();
}


// (fp32 weights, and one instance for row-major bf16: inside a context bf16 models run every GEMM on the MFMA kernel)
#if PPD_INST == 0
template hipError_t launch_gemm_t<float, false, 4>(hipStream_t, const GemmArgs&, int, int, dim3, size_t);
#elif PPD_INST == 1
template hipError_t launch_gemm_t<float, true, 4>(hipStream_t, const GemmArgs&, int, int, dim3, size_t);
#elif PPD_INST == 2
template hipError_t launch_gemm_t<float, false, 2>(hipStream_t, const GemmArgs&, int, int, dim3, size_t);
#elif PPD_INST == 3
template hipError_t launch_gemm_t<float, true, 2>(hipStream_t, const GemmArgs&, int, int, dim3, size_t);
#elif PPD_INST == 6
// bf16 weights as the caller holds them (row-major, not repacked): the stand-alone early prediction
template hipError_t launch_gemm_t<bf16_t, false, 4>(hipStream_t, const GemmArgs&, int, int, dim3, size_t);
#endif
#else
// mmax: the largest row count of the launch's groups (sizes LDS); causal: the prompt-chunk instance
template <int HD>
hipError_t launch_attn_t(hipStream_t stream, const AttnArgs& a, int mmax, dim3 grid, bool causal) {
  if (mmax < 1 || mmax > 16) return hipErrorInvalidValue;
  const size_t lds = sizeof(float) * (size_t)attn_lds_floats<HD>(mmax);
  static_assert(sizeof(float) * attn_lds_floats<HD>(16) <= 64 * 1024, "16 rows fit the default dynamic LDS limit");
  if (lds > 64 * 1024) return hipErrorInvalidValue;
  if (causal) attn_kernel<HD, true><<<grid, dim3(ATT_THREADS), lds, stream>>>(a);
  else attn_kernel<HD, false><<<grid, dim3(ATT_THREADS), lds, stream>>>(a);
  return hipGetLastError();
}

template <int HD>
hipError_t launch_attn_whole(hipStream_t stream, const AttnWholeArgs& w, int mmax, int ngroups, int pmax) {
  static_assert(sizeof(float) * attn_whole_lds_floats<HD>(MAXM) <= 64 * 1024, "MAXM rows fit the default dynamic LDS limit");
  if (mmax < 1 || mmax > MAXM || pmax >= ATT_WHOLE * ATT_CHUNK) return hipErrorInvalidValue;
  attn_whole_kernel<HD><<<dim3(w.a.H, ngroups), dim3(ATT_WHOLE_THREADS), sizeof(float) * (size_t)attn_whole_lds_floats<HD>(mmax), stream>>>(w);
  return hipGetLastError();
}

#if PPD_INST == 4
template hipError_t launch_attn_t<128>(hipStream_t, const AttnArgs&, int, dim3, bool);
template hipError_t launch_attn_whole<128>(hipStream_t, const AttnWholeArgs&, int, int, int);
#elif PPD_INST == 5
template hipError_t launch_attn_t<64>(hipStream_t, const AttnArgs&, int, dim3, bool);
template hipError_t launch_attn_whole<64>(hipStream_t, const AttnWholeArgs&, int, int, int);
#endif
#endif

}  // namespace ppd
