// Kernel instances and launchers of the compute-bound prompt pass (ppd_prefill.h).
#define PPD_PREFILL_TU 1
#include "ppd_prefill.h"


namespace ppd {

hipError_t launch_pack_rows(hipStream_t stream, const PackArgs& a) {
  if (a.M < 1 || a.K < 8 || (a.K & 7) || (a.ld & 3) || a.MT < (a.M + 15) / 16 || a.KT != (a.K + 31) / 32) return hipErrorInvalidValue;
  hipLaunchKernelGGL(pack_rows_kernel, dim3((a.MT + 7) / 8 * 128), dim3(MG_THREADS), 0, stream, a);
  return hipGetLastError();
}

template <bool PAIRED, int TN, int TMB>
static hipError_t launch_pgemm_t(hipStream_t stream, PGemmArgs a) {
  a.MB = (a.MT + TMB - 1) / TMB;
  a.NB = (a.NT + PG_WAVES * TN - 1) / (PG_WAVES * TN);
  a.GM = a.MB < PG_GROUP_M ? a.MB : PG_GROUP_M;
  a.GQ = PG_GROUP_Q;
  a.MBG = (a.MB + a.GM - 1) / a.GM;
  const int nbq = (a.NB + 7) / 8;
  const dim3 grid(8 * ((nbq + a.GQ - 1) / a.GQ) * a.GQ * a.MBG * a.GM);
  hipLaunchKernelGGL((pgemm_kernel<PAIRED, TN, TMB>), grid, dim3(PG_THREADS), (size_t)PG_R * PG_STAGE_BLKS * 1024, stream, a);
  return hipGetLastError();
}

hipError_t launch_pgemm(hipStream_t stream, PGemmArgs a, bool paired) {
  if (a.M < 1 || a.MT != (a.M + 15) / 16 || a.KT < 1 || a.NT < 1) return hipErrorInvalidValue;
  // narrow matrices take two blocks per wave so that the grid still fills the machine
  const int mb = (a.MT + 3) / 4;
  const int tn = ((a.NT + PG_WAVES * 4 - 1) / (PG_WAVES * 4)) * mb >= 384 ? 4 : 2;
  if (paired) return tn == 4 ? launch_pgemm_t<true, 4, 4>(stream, a) : launch_pgemm_t<true, 2, 4>(stream, a);
  return tn == 4 ? launch_pgemm_t<false, 4, 4>(stream, a) : launch_pgemm_t<false, 2, 4>(stream, a);
}

template <bool PAIRED, int TT>
static hipError_t launch_rgemm_t(hipStream_t stream, const RGemmArgs& a, int grid) {
  const size_t lds = (size_t)a.tiles_wg * MG_WAVES * 16 * 16 * sizeof(float) * (a.M > 16 ? 2 : 1);
  if (a.M > 16) hipLaunchKernelGGL((rgemm_kernel<PAIRED, TT, 2>), dim3(grid), dim3(MG_THREADS), lds, stream, a);
  else hipLaunchKernelGGL((rgemm_kernel<PAIRED, TT, 1>), dim3(grid), dim3(MG_THREADS), lds, stream, a);
  return hipGetLastError();
}

hipError_t launch_rgemm(hipStream_t stream, RGemmArgs a, bool paired) {
  if (a.M < 1 || a.M > 32 || a.KT < 1 || a.NT < 1 || (size_t)a.NT * a.KT * 1024 > 0x7fffffffu) return hipErrorInvalidValue;
  a.wbytes = (unsigned)((size_t)a.NT * a.KT * 1024);
  // one workgroup per compute unit, the smallest grid with the same number of tiles in each; more than RG_TILES_MAX tiles do
  // not fit LDS (then more workgroups)
  a.tiles_wg = (a.NT + 255) / 256;
  if (a.tiles_wg > RG_TILES_MAX) a.tiles_wg = RG_TILES_MAX;
  const int grid = (a.NT + a.tiles_wg - 1) / a.tiles_wg;
  // tiles that share their loads of the rows: all of a workgroup's, or half of them past 6 (registers)
  const int tt = a.tiles_wg <= 4 ? a.tiles_wg : (a.tiles_wg <= 6 ? 6 : 4);
  switch (tt) {
    case 1: return paired ? launch_rgemm_t<true, 1>(stream, a, grid) : launch_rgemm_t<false, 1>(stream, a, grid);
    case 2: return paired ? launch_rgemm_t<true, 2>(stream, a, grid) : launch_rgemm_t<false, 2>(stream, a, grid);
    case 3: return paired ? launch_rgemm_t<true, 3>(stream, a, grid) : launch_rgemm_t<false, 3>(stream, a, grid);
    case 4: return paired ? launch_rgemm_t<true, 4>(stream, a, grid) : launch_rgemm_t<false, 4>(stream, a, grid);
    default: return paired ? launch_rgemm_t<true, 6>(stream, a, grid) : launch_rgemm_t<false, 6>(stream, a, grid);
  }
}

template <bool PAIRED, int TT>
static hipError_t rgemm_setup_t() {
  const int lds = RG_TILES_MAX * MG_WAVES * 32 * 16 * (int)sizeof(float);
  hipError_t e = hipFuncSetAttribute((const void*)rgemm_kernel<PAIRED, TT, 1>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e == hipSuccess) e = hipFuncSetAttribute((const void*)rgemm_kernel<PAIRED, TT, 2>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  return e;
}

hipError_t rgemm_setup() {
  hipError_t e = hipSuccess;
  for (auto f : {rgemm_setup_t<true, 4>, rgemm_setup_t<true, 6>, rgemm_setup_t<false, 4>, rgemm_setup_t<false, 6>})
    if (e == hipSuccess) e = f();
  return e;
}

hipError_t launch_pkv_pack(hipStream_t stream, const PKvPackArgs& a, int head_dim) {
  if (a.M < 1 || a.JP != (a.M + 31) / 32 || (head_dim != 64 && head_dim != 128) || (a.d_model & 3)) return hipErrorInvalidValue;
  const dim3 grid(a.JP, a.H);
  if (head_dim == 128) hipLaunchKernelGGL(pkv_pack_kernel<128>, grid, dim3(256), 0, stream, a);
  else hipLaunchKernelGGL(pkv_pack_kernel<64>, grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

template <int HD, int QT>
static hipError_t launch_pattn_t(hipStream_t stream, const PAttnArgs& a) {
  const int MT = (a.M + 15) / 16;
  const dim3 grid((MT + 4 * QT - 1) / (4 * QT), a.H);
  const size_t lds = (size_t)2 * (4 * (HD / 32) + 2 * (HD / 16)) * 1024;
  hipLaunchKernelGGL((pattn_kernel<HD, QT>), grid, dim3(256), lds, stream, a);
  return hipGetLastError();
}

hipError_t launch_pattn(hipStream_t stream, const PAttnArgs& a, int head_dim) {
  if (a.M < 1 || a.JP != (a.M + 31) / 32 || (head_dim != 64 && head_dim != 128) || a.d_model % 32) return hipErrorInvalidValue;
  // rows per workgroup (64 QT): two query tiles per wave once the prompt gives enough workgroups (four would leave
  // one wave per SIMD: measured slower)
  const bool two = a.M >= 1024;
  if (head_dim == 128) return two ? launch_pattn_t<128, 2>(stream, a) : launch_pattn_t<128, 1>(stream, a);
  return two ? launch_pattn_t<64, 2>(stream, a) : launch_pattn_t<64, 1>(stream, a);
}

}  // namespace ppd
