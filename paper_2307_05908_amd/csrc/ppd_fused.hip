// Instances and launcher of the kernel that takes one row through all layers in one launch (ppd_fused.h).
#define PPD_FUSED_TU 1
#include "ppd_fused.h"

namespace ppd {

hipError_t fused_setup(int head_dim, int lds) {
  const void* f = head_dim == 64 ? (const void*)decode_layers_kernel<64> : (const void*)decode_layers_kernel<128>;
  return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
}

hipError_t launch_fused(hipStream_t stream, const FusedArgs& a, int head_dim, int grid, int lds) {
  if (grid < 1 || grid > FU_MAX_WG || (head_dim != 64 && head_dim != 128)) return hipErrorInvalidValue;
  if (head_dim == 64) hipLaunchKernelGGL(decode_layers_kernel<64>, dim3(grid), dim3(FU_THREADS), lds, stream, a);
  else hipLaunchKernelGGL(decode_layers_kernel<128>, dim3(grid), dim3(FU_THREADS), lds, stream, a);
  return hipGetLastError();
}

}  // namespace ppd
