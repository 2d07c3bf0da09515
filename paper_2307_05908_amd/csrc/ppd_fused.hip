// Instances and launcher of the kernel that takes one row through all layers in one launch (ppd_fused.h).
#define PPD_FUSED_TU 1
#include "ppd_fused.h"

namespace ppd {

static const void* fused_kernel(int head_dim, bool narrow) {
  if (head_dim == 64) return narrow ? (const void*)decode_layers_kernel<64, true> : (const void*)decode_layers_kernel<64, false>;
  return narrow ? (const void*)decode_layers_kernel<128, true> : (const void*)decode_layers_kernel<128, false>;
}

hipError_t fused_setup(int head_dim, bool narrow, int lds) {
  return hipFuncSetAttribute(fused_kernel(head_dim, narrow), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
}

hipError_t launch_fused(hipStream_t stream, const FusedArgs& a, int head_dim, bool narrow, int grid, int lds) {
  if (grid < 1 || grid > FU_MAX_WG || (head_dim != 64 && head_dim != 128)) return hipErrorInvalidValue;
  if (head_dim == 64) {
    if (narrow) hipLaunchKernelGGL((decode_layers_kernel<64, true>), dim3(grid), dim3(FU_THREADS), lds, stream, a);
    else hipLaunchKernelGGL((decode_layers_kernel<64, false>), dim3(grid), dim3(FU_THREADS), lds, stream, a);
  } else if (narrow) hipLaunchKernelGGL((decode_layers_kernel<128, true>), dim3(grid), dim3(FU_THREADS), lds, stream, a);
  else hipLaunchKernelGGL((decode_layers_kernel<128, false>), dim3(grid), dim3(FU_THREADS), lds, stream, a);
  return hipGetLastError();
}

}  // namespace ppd
