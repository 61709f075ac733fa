// Instantiations of the two-group W4A16 GEMM for one 16-bit type (-DMOE_DT=0|1: one translation unit each).
#include "gemm_twogroup.hpp"

#ifndef MOE_DT
#error "compile with -DMOE_DT=0|1"
#endif

namespace moe {

static int launch(const TwoGroupParams& p, int fuse, int grid, hipStream_t stream) {
  auto kern = fuse ? w4a16_twogroup_kernel<MOE_DT, 1> : w4a16_twogroup_kernel<MOE_DT, 0>;
  // the dynamic LDS limit of each kernel is raised once per device
  constexpr int kMaxDev = 64;
  static bool allowed[2][kMaxDev] = {};
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return (int)err;
  if (dev < 0 || dev >= kMaxDev || !allowed[fuse ? 1 : 0][dev]) {
    err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kTwoGroupLds);
    if (err != hipSuccess) return (int)err;
    if (dev >= 0 && dev < kMaxDev) allowed[fuse ? 1 : 0][dev] = true;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(512), kTwoGroupLds, stream, p);
  return (int)hipGetLastError();
}

#if MOE_DT == 0
int launch_twogroup_f16(const TwoGroupParams& p, int fuse, int grid, hipStream_t stream) { return launch(p, fuse, grid, stream); }
#else
int launch_twogroup_bf16(const TwoGroupParams& p, int fuse, int grid, hipStream_t stream) { return launch(p, fuse, grid, stream); }
#endif

}  // namespace moe
