// Instantiations of the 64-slot W4A16 GEMM for one 16-bit type (-DMOE_DT=0|1: one translation unit each).
#include "gemm_mid.hpp"

#ifndef MOE_DT
#error "compile with -DMOE_DT=0|1"
#endif

namespace moe {

static int launch(const MidParams& p, int fuse, int pre, int grid, hipStream_t stream) {
  auto kern = fuse ? (pre ? w4a16_mid_kernel<MOE_DT, 1, 1> : w4a16_mid_kernel<MOE_DT, 1, 0>)
                   : (pre ? w4a16_mid_kernel<MOE_DT, 0, 1> : w4a16_mid_kernel<MOE_DT, 0, 0>);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), kMidLds, stream, p);
  return (int)hipGetLastError();
}

#if MOE_DT == 0
int launch_mid_f16(const MidParams& p, int fuse, int pre, int grid, hipStream_t stream) { return launch(p, fuse, pre, grid, stream); }
#else
int launch_mid_bf16(const MidParams& p, int fuse, int pre, int grid, hipStream_t stream) { return launch(p, fuse, pre, grid, stream); }
#endif

}  // namespace moe
