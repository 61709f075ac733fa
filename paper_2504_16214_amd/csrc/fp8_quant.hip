// On-the-fly FP8 quantisation of activations for the FP8 mixture-of-experts layer: one float32
// scale per row and per 128 reduction indices (1 x 128 tiles), codes in OCP e4m3.  Float32
// arithmetic in exactly these steps, because the steps decide integer codes:
//     m = max(max |x| over the tile, 1e-4);  scale = m / 448;  code = e4m3(x * (448 / m))
// (the published fine-grained FP8 recipe of the model family the paper serves; Section VII-D names
// the workload, Table II the kernel).  The second kernel applies SiLU-and-multiply to the gate/up
// product first, rounds the activation to the 16-bit type (it is a 16-bit tensor by the layer's
// definition) and quantises that, so the activation never goes to memory in 16 bits.
//
// Mapping: a tile of 128 elements is handled by 16 lanes with 8 consecutive elements each
// (16-byte loads, 8-byte code stores); a wave covers four tiles; the tile maximum is a four-step
// butterfly inside the 16 lanes.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rows_device.hpp"

namespace fp8 {

template <int DT, int FUSE>
__global__ void __launch_bounds__(256)
quantize_rows_kernel(const uint16_t* __restrict__ X, long long rows, int K, uint8_t* __restrict__ codes,
                     float* __restrict__ scales) {
  quantize_rows<DT, FUSE>(X, rows, K, codes, scales, (long long)blockIdx.x * 256 + threadIdx.x, (long long)gridDim.x * 256);
}

// rows * K / 128 tiles, 16 per workgroup; returns a hipError_t
int launch_fp8_quantize(const void* X, long long rows, int K, int dt, int fuse_silu, uint8_t* codes, float* scales,
                        hipStream_t stream) {
  const long long tiles = rows * (K >> 7);
  if (tiles == 0) return 0;
  long long blocks = (tiles + 15) / 16;
  const long long cap = 256LL * 32;
  if (blocks > cap) blocks = cap;
  const dim3 grid((unsigned)blocks), block(256);
  const uint16_t* x = (const uint16_t*)X;
#define FP8_LAUNCH_Q(DT, F) hipLaunchKernelGGL((quantize_rows_kernel<DT, F>), grid, block, 0, stream, x, rows, K, codes, scales)
  if (dt == moe::kF16) { if (fuse_silu) FP8_LAUNCH_Q(moe::kF16, 1); else FP8_LAUNCH_Q(moe::kF16, 0); }
  else { if (fuse_silu) FP8_LAUNCH_Q(moe::kBF16, 1); else FP8_LAUNCH_Q(moe::kBF16, 0); }
#undef FP8_LAUNCH_Q
  return (int)hipGetLastError();
}

}  // namespace fp8
