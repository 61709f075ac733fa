// Passes over the rows of the activations in front of a layer's first product, as device functions: kernels of their own
// (elementwise.hip, fp8_quant.hip), or beside the bucketing in its launch (align.hip), which has one workgroup's work.
// `thread` of `threads` (whole workgroups) of those that share the pass; 16 lanes for 128 elements, 8 each.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_kernel.hpp"   // 16-bit conversions, element orders, silu_f32

namespace fp8 {

typedef uint32_t q_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t q_u32x2 __attribute__((ext_vector_type(2)));

// two float32 -> two e4m3 codes in the low or high half of a word (round to nearest even; the
// matrix unit's own converter, OCP flavour on this chip)
__device__ __forceinline__ uint32_t pack_e4m3(float a, float b, uint32_t old, bool high) {
  return high ? (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(a, b, (int)old, true)
              : (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(a, b, (int)old, false);
}

// FUSE = 0: X [rows, K] -> codes [rows, K], scales [rows, K / 128]
// FUSE = 1: H [rows, 2K] (columns [0, K) gate, [K, 2K) up) -> the same for act = rnd(silu(gate) * up)
template <int DT, int FUSE>
__device__ __forceinline__ void quantize_rows(const uint16_t* __restrict__ X, long long rows, int K, uint8_t* __restrict__ codes,
                                              float* __restrict__ scales, long long thread, long long threads) {
  const int KB = K >> 7;
  const long long tiles = rows * KB;
  const int lane16 = (int)threadIdx.x & 15;
  const long long group0 = thread >> 4;      // 16-lane group index
  const long long ngroups = threads >> 4;
  for (long long t = group0; t < tiles; t += ngroups) {                           // uniform per 16-lane group
    const long long row = t / KB;
    const int kb = (int)(t - row * KB);
    const int col = kb * 128 + lane16 * 8;
    float x[8];
    if constexpr (FUSE) {
      const uint16_t* hrow = X + row * 2 * (long long)K;
      const q_u32x4 g = *reinterpret_cast<const q_u32x4*>(hrow + col);
      const q_u32x4 u = *reinterpret_cast<const q_u32x4*>(hrow + K + col);
      const uint32_t gw[4] = {g.x, g.y, g.z, g.w}, uw[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float g0 = moe::from_bits16<DT>((uint16_t)gw[i]), g1 = moe::from_bits16<DT>((uint16_t)(gw[i] >> 16));
        const float u0 = moe::from_bits16<DT>((uint16_t)uw[i]), u1 = moe::from_bits16<DT>((uint16_t)(uw[i] >> 16));
        // the activation is a 16-bit tensor: round it before it is quantised
        x[2 * i] = moe::from_bits16<DT>(moe::to_bits16<DT>(moe::silu_f32(g0) * u0));
        x[2 * i + 1] = moe::from_bits16<DT>(moe::to_bits16<DT>(moe::silu_f32(g1) * u1));
      }
    } else {
      const q_u32x4 v = *reinterpret_cast<const q_u32x4*>(X + row * (long long)K + col);
      const uint32_t vw[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[2 * i] = moe::from_bits16<DT>((uint16_t)vw[i]);
        x[2 * i + 1] = moe::from_bits16<DT>((uint16_t)(vw[i] >> 16));
      }
    }
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(x[i]));
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 16));
    m = fmaxf(m, 1e-4f);
    const float ratio = 448.0f / m;          // correctly rounded float32 division
    uint32_t lo = 0u, hi = 0u;
    lo = pack_e4m3(x[0] * ratio, x[1] * ratio, lo, false);
    lo = pack_e4m3(x[2] * ratio, x[3] * ratio, lo, true);
    hi = pack_e4m3(x[4] * ratio, x[5] * ratio, hi, false);
    hi = pack_e4m3(x[6] * ratio, x[7] * ratio, hi, true);
    *reinterpret_cast<q_u32x2*>(codes + row * (long long)K + col) = q_u32x2{lo, hi};
    if (lane16 == 0) scales[t] = m / 448.0f;
  }
}

}  // namespace fp8

namespace moe {

// Activations for the two-group and the 64-slot GEMM.  out (may be null): every run of eight reduction indices in
// the order 0,4,1,5,2,6,3,7 (DEAL: 0,2,4,6,1,3,5,7).  sums (may be null): factor * (sum of the row's 128-index group), float32
// (two-group, bf16: 47, the constant its operands carry; 64-slot, bf16: 16, kZeroUnit).  16 lanes per group, 8 elements each;
// a pure stream (4096 x 7168: 117 MB moved in 24 us).
template <int DT, int DEAL>
__device__ __forceinline__ void prepare_rows(const uint16_t* __restrict__ X, long long groups, uint16_t* __restrict__ out,
                                             float* __restrict__ sums, float factor, long long thread, long long threads) {
  for (long long g = thread >> 4; g < groups; g += threads >> 4) {
    const long long at = g * 128 + (threadIdx.x & 15) * 8;
    const u32x4 v = *reinterpret_cast<const u32x4*>(X + at);
    if (out) *reinterpret_cast<u32x4*>(out + at) = DEAL ? deal8(v) : interleave8(v);
    if (sums) {
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) s += from_bits16<DT>((uint16_t)v[i]) + from_bits16<DT>((uint16_t)(v[i] >> 16));
#pragma unroll
      for (int d = 8; d >= 1; d >>= 1) s += __shfl_xor(s, d, 16);
      if ((threadIdx.x & 15) == 0) sums[g] = factor * s;
    }
  }
}

// One of the passes over X [rows, K] (kind), to run beside the bucketing.
struct RowsJob {
  enum Kind { kNone, kInterleaveF16, kInterleaveBf16, kDealBf16, kQuantizeF16, kQuantizeBf16 };
  int kind = kNone, K = 0;
  const uint16_t* X = nullptr;
  long long rows = 0;
  void* out = nullptr;         // rows in another order, or codes
  float* floats = nullptr;     // group sums (may be null), or scales
  float factor = 0.f;
  long long groups() const { return rows * (K >> 7); }
};

// The job of launch_prepare_rows / launch_fp8_quantize with these arguments.
inline RowsJob prepare_job(const void* X, long long rows, int K, int dt, int deal, void* out, float* sums, float factor) {
  return {dt == kF16 ? RowsJob::kInterleaveF16 : deal ? RowsJob::kDealBf16 : RowsJob::kInterleaveBf16, K, (const uint16_t*)X, rows, out, sums, factor};
}
inline RowsJob quantize_job(const void* X, long long rows, int K, int dt, uint8_t* codes, float* scales) {
  return {dt == kF16 ? RowsJob::kQuantizeF16 : RowsJob::kQuantizeBf16, K, (const uint16_t*)X, rows, codes, scales, 0.f};
}

__device__ __forceinline__ void run_job(const RowsJob& job, long long thread, long long threads) {
  const long long groups = job.rows * (job.K >> 7);
  switch (job.kind) {
    case RowsJob::kInterleaveF16: prepare_rows<kF16, 0>(job.X, groups, (uint16_t*)job.out, job.floats, job.factor, thread, threads); break;
    case RowsJob::kInterleaveBf16: prepare_rows<kBF16, 0>(job.X, groups, (uint16_t*)job.out, job.floats, job.factor, thread, threads); break;
    case RowsJob::kDealBf16: prepare_rows<kBF16, 1>(job.X, groups, (uint16_t*)job.out, job.floats, job.factor, thread, threads); break;
    case RowsJob::kQuantizeF16: fp8::quantize_rows<kF16, 0>(job.X, job.rows, job.K, (uint8_t*)job.out, job.floats, thread, threads); break;
    case RowsJob::kQuantizeBf16: fp8::quantize_rows<kBF16, 0>(job.X, job.rows, job.K, (uint8_t*)job.out, job.floats, thread, threads); break;
    default: break;
  }
}

}  // namespace moe
