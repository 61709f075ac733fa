// The layer for a few tokens: vector times int4 matrix, no bucketing and no matrix instructions.
//
// With a few slots a launch of the tiled GEMM leaves about one wave on a SIMD, and its chain
// load -> LDS -> unpack -> matrix instruction of a stage is exposed (one token of a 7168 x 2048 layer with
// 256 experts, top 8: 118 MB of gate/up weights in 29 us); bucketing and combine are two more launches
// of 5 to 6 us that hardly use the chip.  Here every slot is a vector product of its own: gate/up with
// SiLU-and-multiply is one kernel over (slot, columns), the down projection of all of a token's slots
// with the weighted combine another over (token, columns).  Measured, us, tiled then vector, with the weights in
// the last-level cache (in memory): that token 57.3 / 45.9 (59.7 / 48.8), bf16 60.6 / 43.8 (63.3 / 48.3); one token of
// 4096 x 14336 with 8 experts, top 2, 53.7 / 44.1 (55.9 / 49.3); of 2048 x 1408 with 64, top 6, groups of 128, 29.6 / 17.5
// (31.1 / 21.3); 16 tokens of 256 x 512 with 8, top 2, 18.7 / 9.4 (19.4 / 9.8).
//
// What bounds it: two launches (9 us); in the gate/up launch the vector unit (77 instructions a wave and
// 1 KB of weights, 118 MB in 26 us: 4.5 TB/s), matrix instructions on 4 x 4 x 4 blocks in place of the dot products
// measured 5 to 10 % slower, they issue from the same port; in the down launch (59 MB in 24 us) every workgroup
// stages all act vectors of its token, 36 KB at top 8, for 16 columns.
//
// A wave covers 16 weight rows; 8 lanes share a row, lane i takes reduction indices 256 c + 32 i + [0, 32)
// (16 bytes) of step c: 128 contiguous bytes of a row, or 128-byte runs of the offline repack's blocks
// (256 bytes of 4 rows measured slower: fewer waves fit and a short reduction leaves lanes idle).  A panel
// of four steps (1024 indices, eight groups of 128) is loaded while the previous one is multiplied; lane i
// fetches the scale and zero point of the panel's group i and passes them round.  The order in which a
// row is summed is the same in both weight layouts.  Weights go through the caches: slots that share
// an expert find them there, and a layer that fits the last-level cache stays in it (2048 x 1408 called again
// and again: 17 us against 21 with non-temporal loads, the 256-expert layer the same).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "few_tokens.hpp"
#include "gemm_kernel.hpp"   // 16-bit conversions, interleave8, unpack constants

namespace moe {

// A vector in LDS: chunks of 32 values (four runs of eight, reordered 0,4,1,5,2,6,3,7), 16 bytes of
// padding after every fourth chunk: the 8 lanes of a row read 8 chunks at once, and with it they hit
// different banks.  Behind the values one float32 per chunk.
//   fp16: the unit of the chunk.  The dot product takes subnormal operands as zero, so a chunk is moved up
//         by the power of two that brings its largest value to [2^15, 2^16); values below 2^-29 of
//         that largest one (possible only from 64 on) are lost, which is less than a rounding of its float32
//         sum unless that value's weight is exactly zero.
//   bf16: the sum of its values, which takes the bias of the weights (128 + z) out again.
__host__ __device__ __forceinline__ int vec_bytes(int k) { return 2 * k + (k >> 7) * 16; }
__host__ __device__ __forceinline__ int vec_total(int k) { return vec_bytes(k) + (k >> 5) * 4; }

// c + a.x b.x + a.y b.y in float32
typedef __bf16 bf16_pair __attribute__((ext_vector_type(2)));
template <int DT>
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  if constexpr (DT == kF16)
    return __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, a), __builtin_bit_cast(half2_t, b), c, false);
  else
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16_pair, a), __builtin_bit_cast(bf16_pair, b), c, false);
}

struct DotConst {
  uint32_t hi, lo;           // see UnpackConsts
};
// Eight weights against eight values: fp16 operands are the exact q - z, bf16 operands 128 + q.
template <int DT>
__device__ __forceinline__ float word_mac(uint32_t v, const u32x4& x, half2_t zA, half2_t zB, const DotConst& dc, float c) {
  const uint32_t v8 = v >> 8;
  uint32_t r[4];
  if constexpr (DT == kF16) {
    r[0] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, (v & 0x000F000Fu) | dc.hi) - zA);
    r[1] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, (v & 0x00F000F0u) | dc.lo) - zB);
    r[2] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, (v8 & 0x000F000Fu) | dc.hi) - zA);
    r[3] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, (v8 & 0x00F000F0u) | dc.lo) - zB);
  } else {
    r[0] = (v & 0x000F000Fu) | dc.hi;
    r[1] = ((v >> 4) & 0x000F000Fu) | dc.hi;
    r[2] = (v8 & 0x000F000Fu) | dc.hi;
    r[3] = ((v >> 12) & 0x000F000Fu) | dc.hi;
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) c = dot2<DT>(r[t], x[t], c);
  return c;
}

template <int NR>
struct Panel {
  u32x4 w[NR][4];
  uint32_t sz[NR];        // the lane's own group: scale bits | zero point << 16
};

// NR weight rows per lane (row[q] = the lane's q-th row of the expert) against a vector of K values.
template <int DT, int NR>
struct RowsDot {
  const unsigned char* wbase;
  const uint16_t* sbase;
  const uint8_t* zbase;
  uint32_t woff[NR], goff[NR], wstep, first;
  int K, G, i;
  DotConst dc;
  Panel<NR> cur;

  __device__ __forceinline__ void init(const unsigned char* wb, const uint16_t* sb, const uint8_t* zb, const uint32_t (&row)[NR],
                                       int K_, int pre, int paired) {
    wbase = wb; sbase = sb; zbase = zb; K = K_; G = K_ >> 7; i = threadIdx.x & 7;
    dc.hi = vgpr_const(DT == kF16 ? 0x64006400u : 0x43004300u);
    dc.lo = vgpr_const(0x54005400u);
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const uint32_t r = row[q];
      const uint32_t blk = paired ? ((r >> 5) << 1) | (r & 1) : r >> 4, n = paired ? (r >> 1) & 15 : r & 15;
      goff[q] = r * (uint32_t)G;
      woff[q] = pre ? (blk * (uint32_t)G + (uint32_t)(i >> 2)) * 1024u + (16u * (i & 3) + n) * 16u : r * (uint32_t)(K >> 1) + 16u * i;
    }
    wstep = pre ? 2048u : 128u;
    first = 0u - (pre ? (uint32_t)(i >> 2) * 1024u : 16u * i);     // back to the row's first group
  }
  // A step past the end, or a lane past the end in a last half step, reads bytes of the row's first
  // group, which are not used.
  __device__ __forceinline__ void load(int pn, Panel<NR>& P) const {
    const int g = 8 * pn + i < G ? 8 * pn + i : G - 1;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int st = 4 * pn + c;
      const uint32_t o = 256 * st + 32 * i < K ? (uint32_t)st * wstep : first;
#pragma unroll
      for (int q = 0; q < NR; ++q)
        P.w[q][c] = *reinterpret_cast<const u32x4*>(wbase + (uint32_t)(woff[q] + o));
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) P.sz[q] = (uint32_t)sbase[goff[q] + g] | ((uint32_t)(zbase[goff[q] + g] & 15) << 16);
  }
  template <bool FULL>
  __device__ __forceinline__ void panel(int pn, const unsigned char* xl, const float* xs, float (&acc)[NR]) const {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      int m = 8 * (4 * pn + c) + i;               // the lane's chunk
      if (!FULL && 256 * (4 * pn + c) >= K) break;
      const bool in = FULL || 32 * m < K;
      if (!in) m = 0;
      u32x4 x[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = *reinterpret_cast<const u32x4*>(xl + 64 * m + 16 * (m >> 2) + 16 * j);
      const float xc = xs[m];
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const uint32_t sz = (uint32_t)__shfl((int)cur.sz[q], (int)(threadIdx.x & 56) + 2 * c + (i >> 2), 64), z = sz >> 16;
        const half2_t zA = __builtin_bit_cast(half2_t, 0x64006400u + z * 0x00010001u), zB = __builtin_bit_cast(half2_t, 0x54005400u + z * 0x00100010u);
        float d = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) d = word_mac<DT>(cur.w[q][c][j], x[j], zA, zB, dc, d);
        const float p = DT == kF16 ? d * xc : __builtin_fmaf(-(128.f + (float)z), xc, d);
        const float a = __builtin_fmaf(from_bits16<DT>((uint16_t)sz), p, acc[q]);
        acc[q] = in ? a : acc[q];
      }
    }
  }
  // panels [p0, p1); cur holds panel p0
  __device__ __forceinline__ void run(const unsigned char* xl, const float* xs, int p0, int p1, float (&acc)[NR]) {
    for (int pn = p0; pn < p1; ++pn) {
      Panel<NR> nxt;
      load(pn + 1 < p1 ? pn + 1 : pn, nxt);
      if (1024 * (pn + 1) <= K) panel<true>(pn, xl, xs, acc);
      else panel<false>(pn, xl, xs, acc);
      cur = nxt;
    }
  }
};

// THREADS threads bring n values (rows of K) from src into LDS vectors; `between` runs after the first
// loads are on their way.
template <int DT, int THREADS, bool REORDER, typename F>
__device__ __forceinline__ void stage_vectors(const uint16_t* src, int n, int K, unsigned char* xl, F between) {
  const int vb = vec_bytes(K), vt = vec_total(K);
  u32x4 v[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int k = (c * THREADS + (int)threadIdx.x) * 8;
    v[c] = *reinterpret_cast<const u32x4*>(src + (k < n ? k : 0));
  }
  between();
  auto put = [&](int k, u32x4 x) __attribute__((always_inline)) {
    float s = 0.f;
    if constexpr (DT == kBF16) {
#pragma unroll
      for (int t = 0; t < 4; ++t) s += from_bits16<DT>((uint16_t)x[t]) + from_bits16<DT>((uint16_t)(x[t] >> 16));
      s += __shfl_xor(s, 1, 64);
      s += __shfl_xor(s, 2, 64);
    } else {
      uint32_t m = 0;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const uint32_t a = x[t] & 0x7c00u, b = (x[t] >> 16) & 0x7c00u;
        m = m > a ? m : a;
        m = m > b ? m : b;
      }
      uint32_t o = (uint32_t)__shfl_xor((int)m, 1, 64);
      m = m > o ? m : o;
      o = (uint32_t)__shfl_xor((int)m, 2, 64);
      m = m > o ? m : o;
      const uint32_t e = m >> 10;                                       // 31: an infinity or NaN, nothing moves
      const uint32_t up = e == 31 ? 0u : 30u - (e > 1 ? e : 1u);
      const float f = __builtin_bit_cast(float, (127u + up) << 23);
#pragma unroll
      for (int t = 0; t < 4; ++t)
        x[t] = (uint32_t)to_bits16<DT>(from_bits16<DT>((uint16_t)x[t]) * f) |
               ((uint32_t)to_bits16<DT>(from_bits16<DT>((uint16_t)(x[t] >> 16)) * f) << 16);
      s = __builtin_bit_cast(float, (127u - up) << 23);
    }
    if (k >= n) return;
    const int r = k / K, kr = k - r * K;
    unsigned char* const b = xl + r * vt;
    *reinterpret_cast<u32x4*>(b + 2 * kr + (kr >> 7) * 16) = REORDER ? interleave8(x) : x;
    if ((kr & 31) == 0) *reinterpret_cast<float*>(b + vb + (kr >> 5) * 4) = s;
  };
#pragma unroll
  for (int c = 0; c < 4; ++c) put((c * THREADS + (int)threadIdx.x) * 8, v[c]);
  for (int k0 = 4 * THREADS * 8; k0 < n; k0 += THREADS * 8) {
    const int k = k0 + (int)threadIdx.x * 8;
    put(k, *reinterpret_cast<const u32x4*>(src + (k < n ? k : 0)));
  }
}

// sum over the 8 lanes of a row (every lane ends up with it)
__device__ __forceinline__ float row_sum(float v) {
  v += __shfl_xor(v, 1, 64);
  v += __shfl_xor(v, 2, 64);
  v += __shfl_xor(v, 4, 64);
  return v;
}

// act[slot, :] = round(silu(gate) * up) with gate / up rounded first, runs of eight reordered.
// grid (ceil(N / 32), slots), 4 waves, 8 columns each.  LDS: the token's K activations.
template <int DT>
__global__ void __launch_bounds__(256)
few_gate_up_kernel(const uint16_t* __restrict__ X, const int32_t* ids, const unsigned char* __restrict__ qw,
                   const uint16_t* __restrict__ sc, const uint8_t* __restrict__ zp, uint16_t* __restrict__ act, int topk,
                   int E, int K, int N, int pre) {
  extern __shared__ __align__(16) unsigned char xl[];
  const int slot = blockIdx.y, e = ids[slot];
  if (e < 0 || e >= E) return;                     // (uniform over the workgroup)
  const int lane = threadIdx.x & 63, r = lane >> 3;
  const int col0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 8;
  const int c = (col0 < N ? col0 : 0) + r;         // (N is a multiple of 8: whole waves)
  const uint32_t row[2] = {(uint32_t)c, (uint32_t)(N + c)};
  const size_t eb = (size_t)e * 2 * N;
  RowsDot<DT, 2> rd;
  rd.init(qw + eb * (size_t)(K >> 1), sc + eb * (K >> 7), zp + eb * (K >> 7), row, K, pre, 0);
  stage_vectors<DT, 256, true>(X + (size_t)(slot / topk) * K, K, K, xl, [&]() __attribute__((always_inline)) { rd.load(0, rd.cur); });
  __syncthreads();
  float acc[2] = {0.f, 0.f};
  rd.run(xl, reinterpret_cast<const float*>(xl + vec_bytes(K)), 0, (K + 1023) >> 10, acc);
  const float g = from_bits16<DT>(to_bits16<DT>(row_sum(acc[0])));
  const float u = from_bits16<DT>(to_bits16<DT>(row_sum(acc[1])));
  if ((lane & 7) == 0 && col0 < N) act[(size_t)slot * N + col0 + 2 * (r & 3) + (r >> 2)] = to_bits16<DT>(silu_f32(g) * u);
}

// out[t, :] = sum over j of w[t, j] * (act[slot] . W2[e]), the products unrounded.  grid (K / 16, T), 8 waves,
// 16 columns; a wave takes (slot, part of the reduction) pairs.  LDS: the token's act rows, then the
// pairs' results.
template <int DT>
__global__ void __launch_bounds__(512)
few_down_kernel(const uint16_t* __restrict__ act, const int32_t* ids, const float* __restrict__ wts,
                const unsigned char* __restrict__ qw, const uint16_t* __restrict__ sc, const uint8_t* __restrict__ zp,
                uint16_t* __restrict__ out, int topk, int E, int K, int N, int parts, int pre) {
  extern __shared__ __align__(16) unsigned char xl[];
  const int vt = vec_total(N), vb = vec_bytes(N);
  float* const ys = reinterpret_cast<float*>(xl + (size_t)topk * vt);          // [topk * parts][16]
  const int t = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int np = (N + 1023) >> 10;
  const int c0 = blockIdx.x * 16, r = lane >> 3;
  const uint32_t row[2] = {(uint32_t)(c0 + 2 * r), (uint32_t)(c0 + 2 * r + 1)};
  RowsDot<DT, 2> rd;
  auto start = [&](int u) __attribute__((always_inline)) {       // fetch the pair's first panel; false: nothing to do
    const int j = u / parts, part = u - j * parts;
    const int e = u < topk * parts ? ids[t * topk + j] : -1;
    if (e < 0 || e >= E) return false;
    const size_t eb = (size_t)e * K;
    rd.init(qw + eb * (size_t)(N >> 1), sc + eb * (N >> 7), zp + eb * (N >> 7), row, N, pre, 1);
    rd.load(part * np / parts < np ? part * np / parts : np - 1, rd.cur);
    return true;
  };
  bool some = false;
  stage_vectors<DT, 512, false>(act + (size_t)t * topk * N, topk * N, N, xl, [&]() __attribute__((always_inline)) { some = start(wave); });
  __syncthreads();
  for (int u = wave; u < topk * parts; u += 8) {
    const int j = u / parts, part = u - j * parts;
    if (u != wave) some = start(u);
    float acc[2] = {0.f, 0.f};
    if (some)
      rd.run(xl + (size_t)j * vt, reinterpret_cast<const float*>(xl + (size_t)j * vt + vb), part * np / parts, (part + 1) * np / parts, acc);
    const float y0 = row_sum(acc[0]), y1 = row_sum(acc[1]);
    if ((lane & 7) == 0) { ys[u * 16 + 2 * r] = y0; ys[u * 16 + 2 * r + 1] = y1; }
  }
  __syncthreads();
  if (threadIdx.x < 16) {
    float o = 0.f;
    for (int j = 0; j < topk; ++j) {
      const int e = ids[t * topk + j];
      if (e < 0 || e >= E) continue;
      float y = ys[(j * parts) * 16 + threadIdx.x];
      for (int q = 1; q < parts; ++q) y += ys[(j * parts + q) * 16 + threadIdx.x];
      o = __builtin_fmaf(wts[t * topk + j], y, o);
    }
    out[(size_t)t * K + c0 + threadIdx.x] = to_bits16<DT>(o);
  }
}

bool few_tokens_fit(int topk, int K, int N) {
  return K % 128 == 0 && N % 128 == 0 && (size_t)vec_total(K) <= kFewLds && (size_t)topk * (vec_total(N) + 8 * 64) <= kFewLds;
}

int few_down_parts(int topk, int N) {
  const int parts = topk >= 8 ? 1 : topk >= 4 ? 2 : topk >= 2 ? 4 : 8, panels = (N + 1023) / 1024;
  return parts < panels ? parts : panels;
}

int launch_few_gate_up(const void* X, const int32_t* ids, const int32_t* qw, const void* s, const uint8_t* z, void* act, int T,
                       int topk, int E, int K, int N, int dt, int pre, hipStream_t stream) {
  const dim3 grid((N + 31) / 32, T * topk), block(256);
  const size_t lds = (size_t)vec_total(K);
  if (dt == kF16)
    hipLaunchKernelGGL(few_gate_up_kernel<kF16>, grid, block, lds, stream, (const uint16_t*)X, ids, (const unsigned char*)qw,
                       (const uint16_t*)s, z, (uint16_t*)act, topk, E, K, N, pre);
  else
    hipLaunchKernelGGL(few_gate_up_kernel<kBF16>, grid, block, lds, stream, (const uint16_t*)X, ids, (const unsigned char*)qw,
                       (const uint16_t*)s, z, (uint16_t*)act, topk, E, K, N, pre);
  return (int)hipGetLastError();
}

int launch_few_down(const void* act, const int32_t* ids, const float* w, const int32_t* qw, const void* s, const uint8_t* z,
                    void* out, int T, int topk, int E, int K, int N, int dt, int pre, hipStream_t stream) {
  const int parts = few_down_parts(topk, N);
  const dim3 grid(K / 16, T), block(512);
  const size_t lds = (size_t)topk * (vec_total(N) + parts * 64);
  if (dt == kF16)
    hipLaunchKernelGGL(few_down_kernel<kF16>, grid, block, lds, stream, (const uint16_t*)act, ids, w, (const unsigned char*)qw,
                       (const uint16_t*)s, z, (uint16_t*)out, topk, E, K, N, parts, pre);
  else
    hipLaunchKernelGGL(few_down_kernel<kBF16>, grid, block, lds, stream, (const uint16_t*)act, ids, w, (const unsigned char*)qw,
                       (const uint16_t*)s, z, (uint16_t*)out, topk, E, K, N, parts, pre);
  return (int)hipGetLastError();
}

}  // namespace moe
