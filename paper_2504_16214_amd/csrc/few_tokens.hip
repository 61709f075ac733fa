// The layer for a few tokens: vector times int4 matrix, no bucketing and no matrix instructions.
//
// With a few slots a launch of the tiled GEMM leaves about one wave on a SIMD, and its chain
// load -> LDS -> unpack -> matrix instruction of a stage is exposed (one token of a 7168 x 2048 layer with
// 256 experts, top 8: 118 MB of gate/up weights in 29 us); bucketing and combine are two more launches
// of 5 to 6 us that hardly use the chip.  Here every slot is a vector product of its own: gate/up with
// SiLU-and-multiply is one kernel over (slot, columns), the down projection of all of a token's slots
// with the weighted combine another over (token, columns).  Measured, us, tiled then vector, with the weights in
// the last-level cache (in memory), replayed: that token 57.1 / 41.5 (58.7 / 41.9), bf16 59.0 / 39.6 (59.0 / 39.5); one token of
// 4096 x 14336 with 8 experts, top 2, 54.0 / 42.7 (54.9 / 46.4); 3 of 2048 x 1408 with 64, top 6, groups of 128, 39.3 / 25.7
// (40.0 / 26.8); 16 tokens of 256 x 512 with 8, top 2, 18.7 / 8.2 (19.3 / 8.9).
//
// What bounds it: two launches (9 us); in the gate/up launch the vector unit (77 instructions a wave and
// 1 KB of weights, 118 MB in 26 us: 4.5 TB/s), matrix instructions on 4 x 4 x 4 blocks in place of the dot products
// measured 5 to 10 % slower, they issue from the same port, and two waves for each range of columns with half of the
// reduction each 6 % slower; the down launch (59 MB in 18.6 us) its start, about 5 us, and then the same.  Every workgroup
// of the down launch needs all act vectors of its token, 36 KB at top 8, for 16 columns: they are brought into their final
// form once, by the gate/up kernel, and copied to LDS directly, and both panels of a 2048-long reduction are sent before
// the first is waited for (23.9 us when every workgroup scaled the vectors itself and one panel was in flight).
// With both that token went from 49.2 to 44.0 (another session), bf16 45.4 to 41.4, 4 tokens of 2048 x 1408 37.7 to 30.0.
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
#include "router_device.hpp"

namespace moe {

// A vector: chunks of 32 values, 64 bytes, four runs of eight (each in the order 0,4,1,5,2,6,3,7); run j of
// chunk m lies at position j ^ run_key(m), so that the 8 lanes of a row, which read 8 chunks at once, hit different
// banks.  Behind the values one float32 per chunk.
//   fp16: the unit of the chunk.  The dot product takes subnormal operands as zero, so a chunk is moved up
//         by the power of two that brings its largest value to [2^15, 2^16); values below 2^-29 of
//         that largest one (possible only from 64 on) are lost, which is less than a rounding of its float32
//         sum unless that value's weight is exactly zero.
//   bf16: the sum of its values, which takes the bias of the weights (128 + z) out again.
// The gate/up kernel leaves act in this form in memory (a workgroup produces whole chunks), all values of a token first,
// then its chunks' floats, so that the down kernel copies it to LDS without touching it.
__host__ __device__ __forceinline__ int vec_bytes(int k) { return 2 * k; }
__host__ __device__ __forceinline__ int vec_total(int k) { return vec_bytes(k) + (k >> 5) * 4; }
__device__ __forceinline__ int run_key(int m) { return (m & 3) ^ ((m >> 1) & 2); }

// The power of two for a chunk whose largest exponent field is m (0x7c00 mask): exponent to add
__device__ __forceinline__ uint32_t chunk_up(uint32_t m) {
  const uint32_t e = m >> 10;                                         // 31: an infinity or NaN, nothing moves
  return e == 31 ? 0u : 30u - (e > 1 ? e : 1u);
}

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
  uint32_t s[NR], z[NR];  // the lane's own group: scale bits, zero point (put together at use: here they would be waited for)
};

// NR weight rows per lane (row[q] = the lane's q-th row of the expert) against a vector of K values.
template <int DT, int NR>
struct RowsDot {
  const unsigned char* wbase;
  const uint16_t* sbase;
  const uint8_t* zbase;
  uint32_t woff[NR], goff[NR], wstep, half;
  int K, G, i;
  DotConst dc;
  Panel<NR> ring[2];

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
    half = K % 256 != 0 && i >= 4 ? (pre ? 1024u : 64u) : 0u;        // from a last half step's missing group to the one before
  }
  // What lies past the end reads the last step again, or (a lane past the end in a last half step) its first
  // half; it is not used.
  __device__ __forceinline__ void load_w(int pn, Panel<NR>& P) const {
    const int last = (K - 1) >> 8;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int st = 4 * pn + c < last ? 4 * pn + c : last;
      const unsigned char* const b = wbase + (size_t)st * wstep;
      const uint32_t back = st == last ? half : 0u;
#pragma unroll
      for (int q = 0; q < NR; ++q) P.w[q][c] = *reinterpret_cast<const u32x4*>(b + (uint32_t)(woff[q] - back));
    }
  }
  __device__ __forceinline__ void load_sz(int pn, uint32_t (&s)[NR], uint32_t (&z)[NR]) const {
    const int g = 8 * pn + i < G ? 8 * pn + i : G - 1;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      s[q] = sbase[goff[q] + g];
      z[q] = zbase[goff[q] + g];
    }
  }
  __device__ __forceinline__ void panel(int pn, const Panel<NR>& cur, const unsigned char* xl, const float* xs, float (&acc)[NR]) const {
    uint32_t own[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) own[q] = cur.s[q] | ((cur.z[q] & 15) << 16);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      int m = 8 * (4 * pn + c) + i;               // the lane's chunk
      if (256 * (4 * pn + c) >= K) break;         // (uniform)
      const bool in = 32 * m < K;
      if (!in) m = 0;
      u32x4 x[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = *reinterpret_cast<const u32x4*>(xl + 64 * m + 16 * (j ^ run_key(m)));
      const float xc = xs[m];
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const uint32_t sz = (uint32_t)__shfl((int)own[q], (int)(threadIdx.x & 56) + 2 * c + (i >> 2), 64), z = sz >> 16;
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
  // Panels [p0, p1).  One or two are sent at the start and worked off.  More: one is sent while the one before it is
  // multiplied (two panels in flight, with their code unrolled or the last one read again, are no faster there; a loop over the
  // one or two panels costs 7 us of 19).
  __device__ __forceinline__ void start(int p0, int p1) {
    load_sz(p0, ring[0].s, ring[0].z);
    load_sz(p0 + 1, ring[1].s, ring[1].z);
    load_w(p0, ring[0]);
    if (p1 - p0 == 2) load_w(p0 + 1, ring[1]);
  }
  __device__ __forceinline__ void run(const unsigned char* xl, const float* xs, int p0, int p1, float (&acc)[NR]) {
    if (p1 - p0 > 2) {
      for (int pn = p0; pn < p1; ++pn) {
        const int nx = pn + 1 < p1 ? pn + 1 : pn;
        load_sz(nx, ring[1].s, ring[1].z);
        load_w(nx, ring[1]);
        panel(pn, ring[0], xl, xs, acc);
        ring[0] = ring[1];
      }
    } else {
      panel(p0, ring[0], xl, xs, acc);
      if (p1 - p0 == 2) panel(p0 + 1, ring[1], xl, xs, acc);
    }
  }
};

// 256 threads bring the K activations of a token into an LDS vector; `between` runs after the first loads
// are on their way.
template <int DT, typename F>
__device__ __forceinline__ void stage_row(const uint16_t* src, int K, unsigned char* xl, F between) {
  const int vb = vec_bytes(K);
  u32x4 v[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int k = (c * 256 + (int)threadIdx.x) * 8;
    v[c] = *reinterpret_cast<const u32x4*>(src + (k < K ? k : 0));
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
      const uint32_t up = chunk_up(m);
      const float f = __builtin_bit_cast(float, (127u + up) << 23);
#pragma unroll
      for (int t = 0; t < 4; ++t)
        x[t] = (uint32_t)to_bits16<DT>(from_bits16<DT>((uint16_t)x[t]) * f) |
               ((uint32_t)to_bits16<DT>(from_bits16<DT>((uint16_t)(x[t] >> 16)) * f) << 16);
      s = __builtin_bit_cast(float, (127u - up) << 23);
    }
    if (k >= K) return;
    const int m = k >> 5;
    *reinterpret_cast<u32x4*>(xl + 64 * m + 16 * (((k >> 3) & 3) ^ run_key(m))) = interleave8(x);
    if ((k & 31) == 0) *reinterpret_cast<float*>(xl + vb + m * 4) = s;
  };
#pragma unroll
  for (int c = 0; c < 4; ++c) put((c * 256 + (int)threadIdx.x) * 8, v[c]);
  for (int k0 = 4 * 256 * 8; k0 < K; k0 += 256 * 8) {
    const int k = k0 + (int)threadIdx.x * 8;
    put(k, *reinterpret_cast<const u32x4*>(src + (k < K ? k : 0)));
  }
}

// sum over the 8 lanes of a row (every lane ends up with it)
__device__ __forceinline__ float row_sum(float v) {
  v += __shfl_xor(v, 1, 64);
  v += __shfl_xor(v, 2, 64);
  v += __shfl_xor(v, 4, 64);
  return v;
}

// act[slot, :] = round(silu(gate) * up) with gate / up rounded first, as vectors for the down kernel: the values of
// slot s at vals + s N, the floats of its chunks at units + s N / 32.
// grid (N / 32, slots), 4 waves, 8 columns each: a chunk.  LDS: the token's K activations, a word for each wave, ROUTE:
// the token's ids and weights.
// ROUTE: the ids come from the token's logits; every wave works them out for itself (at most 64 experts: four keys a lane, half
// a microsecond against a launch of 3.5 us), and the first workgroup of a token stores them for the down kernel.
template <int DT, int ROUTE>
__global__ void __launch_bounds__(256, 4)
few_gate_up_kernel(const uint16_t* __restrict__ X, FewRoute route, const int32_t* __restrict__ ids, const unsigned char* __restrict__ qw,
                   const uint16_t* __restrict__ sc, const uint8_t* __restrict__ zp, uint16_t* __restrict__ vals,
                   float* __restrict__ units, int topk, int E, int K, int N, int pre) {
  extern __shared__ __align__(16) unsigned char xl[];
  const int slot = blockIdx.y, lane = threadIdx.x & 63, r = lane >> 3;
  int e;
  if constexpr (ROUTE) {
    int32_t* const rid = reinterpret_cast<int32_t*>(xl + vec_total(K) + 16);
    float* const rw = reinterpret_cast<float*>(rid + kRouter16MaxTopk);
    const int t = slot / topk, j = slot - t * topk;
    route_token_row16<kFewRouteE / 16>(route.logits + (size_t)t * E, route.bias, E, topk, lane, rid, rw);      // (every wave writes the same)
    e = __builtin_amdgcn_readfirstlane(rid[j]);
    if (blockIdx.x == 0 && j == 0 && (int)threadIdx.x < topk) {
      route.ids[slot + threadIdx.x] = rid[threadIdx.x];
      route.weights[slot + threadIdx.x] = rw[threadIdx.x];
    }
  } else {
    e = ids[slot];
  }
  if (e < 0 || e >= E) return;                     // (uniform over the workgroup)
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), chunk = blockIdx.x;
  const int c = 32 * chunk + 8 * wave + r;         // (N is a multiple of 32)
  const uint32_t row[2] = {(uint32_t)c, (uint32_t)(N + c)};
  const size_t eb = (size_t)e * 2 * N;
  const int np = (K + 1023) >> 10;
  RowsDot<DT, 2> rd;
  rd.init(qw + eb * (size_t)(K >> 1), sc + eb * (K >> 7), zp + eb * (K >> 7), row, K, pre, 0);
  stage_row<DT>(X + (size_t)(slot / topk) * K, K, xl, [&]() __attribute__((always_inline)) { rd.start(0, np); });
  __syncthreads();
  float acc[2] = {0.f, 0.f};
  rd.run(xl, reinterpret_cast<const float*>(xl + vec_bytes(K)), 0, np, acc);
  const float g = from_bits16<DT>(to_bits16<DT>(row_sum(acc[0])));
  const float u = from_bits16<DT>(to_bits16<DT>(row_sum(acc[1])));
  const uint16_t a = to_bits16<DT>(silu_f32(g) * u);      // (all 8 lanes of the row hold it)
  // the chunk's float: over the wave's 8 columns, then over the four waves
  uint32_t* const red = reinterpret_cast<uint32_t*>(xl + vec_total(K));
  uint32_t m = a & 0x7c00u;
  float sum = from_bits16<DT>(a);
#pragma unroll
  for (int d = 8; d <= 32; d <<= 1) {
    const uint32_t o = (uint32_t)__shfl_xor((int)m, d, 64);
    m = m > o ? m : o;
    sum += __shfl_xor(sum, d, 64);
  }
  if (lane == 0) red[wave] = DT == kF16 ? m : __builtin_bit_cast(uint32_t, sum);
  __syncthreads();
  const u32x4 all = *reinterpret_cast<const u32x4*>(red);
  uint16_t v = a;
  float unit;
  if constexpr (DT == kF16) {
    const uint32_t m0 = all[0] > all[1] ? all[0] : all[1], m1 = all[2] > all[3] ? all[2] : all[3];
    const uint32_t up = chunk_up(m0 > m1 ? m0 : m1);
    v = to_bits16<DT>(from_bits16<DT>(a) * __builtin_bit_cast(float, (127u + up) << 23));
    unit = __builtin_bit_cast(float, (127u - up) << 23);
  } else {
    const floatx4_t f = __builtin_bit_cast(floatx4_t, all);
    unit = (f[0] + f[1]) + (f[2] + f[3]);
  }
  if ((lane & 7) == 0) vals[(size_t)slot * N + 32 * chunk + 8 * (wave ^ run_key(chunk)) + 2 * (r & 3) + (r >> 2)] = v;
  if (threadIdx.x == 0) units[(size_t)slot * (N >> 5) + chunk] = unit;
}

// out[t, :] = sum over j of w[t, j] * (act[slot] . W2[e]), the products unrounded.  grid (K / 16, T), up to 8 waves,
// 16 columns; a wave takes (slot, part of the reduction) pairs.  LDS: the token's act values, their chunks'
// floats, the pairs' results.
template <int DT>
__global__ void __launch_bounds__(512, 4)
few_down_kernel(const uint16_t* vals, const float* units, const int32_t* __restrict__ ids,
                const float* wts, const unsigned char* qw, const uint16_t* sc,
                const uint8_t* zp, uint16_t* out, int topk, int E, int K, int N, int parts, int pre) {
  extern __shared__ __align__(16) unsigned char xl[];
  const int vbytes = topk * vec_bytes(N), ubytes = topk * (N >> 5) * 4;
  float* const ys = reinterpret_cast<float*>(xl + vbytes + ubytes);          // [topk * parts][16]
  const int t = blockIdx.y, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int np = (N + 1023) >> 10;
  const int c0 = blockIdx.x * 16, r = lane >> 3;
  const uint32_t row[2] = {(uint32_t)(c0 + 2 * r), (uint32_t)(c0 + 2 * r + 1)};
  const int nw = (int)blockDim.x >> 6;              // at most eight waves, and as many pairs
  const int e0 = ids[t * topk + wave / parts];
  // act straight to LDS (both arrays are whole runs of 16 bytes).  (The weights are no __restrict__ pointers: their first
  // loads would be moved behind the barrier.)
  typedef __attribute__((address_space(3))) void* lptr_t;
  const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void*)(vals + (size_t)t * topk * N), 0, vbytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc((void*)(units + (size_t)t * topk * (N >> 5)), 0, ubytes, 0x00020000);
  for (int o = wave * 1024; o < vbytes; o += nw * 1024)
    if (o + lane * 16 < vbytes) __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lptr_t)(xl + o), 16, lane * 16, o, 0, 0);
  for (int o = wave * 1024; o < ubytes; o += nw * 1024)
    if (o + lane * 16 < ubytes) __builtin_amdgcn_raw_ptr_buffer_load_lds(ru, (lptr_t)(xl + vbytes + o), 16, lane * 16, o, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  RowsDot<DT, 2> rd;
  // The pair's first panels, e its expert; false: none, nothing to do.  (The loads are sent all the same, for expert 0: with a
  // branch around them the compiler waits where its paths meet, 23 us instead of 19.5 for one 7168 x 2048 token.)
  auto start = [&](int u, int e) __attribute__((always_inline)) {
    const int j = u / parts, part = u - j * parts;
    const int p1 = (part + 1) * np / parts, p0 = part * np / parts;
    const bool some = e >= 0 && e < E;
    const size_t eb = (size_t)(some ? e : 0) * K;
    rd.init(qw + eb * (size_t)(N >> 1), sc + eb * (N >> 7), zp + eb * (N >> 7), row, N, pre, 1);
    rd.start(p0, p1);
    return some;
  };
  bool some = start(wave, e0);
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0F70);               // vmcnt(0): act has landed (and the first panels, which are next)
  asm volatile("" ::: "memory");
  __syncthreads();
  for (int u = wave; u < topk * parts; u += nw) {
    const int j = u / parts, part = u - j * parts;
    if (u != wave) some = start(u, ids[t * topk + j]);
    float acc[2] = {0.f, 0.f};
    if (some)
      rd.run(xl + (size_t)j * vec_bytes(N), reinterpret_cast<const float*>(xl + vbytes) + (size_t)j * (N >> 5), part * np / parts, (part + 1) * np / parts, acc);
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
  return K % 128 == 0 && N % 128 == 0 && (size_t)vec_total(K) + 16 + kRouter16MaxTopk * 8 <= kFewLds && (size_t)topk * (vec_total(N) + 8 * 64) <= kFewLds;
}

int few_down_parts(int topk, int N) {
  const int parts = topk >= 8 ? 1 : topk >= 4 ? 2 : topk >= 2 ? 4 : 8, panels = (N + 1023) / 1024;
  return parts < panels ? parts : panels;
}

int launch_few_gate_up(const void* X, const FewRoute* route, const int32_t* ids, const int32_t* qw, const void* s, const uint8_t* z, void* act,
                       float* units, int T, int topk, int E, int K, int N, int dt, int pre, hipStream_t stream) {
  const dim3 grid(N / 32, T * topk), block(256);
  const size_t lds = (size_t)vec_total(K) + 16 + (route ? kRouter16MaxTopk * 8 : 0);
#define MOE_LAUNCH_FEW(DT, ROUTE) \
  hipLaunchKernelGGL((few_gate_up_kernel<DT, ROUTE>), grid, block, lds, stream, (const uint16_t*)X, route ? *route : FewRoute{}, ids, \
                     (const unsigned char*)qw, (const uint16_t*)s, z, (uint16_t*)act, units, topk, E, K, N, pre)
  if (dt == kF16) { if (route) MOE_LAUNCH_FEW(kF16, 1); else MOE_LAUNCH_FEW(kF16, 0); }
  else { if (route) MOE_LAUNCH_FEW(kBF16, 1); else MOE_LAUNCH_FEW(kBF16, 0); }
#undef MOE_LAUNCH_FEW
  return (int)hipGetLastError();
}

int launch_few_down(const void* act, const float* units, const int32_t* ids, const float* w, const int32_t* qw, const void* s, const uint8_t* z,
                    void* out, int T, int topk, int E, int K, int N, int dt, int pre, hipStream_t stream) {
  const int parts = few_down_parts(topk, N);
  const int pairs = topk * parts;
  const dim3 grid(K / 16, T), block(64 * (pairs < 8 ? pairs : 8));
  const size_t lds = (size_t)topk * (vec_total(N) + parts * 64);
  if (dt == kF16)
    hipLaunchKernelGGL(few_down_kernel<kF16>, grid, block, lds, stream, (const uint16_t*)act, units, ids, w, (const unsigned char*)qw,
                       (const uint16_t*)s, z, (uint16_t*)out, topk, E, K, N, parts, pre);
  else
    hipLaunchKernelGGL(few_down_kernel<kBF16>, grid, block, lds, stream, (const uint16_t*)act, units, ids, w, (const unsigned char*)qw,
                       (const uint16_t*)s, z, (uint16_t*)out, topk, E, K, N, parts, pre);
  return (int)hipGetLastError();
}

}  // namespace moe
