// The layer for a few tokens: vector times int4 matrix, no bucketing and no tile.
//
// With a few slots a launch of the tiled GEMM leaves about one wave on a SIMD, and its chain
// load -> LDS -> unpack -> matrix instruction of a stage is exposed; bucketing and combine are two more launches
// of 5 to 6 us that hardly use the chip.  Here every slot is a vector product of its own: gate/up with
// SiLU-and-multiply is one kernel over (slot, columns), the down projection of all of a token's slots
// with the weighted combine another over (token, columns).
//
// The products are sums of integers.  A chunk of 32 activations is brought to whole numbers below 2^30 by a power of two
// (its unit), four signed bytes each, digits to the base 256; nibbles as bytes need two masks and a shift for eight
// weights.  The int8 matrix instruction multiplies them: its 16 rows are the 4 digits of the 4 chunks of a quantisation
// group, each zero outside its own chunk, its 16 columns are 16 weight rows.  A lane ends up with the 4 digits' sums of one
// chunk and one weight row and takes the zero point times the chunk's own sums from them, digits 0 and 1 and digits 2 and 3
// together: whole numbers that float32 holds.  So a chunk's sum of (q - z) x is rounded once, when its halves are put
// together; a weight that is its zero point contributes nothing, however large its activation.  Then it multiplies by the
// group's scale.  Some chunks have no such form: fp16 with a value that is no multiple of its unit (only beside one of 64
// and more, 2^19 times as large), bf16 with nothing above 2^-97, either with an infinity or a NaN.  They are kept as
// they are and their weights multiplied one by one in float32 (by_values), unless they are fp16 with kMany values of a 32nd of the largest and more:
// those lose 2^-29 of the largest where a float32 sum that meets but one of the many rounds at 2^-24 of it (simulated on 2048 values, silu(g) u, with
// standard deviations of 4 to 100 and weights of which 3 to 97 % are zero: the same error as float32 sums of all, 5e-9 to 1.5e-8).  Without that most chunks are
// kept where act is in the hundreds, as gates of -10 and less leave a millionth beside it.  bf16 values below 2^-22 of the largest of their
// chunk lose what is below 2^-29 of it: one in a thousand chunks of act has one, and kept as they are they cost 2 to 3 us a
// call; the products with 128 + q that this form replaced lost 2^-24 of 143 times the largest.
//
// What bounds it: two launches of 5 to 6 us each beside the stream of weights (gate/up of one token of 7168 x 2048, 256 experts, top 8, 118 MB from
// memory, 25.6 us and 4.6 TB/s; down 15.9; 44.6 -> 41.5 the call.  With products of float16 pairs on the vector unit, 77 instructions a KB of
// weights where there are 40 now, they took 27.8 and 19.4, and no less with the weights in the cache).  Zero points taken out in whole numbers
// cost 1 % (that call with its weights in the cache 34.4 -> 34.7 us, from memory 43.9 -> 44.7; 12 tokens of 1024 x 1024, 64 experts, top 2, 12.1 -> 12.3 and 18.4).
// Activations as wide as x e^(1.5 y), act in the hundreds: 20 calls of 15 to 100 us that were the slowest beside the float16 pairs while every chunk with
// a loss was kept (0.63 of their speed from the cache, 0.66 from memory) are 1.25 and 1.14 times as fast.
//
// A wave covers 16 weight rows, four groups (4 KB) in flight, the next four asked for as each is used.  The order in which a
// row is summed is the same in both weight layouts.  Weights go through the caches: slots that share
// an expert find them there, and a layer that fits the last-level cache stays in it.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "few_tokens.hpp"
#include "gemm_kernel.hpp"   // 16-bit conversions
#include "router_device.hpp"

namespace moe {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void* lptr_t;

// A vector of k activations: for every group of 128, [half h of a chunk][chunk][digit][16 bytes], the bytes of a half (16
// activations, two weight words) in the order the nibbles are unpacked to: 0, 2, 4, 6, 1, 3, 5, 7 of either word.
// Behind it, two words for every chunk: in the low 24 bits the sum of its digits 0 + 256 digits 1 and that of its digits 2
// + 256 digits 3, in the first one's upper 8 the exponent of its unit.  A chunk that is kept as it is has kAsIs for
// an exponent, and where digits would lie its 16-bit activations, 16 at the start of each half's 64 bytes.
constexpr int kAsIs = -128;
constexpr uint32_t kLossFrom = 0x42800000u;      // 64: below it every fp16 value is a multiple of its chunk's unit
constexpr uint32_t kLarge = 5u << 23;            // (an exponent's difference: a 32nd of the largest)
constexpr int kMany = 4;
__host__ __device__ __forceinline__ int vec_bytes(int k) { return 4 * k; }
__host__ __device__ __forceinline__ int vec_total(int k) { return vec_bytes(k) + (k >> 5) * 8; }
__device__ __forceinline__ int half_at(int chunk, int h) { return (chunk >> 2) * 512 + h * 256 + (chunk & 3) * 64; }      // + 16 digit

// Exponent to add so that the chunk's largest value (float32 bits, no sign) comes to [2^29, 2^30); 126 at most: the factor and the unit
// stay normal numbers.
__device__ __forceinline__ int chunk_up(uint32_t largest) {
  const int up = 29 + 127 - (int)(largest >> 23);
  return up < 126 ? up : 126;
}
__device__ __forceinline__ float power_of_two(int e) { return __builtin_bit_cast(float, (uint32_t)(127 + e) << 23); }
// |v| < 2^30, towards zero to a whole number -> its four signed digits as bytes, each of the first three plus 128
__device__ __forceinline__ uint32_t biased_digits(float v) { return (uint32_t)(int)v + 0x00808080u; }
template <int DT>
__device__ __forceinline__ bool no_digits(uint32_t largest) {      // float32 bits, no sign
  return largest >= 0x7f800000u || (DT == kBF16 && largest - 1u < ((uint32_t)(127 - 97) << 23) - 1u);
}
__device__ __forceinline__ u32x2 chunk_words(bool as_is, int up, int s01, int s23) {
  return as_is ? u32x2{(uint32_t)kAsIs << 24, 0u} : u32x2{((uint32_t)-up << 24) | ((uint32_t)s01 & 0x00FFFFFFu), (uint32_t)s23};
}
// a * (the low 24 bits of b) + c
__device__ __forceinline__ int mad24(int a, uint32_t b, int c) { return a * ((int)(b << 8) >> 8) + c; }

// Over 4 lanes (a quad), over 8, over the lanes (n, 0 ... 3) of a row: every lane ends up with the result.
__device__ __forceinline__ float as_float(uint32_t v) { return __builtin_bit_cast(float, v); }      // (of a vector's element, by value)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true); }
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;
template <int CTRL>
__device__ __forceinline__ uint32_t max_over(uint32_t m) {
  const uint32_t o = dpp<CTRL>(m);
  return m > o ? m : o;
}
template <int CTRL>
__device__ __forceinline__ int sum_over(int v) { return v + (int)dpp<CTRL>((uint32_t)v); }
__device__ __forceinline__ float row_sum(float v) {
  auto h = __builtin_amdgcn_permlane32_swap(bits32(v), bits32(v), false, false);
  v = as_float(h[0]) + as_float(h[1]);
  h = __builtin_amdgcn_permlane16_swap(bits32(v), bits32(v), false, false);
  return as_float(h[0]) + as_float(h[1]);
}

// 16 weight rows against a vector, R groups in flight.  PRE: operand order; register i is group i, lane (n, j) with its own 16 bytes.
// Otherwise registers 2 i and 2 i + 1 are rows 0 ... 7 and 8 ... 15 of groups 2 i and 2 i + 1, a lane with 16 bytes of row lane / 8: 128 bytes in
// a line (64 of each of the 16 rows, the order of the operands, had the caches look up every line twice: 46.7 us for the call
// above where this takes 41.5); pair() brings them to the lanes that want them.
template <int DT, int R, int PRE>
struct Rows16 {
  __amdgpu_buffer_rsrc_t rs, rz;
  const unsigned char* wbase;
  uint32_t woff, soff, wbytes, half, from;
  int G;
  u32x4 w[R];
  uint32_t own[R / 4], nxt_s[R / 4], nxt_z[R / 4];

  // rows: those of one matrix (of one expert); row0: the first of 16, apart: rows from the eighth to the ninth
  __device__ __forceinline__ void init(const unsigned char* wb, const uint16_t* sb, const uint8_t* zb, uint32_t rows, uint32_t row0, uint32_t apart, int K, int paired) {
    const uint32_t lane = threadIdx.x & 63, j = lane >> 4, row = row0 + (lane & 7) + (lane & 8 ? apart : 0);
    G = K >> 7;
    wbytes = rows * (uint32_t)(K >> 1);
    if constexpr (PRE) {
      const uint32_t blk = paired ? ((row >> 5) << 1) | (row & 1) : row >> 4, n = paired ? (row >> 1) & 15 : row & 15;
      woff = blk * (uint32_t)G * 1024u + (16u * j + n) * 16u;
    } else {
      woff = (row0 + (lane >> 3)) * (uint32_t)(K >> 1) + 16u * (lane & 7);
      half = apart * (uint32_t)(K >> 1);
      from = 4u * (8u * (lane & 7) + 4u * ((lane >> 3) & 1) + j);
    }
    soff = row * (uint32_t)G + j;
    wbase = wb;
    rs = __builtin_amdgcn_make_buffer_rsrc((void*)sb, 0, (int)(rows * (uint32_t)G * 2u), 0x00020000);
    rz = __builtin_amdgcn_make_buffer_rsrc((void*)zb, 0, (int)(rows * (uint32_t)G), 0x00020000);
  }
  // Register i, of the pair of groups (g, g + 1) (g even).  A group past the end fetches nothing (a buffer without bytes; the second of an odd
  // row's last pair: an offset past the buffer), and counts as a load all the same.
  __device__ __forceinline__ void load_w(int i, int g, int g1) {
    const bool some = (PRE ? g + (i & 1) : g) < g1;
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)wbase, 0, some ? (int)wbytes : 0, 0x00020000);
    if constexpr (PRE) w[i] = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)woff, (g + (i & 1)) * 1024, 0);
    else w[i] = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(g + 1 < G || !(threadIdx.x & 4) ? woff : 0xFFFFFFF0u), g * 64 + (i & 1 ? (int)half : 0), 0);
  }
  __device__ __forceinline__ void pair(u32x4& a, u32x4& b) const {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t lo = a[t], hi = b[t];
      const int x = __builtin_amdgcn_ds_bpermute((int)from, (int)lo), y = __builtin_amdgcn_ds_bpermute((int)from, (int)hi);
      // (row lane & 7, group lane & 8) of either half -> of either group (row lane & 15)
      a[t] = (uint32_t)__builtin_amdgcn_update_dpp(x, y, 0x128, 0xf, 0xc, false);
      b[t] = (uint32_t)__builtin_amdgcn_update_dpp(y, x, 0x128, 0xf, 0x3, false);
    }
  }
  // scales and zero points of groups [g, g + R): lane group j those of g + j, g + 4 + j ...  (Past a row's end those of
  // the next, past the last row's nothing: not used.)
  __device__ __forceinline__ void load_sz(int g) {
#pragma unroll
    for (int q = 0; q < R / 4; ++q) {
      const uint32_t at = soff + (uint32_t)(g + 4 * q);
      nxt_s[q] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, (int)(2u * at), 0, 0);
      nxt_z[q] = (uint32_t)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(rz, (int)at, 0, 0);
    }
  }
  __device__ __forceinline__ void start(int g0, int g1) {
    load_sz(g0);
#pragma unroll
    for (int i = 0; i < R; ++i) load_w(i, g0 + (i & ~1), g1);
  }
  // The rows' sums over groups [g0, g1), g0 even, against the vector at xl: lane (n, j) has row n's over the chunks j.
  // as_is (uniform): some chunk of the vector may be kept as it is.
  __device__ __forceinline__ float run(const unsigned char* xl, const uint32_t* units, const unsigned char* zeros, int g0, int g1, bool as_is) {
    const int lane = threadIdx.x & 63, n = lane & 15, j = lane >> 4;
    // lanes of the digits of chunk j read them, the others zeros
    const bool mine = (n >> 2) == j;
    const unsigned char* xp = mine ? xl + g0 * 512 + j * 64 + (n & 3) * 16 : zeros;
    const int xstep = mine ? 512 * R : 0;
    const uint32_t* up = units + (size_t)(g0 * 4 + j) * 2;
    float acc = 0.f;
    auto group = [&](int i, int g, const u32x4& v) __attribute__((always_inline)) {
      const u32x4 x0 = *reinterpret_cast<const u32x4*>(xp + 512 * i), x1 = *reinterpret_cast<const u32x4*>(xp + 512 * i + 256);
      const u32x2 u = *reinterpret_cast<const u32x2*>(up + 8 * i);
      const uint32_t sz = (uint32_t)__builtin_amdgcn_ds_bpermute((n + 16 * (i & 3)) * 4, (int)own[i >> 2]);
      const uint32_t m = 0x0F0F0F0Fu;
      i32x4 d = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, x0),
                                                      i32x4{(int)(v.x & m), (int)((v.x >> 4) & m), (int)(v.y & m), (int)((v.y >> 4) & m)}, i32x4{0, 0, 0, 0}, 0, 0, 0);
      d = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(i32x4, x1),
                                                i32x4{(int)(v.z & m), (int)((v.z >> 4) & m), (int)(v.w & m), (int)((v.w >> 4) & m)}, d, 0, 0, 0);
      // |q - z| <= 15, |digit 0 + 256 digit 1| <= 32896, |digit 2 + 256 digit 3| <= 2^14: over 32 weights below 2^24
      const int nz = (int)sz >> 16, exponent = (int)u[0] >> 24;
      const float lo = (float)mad24(nz, u[0], d[0] + (d[1] << 8)), hi = (float)mad24(nz, u[1], d[2] + (d[3] << 8));
      float t = __builtin_ldexpf(__builtin_fmaf(hi, 65536.f, lo), exponent);
      if (__builtin_expect(as_is, 0))
        if (exponent == kAsIs) t = by_values(v, xl + g * 512 + j * 64, nz);
      acc = __builtin_fmaf(from_bits16<DT>((uint16_t)sz), t, acc);
    };
    for (int p = g0; p < g1; p += R) {
#pragma unroll
      for (int q = 0; q < R / 4; ++q) own[q] = nxt_s[q] | ((0u - (nxt_z[q] & 15)) << 16);
      load_sz(p + R);
#pragma unroll
      for (int i = 0; i < R; i += 2) {
        if (p + i >= g1) return acc;
        if constexpr (PRE) {
          group(i, p + i, w[i]);
          load_w(i, p + i + R, g1);
          if (p + i + 1 < g1) group(i + 1, p + i + 1, w[i + 1]);
          load_w(i + 1, p + i + R, g1);
        } else {
          u32x4 a = w[i], b = w[i + 1];
          pair(a, b);
          load_w(i, p + i + R, g1);
          load_w(i + 1, p + i + R, g1);
          group(i, p + i, a);
          if (p + i + 1 < g1) group(i + 1, p + i + 1, b);
        }
      }
      xp += xstep;
      up += 8 * R;
    }
    return acc;
  }
  // A chunk's sum weight by weight, at: its activations as they are, nz: minus the zero point.  (A short loop: straight-line code, 1.4 times as fast where
  // every chunk is kept, cost the calls without one 2 %, cold as a short kernel's instructions are.)
  static __device__ __forceinline__ float by_values(const u32x4& v, const unsigned char* at, int nz) {
    const float z = (float)nz;
    float t = 0.f;
#pragma unroll 1
    for (int i = 0; i < 8; ++i) {
      const uint32_t word = (i < 2 ? v.x : i < 4 ? v.y : i < 6 ? v.z : v.w) >> (16 * (i & 1)), even = word & 0x0F0Fu, odd = (word >> 4) & 0x0F0Fu;
      const u32x2 x = *reinterpret_cast<const u32x2*>(at + 256 * (i >> 2) + 8 * (i & 3));
#pragma unroll
      for (int k = 0; k < 4; ++k)
        t = __builtin_fmaf((float)(uint8_t)((k & 1 ? odd : even) >> (8 * (k >> 1))) + z, from_bits16<DT>((uint16_t)(x[k >> 1] >> (16 * (k & 1)))), t);
    }
    return t;
  }
};

constexpr int kGateThreads = 512;
struct FirstValues { u32x4 v[2]; };
__device__ __forceinline__ FirstValues first_values(const uint16_t* src, int K) {
  FirstValues f;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int k = (c * kGateThreads + (int)threadIdx.x) * 8;
    f.v[c] = *reinterpret_cast<const u32x4*>(src + (k < K ? k : 0));
  }
  return f;
}
// kGateThreads threads bring the K activations of a token into an LDS vector, the first of them loaded already.
// Whether one of the thread's chunks is kept as it is.
template <int DT>
__device__ __forceinline__ bool stage_row(const uint16_t* src, int K, unsigned char* xl, FirstValues& first) {
  bool odd = false;
  uint32_t* const units = reinterpret_cast<uint32_t*>(xl + vec_bytes(K));
  constexpr int step = kGateThreads * 8;
  u32x4 (&v)[2] = first.v;
  auto put = [&](int k, const u32x4& x) __attribute__((always_inline)) {
    // the largest of the chunk, on the 16-bit patterns
    u16x2 top = {0, 0};
#pragma unroll
    for (int t = 0; t < 4; ++t) top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, x[t] & 0x7fff7fffu));
    const uint32_t larger = top.x > top.y ? top.x : top.y;
    const uint32_t m = bits32(from_bits16<DT>((uint16_t)max_over<kXor2>(max_over<kXor1>(larger))));
    if (k >= K) return;                            // (K is a multiple of 32: a chunk's four lanes stay together)
    const int up = chunk_up(m), chunk = k >> 5, word = (k >> 3) & 3;
    const float factor = power_of_two(up);
    auto scaled = [&](int t) __attribute__((always_inline)) { return __builtin_fmaf(from_bits16<DT>((uint16_t)(x[t >> 1] >> (16 * (t & 1)))), factor, 0.f); };
    uint32_t y[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) y[t] = biased_digits(scaled(t));
    bool as_is = no_digits<DT>(m);
    if (DT == kF16 && m >= kLossFrom) {
      const uint32_t large = m + ((uint32_t)up << 23) - kLarge;
      uint32_t rest = 0u;
      int many = 0;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        rest |= bits32(scaled(t) - __builtin_truncf(scaled(t)));
        many += (bits32(scaled(t)) & 0x7fffffffu) >= large;
      }
      rest = max_over<kXor2>(max_over<kXor1>(rest << 1));              // (no sign: what is whole leaves a zero)
      as_is |= rest != 0u && sum_over<kXor2>(sum_over<kXor1>(many)) < kMany;
    }
    // digit planes: bytes of values 0, 2, 4, 6 and of 1, 3, 5, 7
    unsigned char* const at = xl + half_at(chunk, word >> 1) + 8 * (word & 1);
    uint32_t plane[4][2];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const uint32_t a = __builtin_amdgcn_perm(y[2 + o], y[o], 0x05010400u), b = __builtin_amdgcn_perm(y[2 + o], y[o], 0x07030602u);
      const uint32_t c = __builtin_amdgcn_perm(y[6 + o], y[4 + o], 0x05010400u), d = __builtin_amdgcn_perm(y[6 + o], y[4 + o], 0x07030602u);
      plane[0][o] = __builtin_amdgcn_perm(c, a, 0x05040100u) ^ 0x80808080u;
      plane[1][o] = __builtin_amdgcn_perm(c, a, 0x07060302u) ^ 0x80808080u;
      plane[2][o] = __builtin_amdgcn_perm(d, b, 0x05040100u) ^ 0x80808080u;
      plane[3][o] = __builtin_amdgcn_perm(d, b, 0x07060302u);
    }
    int sum[4];
#pragma unroll
    for (int d = 0; d < 4; ++d)
      sum[d] = __builtin_amdgcn_sdot4((int)plane[d][0], 0x01010101, __builtin_amdgcn_sdot4((int)plane[d][1], 0x01010101, 0, false), false);
    const int s01 = sum_over<kXor2>(sum_over<kXor1>(sum[0] + (sum[1] << 8)));
    const int s23 = sum_over<kXor2>(sum_over<kXor1>(sum[2] + (sum[3] << 8)));
    odd |= as_is;
    if (__builtin_expect(as_is, 0)) {
      *reinterpret_cast<u32x4*>(xl + half_at(chunk, word >> 1) + 16 * (word & 1)) = x;
    } else {
#pragma unroll
      for (int d = 0; d < 4; ++d) *reinterpret_cast<u32x2*>(at + 16 * d) = u32x2{plane[d][0], plane[d][1]};
    }
    if (word == 0) *reinterpret_cast<u32x2*>(units + 2 * chunk) = chunk_words(as_is, up, s01, s23);
  };
  // (one copy of the code for all: what a short kernel runs once comes from memory)
#pragma unroll 1
  for (int c = 0; c * step < K; ++c) {
    const int k = c * step + (int)threadIdx.x * 8;
    if (c >= 2) {
      v[0] = *reinterpret_cast<const u32x4*>(src + (k < K ? k : 0));
      __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0), here: behind the branch it would hold for the first loads as well
    }
    put(k, v[0]);
    v[0] = v[1];
  }
  return odd;
}

// Zeros, as long as R groups, that the lanes of the other chunks read.
__host__ __device__ constexpr int zero_bytes(int R) { return 512 * R; }
template <int R>
__device__ __forceinline__ void clear(unsigned char* zeros, int threads) {
  for (int o = 16 * (int)threadIdx.x; o < zero_bytes(R); o += 16 * threads) *reinterpret_cast<u32x4*>(zeros + o) = u32x4{0, 0, 0, 0};
}

// act[slot, :] = round(silu(gate) * up) with gate / up rounded first, as vectors for the down kernel: digits of slot s at
// vals + 4 s N, its chunks' words at units + 2 s N / 32.
// KP 1: grid (N / 64, slots), 8 waves, 8 columns each; KP 2: (N / 32, slots), four times 8 columns, two halves of the reduction.  LDS: the
// token's K activations, zeros, a flag for every wave, the columns' sums, ROUTE: the token's ids and weights.
// ROUTE: the ids come from the token's logits; every wave works them out for itself (at most 64 experts: four keys a lane, half
// a microsecond against a launch of 3.5 us), and the first workgroup of a token stores them for the down kernel.
// (64 registers: four workgroups a CU.)
template <int DT, int ROUTE, int R, int PRE, int KP>
__global__ void __launch_bounds__(kGateThreads, 8)
few_gate_up_kernel(const uint16_t* __restrict__ X, FewRoute route, const int32_t* __restrict__ ids, const unsigned char* __restrict__ qw,
                   const uint16_t* __restrict__ sc, const uint8_t* __restrict__ zp, unsigned char* __restrict__ vals,
                   uint32_t* __restrict__ units, int topk, int E, int K, int N) {
  extern __shared__ __align__(16) unsigned char xl[];
  unsigned char* const zeros = xl + vec_total(K);
  uint32_t* const bad = reinterpret_cast<uint32_t*>(zeros + zero_bytes(R));
  constexpr int COLS = 64 / KP;
  float* const col = reinterpret_cast<float*>(bad + 8);
  const int slot = blockIdx.y, lane = threadIdx.x & 63;
  const uint16_t* const x = X + (size_t)(slot / topk) * K;
  FirstValues first = first_values(x, K);
  int e;
  if constexpr (ROUTE) {
    int32_t* const rid = reinterpret_cast<int32_t*>(col + 128);
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
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), part = KP == 2 ? wave >> 2 : 0, cw = 8 * (KP == 2 ? wave & 3 : wave);
  const size_t eb = (size_t)e * 2 * N;
  const int G = K >> 7, mid = KP == 2 ? 2 * ((G + 2) >> 2) : G, g0 = part ? mid : 0, g1 = part ? G : mid;
  Rows16<DT, R, PRE> rd;       // eight gate rows, the eight up rows of the same columns (N is a multiple of 32)
  rd.init(qw + eb * (size_t)(K >> 1), sc + eb * G, zp + eb * G, 2u * (uint32_t)N, (uint32_t)(COLS * (int)blockIdx.x + cw), (uint32_t)N, K, 0);
  rd.start(g0, g1);
  clear<R>(zeros, kGateThreads);
  const bool odd = stage_row<DT>(x, K, xl, first);
  if (lane == 0) bad[wave] = 0u;
  if (odd) bad[wave] = 1u;
  __syncthreads();
  const u32x4 b0 = *reinterpret_cast<const u32x4*>(bad), b1 = *reinterpret_cast<const u32x4*>(bad + 4);
  const bool odd_row = __builtin_amdgcn_readfirstlane((int)(b0[0] | b0[1] | b0[2] | b0[3] | b1[0] | b1[1] | b1[2] | b1[3])) != 0;
  const float r = rd.run(xl, reinterpret_cast<const uint32_t*>(xl + vec_bytes(K)), zeros, g0, g1, odd_row);
  // [part][gate, up][column]
  const float y = row_sum(r);
  if (lane < 16) col[(2 * part + (lane >> 3)) * COLS + cw + (lane & 7)] = y;
  __syncthreads();
  if ((int)threadIdx.x >= COLS) return;
  float gate = col[threadIdx.x], upper = col[COLS + threadIdx.x];
  if constexpr (KP == 2) {
    gate += col[2 * COLS + threadIdx.x];
    upper += col[3 * COLS + threadIdx.x];
  }
  const float a = from_bits16<DT>(to_bits16<DT>(silu_f32(from_bits16<DT>(to_bits16<DT>(gate))) * from_bits16<DT>(to_bits16<DT>(upper))));
  uint32_t m = max_over<kMirror>(max_over<kHalfMirror>(max_over<kXor2>(max_over<kXor1>(bits32(a) & 0x7fffffffu))));
  const auto both = __builtin_amdgcn_permlane16_swap(m, m, false, false);      // rows 0 and 1 (2 and 3) of 16 lanes
  m = both[0] > both[1] ? both[0] : both[1];
  const int up = chunk_up(m), k = threadIdx.x & 31, chunk = (int)(blockIdx.x * COLS + threadIdx.x) >> 5;
  const float v = a * power_of_two(up);
  bool as_is = no_digits<DT>(m);
  if (DT == kF16) {
    const int half = threadIdx.x & 32;
    const uint32_t rest = (uint32_t)(__ballot(v != __builtin_truncf(v)) >> half), large = (uint32_t)(__ballot((bits32(a) & 0x7fffffffu) >= m - kLarge) >> half);
    as_is |= rest != 0u && __builtin_popcount(large) < kMany;      // (a rest: the largest is 64 or more)
  }
  const uint32_t d = biased_digits(v) ^ 0x00808080u;
  int s01 = ((int)(d << 24) >> 24) + (((int)(d << 16) >> 24) << 8), s23 = ((int)(d << 8) >> 24) + (((int)d >> 24) << 8);
  s01 = sum_over<kMirror>(sum_over<kHalfMirror>(sum_over<kXor2>(sum_over<kXor1>(s01))));
  s23 = sum_over<kMirror>(sum_over<kHalfMirror>(sum_over<kXor2>(sum_over<kXor1>(s23))));
  const auto both01 = __builtin_amdgcn_permlane16_swap((uint32_t)s01, (uint32_t)s01, false, false);
  const auto both23 = __builtin_amdgcn_permlane16_swap((uint32_t)s23, (uint32_t)s23, false, false);
  s01 = (int)(both01[0] + both01[1]);
  s23 = (int)(both23[0] + both23[1]);
  unsigned char* const at = vals + (size_t)slot * vec_bytes(N) + half_at(chunk, k >> 4);
  if (__builtin_expect(as_is, 0)) {
    reinterpret_cast<uint16_t*>(at)[k & 15] = to_bits16<DT>(a);
  } else {
    const int pos = (k & 8) + 4 * (k & 1) + ((k >> 1) & 3);
#pragma unroll
    for (int i = 0; i < 4; ++i) at[16 * i + pos] = (unsigned char)(d >> (8 * i));
  }
  if (k == 0) *reinterpret_cast<u32x2*>(units + ((size_t)slot * (N >> 5) + chunk) * 2) = chunk_words(as_is, up, s01, s23);
}

// out[t, :] = sum over j of w[t, j] * (act[slot] . W2[e]), the products unrounded.  grid (K / 16, T), up to 8 waves,
// 16 columns; a wave takes (slot, part of the reduction) pairs.  LDS: the act vectors of `per` of the token's slots at a time (ROUNDS 0:
// all), their chunks' words, zeros, the results of all pairs.
template <int DT, int R, int PRE, int ROUNDS>
__global__ void __launch_bounds__(512, 4)
few_down_kernel(const unsigned char* vals, const uint32_t* units, const int32_t* __restrict__ ids,
                const float* wts, const unsigned char* qw, const uint16_t* sc,
                const uint8_t* zp, uint16_t* out, int topk, int E, int K, int N, int parts, int per) {
  extern __shared__ __align__(16) unsigned char xl[];
  const int vbytes = (ROUNDS ? per : topk) * vec_bytes(N), ubytes = (ROUNDS ? per : topk) * (N >> 5) * 8;
  unsigned char* const zeros = xl + vbytes + ubytes;
  float* const ys = reinterpret_cast<float*>(zeros + zero_bytes(R));          // [topk * parts][16]
  const int t = blockIdx.y, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int G = N >> 7;
  const int c0 = blockIdx.x * 16;
  const int nw = (int)blockDim.x >> 6;              // at most eight waves, and as many pairs
  Rows16<DT, R, PRE> rd;
  auto range = [&](int part, int& g0, int& g1) __attribute__((always_inline)) {
    const int pairs = (G + 1) >> 1;
    g0 = 2 * (part * pairs / parts);
    g1 = part + 1 == parts ? G : 2 * ((part + 1) * pairs / parts);
  };
  // The pair's first groups, e its expert; false: none, nothing to do.  (The loads are sent all the same, for expert 0: with a
  // branch around them the compiler waits where its paths meet.)
  auto start = [&](int u, int e) __attribute__((always_inline)) {
    int g0, g1;
    range(u % parts, g0, g1);
    const bool some = e >= 0 && e < E;
    const size_t eb = (size_t)(some ? e : 0) * K;
    rd.init(qw + eb * (size_t)(N >> 1), sc + eb * G, zp + eb * G, (uint32_t)K, (uint32_t)c0, 8u, N, 1);
    rd.start(g0, g1);
    return some;
  };
  auto round = [&](int s0, int slots) __attribute__((always_inline)) {
    const int e0 = !ROUNDS || wave / parts < slots ? ids[t * topk + s0 + wave / parts] : -1;
    // act straight to LDS (both arrays are whole runs of 16 bytes)
    const int vb = slots * vec_bytes(N), ub = slots * (N >> 5) * 8;
    const size_t slot0 = (size_t)t * topk + s0;
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void*)(vals + slot0 * vec_bytes(N)), 0, vb, 0x00020000);
    const __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc((void*)((const unsigned char*)units + slot0 * (N >> 5) * 8), 0, ub, 0x00020000);
    for (int o = wave * 1024; o < vb; o += nw * 1024)
      if (o + lane * 16 < vb) __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lptr_t)(xl + o), 16, lane * 16, o, 0, 0);
    for (int o = wave * 1024; o < ub; o += nw * 1024)
      if (o + lane * 16 < ub) __builtin_amdgcn_raw_ptr_buffer_load_lds(ru, (lptr_t)(xl + vbytes + o), 16, lane * 16, o, 0, 0);
    if (s0 == 0) clear<R>(zeros, 64 * nw);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    bool some = start(wave, e0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);             // vmcnt(0): act has landed (and the first groups, which are next)
    asm volatile("" ::: "memory");
    __syncthreads();
    for (int u = wave; u < slots * parts; u += nw) {
      const int j = u / parts;
      int g0, g1;
      range(u - j * parts, g0, g1);
      if (u != wave) some = start(u, ids[t * topk + s0 + j]);
      float r = 0.f;
      if (some) {
        const unsigned char* const xv = xl + (size_t)j * vec_bytes(N);
        const uint32_t* const xu = reinterpret_cast<const uint32_t*>(xl + vbytes) + (size_t)j * (N >> 5) * 2;
        bool odd = false;
        for (int i = 4 * g0 + lane; i < 4 * g1; i += 64) odd |= (int)xu[2 * i] >> 24 == kAsIs;
        r = rd.run(xv, xu, zeros, g0, g1, __ballot(odd) != 0ull);
      }
      const float y = row_sum(r);
      if (lane < 16) ys[(s0 * parts + u) * 16 + lane] = y;
    }
    __syncthreads();
  };
  if constexpr (ROUNDS) {
#pragma unroll 1
    for (int s0 = 0; s0 < topk; s0 += per) round(s0, per < topk - s0 ? per : topk - s0);
  } else {
    round(0, topk);
  }
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

// Groups in flight a wave.  Eight would have more on its way, and twice the code: a kernel of ten to twenty us fetches its
// instructions from memory once, and loses as much on that (1 token of 7168 x 2048, 256 experts, top 8: 40.9 us with four, 42.5 with eight
// in the down kernel; 12 tokens of 1024 x 1024, 64 experts, top 2: 13.4, 14.6 with eight in gate/up).
constexpr int kDeep = 4;
using Zero = std::integral_constant<int, 0>;
using One = std::integral_constant<int, 1>;
using Two = std::integral_constant<int, 2>;

static size_t gate_up_lds(int K, bool route, int R) { return (size_t)vec_total(K) + zero_bytes(R) + 32 + 512 + (route ? kRouter16MaxTopk * 8 : 0); }
static size_t down_lds(int topk, int per, int N, int parts, int R) { return (size_t)per * vec_total(N) + (size_t)topk * parts * 64 + zero_bytes(R); }

bool few_tokens_fit(int topk, int K, int N) {
  return K % 128 == 0 && N % 128 == 0 && gate_up_lds(K, true, kDeep) <= kFewLds && down_lds(topk, topk, N, 8, kDeep) <= kFewLds;
}

size_t few_act_bytes(long long slots, int N) { return (size_t)slots * vec_bytes(N); }
size_t few_unit_bytes(long long slots, int N) { return (size_t)slots * (N >> 5) * 8; }

int few_down_parts(int topk, int N) {
  const int parts = topk >= 8 ? 1 : topk >= 4 ? 2 : topk >= 2 ? 4 : 8, panels = (N + 1023) / 1024;
  return parts < panels ? parts : panels;
}

// Slots whose act lies in LDS at a time: all, unless they leave room for one workgroup on a CU and there are more workgroups than CUs:
// a few in a second round cost as much as a full one.  Then as many as let two workgroups in.  (80 random calls with 257 to 420 workgroups
// 1.08 times as fast from the cache, 1.07 from memory, none slower; one token of 4224 x 3456, 32 experts, top 6, 264 workgroups, bf16 42.1 -> 38.4 and
// 56.7 -> 49.5 us.)
static int few_down_slots(int T, int topk, int K, int N) {
  const int parts = few_down_parts(1, N);      // (an upper bound)
  if ((long long)K / 16 * T <= 256) return topk;
  for (int rounds = 1; rounds <= topk; ++rounds) {
    const int per = (topk + rounds - 1) / rounds;
    if (down_lds(topk, per, N, parts, kDeep) <= 80 * 1024) return per;
  }
  return topk;
}

// Dynamic LDS beyond 64 KB needs the kernel's attribute, remembered per device.
static int allow_lds(const void* kern, size_t lds, bool (&allowed)[64]) {
  if (lds <= 64 * 1024) return 0;
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return (int)err;
  if (dev >= 0 && dev < 64 && allowed[dev]) return 0;
  err = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kFewLds);
  if (err == hipSuccess && dev >= 0 && dev < 64) allowed[dev] = true;
  return (int)err;
}

template <int DT, int ROUTE, int R, int PRE, int KP>
static int gate_up(const void* X, const FewRoute& route, const int32_t* ids, const int32_t* qw, const void* s, const uint8_t* z, void* act,
                   uint32_t* units, int T, int topk, int E, int K, int N, hipStream_t stream) {
  static bool allowed[64] = {};
  const size_t lds = gate_up_lds(K, ROUTE, R);
  const int err = allow_lds(reinterpret_cast<const void*>(few_gate_up_kernel<DT, ROUTE, R, PRE, KP>), lds, allowed);
  if (err != 0) return err;
  hipLaunchKernelGGL((few_gate_up_kernel<DT, ROUTE, R, PRE, KP>), dim3(N / (64 / KP), T * topk), dim3(kGateThreads), lds, stream, (const uint16_t*)X, route, ids,
                     (const unsigned char*)qw, (const uint16_t*)s, z, (unsigned char*)act, units, topk, E, K, N);
  return (int)hipGetLastError();
}

template <int DT, int R, int PRE, int ROUNDS>
static int down(const void* act, const uint32_t* units, const int32_t* ids, const float* w, const int32_t* qw, const void* s, const uint8_t* z,
                void* out, int T, int topk, int per, int E, int K, int N, hipStream_t stream) {
  static bool allowed[64] = {};
  const int parts = few_down_parts(per, N), pairs = per * parts;
  const size_t lds = down_lds(topk, per, N, parts, R);
  auto kern = few_down_kernel<DT, R, PRE, ROUNDS>;
  const int err = allow_lds(reinterpret_cast<const void*>(kern), lds, allowed);
  if (err != 0) return err;
  hipLaunchKernelGGL(kern, dim3(K / 16, T), dim3(64 * (pairs < 8 ? pairs : 8)), lds, stream, (const unsigned char*)act, units, ids, w,
                     (const unsigned char*)qw, (const uint16_t*)s, z, (uint16_t*)out, topk, E, K, N, parts, per);
  return (int)hipGetLastError();
}

int launch_few_gate_up(const void* X, const FewRoute* route, const int32_t* ids, const int32_t* qw, const void* s, const uint8_t* z, void* act,
                       uint32_t* units, int T, int topk, int E, int K, int N, int dt, int pre, hipStream_t stream) {
  const FewRoute r = route ? *route : FewRoute{};
  auto with = [&](auto route_in, auto ordered, auto parts) {
    constexpr int RT = decltype(route_in)::value, PRE = decltype(ordered)::value, KP = decltype(parts)::value;
    return (dt == kF16 ? gate_up<kF16, RT, kDeep, PRE, KP> : gate_up<kBF16, RT, kDeep, PRE, KP>)(X, r, ids, qw, s, z, act, units, T, topk, E, K, N, stream);
  };
  auto pick = [&](auto route_in, auto parts) { return pre ? with(route_in, One{}, parts) : with(route_in, Zero{}, parts); };
  // 64 columns a workgroup, unless that leaves CUs without one, or a few with one more than the rest: then 32, and the reduction in halves.  (4 tokens of
  // 7168 x 2048, top 1, 128 workgroups of 64 columns: 25.5 -> 24.0 us; 16 tokens of 256 x 512, top 2, 256 of them: 8.2, in halves 9.1.  A half of less than
  // two groups is not worth its waves: 11 tokens of 256 x 512, 8.1, in halves 8.7; 4 tokens of 768 x 512, 8.0, in halves 7.5.  257 to 383 and 513 to 639 of
  // them, K 1024 and more: 180 random calls 1.05 times as fast from memory and 1.04 from the cache, 3 % slower at the worst (one token of 5248 x 7040, top 3, 330 of
  // them, 63.7 -> 55.1); 384 to 512 of them 0.98, with K below 1024 1.00 and from the cache 0.95.)
  const long long columns = (long long)N / 64 * T * topk;      // workgroups of 64
  const bool halves = columns < 256 ? K >= 512 : K >= 1024 && columns > 256 && columns < 640 && (columns - 1) % 256 < 127;
  if (route) return halves ? pick(One{}, Two{}) : pick(One{}, One{});
  return halves ? pick(Zero{}, Two{}) : pick(Zero{}, One{});
}

int launch_few_down(const void* act, const uint32_t* units, const int32_t* ids, const float* w, const int32_t* qw, const void* s, const uint8_t* z,
                    void* out, int T, int topk, int E, int K, int N, int dt, int pre, hipStream_t stream) {
  auto with = [&](auto ordered, auto in_rounds, int per) {
    constexpr int PRE = decltype(ordered)::value, ROUNDS = decltype(in_rounds)::value;
    return (dt == kF16 ? down<kF16, kDeep, PRE, ROUNDS> : down<kBF16, kDeep, PRE, ROUNDS>)(act, units, ids, w, qw, s, z, out, T, topk, per, E, K, N, stream);
  };
  const int per = few_down_slots(T, topk, K, N);
  if (per < topk) return pre ? with(One{}, One{}, per) : with(Zero{}, One{}, per);
  return pre ? with(One{}, Zero{}, topk) : with(Zero{}, Zero{}, topk);
}

}  // namespace moe
