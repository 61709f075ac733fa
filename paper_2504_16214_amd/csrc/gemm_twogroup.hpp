// Grouped W4A16 GEMM for large batches: 256 slots x 256 features per workgroup, two wave groups in turn
// on the matrix unit.  Used by the layer (group 128, K_in and N_out multiples of 1024), whose
// activations are stored with every run of eight reduction indices in the order 0,4,1,5,2,6,3,7 (the
// order the nibble unpack produces), so that they go from memory to LDS without passing registers.
//
// Eight waves; wave w owns 32 features for all slots of the block, so each packed weight is unpacked
// once per workgroup; waves w and w + 4 share a SIMD and belong to different groups.  A stage is one
// quantisation group (128 reduction indices, eight packed words per lane, one word per
// v_mfma_f32_32x32x16).  A stage's words are dealt to phases of 7 to 12 matrix instructions: a load phase
// (activation fragments from LDS, the words' unpack, the accumulators' rescale, loads of later stages)
// and a matrix phase, a barrier after each.  The second group runs one phase behind the first: on
// every SIMD one wave multiplies while the other unpacks and loads.  Phases are balanced when neither
// side is longer than eight 32-cycle instructions; 16x16x32 instructions in the same schedule lose
// about 90 cycles per phase to the barrier (16 cycles of work cover it instead of 32) and read each
// operand register twice as often.
//
// The kernel is specialised on the live 32-slot parts of a block (ML), so that a block costs what its
// rows cost; 256-slot blocks then fetch and unpack an expert's weights once per 256 rows.  Up to 64 rows
// its loads come as whole lines through LDS (STREAM below); at 22 rows per expert (bf16, K 7168, N 2048) neither
// side is at its limit: 4.7 TB/s fetched, matrix unit busy 21 % of the cycles, vector unit 49 % (such batches of large
// weights run on the 64-slot tile).  Above it is
// bound by power: at 128 rows the matrix unit is busy 56 % of the cycles at 1.77 GHz (2.4 nominal); without the
// fragment reads from LDS the cycles stay the same and the clock rises to 2.0 GHz (1860 -> 1558 us), without
// weight loads likewise (1607 us).
// Measured, eight-wave 128-slot tile -> this one, gate/up product of 256 experts (K 7168, N 2048), fp16:
// 128 rows per expert 2.09 -> 1.87 ms (even counts; 2.06 with drawn routing), 160 rows 2.87 -> 2.22, 192 rows
// 3.23 -> 2.54, 64 rows 1.32 -> 1.17; layer at 4096 tokens fp16 4.03 -> 3.60 ms, bf16 5.44 -> 4.26 ms.  With its
// stores by offset and four (act: two) columns wide instead of one, with a branch for each: fp16 3.64 -> 3.49 ms, bf16 4.30 -> 4.25.
#pragma once
#include "gemm_kernel.hpp"

namespace moe {

struct TwoGroupParams {
  const void* A;             // [rows, K_in] 16-bit, runs of eight reordered
  const float* bias_rows;    // bf16: [rows, K_in / 128] 47 * (sum of the row's group); fp16: unused
  int row_div;
  const int32_t* qweight;
  const void* scales;
  const uint8_t* zeros;
  const int32_t* sorted_slot_ids;
  const int32_t* block_expert_ids;
  const int32_t* num_padded;
  int num_slots, E, N_out, K_in;
  void* C;                   // FUSE: act [num_slots, N_out / 2] 16-bit, runs of eight reordered; else float32 [num_slots, N_out]
  uint32_t c_bytes;          // bytes of C; 0: rows are stored with a branch (c_plane_bytes)
  int n_tiles;               // 256-feature tiles of a block
  int tiles_per_wg;          // consecutive tiles one workgroup walks
  int pre;                   // 1: qweight in the operand order of the offline repack
};

typedef float floatx16_t __attribute__((ext_vector_type(16)));
template <int DT>
__device__ __forceinline__ floatx16_t mfma32x32x16(const u32x4& a, const u32x4& b, floatx16_t c) {
  if constexpr (DT == kF16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

template <int ML>
struct TwoGroupGeom {
  static constexpr int WPP = ML == 1 ? 8 : ML <= 3 ? 4 : ML <= 6 ? 2 : 1;   // words per phase: 7 ... 12 matrix instructions
  static constexpr int PH = 8 / WPP;                        // phase pairs per stage
  // Up to 64 rows the launch is bound by the weight stream: weights go to LDS as whole 128-byte lines
  // (two stages at a time, three buffers, private to a wave) and the waves run free between one
  // barrier per stage.  Above, weights come straight to registers and the wave groups take turns.
  static constexpr bool STREAM = ML <= 2;
  static constexpr int NBUF = ML == 2 || ML == 5 ? 3 : ML <= 4 ? 4 : 2;
  static constexpr int STAGE = 32 * ML * 256;
  static constexpr int RROWS = ML > 4 ? 256 : 128;          // rows of the row-sum ring
  static constexpr int SR = RROWS / 32;                     // row sums: rows per wave and step
  static constexpr int ROFF = NBUF * STAGE;                 // ring of four groups of four stages
  static constexpr int TOFF = ROFF + 4 * RROWS * 16;        // slot of every tile row
  // Stores by offset hold on to more registers than a block of six parts or more has left (91 spilled instead of 9 at eight: gate/up of 2921 slots
  // by 3 on 120 experts, K 1024, N 6144, 456 -> 562 us).
  static constexpr bool BY_OFFSET = ML <= 5;
  static constexpr int OOFF = TOFF + 256 * 4;               // BY_OFFSET: its offset in C (c_bytes)
  static constexpr int ZOFF = OOFF + (BY_OFFSET ? 256 * 4 : 0);      // zeros, as large as one group of the ring
  static constexpr int WOFF = ZOFF + RROWS * 16;            // STREAM: three buffers of 256 rows x 128 bytes
  static constexpr int LDS = WOFF + (STREAM ? 3 * 32768 : 0);
  static_assert(LDS <= 160 * 1024, "LDS");
};

#define TG_FENCE()                        \
  {                                       \
    __builtin_amdgcn_sched_barrier(0);    \
    asm volatile("" ::: "memory");        \
  }
#define TG_BARRIER()                      \
  {                                       \
    TG_FENCE()                            \
    __builtin_amdgcn_s_barrier();         \
    TG_FENCE()                            \
  }
constexpr int tg_waitcnt(int vm, bool lg) { return (vm & 15) | ((vm >> 4) << 14) | 0x70 | (lg ? 0 : 0xF00); }

template <int DT>
struct TgCtx {
  uint32_t c0, c1;      // fp16: packed (1024 + z), (64 + z); bf16: packed 32.0 + 15 - z, unused
};

// One packed word -> 8 sixteen-bit floats in the order 0,4,1,5,2,6,3,7.  fp16: the integers q - z (see
// dequant_word).  bf16: 47 + (q - z), between 32 and 62, exact in 8 significant bits; the constant is
// the same for every feature, so the accumulators' rescale, which is a multiplication anyway, takes 47
// times the group's row sum away in the same instruction.  (The smallest constant whose range stays
// in one binade; 143 = 128 + 15 saves nothing and triples the rounding error of the sums.)
template <int DT>
__device__ __forceinline__ u32x4 tg_unpack(uint32_t w, const TgCtx<DT>& c, const UnpackConsts& k) {
  uint32_t r[4];
  if constexpr (DT == kF16) {
    const uint32_t w8 = w >> 8;
    const half2_t zA = __builtin_bit_cast(half2_t, c.c0), zB = __builtin_bit_cast(half2_t, c.c1);
    r[0] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, (w & 0x000F000Fu) | k.or_hi) - zA);
    r[1] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, (w & 0x00F000F0u) | k.or_lo) - zB);
    r[2] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, (w8 & 0x000F000Fu) | k.or_hi) - zA);
    r[3] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, (w8 & 0x00F000F0u) | k.or_lo) - zB);
  } else {
    // (nibbles at mantissa bits 2 .. 5 of 32.0)
    const uint32_t w8 = w >> 8;
    r[0] = ((w & 0x000F000Fu) << 2) + c.c0;
    r[1] = ((w >> 2) & 0x003C003Cu) + c.c0;
    r[2] = ((w8 & 0x000F000Fu) << 2) + c.c0;
    r[3] = ((w8 >> 2) & 0x003C003Cu) + c.c0;
  }
  return u32x4{r[0], r[1], r[2], r[3]};
}

template <int DT, int FUSE, int ML>
__device__ __forceinline__ void
tg_tile(const TwoGroupParams& p, unsigned char* lds, int row0, int e, int tile0, int ntl) {
  using G = TwoGroupGeom<ML>;
  constexpr int NBUF = G::NBUF, SR = G::SR, WPP = G::WPP, PH = G::PH;
  constexpr int PDW = ML >= 7 ? 2 : 4;       // weight loads run this many stages ahead (registers)
  constexpr int UNR = 4;                     // stages per trip: one scale panel of four groups
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, lh = lane >> 5;
  const int K_in = p.K_in, nst = K_in >> 7;
  UnpackConsts uk;
  uk.or_hi = vgpr_const(0x64006400u);
  uk.or_lo = vgpr_const(0x54005400u);

  int* const slots = reinterpret_cast<int*>(lds + G::TOFF);
  uint32_t* const out_rows = reinterpret_cast<uint32_t*>(lds + G::OOFF);
  if (tid < 256) {
    const int s = tid < 32 * ML ? p.sorted_slot_ids[row0 + tid] : -1;
    slots[tid] = s >= 0 && s < p.num_slots ? s : -1;
    if constexpr (G::BY_OFFSET) out_rows[tid] = s >= 0 && s < p.num_slots ? (uint32_t)s * (uint32_t)p.N_out * (FUSE ? 1u : 4u) : kNoRow;
  }
  if (DT == kBF16 && tid < G::RROWS) *reinterpret_cast<u32x4*>(lds + G::ZOFF + tid * 16) = u32x4{0, 0, 0, 0};
  __syncthreads();
  auto arow_of = [&](int r) __attribute__((always_inline)) { const int s = slots[r]; return s < 0 ? 0 : s / p.row_div; };

  // ---- activations: global -> LDS.  A row's 256 bytes per stage are 16 chunks, chunk c at position
  // c ^ (row & 15): the 16 lanes an LDS cycle serves (16 rows, different modulo 16) read 16 positions.
  typedef __attribute__((address_space(3))) void* lptr_t;
  uint32_t aoff[ML];
  {
    const int rl = 4 * wave + (lane >> 4), ch = (lane & 15) ^ (rl & 15);
#pragma unroll
    for (int q = 0; q < ML; ++q) aoff[q] = (uint32_t)arow_of(32 * q + rl) * (uint32_t)(K_in * 2) + 16u * (uint32_t)ch;
  }
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void*)p.A, 0, (int)0xffffffffu, 0x00020000);
  const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void*)p.bias_rows, 0, (int)0xffffffffu, 0x00020000);
  auto dma_a = [&](int buf, int q, int st) __attribute__((always_inline)) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lptr_t)(lds + buf + (32 * q + 4 * wave) * 256), 16, (int)aoff[q], st * 256, 0, 0);
  };
  // Row sums (bf16): four groups at a time, SR rows per wave and step, four steps bring all; a block
  // of SR rows is [4 groups][SR rows], so a lane reads its four rows with one load.
  auto sum_row = [&](int t) __attribute__((always_inline)) { return arow_of(((t & 3) * 8 + wave) * SR + (lane & (SR - 1))); };
  auto dma_r = [&](int t, int st, int row) __attribute__((always_inline)) {      // t: flattened step, st: its stage in the row
    if (lane < 4 * SR)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rr, (lptr_t)(lds + G::ROFF + ((t >> 2) & 3) * (G::RROWS * 16) + ((t & 3) * 8 + wave) * (SR * 16)), 4,
          (row * nst + (st & ~3) + lane / SR) * 4, 0, 0, 0);
  };

  // ---- weights: operand order straight from memory.  Lane (n, h) multiplies feature n; word w of its
  // q-th load holds reduction indices 64 q + 32 h + 8 w + [0, 8) of the stage.
  const unsigned char* const wbase = reinterpret_cast<const unsigned char*>(p.qweight) + (size_t)e * p.N_out * (size_t)(K_in >> 1);
  const int wstep = p.pre ? 1024 : 64, qstep = p.pre ? 512 : 32;
  const int half_n = p.N_out >> 1;
  uint32_t woff, sz_row;
  uint32_t wdma[4];                          // STREAM: the lane's rows 8 i + lane / 8 of the wave's 32
  auto wrow_of = [&](int tile, int n) __attribute__((always_inline)) {
    // (fused: lane n & 15 takes the feature whose act lies at that position, runs of eight in operand order: neighbouring lanes
    // store neighbouring columns)
    return FUSE ? (n >> 4) * half_n + tile * 128 + wave * 16 + (n & 8) + ((n >> 1) & 3) + 4 * (n & 1) : tile * 256 + wave * 32 + n;
  };
  // 16-byte chunk j (0 .. 3) of a stage of weight row wrow, bytes from wbase
  auto w_at = [&](uint32_t wrow, uint32_t st, uint32_t j) __attribute__((always_inline)) -> uint32_t {
    // (operand-order blocks hold 16 consecutive rows, or the even / odd ones of 32)
    const uint32_t blk = FUSE ? wrow >> 4 : ((wrow >> 5) << 1) | (wrow & 1), n = FUSE ? wrow & 15 : (wrow >> 1) & 15;
    return p.pre ? (blk * (uint32_t)nst + st) * 1024u + j * 256u + n * 16u : wrow * (uint32_t)(K_in >> 1) + st * 64u + j * 16u;
  };
  auto set_w_rows = [&](int tile) __attribute__((always_inline)) {
    if constexpr (G::STREAM) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int n = 8 * i + (lane >> 3), c = (lane & 7) ^ ((n >> 1) & 7);
        wdma[i] = w_at((uint32_t)wrow_of(tile, n), (uint32_t)(c >> 2), (uint32_t)(c & 3));
      }
    } else {
      woff = w_at((uint32_t)wrow_of(tile, ln), 0u, (uint32_t)lh);
    }
  };
  auto set_sz_rows = [&](int tile) __attribute__((always_inline)) {
    sz_row = ((uint32_t)e * (uint32_t)p.N_out + (uint32_t)wrow_of(tile, ln)) * (uint32_t)nst;
  };
  u32x4 wr[PDW][2];
  int ld_t = 0, ld_st = 0;
  auto load_w = [&](u32x4(&w)[2]) __attribute__((always_inline)) {
    const unsigned char* b = wbase + (size_t)ld_st * wstep;
    asm("" : "+v"(woff));
    w[0] = *reinterpret_cast<const u32x4*>(b + woff);
    w[1] = *reinterpret_cast<const u32x4*>(b + qstep + woff);
    if (__builtin_expect(++ld_st == nst, 0)) {
      asm volatile("");
      ld_st = 0;
      if (++ld_t < ntl) set_w_rows(tile0 + ld_t);      // past the last tile its rows are read again
    }
  };
  // STREAM: row n of the wave's 32 keeps its chunk c (0 .. 7 of two stages) at position c ^ (n / 2 & 7), so
  // that the 16 lanes an LDS cycle serves read 16 positions
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)wbase, 0, (int)0xffffffffu, 0x00020000);
  auto dma_w = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      asm("" : "+v"(wdma[i]));
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lptr_t)(lds + G::WOFF + buf + wave * 4096 + i * 1024), 16, (int)wdma[i], ld_st * wstep, 0, 0);
    }
    ld_st += 2;
    if (__builtin_expect(ld_st == nst, 0)) {
      asm volatile("");
      ld_st = 0;
      if (++ld_t < ntl) set_w_rows(tile0 + ld_t);
    }
  };
  const int wpos = G::WOFF + wave * 4096 + ln * 128 + 16 * (lh ^ ((ln >> 1) & 7));      // ^ 16 * (4 (stage & 1) + 2 q)
  int wbuf0 = 0, wbuf1 = 32768, wbuf2 = 65536;      // buffers of the pair being multiplied, the next, the one after

  // ---- scales and zero points: panels of four groups in registers, one panel ahead
  u32x2 s_cur, s_nxt;
  uint32_t z_cur, z_nxt;
  int sp_t = 0, sp_g = 0;
  auto load_sz = [&]() __attribute__((always_inline)) {
    s_nxt = *reinterpret_cast<const u32x2*>(reinterpret_cast<const uint16_t*>(p.scales) + sz_row + sp_g);
    z_nxt = *reinterpret_cast<const uint32_t*>(p.zeros + sz_row + sp_g);
    sp_g += 4;
    if (__builtin_expect(sp_g == nst, 0)) {
      asm volatile("");
      sp_g = 0;
      if (++sp_t < ntl) set_sz_rows(tile0 + sp_t);
    }
  };

  // ---- prologue ----
  set_w_rows(tile0);
  set_sz_rows(tile0);
  load_sz();
  int la_st = 0;                                    // stage of the next activation load
  int bufs[NBUF];
#pragma unroll
  for (int b = 0; b < NBUF; ++b) bufs[b] = b * G::STAGE;
  int lr_st = 0, rt = 0, rrow = 0;                  // row sums: stage, flattened step, row of the next load
  if constexpr (DT == kBF16) {
#pragma unroll
    for (int t = 0; t < 8; ++t) dma_r(t, t, sum_row(t));
    rt = 8; lr_st = 8 == nst ? 0 : 8;
    rrow = sum_row(0);
  }
#pragma unroll
  for (int b = 0; b < NBUF - 1; ++b) {
#pragma unroll
    for (int q = 0; q < ML; ++q) dma_a(bufs[b], q, la_st);
    if (++la_st == nst) la_st = 0;
  }
  if constexpr (G::STREAM) {
    dma_w(wbuf0);
    dma_w(wbuf1);
  } else {
#pragma unroll
    for (int d = 0; d < PDW; ++d) load_w(wr[d]);
  }
  __builtin_amdgcn_s_waitcnt(tg_waitcnt(0, true));
  TG_BARRIER()
  if (!G::STREAM && wave >= 4) TG_BARRIER()

  floatx16_t acc[ML];
  float unit = 1.f;                                 // scale the accumulators are expressed in
#pragma unroll
  for (int mt = 0; mt < ML; ++mt)
#pragma unroll
    for (int c = 0; c < 16; ++c) acc[mt][c] = 0.f;

  const int abase = ln * 256 + 16 * ((4 * lh) ^ (ln & 15));      // + 8192 mt, ^ 16 * (8 q + w)
  int gst = 0;                                      // flattened stage

  // accumulator register c of a lane: row 8 (c >> 2) + 4 h + (c & 3) of the sub-tile, feature n
  auto store_tile = [&](int tile) __attribute__((always_inline)) {
    if (G::BY_OFFSET && p.c_bytes) {
      const __amdgpu_buffer_rsrc_t rc = c_rows(p.C, p.c_bytes);
      const bool odd = lane & 1;
#pragma unroll
      for (int mt = 0; mt < ML; ++mt) {
#pragma unroll
        for (int c4 = 0; c4 < 4; ++c4) {
          const uint32_t* const rows = out_rows + mt * 32 + 8 * c4 + 4 * lh;
          if constexpr (FUSE) {
            // (see below; then neighbouring lanes put their columns together: one row of two each)
            uint32_t v[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const auto sw = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, acc[mt][4 * c4 + 2 * h] * unit),
                                                               __builtin_bit_cast(uint32_t, acc[mt][4 * c4 + 2 * h + 1] * unit), false, false);
              const float g = from_bits16<DT>(to_bits16<DT>(__builtin_bit_cast(float, (uint32_t)sw[0])));
              const float u = from_bits16<DT>(to_bits16<DT>(__builtin_bit_cast(float, (uint32_t)sw[1])));
              v[h] = to_bits16<DT>(silu_f32(g) * u);
            }
            const uint32_t at = rows[2 * (lane & 1) + ((lane >> 4) & 1)] + (uint32_t)(tile * 128 + wave * 16 + (lane & 14)) * 2u;
            __builtin_amdgcn_raw_buffer_store_b32(pair_columns(v[0], v[1], odd), rc, (int)at, 0, 0);
          } else {
            // four lanes exchange four rows of their columns: a lane then stores four columns of one row
            uint32_t v[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = __builtin_bit_cast(uint32_t, acc[mt][4 * c4 + c] * unit);
            const bool two = lane & 2;
            const uint32_t g0 = from_neighbour(odd ? v[0] : v[1]), g1 = from_neighbour(odd ? v[2] : v[3]);
            const uint32_t r0 = odd ? g0 : v[0], r1 = odd ? v[1] : g0, r2 = odd ? g1 : v[2], r3 = odd ? v[3] : g1;      // columns of a pair: (r0, r1) of row 0 or 1, (r2, r3) of row 2 or 3
            const uint32_t h0 = from_pair(two ? r0 : r2), h1 = from_pair(two ? r1 : r3);
            const uint32_t at = rows[lane & 3] + (uint32_t)(tile * 256 + wave * 32 + (ln & ~3)) * 4u;
            __builtin_amdgcn_raw_buffer_store_b128(two ? u32x4{h0, h1, r2, r3} : u32x4{r0, r1, h0, h1}, rc, (int)at, 0, 0);
          }
        }
      }
    } else {
#pragma unroll
    for (int mt = 0; mt < ML; ++mt) {
#pragma unroll
      for (int c4 = 0; c4 < 4; ++c4) {
        const u32x4 sl = *reinterpret_cast<const u32x4*>(slots + mt * 32 + 8 * c4 + 4 * lh);
        if constexpr (FUSE) {
#pragma unroll
          for (int c = 0; c < 4; c += 2) {
            // lanes 16 .. 31 (up) of one register change places with lanes 0 .. 15 (gate) of the next:
            // a lane then holds gate and up of one row and column
            const auto sw = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, acc[mt][4 * c4 + c] * unit),
                                                             __builtin_bit_cast(uint32_t, acc[mt][4 * c4 + c + 1] * unit), false, false);
            const int slot = (int)((lane & 16) ? sl[c + 1] : sl[c]);
            // round gate/up to the storage type first: the product is a 16-bit tensor by definition
            const float g = from_bits16<DT>(to_bits16<DT>(__builtin_bit_cast(float, (uint32_t)sw[0])));
            const float u = from_bits16<DT>(to_bits16<DT>(__builtin_bit_cast(float, (uint32_t)sw[1])));
            const int col = tile * 128 + wave * 16 + (lane & 15);
            if (slot >= 0) reinterpret_cast<uint16_t*>(p.C)[(size_t)slot * half_n + col] = to_bits16<DT>(silu_f32(g) * u);
          }
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const int slot = (int)sl[c];
            if (slot >= 0)
              reinterpret_cast<float*>(p.C)[(size_t)slot * p.N_out + tile * 256 + wave * 32 + ln] = acc[mt][4 * c4 + c] * unit;
          }
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(tg_waitcnt(0, false));
    }
#pragma unroll
    for (int mt = 0; mt < ML; ++mt)
#pragma unroll
      for (int c = 0; c < 16; ++c) acc[mt][c] = 0.f;
    unit = 1.f;
  };

  // operand constants of a group from its panel; returns the group's scale.  w: the words unpacked with them.
  auto group_ctx = [&](const u32x2& sp, uint32_t zp, int g, TgCtx<DT>& ctx, u32x4(&w)[2]) __attribute__((always_inline)) -> float {
    const uint32_t zz = (zp >> (8 * g)) & 0xfu;      // zero points are 4-bit by contract
    const uint32_t sb = (sp[g >> 1] >> (16 * (g & 1))) & 0xffffu;
    if constexpr (DT == kF16) {
      ctx.c0 = 0x64006400u + zz * 0x00010001u;
      ctx.c1 = 0x54005400u + zz * 0x00100010u;
    } else {
      ctx.c0 = 0x423c423cu - zz * 0x00040004u;
    }
    const float sc = from_bits16<DT>((uint16_t)sb);
    if (__builtin_expect(__ballot(sc == 0.f) != 0ull, 0)) {
      // rare: a group with scale 0 contributes exactly nothing; a real branch.  fp16: q == z everywhere.
      // bf16: operands 0.0, and the caller takes no row sums away (47 * sum from the matrix unit and
      // from the row sums are not added in the same order, so they would not cancel)
      asm volatile("" ::: "memory");
      const uint32_t zw = DT == kF16 ? zz * 0x11111111u : 0u;
      if (sc == 0.f) {
        w[0] = w[1] = u32x4{zw, zw, zw, zw};
        if constexpr (DT == kBF16) ctx.c0 = 0u;
      }
    }
    return sc;
  };
  // Before the barrier at which the first group first reads stage g + 1 every wave has waited for its
  // part of it; the loads sent after it (at least kWait) may stay in flight.
  constexpr int kWait = G::STREAM ? (NBUF - 2) * ML + 4 : (NBUF - 2) * (ML + 2) + 2;
  int c_t = 0, c_st = 0;
  const int trips = ntl * (nst / UNR);
  for (int trip = 0; trip < trips; ++trip) {
    s_cur = s_nxt;
    z_cur = z_nxt;
    load_sz();
    [&]<int... Rs>(std::integer_sequence<int, Rs...>) {
      (([&] {
         constexpr int r = Rs;
         float rs = 1.f;
         // bf16: 47 * (row sum) of the lane's 16 rows of a sub-tile, from `sums` on (zeros: scale 0)
         floatx4_t nr[4];
         int sums = 0;
         auto load_sums = [&](int mt) __attribute__((always_inline)) {
           if constexpr (DT == kBF16) {
#pragma unroll
             for (int c4 = 0; c4 < 4; ++c4) {
               const int row = mt * 32 + 8 * c4 + 4 * lh;
               nr[c4] = *reinterpret_cast<const floatx4_t*>(
                   lds + sums + (row / SR) * (SR * 16) + r * (SR * 4) + (row & (SR - 1)) * 4);
             }
           }
         };
         auto rescale = [&](int mt) __attribute__((always_inline)) {
#pragma unroll
           for (int c = 0; c < 16; ++c) {
             if constexpr (DT == kBF16) acc[mt][c] = __builtin_fmaf(acc[mt][c], rs, -nr[c >> 2][c & 3]);      // (negated addend: keeps the result in acc's register)
             else acc[mt][c] *= rs;
           }
         };
         u32x4(&w)[2] = wr[r % PDW];
         TgCtx<DT> ctx;
#pragma unroll
         for (int ph = 0; ph < PH; ++ph) {
           const int i0 = ph * WPP;
           // the first kEarly sub-tiles are rescaled in the first load phase, the others between the matrix
           // instructions of the phase (bf16: two, its row sums are register-hungry)
           constexpr int kEarly = DT == kBF16 && ML >= 6 ? 2 : (ML + 1) / 2;
           // ---- load phase ----
           u32x4 a[WPP][ML], bw[WPP];
#pragma unroll
           for (int i = 0; i < WPP; ++i) {
             const int k = i0 + i, ab = (abase ^ (16 * (8 * (k >> 2) + (k & 3)))) + bufs[0];
#pragma unroll
             for (int mt = 0; mt < ML; ++mt) a[i][mt] = *reinterpret_cast<const u32x4*>(lds + ab + mt * 8192);
           }
           if constexpr (G::STREAM) {
             if (ph == 0) {
#pragma unroll
               for (int q = 0; q < 2; ++q) w[q] = *reinterpret_cast<const u32x4*>(lds + (wpos ^ (16 * (4 * (r & 1) + 2 * q))) + wbuf0);
             }
           }
           // loads of later stages: activations first
#pragma unroll
           for (int q = 0; q < ML; ++q)
             if ((PH == 1 ? 0 : q * (PH - 1) / ML) == ph) dma_a(bufs[NBUF - 1], q, la_st);
           if constexpr (G::STREAM && (r & 1) == 0) {
             if (ph == PH - 1) dma_w(wbuf2);
           }
           if (ph == 0) {
             if constexpr (DT == kBF16) { dma_r(rt, lr_st, rrow); rrow = sum_row(rt + 1); }
             const float sc = group_ctx(s_cur, z_cur, r, ctx, w);
             rs = sc == 0.f ? 1.f : unit * __builtin_amdgcn_rcpf(sc);
             unit = sc == 0.f ? unit : sc;
             if constexpr (DT == kBF16) sums = sc == 0.f ? G::ZOFF : G::ROFF + ((gst >> 2) & 3) * (G::RROWS * 16);
           }
#pragma unroll
           for (int i = 0; i < WPP; ++i) bw[i] = tg_unpack<DT>(w[(i0 + i) >> 2][(i0 + i) & 3], ctx, uk);
           if (ph == 0) {
#pragma unroll
             for (int mt = 0; mt < kEarly; ++mt) {
               load_sums(mt);
               rescale(mt);
               if constexpr (DT == kBF16 && ML >= 6) __builtin_amdgcn_sched_barrier(0);
             }
             if constexpr (kEarly < ML) load_sums(kEarly);
           }
           if (!G::STREAM && ph == PH - 1) load_w(w);      // this stage's words are used up
           __builtin_amdgcn_sched_barrier(0);
           if (ph == PH - 1) __builtin_amdgcn_s_waitcnt(tg_waitcnt(kWait, true));
           else __builtin_amdgcn_s_waitcnt(tg_waitcnt(63, true));
           if (!G::STREAM || ph == PH - 1) TG_BARRIER()
           // ---- matrix phase ----
           if (!G::STREAM) __builtin_amdgcn_s_setprio(1);
#pragma unroll
           for (int i = 0; i < WPP; ++i) {
#pragma unroll
             for (int mt = 0; mt < ML; ++mt) {
               acc[mt] = mfma32x32x16<DT>(a[i][mt], bw[i], acc[mt]);
               if (ph == 0 && i == 0 && mt + kEarly < ML) {
                 __builtin_amdgcn_sched_barrier(0);
                 rescale(mt + kEarly);
                 if (mt + kEarly + 1 < ML) load_sums(mt + kEarly + 1);
                 __builtin_amdgcn_sched_barrier(0);
               }
             }
           }
           if constexpr (!G::STREAM) {
             __builtin_amdgcn_s_setprio(0);
             TG_BARRIER()
           }
         }
         if constexpr (G::STREAM && (r & 1) == 1) {
           const int t1 = wbuf0;
           wbuf0 = wbuf1; wbuf1 = wbuf2; wbuf2 = t1;
         }
         // the buffer just read takes the stage sent next
         const int t0 = bufs[0];
#pragma unroll
         for (int q = 0; q + 1 < NBUF; ++q) bufs[q] = bufs[q + 1];
         bufs[NBUF - 1] = t0;
         if (++la_st == nst) la_st = 0;
         if constexpr (DT == kBF16) {
           ++rt;
           if (++lr_st == nst) lr_st = 0;
         }
         ++gst;
       }()),
       ...);
    }(std::make_integer_sequence<int, UNR>{});
    c_st += UNR;
    if (c_st == nst) {
      store_tile(tile0 + c_t);
      c_st = 0;
      ++c_t;
    }
  }
  if (!G::STREAM && wave < 4) TG_BARRIER()
  __builtin_amdgcn_s_waitcnt(tg_waitcnt(0, false));      // no direct-to-LDS load outlives the workgroup
}

template <int DT, int FUSE>
__global__ void __launch_bounds__(512, 1)
w4a16_twogroup_kernel(const TwoGroupParams p) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int tgroups = (p.n_tiles + p.tiles_per_wg - 1) / p.tiles_per_wg;
  const int L = xcd_contiguous_index(blockIdx.x, (*p.num_padded / 256) * tgroups);
  if (L < 0) return;
  const int tile0 = (L % tgroups) * p.tiles_per_wg;
  const int ntl = p.n_tiles - tile0 < p.tiles_per_wg ? p.n_tiles - tile0 : p.tiles_per_wg;
  const int blk = L / tgroups, row0 = blk * 256;
  const int e = p.block_expert_ids[blk];
  if (e < 0 || e >= p.E) return;
  int live = 0;                                     // the slots of a block are packed at its front
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int s = p.sorted_slot_ids[row0 + 32 * i];
    live += s >= 0 && s < p.num_slots ? 1 : 0;
  }
  switch (__builtin_amdgcn_readfirstlane(live)) {
    case 1: tg_tile<DT, FUSE, 1>(p, smem, row0, e, tile0, ntl); break;
    case 2: tg_tile<DT, FUSE, 2>(p, smem, row0, e, tile0, ntl); break;
    case 3: tg_tile<DT, FUSE, 3>(p, smem, row0, e, tile0, ntl); break;
    case 4: tg_tile<DT, FUSE, 4>(p, smem, row0, e, tile0, ntl); break;
    case 5: tg_tile<DT, FUSE, 5>(p, smem, row0, e, tile0, ntl); break;
    case 6: tg_tile<DT, FUSE, 6>(p, smem, row0, e, tile0, ntl); break;
    case 7: tg_tile<DT, FUSE, DT == kBF16 ? 8 : 7>(p, smem, row0, e, tile0, ntl); break;      // (bf16: seven would spill registers)
    case 8: tg_tile<DT, FUSE, 8>(p, smem, row0, e, tile0, ntl); break;
    default: break;
  }
}

constexpr int kTwoGroupLds = TwoGroupGeom<2>::LDS;
static_assert(TwoGroupGeom<1>::LDS <= kTwoGroupLds && TwoGroupGeom<2>::LDS <= kTwoGroupLds && TwoGroupGeom<4>::LDS <= kTwoGroupLds && TwoGroupGeom<5>::LDS <= kTwoGroupLds && TwoGroupGeom<7>::LDS <= kTwoGroupLds && TwoGroupGeom<8>::LDS <= kTwoGroupLds, "LDS");

// Launchers (one translation unit per 16-bit type); a hipError_t.
int launch_twogroup_f16(const TwoGroupParams& p, int fuse, int grid, hipStream_t stream);
int launch_twogroup_bf16(const TwoGroupParams& p, int fuse, int grid, hipStream_t stream);

}  // namespace moe
