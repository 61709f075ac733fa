// Grouped W4A16 GEMM for about 10 to 60 rows per expert: 64-slot blocks, 128 features per workgroup, three
// workgroups of four waves on a CU.  Used by the layer (group 128, K_in and N_out multiples of 1024), whose
// activations are stored in operand order beforehand, so that they go from memory to LDS without
// passing registers (on the 32-slot tile their way through registers was a seventh of the time: 16 of 115 vector
// instructions for 16 matrix instructions, and a second barrier per stage).
//
// A wave owns 32 features for all slots of the block.  A weight stage is 256 reduction indices: 128 bytes of every weight
// row, fetched into registers, then through a wave-private LDS tile to operand order; the activations one of their
// stages ahead, straight to LDS, with a barrier after each.  Up to two live parts an activation stage is 256 indices too and the
// weights run two stages ahead; from three on it is 128 (two buffers of 16 KB), so two barriers per weight stage, and
// the weights run one ahead (registers).  The kernel is specialised on the live 16-row parts of a block, so that up to 64 rows of an expert share one fetch and one unpack of its weights
// without paying for padding.  bf16 has no packed subtraction; the other tiles send the zero points through
// a second matrix instruction for every one.  Here the conversion unit produces the integers q and the zero points
// cost one float32 matrix instruction per four groups (see mid_tile): half the matrix instructions, 7 vector
// instructions a word, and smaller rounding errors, since no bias passes through the sums.
//
// Measured, former tiles -> this one, layer of 256 experts (K 7168, N 2048): fp16 512 tokens 1.30 -> 1.23 ms, 1024
// 1.67 -> 1.51; bf16 512 1.59 -> 1.29, 717 1.70 -> 1.41, 1024 1.89 -> 1.57; 8 experts (K 4096, N 14336), 64 tokens,
// fp16 175 -> 167 us.  What bounds it: gate/up at 22 rows takes 0.80 ms, without weight loads 0.53, without
// computation 0.67 (4.3 GB at 6.5 TB/s; a tenth more than the weights, scale lines that are fetched again);
// vector and matrix instructions of a SIMD share its issue and add up.  Not better: 64 features a wave on 32x32x16
// instructions with two workgroups on a CU (half the activation reads, 0.78 ms at 22 rows, but 8 % slower at 32
// and 64 rows).  Where the unpacking stands makes little difference: see `groups`.
#pragma once
#include "gemm_kernel.hpp"
#include "mid_order.hpp"

namespace moe {

struct MidParams {
  const void* A;             // [rows, K_in] 16-bit, runs of eight reordered (mid_unpack)
  const float* sums;         // bf16: [rows, K_in / 128] 16 times the sums of the row's groups (kZeroUnit); fp16: unused
  int row_div;
  const int32_t* qweight;
  const void* scales;
  const uint8_t* zeros;
  const int32_t* sorted_slot_ids;
  const int32_t* block_expert_ids;
  const int32_t* num_padded;
  int num_slots, E, N_out, K_in;
  void* C;                   // FUSE: act [num_slots, N_out / 2] 16-bit, runs of eight reordered; else float32 [num_slots, N_out]
  int n_tiles;               // 128-feature tiles of a block
  int tiles_per_wg;          // consecutive tiles one workgroup walks
  int k_splits, k_span;      // ranges of the reduction (whole panels of 1024), one workgroup each
  long long split_stride;    // float32 plane of a range: C + split * split_stride
};

constexpr int kMidRows = 64, kMidXBytes = 32768, kMidWBytes = 4096;      // activations (two buffers), weights per wave
constexpr int kMidSlots = kMidXBytes + 4 * kMidWBytes, kMidLds = kMidSlots + kMidRows * 4;
static_assert(kMidLds <= 64 * 1024, "no kernel attribute is needed for this much");

// A word's eight weights in the order of its activations.
//   fp16: the integers q - z, order 0,4,1,5,2,6,3,7.
//   bf16: the integers q, order 0,2,4,6,1,3,5,7: a byte that holds a nibble is the e4m3 code of q / 512 (linear
//         up to 15), which the conversion unit turns into bf16, two a time.  The zero points follow by the
//         rows' sums (see mid_tile).
template <int DT>
__device__ __forceinline__ u32x4 mid_unpack(uint32_t w, const DeqCtx<kF16, 0>& c, const UnpackConsts& k) {
  if constexpr (DT == kF16) {
    return dequant_word<kF16, 0>(w, c, k);
  } else {
    return nibbles_bf16(w);
  }
}

#define MID_FENCE()                       \
  {                                       \
    __builtin_amdgcn_sched_barrier(0);    \
    asm volatile("" ::: "memory");        \
  }
// vmcnt(n) (six bits, split 4 + 2), lgkmcnt(0), then the barrier
#define MID_BARRIER(VM)                                                                \
  {                                                                                    \
    MID_FENCE()                                                                        \
    __builtin_amdgcn_s_waitcnt(((VM) & 15) | (((VM) >> 4) << 14) | 0x70);              \
    __builtin_amdgcn_s_barrier();                                                      \
    MID_FENCE()                                                                        \
  }

// ML: live 16-row parts of the block
template <int DT, int FUSE, int PRE, int ML>
__device__ __forceinline__ void mid_tile(const MidParams& p, unsigned char* lds, int row0, int e, int tile0, int ntl, int split) {
  constexpr int XS = ML <= 2 ? 256 : 128;          // reduction indices per activation stage (two buffers of at most 16 KB)
  constexpr int XSTEPS = 256 / XS;                 // activation stages per weight stage
  constexpr int XP = XS * 2;                       // bytes per row and stage
  constexpr int XBUF = kMidXBytes / 2;
  constexpr int XQ = 16 * ML * XP / 4096;          // direct-to-LDS loads per wave and stage
  constexpr int RPQ = 1024 / XP;                   // rows per load
  constexpr int PDW = ML <= 2 ? 2 : 1;             // weight loads run this many stages ahead (registers)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 15, lj = lane >> 4;
  const int K_in = p.K_in, G = K_in >> 7;
  const int k0 = split * p.k_span, K_ext = K_in - k0 < p.k_span ? K_in - k0 : p.k_span;
  const int nst = K_ext >> 8, npan = K_ext >> 10;
  UnpackConsts uk;
  uk.or_hi = vgpr_const(0x64006400u);
  uk.or_lo = vgpr_const(0x54005400u);

  int* const slots = reinterpret_cast<int*>(lds + kMidSlots);
  if (tid < kMidRows) {
    const int s = p.sorted_slot_ids[row0 + tid];
    slots[tid] = s >= 0 && s < p.num_slots ? s : -1;
  }
  __syncthreads();
  auto arow_of = [&](int r) __attribute__((always_inline)) { const int s = slots[r]; return (uint32_t)(s < 0 ? 0 : s / p.row_div); };

  // ---- activations: global -> LDS.  A row's 256 bytes of a group are 16 chunks, chunk c at position c ^ (row & 15):
  // the 16 lanes an LDS cycle serves (16 rows) read 16 positions.
  typedef __attribute__((address_space(3))) void* lptr_t;
  uint32_t aoff[XQ];
  {
    const int pos = lane & (XP / 16 - 1);
#pragma unroll
    for (int q = 0; q < XQ; ++q) {
      const int r = (q * 4 + wave) * RPQ + lane / (64 / RPQ);
      aoff[q] = arow_of(r) * (uint32_t)(K_in * 2) + (uint32_t)k0 * 2u + 256u * (pos >> 4) + 16u * (uint32_t)((pos & 15) ^ (r & 15));
    }
  }
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void*)p.A, 0, (int)0xffffffffu, 0x00020000);
  int lx = 0;                                      // stage of the next activation load (every tile reads the same rows)
  const int nxst = K_ext / XS;
  auto dma_x = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < XQ; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lptr_t)(lds + buf * XBUF + (q * 4 + wave) * 1024), 16, (int)aoff[q], lx * XP, 0, 0);
    if (++lx == nxst) lx = 0;
  };
  const int xbase = ln * XP + 16 * ((4 * lj) ^ ln);      // + 16 mt XP + 256 u, ^ 16 i

  // ---- weights.  Feature f = 16 s + n of the wave: fused, 16 gate columns, then up; otherwise the even ones of
  // 32 columns, then the odd ones, so that a lane ends up with pairs.  Stated layout: eight contiguous rows
  // x 128 bytes per load, through a wave-private LDS tile; chunk c (0 .. 7) of LDS row r at position c ^ (r / 2 & 7), feature
  // f in row f (paired: f ^ s), so that the 16 lanes an LDS cycle serves hit different banks, reading and writing.
  // Offline repack: operand blocks straight to registers.
  unsigned char* const wsw = lds + kMidXBytes + wave * kMidWBytes;
  const unsigned char* const wbase = reinterpret_cast<const unsigned char*>(p.qweight) + (size_t)e * p.N_out * (size_t)(K_in >> 1) +
                                     (PRE ? (size_t)(k0 >> 7) * 1024 : (size_t)(k0 >> 1));
  const int half_n = p.N_out >> 1;
  // weight row of feature n of the wave's sub-tile s
  auto wrow_of = [&](int tile, int s, int n) __attribute__((always_inline)) {
    return (uint32_t)(FUSE ? s * half_n + tile * 64 + wave * 16 + n : tile * 128 + wave * 32 + 2 * n + s);
  };
  uint32_t woff[4];
  auto set_w_rows = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if constexpr (PRE) {       // load q: group q & 1 of sub-tile q >> 1
        const uint32_t r = wrow_of(tile, q >> 1, 0), blk = FUSE ? r >> 4 : ((r >> 5) << 1) | (uint32_t)(q >> 1);
        woff[q] = (blk * (uint32_t)G + (uint32_t)(q & 1)) * 1024u + (uint32_t)(lane * 16);
      } else {                   // load q: rows 8 q ... 8 q + 7 of the wave's 32
        const int rw = 8 * q + (lane >> 3);
        const uint32_t r = FUSE ? wrow_of(tile, rw >> 4, rw & 15) : (uint32_t)(tile * 128 + wave * 32 + rw);
        woff[q] = r * (uint32_t)(K_in >> 1) + (uint32_t)((lane & 7) * 16);
      }
    }
  };
  u32x4 wr[PDW][4];
  int ld_t = 0, ld_st = 0;
  auto load_w = [&](u32x4(&w)[4]) __attribute__((always_inline)) {
    const unsigned char* b = wbase + (size_t)ld_st * (PRE ? 2048 : 128);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      asm("" : "+v"(woff[q]));
      w[q] = load_weights<true>(b + woff[q]);
    }
    if (__builtin_expect(++ld_st == nst, 0)) {
      asm volatile("");
      ld_st = 0;
      if (++ld_t < ntl) set_w_rows(tile0 + ld_t);      // past the last tile its rows are read again
    }
  };
  const int wput = [&]() {
    const int r = lane >> 3, c = lane & 7, x = FUSE ? r : (r >> 1) ^ (r & 1);      // LDS row 8 q + x; paired: 16 s + 4 q + x
    return (FUSE ? r : 16 * (r & 1) + x) * 128 + 16 * (c ^ (x >> 1));
  }();
  auto put_w = [&](const u32x4(&w)[4]) __attribute__((always_inline)) {
    if constexpr (!PRE) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<u32x4*>(wsw + (FUSE ? (wput ^ (64 * (q & 1))) + 1024 * q : (wput ^ (32 * q)) + 512 * q)) = w[q];
    }
  };
  int wget[2];                                     // the lane's chunk of the first group, ^ 64 (second)
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int r = 16 * s + (FUSE ? ln : ln ^ s);
    wget[s] = r * 128 + 16 * (lj ^ ((r >> 1) & 7));
  }

  // ---- scales and zero points: panels of eight groups in registers, one panel ahead.  bf16: for the product of the
  // zero points, at the end of a panel, a lane fetches groups 2 j, 2 j + 1 in the middle of it: scales and
  // zero points of its features, sums of its rows.  Four parts have no registers for that (they spilled 10 to 21) and
  // fetch at the end: 3 to 5 % less at 48 to 63 rows per expert, the same or less with fewer parts.  3 to 13 are spilled still,
  // in fp16 with four parts and the stated layout 4 to 8.
  u32x4 s_cur[2], s_nxt[2];
  u32x2 z_cur[2], z_nxt[2];
  uint32_t sp[2], zp[2];
  floatx2_t rsum[ML];
  uint32_t sz_row[2], roff[ML];
  auto set_sz_rows = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 2; ++s) sz_row[s] = ((uint32_t)e * (uint32_t)p.N_out + wrow_of(tile, s, ln)) * (uint32_t)G + (uint32_t)(k0 >> 7);
  };
  if constexpr (DT == kBF16) {
#pragma unroll
    for (int mt = 0; mt < ML; ++mt) roff[mt] = arow_of(16 * mt + ln) * (uint32_t)G + (uint32_t)(k0 >> 7) + 2u * lj;
  }
  int sp_t = 0, sp_pan = 0;
  auto load_panel = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      s_nxt[s] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(p.scales) + sz_row[s] + 8 * sp_pan);
      if constexpr (DT == kF16) z_nxt[s] = *reinterpret_cast<const u32x2*>(p.zeros + sz_row[s] + 8 * sp_pan);
    }
    if (__builtin_expect(++sp_pan == npan, 0)) {
      asm volatile("");
      sp_pan = 0;
      if (++sp_t < ntl) set_sz_rows(tile0 + sp_t);
    }
  };
  uint32_t zo_row[2];        // bf16: the features' rows in the tile being multiplied
  auto set_zo_rows = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 2; ++s) zo_row[s] = ((uint32_t)e * (uint32_t)p.N_out + wrow_of(tile, s, ln)) * (uint32_t)G + (uint32_t)(k0 >> 7) + 2u * lj;
  };
  auto load_zero_operands = [&](int pan) __attribute__((always_inline)) {
    if constexpr (DT == kBF16) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        sp[s] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint16_t*>(p.scales) + zo_row[s] + 8 * pan);
        zp[s] = *reinterpret_cast<const uint16_t*>(p.zeros + zo_row[s] + 8 * pan);
      }
#pragma unroll
      for (int mt = 0; mt < ML; ++mt) rsum[mt] = *reinterpret_cast<const floatx2_t*>(p.sums + roff[mt] + 8 * pan);
    }
  };
  auto adopt_panel = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      s_cur[s] = s_nxt[s];
      if constexpr (DT == kF16) z_cur[s] = z_nxt[s] & 0x0f0f0f0fu;        // zero points are 4-bit by contract
    }
  };

  floatx4_t acc[ML][2];
#pragma unroll
  for (int mt = 0; mt < ML; ++mt)
#pragma unroll
    for (int s = 0; s < 2; ++s) acc[mt][s] = floatx4_t{0.f, 0.f, 0.f, 0.f};

  u32x4 wcur[4];            // PRE: the words of the stage being multiplied
  // NG consecutive groups of the panel from GP0 on (one activation stage).  Every word's unpack stands between the
  // matrix instructions of the word before it, and the sums of a group between those of the next.  (Unpacking a word before
  // its own matrix instructions, in separate blocks, takes the same time at 10 to 30 rows per expert and 1 to 2 %
  // less at 48 to 63, bf16.)
  auto groups = [&](auto gpc, int xbuf) __attribute__((always_inline)) {
    constexpr int GP0 = decltype(gpc)::value, NG = XS / 128;
    u32x4 w[2][NG];
    DeqCtx<kF16, 0> ctx[2];
    float scl[2][NG];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const int u = (GP0 + g) & 1;
        if constexpr (PRE) w[s][g] = wcur[2 * s + u];
        else w[s][g] = *reinterpret_cast<const u32x4*>(wsw + (wget[s] ^ (64 * u)));
      }
    }
    floatx4_t part[NG][ML][2];
    u32x4 a_nxt[ML], b_nxt[2];
    auto read_x = [&](int t) __attribute__((always_inline)) {
#pragma unroll
      for (int mt = 0; mt < ML; ++mt)
        a_nxt[mt] = *reinterpret_cast<const u32x4*>(lds + xbuf * XBUF + 16 * mt * XP + 256 * (t >> 2) + (xbase ^ (16 * (t & 3))));
    };
    auto unpack = [&](auto tc, int s) __attribute__((always_inline)) {
      constexpr int t = decltype(tc)::value, g = t >> 2, GP = GP0 + g;
      if constexpr ((t & 3) == 0) {
        if constexpr (DT == kF16) {
          ctx[s] = DeqCtx<kF16, 0>::from_panel(GP, s_cur[s][GP >> 1], z_cur[s][GP >> 2], z_cur[s][GP >> 2] << 4, uk);
          scl[s][g] = ctx[s].s;
        } else {
          scl[s][g] = __builtin_bit_cast(float, (GP & 1) ? (s_cur[s][GP >> 1] & 0xffff0000u) : (s_cur[s][GP >> 1] << 16));
        }
      }
      b_nxt[s] = mid_unpack<DT>(w[s][g][t & 3], ctx[s], uk);
    };
    auto add = [&](int g, int mt) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[mt][s][c] = __builtin_fmaf(scl[s][g], part[g][mt][s][c], acc[mt][s][c]);
      asm volatile("" : "+v"(acc[mt][0]), "+v"(acc[mt][1]));      // (here, not at the panel's end)
    };
    if constexpr (ML < 4) read_x(0);
    unpack(std::integral_constant<int, 0>{}, 0);
    unpack(std::integral_constant<int, 0>{}, 1);
    [&]<int... Ts>(std::integer_sequence<int, Ts...>) {
      (([&] {
         constexpr int t = Ts, g = t >> 2;
         u32x4 a[ML], b[2];
         if constexpr (ML == 4) read_x(t);      // (no registers for fragments ahead)
#pragma unroll
         for (int mt = 0; mt < ML; ++mt) a[mt] = a_nxt[mt];
#pragma unroll
         for (int s = 0; s < 2; ++s) b[s] = b_nxt[s];
         if constexpr (ML < 4 && t + 1 < 4 * NG) read_x(t + 1);
         __builtin_amdgcn_sched_barrier(0);
#pragma unroll
         for (int s = 0; s < 2; ++s) {
#pragma unroll
           for (int mt = 0; mt < ML; ++mt) part[g][mt][s] = mfma16x16x32<DT>(a[mt], b[s], (t & 3) == 0 ? floatx4_t{0.f, 0.f, 0.f, 0.f} : part[g][mt][s]);
           __builtin_amdgcn_sched_barrier(0);
           if constexpr (t + 1 < 4 * NG) unpack(std::integral_constant<int, t + 1>{}, s);
           if constexpr (g > 0 && (t & 3) == 0) {
             if (s < ML) add(g - 1, s);
             if (s + 2 < ML) add(g - 1, s + 2);
           }
           __builtin_amdgcn_sched_barrier(0);
         }
       }()),
       ...);
    }(std::make_integer_sequence<int, 4 * NG>{});
#pragma unroll
    for (int mt = 0; mt < ML; ++mt) add(NG - 1, mt);
  };

  auto store_tile = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
    for (int mt = 0; mt < ML; ++mt) {
      const u32x4 sl = *reinterpret_cast<const u32x4*>(slots + 16 * mt + 4 * lj);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int slot = (int)sl[c];
        if (slot < 0) continue;
        if constexpr (FUSE) {
          // round gate/up to the storage type first: the product is a 16-bit tensor by definition
          const float g = from_bits16<DT>(to_bits16<DT>(acc[mt][0][c])), u = from_bits16<DT>(to_bits16<DT>(acc[mt][1][c]));
          const int col = tile * 64 + wave * 16 + (ln & 8) + (DT == kF16 ? 2 * (ln & 3) + ((ln >> 2) & 1) : ((ln >> 1) & 3) + 4 * (ln & 1));
          reinterpret_cast<uint16_t*>(p.C)[(size_t)slot * half_n + col] = to_bits16<DT>(silu_f32(g) * u);
        } else {
          float* dst = reinterpret_cast<float*>(p.C) + (size_t)split * p.split_stride + (size_t)slot * p.N_out + tile * 128 + wave * 32 + 2 * ln;
          *reinterpret_cast<floatx2_t*>(dst) = floatx2_t{acc[mt][0][c], acc[mt][1][c]};
        }
      }
    }
#pragma unroll
    for (int mt = 0; mt < ML; ++mt)
#pragma unroll
      for (int s = 0; s < 2; ++s) acc[mt][s] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  };

  // ---- pipeline.  Activations run one of their stages ahead (two buffers), weights PDW stages; one barrier per
  // activation stage.  Every step sends its activations before its weights, so the wait for the former
  // leaves the latter in flight.
  set_w_rows(tile0);
  set_sz_rows(tile0);
  if constexpr (DT == kBF16) set_zo_rows(tile0);
  dma_x(0);
  load_panel();
#pragma unroll
  for (int d = 0; d < PDW; ++d) load_w(wr[d]);
  adopt_panel();
  put_w(wr[0]);
  if constexpr (!PRE && PDW == 1) load_w(wr[0]);
  MID_BARRIER(0)

  int c_t = 0, c_pan = 0;
  const int trips = ntl * npan;
  for (int trip = 0; trip < trips; ++trip) {
    [&]<int... Rs>(std::integer_sequence<int, Rs...>) {
      (([&] {
         constexpr int r = Rs / XSTEPS, h = Rs % XSTEPS;      // weight stage of the panel, activation stage in it
         constexpr int buf = Rs & 1;
         MID_FENCE()
         if constexpr (r == 2 && h == 0) {
           if constexpr (ML < 4) load_zero_operands(c_pan);
           load_panel();
         }
         dma_x(buf ^ 1);
         MID_FENCE()
         if constexpr (h == 0) {
           if constexpr (PRE) {
#pragma unroll
             for (int q = 0; q < 4; ++q) wcur[q] = wr[r % PDW][q];
             load_w(wr[r % PDW]);
           } else if constexpr (PDW == 2) {
             load_w(wr[r % PDW]);
           }
         }
         MID_FENCE()
         groups(std::integral_constant<int, 2 * r + h>{}, buf);
         if constexpr (h == XSTEPS - 1 && !PRE) {
           put_w(wr[(r + 1) % PDW]);
           if constexpr (PDW == 1) load_w(wr[0]);
         }
         // (activations sent last in this step unless weights followed them)
         MID_BARRIER((h == 0 && (PRE || PDW == 2)) || (h == XSTEPS - 1 && !PRE && PDW == 1) ? 4 : 0)
       }()),
       ...);
    }(std::make_integer_sequence<int, 4 * XSTEPS>{});
    if constexpr (DT == kBF16) {
      if constexpr (ML == 4) load_zero_operands(c_pan);
      // the panel's zero points: four groups per instruction, float32 operands (scale * z / 16 stays in range, see kZeroUnit)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const float sz = -__builtin_bit_cast(float, h ? sp[s] & 0xffff0000u : sp[s] << 16) * ((float)((zp[s] >> (8 * h)) & 15u) * (1.f / kZeroUnit));
#pragma unroll
          for (int mt = 0; mt < ML; ++mt) acc[mt][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(rsum[mt][h], sz, acc[mt][s], 0, 0, 0);
        }
    }
    adopt_panel();
    if (++c_pan == npan) {
      store_tile(tile0 + c_t);
      c_pan = 0;
      ++c_t;
      if constexpr (DT == kBF16) set_zo_rows(tile0 + (c_t < ntl ? c_t : ntl - 1));
    }
  }
  __builtin_amdgcn_s_waitcnt(0x70 | 0xF00);        // vmcnt(0): no direct-to-LDS load outlives the workgroup
}

template <int DT, int FUSE, int PRE>
__global__ void __launch_bounds__(256, 3)
w4a16_mid_kernel(const MidParams p) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int tgroups = (p.n_tiles + p.tiles_per_wg - 1) / p.tiles_per_wg;
  const int nwork = tgroups * p.k_splits;
  int blk, work;
  if (!mid_work(blockIdx.x, *p.num_padded / kMidRows, nwork, blk, work)) return;
  const int row0 = blk * kMidRows, split = work % p.k_splits, tile0 = work / p.k_splits * p.tiles_per_wg;
  const int ntl = p.n_tiles - tile0 < p.tiles_per_wg ? p.n_tiles - tile0 : p.tiles_per_wg;
  const int e = p.block_expert_ids[blk];
  if (e < 0 || e >= p.E) return;
  const int slot = p.sorted_slot_ids[row0 + (threadIdx.x & 63)];
  const unsigned long long any = __ballot(slot >= 0 && slot < p.num_slots);
  const int parts = any ? (64 - __builtin_clzll(any) + 15) / 16 : 0;
  switch (__builtin_amdgcn_readfirstlane(parts)) {
    case 1: mid_tile<DT, FUSE, PRE, 1>(p, smem, row0, e, tile0, ntl, split); break;
    case 2: mid_tile<DT, FUSE, PRE, 2>(p, smem, row0, e, tile0, ntl, split); break;
    case 3: mid_tile<DT, FUSE, PRE, 3>(p, smem, row0, e, tile0, ntl, split); break;
    case 4: mid_tile<DT, FUSE, PRE, 4>(p, smem, row0, e, tile0, ntl, split); break;
    default: break;
  }
}

// Launchers (one translation unit per 16-bit type); a hipError_t.
int launch_mid_f16(const MidParams& p, int fuse, int pre, int grid, hipStream_t stream);
int launch_mid_bf16(const MidParams& p, int fuse, int pre, int grid, hipStream_t stream);

}  // namespace moe
