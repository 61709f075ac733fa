// Blockwise-scaled FP8 GEMM for gfx950:
//   C[m, n] = sum_kb a_scale[m, kb] * b_scale[n / 128, kb] * sum_{k in block kb} A[m, k] * B[n, k]
// A [M, K], B [N, K] e4m3 codes (OCP), scales float32, one reduction block = 128 = the depth of one
// v_mfma_f32_16x16x128_f8f6f4, so every matrix instruction starts from a zero accumulator and its
// result is folded into the float32 accumulator with one scaled FMA per register.
//
// Mapping.  A workgroup of WM x WN waves owns BM rows of A ("tokens") and BN rows of B ("features").
// The features are the matrix instruction's row operand and the tokens its column operand, so a
// lane ends up with one token and runs of its features: 16-byte stores, one activation scale
// per lane and row block.
//   * Both operands go global -> LDS with direct-to-LDS loads (global_load_lds_dwordx4: no staging
//     registers, no ds_write) -> operand registers.  The global side is fully coalesced (eight lanes
//     per 128-byte row block); operand-order loads straight from global memory (one row per lane)
//     cost the texture path four times the cycles and were the bottleneck of a first version.  LDS
//     rows are 128 bytes with their 16-byte chunks XOR-swizzled by the row index (the swizzle is
//     applied on the global side: which chunk a lane fetches), a ring of NS buffers (two in every
//     compiled variant), one barrier per reduction block; every wave waits for its own loads of the
//     next block (vmcnt) before that barrier.
//   * The order of the 128 reduction indices inside an instruction is free as long as both
//     operands use the same one: lane group j takes bytes [16 j, +16) and [64 + 16 j, +16) of a row.
//   * The activation scales of a block travel through LDS with the tile (one 4-byte direct-to-LDS
//     load per token).
//   * Split reduction: blockIdx also selects a range of reduction blocks; split i writes plane i
//     of a float32 buffer and a second kernel adds the planes in order and rounds once.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "fp8_gemm.hpp"

namespace fp8 {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
// two float32 -> two 16-bit values in a word, round to nearest even (one v_cvt_pk_bf16_f32, or two
// v_cvt_f16_f32 and a pack)
template <int BF16>
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  if constexpr (BF16) return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
  else return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), f16x2));
}

// Workgroup = WM x WN waves; wave (wm, wn) owns tokens [16 MT wm, 16 MT (wm + 1)) and features
// [16 NT wn, 16 NT (wn + 1)) of the BM x BN tile (BM = 16 MT WM, BN = 16 NT WN).
template <int WM, int WN, int MT, int NT, int NS>
struct Geom {
  static constexpr int T = 64 * WM * WN;                 // threads
  static constexpr int BM = 16 * MT * WM, BN = 16 * NT * WN;
  static constexpr int RPP = T / 8;                      // tile rows one pass of the workgroup loads
  static constexpr int AROWS = (BM + RPP - 1) / RPP * RPP;   // activation rows held in LDS (padded to whole passes)
  static constexpr int CHA = AROWS / RPP, CHB = BN / RPP;    // 16-byte chunks per thread and block
  static constexpr int SCALES = T;                          // activation-scale slots: one per thread (slots past BM repeat the last row)
  static constexpr int STAGE = (AROWS + BN) * 128 + SCALES * 4;  // bytes: A rows, B rows, activation scales
  static constexpr int LDS = NS * STAGE;                    // NS buffers: NS - 1 blocks in flight
  static constexpr int LPB = CHA + CHB + 1;                 // vector-memory loads per wave and block
  static_assert(BM <= T, "one activation scale per thread");
  static_assert(LPB * (NS - 2) <= 63, "vmcnt is six bits");
  static_assert(BN % RPP == 0, "feature tile must be whole passes");
};

// Which of a wave's 16 NT features LDS row q (operand row q & 15 of sub-tile q >> 4) holds.  Lane group j of a token
// ends up with operand rows 4 j ... 4 j + 3 of every sub-tile.  The rows are dealt so that the four groups' 16 bytes
// of one store lie side by side, 64 bytes of a token: float32 stores a sub-tile at a time (the identity), 16-bit types
// two.  (With 4 NT consecutive features in a lane a store touched every fourth or second 16 bytes: float32 tiles, written
// only, 3.3 TB/s against 5.4.  Grouped 256 x 256 tile, 256 rows for each of 256 experts, K 2048, N 7168, float32, 1600 ->
// 1430 us; FP8 layer, 4096 tokens, 256 experts 3.09 -> 3.05 ms, 64 experts, K 2048, N 1408 457 -> 428 us; dense the same.)
template <int NT>
__device__ __forceinline__ int feature_of_row(int q, bool f32) {
  const int nt = q >> 4, l = q & 15;
  return NT == 1 || f32 ? q : 32 * (nt >> 1) + 8 * (l >> 2) + 4 * (nt & 1) + (l & 3);
}

// Row block mb and feature block nb of tile L inside a split.  Tiles are walked in groups of group_m row
// blocks: feature block by feature block inside a group, so that the workgroups that run together share
// both their A rows and their B rows.  Row blocks of different experts share no B rows: a group without two
// blocks of one expert goes row block by row block, and an XCD works on all feature blocks of one or two
// experts, whose rows of A stay in its L2 (FP8 layer of 256 experts, K 7168, N 2048: 4096 tokens 3.19 -> 3.07 ms,
// 128 tokens 1.90 -> 1.88; in that order whatever the experts, 267 tokens of skewed routing took 571 for 505 us).
__device__ __forceinline__ void tile_of(const GemmParams& p, bool grouped, int m_blocks, int n_blocks, int L, int& mb, int& nb) {
  const int per_group = p.group_m * n_blocks, grp = L / per_group, rem = L - grp * per_group, m0 = grp * p.group_m;
  const int m_in = m_blocks - m0 < p.group_m ? m_blocks - m0 : p.group_m;
  bool share = !grouped;
  for (int i = 1; i < m_in && !share; ++i) share = p.block_expert_ids[m0 + i] == p.block_expert_ids[m0 + i - 1];
  nb = share ? rem / m_in : rem % n_blocks;
  mb = m0 + (share ? rem % m_in : rem / n_blocks);
}

// Lane group j's share of a token's 16 NT features (see feature_of_row) in the output type (p.out_bf16: 0 fp16, 1 bf16,
// 2 float32); at: the first of them.
template <int NT>
__device__ __forceinline__ void store_row(const GemmParams& p, size_t at, int j, const f32x4 (&v)[NT]) {
  if (p.k_splits > 1 || p.out_bf16 == 2) {      // a partial plane, or the result itself
    float* dst = reinterpret_cast<float*>(p.C) + at + 4 * j;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) *reinterpret_cast<f32x4*>(dst + 16 * nt) = v[nt];
    return;
  }
  uint32_t w[2 * NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    if (p.out_bf16 == 1) {
      w[2 * nt] = pack2<1>(v[nt][0], v[nt][1]);
      w[2 * nt + 1] = pack2<1>(v[nt][2], v[nt][3]);
    } else {
      w[2 * nt] = pack2<0>(v[nt][0], v[nt][1]);
      w[2 * nt + 1] = pack2<0>(v[nt][2], v[nt][3]);
    }
  }
  uint16_t* dst = reinterpret_cast<uint16_t*>(p.C) + at + (NT == 1 ? 4 : 8) * j;
  if constexpr (NT == 1) {
    *reinterpret_cast<u32x2*>(dst) = u32x2{w[0], w[1]};
  } else {
#pragma unroll
    for (int h = 0; h < NT / 2; ++h)
      *reinterpret_cast<u32x4*>(dst + 32 * h) = u32x4{w[4 * h], w[4 * h + 1], w[4 * h + 2], w[4 * h + 3]};
  }
}

// KG > 1: KG groups of WM x WN waves share the tile, each with a part of the reduction and its own ring of buffers;
// their sums meet in LDS (dense, unsplit launches).
template <int WM, int WN, int MT, int NT, int NS, int KG = 1>
__global__ void __launch_bounds__(64 * WM * WN * KG, (WM * WN * KG == 4 && MT * NT <= 16 ? 2 : 1))
fp8_blockwise_gemm_kernel(const GemmParams p) {
  using G = Geom<WM, WN, MT, NT, NS>;
  constexpr int T = G::T, BM = G::BM, BN = G::BN, RPP = G::RPP, AROWS = G::AROWS, CHA = G::CHA, CHB = G::CHB;
  extern __shared__ __attribute__((aligned(16))) unsigned char all_lds[];

  const int kgroup = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / T);
  unsigned char* const lds = all_lds + kgroup * G::LDS;
  const int tid = KG == 1 ? (int)threadIdx.x : (int)threadIdx.x - kgroup * T, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave - wm * WN;
  const int ln = lane & 15, lj = lane >> 4;

  // hardware block id -> logical tile: consecutive ids go round the 8 XCDs, so give every XCD a
  // contiguous range of tiles.  The grouped launch is sized for the bucketing capacity; its ranges
  // are cut over the row blocks that really exist (num_padded), so the unused capacity does not
  // leave the last XCDs without work, and the surplus workgroups exit here.
  const bool grouped = p.sorted_slot_ids != nullptr;
  const int n_blocks = p.N / BN;
  const int m_blocks = grouped ? *p.num_padded / BM : (p.M + BM - 1) / BM;
  const int total = grouped ? m_blocks * n_blocks : (int)gridDim.x;
  int L;
  {
    const int id = blockIdx.x, q = total >> 3, r = total & 7, x = id & 7, idx = id >> 3;
    if (idx >= q + (x < r ? 1 : 0)) return;       // (uniform over the workgroup: nobody reaches a barrier)
    L = x * q + (x < r ? x : r) + idx;
  }
  const int split = L / (m_blocks * n_blocks);
  L -= split * (m_blocks * n_blocks);
  int mb, nb;
  tile_of(p, grouped, m_blocks, n_blocks, L, mb, nb);
  const int row0 = mb * BM;                       // first token of the tile
  const int n0 = nb * BN;                         // first feature of the tile
  const int KB = p.K >> 7;
  const int kb0 = KG == 1 ? split * p.kb_per_split : kgroup * KB / KG;
  int kb1 = KG == 1 ? kb0 + p.kb_per_split : (kgroup + 1) * KB / KG;
  if (kb1 > KB) kb1 = KB;
  const int nkb = kb1 - kb0;                      // >= 1 by construction of the grid
  const int trips = KG == 1 ? nkb : (KB + KG - 1) / KG;      // (every group meets every barrier)

  // ---- global -> LDS: direct-to-LDS loads (no staging registers, no ds_write) ----
  // LDS row r keeps its chunk c at position c ^ (r & 7): the operand reads below (16 rows, one
  // chunk position per lane group) then touch every bank group once.  One load instruction of a
  // wave fills 1 KiB of LDS in lane order = 8 rows x 8 positions; the lane at position s of row r
  // therefore fetches chunk s ^ (r & 7) of that row.  Pass i of the workgroup covers tile rows
  // [RPP i, RPP (i + 1)), wave w rows 8 w .. 8 w + 7 of the pass.
  const int srow = tid >> 3, sc = tid & 7;
  const uint8_t* Bmat = p.B;
  const float* bsmat = p.b_scale;
  if (grouped) {
    // row blocks past the bucketed slots, and blocks without an expert, have nothing to do
    // (uniform over the workgroup: nobody reaches a barrier)
    if (row0 >= *p.num_padded) return;
    const int e = p.block_expert_ids[mb];
    if (e < 0) return;
    Bmat += (size_t)e * p.b_expert_stride;
    bsmat += (size_t)e * p.bs_expert_stride;
  }
  // A row behind a tile row: dense = the row itself (rows past the matrix repeat its last row and
  // are never stored); grouped = slot / row_div (padding rows read row 0)
  auto a_row_of = [&](int r) __attribute__((always_inline)) -> int {
    if (grouped) {
      const int slot = p.sorted_slot_ids[row0 + r];
      return (slot >= 0 && slot < p.num_slots) ? slot / p.row_div : 0;
    }
    const int g = row0 + r;
    return g >= p.M ? p.M - 1 : g;
  };
  const bool f32 = KG > 1 || p.k_splits > 1 || p.out_bf16 == 2;      // a partial sum, or the result itself
  uint32_t aoff[CHA], boff[CHB];                  // byte offsets from A / B (host checks they fit 32 bits)
#pragma unroll
  for (int i = 0; i < CHA; ++i) {
    int r = srow + RPP * i;
    if (r >= BM) r = BM - 1;                      // LDS rows past the token tile (padding of the pass) repeat its last row
    aoff[i] = (uint32_t)a_row_of(r) * (uint32_t)p.K + 16u * (sc ^ (srow & 7));
  }
#pragma unroll
  for (int i = 0; i < CHB; ++i) {
    const int r = srow + RPP * i, q = r % (16 * NT);
    boff[i] = (uint32_t)(n0 + r - q + feature_of_row<NT>(q, f32)) * (uint32_t)p.K + 16u * (sc ^ (srow & 7));
  }
  // activation scale of tile row tid (threads past BM repeat the last row)
  const float* assrc = p.a_scale + (size_t)a_row_of(tid < BM ? tid : BM - 1) * KB;
  const float* bssrc = bsmat + (size_t)((n0 + wn * 16 * NT) >> 7) * KB;      // wave-uniform

  // ---- operand read positions ----
  const int xrow = wm * 16 * MT + ln;             // + 16 mt
  const int xpos = 16 * (lj ^ (ln & 7));          // tile rows are multiples of 16 apart: (row & 7) == (ln & 7)
  const int wpos0 = (AROWS + wn * 16 * NT + ln) * 128 + xpos;      // + 2048 nt

  f32x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

  float sb[NS];               // weight-block scale of the block in each LDS buffer

  typedef const __attribute__((address_space(1))) void* gptr_t;
  typedef __attribute__((address_space(3))) void* lptr_t;
  auto dma_block = [&](int buf, int kb) __attribute__((always_inline)) {
    const uint8_t* ab = p.A + (size_t)kb * 128;
    const uint8_t* bb = Bmat + (size_t)kb * 128;
    unsigned char* st = lds + buf * G::STAGE + 1024 * wave;            // this wave's 8 rows of every pass
#pragma unroll
    for (int i = 0; i < CHB; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(bb + boff[i]), (lptr_t)(st + (AROWS + RPP * i) * 128), 16, 0, 0);
#pragma unroll
    for (int i = 0; i < CHA; ++i)
      __builtin_amdgcn_global_load_lds((gptr_t)(ab + aoff[i]), (lptr_t)(st + RPP * i * 128), 16, 0, 0);
    __builtin_amdgcn_global_load_lds((gptr_t)(assrc + kb),
                                     (lptr_t)(lds + buf * G::STAGE + (AROWS + BN) * 128 + 256 * wave), 4, 0, 0);
    sb[buf] = bssrc[kb];
  };
  auto read_op = [&](const unsigned char* st, int off) __attribute__((always_inline)) -> i32x8 {
    // chunk positions c and c ^ 4 of the row: reduction indices [16 lj, +16) and [64 + 16 lj, +16)
    const i32x4 lo = *reinterpret_cast<const i32x4*>(st + off);
    const i32x4 hi = *reinterpret_cast<const i32x4*>(st + (off ^ 64));
    return i32x8{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
  };
  i32x8 wa[NT];
  float sp[MT];                // a_scale * b_scale of the lane's token in every row block
  auto read_w = [&](int ring) __attribute__((always_inline)) {
    const unsigned char* st = lds + ring * G::STAGE;
    const float* ss = reinterpret_cast<const float*>(st + (AROWS + BN) * 128) + xrow;
    const float bs = sb[ring];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) sp[mt] = ss[16 * mt] * bs;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) wa[nt] = read_op(st, wpos0 + 2048 * nt);
  };
  // row blocks [MLO, MHI) of the tile against the wave's NT weight operands
  auto compute = [&](int ring, auto mlo, auto mhi) __attribute__((always_inline)) {
    constexpr int MLO = decltype(mlo)::value, MHI = decltype(mhi)::value;
    const unsigned char* st = lds + ring * G::STAGE;
    // software pipeline: the activation operand of row block mt + 1 is read from LDS, and the
    // partial sums of row block mt - 1 are folded into the accumulators, while row block mt is
    // in the matrix unit
    i32x8 xa = read_op(st, (xrow + 16 * MLO) * 128 + xpos);
    f32x4 pprev[NT];
#pragma unroll
    for (int mt = MLO; mt < MHI; ++mt) {
      i32x8 xn = xa;
      if (mt + 1 < MHI) xn = read_op(st, (xrow + 16 * (mt + 1)) * 128 + xpos);
      f32x4 part[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        part[nt] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
            wa[nt], xa, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0, 0, 0, 0);   // e4m3 x e4m3, no block exponents
      if (mt > MLO) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt - 1][nt] += pprev[nt] * sp[mt - 1];
      }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) pprev[nt] = part[nt];
      xa = xn;
      // Instruction order.  Left to itself the scheduler gathers every FMA of the block at its
      // end, which keeps all partial sums alive.  An empty asm that takes the accumulators just
      // updated and the next activation operand ties them together: the matrix instructions of
      // row block mt + 1 cannot start before the FMAs of row block mt - 1 are done.
      if (mt > MLO) {
        if constexpr (NT == 4)
          asm volatile("" : "+v"(acc[mt - 1][0]), "+v"(acc[mt - 1][1]), "+v"(acc[mt - 1][2]), "+v"(acc[mt - 1][3]), "+v"(xa));
        else if constexpr (NT == 2)
          asm volatile("" : "+v"(acc[mt - 1][0]), "+v"(acc[mt - 1][1]), "+v"(xa));
        else
          asm volatile("" : "+v"(acc[mt - 1][0]), "+v"(xa));
      }
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[MHI - 1][nt] += pprev[nt] * sp[MHI - 1];
  };
  using std::integral_constant;
  // vmcnt(n): at most n of this wave's vector-memory loads still in flight (six bits, split 4 + 2)
  constexpr int kLanded = ((G::LPB * (NS - 2)) & 15) | (((G::LPB * (NS - 2)) >> 4) << 14) | 0x0F70;
  // One block.  Buffer cur is multiplied; the block NS - 1 ahead is sent to the buffer that was
  // multiplied last (every wave is past the barrier that followed it); before the closing barrier
  // each wave waits until its own part of the NEXT block has landed.
  auto stage = [&](auto cur_c, int kb_far, bool live) __attribute__((always_inline)) {
    constexpr int cur = decltype(cur_c)::value;
    if (KG == 1 || live) {
      read_w(cur);
      __builtin_amdgcn_sched_barrier(0);       // the LDS reads above are issued before the far block's loads
      dma_block((cur + NS - 1) % NS, kb_far);
      __builtin_amdgcn_sched_barrier(0);
      compute(cur, integral_constant<int, 0>{}, integral_constant<int, MT>{});
    }
    __builtin_amdgcn_s_waitcnt(kLanded);
    __syncthreads();
  };

  // ---- pipeline: NS - 1 blocks in flight while one is multiplied ----
  // (block indices past the end are clamped: a valid block is loaded and never consumed, so every
  // wave issues the same number of loads per stage and the vmcnt arithmetic holds)
  auto clampk = [&](int i) __attribute__((always_inline)) { return kb0 + (i < nkb ? i : nkb - 1); };
#pragma unroll
  for (int s = 0; s < NS - 1; ++s) dma_block(s, clampk(s));
  __builtin_amdgcn_s_waitcnt(kLanded);
  __syncthreads();
  for (int it = 0; it < trips; it += NS) {
    stage(integral_constant<int, 0>{}, clampk(it + NS - 1), it < nkb);
    if constexpr (NS >= 2) { if (it + 1 < trips) stage(integral_constant<int, 1>{}, clampk(it + NS), it + 1 < nkb); }
    if constexpr (NS >= 3) { if (it + 2 < trips) stage(integral_constant<int, 2>{}, clampk(it + NS + 1), it + 2 < nkb); }
    if constexpr (NS >= 4) { if (it + 3 < trips) stage(integral_constant<int, 3>{}, clampk(it + NS + 2), it + 3 < nkb); }
  }
  if constexpr (KG > 1) {
    // the groups' sums (operand rows are features in order, see f32), added in the order of the reduction
    static_assert(BM * BN * 4 <= G::LDS, "a group's sums fit in its buffers");
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) *reinterpret_cast<f32x4*>(lds + ((xrow + 16 * mt) * BN + wn * 16 * NT + 16 * nt + 4 * lj) * 4) = acc[mt][nt];
    __syncthreads();
    for (int q = threadIdx.x; q < BM * BN / 4; q += T * KG) {
      const int t = q / (BN / 4), f = 4 * (q % (BN / 4));
      if (row0 + t >= p.M) continue;
      f32x4 v = *reinterpret_cast<const f32x4*>(all_lds + 16 * q);
#pragma unroll
      for (int g = 1; g < KG; ++g) v += *reinterpret_cast<const f32x4*>(all_lds + g * G::LDS + 16 * q);
      const size_t at = (size_t)(row0 + t) * p.N + n0 + f;
      if (p.out_bf16 == 2) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p.C) + at) = v;
      else
        *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(p.C) + at) =
            p.out_bf16 == 1 ? u32x2{pack2<1>(v[0], v[1]), pack2<1>(v[2], v[3])} : u32x2{pack2<0>(v[0], v[1]), pack2<0>(v[2], v[3])};
    }
    return;
  }

  // ---- epilogue: the lane's token ----
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    int t = row0 + xrow + 16 * mt;               // dense: the token; grouped: the slot behind the tile row
    if (grouped) {
      t = p.sorted_slot_ids[t];
      if (t < 0 || t >= p.num_slots) continue;   // padding row
    } else if (t >= p.M) {
      continue;
    }
    store_row<NT>(p, ((size_t)split * p.M + t) * p.N + n0 + wn * 16 * NT, lj, acc[mt]);
  }
}

// ---- the 256 x 256 tile: two wave groups in turn on the matrix unit -------------------------------
// Eight waves, two groups of four; a wave owns 64 features and every other 16-row sub-tile of the
// workgroup's rows, waves w and w + 4 (one of each group) share a SIMD.  A reduction block is worked
// off in clusters of two sub-tiles per wave (64 rows of the tile): a load phase (operand reads from
// LDS, direct-to-LDS loads of later blocks) and a matrix phase (eight matrix instructions, each
// followed by the scaled FMAs of the one three before it), a barrier after each.  The second group
// runs one phase behind the first: on every SIMD one wave multiplies while the other loads.
//
// ML = live sub-tiles per wave (1 .. 8): rows past the matrix, or past an expert's slots, cost
// nothing beyond the rounding to 32 rows.  The feature rows' operands stay in registers for a block.
//
// Why this shape.  Matrix instructions and the scaled FMAs (four per instruction) overlap fully when
// they come from different waves of a SIMD or are three instructions apart; run in lockstep between
// two barriers per block, as the former 256 x 256 tile did, the waves read LDS together, wait
// together and sit in the wait states between an instruction and its own FMAs (matrix unit busy 41 %
// of 4980 cycles per block).  In turns it is busy 57 % (8192^3, 2.14 GHz) and 51 % (4096 x 51200 x 5120, 1.84 GHz):
// the clock is power-limited.
// Measured, former tile -> this one: 4096 x 51200 x 5120 1.18 -> 1.00 ms (1.82 -> 2.15 PFLOP/s), 8192^3
// 0.51 -> 0.46 ms; FP8 layer of 256 experts at 4096 tokens (128-slot blocks on the 128 x 128 tile
// before): gate/up product 2.44 -> 1.65 ms (4.5 TB/s of weights, each fetched once), layer 4.21 ->
// 3.09 ms.  What is left: dense, the exposed stores of a round (110 of 1020 us) and power; grouped, loads (half
// of the wave cycles wait, 2.1 GHz, matrix unit busy 25 %).
template <int ML>
struct PingGeom {
  static constexpr int T = 512, BM = 256, BN = 256, NT = 4;
  static constexpr int C = (ML + 1) / 2;                   // clusters per block
  static constexpr int NBUF = C <= 2 ? 3 : 2;              // operand buffers
  static constexpr int ROWS = C <= 2 ? 128 : 256;          // tile rows a buffer has room for
  static constexpr int BOFF = ROWS * 128;
  static constexpr int STAGE = BOFF + BN * 128;            // bytes per buffer: A rows, B rows
  static constexpr int SR = ROWS / 32;                     // scale rows per wave and step
  static constexpr int SOFF = NBUF * STAGE;                // activation scales: ring of four groups of four blocks
  static constexpr int TOFF = SOFF + 4 * ROWS * 16;        // A row behind every tile row
  static constexpr int OOFF = TOFF + ROWS * 4;             // row of C behind every tile row, -1: none
  static constexpr int LDS = OOFF + ROWS * 4;
  static_assert(LDS <= 160 * 1024, "LDS");
};
constexpr int kPingLds = PingGeom<4>::LDS > PingGeom<8>::LDS ? PingGeom<4>::LDS : PingGeom<8>::LDS;

#define FP8_PHASE_FENCE()                 \
  {                                       \
    __builtin_amdgcn_sched_barrier(0);    \
    asm volatile("" ::: "memory");        \
  }
#define FP8_PHASE_BARRIER()               \
  {                                       \
    FP8_PHASE_FENCE()                     \
    __builtin_amdgcn_s_barrier();         \
    FP8_PHASE_FENCE()                     \
  }
// vmcnt(n) (six bits, split 4 + 2), lgkmcnt(0) if lg
constexpr int waitcnt_imm(int vm, bool lg) { return (vm & 15) | ((vm >> 4) << 14) | 0x70 | (lg ? 0 : 0xF00); }

// One tile.  row0: first row (dense) or first slot-table entry (grouped); B, bs: the tile's weight
// matrix and block scales; [kb0, kb0 + nkb): its reduction blocks.
template <int ML>
__device__ __forceinline__ void
ping_tile(const GemmParams& p, unsigned char* lds, int row0, int n0, const uint8_t* B, const float* bs, int kb0, int nkb,
          int split) {
  using G = PingGeom<ML>;
  constexpr int NT = G::NT, C = G::C, NBUF = G::NBUF, BN = G::BN, SR = G::SR;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int ln = lane & 15, lj = lane >> 4;
  const bool grouped = p.sorted_slot_ids != nullptr;
  const int KB = p.K >> 7;

  // A row behind a tile row: dense = the row itself (rows past the matrix repeat its last row and are
  // never stored); grouped = slot / row_div (padding rows read row 0)
  int* const atab = reinterpret_cast<int*>(lds + G::TOFF);
  int* const otab = reinterpret_cast<int*>(lds + G::OOFF);      // (the table's entries: fetched at the end, each store waited for one)
  if (tid < G::ROWS) {
    int r, o;
    if (grouped) {
      const int slot = p.sorted_slot_ids[row0 + tid];
      o = (slot >= 0 && slot < p.num_slots) ? slot : -1;
      r = o >= 0 ? slot / p.row_div : 0;
    } else {
      o = row0 + tid < p.M ? row0 + tid : -1;
      r = o >= 0 ? o : p.M - 1;
    }
    atab[tid] = r;
    otab[tid] = o;
  }
  __syncthreads();

  // DMA sources: lane (8 lanes per row) at position sc of tile row r fetches chunk sc ^ (r & 7).  A wave
  // sends rows of its own group only (cluster c: 64 c + 32 (wn >> 1) + 16 wm + 8 (wn & 1) + [0, 8)), so
  // their buffer is free as soon as the group has read it.
  const int srow = lane >> 3, sc = lane & 7;
  const uint32_t chunk = 16u * (uint32_t)(sc ^ (srow & 7));
  const int arow = 32 * (wn >> 1) + 16 * wm + 8 * (wn & 1);
  uint32_t aoff[C], boff[4];
#pragma unroll
  for (int c = 0; c < C; ++c) aoff[c] = (uint32_t)atab[64 * c + arow + srow] * (uint32_t)p.K + chunk;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    boff[i] = (uint32_t)(n0 + 64 * i + feature_of_row<NT>(8 * wave + srow, p.k_splits > 1 || p.out_bf16 == 2)) * (uint32_t)p.K + chunk;
  }
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void*)p.A, 0, (int)0xffffffffu, 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)B, 0, (int)0xffffffffu, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)p.a_scale, 0, (int)0xffffffffu, 0x00020000);
  const float* bssrc = bs + (size_t)((n0 + wn * 64) >> 7) * KB + kb0;
  typedef __attribute__((address_space(3))) void* lptr_t;
  // (block indices past the end are clamped: a valid block is loaded and never consumed, so every wave
  // issues the same number of loads per block and the vmcnt arithmetic holds)
  auto clampk = [&](int i) __attribute__((always_inline)) { return i < nkb ? i : nkb - 1; };
  auto dma_a = [&](int base, int c, int kb) __attribute__((always_inline)) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lptr_t)(lds + base + (64 * c + arow) * 128), 16, (int)aoff[c], (kb0 + kb) * 128, 0, 0);
  };
  auto dma_b = [&](int base, int i, int kb) __attribute__((always_inline)) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lptr_t)(lds + base + G::BOFF + (64 * i + 8 * wave) * 128), 16, (int)boff[i], (kb0 + kb) * 128, 0, 0);
  };
  // Activation scales: four blocks at a time, so that a row's scales share a cache line (one 4-byte
  // load per row and block touches 256 lines per block, half as many as the operands do).  Step t
  // brings SR rows' scales of block group t / 4 per wave; four steps bring all.
  auto scale_row = [&](int t) __attribute__((always_inline)) { return atab[((t & 3) * 8 + wave) * SR + ((lane >> 2) & (SR - 1))]; };
  auto dma_s = [&](int t, int r) __attribute__((always_inline)) {
    if (lane < 4 * SR) {
      int k = (t & ~3) + (lane & 3);
      if (k >= nkb) k = nkb - 1;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rs, (lptr_t)(lds + G::SOFF + ((t >> 2) & 3) * (G::ROWS * 16) + ((t & 3) * 8 + wave) * (SR * 16)), 4,
          (r * KB + kb0 + k) * 4, 0, 0, 0);
    }
  };

  // operand positions inside a buffer (sub-tile 2 mt + wm of the tile is the wave's mt)
  const int xpos = (16 * wm + ln) * 128 + 16 * (lj ^ (ln & 7));                   // + 4096 mt
  const int wpos = G::BOFF + (wn * 64 + ln) * 128 + 16 * (lj ^ (ln & 7));         // + 2048 nt
  const int spos = G::SOFF + (16 * wm + ln) * 16;                                 // + 512 mt
  auto read_op = [&](int at) __attribute__((always_inline)) -> i32x8 {
    const i32x4 lo = *reinterpret_cast<const i32x4*>(lds + at);
    const i32x4 hi = *reinterpret_cast<const i32x4*>(lds + (at ^ 64));
    return i32x8{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
  };

  f32x4 acc[ML][NT];
#pragma unroll
  for (int mt = 0; mt < ML; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  i32x8 wa[NT], xa[2];
  f32x4 part[4];
  float sp[2], spp[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) part[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  sp[0] = sp[1] = spp[0] = spp[1] = 0.f;
  auto read_w = [&](int base, int nt) __attribute__((always_inline)) {
    wa[nt] = read_op((base + wpos) + 2048 * nt);
  };

  // ---- when what is sent --------------------------------------------------------------------------
  // C <= 2 (three buffers): load phase 0 of block kb sends all of block kb + 2 into the buffer of block
  // kb - 1, which both groups have read; the block's feature operands are read in its load phase 0.
  // C >= 3 (two buffers): block kb + 2 goes to the buffer of block kb while that is still being worked
  // off: the feature rows once both groups hold them in registers (from load phase 1 on), a cluster's
  // rows once its group has read them; the last cluster's rows follow in load phase 0 of block kb + 1.
  // The next block's feature operands are read in the last matrix phase, each after its last use.
  // Before the barrier at which a group first reads block kb + 1 every wave has waited for its part of
  // it, in a load phase whose younger loads (kWait of them) may stay in flight.
  constexpr bool REFILL = C >= 3;
  constexpr int kWaitPhase = C >= 3 ? C - 2 : 0;
  constexpr int kWait = C == 4 ? 1 + 3 + 4 : C == 3 ? 1 + 4 : 4 + C + 1;
  auto send_prologue = [&](int base, int kb) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) dma_b(base, i, kb);
#pragma unroll
    for (int c = 0; c < (REFILL ? C - 1 : C); ++c) dma_a(base, c, kb);
  };
#pragma unroll
  for (int t = 0; t < 8; ++t) dma_s(t, scale_row(t));
  send_prologue(0, 0);
  if constexpr (REFILL) dma_a(0, C - 1, 0);
  send_prologue(G::STAGE, clampk(1));
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(REFILL ? 4 + C - 1 : 4 + C, true));      // block 0 has landed
  FP8_PHASE_BARRIER()
  if (wm == 1) FP8_PHASE_BARRIER()
  if constexpr (REFILL) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) read_w(0, nt);
  }

  int srow_next = scale_row(0);      // the row behind the lane's next scale (step kb + 8)
  float sb = bssrc[0];
  int cur = 0, nxt = G::STAGE, far = NBUF == 3 ? 2 * G::STAGE : 0;      // buffers of blocks kb, kb + 1, kb + 2
  for (int kb = 0; kb < nkb; ++kb) {
    const int kn = clampk(kb + 1), kf = clampk(kb + 2);
    const float sb_next = bssrc[kn];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int H = 2 * c + 1 < ML ? 2 : 1;                 // sub-tiles of this cluster
      const int HP = c > 0 ? 2 : ((ML & 1) ? 1 : 2);        // ... of the previous one
      const int cp = c > 0 ? c - 1 : C - 1;
      // ---- load phase ----
      if constexpr (!REFILL) {
        if (c == 0) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) read_w(cur, nt);
        }
      }
      float sa[2] = {0.f, 0.f};
#pragma unroll
      for (int h = 0; h < H; ++h) xa[h] = read_op((cur + xpos) + (2 * c + h) * 4096);
#pragma unroll
      for (int h = 0; h < H; ++h)
        sa[h] = *reinterpret_cast<const float*>(lds + spos + ((kb >> 2) & 3) * (G::ROWS * 16) + (kb & 3) * 4 + (2 * c + h) * 512);
      if constexpr (C == 4) {
        if (c == 0) dma_a(nxt, 3, kn);
        if (c == 1) { dma_b(far, 0, kf); dma_b(far, 1, kf); dma_s(kb + 8, srow_next); }
        if (c == 2) { dma_b(far, 2, kf); dma_b(far, 3, kf); dma_a(far, 0, kf); dma_a(far, 1, kf); }
        if (c == 3) dma_a(far, 2, kf);
      } else if constexpr (C == 3) {
        if (c == 0) dma_a(nxt, 2, kn);
        if (c == 1) { dma_b(far, 0, kf); dma_b(far, 1, kf); dma_s(kb + 8, srow_next); dma_a(far, 0, kf); }
        if (c == 2) { dma_b(far, 2, kf); dma_b(far, 3, kf); dma_a(far, 1, kf); }
      } else {
        if (c == 0) { send_prologue(far, kf); dma_s(kb + 8, srow_next); }
      }
      if (c == (C > 1 ? 1 : 0)) srow_next = scale_row(kb + 1);
      __builtin_amdgcn_sched_barrier(0);
      if (c == kWaitPhase) __builtin_amdgcn_s_waitcnt(waitcnt_imm(kWait, true));
      else __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, true));
      FP8_PHASE_BARRIER()
      // ---- matrix phase ----
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int h = 0; h < H; ++h) sp[h] = sa[h] * sb;
#pragma unroll
      for (int i = 0; i < 4 * H; ++i) {
        const int nt = H == 2 ? i >> 1 : i, h = H == 2 ? i & 1 : 0;
        part[i & 3] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wa[nt], xa[h], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        // fold in the product of three instructions ago (of the previous cluster for the first three)
        if (i >= 3) {
          const int j = i - 3, jn = H == 2 ? j >> 1 : j, jh = H == 2 ? j & 1 : 0;
          acc[2 * c + jh][jn] += part[j & 3] * sp[jh];
        } else {
          const int j = i + 4 * HP - 3, jn = HP == 2 ? j >> 1 : j, jh = HP == 2 ? j & 1 : 0;
          acc[2 * cp + jh][jn] += part[j & 3] * spp[jh];
        }
        if constexpr (REFILL) {
          if (c == C - 1 && h == H - 1) read_w(nxt, nt);      // the operand's last use: fetch the next block's
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_setprio(0);
#pragma unroll
      for (int h = 0; h < H; ++h) spp[h] = sp[h];
      FP8_PHASE_BARRIER()
    }
    sb = sb_next;
    const int t = cur;
    cur = nxt; nxt = NBUF == 3 ? far : t; far = NBUF == 3 ? t : cur;
  }
  {
    constexpr int HP = (ML & 1) ? 1 : 2;
#pragma unroll
    for (int j = 4 * HP - 3; j < 4 * HP; ++j) {
      const int jn = HP == 2 ? j >> 1 : j, jh = HP == 2 ? j & 1 : 0;
      acc[2 * (C - 1) + jh][jn] += part[j & 3] * spp[jh];
    }
  }
  if (wm == 0) FP8_PHASE_BARRIER()
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, false));      // no direct-to-LDS load outlives the workgroup

  int rows[ML];
#pragma unroll
  for (int mt = 0; mt < ML; ++mt) rows[mt] = otab[32 * mt + 16 * wm + ln];
#pragma unroll
  for (int mt = 0; mt < ML; ++mt) {
    const int t = rows[mt];
    if (t < 0) continue;
    store_row<NT>(p, ((size_t)split * p.M + t) * p.N + n0 + wn * 64, lj, acc[mt]);
  }
}

__global__ void __launch_bounds__(512, 1)
fp8_pingpong_kernel(const GemmParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  constexpr int BM = 256, BN = 256;
  const bool grouped = p.sorted_slot_ids != nullptr;
  const int n_blocks = p.N / BN;
  const int m_blocks = grouped ? *p.num_padded / BM : (p.M + BM - 1) / BM;
  const int total = grouped ? m_blocks * n_blocks : (int)gridDim.x;
  int L;
  {
    const int id = blockIdx.x, q = total >> 3, r = total & 7, x = id & 7, idx = id >> 3;
    if (idx >= q + (x < r ? 1 : 0)) return;       // (uniform over the workgroup: nobody reaches a barrier)
    L = x * q + (x < r ? x : r) + idx;
  }
  const int split = L / (m_blocks * n_blocks);
  L -= split * (m_blocks * n_blocks);
  int mb, nb;
  tile_of(p, grouped, m_blocks, n_blocks, L, mb, nb);
  const int row0 = mb * BM, n0 = nb * BN;
  const int KB = p.K >> 7, kb0 = split * p.kb_per_split;
  const int nkb = KB - kb0 < p.kb_per_split ? KB - kb0 : p.kb_per_split;      // >= 1 by construction of the grid
  const uint8_t* B = p.B;
  const float* bs = p.b_scale;
  // live rows: to the end of the matrix, or to the last slot in the block's table (in whole 32-row parts)
  int live = p.M - row0 < BM ? p.M - row0 : BM;
  if (grouped) {
    const int e = p.block_expert_ids[mb];
    if (e < 0) return;
    B += (size_t)e * p.b_expert_stride;
    bs += (size_t)e * p.bs_expert_stride;
    live = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int slot = p.sorted_slot_ids[row0 + 64 * i + (threadIdx.x & 63)];
      const unsigned long long any = __ballot(slot >= 0 && slot < p.num_slots);
      if (any) live = 64 * i + (any >> 32 ? 64 : 32);
    }
  }
  const int ml = __builtin_amdgcn_readfirstlane((live + 31) / 32);
  switch (ml) {
    case 1: ping_tile<1>(p, lds, row0, n0, B, bs, kb0, nkb, split); break;
    case 2: ping_tile<2>(p, lds, row0, n0, B, bs, kb0, nkb, split); break;
    case 3: ping_tile<3>(p, lds, row0, n0, B, bs, kb0, nkb, split); break;
    case 4: ping_tile<4>(p, lds, row0, n0, B, bs, kb0, nkb, split); break;
    case 5: ping_tile<5>(p, lds, row0, n0, B, bs, kb0, nkb, split); break;
    case 6: ping_tile<6>(p, lds, row0, n0, B, bs, kb0, nkb, split); break;
    case 7: ping_tile<7>(p, lds, row0, n0, B, bs, kb0, nkb, split); break;
    case 8: ping_tile<8>(p, lds, row0, n0, B, bs, kb0, nkb, split); break;
    default: break;
  }
}

// Sum of the float32 planes in plane order, one rounding.  n4 = M * N / 4.
__global__ void __launch_bounds__(256)
fp8_split_reduce_kernel(const f32x4* __restrict__ planes, int k_splits, long long n4, void* __restrict__ C,
                        int out_type) {
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n4; i += (long long)gridDim.x * 256) {
    f32x4 s = planes[i];
    for (int k = 1; k < k_splits; ++k) s += planes[(long long)k * n4 + i];
    if (out_type == 2) reinterpret_cast<f32x4*>(C)[i] = s;
    else
      reinterpret_cast<u32x2*>(C)[i] = out_type == 1 ? u32x2{pack2<1>(s[0], s[1]), pack2<1>(s[2], s[3])}
                                                     : u32x2{pack2<0>(s[0], s[1]), pack2<0>(s[2], s[3])};
  }
}

template <int WM, int WN, int MT, int NT, int NS, int KG = 1>
static int launch_one(const GemmParams& p, hipStream_t stream) {
  using G = Geom<WM, WN, MT, NT, NS>;
  static_assert(G::LDS * KG <= 160 * 1024, "LDS");
  auto kern = fp8_blockwise_gemm_kernel<WM, WN, MT, NT, NS, KG>;
  if (G::LDS * KG > 64 * 1024) {
    // raise the dynamic LDS limit of this kernel once per device
    constexpr int kMaxDev = 64;
    static bool allowed[kMaxDev] = {};
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return (int)err;
    if (dev < 0 || dev >= kMaxDev || !allowed[dev]) {
      err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                G::LDS * KG);
      if (err != hipSuccess) return (int)err;
      if (dev >= 0 && dev < kMaxDev) allowed[dev] = true;
    }
  }
  const int grid = ((p.M + G::BM - 1) / G::BM) * (p.N / G::BN) * p.k_splits;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(G::T * KG), G::LDS * KG, stream, p);
  return (int)hipGetLastError();
}

// Tiles.  bm = tokens per workgroup in {16, 32, 64, 128, 256}, bn = features per workgroup in
// {64, 128, 256}; bm = 256 runs eight waves (the two-group tile at bn = 256, 2 x 4 waves in step at
// bn = 128), everything else four (1 x 4).  Returns a
// hipError_t, or -1 for an unknown tile.  Measured and not compiled in: three LDS buffers (two
// blocks in flight: no gain on the small tiles, -30 % on 128 x 128 where it costs the second
// workgroup per CU) and the non-temporal cache policy on the weight loads (-18 % on streaming
// shapes).
static int launch_ping(const GemmParams& p, hipStream_t stream) {
  auto kern = fp8_pingpong_kernel;
  constexpr int kMaxDev = 64;
  static bool allowed[kMaxDev] = {};
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return (int)err;
  if (dev < 0 || dev >= kMaxDev || !allowed[dev]) {
    err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kPingLds);
    if (err != hipSuccess) return (int)err;
    if (dev >= 0 && dev < kMaxDev) allowed[dev] = true;
  }
  const int grid = ((p.M + 255) / 256) * (p.N / 256) * p.k_splits;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(512), kPingLds, stream, p);
  return (int)hipGetLastError();
}

int launch_fp8_gemm(const GemmParams& p, int bm, int bn, hipStream_t stream) {
  if (bm == 256 && bn == 256) return launch_ping(p, stream);
#define FP8_TILE(BMv, BNv, WMv, WNv, MTv, NTv, NSv)                                   \
  if (bm == BMv && bn == BNv) return launch_one<WMv, WNv, MTv, NTv, NSv>(p, stream);
  FP8_TILE(16, 64, 1, 4, 1, 1, 2)   FP8_TILE(16, 128, 1, 4, 1, 2, 2)   FP8_TILE(16, 256, 1, 4, 1, 4, 2)
  FP8_TILE(32, 64, 1, 4, 2, 1, 2)   FP8_TILE(32, 128, 1, 4, 2, 2, 2)   FP8_TILE(32, 256, 1, 4, 2, 4, 2)
  FP8_TILE(64, 64, 1, 4, 4, 1, 2)   FP8_TILE(64, 128, 1, 4, 4, 2, 2)   FP8_TILE(64, 256, 1, 4, 4, 4, 2)
  FP8_TILE(128, 64, 1, 4, 8, 1, 2)  FP8_TILE(128, 128, 1, 4, 8, 2, 2)  FP8_TILE(128, 256, 1, 4, 8, 4, 2)
  FP8_TILE(256, 128, 2, 4, 8, 2, 2)
#undef FP8_TILE
  return -1;
}

// Tiles whose reduction is split among kg groups of waves (bm in {16, 32, 64}; bn, kg below).  Why: up to 64 rows a
// launch is a chain of loads, and what the planes of a split cost, a second launch (2.5 us of 8 to 12) and their trip through
// memory, is most of what can be saved; a CU takes in 70 to 90 kB a microsecond from the caches however its waves
// are dealt, so few fat workgroups stream as fast as many thin ones.  Deeper rings (three and four buffers) measured the same.
int launch_fp8_kgroups(const GemmParams& p, int bm, int bn, int kg, hipStream_t stream) {
  if (p.K / 128 < kg || p.sorted_slot_ids || p.k_splits != 1) return (int)hipErrorInvalidValue;      // (every group has a block of the reduction)
#define FP8_KG(BMv, BNv, WNv, MTv, KGv) if (bm == BMv && bn == BNv && kg == KGv) return launch_one<1, WNv, MTv, 1, 2, KGv>(p, stream);
  FP8_KG(16, 16, 1, 1, 4) FP8_KG(16, 16, 1, 1, 8) FP8_KG(16, 32, 2, 1, 4)
  FP8_KG(32, 16, 1, 2, 4) FP8_KG(32, 32, 2, 2, 4) FP8_KG(32, 64, 4, 2, 2)
  FP8_KG(64, 16, 1, 4, 4) FP8_KG(64, 32, 2, 4, 4) FP8_KG(64, 64, 4, 4, 2)
#undef FP8_KG
  return (int)hipErrorInvalidValue;
}

// Register-resident loop of the FP8 matrix instruction (the achievable matrix-unit roof).
__global__ void __launch_bounds__(256)
fp8_mfma_loop_kernel(float* __restrict__ sink, int iters) {
  i32x8 a, b;
#pragma unroll
  for (int i = 0; i < 8; ++i) { a[i] = 0x38383838; b[i] = 0x30303030 + (int)(threadIdx.x & 1); }
  f32x4 c0 = {0, 0, 0, 0}, c1 = c0, c2 = c0, c3 = c0;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      c0 = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c0, 0, 0, 0, 0, 0, 0);
      c1 = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c1, 0, 0, 0, 0, 0, 0);
      c2 = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c2, 0, 0, 0, 0, 0, 0);
      c3 = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c3, 0, 0, 0, 0, 0, 0);
    }
  }
  sink[(size_t)blockIdx.x * 256 + threadIdx.x] = c0[0] + c1[1] + c2[2] + c3[3];
}

int launch_fp8_mfma_loop(float* sink, int grid, int iters, hipStream_t stream) {
  hipLaunchKernelGGL(fp8_mfma_loop_kernel, dim3(grid), dim3(256), 0, stream, sink, iters);
  return (int)hipGetLastError();
}

int launch_fp8_split_reduce(const float* planes, int k_splits, long long mn, void* C, int out_bf16,
                            hipStream_t stream) {
  const long long n4 = mn / 4;
  long long blocks = (n4 + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(fp8_split_reduce_kernel, dim3((int)blocks), dim3(256), 0, stream, (const f32x4*)planes,
                     k_splits, n4, C, out_bf16);
  return (int)hipGetLastError();
}

}  // namespace fp8
