// Host side of the C ABI declared in include/moe_w4a16.h: argument validation, tile choice,
// workspace carving and kernel launches.  No allocation, no synchronisation, caller's stream.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>

#include <math.h>

#include "../../include/fp8_blockwise_gemm.h"
#include "../../include/moe_w4a16.h"
#include "few_tokens.hpp"
#include "fp8_gemm.hpp"
#include "gemm_kernel.hpp"
#include "gemm_mid.hpp"
#include "gemm_twogroup.hpp"
#include "rows_device.hpp"


namespace moe {

int launch_align(const int32_t*, int, int, int, int, int32_t*, int32_t*, int32_t*, int32_t*, int32_t*,
                 const RowsJob*, hipStream_t);
int launch_silu_mul(const void*, void*, long long, int, int, hipStream_t);
int launch_prepare_rows(const void*, long long, int, int, int, void*, float*, float, hipStream_t);
int launch_repack(const int32_t*, int, int, int, int, int32_t*, hipStream_t);
int launch_awq_import(const int32_t*, const int32_t*, const void*, int, int, int, int, int32_t*, void*, uint8_t*,
                      hipStream_t);
int launch_route_topk(const float*, const float*, int, int, int, int32_t*, float*, hipStream_t);
int launch_route_align(const float*, const float*, int, int, int, int32_t*, float*, int, int, int32_t*, int32_t*,
                       int32_t*, int32_t*, int32_t*, const RowsJob*, hipStream_t);
int launch_stream_read(const void*, size_t, uint32_t*, int, hipStream_t);
int launch_mfma_loop(float*, int, int, hipStream_t);
int launch_issue_mix(float*, int, int, int, hipStream_t);
int launch_combine(const void*, int, int, const float*, const int32_t*, int, void*, long long, int, int, int,
                   hipStream_t);
}  // namespace moe
namespace fp8 {
int launch_fp8_quantize(const void*, long long, int, int, int, uint8_t*, float*, hipStream_t);
}
static bool few_tokens_pay(int T, int topk, int E, int K, int N, int dt, int pre);

namespace moe {

// ---- table of compiled GEMM variants ------------------------------------------------------
#define MOE_DECL(DT, MT, NT, KS, KW, F, Z) \
  extern template int launch_w4a16_gemm<DT, MT, NT, KS, KW, F, Z, 0, 4>(const GemmParams&, int, hipStream_t);
#define MOE_DECL_PRE(DT, MT, NT, KS, F) \
  extern template int launch_w4a16_gemm<DT, MT, NT, KS, 4, F, 1, 1, 4>(const GemmParams&, int, hipStream_t);
#define MOE_DECL_WIDE(DT, MT, NT, KS, F, WV) \
  extern template int launch_w4a16_gemm<DT, MT, NT, KS, 4, F, 1, 2, WV>(const GemmParams&, int, hipStream_t);
#define MOE_ALL_DT_KW(M, MT, NT, KS, F) \
  M(0, MT, NT, KS, 1, F, 0) M(0, MT, NT, KS, 2, F, 0) M(0, MT, NT, KS, 4, F, 0) \
  M(1, MT, NT, KS, 1, F, 0) M(1, MT, NT, KS, 2, F, 0) M(1, MT, NT, KS, 4, F, 0)
#define MOE_TILE(MT, NT, KS) MOE_ALL_DT_KW(MOE_DECL, MT, NT, KS, 0)
#define MOE_TILE_FUSE(MT, NT, KS) MOE_ALL_DT_KW(MOE_DECL, MT, NT, KS, 1)
#include "gemm_variants.def"
#define MOE_TILE_SZR(MT, NT, KS) MOE_DECL(0, MT, NT, KS, 4, 0, 1) MOE_DECL(1, MT, NT, KS, 4, 0, 1)
#define MOE_TILE_SZR_FUSE(MT, NT, KS) MOE_DECL(0, MT, NT, KS, 4, 1, 1) MOE_DECL(1, MT, NT, KS, 4, 1, 1)
#include "gemm_variants_szr.def"
#define MOE_TILE_PRE(MT, NT, KS) MOE_DECL_PRE(0, MT, NT, KS, 0) MOE_DECL_PRE(1, MT, NT, KS, 0)
#define MOE_TILE_PRE_FUSE(MT, NT, KS) MOE_DECL_PRE(0, MT, NT, KS, 1) MOE_DECL_PRE(1, MT, NT, KS, 1)
#include "gemm_variants_pre.def"
#define MOE_TILE_WIDE(MT, NT, KS, WV) MOE_DECL_WIDE(0, MT, NT, KS, 0, WV) MOE_DECL_WIDE(1, MT, NT, KS, 0, WV)
#define MOE_TILE_WIDE_FUSE(MT, NT, KS, WV) MOE_DECL_WIDE(0, MT, NT, KS, 1, WV) MOE_DECL_WIDE(1, MT, NT, KS, 1, WV)
#include "gemm_variants_wide.def"
#define MOE_ONE_BUFFER(M, F) M(0, 1, F) M(0, 2, F) M(0, 4, F) M(1, 1, F) M(1, 2, F) M(1, 4, F)
#define MOE_DECL_ONE(DT, KW, F) extern template int launch_w4a16_gemm<DT, 4, 2, 128, KW, F, 0, 0, 4, 1>(const GemmParams&, int, hipStream_t);
MOE_ONE_BUFFER(MOE_DECL_ONE, 0) MOE_ONE_BUFFER(MOE_DECL_ONE, 1)
#define MOE_NOT_AHEAD(M) M(1, 0) M(1, 1) M(2, 0) M(2, 1)
#define MOE_DECL_NOT_AHEAD(KW, F) extern template int launch_w4a16_gemm<0, 2, 2, 256, KW, F, 0, 0, 4, 1, 0>(const GemmParams&, int, hipStream_t);
MOE_NOT_AHEAD(MOE_DECL_NOT_AHEAD)

typedef int (*GemmLaunchFn)(const GemmParams&, int, hipStream_t);
// pre: 0 = weight tile staged in LDS, 1 = operand-order (repacked) weights, 2 = row-major weights
// loaded in operand order; wv = wavefronts per workgroup; alt = the tile's other form:
// 64x128 with one activation buffer, 32x128 without words read ahead
struct GemmVariant { int dt, mt, nt, ks, kw, fuse, szr, pre, wv; GemmLaunchFn fn; int alt = 0; };
#define MOE_ENTRY(DT, MT, NT, KS, KW, F, Z) {DT, MT, NT, KS, KW, F, Z, 0, 4, &launch_w4a16_gemm<DT, MT, NT, KS, KW, F, Z, 0, 4>},
#define MOE_ENTRY_PRE(DT, MT, NT, KS, F) {DT, MT, NT, KS, 4, F, 1, 1, 4, &launch_w4a16_gemm<DT, MT, NT, KS, 4, F, 1, 1, 4>},
#define MOE_ENTRY_WIDE(DT, MT, NT, KS, F, WV) {DT, MT, NT, KS, 4, F, 1, 2, WV, &launch_w4a16_gemm<DT, MT, NT, KS, 4, F, 1, 2, WV>},
static const GemmVariant kVariants[] = {
#define MOE_TILE(MT, NT, KS) MOE_ALL_DT_KW(MOE_ENTRY, MT, NT, KS, 0)
#define MOE_TILE_FUSE(MT, NT, KS) MOE_ALL_DT_KW(MOE_ENTRY, MT, NT, KS, 1)
#include "gemm_variants.def"
#define MOE_TILE_SZR(MT, NT, KS) MOE_ENTRY(0, MT, NT, KS, 4, 0, 1) MOE_ENTRY(1, MT, NT, KS, 4, 0, 1)
#define MOE_TILE_SZR_FUSE(MT, NT, KS) MOE_ENTRY(0, MT, NT, KS, 4, 1, 1) MOE_ENTRY(1, MT, NT, KS, 4, 1, 1)
#include "gemm_variants_szr.def"
#define MOE_TILE_PRE(MT, NT, KS) MOE_ENTRY_PRE(0, MT, NT, KS, 0) MOE_ENTRY_PRE(1, MT, NT, KS, 0)
#define MOE_TILE_PRE_FUSE(MT, NT, KS) MOE_ENTRY_PRE(0, MT, NT, KS, 1) MOE_ENTRY_PRE(1, MT, NT, KS, 1)
#include "gemm_variants_pre.def"
#define MOE_TILE_WIDE(MT, NT, KS, WV) MOE_ENTRY_WIDE(0, MT, NT, KS, 0, WV) MOE_ENTRY_WIDE(1, MT, NT, KS, 0, WV)
#define MOE_TILE_WIDE_FUSE(MT, NT, KS, WV) MOE_ENTRY_WIDE(0, MT, NT, KS, 1, WV) MOE_ENTRY_WIDE(1, MT, NT, KS, 1, WV)
#include "gemm_variants_wide.def"
#define MOE_ENTRY_ONE(DT, KW, F) {DT, 4, 2, 128, KW, F, 0, 0, 4, &launch_w4a16_gemm<DT, 4, 2, 128, KW, F, 0, 0, 4, 1>, 1},
  MOE_ONE_BUFFER(MOE_ENTRY_ONE, 0) MOE_ONE_BUFFER(MOE_ENTRY_ONE, 1)
#define MOE_ENTRY_NOT_AHEAD(KW, F) {0, 2, 2, 256, KW, F, 0, 0, 4, &launch_w4a16_gemm<0, 2, 2, 256, KW, F, 0, 0, 4, 1, 0>, 1},
  MOE_NOT_AHEAD(MOE_ENTRY_NOT_AHEAD)
};

static const GemmVariant* find_variant(int dt, int mt, int nt, int kw, int fuse, int szr, int pre = 0, int wv = 4, int alt = 0) {
  for (const GemmVariant& v : kVariants)
    if (v.dt == dt && v.mt == mt && v.nt == nt && v.kw == kw && v.fuse == fuse && v.szr == szr && v.pre == pre &&
        v.wv == wv && v.alt == alt)
      return &v;
  return nullptr;
}

// ---- thread-local state -----------------------------------------------------------------
static thread_local char g_err[512] = "";
static thread_local void* g_events[7] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
static thread_local int g_nevents = 0;
static thread_local int g_force_mt = 0, g_force_nt = 0;
static thread_local int g_scale_path = 0;   // 0 auto, 1 LDS table, 2 registers
static thread_local int g_force_tpw = 0;    // feature tiles per workgroup (register-scale kernels), 0 = auto
static thread_local int g_force_ksplit = 0; // reduction splits of the layer's down projection, 0 = auto
static thread_local int g_force_block_m = 0; // bucketing block of the layer, 0 = auto
static thread_local int g_wide_mode = 0;     // eight-wave 128-token tiles: 0 = when the shape allows, 1 = never
static thread_local int g_last_plan[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};   // what the last grouped GEMM launch used

static int fail(int status, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return status;
}
static int hip_fail(int err, const char* what) {
  return fail(MOE_HIP_ERROR, "%s: %s", what, hipGetErrorString((hipError_t)err));
}

static bool valid_block_m(int b) { return b == 16 || b == 32 || b == 64 || b == 128 || b == 256; }
static size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
static size_t align_capacity(long long S, int E, int block_m) {
  const long long worst = S + (S < E ? S : E) * (long long)(block_m - 1);
  return (size_t)((worst + block_m - 1) / block_m * block_m);
}
constexpr size_t kLdsLimit = 160 * 1024;
constexpr int kMaxGroups = 512;

static size_t gemm_lds_bytes(int mt, int nt, int ks, int G, int szr) {
  const size_t M_T = 16 * mt, NW = 16 * nt;
  return kXBufs(mt, ks) * M_T * (ks * 2 + kXRowPad) + 4 * NW * (ks / 2 + kWRowPad(ks)) + (szr ? 0 : (size_t)G * 64 * nt * 4) + M_T * 4;
}

// The eight-wave 128-token tile serves 128-slot blocks of register-scale shapes in the stated
// weight layout (group 128, 16-byte aligned scale rows).
static bool wide_tile_usable(int block_m, int szr_ok, int pre) {
  return block_m >= 128 && szr_ok && !pre && g_wide_mode != 1 && g_force_mt == 0 && g_force_nt == 0;
}

// Tile choice.  Tokens per tile follow the bucketing block; the feature width per workgroup is
// as wide as LDS allows while still giving every CU a couple of workgroups (256 CUs).
static int choose_tile(int num_slots, int E, int feat, int G, int block_m, int fuse, int szr_ok, int dt, int pre,
                       int& mt, int& nt, int& ks, int& szr) {
  mt = block_m / 16;
  if (mt > 8) mt = 8;
  if (g_force_mt > 0) {
    if ((block_m / 16) % g_force_mt != 0) return -1;
    mt = g_force_mt;
  }
  ks = mt >= 4 ? 128 : 256;
  const int min_nt = (fuse || mt >= 4) ? 2 : 1;
  // register-resident scales when the shape allows it and such a variant is compiled
  auto pick_szr = [&](int nt_) {
    if ((g_scale_path == 1 && !pre) || !szr_ok) return 0;
    return find_variant(dt, mt, nt_, 4, fuse, 1, pre) ? 1 : 0;
  };
  if (g_force_nt > 0) {
    nt = g_force_nt;
    szr = pick_szr(nt);
    if ((g_scale_path == 2 || pre) && !szr) return -1;
    return (nt >= min_nt && (nt == 1 || nt == 2 || nt == 4) && gemm_lds_bytes(mt, nt, ks, G, szr) <= kLdsLimit) ? 0 : -1;
  }
  const long long est_blocks = (num_slots + 16 * mt - 1) / (16 * mt) + (num_slots < E ? num_slots : E) / 2;
  // 256-feature tiles only pay off with register-resident scales (two workgroups per CU)
  nt = (mt >= 4 && pick_szr(4)) ? 4 : 2;
  for (;;) {
    const int fpw = fuse ? 32 * nt : 64 * nt;
    const long long wgs = est_blocks * ((feat + fpw - 1) / fpw);
    szr = pick_szr(nt);
    if ((g_scale_path == 2 || pre) && !szr) { if (nt == min_nt) return -1; nt >>= 1; continue; }
    const bool fits = gemm_lds_bytes(mt, nt, ks, G, szr) <= kLdsLimit;
    // 128-feature tiles stay even when they leave fewer than two workgroups per CU: measured
    // faster than twice as many 64-feature tiles (same bytes in flight, less activation staging)
    if (fits && (wgs >= 512 || nt <= 2 || nt == min_nt)) return 0;
    if (nt == min_nt) return -1;
    nt >>= 1;
  }
}

// Does the 64x128 tile with its scales in LDS run with one activation buffer?  One frees 18 KB of LDS, for a third
// workgroup on a CU (where many groups fill the LDS, for a second), and costs a second barrier per stage.  So the
// launch has to have more than two and a half workgroups (one and a quarter) for every CU, and more than a few stages.  Layer,
// time with two buffers over time with one, 600 shapes, mean (worst), by workgroups of the larger product up to 512 /
// 512 ... 768 / above 1500: fp16, chunk-steps of 32 and 64 k 0.99 (0.97) / 1.06 (0.97) / 1.16 (0.98), 128 k 0.98 (0.96) / 0.99
// (0.97) / 1.07 (0.98); bf16, 32 and 64 k 0.99 (0.95) / 1.06 (0.98) / 1.15 (0.97).  Reductions of 128 ... 320 with 1000 workgroups
// 0.95 ... 0.97.  bf16, 128 k: always, its row sums (ZS) outweigh the barrier, 1.02 (1.00) / 1.07 (1.02) / 1.14 (1.00).
static bool one_buffer_pays(int num_slots, int E, int feat, int fuse, int K_in, int G, int dt, int kw) {
  if (dt == MOE_BF16 && kw == 4) return true;
  const size_t two = gemm_lds_bytes(4, 2, 128, G, 0), one = two - 64 * (128 * 2 + kXRowPad), cu = 160 * 1024;
  const int fit_two = (int)std::min<size_t>(2, cu / two), fit_one = (int)std::min<size_t>(3, cu / one);
  const long long blocks = (num_slots + 63) / 64 + (num_slots < E ? num_slots : E) / 2, n_tiles = (feat + (fuse ? 63 : 127)) / (fuse ? 64 : 128);
  return fit_one > fit_two && K_in >= 512 && blocks * n_tiles > 320 * fit_two;
}

// Does the 32x128 tile, which reads its words ahead in fp16 with groups below 128, do better without?  The registers
// of that (118 and 127 -> 144) leave three workgroups on a CU; up to five groups the LDS holds four.  So with groups of
// 64 a launch of more than three for every CU does (an estimate: what a uniform routing has); with groups of 32 and
// reductions this short, one stage that is half empty, any launch.  Layer, time with over time without, 4200 shapes, products of up
// to five groups by workgroups up to 768 / 768 ... 1024 / above, mean: groups of 32 1.005 / 1.045 / 1.05, of 64 0.987 / 1.03 / 1.03;
// of six to eight groups, any launch, 0.985.
static bool read_ahead_costs(int num_slots, int E, int feat, int fuse, int G, int dt, int kw) {
  const long long blocks = (num_slots + 31) / 32 + (num_slots < E ? num_slots : E) / 2, n_tiles = (feat + (fuse ? 63 : 127)) / (fuse ? 64 : 128);
  return kReadAhead(dt, 2, 2, kw, 0) && 4 * gemm_lds_bytes(2, 2, 256, G, 0) <= 160 * 1024 && (kw == 1 || blocks * n_tiles > 768);
}

struct GemmArgs {
  const void* A; int row_div;
  const int32_t* qweight; const void* scales; const uint8_t* zeros;
  const int32_t* sorted_slot_ids; const int32_t* block_expert_ids; const int32_t* num_padded;
  int num_slots, E, N_out, K_in, group, block_m, dt;
  void* C; int ldc; int fuse_half_n; int out_f32;
  int dense = 0;             // 1: plain GEMM, no routing tables (the three table pointers are null)
  int pre = 0;               // 1: qweight is in the operand-order layout of moe_repack_qweight
  int k_splits = 1;          // wanted reduction splits (float32 output planes num_slots*ldc apart)
  int* used_splits = nullptr;  // out: the number of planes the launch really wrote
};

static int run_gemm(const GemmArgs& a, hipStream_t stream) {
  if (a.dt != MOE_F16 && a.dt != MOE_BF16) return fail(MOE_INVALID_ARGUMENT, "dt must be MOE_F16 or MOE_BF16");
  if (a.num_slots < 0 || a.E < 1 || a.row_div < 1 || a.N_out < 1 || a.K_in < 1 || a.group < 1)
    return fail(MOE_INVALID_ARGUMENT, "sizes must be positive (num_slots >= 0)");
  if (!valid_block_m(a.block_m)) return fail(MOE_INVALID_ARGUMENT, "block_m must be 16, 32, 64, 128 or 256");
  if (a.group % 32 != 0) return fail(MOE_UNSUPPORTED_SHAPE, "group_size %d is not a multiple of 32", a.group);
  if (a.K_in % a.group != 0) return fail(MOE_UNSUPPORTED_SHAPE, "K_in %d is not a multiple of group_size %d", a.K_in, a.group);
  if (a.N_out % 16 != 0) return fail(MOE_UNSUPPORTED_SHAPE, "N_out %d is not a multiple of 16", a.N_out);
  const int G = a.K_in / a.group;
  if (G > kMaxGroups) return fail(MOE_UNSUPPORTED_SHAPE, "K_in/group_size = %d exceeds %d", G, kMaxGroups);
  if (a.num_slots == 0) return MOE_OK;
  if (!a.A || !a.qweight || !a.scales || !a.zeros || !a.C ||
      (!a.dense && (!a.sorted_slot_ids || !a.block_expert_ids || !a.num_padded)))
    return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  if (((uintptr_t)a.A | (uintptr_t)a.qweight) % 16 != 0)
    return fail(MOE_INVALID_ARGUMENT, "A and qweight must be 16-byte aligned");
  if ((uintptr_t)a.scales % 2 != 0 || (uintptr_t)a.C % (a.out_f32 ? 8 : 4) != 0)
    return fail(MOE_INVALID_ARGUMENT, "scales must be 2-byte aligned and C 4-byte aligned");

  // kernels address with 32-bit per-lane byte offsets from a per-expert / per-matrix base
  if ((long long)a.N_out * (a.K_in / 2) >= (1LL << 31))
    return fail(MOE_UNSUPPORTED_SHAPE, "one expert's packed weights must stay below 2 GiB");
  if (((long long)(a.num_slots + a.row_div - 1) / a.row_div) * a.K_in * 2 >= (1LL << 31))
    return fail(MOE_UNSUPPORTED_SHAPE, "the A matrix must stay below 2 GiB");
  const int fuse = a.fuse_half_n > 0 ? 1 : 0;
  const int feat = fuse ? a.fuse_half_n : a.N_out;
  const int kw = a.group % 128 == 0 ? 4 : (a.group % 64 == 0 ? 2 : 1);
  int mt, nt, ks, szr;
  const int sz_vec = (G % 8 == 0 && (uintptr_t)a.scales % 16 == 0 && (uintptr_t)a.zeros % 8 == 0) ? 1 : 0;
  const int szr_ok = sz_vec && a.group == 128 && (long long)a.E * a.N_out * G < (1LL << 31);
  if (a.pre && (!szr_ok || (!fuse && a.N_out % 32 != 0)))
    return fail(MOE_UNSUPPORTED_SHAPE, "operand-order weights need group_size 128, K_in %% 1024 == 0, 16-byte aligned "
                "scale rows and (down projection) N_out %% 32 == 0");
  int wv = 4, pre = a.pre;
  if (wide_tile_usable(a.block_m, szr_ok, a.pre) && find_variant(a.dt, 8, 2, 4, fuse, 1, 2, 8)) {
    mt = 8; nt = 2; ks = 128; szr = 1; wv = 8; pre = 2;
  } else if (choose_tile(a.num_slots, a.E, feat, G, a.block_m, fuse, szr_ok, a.dt, a.pre, mt, nt, ks, szr) != 0) {
    return fail(MOE_UNSUPPORTED_SHAPE, "no GEMM tile fits (K_in/group_size = %d, block_m = %d, override %d/%d)",
                G, a.block_m, g_force_mt, g_force_nt);
  }
  const int alt = !szr && nt == 2 && (mt == 4 ? one_buffer_pays(a.num_slots, a.E, feat, fuse, a.K_in, G, a.dt, kw)
                                              : mt == 2 && read_ahead_costs(a.num_slots, a.E, feat, fuse, G, a.dt, kw));
  const GemmVariant* v = find_variant(a.dt, mt, nt, kw, fuse, szr, pre, wv, alt);
  if (!v) return fail(MOE_UNSUPPORTED_SHAPE, "GEMM variant mt=%d nt=%d kw=%d fuse=%d szr=%d is not compiled", mt, nt, kw, fuse, szr);

  GemmParams p;
  p.A = a.A; p.row_div = a.row_div;
  p.qweight = a.qweight; p.scales = a.scales; p.zeros = a.zeros;
  p.sorted_slot_ids = a.sorted_slot_ids; p.block_expert_ids = a.block_expert_ids; p.num_padded = a.num_padded;
  p.num_slots = a.num_slots; p.E = a.E; p.N_out = a.N_out; p.K_in = a.K_in; p.group = a.group;
  p.block_m = a.block_m; p.C = a.C; p.ldc = a.ldc;
  const int fpw = (fuse ? 8 : 16) * nt * wv;     // features (act columns when fused) per workgroup tile
  p.n_tiles = (feat + fpw - 1) / fpw;
  p.G = G;
  p.cpg = a.group / (32 * kw);
  p.half_n = a.fuse_half_n;
  p.out_f32 = a.out_f32;
  p.c_bytes = c_plane_bytes(a.num_slots, (long long)a.ldc * (a.out_f32 ? 4 : 2));
  p.sz_vec = sz_vec;
  p.dense = a.dense;
  // Split reduction: whole scale panels (4 pipeline stages) per range, every range non-empty.
  int ksp = 1, kspan = a.K_in;
  if (a.k_splits > 1 && szr && a.out_f32 && !fuse) {
    const int pan = ks >= 256 ? 1024 : 512, npan = a.K_in / pan;   // one scale panel of the kernel
    const int pps = (npan + a.k_splits - 1) / a.k_splits;
    ksp = (npan + pps - 1) / pps;
    kspan = pps * pan;
  }
  p.k_splits = ksp; p.k_span = kspan; p.split_stride = (long long)a.num_slots * a.ldc;
  if (a.used_splits) *a.used_splits = ksp;
  const size_t cap = align_capacity(a.num_slots, a.E, a.block_m);
  // Register-scale kernels can walk several feature tiles per workgroup: aim for about 48
  // pipeline stages per workgroup at small token tiles (the start-up of a workgroup costs about
  // as much as ten of their stages) while keeping a few thousand workgroups in the launch.
  int tpw = 1;
  if (szr) {
    const int nst = kspan / ks;
    const int target = mt <= 2 ? 48 : 24;       // large token tiles: stages are long, start-up matters less
    tpw = (target + nst - 1) / nst;
    if (tpw > 8) tpw = 8;
    if (tpw > p.n_tiles) tpw = p.n_tiles;
    // prefer a count that divides the tiles of a block evenly (no short last group)
    for (int t = tpw; t <= tpw + 2 && t <= 8 && t <= p.n_tiles; ++t)
      if (p.n_tiles % t == 0) { tpw = t; break; }
    // Enough workgroups for the chip: two rounds of the 768 that are resident, and with a few rows per expert
    // (16-row blocks, a workgroup is all weight streaming) a third one, which evens out the tail, as long as a workgroup keeps
    // 16 stages to make up for its start.  A count that leaves a short last group is lowered to the next that does not, if
    // that costs less than half of it and leaves 16 stages.  Down projection of 256 experts, 2048 -> 7168 (56 tiles), f16:
    // 128 tokens 4 or 7 tiles 358 us, 10 379, 12 403; 37 tokens on repacked weights 2 tiles 222 us,
    // 4 228, 6 (what 1536 workgroups alone gave) 235.  The whole layer, replayed: 37 to 96 tokens 1 to 3 % less, others within 1.5 %.
    // Products where two rounds alone choose another count: 144 of gate/up 1.8 % less on average (8 % more at most), 7 of down 1 % less;
    // without the 16 stages a gate/up reduction of 1024 lost up to 11 %, 157 of down 3 % on average.
    const long long est_blocks = (a.num_slots + 16 * mt - 1) / (16 * mt) + (a.num_slots < a.E ? a.num_slots : a.E) / 2;
    auto workgroups = [&](int t) { return est_blocks * ((p.n_tiles + t - 1) / t) * ksp; };
    while (tpw > 1 && workgroups(tpw) < 1536) --tpw;
    while (mt == 1 && (tpw - 1) * nst >= 16 && workgroups(tpw) < 2304) --tpw;
    for (int t = tpw; mt == 1 && 2 * t > tpw && (t == tpw || t * nst >= 16); --t)
      if (p.n_tiles % t == 0) { tpw = t; break; }
  }
  if (g_force_tpw > 0) tpw = szr ? (g_force_tpw < p.n_tiles ? g_force_tpw : p.n_tiles) : 1;
  p.tiles_per_wg = tpw;
  const long long grid = (long long)(cap / (16 * mt)) * ((p.n_tiles + tpw - 1) / tpw) * ksp;
  if (grid > 0x7fffffffLL) return fail(MOE_UNSUPPORTED_SHAPE, "grid too large");
  g_last_plan[0] = mt; g_last_plan[1] = nt; g_last_plan[2] = ks; g_last_plan[3] = szr;
  g_last_plan[4] = tpw; g_last_plan[5] = ksp; g_last_plan[6] = kspan; g_last_plan[7] = fuse;
  g_last_plan[8] = wv;
  const int err = v->fn(p, (int)grid, stream);
  if (err != 0) return hip_fail(err, "grouped GEMM launch");
  return MOE_OK;
}

// wide_shape: the layer's shapes admit the eight-wave tile; wide_tile: it will be used (not with
// operand-order weights, which only the four-wave tiles read)
static int pick_block_m(long long S, int E, bool wide_shape = false, bool wide_tile = false) {
  const long long avg = S / (E > 0 ? E : 1);
  if (avg <= 8) return 16;
  if (avg <= (wide_shape ? 28 : 24)) return 32;
  // 128-slot blocks only for the eight-wave tile (every unpacked weight feeds up to eight matrix
  // instructions and its main loop skips the block's empty 16-row sub-tiles, so a block that is a
  // quarter full costs a quarter of the matrix work); the four-wave 128-slot tiles run one
  // workgroup per CU and lose to 64-slot ones.  Measured on the 256-expert layer shape: 32 rows per
  // expert 1.73 against 1.88 ms, 48 rows a tie, 64 rows 2.40 against 2.90 ms; up to 28 rows the
  // 32-slot tile wins (28 rows: 1.65 ms for both, 64-slot blocks 1.86).
  if (wide_tile) return 128;
  return 64;
}

// Can both projections of a layer run on the eight-wave tile?  (group 128, whole 8-group scale
// panels in K and N; pointer alignment is checked again at launch)
static bool layer_wide_ok(int K, int N, int group_size) {
  return group_size == 128 && K % 1024 == 0 && N % 1024 == 0 && g_wide_mode != 1 && g_force_mt == 0 && g_force_nt == 0;
}

// Reduction splits of the layer's down projection.  With few experts and few rows the launch has
// too few workgroups to keep enough loads in flight; cutting the reduction multiplies them (the
// combine adds the partial planes).  Only for small token tiles: large ones have rows to spare.
static int pick_k_splits(long long S, int E, int K, int N, int block_m) {
  if (block_m > 32) return 1;
  const long long est_blocks = (S + block_m - 1) / block_m + (S < E ? S : E) / 2;
  const long long wgs = est_blocks * ((K + 127) / 128);
  if (wgs <= 0 || wgs >= 768) return 1;
  long long want = (768 + wgs - 1) / wgs;      // about one workgroup per resident slot (3 per CU)
  const int npan = N / 1024;
  if (want > npan) want = npan;
  if (want > 8) want = 8;
  return want < 1 ? 1 : (int)want;
}

// Does the layer run on the two-group 256-slot tile (gemm_twogroup.hpp)?  It fetches and unpacks an
// expert's weights once per 256 rows and keeps the matrix unit busier; below, the 32-slot and the
// eight-wave 128-slot tiles stream the weights as fast or spread a small launch over more workgroups.
// Measured (us, former choice -> two-group; 256 experts, K 7168, N 2048): fp16 512 tokens 1304 -> 1407,
// 1024 1714 -> 1657, 1536 1991 -> 1915, 4096 4026 -> 3596; bf16, whose zero points cost the other
// tiles a second matrix instruction, 512 tokens a tie, 717 1723 -> 1690, 1024 1933 -> 1912, 4096 5436
// -> 4258 (the 64-slot tile, asked first, now has the 717 and 1024: 1407 and 1570 in bf16, 1510 in fp16).  Launches of few tiles lose by their last round: fp16 16 experts (K 4096, N 2048), 2048
// tokens (768 tiles) 324 -> 359, 4096 tokens (1280) 562 -> 583, 8 experts (K 4096, N 14336), 1024
// tokens (1536) 1008 -> 940; bf16 64 experts (K 2048, N 1024), 512 tokens (704) 113 -> 124, 1024
// tokens (896) 186 -> 180, 16 experts, 2048 tokens (768) 440 -> 412.
// Two more conditions come from 24000 layer calls on the former tiles and on this one (8 to 256 experts, K and N
// 1024 ... 14336, 8 to 192 rows per expert, uniform and power-law routing, both weight layouts):
//   * Skewed routing packs the rows into far fewer blocks than uniform routing, and the host does not know which
//     it is.  So even if every block were full there have to be some rounds of tiles (`packed`), or so many
//     rows per expert that the 128-slot tile needs a second block.  Former time over this one's, geometric mean
//     (share of calls more than 5 % slower) of the calls these conditions keep / take away: bf16 uniform 1.09 (3 %) /
//     0.98 (33 %), skewed 1.12 (12 %) / 0.92 (56 %); fp16 uniform 1.07 (4 %) / 1.03 (12 %), skewed 0.96 (39 %) / 0.87 (80 %).
//   * Operand-order weights run on 64-slot four-wave tiles otherwise, which lose less at few rows: bf16 20 to 26
//     rows per expert 4 to 7 % faster there (256 experts, K 7168, N 2048), 28 a tie, 32 17 % slower.  Kept / taken
//     away: bf16 uniform 1.15 (6 %) / 0.96 (53 %), skewed 1.03 (31 %) / 0.82 (77 %); fp16 1.12 (3 %) / 1.01 (29 %) and
//     0.96 (45 %) / 0.81 (94 %).
static bool twogroup_pays(long long S, int E, int K, int N, int dt, int pre) {
  const long long avg = S / (E > 0 ? E : 1), feat = (2LL * N + K) / 256;
  const long long tiles = (S / 256 + (S < E ? S : E) / 2) * feat, packed = S / 256 * feat;      // of both products
  if (dt == MOE_BF16) return avg >= (pre ? 28 : 20) && tiles >= 750 && (packed >= 600 || avg >= 112);
  return avg >= 29 && tiles >= 1400 && (packed >= 1000 || avg >= 112);
}

// Does the layer run on the 64-slot tile (gemm_mid.hpp)?  It reads an expert's weights once for up to 64 rows, works
// off whole 16-row parts only, and takes activations that were put in order first (beside the bucketing, or from 2^23 of them on by a launch of
// their own; in bf16 act's sums are another launch), so the launch has to be large: a quarter of a billion weights in each of an expert's
// matrices together and two workgroups for each of three on a CU.  (All figures were taken when the reorder was always a launch of 4 us: the line errs
// to the side of the other tiles, as that of twogroup_pays does.)  Former choice over this tile, lower of two draws, by rows per
// expert: even routing / experts weighted as 1 / rank / as rank ** -2.4 (2900 calls, 11 shapes, both layouts), stated layout:
//   256 experts, K 7168, N 2048,  fp16  9: 1.18/1.28/1.12  16: 1.09/1.23/1.23  28: 1.14/1.27/1.28  40: 1.12/1.56/0.97  54: 0.99/1.41/0.93
//                                 bf16  9: 1.39/1.49/1.43  16: 1.26/1.47/1.38  28: 1.19/1.84/1.09  48: 1.13/1.63/1.01  60: 1.00/1.50/0.96  72: 0.93/1.48/0.93
//   64 experts, K 7168, N 2048,   fp16  9: 1.15/1.16/1.22  16: 1.04/1.16/1.19  28: 1.07/1.27/1.24  40: 1.16/1.63/1.35  54: 1.07/1.48/1.25
//                                 bf16  9: 1.35/1.41/1.38  16: 1.23/1.32/1.37  28: 1.22/1.52/1.45  48: 1.16/1.97/1.65  60: 1.09/1.90/1.64  72: 0.90/1.64/1.25
//   8 experts, K 4096, N 14336,   fp16  9: 1.23/1.20/1.24  16: 1.04/1.26/1.21  20: 1.05/1.15/1.07  28: 1.15/1.24/1.22  40: 1.44/1.90/1.92
//                                 bf16  9: 1.39/1.36/1.34  16: 1.19/1.39/1.36  20: 1.15/1.21/1.14  48: 1.45/2.25/2.29  60: 1.40/2.01/1.98  72: 1.05/1.81/1.79
//   16 experts, K 5120, N 8192,   fp16  9: 1.10/1.05/1.04  20: 0.95/1.18/1.25  28: 1.03/1.24/1.24  40: 1.25/1.85/1.12;  bf16  60: 1.13/1.95/1.38  78: 0.88/1.77/1.70
//   64 experts, K = N = 2048,     fp16  9: 1.13/1.12/1.04  20: 0.94/1.10/1.15  28: 0.99/1.12/1.20  40: 1.06/1.44/1.35;  bf16  60: 0.95/1.76/1.40  72: 0.82/1.70/1.44
//   32 experts, K 2048, N 4096,   fp16  9: 1.04/1.15/1.11  20: 0.93/1.15/1.18  28: 1.03/1.17/1.27  48: 0.99/1.43/1.22;  bf16  60: 0.95/1.88/1.35  72: 0.83/1.95/1.17
//   8 experts, K 2048, N 20480,   fp16  9: 1.12/1.14/1.21  20: 0.99/1.05/1.17  28: 1.06/1.12/1.23  48: 1.69/2.36/2.35;  bf16  60: 1.73/2.59/2.61  72: 1.38/2.39/2.39
// What the numbers set.  fp16 below half a billion weights: from 28 rows on; below that only where the former choice splits
// a short down product or unpacks operand-order words, and the reduction is not the shortest (8 experts, K 1024, N 31744,
// operand order, 16 rows 0.91).  The end is where even routing turns (from 64 rows on half the experts need a second block); later,
// bf16, where the down product had too few tiles before (E * K), or for operand-order weights that are not on the
// two-group tile (72 rows 1.09 ... 1.36).  Not used: 8 experts, K 4096, N 14336 gain up to 96 rows (1.1 ... 1.3 in runs of blocks).
static bool mid_pays(long long S, int E, int K, int N, int dt, int pre) {
  const long long avg = S / (E > 0 ? E : 1), weights = (long long)E * N * K;
  if (avg < 9 || weights < 250000000LL || (long long)E * N < 96000) return false;
  const bool two_group = twogroup_pays(S, E, K, N, dt, pre);
  if (dt == MOE_F16)
    return avg < (!pre ? 56 : two_group ? 64 : 72) && (weights >= 500000000LL || avg >= 28 || (K >= 2048 && (pre || (long long)E * K <= 50000)));
  return avg < ((long long)E * K <= 40000 || (pre && !two_group) ? 80 : 64);
}

// Reduction splits of its down projection: about one workgroup for each of three on a CU.
static int mid_splits(long long S, int E, int K, int N) {
  const long long wgs = (S < E ? S : E) * (K / 128);
  int s = wgs >= 768 ? 1 : (int)((768 + wgs / 2) / (wgs > 0 ? wgs : 1)), npan = N / 1024;
  if (s > npan) s = npan;
  if (s > 8) s = 8;
  return s < 1 ? 1 : s;
}

// Scratch inside the library, for the layer call that carries no workspace.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;

struct Workspace {
  size_t counts, offsets, num_padded, sorted, blocks, act, Y, base, sums, mid_splits, few_units, few_end, total;
};
// Bytes up to the end of `planes` partial planes at Y; the row sums of act lie there.
static size_t end_of_planes(const Workspace& w, size_t plane, size_t planes) {
  return std::max(w.base, w.Y + round_up(plane * planes, 256));
}
static Workspace carve(long long T, int K, int N, int E, int topk, int dt) {
  const long long S = T * topk;
  Workspace w;
  size_t o = 0;
  w.counts = o;      o += round_up((size_t)E * 4, 256);
  w.offsets = o;     o += round_up((size_t)(E + 1) * 4, 256);
  w.num_padded = o;  o += 256;
  w.sorted = o;      o += round_up(align_capacity(S, E, 256) * 4, 256);   // the largest block any caller can force
  w.blocks = o;      o += round_up((align_capacity(S, E, 16) / 16 + 1) * 4, 256);
  w.act = o;         o += round_up((size_t)S * N * 2, 256);
  // float32 (combined unrounded); one plane per reduction split (at most 8, small batches only)
  w.Y = o;           o += round_up((size_t)S * K * 4 * std::max(pick_k_splits(S, E, K, N, pick_block_m(S, E)),
                                                            pick_k_splits(S, E, K, N, pick_block_m(S, E, true))), 256);
  w.base = o;        // what the layer cannot do without
  // row sums of act for the bf16 operands of the two-group and the 64-slot tile; a caller's workspace
  // without them runs the layer on another tile instead.  (Where only the 64-slot tile wants them they are
  // reserved for either type, so that as a rule the query says the same for both.)
  const bool ordered = K % 1024 == 0 && N % 1024 == 0, rows_for_two = ordered && twogroup_pays(S, E, K, N, MOE_BF16, 0);
  const bool mid = ordered && (mid_pays(S, E, K, N, dt, 0) || mid_pays(S, E, K, N, dt, 1));     // (the query does not know the layout)
  const size_t row_sums = (size_t)S * (N / 128) * 4;
  w.sums = dt == MOE_BF16 ? row_sums : 0;
  if (rows_for_two ? dt == MOE_BF16 : mid) o += round_up(row_sums, 256);
  // The vector products of a few tokens hold act in twice the bytes, from its place on into that of Y.
  w.few_units = w.act + round_up(few_act_bytes(S, N), 256);
  w.few_end = w.few_units + few_unit_bytes(S, N);
  // Planes of the 64-slot tile's split down product.  A workspace without them runs it in fewer splits, whose sums are
  // rounded in another order, so sizes that the built-in array serves get no more of them than it holds: the two
  // calls then have the same bits.
  const size_t plane = (size_t)S * K * 4;
  auto with_planes = [&](size_t planes) { return end_of_planes(w, plane, planes) + round_up(w.sums, 256); };
  const size_t most = w.base <= kStaticScratchBytes ? std::max(kStaticScratchBytes, with_planes(0)) : ~(size_t)0;
  w.mid_splits = mid_splits(S, E, K, N);
  while (w.mid_splits > 1 && (mid ? with_planes(w.mid_splits) > most : w.Y + plane * w.mid_splits > w.base)) --w.mid_splits;
  w.total = mid ? std::max(o, with_planes(w.mid_splits)) : o;
  return w;
}
// What the size query answers: room for T tokens, and for the most of fewer tokens that run as vector products, whose act
// may be longer than everything the tiles need for T (13 to 16 tokens of 256 x 1024, 8 experts, top 2, with the size of 17 to 22).
static size_t layer_workspace(int T, int K, int N, int E, int topk, int dt) {
  size_t o = carve(T, K, N, E, topk, dt).total;
  if (few_tokens_fit(topk, K, N))
    for (int t = std::min(T, 32 / topk); t > 0; --t)
      if (few_tokens_pay(t, topk, E, K, N, dt, 0) || few_tokens_pay(t, topk, E, K, N, dt, 1))
        return std::max(o, round_up(carve(t, K, N, E, topk, dt).few_end, 256));
  return o;
}

}  // namespace moe

using namespace moe;

// ---- blockwise-scaled FP8 GEMM: tile and split choice --------------------------------------
static thread_local int g_fp8_mt = 0, g_fp8_nt = 0, g_fp8_splits = 0, g_fp8_group_m = 0;

struct Fp8Plan { int bm, bn, splits, kb_per_split; };

// at least four blocks of the reduction in a split
static int fp8_splits_for(int want, int most, int KB) {
  int s = want < most ? want : most;
  if (s > KB / 4) s = KB / 4;
  return s < 1 ? 1 : s;
}

// 65 rows and more that do not fill the 256 x 256 tile: tile and split by the time they should take.  A
// workgroup needs t microseconds for a block of 128 reduction indices with two workgroups on its CU (the
// value depends little on the second one), about four blocks to start and end; a last round that
// is partly full costs 0.4 of what is missing; a split costs a launch and 8 bytes an output.  Fitted to
// 30 shapes of 65 to 1024 rows (N 2048 ... 10240, K 5120 ... 25600), it is within 12 % of the times of
// the tiles that matter.  us, with the former rule (768 workgroups wanted, no split from 256 on) / now:
//   128 x 10240 x 5120 29.9 / 22.2, 256 x 5120 x 8192 38.1 / 25.5, 200 x 5120 x 25600 107 / 51,
//   512 x 5120 x 25600 126 / 89, 1024 x 2048 x 7168 39.3 / 31.6
static void fp8_medium_plan(int M, int N, int KB, int& bm, int& bn, int& splits) {
  static const struct { int bm, bn; double t; } kTiles[] = {{64, 128, 0.65}, {128, 128, 1.02}, {64, 64, 0.5}, {128, 64, 0.75}};
  double best = -1;
  for (const auto& c : kTiles) {
    if (N % c.bn != 0 || (c.bm == 128 && c.bn == 64 && N % 128 == 0)) continue;
    const double wgs = (double)((M + c.bm - 1) / c.bm) * (N / c.bn);
    for (int s = 1; s <= fp8_splits_for(16, 16, KB); ++s) {
      const double r = wgs * s / 512, full = ceil(r), f = r <= 1 ? 1 : r + 0.4 * (full - r);
      const double us = f * ((KB + s - 1) / s + 4) * c.t + (s > 1 ? 4 + (double)s * M * N / 750e3 : 0);
      if (best < 0 || us < best) { best = us; bm = c.bm; bn = c.bn; splits = s; }
    }
  }
}

// Up to 64 rows: does the kernel whose workgroups split the reduction among their waves (launch_fp8_kgroups) take the
// call?  It has no planes and no second launch, but a workgroup reads the activations of its whole reduction for 16 to 64
// features, where planes give it a part for 64 or 128.  So by the time both should take, mean of weights in the cache and in memory, in
// us.  Groups: a start; the kilobytes of the fullest CU and of the mean one; the blocks of one group (and by rows); the
// workgroups of the fullest CU (and by rows); its blocks by rows squared.  Planes: a start; a second launch; the blocks of a
// workgroup (and by rows); a million weights; outputs of all planes; activations.  Fitted to 7348 random calls (N 64 ... 51200,
// K 128 ... 28160), mean error 6 to 8 %.  Beyond 64 million weights there is little to gain.  A tenth has to be gained, a quarter where the planes
// are one and no second launch goes away, or where the activations are large: below that 23 of 1600 calls were slower by more than 3 % with weights
// in one of the two places (15 x 2432 x 13952, from memory 17.2 / 20.3 the worst; 5 % at unsplit ones, from the cache), and now one is (0.969) of the 2565 of 2800
// random calls that are still taken, 1.41x on average from the cache and 1.44x from memory.  The plan is that of a full workspace: up to 64 rows none is accepted with fewer planes.
// us, planes then groups, weights in the cache (in memory): 16 x 3968 x 3328 7.8 / 4.8 (9.1 / 6.6), 54 x 6016 x 1408 7.6 / 5.8 (11.6 / 9.1),
// 1 x 2048 x 7168 8.4 / 5.8 (9.8 / 7.7), 16 x 12800 x 1024 6.9 / 4.7 (7.9 / 5.9), 1 x 10240 x 5120 12.6 / 10.7 (15.7 / 12.9);
// left with planes 64 x 10240 x 5120 16.6 / 19.7 (23.6 / 28.5), 16 x 5120 x 25600 25.4 / 32.6 (30.6 / 51).
static bool fp8_groups_pay(int M, int N, int K, const Fp8Plan& pl, int& bn, int& groups) {
  const int KB = K / 128;
  if (M > 64 || (long long)N * K > 64000000LL) return false;
  static const struct { int bn, groups; double start, most, mean, blocks, blocks_rows, wgs, wgs_rows, rows2; } kFit[] = {
      {16, 4, 1.9, 0.00224, 0.0115, 0.309, 0, 0.18, 0.238, 0.0423}, {16, 8, 1.63, 0.00178, 0.0112, 0.272, 0, 0.93, 0.288, 0.156},
      {32, 4, 1.87, 0.0042, 0.0139, 0.375, 0, 0.412, 0.353, 0.0322}, {64, 2, 2.29, 0.007, 0.0159, 0.311, 0.0334, 0.0771, 0.246, 0.00115}};
  const double rows = pl.bm / 16, nk = (double)N * K / 1e6;
  const int per = (KB + pl.splits - 1) / pl.splits;
  const double planes = 2.64 + (pl.splits > 1 ? 2.84 : 0) + per * (0.293 + 0.00617 * rows) + 0.114 * nk + 1.18 * pl.splits * (double)M * N / 1e6 + 4.19 * (double)M * K / 1e6;
  double best = planes / (pl.splits == 1 || (long long)M * K >= 65536 ? 1.25 : 1.1);
  bool pays = false;
  for (const auto& f : kFit) {
    // (eight groups of 32 rows are never the best, of 64 they do not fit the LDS; 64 features of 16 rows gain too little)
    if (KB < f.groups || (f.groups == 8 && pl.bm > 16) || (f.bn == 64 && pl.bm == 16)) continue;
    const int pass = f.bn / 2, a_rows = (pl.bm + pass - 1) / pass * pass;      // rows of a load pass; activation rows held
    const double kb = ((a_rows + f.bn) * 128 + f.bn * 16) / 1e3, wgs = (double)(N / f.bn) / 256, full = ceil(wgs), b = (KB + f.groups - 1) / f.groups;
    const double us = f.start + f.most * full * KB * kb + f.mean * wgs * KB * kb + b * (f.blocks + f.blocks_rows * rows) + full * (f.wgs + f.wgs_rows * rows) + f.rows2 * full * KB * rows * rows / 10;
    if (us < best) { best = us; bn = f.bn; groups = f.groups; pays = true; }
  }
  return pays;
}

// The splits a workspace was sized for before the tiles and splits above were chosen by time: up to 768
// workgroups of the four-wave tiles.  A caller who brings planes for them, by a size kept from an earlier
// release, still runs: a shape that needed none unsplit, one that needed fewer than it is now given
// with those it has room for.
static int fp8_four_wave_rows(int M, int N) {
  return M <= 16 ? 16 : M <= 32 ? 32 : M <= 64 ? 64 : M > 128 && N % 128 == 0 && (long long)((M + 127) / 128) * (N / 128) < 512 ? 64 : 128;
}
static int fp8_splits_needed(int M, int N, int K) {
  const int bm = fp8_four_wave_rows(M, N), KB = K / 128;
  const long long mb = (M + bm - 1) / bm;
  const long long wgs = N % 128 == 0 && mb * (N / 128) >= 256 ? mb * (N / 128) : mb * (N / 64);
  if (wgs >= 256) return 1;
  const int want = fp8_splits_for((int)((768 + wgs - 1) / wgs), 16, KB), per = (KB + want - 1) / want;
  return (KB + per - 1) / per;                         // no empty split
}

// false: the (forced) plan does not fit the shape
static bool fp8_plan(int M, int N, int K, Fp8Plan& pl) {
  const int KB = K / 128;
  int bm = fp8_four_wave_rows(M, N);
  // 128 features per workgroup measured fastest at every four-wave token-tile height up to 128 (two
  // or more workgroups per CU; 256 wide costs occupancy, 64 wide LDS traffic per matrix instruction).
  int bn = 128;
  // More than 64 rows take the 256 x 256 two-group tile where its rounds over the 256 CUs are at
  // least 60 % full: 4096 x 51200 x 5120 0.99 against 1.15 ms with the former 256 x 256 tile, 512 x
  // 51200 151 against 205 us, 128 x 51200 61 against 76 us, 1024 x 10240 (160 tiles) 67 against 78 us;
  // 320 tiles (62 %) tie, 80 tiles lose (200 x 20480: 60 against 44 us).  At 64 rows and fewer the
  // small tiles stream the weights as fast with more workgroups in flight (64 x 65536 x 8192: 126
  // against 134 us).
  const long long tiles256 = (long long)((M + 255) / 256) * (N / 256);
  // A reduction of fewer than four blocks does not hide its start and its write-out (4096 x 12800 x 256:
  // 47 against 45 us).
  const bool two_group = !g_fp8_mt && !g_fp8_nt && M > 64 && N % 256 == 0 && KB >= 4 &&
                         tiles256 * 5 >= 3 * 256 * ((tiles256 + 255) / 256);
  if (g_fp8_mt) bm = 16 * g_fp8_mt;
  else if (g_fp8_nt && M > 128 && N % 256 == 0 && tiles256 >= 512) bm = 256;      // (a forced width picks its height)
  if (bm != 16 && bm != 32 && bm != 64 && bm != 128 && bm != 256) return false;
  int splits = 1;
  if (two_group) {
    bm = bn = 256;
  } else if (M > 64 && !g_fp8_mt && !g_fp8_nt) {
    fp8_medium_plan(M, N, KB, bm, bn, splits);
  } else {
    const long long m_blocks = (M + bm - 1) / bm;
    while (bn > 64 && N % bn != 0) bn >>= 1;
    // small problems: narrower feature tiles first (more workgroups streaming weights) ...
    while (bn > 64 && m_blocks * (N / bn) < 256) bn >>= 1;
    if (g_fp8_nt) bn = 64 * g_fp8_nt;
    if ((bn != 64 && bn != 128 && bn != 256) || N % bn != 0 || (bm == 256 && bn == 64)) return false;
    // ... then a split of the reduction, each split at least four blocks long: up to two workgroups per CU, or
    // for 32 rows and fewer, whose planes (8 bytes an output and split) are small and whose workgroups
    // have less to load, about 2.75.  us by splits, weights in memory (in the cache):
    //   64 x 10240 x 5120 (160 workgroups a split) 3: 24.7 (16.7), 4: 27.2 (19.1), 5: 28.9 (20.3);  64 x 5120 x 25600 (80) 6: 44 (29), 10: 52 (35)
    //   16 x 10240 x 5120 3: 19.1 (13.3), 4: 17.9 (13.6), 5: 18.8 (14.8);  1 x 5120 x 25600 6: 36 (24), 8: 31 (23), 10: 31 (25)
    //   32 x 14336 x 4096 (224) 2: 21.3 (14.6), 3: 19.2 (14.7), 4: 20.1 (15.9);  1 x 2048 x 7168 (32) 8: 11.3 (7.4), 12: 11.0 (8.3), 14: 10.8 (8.6)
    const long long wgs = m_blocks * (N / bn);
    if (wgs < 256)
      splits = bm <= 32 ? fp8_splits_for((704 + (int)wgs / 2) / (int)wgs, wgs < 32 ? 16 : 12, KB) : fp8_splits_for(512 / (int)wgs, wgs < 32 ? 16 : 8, KB);
  }
  if (g_fp8_splits) splits = g_fp8_splits;
  if (splits < 1 || splits > KB) return false;
  const int per = (KB + splits - 1) / splits;
  splits = (KB + per - 1) / per;                       // no empty split
  pl = Fp8Plan{bm, bn, splits, per};
  return true;
}

extern "C" {

const char* moe_last_error(void) { return g_err; }

size_t moe_align_capacity(int T, int topk, int E, int block_m) {
  if (T < 0 || topk < 1 || E < 1 || !valid_block_m(block_m)) return 0;
  return align_capacity((long long)T * topk, E, block_m);
}

int moe_align_by_expert(const int32_t* topk_ids, int T, int topk, int E, int block_m,
                        int32_t* expert_counts, int32_t* expert_offsets, int32_t* sorted_slot_ids,
                        int32_t* block_expert_ids, int32_t* num_padded, void* stream) {
  if (T < 0 || topk < 1 || E < 1) return fail(MOE_INVALID_ARGUMENT, "need T >= 0, topk >= 1, E >= 1");
  if (!valid_block_m(block_m)) return fail(MOE_INVALID_ARGUMENT, "block_m must be 16, 32, 64, 128 or 256");
  if (E > 1024) return fail(MOE_UNSUPPORTED_SHAPE, "E = %d exceeds 1024", E);
  const long long S = (long long)T * topk;
  if (S > 0x7fffffffLL / 2) return fail(MOE_UNSUPPORTED_SHAPE, "T*topk too large");
  if (!expert_counts || !expert_offsets || !num_padded || (S > 0 && (!topk_ids || !sorted_slot_ids || !block_expert_ids)))
    return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  const size_t cap = align_capacity(S, E, block_m);
  const int err = launch_align(topk_ids, (int)S, E, block_m, (int)cap, expert_counts, expert_offsets,
                               sorted_slot_ids, block_expert_ids, num_padded, nullptr, (hipStream_t)stream);
  if (err != 0) return hip_fail(err, "align launch");
  return MOE_OK;
}

int moe_w4a16_grouped_gemm(const void* A, int row_div, const int32_t* qweight, const void* scales,
                           const uint8_t* zeros, const int32_t* sorted_slot_ids,
                           const int32_t* block_expert_ids, const int32_t* num_padded, int num_slots,
                           int E, int N_out, int K_in, int group_size, int block_m, moe_dtype dt,
                           void* C, void* stream) {
  GemmArgs a{A, row_div, qweight, scales, zeros, sorted_slot_ids, block_expert_ids, num_padded,
             num_slots, E, N_out, K_in, group_size, block_m, (int)dt, C, N_out, 0, 0};
  return run_gemm(a, (hipStream_t)stream);
}

int moe_w4a16_dense_gemm(const void* A, const int32_t* qweight, const void* scales, const uint8_t* zeros,
                         int M, int N_out, int K_in, int group_size, moe_dtype dt, void* C, void* stream) {
  if (M < 0) return fail(MOE_INVALID_ARGUMENT, "need M >= 0");
  const int block_m = M <= 16 ? 16 : (M <= 32 ? 32 : 64);
  GemmArgs a{A, 1, qweight, scales, zeros, nullptr, nullptr, nullptr,
             M, 1, N_out, K_in, group_size, block_m, (int)dt, C, N_out, 0, 0};
  a.dense = 1;
  return run_gemm(a, (hipStream_t)stream);
}

int moe_route_topk(const float* logits, const float* bias, int T, int E, int topk,
                   int32_t* topk_ids, float* topk_weights, void* stream) {
  if (T < 0 || E < 1 || topk < 1) return fail(MOE_INVALID_ARGUMENT, "need T >= 0, E >= 1, topk >= 1");
  if (E > 1024) return fail(MOE_UNSUPPORTED_SHAPE, "E = %d exceeds 1024", E);
  if (topk > E || topk > 64) return fail(MOE_UNSUPPORTED_SHAPE, "topk = %d exceeds min(E, 64)", topk);
  if (T == 0) return MOE_OK;
  if (!logits || !topk_ids || !topk_weights) return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  const int err = launch_route_topk(logits, bias, T, E, topk, topk_ids, topk_weights, (hipStream_t)stream);
  if (err != 0) return hip_fail(err, "router launch");
  return MOE_OK;
}

int moe_probe_stream_read(const void* src, size_t bytes, void* sink, void* stream) {
  if (!src || !sink || bytes < 16 || ((uintptr_t)src % 16) != 0)
    return fail(MOE_INVALID_ARGUMENT, "probe needs a 16-byte aligned source of at least 16 bytes and a sink");
  const int err = launch_stream_read(src, bytes, (uint32_t*)sink, 256 * 16, (hipStream_t)stream);
  if (err != 0) return hip_fail(err, "stream-read probe launch");
  return MOE_OK;
}

int moe_probe_mfma(void* sink, int iters, void* stream) {
  if (!sink || iters < 1) return fail(MOE_INVALID_ARGUMENT, "probe needs a sink and iters >= 1");
  const int err = launch_mfma_loop((float*)sink, 512, iters, (hipStream_t)stream);
  if (err != 0) return hip_fail(err, "MFMA probe launch");
  return MOE_OK;
}

int moe_probe_issue_mix(void* sink, int iters, int valu_per_mfma, int lds_reads_per_8_mfma, void* stream) {
  if (!sink || iters < 1) return fail(MOE_INVALID_ARGUMENT, "probe needs a sink and iters >= 1");
  const int err = launch_issue_mix((float*)sink, iters, valu_per_mfma, lds_reads_per_8_mfma, (hipStream_t)stream);
  if (err == -1)
    return fail(MOE_UNSUPPORTED_SHAPE, "issue-mix probe: valu_per_mfma must be 0, 1, 2, 3, 4 or 6 and "
                "lds_reads_per_8_mfma 0, 2, 4 or 8");
  if (err != 0) return hip_fail(err, "issue-mix probe launch");
  return MOE_OK;
}

int moe_silu_mul(const void* H, void* act, int S, int N, moe_dtype dt, void* stream) {
  if (S < 0 || N < 1) return fail(MOE_INVALID_ARGUMENT, "need S >= 0 and N >= 1");
  if (dt != MOE_F16 && dt != MOE_BF16) return fail(MOE_INVALID_ARGUMENT, "dt must be MOE_F16 or MOE_BF16");
  if (S == 0) return MOE_OK;
  if (!H || !act) return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  if (N % 8 == 0 && ((uintptr_t)H | (uintptr_t)act) % 16 != 0)
    return fail(MOE_INVALID_ARGUMENT, "H and act must be 16-byte aligned");
  const int err = launch_silu_mul(H, act, S, N, (int)dt, (hipStream_t)stream);
  if (err != 0) return hip_fail(err, "silu_mul launch");
  return MOE_OK;
}

int moe_combine(const void* Y, const float* topk_weights, void* out, int T, int topk, int K, moe_dtype dt,
                void* stream) {
  if (T < 0 || topk < 1 || K < 1) return fail(MOE_INVALID_ARGUMENT, "need T >= 0, topk >= 1, K >= 1");
  if (dt != MOE_F16 && dt != MOE_BF16) return fail(MOE_INVALID_ARGUMENT, "dt must be MOE_F16 or MOE_BF16");
  if (T == 0) return MOE_OK;
  if (!Y || !topk_weights || !out) return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  if (K % 8 == 0 && ((uintptr_t)Y | (uintptr_t)out) % 16 != 0)
    return fail(MOE_INVALID_ARGUMENT, "Y and out must be 16-byte aligned");
  const int err = launch_combine(Y, 0, 1, topk_weights, nullptr, 0, out, T, topk, K, (int)dt, (hipStream_t)stream);
  if (err != 0) return hip_fail(err, "combine launch");
  return MOE_OK;
}

int moe_combine_masked(const void* Y, const float* topk_weights, const int32_t* topk_ids, int E, void* out, int T,
                       int topk, int K, moe_dtype dt, void* stream) {
  if (T < 0 || topk < 1 || K < 1 || E < 1) return fail(MOE_INVALID_ARGUMENT, "need T >= 0, topk >= 1, K >= 1, E >= 1");
  if (dt != MOE_F16 && dt != MOE_BF16) return fail(MOE_INVALID_ARGUMENT, "dt must be MOE_F16 or MOE_BF16");
  if (T == 0) return MOE_OK;
  if (!Y || !topk_weights || !topk_ids || !out) return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  if (K % 8 == 0 && ((uintptr_t)Y | (uintptr_t)out) % 16 != 0)
    return fail(MOE_INVALID_ARGUMENT, "Y and out must be 16-byte aligned");
  const int err = launch_combine(Y, 0, 1, topk_weights, topk_ids, E, out, T, topk, K, (int)dt, (hipStream_t)stream);
  if (err != 0) return hip_fail(err, "combine launch");
  return MOE_OK;
}

size_t moe_w4a16_layer_workspace_bytes(int T, int K, int N, int E, int topk, moe_dtype dt) {
  if (T < 0 || K < 1 || N < 1 || E < 1 || topk < 1) return 0;
  return layer_workspace(T, K, N, E, topk, (int)dt);
}

int moe_layer_block_m(int T, int E, int topk) {
  if (T < 0 || E < 1 || topk < 1) return 0;
  return pick_block_m((long long)T * topk, E);
}

int moe_layer_block_m_for(int T, int K, int N, int E, int topk, int group_size) {
  if (T < 0 || K < 1 || N < 1 || E < 1 || topk < 1 || group_size < 1) return 0;
  if (g_force_block_m > 0) return g_force_block_m;
  return pick_block_m((long long)T * topk, E, layer_wide_ok(K, N, group_size), layer_wide_ok(K, N, group_size));
}

}  // extern "C"

// Up to this many tokens the router runs inside the bucketing workgroup (one launch); beyond it the
// many-workgroup router kernel plus the bucketing kernel are faster than one CU routing everything
// (measured, 256 experts, top-8: fused 10.6 / 15.0 / 23.4 us at 16 / 64 / 128 tokens against
// 15.1 us for the two launches).
constexpr int kFusedRouteMaxTokens = 64;

struct RouteArgs {            // routed layer: the layer's first step computes ids / weights itself
  const float* logits = nullptr;
  const float* bias = nullptr;
  int32_t* ids = nullptr;     // [T, topk] tables to fill (inside the caller's workspace)
  float* weights = nullptr;
};

// Does the pass over the activations run in the launch of the bucketing?  A launch and its gap less, 2.5 us (64 tokens of 4096 x 14336
// 167.0 -> 164.6, 512 of 2048 x 2048 147.5 -> 144.9, FP8 64 of 2048 x 1408 129.2 -> 126.6).  Where the pass is long the bucketing, one workgroup that
// now shares its CU and the caches with it, takes longer: 4096 tokens of 7168 3405 -> 3429 us, FP8 the same either way; 4096 of 2048
// in FP8 419 -> 415.
static bool runs_beside(long long T, int K) { return T * K <= 1LL << 23; }

// router (+ bucketing): one launch for small batches, two otherwise
static int route_and_align(const RouteArgs& r, int T, int E, int topk, int block_m, int32_t* counts, int32_t* offsets,
                           int32_t* sorted, int32_t* blocks, int32_t* num_padded, const RowsJob* job, hipStream_t stream) {
  const long long S = (long long)T * topk;
  const int cap = (int)align_capacity(S, E, block_m);
  int err;
  if (T <= kFusedRouteMaxTokens) {
    err = launch_route_align(r.logits, r.bias, T, E, topk, r.ids, r.weights, block_m, cap, counts, offsets, sorted,
                             blocks, num_padded, job, stream);
    if (err != 0) return hip_fail(err, "router + align launch");
    return MOE_OK;
  }
  err = launch_route_topk(r.logits, r.bias, T, E, topk, r.ids, r.weights, stream);
  if (err != 0) return hip_fail(err, "router launch");
  err = launch_align(r.ids, (int)S, E, block_m, cap, counts, offsets, sorted, blocks, num_padded, job, stream);
  if (err != 0) return hip_fail(err, "align launch");
  return MOE_OK;
}

// One product of the layer on the two-group tile.
static int run_twogroup(const void* A, const float* bias_rows, int row_div, const int32_t* qw, const void* sc,
                        const uint8_t* z, const int32_t* sorted, const int32_t* blocks, const int32_t* num_padded,
                        int num_slots, int E, int N_out, int K_in, int dt, int fuse, int pre, void* C, hipStream_t stream) {
  TwoGroupParams p;
  p.A = A; p.bias_rows = bias_rows; p.row_div = row_div;
  p.qweight = qw; p.scales = sc; p.zeros = z;
  p.sorted_slot_ids = sorted; p.block_expert_ids = blocks; p.num_padded = num_padded;
  p.num_slots = num_slots; p.E = E; p.N_out = N_out; p.K_in = K_in; p.C = C; p.pre = pre;
  p.c_bytes = c_plane_bytes(num_slots, fuse ? N_out : 4LL * N_out);      // 16-bit act of half the columns, or float32
  p.n_tiles = N_out / 256;
  // Several tiles per workgroup where the reduction is short (a tile's start and end cost about as
  // much as four stages), as long as a few rounds over the CUs remain.
  const long long est_blocks = (num_slots + 255) / 256 + (num_slots < E ? num_slots : E) / 2;
  int tpw = 56 / (K_in / 128);
  if (tpw < 1) tpw = 1;
  if (tpw > p.n_tiles) tpw = p.n_tiles;
  while (tpw > 1 && (p.n_tiles % tpw != 0 || est_blocks * (p.n_tiles / tpw) < 1024)) --tpw;
  if (g_force_tpw > 0) tpw = g_force_tpw < p.n_tiles ? g_force_tpw : p.n_tiles;
  p.tiles_per_wg = tpw;
  const long long grid = (long long)(align_capacity(num_slots, E, 256) / 256) * ((p.n_tiles + tpw - 1) / tpw);
  if (grid > 0x7fffffffLL) return fail(MOE_UNSUPPORTED_SHAPE, "grid too large");
  const int plan[9] = {16, 2, 128, 1, tpw, 1, K_in, fuse, 8};
  for (int i = 0; i < 9; ++i) g_last_plan[i] = plan[i];
  const int err = (dt == MOE_F16 ? launch_twogroup_f16 : launch_twogroup_bf16)(p, fuse, (int)grid, stream);
  if (err != 0) return hip_fail(err, "two-group GEMM launch");
  return MOE_OK;
}

// One product of the layer on the 64-slot tile.
static int run_mid(const void* A, const float* sums, int row_div, const int32_t* qw, const void* sc, const uint8_t* z,
                   const int32_t* sorted, const int32_t* blocks, const int32_t* num_padded, int num_slots, int E, int N_out,
                   int K_in, int dt, int fuse, int pre, int want_splits, void* C, int* used_splits, hipStream_t stream) {
  MidParams p;
  p.A = A; p.sums = sums; p.row_div = row_div;
  p.qweight = qw; p.scales = sc; p.zeros = z;
  p.sorted_slot_ids = sorted; p.block_expert_ids = blocks; p.num_padded = num_padded;
  p.num_slots = num_slots; p.E = E; p.N_out = N_out; p.K_in = K_in; p.C = C;
  p.n_tiles = N_out / 128;
  p.k_splits = 1; p.k_span = K_in; p.split_stride = (long long)num_slots * N_out;
  if (want_splits > 1) {               // whole panels of 1024, every range non-empty
    const int npan = K_in / 1024, per = (npan + want_splits - 1) / want_splits;
    p.k_splits = (npan + per - 1) / per;
    p.k_span = per * 1024;
  }
  if (used_splits) *used_splits = p.k_splits;
  const long long est_blocks = (num_slots + 63) / 64 + (num_slots < E ? num_slots : E) / 2;
  int tpw = (48 + p.k_span / 256 - 1) / (p.k_span / 256);
  if (tpw > 8) tpw = 8;
  if (tpw > p.n_tiles) tpw = p.n_tiles;
  while (tpw > 1 && (p.n_tiles % tpw != 0 || est_blocks * (p.n_tiles / tpw) * p.k_splits < 1536)) --tpw;
  if (g_force_tpw > 0) tpw = g_force_tpw < p.n_tiles ? g_force_tpw : p.n_tiles;
  p.tiles_per_wg = tpw;
  const long long grid = mid_grid(align_capacity(num_slots, E, 64) / 64, (p.n_tiles + tpw - 1) / tpw * p.k_splits);
  if (grid > 0x7fffffffLL) return fail(MOE_UNSUPPORTED_SHAPE, "grid too large");
  const int plan[9] = {4, 2, 256, 1, tpw, p.k_splits, p.k_span, fuse, 4};
  for (int i = 0; i < 9; ++i) g_last_plan[i] = plan[i];
  const int err = (dt == MOE_F16 ? launch_mid_f16 : launch_mid_bf16)(p, fuse, pre, (int)grid, stream);
  if (err != 0) return hip_fail(err, "64-slot GEMM launch");
  return MOE_OK;
}

// Do the vector-product kernels (few_tokens.hip) take the call?  They have two launches instead of four, but
// read an expert's weights once for every slot.  So up to 32 slots, and by the time both sides should take, in us with
// weights that are not in a cache: a start, then the vectors by the weights of every slot and by the activations a workgroup of gate/up
// stages, the tiles by the weights of every expert met, by the reduction that a workgroup walks and by what a reduction that is no multiple
// of 1024 loses (no register scales, no splits).  The host does not know the routing: the experts met are the mean of
// what independent tokens meet and of what tokens meet that all choose the same.  Fitted to 5180 calls of 1 to 32 tokens (K 128 ... 8192,
// N 128 ... 14336, 4 to 256 experts, top 1 to 10), within 10 % (vector) and 6 % (tiled) on average.
// Calls it takes that are slower than on the tiles by more than 3 %, cached or not / calls it leaves there that would be faster by more:
// independent tokens 0 / 846 of 8538 (the fits saw 5180 of them), experts weighted as 1 / rank 5 / 116 of 2073, all tokens alike 9 / 72 of
// 2089 (20 % at most), all counted with the products' former times.  Above 128 million weights for all slots there is least to gain (0.8 to 1) and alike tokens
// cost most (31 of the 2089 with twice that).  The products' present form is 2 to 15 % faster, so the line errs to the side of the tiles: of 4440 random calls that it
// takes (independent tokens, a third of them with wide activations, plain layout) all are faster than on the tiles, 1.08x the least, 2.3x on average with weights in the cache and
// 2.0x in memory.  More than 16 tokens, one expert each, keep the line they had, five rounds of down workgroups; 150 of the calls left
// are beyond it.
// Tiled / vector, weights in memory (in the cache), fp16, experts drawn from 64 where there are 256:
//   7168x2048, 256 experts, top 8: 1 token 62.1 / 44.9 (56.5 / 35.0);   top 1: 4 tokens 47.6 / 27.6 (43.5 / 19.7), 8 57.6 / 42.6
//   4096x14336, 8, top 2: 1 token 57.9 / 46.1 (52.1 / 35.5);   2048x1408, 64, top 6: 4 tokens 43.9 / 33.6, 5 48.5 / 38.2
//   2048x2048, 64: top 1, 6 tokens 28.2 / 18.7, 8 29.1 / 20.5, 16 38.7 / 28.5
//   1024x1024, 64: top 2, 12 tokens 28.0 / 18.3, 16 29.0 / 19.3;   256x512, 8, top 2: 16 tokens 22.0 / 9.1
static bool few_tokens_pay(int T, int topk, int E, int K, int N, int dt, int pre) {
  const long long S = (long long)T * topk, nk = (long long)N * K;
  if (S > 32 || S * nk > 128000000LL || (T > 16 && T * (long long)K > 20480)) return false;
  static const struct { double vector, slot, stage, tiled, expert, walk, odd_k, odd_n; } kFit[2][2] = {      // [operand order][bf16]; sizes in thousands
      {{8.1, 0.288, 0.85, 18.0, 0.260, 2.17, 0.78, 3.23}, {8.1, 0.268, 0.75, 18.2, 0.253, 2.40, 0.69, 3.29}},
      {{8.6, 0.293, 0.52, 18.9, 0.265, 1.15, 0, 0}, {8.25, 0.270, 0.68, 18.9, 0.256, 1.48, 0, 0}}};
  const auto& f = kFit[pre ? 1 : 0][dt == MOE_BF16 ? 1 : 0];
  const double mw = nk / 1e6, k = K / 1e3, n = N / 1e3;        // a million weights of one of an expert's three matrices
  const double alike = topk < E ? topk : E, experts = 0.5 * (E * (1 - pow(1 - alike / E, T)) + alike);
  return f.vector + f.slot * S * mw + f.stage * k < f.tiled + f.expert * experts * mw + f.walk * k + (K % 1024 ? f.odd_k * k : 0) + (N % 1024 ? f.odd_n * n : 0);
}
static int layer_impl(const void* X, const int32_t* topk_ids, const float* topk_weights,
                      const int32_t* qw1, const void* s1, const uint8_t* z1,
                      const int32_t* qw2, const void* s2, const uint8_t* z2,
                      void* out, int T, int K, int N, int E, int topk, int group_size, moe_dtype dt,
                      void* workspace, size_t workspace_bytes, void* stream_v, int pre,
                      const RouteArgs* route = nullptr) {
  hipStream_t stream = (hipStream_t)stream_v;
  if (T < 0 || K < 1 || N < 1 || E < 1 || topk < 1 || group_size < 1)
    return fail(MOE_INVALID_ARGUMENT, "need T >= 0 and positive K, N, E, topk, group_size");
  if (dt != MOE_F16 && dt != MOE_BF16) return fail(MOE_INVALID_ARGUMENT, "dt must be MOE_F16 or MOE_BF16");
  if (E > 1024) return fail(MOE_UNSUPPORTED_SHAPE, "E = %d exceeds 1024", E);
  if (group_size % 32 != 0 || K % group_size != 0 || N % group_size != 0)
    return fail(MOE_UNSUPPORTED_SHAPE, "group_size %d must be a multiple of 32 dividing K=%d and N=%d", group_size, K, N);
  if (K % 16 != 0 || N % 16 != 0) return fail(MOE_UNSUPPORTED_SHAPE, "K and N must be multiples of 16");
  if (K / group_size > kMaxGroups || N / group_size > kMaxGroups)
    return fail(MOE_UNSUPPORTED_SHAPE, "more than %d quantisation groups per row", kMaxGroups);
  if (T == 0) return MOE_OK;
  if (!X || !topk_ids || !topk_weights || !qw1 || !s1 || !z1 || !qw2 || !s2 || !z2 || !out || !workspace)
    return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  if (((uintptr_t)workspace % 256) != 0) return fail(MOE_INVALID_ARGUMENT, "workspace must be 256-byte aligned");
  if (((uintptr_t)out % 16) != 0) return fail(MOE_INVALID_ARGUMENT, "out must be 16-byte aligned");
  const Workspace w = carve(T, K, N, E, topk, (int)dt);
  if (workspace_bytes < w.base)
    return fail(MOE_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", workspace_bytes, layer_workspace(T, K, N, E, topk, (int)dt));
  const long long S = (long long)T * topk;
  if (S > 0x7fffffffLL / 2) return fail(MOE_UNSUPPORTED_SHAPE, "T*topk too large");
  // Operand-order weights: the same shapes and alignments at every token number, whichever kernel runs.
  if (pre) {
    if ((((uintptr_t)X | (uintptr_t)qw1 | (uintptr_t)qw2) % 16) != 0 || (((uintptr_t)s1 | (uintptr_t)s2) % 2) != 0)
      return fail(MOE_INVALID_ARGUMENT, "X and the packed weights must be 16-byte, scales 2-byte aligned");
    if (group_size != 128 || K % 1024 != 0 || N % 1024 != 0 || (((uintptr_t)s1 | (uintptr_t)s2) % 16) != 0 ||
        (((uintptr_t)z1 | (uintptr_t)z2) % 8) != 0 || (long long)E * 2 * N * (K / 128) >= (1LL << 31))
      return fail(MOE_UNSUPPORTED_SHAPE, "operand-order weights need group_size 128, K %% 1024 == 0, N %% 1024 == 0, "
                  "16-byte aligned scales and 8-byte aligned zero points");
  }

  unsigned char* base = (unsigned char*)workspace;
  int32_t* counts = (int32_t*)(base + w.counts);
  int32_t* offsets = (int32_t*)(base + w.offsets);
  int32_t* num_padded = (int32_t*)(base + w.num_padded);
  int32_t* sorted = (int32_t*)(base + w.sorted);
  int32_t* blocks = (int32_t*)(base + w.blocks);
  void* act = base + w.act;
  void* Y = base + w.Y;
  // Two-group and 64-slot tile: their shapes, every tuning hook that asks for another kernel at rest, 32-bit offsets
  // in range, room for the row sums (bf16), and the alignment of the other register-scale tiles, so
  // that scales and zero points of less are taken or refused alike at every token number.
  const bool ordered =
      layer_wide_ok(K, N, group_size) && g_scale_path != 1 && workspace_bytes >= w.base + w.sums &&
      (((uintptr_t)X | (uintptr_t)qw1 | (uintptr_t)qw2) % 16) == 0 && (((uintptr_t)s1 | (uintptr_t)s2) % 16) == 0 &&
      (((uintptr_t)z1 | (uintptr_t)z2) % 8) == 0 && (long long)N * K < (1LL << 31) &&
      (long long)E * 2 * N * (K / 128) < (1LL << 31) && (long long)T * K * 2 < (1LL << 31) && S * N * 2 < (1LL << 31);
  const bool mid_fits = mid_pays(S, E, K, N, (int)dt, pre);
  const bool mid = ordered && (g_force_block_m == 64 || (g_force_block_m == 0 && mid_fits));
  const bool two_group = ordered && g_force_ksplit == 0 &&
                         (g_force_block_m == 256 || (g_force_block_m == 0 && !mid_fits && twogroup_pays(S, E, K, N, (int)dt, pre)));
  // a forced bucketing block wins; a forced token tile (tuning hook) also fixes the block
  const int block_m = two_group ? 256 : mid ? 64 : g_force_block_m > 0 ? g_force_block_m
                      : (g_force_mt == 1 || g_force_mt == 2 || g_force_mt == 4 || g_force_mt == 8)
                          ? 16 * g_force_mt : pick_block_m(S, E, layer_wide_ok(K, N, group_size), !pre && layer_wide_ok(K, N, group_size));
  const bool ev = g_nevents == 5;
  auto mark = [&](int i) { if (ev) (void)hipEventRecord((hipEvent_t)g_events[i], stream); };
  int err;
  // A few tokens: vector products, unless a tuning hook asks for a tile; whole groups of 128, 16-byte
  // aligned words and activations, 32-bit offsets into an expert, room for act's vectors.
  const bool few = few_tokens_pay(T, topk, E, K, N, (int)dt, pre) && group_size == 128 && few_tokens_fit(topk, K, N) && g_force_block_m == 0 &&
                   w.few_end <= workspace_bytes &&
                   g_force_mt == 0 && g_force_nt == 0 && g_force_ksplit == 0 && g_scale_path == 0 && g_force_tpw == 0 && g_wide_mode == 0 &&
                   (((uintptr_t)X | (uintptr_t)qw1 | (uintptr_t)qw2) % 16) == 0 && (((uintptr_t)s1 | (uintptr_t)s2) % 2) == 0 &&
                   (long long)N * K < (1LL << 31);
  if (few) {
    mark(0);
    const FewRoute inside{route ? route->logits : nullptr, route ? route->bias : nullptr, route ? route->ids : nullptr, route ? route->weights : nullptr};
    const bool fused = route && E <= kFewRouteE && topk <= kFewRouteTopk;
    if (route && !fused) {
      err = launch_route_topk(route->logits, route->bias, T, E, topk, route->ids, route->weights, stream);
      if (err != 0) return hip_fail(err, "router launch");
    }
    mark(1);
    err = launch_few_gate_up(X, fused ? &inside : nullptr, topk_ids, qw1, s1, z1, act, (uint32_t*)(base + w.few_units), T, topk, E, K, N, (int)dt, pre, stream);
    if (err != 0) return hip_fail(err, "few-token gate/up launch");
    mark(2);
    err = launch_few_down(act, (const uint32_t*)(base + w.few_units), topk_ids, topk_weights, qw2, s2, z2, out, T, topk, E, K, N, (int)dt, pre, stream);
    if (err != 0) return hip_fail(err, "few-token down launch");
    for (int& v : g_last_plan) v = 0;       // no tile
    mark(3);
    mark(4);
    return MOE_OK;
  }

  // The two-group and the 64-slot tile read the rows of X in another order (bf16: and their sums); they live where Y will be
  // written: Y is written last.
  float* const xsum = dt == MOE_BF16 ? (float*)((unsigned char*)Y + round_up((size_t)T * K * 2, 256)) : nullptr;
  const bool reorder = two_group || mid, beside = reorder && runs_beside(T, K);
  const int deal = two_group ? 0 : 1;
  const float factor = two_group ? 47.f : kZeroUnit;
  RowsJob job;
  if (beside) job = prepare_job(X, T, K, (int)dt, deal, Y, xsum, factor);
  mark(0);
  if (route) {
    const int rst = route_and_align(*route, T, E, topk, block_m, counts, offsets, sorted, blocks, num_padded, &job, stream);
    if (rst != MOE_OK) return rst;
  } else {
    err = launch_align(topk_ids, (int)S, E, block_m, (int)align_capacity(S, E, block_m), counts, offsets,
                       sorted, blocks, num_padded, &job, stream);
    if (err != 0) return hip_fail(err, "align launch");
  }
  if (reorder && !beside) {
    err = launch_prepare_rows(X, T, K, (int)dt, deal, Y, xsum, factor, stream);
    if (err != 0) return hip_fail(err, "activation reorder launch");
  }

  if (two_group) {
    float* const asum = dt == MOE_BF16 ? (float*)(base + w.base) : nullptr;
    mark(1);
    int st = run_twogroup(Y, xsum, topk, qw1, s1, z1, sorted, blocks, num_padded, (int)S, E, 2 * N, K, (int)dt, 1, pre, act, stream);
    if (st != MOE_OK) return st;
    mark(2);
    if (asum) {
      err = launch_prepare_rows(act, S, N, (int)dt, 0, nullptr, asum, 47.f, stream);
      if (err != 0) return hip_fail(err, "row sum launch");
    }
    st = run_twogroup(act, asum, 1, qw2, s2, z2, sorted, blocks, num_padded, (int)S, E, K, N, (int)dt, 0, pre, Y, stream);
    if (st != MOE_OK) return st;
    mark(3);
    err = launch_combine(Y, 1, 1, topk_weights, topk_ids, E, out, T, topk, K, (int)dt, stream);
    if (err != 0) return hip_fail(err, "combine launch");
    mark(4);
    return MOE_OK;
  }
  if (mid) {
    // reduction splits of the down product: as many partial planes as the caller's workspace holds
    const size_t plane = (size_t)S * K * 4;
    size_t want = g_force_ksplit > 0 ? (size_t)g_force_ksplit : w.mid_splits;
    while (want > 1 && end_of_planes(w, plane, want) + w.sums > workspace_bytes) --want;
    float* const asum = dt == MOE_BF16 ? (float*)(base + end_of_planes(w, plane, want)) : nullptr;
    mark(1);
    int st = run_mid(Y, xsum, topk, qw1, s1, z1, sorted, blocks, num_padded, (int)S, E, 2 * N, K, (int)dt, 1, pre, 1, act, nullptr, stream);
    if (st != MOE_OK) return st;
    mark(2);
    if (asum) {
      // (act's runs are in the order the kernel reads; the sums do not mind)
      err = launch_prepare_rows(act, S, N, (int)dt, 1, nullptr, asum, kZeroUnit, stream);
      if (err != 0) return hip_fail(err, "row sum launch");
    }
    int planes = 1;
    st = run_mid(act, asum, 1, qw2, s2, z2, sorted, blocks, num_padded, (int)S, E, K, N, (int)dt, 0, pre, (int)want, Y, &planes, stream);
    if (st != MOE_OK) return st;
    mark(3);
    err = launch_combine(Y, 1, planes, topk_weights, topk_ids, E, out, T, topk, K, (int)dt, stream);
    if (err != 0) return hip_fail(err, "combine launch");
    mark(4);
    return MOE_OK;
  }
  mark(1);
  GemmArgs g1{X, topk, qw1, s1, z1, sorted, blocks, num_padded, (int)S, E, 2 * N, K, group_size, block_m,
              (int)dt, act, N, N, 0};
  g1.pre = pre;
  int st = run_gemm(g1, stream);
  if (st != MOE_OK) return st;

  mark(2);
  GemmArgs g2{act, 1, qw2, s2, z2, sorted, blocks, num_padded, (int)S, E, K, N, group_size, block_m,
              (int)dt, Y, K, 0, 1};
  // reduction splits: as many partial planes as the caller's workspace holds
  int want = g_force_ksplit > 0 ? g_force_ksplit : pick_k_splits(S, E, K, N, block_m);
  const size_t planes_fit = (workspace_bytes - w.Y) / ((size_t)S * K * 4);
  if ((size_t)want > planes_fit) want = (int)planes_fit;
  int planes = 1;
  g2.k_splits = want;
  g2.used_splits = &planes;
  g2.pre = pre;
  st = run_gemm(g2, stream);
  if (st != MOE_OK) return st;

  mark(3);
  err = launch_combine(Y, 1, planes, topk_weights, topk_ids, E, out, T, topk, K, (int)dt, stream);
  if (err != 0) return hip_fail(err, "combine launch");
  mark(4);
  return MOE_OK;
}

extern "C" {

int moe_w4a16_layer(const void* X, const int32_t* topk_ids, const float* topk_weights,
                    const int32_t* qw1, const void* s1, const uint8_t* z1,
                    const int32_t* qw2, const void* s2, const uint8_t* z2,
                    void* out, int T, int K, int N, int E, int topk, int group_size, moe_dtype dt,
                    void* workspace, size_t workspace_bytes, void* stream) {
  return layer_impl(X, topk_ids, topk_weights, qw1, s1, z1, qw2, s2, z2, out, T, K, N, E, topk, group_size, dt,
                    workspace, workspace_bytes, stream, 0);
}

int moe_w4a16_layer_prepacked(const void* X, const int32_t* topk_ids, const float* topk_weights,
                              const int32_t* qw1p, const void* s1, const uint8_t* z1,
                              const int32_t* qw2p, const void* s2, const uint8_t* z2,
                              void* out, int T, int K, int N, int E, int topk, int group_size, moe_dtype dt,
                              void* workspace, size_t workspace_bytes, void* stream) {
  return layer_impl(X, topk_ids, topk_weights, qw1p, s1, z1, qw2p, s2, z2, out, T, K, N, E, topk, group_size, dt,
                    workspace, workspace_bytes, stream, 1);
}

// ---- the layer for callers that cannot allocate ---------------------------------------------
// Same kernels as moe_w4a16_layer; the bucketing tables, `act` and the float32 down-projection
// planes live in a fixed device array of this module instead of a caller workspace.  Every GPU
// the library runs on holds its own copy of the array (at its own address) until the process ends.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Device address of `scratch` on the current device, resolved once per device.  (In host code the
// array's name is only a handle for hipGetSymbolAddress, never an address to hand to a kernel.)
static int static_scratch(void** ptr) {
  constexpr int kMaxDev = 64;
  static void* ptrs[kMaxDev] = {};
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return hip_fail((int)err, "hipGetDevice");
  if (dev < 0 || dev >= kMaxDev) return fail(MOE_UNSUPPORTED_SHAPE, "device index %d outside [0, %d)", dev, kMaxDev);
  void* p = __atomic_load_n(&ptrs[dev], __ATOMIC_ACQUIRE);
  if (!p) {
    err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (err != hipSuccess || !p) return hip_fail((int)err, "hipGetSymbolAddress(scratch)");
    __atomic_store_n(&ptrs[dev], p, __ATOMIC_RELEASE);      // racing first calls resolve the same address
  }
  *ptr = p;
  return MOE_OK;
}

int moe_w4a16_layer_noalloc(const void* X, const int32_t* topk_ids, const float* topk_weights,
                            const int32_t* qw1, const void* s1, const uint8_t* z1,
                            const int32_t* qw2, const void* s2, const uint8_t* z2,
                            void* out, int T, int K, int N, int E, int topk, int group_size, moe_dtype dt,
                            void* stream) {
  if (T < 0 || K < 1 || N < 1 || E < 1 || topk < 1)
    return fail(MOE_INVALID_ARGUMENT, "need T >= 0 and positive K, N, E, topk, group_size");
  const size_t need = carve(T, K, N, E, topk, (int)dt).base;
  if (need > kStaticScratchBytes)
    return fail(MOE_WORKSPACE_TOO_SMALL,
                "moe_w4a16_layer_noalloc: these sizes need %zu bytes of scratch, the built-in array holds %zu; "
                "use moe_w4a16_layer with a caller workspace", need, kStaticScratchBytes);
  void* ptr = nullptr;
  const int st = static_scratch(&ptr);
  if (st != MOE_OK) return st;
  // nothing in the array has to start at zero: the bucketing kernel writes every table entry it or
  // the GEMMs read, and act / Y rows are read only for slots whose rows this call wrote
  return layer_impl(X, topk_ids, topk_weights, qw1, s1, z1, qw2, s2, z2, out, T, K, N, E, topk, group_size, dt,
                    ptr, kStaticScratchBytes, stream, 0);
}

int moe_repack_qweight(const int32_t* qweight, int E, int N_out, int K_in, int paired, int32_t* out, void* stream) {
  if (E < 1 || N_out < 1 || K_in < 1) return fail(MOE_INVALID_ARGUMENT, "need positive E, N_out, K_in");
  if (K_in % 128 != 0 || N_out % (paired ? 32 : 16) != 0)
    return fail(MOE_UNSUPPORTED_SHAPE, "repack needs K_in %% 128 == 0 and N_out %% %d == 0", paired ? 32 : 16);
  if (!qweight || !out || qweight == out) return fail(MOE_INVALID_ARGUMENT, "null or aliased pointer argument");
  if ((((uintptr_t)qweight | (uintptr_t)out) % 16) != 0)
    return fail(MOE_INVALID_ARGUMENT, "qweight and out must be 16-byte aligned");
  const int err = launch_repack(qweight, E, N_out, K_in, paired ? 1 : 0, out, (hipStream_t)stream);
  if (err != 0) return hip_fail(err, "repack launch");
  return MOE_OK;
}

int moe_import_awq(const int32_t* awq_qweight, const int32_t* awq_qzeros, const void* awq_scales, int E, int K_in,
                   int N_out, int group_size, int32_t* qweight, void* scales, uint8_t* zeros, void* stream) {
  if (E < 1 || K_in < 1 || N_out < 1 || group_size < 1)
    return fail(MOE_INVALID_ARGUMENT, "need positive E, K_in, N_out, group_size");
  if (E > 65535) return fail(MOE_UNSUPPORTED_SHAPE, "import handles at most 65535 experts per call");
  if (K_in % 8 != 0 || N_out % 8 != 0 || K_in % group_size != 0)
    return fail(MOE_UNSUPPORTED_SHAPE, "import needs K_in %% 8 == 0, N_out %% 8 == 0, K_in %% group_size == 0");
  if (!awq_qweight || !awq_qzeros || !awq_scales || !qweight || !scales || !zeros)
    return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  if ((const void*)awq_qweight == (const void*)qweight || awq_scales == (const void*)scales)
    return fail(MOE_INVALID_ARGUMENT, "the import does not work in place");
  if (((uintptr_t)awq_qweight | (uintptr_t)awq_qzeros | (uintptr_t)qweight) % 4 != 0 ||
      ((uintptr_t)awq_scales | (uintptr_t)scales) % 2 != 0)
    return fail(MOE_INVALID_ARGUMENT, "word tensors must be 4-byte, scale tensors 2-byte aligned");
  const int err = launch_awq_import(awq_qweight, awq_qzeros, awq_scales, E, K_in, N_out, group_size, qweight, scales,
                                    zeros, (hipStream_t)stream);
  if (err != 0) return hip_fail(err, "AWQ import launch");
  return MOE_OK;
}

size_t moe_w4a16_routed_layer_workspace_bytes(int T, int K, int N, int E, int topk, moe_dtype dt) {
  const size_t layer = moe_w4a16_layer_workspace_bytes(T, K, N, E, topk, dt);
  if (layer == 0 && T != 0) return 0;
  if (T < 0 || topk < 1) return 0;
  // routing tables in front of the layer's own workspace: ids int32 [S], weights float32 [S]
  return 2 * round_up((size_t)T * topk * 4, 256) + layer;
}

int moe_w4a16_routed_layer(const void* X, const float* logits, const float* bias,
                           const int32_t* qw1, const void* s1, const uint8_t* z1,
                           const int32_t* qw2, const void* s2, const uint8_t* z2,
                           void* out, int T, int K, int N, int E, int topk, int group_size, moe_dtype dt,
                           void* workspace, size_t workspace_bytes, void* stream) {
  if (T < 0 || topk < 1 || E < 1) return fail(MOE_INVALID_ARGUMENT, "need T >= 0, topk >= 1, E >= 1");
  if (T == 0) return MOE_OK;
  if (!workspace) return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  if (((uintptr_t)workspace % 256) != 0) return fail(MOE_INVALID_ARGUMENT, "workspace must be 256-byte aligned");
  const size_t table = round_up((size_t)T * topk * 4, 256);
  if (workspace_bytes < 2 * table)
    return fail(MOE_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", workspace_bytes,
                moe_w4a16_routed_layer_workspace_bytes(T, K, N, E, topk, dt));
  if (E > 1024) return fail(MOE_UNSUPPORTED_SHAPE, "E = %d exceeds 1024", E);
  if (topk > E || topk > 64) return fail(MOE_UNSUPPORTED_SHAPE, "topk = %d exceeds min(E, 64)", topk);
  if (!logits) return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  unsigned char* base = (unsigned char*)workspace;
  RouteArgs r;
  r.logits = logits; r.bias = bias;
  r.ids = (int32_t*)base;
  r.weights = (float*)(base + table);
  return layer_impl(X, r.ids, r.weights, qw1, s1, z1, qw2, s2, z2, out, T, K, N, E, topk, group_size, dt,
                    base + 2 * table, workspace_bytes - 2 * table, stream, 0, &r);
}

int moe_route_align(const float* logits, const float* bias, int T, int E, int topk, int block_m,
                    int32_t* topk_ids, float* topk_weights, int32_t* expert_counts, int32_t* expert_offsets,
                    int32_t* sorted_slot_ids, int32_t* block_expert_ids, int32_t* num_padded, void* stream) {
  if (T < 0 || E < 1 || topk < 1) return fail(MOE_INVALID_ARGUMENT, "need T >= 0, E >= 1, topk >= 1");
  if (!valid_block_m(block_m)) return fail(MOE_INVALID_ARGUMENT, "block_m must be 16, 32, 64, 128 or 256");
  if (E > 1024) return fail(MOE_UNSUPPORTED_SHAPE, "E = %d exceeds 1024", E);
  if (topk > E || topk > 64) return fail(MOE_UNSUPPORTED_SHAPE, "topk = %d exceeds min(E, 64)", topk);
  const long long S = (long long)T * topk;
  if (S > 0x7fffffffLL / 2) return fail(MOE_UNSUPPORTED_SHAPE, "T*topk too large");
  if (!expert_counts || !expert_offsets || !num_padded ||
      (S > 0 && (!logits || !topk_ids || !topk_weights || !sorted_slot_ids || !block_expert_ids)))
    return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  RouteArgs r;
  r.logits = logits; r.bias = bias; r.ids = topk_ids; r.weights = topk_weights;
  return route_and_align(r, T, E, topk, block_m, expert_counts, expert_offsets, sorted_slot_ids, block_expert_ids,
                         num_padded, nullptr, (hipStream_t)stream);
}

int moe_set_stage_events(void* const* events, int n) {
  if (n == 0 || events == nullptr) { g_nevents = 0; return MOE_OK; }
  if (n != 5 && n != 7) return fail(MOE_INVALID_ARGUMENT, "expected 5 events (16-bit layer) or 7 (FP8 layer)");
  for (int i = 0; i < n; ++i) g_events[i] = events[i];
  g_nevents = n;
  return MOE_OK;
}

int moe_set_scale_path(int mode) {
  if (mode < 0 || mode > 2) return fail(MOE_INVALID_ARGUMENT, "scale path mode must be 0, 1 or 2");
  g_scale_path = mode;
  return MOE_OK;
}

int moe_set_tiles_per_workgroup(int n) {
  if (n < 0 || n > 64) return fail(MOE_INVALID_ARGUMENT, "tiles per workgroup must be in 0..64");
  g_force_tpw = n;
  return MOE_OK;
}

int moe_set_reduction_splits(int n) {
  if (n < 0 || n > 64) return fail(MOE_INVALID_ARGUMENT, "reduction splits must be in 0..64");
  g_force_ksplit = n;
  return MOE_OK;
}

int moe_set_block_m_override(int block_m) {
  if (block_m != 0 && !valid_block_m(block_m))
    return fail(MOE_INVALID_ARGUMENT, "block_m override must be 0, 16, 32, 64, 128 or 256");
  g_force_block_m = block_m;
  return MOE_OK;
}

int moe_last_gemm_plan(int* plan9) {
  if (!plan9) return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  for (int i = 0; i < 9; ++i) plan9[i] = g_last_plan[i];
  return MOE_OK;
}

int moe_set_wide_tiles(int mode) {
  if (mode < 0 || mode > 1) return fail(MOE_INVALID_ARGUMENT, "wide tile mode must be 0 (when usable) or 1 (never)");
  g_wide_mode = mode;
  return MOE_OK;
}

int moe_set_tile_override(int mt, int nt) {
  if (mt < 0 || nt < 0) return fail(MOE_INVALID_ARGUMENT, "negative tile override");
  g_force_mt = mt; g_force_nt = nt;
  return MOE_OK;
}

// ---- blockwise-scaled FP8 GEMM (include/fp8_blockwise_gemm.h) -------------------------------
size_t fp8_blockwise_gemm_workspace_bytes(int M, int N, int K) {
  if (M < 1 || N < 64 || K < 128 || K % 128 != 0 || N % 64 != 0) return 0;
  Fp8Plan pl;
  if (!fp8_plan(M, N, K, pl)) return 0;
  return pl.splits > 1 ? round_up((size_t)pl.splits * (size_t)M * (size_t)N * sizeof(float), 256) : 0;
}

int fp8_blockwise_gemm(const uint8_t* A, const float* a_scale, const uint8_t* B, const float* b_scale, void* C,
                       int M, int N, int K, int out_dtype, void* workspace, size_t workspace_bytes, void* stream) {
  if (M < 0 || N < 1 || K < 1) return fail(MOE_INVALID_ARGUMENT, "need M >= 0, N >= 1, K >= 1");
  if (out_dtype < 0 || out_dtype > 2)
    return fail(MOE_INVALID_ARGUMENT, "out_dtype must be 0 (fp16), 1 (bf16) or 2 (float32)");
  if (K % 128 != 0 || N % 64 != 0)
    return fail(MOE_UNSUPPORTED_SHAPE, "the FP8 GEMM needs K %% 128 == 0 and N %% 64 == 0 (got N=%d K=%d)", N, K);
  if (M == 0) return MOE_OK;
  if (!A || !a_scale || !B || !b_scale || !C) return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  if (((uintptr_t)A | (uintptr_t)B | (uintptr_t)C) % 16 != 0 || ((uintptr_t)a_scale | (uintptr_t)b_scale) % 4 != 0)
    return fail(MOE_INVALID_ARGUMENT, "A, B, C must be 16-byte aligned, the scales 4-byte aligned");
  if (C == (const void*)A || C == (const void*)B) return fail(MOE_INVALID_ARGUMENT, "C must not alias an input");
  const size_t plane = (size_t)M * (size_t)N * sizeof(float);
  Fp8Plan pl;
  if (!fp8_plan(M, N, K, pl)) return fail(MOE_UNSUPPORTED_SHAPE, "the forced FP8 plan does not fit M=%d N=%d K=%d", M, N, K);
  if ((unsigned long long)M * (unsigned long long)K >= (1ull << 32) ||
      (unsigned long long)N * (unsigned long long)K >= (1ull << 32))
    return fail(MOE_UNSUPPORTED_SHAPE, "the FP8 GEMM addresses A and B with 32-bit offsets: M * K and N * K must be below 2^32");
  if (!g_fp8_mt && !g_fp8_nt && !g_fp8_splits) {
    const int KB = K / 128, least = fp8_splits_needed(M, N, K);
    const bool misaligned = (uintptr_t)workspace % 256 != 0;
    if (least > 1 && misaligned) return fail(MOE_INVALID_ARGUMENT, "workspace must be 256-byte aligned");
    const int fit = workspace && !misaligned ? (int)std::min<size_t>(workspace_bytes / plane, 16) : 0;
    if (fit < pl.splits && fit >= (least > 1 ? least : 0)) {
      pl.kb_per_split = fit > 1 ? (KB + fit - 1) / fit : KB;
      pl.splits = (KB + pl.kb_per_split - 1) / pl.kb_per_split;
    }
  }
  const long long m_blocks = (M + pl.bm - 1) / pl.bm;
  const long long grid = m_blocks * (N / pl.bn) * pl.splits;
  if (grid > 0x7fffffffLL) return fail(MOE_UNSUPPORTED_SHAPE, "too many workgroups");
  fp8::GemmParams p = {};
  p.A = A; p.a_scale = a_scale; p.B = B; p.b_scale = b_scale;
  p.M = M; p.N = N; p.K = K;
  p.k_splits = pl.splits; p.kb_per_split = pl.kb_per_split; p.out_bf16 = out_dtype;
  // row blocks per tile group: 4 for the 256 x 256 tile (8192^3 459 against 470 us at 8), 4 ... 16 alike elsewhere
  p.group_m = g_fp8_group_m ? g_fp8_group_m : pl.bm == 256 ? 4 : 8;
  if (pl.splits > 1) {
    const size_t need = round_up((size_t)pl.splits * plane, 256);
    if (!workspace || workspace_bytes < need)
      return fail(MOE_WORKSPACE_TOO_SMALL, "FP8 GEMM workspace: need %zu bytes, got %zu", need, workspace_bytes);
    if ((uintptr_t)workspace % 256 != 0) return fail(MOE_INVALID_ARGUMENT, "workspace must be 256-byte aligned");
    p.C = workspace;
  } else {
    p.C = C;
  }
  int kbn, kgroups;
  if (!g_fp8_mt && !g_fp8_nt && !g_fp8_splits && fp8_groups_pay(M, N, K, pl, kbn, kgroups)) {
    p.C = C; p.k_splits = 1; p.kb_per_split = K / 128;
    const int err = fp8::launch_fp8_kgroups(p, pl.bm, kbn, kgroups, (hipStream_t)stream);
    if (err != 0) return hip_fail(err, "FP8 GEMM launch");
    return MOE_OK;
  }
  int err = fp8::launch_fp8_gemm(p, pl.bm, pl.bn, (hipStream_t)stream);
  if (err == -1) return fail(MOE_UNSUPPORTED_SHAPE, "no FP8 GEMM variant for tile %d x %d", pl.bm, pl.bn);
  if (err != 0) return hip_fail(err, "FP8 GEMM launch");
  if (pl.splits > 1) {
    err = fp8::launch_fp8_split_reduce((const float*)workspace, pl.splits, (long long)M * N, C, out_dtype,
                                       (hipStream_t)stream);
    if (err != 0) return hip_fail(err, "FP8 split reduction launch");
  }
  return MOE_OK;
}

int fp8_moe_grouped_gemm(const uint8_t* A, const float* a_scale, int row_div, const uint8_t* B,
                         const float* b_scale, const int32_t* sorted_slot_ids, const int32_t* block_expert_ids,
                         const int32_t* num_padded, int num_slots, int E, int N, int K, int block_m, int out_dtype,
                         void* C, void* stream) {
  if (num_slots < 0 || E < 1 || E > 1024 || N < 1 || K < 1 || row_div < 1)
    return fail(MOE_INVALID_ARGUMENT, "need num_slots >= 0, 1 <= E <= 1024, N >= 1, K >= 1, row_div >= 1");
  if (out_dtype < 0 || out_dtype > 2)
    return fail(MOE_INVALID_ARGUMENT, "out_dtype must be 0 (fp16), 1 (bf16) or 2 (float32)");
  if (!valid_block_m(block_m)) return fail(MOE_INVALID_ARGUMENT, "block_m must be 16, 32, 64, 128 or 256");
  if (K % 128 != 0 || N % 64 != 0 || (block_m == 256 && N % 128 != 0))
    return fail(MOE_UNSUPPORTED_SHAPE,
                "the grouped FP8 GEMM needs K %% 128 == 0 and N %% 64 == 0 (N %% 128 == 0 at block_m 256); got N=%d K=%d",
                N, K);
  if (num_slots == 0) return MOE_OK;
  if (!A || !a_scale || !B || !b_scale || !sorted_slot_ids || !block_expert_ids || !num_padded || !C)
    return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  if (((uintptr_t)A | (uintptr_t)B | (uintptr_t)C) % 16 != 0 || ((uintptr_t)a_scale | (uintptr_t)b_scale) % 4 != 0)
    return fail(MOE_INVALID_ARGUMENT, "A, B, C must be 16-byte aligned, the scales 4-byte aligned");
  if (C == (const void*)A || C == (const void*)B) return fail(MOE_INVALID_ARGUMENT, "C must not alias an input");
  const unsigned long long rows_a = ((unsigned long long)num_slots + row_div - 1) / row_div;
  if (rows_a * (unsigned long long)K >= (1ull << 32) || (unsigned long long)N * (unsigned long long)K >= (1ull << 32))
    return fail(MOE_UNSUPPORTED_SHAPE, "32-bit operand offsets: rows(A) * K and N * K must be below 2^32");
  const size_t cap = align_capacity(num_slots, E, block_m);
  const int bn = block_m == 256 && N % 256 == 0 ? 256 : N % 128 == 0 ? 128 : 64;
  const long long grid = (long long)(cap / block_m) * (N / bn);
  if (cap > 0x7fffffffULL || grid > 0x7fffffffLL) return fail(MOE_UNSUPPORTED_SHAPE, "too many workgroups");
  fp8::GemmParams p = {};
  p.A = A; p.a_scale = a_scale; p.B = B; p.b_scale = b_scale; p.C = C;
  p.M = (int)cap; p.N = N; p.K = K;
  p.k_splits = 1; p.kb_per_split = K / 128; p.out_bf16 = out_dtype;
  p.group_m = g_fp8_group_m ? g_fp8_group_m : 8;
  p.sorted_slot_ids = sorted_slot_ids; p.block_expert_ids = block_expert_ids; p.num_padded = num_padded;
  p.num_slots = num_slots; p.row_div = row_div;
  p.b_expert_stride = (size_t)N * (size_t)K;
  p.bs_expert_stride = (size_t)((N + 127) / 128) * (size_t)(K / 128);
  const int err = fp8::launch_fp8_gemm(p, block_m, bn, (hipStream_t)stream);
  if (err == -1) return fail(MOE_UNSUPPORTED_SHAPE, "no FP8 GEMM variant for tile %d x %d", block_m, bn);
  if (err != 0) return hip_fail(err, "grouped FP8 GEMM launch");
  return MOE_OK;
}

// ---- FP8 mixture-of-experts layer ------------------------------------------------------------
int fp8_quantize_rows(const void* X, int rows, int K, int dt, uint8_t* codes, float* scales, void* stream) {
  if (rows < 0 || K < 1) return fail(MOE_INVALID_ARGUMENT, "need rows >= 0 and K >= 1");
  if (dt != MOE_F16 && dt != MOE_BF16) return fail(MOE_INVALID_ARGUMENT, "dt must be MOE_F16 or MOE_BF16");
  if (K % 128 != 0) return fail(MOE_UNSUPPORTED_SHAPE, "the activation quantiser needs K %% 128 == 0 (got %d)", K);
  if (rows == 0) return MOE_OK;
  if (!X || !codes || !scales) return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  if ((uintptr_t)X % 16 != 0 || (uintptr_t)codes % 8 != 0 || (uintptr_t)scales % 4 != 0)
    return fail(MOE_INVALID_ARGUMENT, "X must be 16-byte, codes 8-byte, scales 4-byte aligned");
  const int err = fp8::launch_fp8_quantize(X, rows, K, (int)dt, 0, codes, scales, (hipStream_t)stream);
  if (err != 0) return hip_fail(err, "activation quantiser launch");
  return MOE_OK;
}

int fp8_silu_mul_quantize(const void* H, int S, int N, int dt, uint8_t* codes, float* scales, void* stream) {
  if (S < 0 || N < 1) return fail(MOE_INVALID_ARGUMENT, "need S >= 0 and N >= 1");
  if (dt != MOE_F16 && dt != MOE_BF16) return fail(MOE_INVALID_ARGUMENT, "dt must be MOE_F16 or MOE_BF16");
  if (N % 128 != 0) return fail(MOE_UNSUPPORTED_SHAPE, "the activation quantiser needs N %% 128 == 0 (got %d)", N);
  if (S == 0) return MOE_OK;
  if (!H || !codes || !scales) return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  if ((uintptr_t)H % 16 != 0 || (uintptr_t)codes % 8 != 0 || (uintptr_t)scales % 4 != 0)
    return fail(MOE_INVALID_ARGUMENT, "H must be 16-byte, codes 8-byte, scales 4-byte aligned");
  const int err = fp8::launch_fp8_quantize(H, S, N, (int)dt, 1, codes, scales, (hipStream_t)stream);
  if (err != 0) return hip_fail(err, "SiLU-and-multiply quantiser launch");
  return MOE_OK;
}

static thread_local int g_fp8_layer_block_m = 0;

static int fp8_pick_block_m(long long S, int E, int K, int N) {
  if (g_fp8_layer_block_m > 0) return g_fp8_layer_block_m;
  const long long avg = S / (E > 0 ? E : 1);
  // 256-slot blocks (the two-group tile of fp8_moe_grouped_gemm, which skips a block's empty 32-row
  // parts): every weight is fetched once per 256 rows.  From 64 rows per expert on if the smaller
  // product's tiles fill their rounds over the CUs to 70 % (64 experts, K 2048, N 1408: 1000 tokens 197
  // against 218 us, 3000 tokens 369 against 448; 8 experts, 144 tiles: 142 against 130), from 16 on
  // in launches of many rounds (256 experts, K 7168, N 2048: 512 tokens 2.06 against 2.09 ms, 1024
  // 2.25 against 2.49, 4096 3.07 against 3.95; at 8 rows per expert 32-slot blocks win by 1 %).
  // Skewed routing packs the rows into fewer blocks; the second case also asks for 100 tiles if every block were
  // full (former time over this tile's below / at 100 ... 160 / from 260 on, geometric mean: even routing 1.04 / 1.15 /
  // 1.15, power law 0.85 / 0.96 / 1.09).
  if (K % 256 == 0 && N % 128 == 0) {
    const long long per_block = (K < 2 * N ? K : 2 * N) / 256, tiles = (S / 256 + (S < E ? S : E) / 2) * per_block;
    if (tiles >= 1024 ? avg >= 16 : avg >= 64 && tiles * 10 >= 7 * 256 * ((tiles + 255) / 256) && S / 256 * per_block >= 100) return 256;
  }
  if (avg <= 32) return 32;      // measured: 32-token tiles stream the weights fastest at a few rows per expert
  if (avg >= 96) return 128;     // about one row block per expert: its weights are fetched once (measured +2 %)
  return 64;
}

struct Fp8Workspace { size_t counts, offsets, num_padded, sorted, blocks, xq, sx, H, aq, sa, Y, total; };
static Fp8Workspace fp8_carve(long long T, int K, int N, int E, int topk) {
  const long long S = T * topk;
  Fp8Workspace w;
  size_t o = 0;
  w.counts = o;      o += round_up((size_t)E * 4, 256);
  w.offsets = o;     o += round_up((size_t)(E + 1) * 4, 256);
  w.num_padded = o;  o += 256;
  w.sorted = o;      o += round_up(align_capacity(S, E, 256) * 4, 256);
  w.blocks = o;      o += round_up((align_capacity(S, E, 16) / 16 + 1) * 4, 256);
  w.xq = o;          o += round_up((size_t)T * K, 256);
  w.sx = o;          o += round_up((size_t)T * (K / 128) * 4, 256);
  w.H = o;           o += round_up((size_t)S * 2 * N * 2, 256);
  w.aq = o;          o += round_up((size_t)S * N, 256);
  w.sa = o;          o += round_up((size_t)S * (N / 128) * 4, 256);
  w.Y = o;           o += round_up((size_t)S * K * 4, 256);
  w.total = o;
  return w;
}

size_t fp8_moe_layer_workspace_bytes(int T, int K, int N, int E, int topk) {
  if (T < 0 || K < 128 || N < 128 || E < 1 || topk < 1 || K % 128 != 0 || N % 128 != 0) return 0;
  return fp8_carve(T, K, N, E, topk).total;
}

int fp8_set_layer_block_m(int block_m) {
  if (block_m != 0 && !valid_block_m(block_m))
    return fail(MOE_INVALID_ARGUMENT, "block_m override must be 0, 16, 32, 64, 128 or 256");
  g_fp8_layer_block_m = block_m;
  return MOE_OK;
}

int fp8_moe_layer(const void* X, const int32_t* topk_ids, const float* topk_weights,
                  const uint8_t* w1, const float* w1_scale, const uint8_t* w2, const float* w2_scale,
                  void* out, int T, int K, int N, int E, int topk, int dt,
                  void* workspace, size_t workspace_bytes, void* stream_v) {
  hipStream_t stream = (hipStream_t)stream_v;
  if (T < 0 || K < 1 || N < 1 || E < 1 || topk < 1)
    return fail(MOE_INVALID_ARGUMENT, "need T >= 0 and positive K, N, E, topk");
  if (dt != MOE_F16 && dt != MOE_BF16) return fail(MOE_INVALID_ARGUMENT, "dt must be MOE_F16 or MOE_BF16");
  if (E > 1024) return fail(MOE_UNSUPPORTED_SHAPE, "E = %d exceeds 1024", E);
  if (K % 128 != 0 || N % 128 != 0)
    return fail(MOE_UNSUPPORTED_SHAPE, "the FP8 layer needs K %% 128 == 0 and N %% 128 == 0 (got K=%d N=%d)", K, N);
  if (T == 0) return MOE_OK;
  if (!X || !topk_ids || !topk_weights || !w1 || !w1_scale || !w2 || !w2_scale || !out || !workspace)
    return fail(MOE_INVALID_ARGUMENT, "null pointer argument");
  if (((uintptr_t)workspace % 256) != 0) return fail(MOE_INVALID_ARGUMENT, "workspace must be 256-byte aligned");
  if (((uintptr_t)X | (uintptr_t)out | (uintptr_t)w1 | (uintptr_t)w2) % 16 != 0)
    return fail(MOE_INVALID_ARGUMENT, "X, out and the weight tensors must be 16-byte aligned");
  const long long S = (long long)T * topk;
  if (S > 0x7fffffffLL / 2) return fail(MOE_UNSUPPORTED_SHAPE, "T*topk too large");
  const Fp8Workspace w = fp8_carve(T, K, N, E, topk);
  if (workspace_bytes < w.total)
    return fail(MOE_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", workspace_bytes, layer_workspace(T, K, N, E, topk, (int)dt));
  unsigned char* base = (unsigned char*)workspace;
  int32_t* counts = (int32_t*)(base + w.counts);
  int32_t* offsets = (int32_t*)(base + w.offsets);
  int32_t* num_padded = (int32_t*)(base + w.num_padded);
  int32_t* sorted = (int32_t*)(base + w.sorted);
  int32_t* blocks = (int32_t*)(base + w.blocks);
  uint8_t* xq = base + w.xq;
  float* sx = (float*)(base + w.sx);
  void* H = base + w.H;
  uint8_t* aq = base + w.aq;
  float* sa = (float*)(base + w.sa);
  float* Y = (float*)(base + w.Y);
  const int block_m = fp8_pick_block_m(S, E, K, N);
  const bool ev = g_nevents == 7;
  auto mark = [&](int i) { if (ev) (void)hipEventRecord((hipEvent_t)g_events[i], stream); };

  mark(0);
  const bool beside = runs_beside(T, K);
  const RowsJob job = beside ? quantize_job(X, T, K, (int)dt, xq, sx) : RowsJob{};
  int err = launch_align(topk_ids, (int)S, E, block_m, (int)align_capacity(S, E, block_m), counts, offsets, sorted,
                         blocks, num_padded, &job, stream);
  if (err != 0) return hip_fail(err, "align and quantiser launch");
  mark(1);
  if (!beside) {
    err = fp8::launch_fp8_quantize(X, T, K, (int)dt, 0, xq, sx, stream);
    if (err != 0) return hip_fail(err, "activation quantiser launch");
  }
  mark(2);
  int st = fp8_moe_grouped_gemm(xq, sx, topk, w1, w1_scale, sorted, blocks, num_padded, (int)S, E, 2 * N, K, block_m,
                                (int)dt, H, stream);
  if (st != MOE_OK) return st;
  mark(3);
  // rows of slots that were not bucketed hold stale bytes: they are quantised like any other row
  // and never read again (the second product only gathers bucketed slots)
  err = fp8::launch_fp8_quantize(H, S, N, (int)dt, 1, aq, sa, stream);
  if (err != 0) return hip_fail(err, "SiLU-and-multiply quantiser launch");
  mark(4);
  st = fp8_moe_grouped_gemm(aq, sa, 1, w2, w2_scale, sorted, blocks, num_padded, (int)S, E, K, N, block_m, 2, Y, stream);
  if (st != MOE_OK) return st;
  mark(5);
  err = launch_combine(Y, 1, 1, topk_weights, topk_ids, E, out, T, topk, K, (int)dt, stream);
  if (err != 0) return hip_fail(err, "combine launch");
  mark(6);
  return MOE_OK;
}

int fp8_set_plan_override(int mt, int nt, int k_splits, int group_m) {
  if (mt < 0 || nt < 0 || k_splits < 0 || group_m < 0) return fail(MOE_INVALID_ARGUMENT, "negative plan override");
  g_fp8_mt = mt; g_fp8_nt = nt; g_fp8_splits = k_splits; g_fp8_group_m = group_m;
  return MOE_OK;
}

int fp8_probe_mfma(void* sink, int iters, void* stream) {
  if (!sink || iters < 1) return fail(MOE_INVALID_ARGUMENT, "probe needs a sink and iters >= 1");
  const int err = fp8::launch_fp8_mfma_loop((float*)sink, 512, iters, (hipStream_t)stream);
  if (err != 0) return hip_fail(err, "FP8 MFMA probe launch");
  return MOE_OK;
}

}  // extern "C"
