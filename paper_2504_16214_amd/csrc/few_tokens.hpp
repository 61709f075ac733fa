// Launch interface of the few-token layer kernels (few_tokens.hip), used by the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace moe {

constexpr size_t kFewLds = 136 * 1024;     // LDS either kernel may take

// K and N whole groups of 128, the vectors within the LDS budget.
bool few_tokens_fit(int topk, int K, int N);
// Parts of the reduction that a slot's down product is cut into: about eight (slot, part) pairs for the eight waves.
int few_down_parts(int topk, int N);
// Routing inside the gate/up launch: up to kFewRouteE experts and 16 experts a token; fills ids and weights [T, topk].
// (Sixteen keys a lane instead of four, for 65 to 256 experts, would take 1 to 13 % off such calls: 1 token of 7168 x 2048, 256 experts,
// 48.9 -> 47.9 us, 128 experts 47.9 -> 46.1, 8 tokens of 256 x 512, 72 experts, 10.6 -> 9.4.  Not built.)
constexpr int kFewRouteE = 64, kFewRouteTopk = 16;
struct FewRoute {
  const float* logits;
  const float* bias;         // may be null
  int32_t* ids;
  float* weights;
};
// What act and its chunks' words take.
size_t few_act_bytes(long long slots, int N);
size_t few_unit_bytes(long long slots, int N);
// act as vectors of the down kernel (few_act_bytes, 16-byte aligned) with their chunks' words in units (few_unit_bytes, 16-byte aligned),
// then out [T, K]; ids outside [0, E) contribute zero.  route (may be null): the ids come from there.  Group 128; X, act, out
// and the packed words 16-byte aligned; pre: the words are in operand order.
int launch_few_gate_up(const void* X, const FewRoute* route, const int32_t* ids, const int32_t* qw, const void* s, const uint8_t* z, void* act,
                       uint32_t* units, int T, int topk, int E, int K, int N, int dt, int pre, hipStream_t stream);
int launch_few_down(const void* act, const uint32_t* units, const int32_t* ids, const float* w, const int32_t* qw, const void* s, const uint8_t* z,
                    void* out, int T, int topk, int E, int K, int N, int dt, int pre, hipStream_t stream);

}  // namespace moe
