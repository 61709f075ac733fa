// Launch interface of the few-token layer kernels (few_tokens.hip), used by the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace moe {

constexpr size_t kFewLds = 64 * 1024;      // LDS either kernel may take (no attribute needed up to here)

// K and N whole groups of 128, the vectors within the LDS budget.
bool few_tokens_fit(int topk, int K, int N);
// Parts of the reduction that a slot's down product is cut into: about eight (slot, part) pairs for the eight waves.
int few_down_parts(int topk, int N);
// act [T * topk, N] (runs of eight reordered), then out [T, K]; ids outside [0, E) contribute zero.  Group
// 128; X, act, out and the packed words 16-byte aligned; pre: the words are in operand order.
int launch_few_gate_up(const void* X, const int32_t* ids, const int32_t* qw, const void* s, const uint8_t* z, void* act, int T,
                       int topk, int E, int K, int N, int dt, int pre, hipStream_t stream);
int launch_few_down(const void* act, const int32_t* ids, const float* w, const int32_t* qw, const void* s, const uint8_t* z,
                    void* out, int T, int topk, int E, int K, int N, int dt, int pre, hipStream_t stream);

}  // namespace moe
