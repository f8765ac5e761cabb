// Training step of the learned min-sum decoder with a frame on one compute
// unit (train.hip).  Called by ldpc_nms_train_forward / _backward for the
// codes it covers; the message packages of decode.hip take the rest.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "internal.h"

namespace ldpc {

// Workspace of a step of `gamma` frames and T iterations, 0 when the code is
// not covered: full bases of 3 rows of weight 6, 9 or 18, or of 4 rows of
// weight 24 with p <= 768, two arrays of n floats in LDS.
size_t train_onchip_bytes(const ldpc_graph* g, int gamma, int T);

// Enqueue the forward and the backward pass (arguments as the entry points);
// false when a launch failed.
bool train_onchip_forward(const ldpc_graph* g, const float* llr, int gamma, int T, const float* w, float* loss,
                          void* ws, hipStream_t st);
bool train_onchip_backward(const ldpc_graph* g, int gamma, int T, const float* w, const float* dloss, float* grad,
                           void* ws, hipStream_t st);

}  // namespace ldpc
