// Sliding-window decoder with messages in registers (window.hip).  Called by
// ldpc_decode_window for the codes it covers; window_lds_kernel of decode.hip,
// whose ring of messages needs more LDS, or the launches take the others.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "internal.h"

namespace ldpc {

// Enqueues the whole decode (arguments as ldpc_decode_window).  Returns 1 once
// launched, 0 (nothing enqueued) when the code or window is not covered, -1
// when the launch failed.
int window_decode(const ldpc_graph* g, const float* llr, int gamma, int W, int K, float* post, uint8_t* bits,
                  hipStream_t st);

}  // namespace ldpc
