// Message-package decoder of a short code with a frame's packages in LDS
// (small.hip).  Called by ldpc_decode and the plans for codes that no other
// one-unit kernel takes; outputs equal the launch-per-phase form's bit for
// bit.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "internal.h"

namespace ldpc {

// Whether the rule chooses this decoder for a batch of gamma frames on the
// current device (and the environment variable LDPC_BLOCK_PATH is not
// "packages").
bool small_selected(const ldpc_graph* g, int gamma);

// Enqueues the whole decode (arguments as ldpc_decode).  Returns 1 once
// launched, 0 (having enqueued nothing) when not chosen, -1 when the launch
// failed.
int small_decode(const ldpc_graph* g, const float* llr, int gamma, int max_iters, int early, float* post,
                 uint8_t* bits, int32_t* iters, uint8_t* converged, hipStream_t st);

}  // namespace ldpc
