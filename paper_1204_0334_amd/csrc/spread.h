// Block decoder with a frame on several compute units (spread.hip), for
// batches that would leave most of the chip idle.  Called by ldpc_decode and
// the plans before the one-unit decoder of onchip.hip, whose results it
// returns bit for bit, and in place of the message packages, whose results it
// returns bit for bit, for longer codes.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "internal.h"

namespace ldpc {

// Workspace of a batch of gamma frames on the current device, 0 when the rule
// does not choose this decoder (or the environment variable LDPC_BLOCK_PATH is
// "packages" or "onchip").
size_t spread_bytes(const ldpc_graph* g, int gamma);

// Whether outputs lie on inputs: members read channel LLRs while others, done
// already, write outputs, and a frame may be decoded a second time.
bool spread_in_place(const ldpc_graph* g, int gamma, const float* llr, const float* post, const uint8_t* bits);

// Enqueues the whole decode (arguments as ldpc_decode, nms_w as
// ldpc_nms_decode's weights or NULL) in the workspace of ws_bytes.  Returns 1
// once launched, 0 (having enqueued nothing) when the rule does not choose
// it or outputs lie on inputs, -1 when a launch failed.
int spread_decode(const ldpc_graph* g, const float* llr, int gamma, int max_iters, int early, float* post,
                  uint8_t* bits, int32_t* iters, uint8_t* converged, void* ws, size_t ws_bytes, hipStream_t st,
                  const float* nms_w);

}  // namespace ldpc
