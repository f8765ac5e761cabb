// Pipelined decoder with a stream on one compute unit (sweep.hip).  Called by
// ldpc_decode_pipeline for the codes and sizes it covers; the ring of
// decode.hip takes the rest.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "internal.h"

namespace ldpc {

// The messages and sums between sweeps of a batch of streams stay within
// kSweepMostBytes; a batch of fewer streams than compute units (of more) would
// leave some idle, and longer chains go to the ring, whose memory does not grow
// with them.
constexpr size_t kSweepMostBytes = (size_t)4 << 30;

struct SweepPlan {
    int sweeps, batch;                   // launches per batch, streams per batch
    size_t lds_limit;                    // LDS a workgroup may take
    size_t alpha_floats, sum_floats;     // per stream, between sweeps
    size_t bytes;                        // workspace of a batch
};

// Whether the sweeps cover g at this batch and processor count (full bases of
// one circulant row per layer: T = 3 with 2 columns per position, T = 4 with 6).
bool sweep_plan(const ldpc_graph* g, int gamma, int iters, SweepPlan& plan);

// Whether they cover g at some batch.  The ring forms messages and sums of such a
// code as the sweeps do, so that results do not depend on which of them runs.
bool sweep_takes(const ldpc_graph* g);

// Enqueues the decode; false when a launch failed.
bool sweep_decode(const ldpc_graph* g, const SweepPlan& plan, const float* llr, int gamma, int iters, float* post,
                  uint8_t* bits, void* workspace, hipStream_t st);

}  // namespace ldpc
