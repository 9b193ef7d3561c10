// Device side: the pack/unpack kernels and their launcher.
#pragma once

#include <hip/hip_runtime_api.h>

#include "plan.hpp"
#include "signal.hpp"

namespace tp {

// Enqueues one planned launch on `stream`.  Returns hipSuccess or the launch error.
hipError_t enqueue(const Launch& launch, bool unpack, hipStream_t stream);

// Whether a launch that is a synchronous call's only one should signal its own end (signal.hpp).
bool signals_itself(const Launch& launch);
// Enqueues such a launch: its kernel signals when all it stores is in memory.
hipError_t enqueue_signalled(const Launch& launch, bool unpack, hipStream_t stream, const SignalParams& signal);

// Enqueues one batched launch (see plan.hpp: BatchParams).
hipError_t enqueue_batch(const BatchParams& batch, bool unpack, hipStream_t stream);

}  // namespace tp
