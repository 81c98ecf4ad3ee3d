// sw2d_handle.h - host-side access to a single-grid handle for the other C-ABI sources.
#pragma once

#include <hip/hip_runtime.h>

#include "sw2d.h"
#include "sw2d_internal.h"

namespace sw2d {
namespace detail {
// The stream and grid size of a single-grid handle (false for a null handle).
bool handle_info(sw2d_t h, hipStream_t* stream, int* nx, int* ny);

// Steps whose folds wait in a handle's partials. A caller that enqueues several runs of steps in one
// call shares one queue among them, and empties it before it returns.
struct FoldQueue {
    FoldRuns runs{};
    int pending = 0;    // steps
    int64_t used = 0;   // slots
};
int step_queued(sw2d_t h, int32_t nsteps, FoldQueue& q);
// Whether a single step of the handle can add a correction as it stores its state (plain model over
// tiles), and such a step.
bool corrects_in_step(sw2d_t h);
int step_corrected(sw2d_t h, const StepCorrection& fix, FoldQueue& q);
int flush_folds(sw2d_t h, FoldQueue& q);
}  // namespace detail
}  // namespace sw2d
