// Sticky error bits that kernels set in a stage's error word, and the status
// that moe_stage_sync makes of them.
#pragma once

#include "moe_stage.h"

namespace moe {

constexpr int kErrBadId = 1;
constexpr int kErrBadLayer = 2;
constexpr int kErrIngestTimeout = 4;
constexpr int kErrBadCount = 8;       // pre-grouped counts negative or past the rows buffer
constexpr int kErrStalled = 16;       // a work item's inputs never became ready (ffn_sched.h)

// One status for all bits, which are cleared together.  A stalled pass comes
// first: it alone says that rows were computed from inputs that were not there,
// with nothing wrong in what the caller passed.
constexpr moe_status sticky_status(int err)
{
    return (err & kErrStalled)         ? MOE_EHIP
           : (err & kErrBadId)         ? MOE_EBADID
           : (err & kErrBadLayer)      ? MOE_EBADLAYER
           : (err & kErrBadCount)      ? MOE_EBADCOUNT
           : (err & kErrIngestTimeout) ? MOE_ETIMEOUT
                                       : MOE_OK;
}

}  // namespace moe
