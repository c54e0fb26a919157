// Internal interface of the one-lane-per-operation bulk kernels
// (lpht_lane.hip).  Not part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lpht_internal.h"

namespace lpht {

// One bulk call (a.kinds must be null or valid for a.n) in workgroups of
// at most `threads` (a multiple of 64); `dense`: the table may be more than
// half full.
hipError_t launch_lane(OpKind op, const BulkArgs &a, uint32_t threads, bool dense, hipStream_t s);

// Descriptors of a multi-table launch that fit its kernel arguments.
constexpr uint32_t kLaneDescs = 28;

// As launch_lane_multi, from up to kLaneDescs descriptors in host memory: they
// travel as kernel arguments, so nothing has to be uploaded before the launch.
hipError_t launch_lane_few(OpKind op, uint32_t up, uint32_t layout, const BulkArgs *descs, uint32_t ndesc,
                           hipStream_t s);

// As launch_bulk_multi, with group width 1.
hipError_t launch_lane_multi(OpKind op, uint32_t up, uint32_t layout, const BulkArgs *descs,
                             const uint64_t *round_start, uint32_t ndesc, uint64_t total_rounds, hipStream_t s);

}  // namespace lpht
