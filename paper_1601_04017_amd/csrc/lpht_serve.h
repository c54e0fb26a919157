// Internal interface of the serving copy kernel (lpht_serve.hip).  Not part
// of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "lpht_internal.h"

namespace lpht {

// One contiguous copy between device staging and memory of the caller that
// the device can address (pinned host memory or device memory); no alignment
// is asked of either side.
struct ServeSeg {
  void *dst;
  const void *src;
  uint64_t bytes;
  uint32_t caller_is_src;  // which side is the caller's
  uint32_t first;          // set by the launcher: first work item of the segment
};

// A table's exact counts: out[0..2] = used, live, error bits (out may be
// pinned host memory).
struct ServeCount {
  const DevStatus *st;
  uint64_t *out;
};

// All copies of one wave of requests and the counts of its tables, in as few
// launches as their descriptors fit kernel arguments (no upload).
hipError_t launch_serve_copy(const std::vector<ServeSeg> &segs, const std::vector<ServeCount> &counts, hipStream_t s);

}  // namespace lpht
