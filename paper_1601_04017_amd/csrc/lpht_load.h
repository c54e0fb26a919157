// Internal interface of the region load (lpht_load.hip): large inserting
// calls on tables that are nearly empty.  Not part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lpht_internal.h"

namespace lpht {

// Whether the region load takes a call of n insertions (or insert-or-assigns)
// on a table of 2^log2c cells of which at most `used0` are not empty.
bool load_applies(uint64_t n, uint32_t log2c, uint32_t layout, uint64_t used0, bool with_flags);

// Its device scratch in bytes.
size_t load_scratch_bytes(uint64_t n, uint32_t log2c, uint32_t layout, bool with_flags);

// Enqueues OP_INSERT, or OP_UPSERT with a.up == 0, for a call that
// load_applies takes.  `fresh`: the table has no non-empty cell.
hipError_t launch_load(OpKind op, const BulkArgs &a, bool fresh, void *scratch, hipStream_t s);

}  // namespace lpht
