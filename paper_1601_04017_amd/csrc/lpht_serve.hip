// Copies of the serving waves: the keys and kinds of all requests of a wave
// into device staging in one launch, and their values, flags and the tables'
// counts back in another.
//
// What bounds it: the PCIe link (about 57 GB/s each way for long sequential
// runs) once the launches are few.  A wave of 16 requests used to queue 64
// copies and 16 count kernels of 4 us each behind one another on its stream;
// here a workgroup moves 16 KiB of some request, 16 bytes per lane and access,
// aligned on the caller's side, where a partial access would cost a link
// transaction, and unaligned on the staging side.  Segment descriptors travel
// in the kernel's arguments, so no upload precedes the launch.  Trace of 96
// requests over 16 tables (2.5 million operations, 64 clients, four streams),
// with the phases' descriptors in kernel arguments too: 9.0 -> 3.2 ms.

#include <hip/hip_runtime.h>

#include <algorithm>

#include "lpht_device.h"
#include "lpht_serve.h"

namespace lpht {

namespace {

constexpr uint32_t kThreads = 256;
constexpr uint32_t kVecs = 4;                            // 16-byte accesses in flight per lane
constexpr uint32_t kItem = kThreads * kVecs * 16;        // bytes a workgroup moves
constexpr uint32_t kSegs = 64, kCounts = 64;             // per launch: 3 KiB of kernel arguments

struct ServeArgs {
  ServeSeg seg[kSegs];
  ServeCount count[kCounts];
  uint32_t nseg, ncount, items, pad;
};
static_assert(sizeof(ServeArgs) <= 4096, "kernel arguments");

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
struct __attribute__((packed, aligned(1))) Unaligned {
  u32x4 v;
};

__global__ void __launch_bounds__(kThreads) k_serve_copy(ServeArgs A) {
  if (blockIdx.x >= A.items) {
    // one wavefront per table: the sums of its count slots
    const uint32_t c = (blockIdx.x - A.items) * (kThreads / 64) + (threadIdx.x >> 6);
    if (c >= A.ncount) return;
    const uint32_t lane = threadIdx.x & 63;
    static_assert(kCountSlots == 64, "one slot per lane");
    const DevStatus *st = A.count[c].st;
    const long long u = wave_sum((long long)st->slot[lane].used);
    const long long l = wave_sum((long long)st->slot[lane].live);
    if (lane == 0) {
      uint64_t *out = A.count[c].out;
      out[0] = (uint64_t)u;
      out[1] = (uint64_t)l;
      out[2] = st->err;
    }
    return;
  }
  uint32_t lo = 0, hi = A.nseg;  // last segment with first <= blockIdx.x
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (A.seg[mid].first <= blockIdx.x) lo = mid; else hi = mid;
  }
  unsigned char *dst = (unsigned char *)A.seg[lo].dst;
  const unsigned char *src = (const unsigned char *)A.seg[lo].src;
  const uint64_t bytes = A.seg[lo].bytes;
  const bool in = A.seg[lo].caller_is_src != 0;
  // bytes before the caller's first 16-byte boundary, then whole 16-byte
  // pieces, then the rest
  const uint64_t caller = (uint64_t)(in ? src : dst);
  const uint64_t head = std::min<uint64_t>((0 - caller) & 15, bytes);
  const uint64_t pieces = (bytes - head) / 16;
  const uint64_t item = blockIdx.x - A.seg[lo].first;
  const uint64_t p0 = item * (kItem / 16);
  u32x4 v[kVecs];
#pragma unroll
  for (uint32_t j = 0; j < kVecs; ++j) {
    const uint64_t p = p0 + j * kThreads + threadIdx.x;
    if (p < pieces) {
      const unsigned char *a = src + head + 16 * p;
      v[j] = in ? *(const u32x4 *)a : ((const Unaligned *)a)->v;
    }
  }
#pragma unroll
  for (uint32_t j = 0; j < kVecs; ++j) {
    const uint64_t p = p0 + j * kThreads + threadIdx.x;
    if (p < pieces) {
      unsigned char *a = dst + head + 16 * p;
      if (in)
        ((Unaligned *)a)->v = v[j];
      else
        *(u32x4 *)a = v[j];
    }
  }
  if (item == 0) {
    // head and tail: at most 15 bytes each
    const uint64_t tail = head + 16 * pieces;
    const uint32_t t = threadIdx.x;
    if (t < 16) {
      if (t < head) dst[t] = src[t];
    } else if (t < 32) {
      const uint64_t i = tail + (t - 16);
      if (i < bytes) dst[i] = src[i];
    }
  }
}

}  // namespace

hipError_t launch_serve_copy(const std::vector<ServeSeg> &segs, const std::vector<ServeCount> &counts,
                             hipStream_t s) {
  drop_stale_error();
  size_t i = 0, c = 0;
  while (i < segs.size() || c < counts.size()) {
    ServeArgs A{};
    uint64_t items = 0;
    // (a segment of 2^31 operations is 2^20 items: far below the grid's limit)
    while (i < segs.size() && A.nseg < kSegs && items < (1u << 22)) {
      ServeSeg g = segs[i++];
      if (g.bytes == 0) continue;
      g.first = (uint32_t)items;
      items += (g.bytes + kItem - 1) / kItem;
      A.seg[A.nseg++] = g;
    }
    while (c < counts.size() && A.ncount < kCounts) A.count[A.ncount++] = counts[c++];
    A.items = (uint32_t)items;
    const uint32_t grid = (uint32_t)items + (A.ncount + kThreads / 64 - 1) / (kThreads / 64);
    if (grid == 0) continue;
    hipLaunchKernelGGL(k_serve_copy, dim3(grid), dim3(kThreads), 0, s, A);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace lpht
