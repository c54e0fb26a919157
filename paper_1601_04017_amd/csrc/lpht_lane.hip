// Bulk operations with one lane per operation (group width 1): the default
// form of every single-table call and of the batch API's multi-table calls.
//
// What bounds it: random lines for finds (51 G lines/s measured on this
// card), random compare-and-swap for insertions (17.9 G/s), launch and memory
// latency for small calls.  So a lane carries exactly one operation from its
// key to its result: no staging in LDS, no hash tables to build, no barrier
// before the first probe, and the hardware's own dispatch of workgroups in
// place of a persistent grid.  A lane looks at its home cell alone (below
// fill 1/2 two in three operations end there, and a wavefront's 64 scattered
// loads cost the address path 64 lines whatever their width), and from then
// on at W cells an iteration, whose loads are in flight together: the wave
// waits for its longest probe run, and W divides the number of waits.
//
// Measured against the staged form (128-operation rounds per wavefront, LDS
// hash tables), KV64 finds: 1500 in 2^12 cells 13.5 -> 7.0 us, 300 007 in 2^24
// 16.5 -> 9.8 us, 2^20 in 2^24 33.3 -> 26.6 us, 10^8 in 2^28 2.95 -> 2.74 ms
// (the same kernel stopping after one cell: 2.66 ms); inserts: 24.5 -> 9.1 us,
// 38 -> 25 us, 83 -> 81 us, 6.1 -> 5.8 ms.

#include <hip/hip_runtime.h>

#include <algorithm>

#include "lpht_device.h"
#include "lpht_lane.h"
#include "lpht_lane_op.h"

namespace lpht {

namespace {

// Adds the wavefront's changes to the counts: insertions (both counts) or
// erasures (live), one atomic per workgroup and count.
template <int OP>
__device__ __forceinline__ void lane_counts(DevStatus *st, uint32_t slot, uint32_t wave_hits, uint32_t *s_hits) {
  if (OP == OP_FIND || OP == OP_UPDATE) return;
  const uint32_t wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) s_hits[wave] = wave_hits;
  __syncthreads();
  if (threadIdx.x == 0) {
    u64 t = 0;
    for (uint32_t w = 0; w < (blockDim.x >> 6); ++w) t += s_hits[w];
    CountSlot *cs = &st->slot[slot % kCountSlots];
    if (t) {
      if (OP == OP_ERASE) {
        add64(&cs->live, 0 - t);
      } else {
        add64(&cs->used, t);
        add64(&cs->live, t);
      }
    }
  }
}

// Operation i of A; returns its flag (0xFD: an operation of another phase).
template <int LAYOUT, int OP, int UP, int W>
__device__ __forceinline__ uint8_t lane_at(const BulkArgs &A, u64 i, uint32_t &err) {
  u64 out = 0;
  uint8_t flag = 0xFD;
  if (!A.kinds || A.kinds[i] == A.kind_sel) {
    const u64 k = word_in<LAYOUT>(A.keys, i);
    if (k == kEmpty || k == kTomb) {
      flag = 0xFE;
      err |= kErrReserved;
    } else {
      const u64 d = OP != OP_FIND && OP != OP_ERASE && A.vals ? word_in<LAYOUT>(A.vals, i) : 1;
      flag = lane_op<LAYOUT, OP, UP, W>(A, k, d, out);
      if (flag == 0xFF) err |= kErrFull;
    }
    if (A.flags) A.flags[i] = flag;
  }
  if (OP == OP_FIND && A.vals_out) {
    if (LAYOUT == 0)
      ((uint32_t *)A.vals_out)[i] = (uint32_t)out;
    else
      ((u64 *)A.vals_out)[i] = out;
  }
  return flag;
}

// Threads per workgroup at most, whatever the tuning asks of the wider group
// kernels: a workgroup's slots free up only when its longest probe run ends
// (10^8 finds in 2^28 KV64 cells: 2.74 / 2.99 ms with 64 to 256 threads,
// 2.84 / 3.18 ms with 512, 2.97 / 3.39 ms with 1024).
constexpr uint32_t kMostThreads = 256;

// One call on one table.
template <int LAYOUT, int OP, int UP, int W>
__global__ void __launch_bounds__(kMostThreads) k_lane(BulkArgs A) {
  __shared__ uint32_t s_hits[kMostThreads / 64];
  uint32_t err = 0, hits = 0;
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 base = (u64)blockIdx.x * blockDim.x; base < A.n; base += stride) {
    const u64 i = base + threadIdx.x;
    uint8_t flag = 0;
    if (i < A.n) flag = lane_at<LAYOUT, OP, UP, W>(A, i, err);
    hits += (uint32_t)__popcll(__ballot(flag == 1));
  }
  lane_errors(A.status, err);
  lane_counts<OP>(A.status, blockIdx.x, hits, s_hits);
}

// One round of kRound operations by a workgroup of kRound threads.
template <int LAYOUT, int OP, int UP, int W>
__device__ __forceinline__ void lane_round(const BulkArgs &A, u64 round, uint32_t slot, uint32_t *s_hits) {
  const u64 i = round * kRound + threadIdx.x;
  uint32_t err = 0;
  uint8_t flag = 0;
  if (i < A.n) flag = lane_at<LAYOUT, OP, UP, W>(A, i, err);
  const uint32_t hits = (uint32_t)__popcll(__ballot(flag == 1));
  lane_errors(A.status, err);
  lane_counts<OP>(A.status, slot, hits, s_hits);
}

// Descriptor j covers rounds [round_start[j], round_start[j + 1]) of kRound
// operations; a workgroup of kRound threads takes a round.
template <int LAYOUT, int OP, int UP, int W>
__global__ void __launch_bounds__(kRound) k_lane_multi(const BulkArgs *descs, const u64 *round_start,
                                                       uint32_t ndesc) {
  __shared__ uint32_t s_hits[kRound / 64];
  const u64 total = round_start[ndesc];
  for (u64 r = blockIdx.x; r < total; r += gridDim.x) {
    uint32_t lo = 0, hi = ndesc;  // last j with round_start[j] <= r
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (round_start[mid] <= r) lo = mid; else hi = mid;
    }
    const BulkArgs A = descs[lo];
    lane_round<LAYOUT, OP, UP, W>(A, r - round_start[lo], (uint32_t)r, s_hits);
    __syncthreads();  // s_hits is written again by the next round
  }
}

// The same from kernel arguments: few descriptors, each of its first round's
// number and the fields a lane needs.
struct LaneDesc {
  void *cells;
  DevStatus *status;
  const void *keys, *vals;
  void *vals_out;
  uint8_t *flags;
  const uint8_t *kinds;
  u64 n, mul;
  u64 first;
  uint32_t log2c, crc_hi, crc_lo, kind_sel;
};
struct LaneFew {
  LaneDesc d[kLaneDescs];
  u64 rounds;
  uint32_t n, pad;
};
static_assert(sizeof(LaneFew) <= 4096, "kernel arguments");

template <int LAYOUT, int OP, int UP, int W>
__global__ void __launch_bounds__(kRound) k_lane_few(LaneFew F) {
  __shared__ uint32_t s_hits[kRound / 64];
  for (u64 r = blockIdx.x; r < F.rounds; r += gridDim.x) {
    uint32_t lo = 0, hi = F.n;
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (F.d[mid].first <= r) lo = mid; else hi = mid;
    }
    const LaneDesc &D = F.d[lo];
    BulkArgs A{};
    A.cells = D.cells;
    A.log2c = D.log2c;
    A.crc_hi = D.crc_hi;
    A.crc_lo = D.crc_lo;
    A.status = D.status;
    A.keys = D.keys;
    A.vals = D.vals;
    A.n = D.n;
    A.vals_out = D.vals_out;
    A.flags = D.flags;
    A.kinds = D.kinds;
    A.kind_sel = D.kind_sel;
    A.mul = D.mul;
    lane_round<LAYOUT, OP, UP, W>(A, r - D.first, (uint32_t)r, s_hits);
    __syncthreads();
  }
}

// Workgroups of a launch: HIP bounds the threads of a grid by 2^32.
constexpr u64 kMaxThreads = 1ull << 31;

// Lookahead: 2 cells up to fill 1/2, 4 above.  KV64, 10^8 finds in 2^28 cells
// at fill 0.37 (hits / misses): W = 2 2.74 / 3.00 ms, W = 4 2.85 / 3.20 ms
// (fetched cells that most lanes do not need); 1.6 * 10^6 in 2^21 at fill 0.75:
// 69.5 / 127.6 us and 56.5 / 92.7 us (long runs, half the waits).
template <int LAYOUT, int OP, int UP>
void lane_launch(const BulkArgs &a, uint32_t threads, bool dense, hipStream_t s) {
  threads = std::min(threads, kMostThreads);
  const u64 blocks = std::min<u64>((a.n + threads - 1) / threads, kMaxThreads / threads);
  if (dense)
    hipLaunchKernelGGL((k_lane<LAYOUT, OP, UP, 4>), dim3((uint32_t)blocks), dim3(threads), 0, s, a);
  else
    hipLaunchKernelGGL((k_lane<LAYOUT, OP, UP, 2>), dim3((uint32_t)blocks), dim3(threads), 0, s, a);
}

// The host does not know every table's fill here: W = 4, which costs small
// calls nothing.
template <int LAYOUT, int OP, int UP>
void lane_launch_multi(const BulkArgs *d, const u64 *rs, uint32_t nd, u64 total, hipStream_t s) {
  const u64 blocks = std::min<u64>(total, kMaxThreads / kRound);
  hipLaunchKernelGGL((k_lane_multi<LAYOUT, OP, UP, 4>), dim3((uint32_t)blocks), dim3(kRound), 0, s, d, rs, nd);
}

template <int LAYOUT, int OP, int UP>
void lane_launch_few(const LaneFew &f, hipStream_t s) {
  const u64 blocks = std::min<u64>(f.rounds, kMaxThreads / kRound);
  hipLaunchKernelGGL((k_lane_few<LAYOUT, OP, UP, 4>), dim3((uint32_t)blocks), dim3(kRound), 0, s, f);
}

}  // namespace

#define LPHT_LANE_OPS(CALL, op, up)                        \
  switch (op) {                                            \
    case OP_FIND: CALL(OP_FIND, 0); break;                 \
    case OP_INSERT: CALL(OP_INSERT, 0); break;             \
    case OP_UPSERT:                                        \
      if (up) CALL(OP_UPSERT, 1); else CALL(OP_UPSERT, 0); \
      break;                                               \
    case OP_UPDATE:                                        \
      if (up) CALL(OP_UPDATE, 1); else CALL(OP_UPDATE, 0); \
      break;                                               \
    case OP_ERASE: CALL(OP_ERASE, 0); break;               \
    default: return hipErrorInvalidValue;                  \
  }

hipError_t launch_lane(OpKind op, const BulkArgs &a, uint32_t threads, bool dense, hipStream_t s) {
  drop_stale_error();
#define LPHT_CALL(OP, UP) \
  (a.layout == 0 ? lane_launch<0, OP, UP>(a, threads, dense, s) : lane_launch<1, OP, UP>(a, threads, dense, s))
  LPHT_LANE_OPS(LPHT_CALL, op, a.up)
#undef LPHT_CALL
  return hipGetLastError();
}

hipError_t launch_lane_few(OpKind op, uint32_t up, uint32_t layout, const BulkArgs *descs, uint32_t ndesc,
                           hipStream_t s) {
  drop_stale_error();
  if (ndesc > kLaneDescs) return hipErrorInvalidValue;
  LaneFew f{};
  for (uint32_t j = 0; j < ndesc; ++j) {
    const BulkArgs &a = descs[j];
    f.d[j] = {a.cells, a.status, a.keys,   a.vals,  a.vals_out, a.flags,  a.kinds,
              a.n,     a.mul,    f.rounds, a.log2c, a.crc_hi,   a.crc_lo, a.kind_sel};
    f.rounds += (a.n + kRound - 1) / kRound;
  }
  f.n = ndesc;
  if (f.rounds == 0) return hipSuccess;
#define LPHT_CALL(OP, UP) (layout == 0 ? lane_launch_few<0, OP, UP>(f, s) : lane_launch_few<1, OP, UP>(f, s))
  LPHT_LANE_OPS(LPHT_CALL, op, up)
#undef LPHT_CALL
  return hipGetLastError();
}

hipError_t launch_lane_multi(OpKind op, uint32_t up, uint32_t layout, const BulkArgs *descs,
                             const uint64_t *round_start, uint32_t ndesc, uint64_t total_rounds, hipStream_t s) {
  drop_stale_error();
  const u64 *rs = (const u64 *)round_start;
  const u64 total = (u64)total_rounds;
#define LPHT_CALL(OP, UP)                                              \
  (layout == 0 ? lane_launch_multi<0, OP, UP>(descs, rs, ndesc, total, s) \
               : lane_launch_multi<1, OP, UP>(descs, rs, ndesc, total, s))
  LPHT_LANE_OPS(LPHT_CALL, op, up)
#undef LPHT_CALL
  return hipGetLastError();
}

}  // namespace lpht
