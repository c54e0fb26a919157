// Partitioned insertOrUpdate with the "add" update function (Algorithm 1
// with fetch-and-add) for large calls.
//
// Equal keys can only be combined while they are in one workgroup's LDS at
// the same time.  A skewed stream (Zipf keys) repeats its rare keys a few
// times across the whole batch, so chunk-local combining leaves one global
// atomic per occurrence for them, and the device's atomics (about 18 G/s,
// whether the addresses are spread over HBM or confined to a small region)
// bound the call.  Here the batch is first partitioned by the top bits of the
// table's hash, which is also a partition of the table into regions (the
// position is the top log2 c bits of the hash, Sec. 5.3.1): every occurrence
// of a key lands in the same bucket, a bucket's operations are combined in a
// large LDS table by one workgroup, and each distinct key costs one upsert
// into its region of the table.  This is the bulk-operation idea of Sec. 5.5
// (sort the batch by hash before touching the table) with a one-level
// partition instead of a full sort, since the result of "add" does not depend
// on the order.
//
// Passes: the partition runs in two levels, 128 buckets of the top 7 hash
// bits and then 64 sub-buckets of the next 6 bits inside each (on tables of
// 2^21 cells or more).  A count (histograms over all buckets of contiguous
// shares) and a scan by one workgroup give every bucket's start in both
// levels, and two scatters, tile by tile through LDS, bring keys, values and
// indices into bucket order: bound by memory, 1.6 GB per 10^8 keys and level
// at 4.1 TB/s.  Skewed streams put one key on most lanes of a wavefront, so
// the LDS atomics of the count and of the apply first combine the lanes that
// share the leading lane's bucket or key.  The scan also lays out the work
// items (at most kItemOps operations inside one bucket).
// 10^8 keys of a Zipf(1) stream: count 0.21 ms, sum and scan 0.04, scatters
// 0.40 and 0.39 ms (a count of each level, 0.49 ms, and scatters of single
// elements behind cursors, 0.80 and 0.53 ms, before).  Then apply: one
// workgroup per work item combines the item in LDS and makes one single-lane
// upsert per distinct key.  When a bucket is a single work item, every
// operation on its keys is in that workgroup, and after the workgroup
// barrier each combined key is applied by one lane only: a new key is
// claimed with compare-and-swap and its sum written by a plain store, which
// halves the atomics of a fresh table; on a KV64 table without a used cell, in a
// call without flags, no compare-and-swap is needed at all (FRESH below).
// Flags: the count pass writes 0 for
// every operation (0xFE for reserved keys), and the operation with the
// smallest index among a slot's operations receives the upsert's result.
// Keys that find no LDS slot (the table is three quarters full, or kProbe
// steps found none) are applied on their own, which keeps "add" exact and
// gives a key's inserted flag to exactly one operation.

#include <hip/hip_runtime.h>

#include <algorithm>

#include "lpht_device.h"
#include "lpht_lane_op.h"
#include "lpht_part.h"

namespace lpht {

namespace {

constexpr uint32_t kBits1 = 7;          // first-level buckets: 128
constexpr uint32_t kMaxBits = 13;       // at most 8192 buckets in all
constexpr uint32_t kCountWG = 512;      // workgroups of the count pass
constexpr uint32_t kCountThreads = 512;
constexpr uint32_t kTile = 4096;        // elements of one scatter workgroup
constexpr uint32_t kPad = 32;           // first-level cursors on lines of their own
constexpr uint32_t kSumSplit = 8;       // rows of workgroups a bucket's total is summed in
// apply workgroups: without flags two per CU (one combines while the other
// makes its upserts), with flags one
// The apply waits for LDS: 1024 threads of four operations each (64 VGPRs) in
// place of 512 of eight, 2^24 Zipf(1) keys 519 -> 460 us for the call, PACKED32
// 643 -> 508.
constexpr uint32_t kApplyThreads = 1024;
constexpr uint32_t kApplyUnroll = 4;
constexpr uint32_t kItemOps = 32768;    // operations per apply work item
// LDS combining slots: 4096 of 16 B (64 KiB, two workgroups per CU; with
// flags each slot also keeps its representative's index) hold the ~2.2k
// distinct keys of a bucket of a 10^8-key Zipf(1) batch in 8192 buckets
constexpr uint32_t kSlotsNoFlags = 4096;
constexpr uint32_t kSlotsFlags = 4096;
constexpr uint32_t kProbe = 32;
constexpr uint32_t kUnroll = 8;         // loads in flight per lane in the count

struct PartK {
  BulkArgs A;
  uint32_t nwg;          // workgroups of the count pass
  uint32_t bits;         // buckets in all: the top `bits` bits of the hash
  uint64_t chunk;        // elements per count workgroup (contiguous)
  uint32_t *hist;        // [nwg][buckets]: the count workgroups' counts
  uint64_t *btot;        // [buckets + 1]: totals (zeroed), then bucket starts; the last: all elements
  uint32_t *cur[2];      // by level: next free position of each bucket (the first level's kPad apart)
  uint32_t *tiles;       // [first-level buckets + 1]: first second-level tile of each
  uint32_t *items;       // [buckets + 1]: first work item of each bucket
  // [items + 1]: first element of each work item, bit 63 set when the item is
  // its bucket's only one; the last entry is the total
  uint64_t *istart;
  // keys put off (a fresh table), in the first level's arrays, which are free by
  // then: with values, off[0] of keys and values; without, off[0] keys of one
  // operation from the front and off[1] keys with their sums from the back
  uint32_t *off;
  // work items taken, past the two each apply workgroup begins with (items
  // differ: of a hot key, of a short bucket; dealt out in turn, 10^8 Zipf(1)
  // keys took 1.07 ms in the apply, now 0.96)
  uint32_t *next;
  // by level: keys, values (calls with values) and operation indices (calls
  // with flags) in bucket order
  void *keys[2], *vals[2];
  uint32_t *idx[2];
};

uint32_t bucket_bits(uint32_t log2c) { return std::min<uint32_t>(kMaxBits, log2c - 8); }

size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

template <int L>
__device__ __forceinline__ u64 part_key(const void *p, u64 i) {
  return L == 0 ? (u64)((const uint32_t *)p)[i] : ((const u64 *)p)[i];
}

template <int L>
__device__ __forceinline__ u64 part_key_nt(const void *p, u64 i) {
  return L == 0 ? (u64)__builtin_nontemporal_load((const uint32_t *)p + i)
                : __builtin_nontemporal_load((const u64 *)p + i);
}

// LDS slot of a key: a mix of all its bits (the table hash's top bits are the
// same for every key of a bucket) by 32-bit products, which take a fifth of
// the VALU's time for a 64-bit one.
__device__ __forceinline__ uint32_t lds_slot(u64 key, uint32_t bits) {
  uint32_t z = (uint32_t)key ^ ((uint32_t)(key >> 32) * 0x85EBCA6Bu);
  z = (z ^ (z >> 15)) * 0xC2B2AE35u;
  z = (z ^ (z >> 13)) * 0x9E3779B1u;
  return z >> (32 - bits);
}

// Reports the wavefront's sticky error bits once.
__device__ __forceinline__ void wave_err(DevStatus *st, uint32_t err) {
  if (__ballot(err != 0)) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) err |= __shfl_xor(err, o, 64);
    if ((threadIdx.x & 63) == 0) atomicOr(&st->err, err);
  }
}

// Wavefront-level aggregation: the mask of the active lanes whose tag equals
// the first active lane's, that lane and its tag (read as scalars).  Skewed
// streams put one key (or bucket) on most lanes of a wavefront; combining them
// first turns up to 64 serialised LDS atomics on one address into one.
template <class Tag>
__device__ __forceinline__ u64 match_first(bool active, Tag tag, Tag &lead_tag, uint32_t &lead) {
  const u64 act = __ballot(active);
  if (!act) return 0;
  lead = (uint32_t)__builtin_ctzll(act);
  lead_tag = (Tag)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)tag, (int)lead);
  if constexpr (sizeof(Tag) == 8)
    lead_tag |= (Tag)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((u64)tag >> 32), (int)lead) << 32;
  return __ballot(active && tag == lead_tag);
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint32_t t = __shfl_xor(v, o, 64);
    v = t < v ? t : v;
  }
  return v;
}

constexpr int kAggRounds = 2;  // leading tags combined per wavefront step
// lanes of one tag worth combining: fewer cost the LDS less than the round
constexpr int kAggLanes = 6;

__global__ void __launch_bounds__(1024) k_part_zero(PartK k) {
  for (uint32_t b = threadIdx.x; b <= (1u << k.bits); b += blockDim.x) k.btot[b] = 0;
  if (threadIdx.x < 2) k.off[threadIdx.x] = 0;
  if (threadIdx.x == 2) *k.next = 0;
}

// Count pass: histogram of this workgroup's contiguous share over all buckets
// (both levels are laid out from it; a count of the first level's output for
// the second, 245 us per 10^8 keys, is not needed).
template <int L>
__global__ void __launch_bounds__(kCountThreads) k_part_count(PartK k) {
  __shared__ uint32_t T[8][256];
  __shared__ uint32_t h[1u << kMaxBits];
  crc_tables_build(T);
  const uint32_t nb = 1u << k.bits;
  for (uint32_t b = threadIdx.x; b < nb; b += blockDim.x) h[b] = 0;
  __syncthreads();
  const BulkArgs &A = k.A;
  const u64 n = A.n;
  const u64 lo = (u64)blockIdx.x * k.chunk;
  const u64 hi = lo + k.chunk < n ? lo + k.chunk : n;
  uint32_t err = 0;
  // kUnroll independent loads per lane before any is used, and the next
  // tile's loads issued before this tile is counted: enough bytes in flight
  // to cover the memory latency
  const u64 step = (u64)blockDim.x * kUnroll;
  u64 key[kUnroll];
  auto load = [&](u64 base) {
#pragma unroll
    for (uint32_t j = 0; j < kUnroll; ++j) {
      const u64 i = base + (u64)j * blockDim.x + threadIdx.x;
      key[j] = i < hi ? part_key<L>(A.keys, i) : 0;
    }
  };
  if (lo < hi) load(lo);
  for (u64 base = lo; base < hi; base += step) {
    u64 ck[kUnroll];
#pragma unroll
    for (uint32_t j = 0; j < kUnroll; ++j) ck[j] = key[j];
    if (base + step < hi) load(base + step);
#pragma unroll
    for (uint32_t j = 0; j < kUnroll; ++j) {
      const u64 i = base + (u64)j * blockDim.x + threadIdx.x;
      bool act = i < hi;
      if (act) {
        if (ck[j] == kEmpty || ck[j] == kTomb) {
          err |= kErrReserved;
          if (A.flags) A.flags[i] = 0xFE;
          act = false;
        } else if (A.flags) {
          A.flags[i] = 0;
        }
      }
      const uint32_t b = act ? (uint32_t)(hash_of<L>(T, ck[j], A.crc_hi, A.crc_lo, A.mul) >> (64 - k.bits)) : 0;
      for (int r = 0; r < kAggRounds; ++r) {
        uint32_t lt = 0, ll = 0;
        const u64 m = match_first(act, b, lt, ll);
        if (__popcll(m) < kAggLanes) break;
        if ((threadIdx.x & 63) == ll) atomicAdd(&h[lt], (uint32_t)__popcll(m));
        if ((m >> (threadIdx.x & 63)) & 1) act = false;
      }
      if (act) atomicAdd(&h[b], 1u);
    }
  }
  wave_err(A.status, err);
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < nb; b += blockDim.x) k.hist[(u64)blockIdx.x * nb + b] = h[b];
}

// Bucket totals: the columns of the count workgroups' histograms, in
// kSumSplit parts (an atomic per workgroup and bucket would be 4 million).
__global__ void __launch_bounds__(256) k_part_sum(PartK k) {
  const uint32_t b = blockIdx.x * 256 + threadIdx.x, nb = 1u << k.bits;
  u64 sum = 0;
#pragma unroll 8
  for (uint32_t w = blockIdx.y; w < k.nwg; w += kSumSplit) sum += k.hist[(u64)w * nb + b];
  if (sum) atomicAdd((unsigned long long *)&k.btot[b], (unsigned long long)sum);
}

// Exclusive scan of one value per thread over a workgroup of 1024 threads.
__device__ __forceinline__ u64 block_scan_1024(u64 v, u64 *s_w, u64 *total) {
  const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  u64 x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const u64 t = __shfl_up(x, o, 64);
    if (lane >= (uint32_t)o) x += t;
  }
  if (lane == 63) s_w[w] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    u64 run = 0;
    for (uint32_t i = 0; i < blockDim.x / 64; ++i) {
      const u64 t = s_w[i];
      s_w[i] = run;
      run += t;
    }
    *total = run;
  }
  __syncthreads();
  return s_w[w] + x - v;
}

// One workgroup of 1024 threads, up to eight buckets per thread: bucket
// starts, the first work item of each bucket and each item's range, the
// cursors of both levels and the second level's tiles.
__global__ void __launch_bounds__(1024) k_part_scan(PartK k) {
  __shared__ u64 s_w[16];
  __shared__ u64 s_tot;
  const uint32_t nb = 1u << k.bits;
  const uint32_t per = (nb + blockDim.x - 1) / blockDim.x;
  const uint32_t b0 = threadIdx.x * per;
  u64 tot[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  u64 els = 0, its = 0;
  for (uint32_t j = 0; j < per && j < 8; ++j) {
    const uint32_t b = b0 + j;
    if (b < nb) {
      tot[j] = k.btot[b];
      els += tot[j];
      its += (tot[j] + kItemOps - 1) / kItemOps;
    }
  }
  const u64 e0 = block_scan_1024(els, s_w, &s_tot);
  const u64 etotal = s_tot;
  __syncthreads();
  const u64 i0 = block_scan_1024(its, s_w, &s_tot);
  const u64 itotal = s_tot;
  u64 e = e0, it = i0;
  for (uint32_t j = 0; j < per && j < 8; ++j) {
    const uint32_t b = b0 + j;
    if (b < nb) {
      k.btot[b] = e;
      k.cur[1][b] = (uint32_t)e;
      const u64 ni = (tot[j] + kItemOps - 1) / kItemOps;
      k.items[b] = (uint32_t)it;
      for (u64 q = 0; q < ni; ++q) k.istart[it + q] = (e + q * kItemOps) | (ni == 1 ? 1ull << 63 : 0);
      e += tot[j];
      it += ni;
    }
  }
  if (threadIdx.x == 0) {
    k.btot[nb] = etotal;
    k.items[nb] = (uint32_t)itotal;
    k.istart[itotal] = etotal;
  }
  __syncthreads();
  const uint32_t sub = k.bits - kBits1, f = threadIdx.x;
  u64 start = 0, tiles = 0;
  if (f < (1u << kBits1)) {
    start = k.btot[f << sub];
    tiles = (k.btot[(f + 1) << sub] - start + kTile - 1) / kTile;
  }
  const u64 t0 = block_scan_1024(tiles, s_w, &s_tot);
  if (f < (1u << kBits1)) {
    k.cur[0][f * kPad] = (uint32_t)start;
    k.tiles[f] = (uint32_t)t0;
  }
  if (f == 0) k.tiles[1u << kBits1] = (uint32_t)s_tot;
}

// Scatter pass of level LV in tiles of 4096 elements: ranked inside their
// bucket by LDS atomics, put in bucket order in LDS and written as runs behind
// one reservation per bucket and tile (of a uniform hash 32 elements a run in
// the first level and 64 in the second, so most written lines are whole;
// written one by one, behind cursors in LDS, L2 wrote lines back part-filled).
// The first level's tiles are those of the batch, the second level's lie in
// one first-level bucket each.  VALS, IDX: the level moves values and
// operation indices along with the keys.  Equal keys cost same-address LDS
// atomics and still one reservation per tile; a wavefront whose elements all
// lie in one bucket ranks itself (2^24 operations on one key: the call 357 ->
// 309 us; 402 with single elements behind cursors).
// A KV64 call with values and indices needs 92 KiB of LDS, so one workgroup
// per CU: of twice the wavefronts then.
template <int L, bool VALS, bool IDX>
constexpr uint32_t scatter_threads() { return L == 1 && VALS && IDX ? 1024 : 512; }

template <int L, bool VALS, bool IDX, int LV>
__global__ void __launch_bounds__((scatter_threads<L, VALS, IDX>()), 4) k_part_scatter(PartK k) {
  using Word = typename std::conditional<L == 0, uint32_t, u64>::type;
  constexpr uint32_t NT = scatter_threads<L, VALS, IDX>(), PER = kTile / NT;
  constexpr uint32_t NB = 1u << (LV == 0 ? kBits1 : kMaxBits - kBits1);
  __shared__ Word kbuf[kTile];
  __shared__ Word vbuf[VALS ? kTile : 1];
  __shared__ uint32_t ibuf[IDX ? kTile : 1];
  __shared__ uint16_t bkt[kTile];
  // by bucket: elements, their start in the tile, then their position less that
  __shared__ uint32_t toff[NB];
  __shared__ uint32_t T[1024];
  __shared__ uint32_t s_w[NB / 64], s_f;
  const BulkArgs &A = k.A;
  const uint32_t sub = k.bits - kBits1, nb = LV == 0 ? NB : 1u << sub, lane = threadIdx.x & 63;
  u64 base;
  uint32_t m, f = 0;
  if (LV == 0) {
    base = (u64)blockIdx.x * kTile;
    m = (uint32_t)std::min<u64>(kTile, A.n - base);
  } else {
    // each XCD (workgroups are dealt out over eight) takes a range of the
    // tiles, so that one L2 joins the runs of a bucket
    const uint32_t all = k.tiles[1u << kBits1];
    const uint32_t t = (blockIdx.x & 7) * ((all + 7) / 8) + (blockIdx.x >> 3);
    if (blockIdx.x >> 3 >= (all + 7) / 8 || t >= all) return;
    if (threadIdx.x < (1u << kBits1) && k.tiles[threadIdx.x] <= t && t < k.tiles[threadIdx.x + 1]) s_f = threadIdx.x;
    __syncthreads();
    f = s_f;
    base = k.btot[f << sub] + (u64)(t - k.tiles[f]) * kTile;
    m = (uint32_t)std::min<u64>(kTile, k.btot[(f + 1) << sub] - base);
  }
  crc_slices_load(T);
  if (threadIdx.x < nb) toff[threadIdx.x] = 0;
  Word key[PER], val[PER];
  uint32_t ix[PER], at[PER];
  bool ok[PER];
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    const uint32_t t = j * NT + threadIdx.x;
    const u64 i = base + t;
    ok[j] = t < m;
    key[j] = ok[j] ? (Word)part_key_nt<L>(LV == 0 ? A.keys : k.keys[0], i) : 0;
    val[j] = VALS && ok[j] ? (Word)part_key_nt<L>(LV == 0 ? A.vals : k.vals[0], i) : 0;
    ix[j] = IDX && ok[j] ? (LV == 0 ? (uint32_t)i : __builtin_nontemporal_load(k.idx[0] + i)) : 0;
    if (LV == 0) ok[j] = key[j] != (Word)kEmpty && key[j] != (Word)kTomb;  // kEmpty past the end, too
  }
  __syncthreads();
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    const uint32_t all = (uint32_t)(hash_sliced<L>(T, (u64)key[j], A.crc_hi, A.crc_lo, A.mul) >> (64 - k.bits));
    const uint32_t b = LV == 0 ? all >> sub : all & (nb - 1);
    // a wavefront of one bucket ranks itself
    if (__all(ok[j] && b == (uint32_t)__builtin_amdgcn_readfirstlane((int)b))) {
      uint32_t r = 0;
      if (lane == 0) r = atomicAdd(&toff[b], 64u);
      at[j] = b | (((uint32_t)__builtin_amdgcn_readfirstlane((int)r) + lane) << 16);
      continue;
    }
    if (ok[j]) at[j] = b | (atomicAdd(&toff[b], 1u) << 16);
  }
  __syncthreads();
  uint32_t to = 0;
  {
    const uint32_t c = threadIdx.x < nb ? toff[threadIdx.x] : 0;
    uint32_t x = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if (lane >= (uint32_t)o) x += y;
    }
    if (threadIdx.x < NB && lane == 63) s_w[threadIdx.x >> 6] = x;
    if (c) to = atomicAdd(LV == 0 ? &k.cur[0][threadIdx.x * kPad] : &k.cur[1][((u64)f << sub) + threadIdx.x], c);
    __syncthreads();
    uint32_t before = x - c;
    if (threadIdx.x < NB)
      for (uint32_t w = 0; w < (threadIdx.x >> 6); ++w) before += s_w[w];
    if (threadIdx.x < nb) toff[threadIdx.x] = before;
    to -= before;
  }
  __syncthreads();
  uint32_t total = 0;
  for (uint32_t w = 0; w < NB / 64; ++w) total += s_w[w];
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    if (!ok[j]) continue;
    const uint32_t b = at[j] & 0xFFFFu, p = toff[b] + (at[j] >> 16);
    kbuf[p] = key[j];
    bkt[p] = (uint16_t)b;
    if (VALS) vbuf[p] = val[j];
    if (IDX) ibuf[p] = ix[j];
  }
  __syncthreads();
  if (threadIdx.x < nb) toff[threadIdx.x] = to;
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < total; i += NT) {
    const u64 q = toff[bkt[i]] + i;
    ((Word *)k.keys[LV])[q] = kbuf[i];
    if (VALS) ((Word *)k.vals[LV])[q] = vbuf[i];
    if (IDX) k.idx[LV][q] = ibuf[i];
  }
}

template <int L, bool VALS, bool IDX>
hipError_t launch_scatters(const PartK &k, hipStream_t s) {
  const uint32_t tiles = (uint32_t)((k.A.n + kTile - 1) / kTile);
  constexpr uint32_t NT = scatter_threads<L, VALS, IDX>();
  hipLaunchKernelGGL((k_part_scatter<L, VALS, IDX, 0>), dim3(tiles), dim3(NT), 0, s, k);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // a first-level bucket's last tile may be short; a multiple of eight
  const uint32_t tiles2 = (tiles + (1u << kBits1) + 7) & ~7u;
  hipLaunchKernelGGL((k_part_scatter<L, VALS, IDX, 1>), dim3(tiles2), dim3(NT), 0, s, k);
  return hipGetLastError();
}

// insertOrUpdate(k, d, add) by the only lane that updates k in this call
// (its bucket is one work item and the item's combined keys are applied one
// per lane): a new key is claimed with compare-and-swap and its value, 0 in
// an empty cell, set by a plain store; a present key gets fetch-and-add.
__device__ __forceinline__ uint8_t upsert_add_excl_kv64(const BulkArgs &A, const uint32_t (*T)[256], u64 k,
                                                        u64 d, long long &d_used, long long &d_live,
                                                        uint32_t &err) {
  const u64 cap = 1ull << A.log2c, mask = cap - 1;
  u64 p = home_of<1>(T, k, A.crc_hi, A.crc_lo, A.mul, A.log2c);
  for (u64 probes = 0; probes < cap; ++probes, p = (p + 1) & mask) {
    u64 *kp = (u64 *)A.cells + 2 * p;
    u64 ck = *kp;
    if (ck == kEmpty) {
      const u64 old = cas64(kp, kEmpty, k);
      if (old == kEmpty) {
        kp[1] = d;
        d_used += 1;
        d_live += 1;
        return 1;
      }
      ck = old;
    }
    if (ck == k) {
      add64(kp + 1, d);
      return 0;
    }
  }
  err |= kErrFull;
  return 0xFF;
}

// A key that found no cell in its bucket's region of a fresh table.  Without
// values a sum is a number of operations, so that keys and sums of two and
// more take no more words than the operations they combine.
__device__ __forceinline__ void put_off(const PartK &k, u64 key, u64 d) {
  u64 *keys = (u64 *)k.keys[0];
  if (k.vals[0]) {
    const uint32_t i = atomicAdd(&k.off[0], 1u);
    keys[i] = key;
    ((u64 *)k.vals[0])[i] = d;
  } else if (d == 1) {
    keys[atomicAdd(&k.off[0], 1u)] = key;
  } else {
    u64 *e = keys + (k.A.n - 2 - 2 * (u64)atomicAdd(&k.off[1], 1u));
    e[0] = d;
    e[1] = key;
  }
}

// insertOrUpdate(k, d, add) from cell p up to the cell `end` of the bucket's
// region; false: no cell found.
__device__ __forceinline__ bool upsert_add_region(void *cells, u64 p, u64 end, u64 key, u64 d, long long &d_new) {
  for (; p < end; ++p) {
    u64 *kp = (u64 *)cells + 2 * p;
    u64 ck = *kp;
    if (ck == kEmpty) {
      ck = cas64(kp, kEmpty, key);
      if (ck == kEmpty) {
        add64(kp + 1, d);
        d_new += 1;
        return true;
      }
    }
    if (ck == key) {
      add64(kp + 1, d);
      return true;
    }
  }
  return false;
}

// FRESH (KV64 without flags; the table has no used cell): a bucket that is one
// work item owns its region of the table, and its combined keys are distinct,
// so each takes a cell by one bit of a map in LDS and writes key and sum with
// one store; no compare-and-swap, whose memory-side rate (17.9 G/s) bounds the
// other form.  Probes that run past the region's end are put off until all
// regions are done (k_part_rest), also those of the buckets that go by
// compare-and-swap here: of several items, or with more keys than LDS slots.
// 10^8 keys of a Zipf(1) stream (18 * 10^6 distinct) on 2^28 cells: the apply
// 1.60 -> 1.23 ms; 2^24 distinct keys on 2^26 cells: the call 1646 -> 751 us.
// Of what is left (0.96 ms) 0.24 are loads, 0.2 the stores, and the rest the
// combining in LDS.
constexpr uint32_t kFreshBits = 16;  // cells of a region: at most 2^16 (a map of 8 KiB; two workgroups per CU)

template <int L, bool VALS, bool FL, bool FRESH>
__global__ void __launch_bounds__(kApplyThreads, FL ? 4 : 8) k_part_apply(PartK k) {
  constexpr uint32_t S = FL ? kSlotsFlags : kSlotsNoFlags;
  constexpr uint32_t SB = 12;
  static_assert((1u << SB) == S, "slot bits");
  static_assert(!FRESH || (L == 1 && !FL), "fresh: KV64 without flags");
  __shared__ uint32_t T[FRESH ? 4 : 8][256];
  __shared__ uint32_t s_taken[FRESH ? (1u << kFreshBits) / 32 : 1];
  __shared__ uint32_t s_spilled[2];  // by turn: some key of the item found no LDS slot
  __shared__ u64 s_key[S];
  __shared__ u64 s_sum[S];
  __shared__ uint32_t s_rep[FL ? S : 1];
  __shared__ uint32_t s_claims, s_next;
  __shared__ long long s_acc[2];
  __shared__ uint32_t s_err;
  const uint32_t rbits = k.A.log2c - k.bits, map = FRESH ? ((1u << rbits) + 31) / 32 : 0;
  if constexpr (FRESH) {
    crc_slices_load(&T[0][0]);
    for (uint32_t q = threadIdx.x; q < map; q += blockDim.x) s_taken[q] = 0;
  } else {
    crc_tables_build(T);
  }
  if (threadIdx.x < 2) s_spilled[threadIdx.x] = 0;
  for (uint32_t q = threadIdx.x; q < S; q += blockDim.x) {
    s_key[q] = 0;
    s_sum[q] = 0;
    if (FL) s_rep[q] = ~0u;
  }
  if (threadIdx.x == 0) s_claims = 0;
  __syncthreads();
  const BulkArgs &A = k.A;
  long long d_used = 0, d_live = 0;
  uint32_t err = 0;
  const uint32_t nitems = k.items[1u << k.bits];
  const u64 step = (u64)blockDim.x * kApplyUnroll;
  constexpr u64 kAlone = 1ull << 63;
  u64 keys[kApplyUnroll], ds[kApplyUnroll];
  uint32_t idxs[kApplyUnroll];
  auto load = [&](u64 pb, u64 hi) {
#pragma unroll
    for (uint32_t u = 0; u < kApplyUnroll; ++u) {
      const u64 p = pb + (u64)u * blockDim.x + threadIdx.x;
      const bool in = p < hi;
      keys[u] = in ? part_key<L>(k.keys[1], p) : 0;
      ds[u] = VALS ? (in ? part_key<L>(k.vals[1], p) : 0) : 1;
      idxs[u] = in && FL ? k.idx[1][p] : 0;
    }
  };
  // item j covers [istart[j], istart[j + 1]) without the flag bit
  u64 lo = 0, hi = 0;
  bool alone = false;
  if (blockIdx.x < nitems) {
    const u64 s0 = k.istart[blockIdx.x];
    lo = s0 & ~kAlone;
    hi = k.istart[blockIdx.x + 1] & ~kAlone;
    alone = (s0 & kAlone) != 0;
    load(lo, hi);
  }
  uint32_t turn = 0;
  for (uint32_t it = blockIdx.x, nx = it + gridDim.x; it < nitems; turn ^= 1) {
    for (u64 pb = lo; pb < hi; pb += step) {
     u64 ck[kApplyUnroll], cd[kApplyUnroll];
     uint32_t ci[kApplyUnroll];
#pragma unroll
     for (uint32_t u = 0; u < kApplyUnroll; ++u) {
       ck[u] = keys[u];
       cd[u] = ds[u];
       ci[u] = idxs[u];
     }
     // the next tile's loads (this item's, else the next item's first) are
     // in flight while this one is combined
     if (pb + step < hi) {
       load(pb + step, hi);
     } else if (nx < nitems) {
       load(k.istart[nx] & ~kAlone, k.istart[nx + 1] & ~kAlone);
     }
#pragma unroll
     for (uint32_t u = 0; u < kApplyUnroll; ++u) {
      // equal keys on the lanes of this step first (a batch key is never 0
      // here, so 0 marks lanes past the end)
      bool act = ck[u] != 0;
      bool open = act;  // not yet in a group
      const u64 key = ck[u];
      u64 d = cd[u];
      uint32_t idx = ci[u];
      // every lane runs every round (the shuffles read all lanes)
      for (int r = 0; r < kAggRounds; ++r) {
        u64 lk = 0;
        uint32_t ll = 0;
        const u64 m = match_first(open, key, lk, ll);
        if (__popcll(m) < kAggLanes) break;
        const bool in = (m >> (threadIdx.x & 63)) & 1;
        // without values every operation adds 1
        const u64 sum = VALS ? (u64)wave_sum(in ? (long long)d : 0) : (u64)__popcll(m);
        const uint32_t imin = FL ? wave_min_u32(in ? idx : ~0u) : 0;
        if (in) {
          open = false;
          if ((threadIdx.x & 63) == ll) {
            // the leading lane carries the group on
            d = sum;
            idx = imin;
          } else {
            act = false;
          }
        }
      }
      if (!act) continue;
      const bool claim = __hip_atomic_load(&s_claims, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) <
                         S / 4 * 3;
      // two slots a step: most keys are present, and a wavefront goes on until
      // its last lane has found its own
      auto slot_key = [&](uint32_t q) {
        return __hip_atomic_load(&s_key[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      };
      uint32_t slot = lds_slot(key, SB - 1) * 2;
      bool held = false;
      for (uint32_t t = 0; t < kProbe;) {
        const u64 k0 = slot_key(slot), k1 = slot_key(slot + 1);
        const uint32_t at = slot + (k0 == key || k0 == 0 ? 0 : 1);
        u64 cur = k0 == key || k0 == 0 ? k0 : k1;
        if (cur == 0) {
          if (!claim) break;  // absent: no lane claims slots any more in this item
          cur = atomicCAS((unsigned long long *)&s_key[at], 0ull, (unsigned long long)key);
          if (cur == 0) {
            atomicAdd(&s_claims, 1u);
            cur = key;
          } else if (cur != key) {
            continue;  // another key took it: the pair again
          }
        }
        if (cur == key) {
          slot = at;
          held = true;
          break;
        }
        slot = (slot + 2) & (S - 1);
        t += 2;
      }
      if (held) {
        atomicAdd((unsigned long long *)&s_sum[slot], (unsigned long long)d);
        if (FL) atomicMin(&s_rep[slot], idx);
      } else {
        // applied on its own, by atomics, before the barrier below
        if constexpr (FRESH) {
          const u64 p = hash_sliced<1>(&T[0][0], key, A.crc_hi, A.crc_lo, A.mul) >> (64 - A.log2c);
          if (!upsert_add_region(A.cells, p, ((p >> rbits) + 1) << rbits, key, d, d_used)) put_off(k, key, d);
          s_spilled[turn] = 1;
        } else {
          const uint8_t f = upsert_add_one<L>(A, T, key, d, d_used, d_live, err);
          if (FL) A.flags[idx] = f;
        }
      }
     }
    }
    __syncthreads();
    // nothing reads the claim count again before the barrier that ends the item
    if (threadIdx.x == 0) {
      s_claims = 0;
      s_spilled[turn ^ 1] = 0;  // (the next item's)
      s_next = 2 * gridDim.x + atomicAdd(k.next, 1u);
    }
    const bool own = FRESH && alone && !s_spilled[turn];
    // one upsert per distinct key of the item
    for (uint32_t q = threadIdx.x; q < S; q += blockDim.x) {
      const u64 key = s_key[q];
      if (key == 0) continue;
      if constexpr (FRESH) {
        const u64 d = s_sum[q], p = hash_sliced<1>(&T[0][0], key, A.crc_hi, A.crc_lo, A.mul) >> (64 - A.log2c);
        const u64 first = p >> rbits << rbits;
        if (own) {
          uint32_t c = (uint32_t)(p - first);
          while (c < (1u << rbits)) {
            const uint32_t free = ~s_taken[c >> 5] & (~0u << (c & 31));
            if (free) {
              c = (c & ~31u) | (uint32_t)__builtin_ctz(free);
              if (!(atomicOr(&s_taken[c >> 5], 1u << (c & 31)) >> (c & 31) & 1u)) break;
            } else {
              c = (c | 31u) + 1;
            }
          }
          if (c < (1u << rbits)) {
            ((u64x2 *)A.cells)[first + c] = u64x2{key, d};
            d_used += 1;
          } else {
            put_off(k, key, d);
          }
        } else if (!upsert_add_region(A.cells, p, first + (1ull << rbits), key, d, d_used)) {
          put_off(k, key, d);
        }
        s_key[q] = 0;
        s_sum[q] = 0;
        continue;
      }
      const uint8_t f = (L == 1 && alone) ? upsert_add_excl_kv64(A, T, key, s_sum[q], d_used, d_live, err)
                                          : upsert_add_one<L>(A, T, key, s_sum[q], d_used, d_live, err);
      if (FL) {
        A.flags[s_rep[q]] = f;
        s_rep[q] = ~0u;
      }
      s_key[q] = 0;
      s_sum[q] = 0;
    }
    __syncthreads();
    if (own)
      for (uint32_t q = threadIdx.x; q < map; q += blockDim.x) s_taken[q] = 0;
    if (nx < nitems) {
      const u64 s0 = k.istart[nx];
      lo = s0 & ~kAlone;
      hi = k.istart[nx + 1] & ~kAlone;
      alone = (s0 & kAlone) != 0;
    }
    it = nx;
    nx = s_next;
  }
  if (FRESH) d_live = d_used;
  flush_counts(A.status, d_used, d_live, err, s_acc, &s_err);
}

// The keys put off, one lane each on the whole table.
__global__ void __launch_bounds__(256) k_part_rest(PartK k) {
  __shared__ long long s_acc[2];
  __shared__ uint32_t s_err;
  const u64 *keys = (const u64 *)k.keys[0];
  const u64 n0 = k.off[0], n = n0 + k.off[1];
  long long d_used = 0;
  uint32_t err = 0;
  for (u64 i = (u64)blockIdx.x * 256 + threadIdx.x; i < n; i += (u64)gridDim.x * 256) {
    u64 key, d = 1, none;
    if (i < n0) {
      key = keys[i];
      if (k.vals[0]) d = ((const u64 *)k.vals[0])[i];
    } else {
      const u64 *e = keys + (k.A.n - 2 - 2 * (i - n0));
      d = e[0];
      key = e[1];
    }
    const uint8_t f = lane_op<1, OP_UPSERT, 1, 4>(k.A, key, d, none);
    if (f == 0xFF)
      err |= kErrFull;
    else
      d_used += f;
  }
  flush_counts(k.A.status, d_used, d_used, err, s_acc, &s_err);
}

// As many apply workgroups as fit at once (LDS bounds them).
template <int L, bool VALS>
hipError_t launch_apply(const PartK &k, bool fresh, uint32_t num_cus, hipStream_t s) {
  const uint32_t cus = std::max<uint32_t>(1, num_cus);
  if (k.A.flags) {
    hipLaunchKernelGGL((k_part_apply<L, VALS, true, false>), dim3(cus), dim3(kApplyThreads), 0, s, k);
    return hipGetLastError();
  }
  if constexpr (L == 1) {
    if (fresh && k.A.log2c - k.bits <= kFreshBits) {
      hipLaunchKernelGGL((k_part_apply<L, VALS, false, true>), dim3(2 * cus), dim3(kApplyThreads), 0, s, k);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(k_part_rest, dim3(cus), dim3(256), 0, s, k);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_part_apply<L, VALS, false, false>), dim3(2 * cus), dim3(kApplyThreads), 0, s, k);
  return hipGetLastError();
}

struct Carved {
  size_t off, btot, hist, cur[2], tiles, items, istart, keys[2], vals[2], idx[2], total;
};

Carved carve(uint64_t n, uint32_t log2c, uint32_t layout, bool with_vals, bool with_flags, uint32_t nwg) {
  const uint32_t nb0 = 1u << kBits1, nb = 1u << bucket_bits(log2c);
  const size_t kb = layout == 0 ? 4 : 8;
  Carved o{};
  size_t at = 0;
  auto take = [&](size_t bytes) {
    const size_t p = at;
    at += round256(bytes);
    return p;
  };
  o.off = take(16);
  o.btot = take(((size_t)nb + 1) * 8);
  o.hist = take((size_t)nwg * nb * 4);
  o.cur[0] = take((size_t)nb0 * kPad * 4);
  o.cur[1] = take((size_t)nb * 4);
  o.tiles = take(((size_t)nb0 + 1) * 4);
  o.items = take(((size_t)nb + 1) * 4);
  // a bucket of c elements has ceil(c / kItemOps) items
  o.istart = take((n / kItemOps + nb + 2) * 8);
  for (int lv = 0; lv < 2; ++lv) {
    o.keys[lv] = take(n * kb);
    o.vals[lv] = take(with_vals ? n * kb : 0);
    o.idx[lv] = take(with_flags ? n * 4 : 0);
  }
  o.total = at;
  return o;
}

uint32_t count_wgs(uint64_t n) {
  const uint64_t w = (n + 4095) / 4096;
  return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(kCountWG, w));
}

}  // namespace

bool part_applies(uint64_t n, uint32_t log2c) {
  return n >= (1ull << 22) && n < (1ull << 32) - 1 && log2c >= 20;
}

size_t part_scratch_bytes(uint64_t n, uint32_t log2c, uint32_t layout, bool with_vals, bool with_flags,
                          uint32_t num_cus) {
  (void)num_cus;
  return carve(n, log2c, layout, with_vals, with_flags, count_wgs(n)).total;
}

hipError_t launch_upsert_add_part(const BulkArgs &a, bool fresh, void *scratch, uint32_t num_cus, hipStream_t s) {
  drop_stale_error();
  if (a.n == 0) return hipSuccess;
  if (!part_applies(a.n, a.log2c) || a.layout > 1 || !scratch || a.kinds) return hipErrorInvalidValue;
  PartK k{};
  k.A = a;
  k.nwg = count_wgs(a.n);
  k.chunk = (a.n + k.nwg - 1) / k.nwg;
  const Carved o = carve(a.n, a.log2c, a.layout, a.vals != nullptr, a.flags != nullptr, k.nwg);
  unsigned char *base = (unsigned char *)scratch;
  k.bits = bucket_bits(a.log2c);
  k.off = (uint32_t *)(base + o.off);
  k.next = k.off + 2;
  k.btot = (uint64_t *)(base + o.btot);
  k.hist = (uint32_t *)(base + o.hist);
  k.tiles = (uint32_t *)(base + o.tiles);
  k.items = (uint32_t *)(base + o.items);
  k.istart = (uint64_t *)(base + o.istart);
  for (int lv = 0; lv < 2; ++lv) {
    k.cur[lv] = (uint32_t *)(base + o.cur[lv]);
    k.keys[lv] = base + o.keys[lv];
    k.vals[lv] = a.vals ? (void *)(base + o.vals[lv]) : nullptr;
    k.idx[lv] = a.flags ? (uint32_t *)(base + o.idx[lv]) : nullptr;
  }
  hipError_t e;
  hipLaunchKernelGGL(k_part_zero, dim3(1), dim3(1024), 0, s, k);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (a.layout == 0)
    hipLaunchKernelGGL(k_part_count<0>, dim3(k.nwg), dim3(kCountThreads), 0, s, k);
  else
    hipLaunchKernelGGL(k_part_count<1>, dim3(k.nwg), dim3(kCountThreads), 0, s, k);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_part_sum, dim3((1u << k.bits) / 256, kSumSplit), dim3(256), 0, s, k);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_part_scan, dim3(1), dim3(1024), 0, s, k);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const bool vals = a.vals != nullptr, idx = a.flags != nullptr;
  if (a.layout == 0)
    e = vals ? (idx ? launch_scatters<0, true, true>(k, s) : launch_scatters<0, true, false>(k, s))
             : (idx ? launch_scatters<0, false, true>(k, s) : launch_scatters<0, false, false>(k, s));
  else
    e = vals ? (idx ? launch_scatters<1, true, true>(k, s) : launch_scatters<1, true, false>(k, s))
             : (idx ? launch_scatters<1, false, true>(k, s) : launch_scatters<1, false, false>(k, s));
  if (e != hipSuccess) return e;
  if (a.layout == 0)
    e = vals ? launch_apply<0, true>(k, fresh, num_cus, s) : launch_apply<0, false>(k, fresh, num_cus, s);
  else
    e = vals ? launch_apply<1, true>(k, fresh, num_cus, s) : launch_apply<1, false>(k, fresh, num_cus, s);
  return e;
}

}  // namespace lpht
