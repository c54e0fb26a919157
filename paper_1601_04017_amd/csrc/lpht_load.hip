// Region load: insertions (and insert-or-assigns) of large batches into a
// table that is nearly empty.
//
// One lane per operation is bound by the memory-side compare-and-swap (17.9 G/s
// on this card, wherever the addresses lie).  Loading a table touches nearly
// every line of it, so here the batch is first partitioned by table region
// (the position is the top log2 c bits of the hash, Sec. 5.3.1, so a region is a
// range of hashes; Sec. 5.5 orders bulk insertions the same way), and one
// workgroup then holds a region in LDS, inserts the region's operations by LDS
// compare-and-swap and writes the region once.
//
//   scatter   in tiles of 4096 operations: ranked inside their bucket by LDS
//             atomics, put in bucket order in LDS, written as runs behind one
//             reservation per bucket and tile.  One level of up to 512 buckets,
//             or two.  Buckets have a fixed room, the expected number of
//             operations and eight standard deviations, so nothing is counted
//             first; an operation that finds its bucket full (equal keys, an
//             uneven hash) is carried out on the table right there.
//   apply     one workgroup per region of 64 KiB.  A table without used cells is
//             not read, and its all-empty lines are not written.  A probe that
//             runs past the region's end is put off: the next region belongs to
//             another workgroup.
//   rest      the operations put off, one lane each on the table.
//
// Equal keys: all operations of a key find the same cells of the region taken
// (cells are never freed here), so one of them inserts and the others meet it,
// or all of them are put off, or are carried out on the table before the region
// is read.  Which of them inserts is open, as in any call.
// Flags: the first scatter writes 1 for every operation, and only the
// exceptions are written later (single bytes at random: the reason why calls
// that want flags stay with one lane per operation beyond kMaxFlagged).
// The batch is sampled first: where keys repeat (all but one operation of a key
// are lookups for a lane, and of a frequent key they fill their bucket and are
// carried out one by one), the first scatter carries its tiles out on the table,
// one lane per operation, and the other passes return at once.
// KV64, 10^8 distinct keys into an empty table of 2^28 cells: 5.84 -> 2.95 ms
// (scatters 0.89 and 0.96 ms, 3.5 TB/s; apply 1.07 ms, 5.5 TB/s); PACKED32, 2^20
// with flags into 2^21 cells: 69 -> 50 us.  Scatter and apply hash by sliced
// tables in LDS: with the lanes' direct hash (130 VALU instructions a key) they
// were bound by the VALU where the batch is small (a pass of 2^20 PACKED32
// insertions with flags and their finds: 102 -> 98 us; 3 * 10^6 KV64 inserted,
// assigned, found and erased: 652 -> 624 us).

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "lpht_device.h"
#include "lpht_lane_op.h"
#include "lpht_load.h"

namespace lpht {

namespace {

constexpr uint32_t kTile = 4096;
constexpr uint32_t kMaxBits = 9;             // buckets of one level: 512
constexpr uint32_t kImageBytes = 64 * 1024;  // a region in LDS: two workgroups per CU
constexpr uint32_t kApplyThreads = 1024;
constexpr uint32_t kPad = 32;                // first-level counters on lines of their own
constexpr uint64_t kMinOps = 1ull << 20;
constexpr uint64_t kMaxFlagged = 1ull << 23;
constexpr uint64_t kSampled = 1ull << 24;
// Workgroups of the apply at most, so that it returns soon where the sample says
// so (with their LDS, 65536 workgroups take 130 us to do nothing).
constexpr uint32_t kMostGroups = 8192;

// region cells: 8192 of 8 bytes, 4096 of 16
constexpr uint32_t region_bits(uint32_t layout) { return layout == 0 ? 13 : 12; }

template <int L>
using Elem = typename std::conditional<L == 0, u64, u64x2>::type;

template <int L>
__device__ __forceinline__ Elem<L> make_elem(u64 key, u64 val) {
  if constexpr (L == 0)
    return (val << 32) | key;
  else
    return u64x2{key, val};
}
template <int L>
__device__ __forceinline__ u64 elem_key(const Elem<L> &e) {
  if constexpr (L == 0)
    return e & 0xFFFFFFFFull;
  else
    return e.x;
}
template <int L>
__device__ __forceinline__ u64 elem_val(const Elem<L> &e) {
  if constexpr (L == 0)
    return e >> 32;
  else
    return e.y;
}

constexpr uint32_t kClasses = 4;  // of keys, each sampled by a workgroup of its own
struct LoadCtl {
  // by class, of the sampled keys: those equal to an earlier one, and the
  // distinct keys among them
  uint32_t repeats[kClasses], repeated[kClasses];
  uint32_t spilled;  // some operation was carried out on the table during a scatter
};

struct LoadK {
  BulkArgs A;
  LoadCtl *ctl;
  void *elem[2];     // by level: bucket b has room for cap[level] elements from b * cap[level]
  uint32_t *idx[2];  // their operations' indices (calls with flags)
  uint32_t *cnt[2];  // reserved so far (may exceed the room); the first level's padded
  uint32_t cap[2];
  uint16_t *put_off;   // by region (of the last level's room): elements for the rest pass
  uint32_t *n_put_off;
  uint32_t rbits, bits[2];  // cells of a region; buckets per level (bits[1] = 0: one level)
  uint32_t tiles2;          // tiles a first-level bucket may have
  uint32_t fresh;
  uint32_t per;             // keys each of a sampling workgroup's threads reads; 0: no sample
  uint32_t slots;           // of a sampling workgroup's table
  uint32_t most_repeats, most_repeated;  // in the sample of a batch that goes by region
};

// Whether keys repeat too often in the sample for the passes by region.
__device__ __forceinline__ bool repetitive(const LoadK &k) {
  if (k.per == 0) return false;
  uint32_t all = 0, keys = 0;
#pragma unroll
  for (uint32_t c = 0; c < kClasses; ++c) {
    all += k.ctl->repeats[c];
    keys += k.ctl->repeated[c];
  }
  return all > k.most_repeats || keys > k.most_repeated;
}

// First launch.  Workgroups [0, kClasses) of a sampled batch: the sample, 1024 * per keys in runs of
// 16 spread over the batch, of which each workgroup puts its class (two bits of a
// mix of the key) into a table in LDS; the others zero the counters.
constexpr uint32_t kSampleSlots = 1u << 15;  // 128 KiB for a quarter of at most 65536 keys
constexpr uint32_t kMostPer = 64;
constexpr uint32_t kReads = 16;  // in flight together
template <int L>
__global__ void __launch_bounds__(1024) k_load_begin(LoadK k, uint32_t n1, uint32_t n2) {
  __shared__ __attribute__((aligned(16))) uint32_t slot[kSampleSlots];  // 31 bits of the mix, and whether the key came again; 0: none
  __shared__ uint32_t s_repeats, s_repeated;
  const uint32_t first = k.per ? kClasses : 0;
  if (blockIdx.x >= first) {
    const uint32_t i = (blockIdx.x - first) * 1024 + threadIdx.x;
    if (i < n1) k.cnt[0][i] = 0;
    if (i < n2) k.cnt[1][i] = 0;
    if (i == 0) k.ctl->spilled = 0;
    return;
  }
  const u64 stride = k.A.n / (64 * k.per);  // between runs: 64 * per of them
  u64 key[kReads];
  auto read = [&](uint32_t j0) {
#pragma unroll
    for (uint32_t j = 0; j < kReads; ++j) {
      const uint32_t t = (j0 + j) * 1024 + threadIdx.x;
      key[j] = j0 + j < k.per ? word_in<L>(k.A.keys, (t >> 4) * stride + (t & 15)) : 0;
    }
  };
  read(0);
  for (uint32_t i = threadIdx.x; i < k.slots / 4; i += 1024) ((uint4 *)slot)[i] = uint4{0, 0, 0, 0};
  if (threadIdx.x == 0) s_repeats = s_repeated = 0;
  __syncthreads();
  uint32_t repeats = 0, repeated = 0;
  for (uint32_t j0 = 0; j0 < k.per;) {
#pragma unroll
    for (uint32_t j = 0; j < kReads; ++j) {
      const u64 z = key[j] * 0x9E3779B97F4A7C15ull;
      if (key[j] <= kTomb || (uint32_t)(z >> 62) != blockIdx.x) continue;
      const uint32_t tag = std::max(2u, (uint32_t)(z >> 16) & ~1u);
      uint32_t p = (uint32_t)(z >> 47) & (k.slots - 1);
      while (true) {
        const uint32_t old = atomicCAS(&slot[p], 0u, tag);
        if (old == 0) break;
        if ((old & ~1u) == tag) {
          ++repeats;
          if (!(old & 1u) && !(atomicOr(&slot[p], 1u) & 1u)) ++repeated;
          break;
        }
        p = (p + 1) & (k.slots - 1);
      }
    }
    j0 += kReads;
    if (j0 < k.per) read(j0);
  }
  if (repeats) atomicAdd(&s_repeats, repeats);
  if (repeated) atomicAdd(&s_repeated, repeated);
  __syncthreads();
  if (threadIdx.x == 0) {
    k.ctl->repeats[blockIdx.x] = s_repeats;
    k.ctl->repeated[blockIdx.x] = s_repeated;
  }
}

// KV64 with indices needs 94 KiB of LDS, so one workgroup per CU: of twice the
// wavefronts then.
template <int L, bool IDX>
constexpr uint32_t scatter_threads() { return L == 1 && IDX ? 1024 : 512; }

template <int L, int OP, bool IDX, int LV>
__global__ void __launch_bounds__((scatter_threads<L, IDX>()), 4) k_load_scatter(LoadK k) {
  constexpr uint32_t NT = scatter_threads<L, IDX>(), PER = kTile / NT;
  constexpr uint32_t NB = 1u << kMaxBits;
  __shared__ Elem<L> buf[kTile];
  __shared__ uint32_t ibuf[IDX ? kTile : 1];
  __shared__ uint16_t bkt[kTile];
  __shared__ uint32_t toff[NB];  // by bucket: elements, their start in the tile, then start in the room less that
  __shared__ uint32_t T[1024];
  __shared__ uint32_t s_w[NT / 64];
  const BulkArgs &A = k.A;
  const uint32_t nb = 1u << k.bits[LV], lane = threadIdx.x & 63;
  uint32_t err = 0;
  if (repetitive(k)) {
    if (LV == 1) return;
    uint32_t hits = 0;
    const u64 i0 = (u64)blockIdx.x * kTile + threadIdx.x;
    u64 next = i0 < A.n ? word_in<L>(A.keys, i0) : 0;
#pragma unroll 1
    for (uint32_t j = 0; j < PER; ++j) {
      const u64 i = i0 + j * NT, key = next;
      if (i + NT < A.n && j + 1 < PER) next = word_in<L>(A.keys, i + NT);
      uint8_t f = 0;
      if (i < A.n) {
        u64 none;
        if (key == kEmpty || key == kTomb) {
          f = 0xFE;
          err |= kErrReserved;
        } else {
          f = lane_op<L, OP, 0, 2>(A, key, A.vals ? word_in<L>(A.vals, i) : 1, none);
          if (f == 0xFF) err |= kErrFull;
        }
        if (IDX) A.flags[i] = f;
      }
      hits += (uint32_t)__popcll(__ballot(f == 1));
    }
    if (lane == 0) s_w[threadIdx.x >> 6] = hits;
    __syncthreads();
    if (threadIdx.x == 0) {
      u64 all = 0;
      for (uint32_t w = 0; w < NT / 64; ++w) all += s_w[w];
      CountSlot *cs = &A.status->slot[blockIdx.x % kCountSlots];
      if (all) {
        add64(&cs->used, all);
        add64(&cs->live, all);
      }
    }
    lane_errors(A.status, err);
    return;
  }
  crc_slices_load(T);
  // this workgroup's elements [base, base + m) of the batch, or of bucket b of
  // the first level (all tiles of a bucket have the same index modulo the number
  // of buckets, hence the same XCD, whose L2 joins their runs)
  u64 base;
  uint32_t m, b = 0;
  if (LV == 0) {
    base = (u64)blockIdx.x * kTile;
    m = (uint32_t)std::min<u64>(kTile, A.n - base);
  } else {
    b = blockIdx.x & ((1u << k.bits[0]) - 1);
    const uint32_t t = blockIdx.x >> k.bits[0];
    const uint32_t have = std::min(k.cnt[0][(u64)b * kPad], k.cap[0]);
    if ((u64)t * kTile >= have) return;
    base = (u64)b * k.cap[0] + (u64)t * kTile;
    m = std::min(kTile, have - t * kTile);
  }
  for (uint32_t i = threadIdx.x; i < nb; i += NT) toff[i] = 0;
  __syncthreads();
  Elem<L> e[PER];
  uint32_t ix[PER], at[PER];
  bool ok[PER];
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    const uint32_t t = j * NT + threadIdx.x;
    const u64 i = base + t;
    ok[j] = t < m;
    e[j] = Elem<L>{};
    ix[j] = 0;
    if (!ok[j]) continue;
    if (LV == 0) {
      const u64 key = word_in<L>(A.keys, i);
      e[j] = make_elem<L>(key, A.vals ? word_in<L>(A.vals, i) : 1);
      ix[j] = (uint32_t)i;
    } else {
      e[j] = ((const Elem<L> *)k.elem[0])[i];
      if (IDX) ix[j] = k.idx[0][i];
    }
  }
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    if (LV == 0 && ok[j]) {
      const u64 key = elem_key<L>(e[j]);
      if (key == kEmpty || key == kTomb) {
        ok[j] = false;
        err |= kErrReserved;
      }
      if (IDX) A.flags[ix[j]] = ok[j] ? 1 : 0xFE;
    }
    if (ok[j]) {
      const u64 pos = hash_sliced<L>(T, elem_key<L>(e[j]), A.crc_hi, A.crc_lo, A.mul) >> (64 - A.log2c);
      const uint32_t region = (uint32_t)(pos >> k.rbits);
      const uint32_t bk = LV == 0 ? region >> k.bits[1] : region & (nb - 1);
      at[j] = bk | (atomicAdd(&toff[bk], 1u) << 16);
    }
  }
  __syncthreads();
  uint32_t room_at = 0;
  {
    // where each bucket's elements begin in the tile, and in the bucket
    const uint32_t c = threadIdx.x < nb ? toff[threadIdx.x] : 0;
    uint32_t x = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if (lane >= (uint32_t)o) x += y;
    }
    if (lane == 63) s_w[threadIdx.x >> 6] = x;
    uint32_t g = 0;
    if (c) g = atomicAdd(LV == 0 ? &k.cnt[0][threadIdx.x * kPad] : &k.cnt[1][((u64)b << k.bits[1]) + threadIdx.x], c);
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t w = 0; w < (threadIdx.x >> 6); ++w) before += s_w[w];
    if (threadIdx.x < nb) toff[threadIdx.x] = before + x - c;
    room_at = g - (before + x - c);
  }
  __syncthreads();
  uint32_t total = 0;
  for (uint32_t w = 0; w < NT / 64; ++w) total += s_w[w];
#pragma unroll
  for (uint32_t j = 0; j < PER; ++j) {
    if (!ok[j]) continue;
    const uint32_t bk = at[j] & 0xFFFFu, p = toff[bk] + (at[j] >> 16);
    buf[p] = e[j];
    bkt[p] = (uint16_t)bk;
    if (IDX) ibuf[p] = ix[j];
  }
  __syncthreads();
  if (threadIdx.x < nb) toff[threadIdx.x] = room_at;
  __syncthreads();
  const uint32_t cap = k.cap[LV];
  uint32_t hits = 0;
  for (uint32_t i0 = 0; i0 < total; i0 += NT) {
    const uint32_t i = i0 + threadIdx.x;
    bool spill = false;
    if (i < total) {
      const uint32_t bk = bkt[i], q = toff[bk] + i;
      spill = q >= cap;
      if (!spill) {
        const u64 to = (((LV == 0 ? 0ull : (u64)b << k.bits[1]) + bk) * cap) + q;
        ((Elem<L> *)k.elem[LV])[to] = buf[i];
        if (IDX) k.idx[LV][to] = ibuf[i];
      }
    }
    if (__any(spill)) {
      uint8_t f = 0;
      if (spill) {
        u64 none;
        f = lane_op<L, OP, 0, 4>(A, elem_key<L>(buf[i]), elem_val<L>(buf[i]), none);
        if (f == 0xFF) err |= kErrFull;
        if (IDX) A.flags[ibuf[i]] = f;
        k.ctl->spilled = 1;
      }
      hits += (uint32_t)__popcll(__ballot(f == 1));
    }
  }
  if (lane == 0 && hits) {
    CountSlot *cs = &A.status->slot[blockIdx.x % kCountSlots];
    add64(&cs->used, hits);
    add64(&cs->live, hits);
  }
  lane_errors(A.status, err);
}

template <int L, int OP, bool IDX>
__global__ void __launch_bounds__(kApplyThreads) k_load_apply(LoadK k, uint32_t regions) {
  __shared__ __attribute__((aligned(16))) u64 img[kImageBytes / 8];  // the region's cells
  __shared__ uint32_t T[1024];
  __shared__ uint32_t s_hits, s_off;
  if (repetitive(k)) return;
  const BulkArgs &A = k.A;
  constexpr uint32_t R = 1u << region_bits(L);
  const int lv = k.bits[1] ? 1 : 0;
  const uint32_t cap = k.cap[lv];
  crc_slices_load(T);
  const bool fresh = k.fresh && !k.ctl->spilled;
  for (uint32_t r = blockIdx.x; r < regions; r += gridDim.x) {
    const uint32_t m = std::min(lv ? k.cnt[1][r] : k.cnt[0][(u64)r * kPad], cap);
    if (threadIdx.x == 0) {
      s_hits = 0;
      s_off = 0;
    }
    if (m == 0) {
      if (threadIdx.x == 0) k.n_put_off[r] = 0;
      continue;
    }
    u64x2 *cells = (u64x2 *)((unsigned char *)A.cells + (u64)r * kImageBytes);
    constexpr uint32_t N16 = kImageBytes / 16, PER = N16 / kApplyThreads;
    if (fresh) {
#pragma unroll
      for (uint32_t j = 0; j < PER; ++j) ((u64x2 *)img)[j * kApplyThreads + threadIdx.x] = u64x2{0, 0};
    } else {
      u64x2 c[PER];
#pragma unroll
      for (uint32_t j = 0; j < PER; ++j) c[j] = cells[j * kApplyThreads + threadIdx.x];
#pragma unroll
      for (uint32_t j = 0; j < PER; ++j) ((u64x2 *)img)[j * kApplyThreads + threadIdx.x] = c[j];
    }
    const Elem<L> *src = (const Elem<L> *)k.elem[lv] + (u64)r * cap;
    const uint32_t *sidx = IDX ? k.idx[lv] + (u64)r * cap : nullptr;
    uint32_t hits = 0;
    Elem<L> next = Elem<L>{};
    if (threadIdx.x < m) next = src[threadIdx.x];
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < m; i += kApplyThreads) {
      const Elem<L> e = next;
      if (i + kApplyThreads < m) next = src[i + kApplyThreads];
      const u64 key = elem_key<L>(e), val = elem_val<L>(e);
      uint32_t p = (uint32_t)(hash_sliced<L>(T, key, A.crc_hi, A.crc_lo, A.mul) >> (64 - A.log2c)) & (R - 1);
      while (true) {
        if (p == R) {
          k.put_off[(u64)r * cap + atomicAdd(&s_off, 1u)] = (uint16_t)i;
          break;
        }
        u64 *w = img + (L == 0 ? p : 2 * p);
        const u64 old = atomicCAS((unsigned long long *)w, 0ull,
                                  (unsigned long long)(L == 0 ? (val << 32) | key : key));
        if (old == 0) {
          if (L == 1) w[1] = val;
          ++hits;
          break;
        }
        if ((L == 0 ? old & 0xFFFFFFFFull : old) == key) {
          // present: insert leaves the value, insert-or-assign overwrites it
          if (OP == OP_UPSERT) {
            if (L == 0)
              ((uint32_t *)w)[1] = (uint32_t)val;
            else
              w[1] = val;
          }
          if (IDX) A.flags[sidx[i]] = 0;
          break;
        }
        ++p;
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) hits += __shfl_xor(hits, o, 64);
    if ((threadIdx.x & 63) == 0 && hits) atomicAdd(&s_hits, hits);
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
      const u64x2 c = ((const u64x2 *)img)[j * kApplyThreads + threadIdx.x];
      // eight lanes hold a line; in a table that was empty a line of empty
      // cells is what is there
      const u64 any = __ballot(c.x != 0 || (L == 0 && c.y != 0));
      if (!fresh || ((any >> (threadIdx.x & 56u)) & 0xFFull))
        __builtin_nontemporal_store(c, cells + j * kApplyThreads + threadIdx.x);
    }
    if (threadIdx.x == 0) {
      k.n_put_off[r] = s_off;
      CountSlot *cs = &A.status->slot[r % kCountSlots];
      if (s_hits) {
        add64(&cs->used, s_hits);
        add64(&cs->live, s_hits);
      }
    }
    __syncthreads();  // the next region's counts and cells take the place of these
  }
}

// A wavefront per region.
template <int L, int OP, bool IDX>
__global__ void __launch_bounds__(256) k_load_rest(LoadK k, uint32_t regions) {
  if (repetitive(k)) return;
  const BulkArgs &A = k.A;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= regions) return;
  const int lv = k.bits[1] ? 1 : 0;
  const uint32_t off = k.n_put_off[r];
  const u64 at = (u64)r * k.cap[lv];
  uint32_t hits = 0, err = 0;
  for (uint32_t i0 = 0; i0 < off; i0 += 64) {
    uint8_t f = 0;
    if (i0 + lane < off) {
      const u64 i = at + k.put_off[at + i0 + lane];
      const Elem<L> e = ((const Elem<L> *)k.elem[lv])[i];
      u64 none;
      f = lane_op<L, OP, 0, 4>(A, elem_key<L>(e), elem_val<L>(e), none);
      if (f == 0xFF) err |= kErrFull;
      if (IDX && f != 1) A.flags[k.idx[lv][i]] = f;
    }
    hits += (uint32_t)__popcll(__ballot(f == 1));
  }
  if (lane == 0 && hits) {
    CountSlot *cs = &A.status->slot[r % kCountSlots];
    add64(&cs->used, hits);
    add64(&cs->live, hits);
  }
  lane_errors(A.status, err);
}

struct Plan {
  uint32_t rbits, bits[2], cap[2], tiles2;
  uint32_t regions;
  size_t ctl, cnt[2], n_put_off, put_off, elem[2], idx[2], total;
  bool ok;
};

size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

// Room of a bucket that takes 2^-bits of n operations: eight standard
// deviations above the mean, in whole lines.
uint64_t room(uint64_t n, uint32_t bits) {
  const double mean = std::ldexp((double)n, -(int)bits);
  return ((uint64_t)(mean + 8.0 * std::sqrt(mean)) + 64) & ~15ull;
}

Plan plan_of(uint64_t n, uint32_t log2c, uint32_t layout, bool with_flags) {
  Plan p{};
  p.rbits = region_bits(layout);
  const uint32_t bits = log2c > p.rbits ? log2c - p.rbits : 0;
  p.bits[0] = bits <= kMaxBits ? bits : (bits + 1) / 2;
  p.bits[1] = bits - p.bits[0];
  p.regions = 1u << bits;
  const uint64_t c0 = room(n, p.bits[0]), c1 = p.bits[1] ? room(n, bits) : 0;
  const uint64_t last = p.bits[1] ? c1 : c0;
  p.ok = bits >= 4 && p.bits[0] <= kMaxBits && p.bits[1] <= kMaxBits && c0 < (1ull << 31) && last < (1u << 16);  // put_off has 16 bits
  if (!p.ok) return p;
  p.cap[0] = (uint32_t)c0;
  p.cap[1] = (uint32_t)c1;
  p.tiles2 = (uint32_t)((c0 + kTile - 1) / kTile);
  const size_t eb = layout == 0 ? 8 : 16;
  size_t at = 0;
  auto take = [&](size_t bytes) {
    const size_t here = at;
    at += round256(bytes);
    return here;
  };
  p.ctl = take(sizeof(LoadCtl));
  p.cnt[0] = take(((size_t)kPad << p.bits[0]) * 4);
  p.cnt[1] = take((size_t)p.regions * 4);
  p.n_put_off = take((size_t)p.regions * 4);
  p.put_off = take((size_t)p.regions * last * 2);
  for (int lv = 0; lv < 2; ++lv) {
    const size_t els = lv == 0 ? (size_t)c0 << p.bits[0] : (size_t)c1 * (p.bits[1] ? p.regions : 0);
    p.elem[lv] = take(els * eb);
    p.idx[lv] = take(with_flags ? els * 4 : 0);
  }
  p.total = at;
  return p;
}

template <int L, int OP, bool IDX>
hipError_t enqueue(const LoadK &k, const Plan &p, hipStream_t s) {
  const uint32_t n1 = kPad << p.bits[0], n2 = p.bits[1] ? p.regions : 0;
  hipLaunchKernelGGL((k_load_begin<L>), dim3((k.per ? kClasses : 0) + (std::max(n1, n2) + 1023) / 1024), dim3(1024), 0, s, k, n1, n2);
  constexpr uint32_t nt = scatter_threads<L, IDX>();
  hipLaunchKernelGGL((k_load_scatter<L, OP, IDX, 0>), dim3((uint32_t)((k.A.n + kTile - 1) / kTile)), dim3(nt), 0, s, k);
  if (p.bits[1])
    hipLaunchKernelGGL((k_load_scatter<L, OP, IDX, 1>), dim3(p.tiles2 << p.bits[0]), dim3(nt), 0, s, k);
  hipLaunchKernelGGL((k_load_apply<L, OP, IDX>), dim3(std::min(p.regions, kMostGroups)), dim3(kApplyThreads), 0, s, k,
                     p.regions);
  hipLaunchKernelGGL((k_load_rest<L, OP, IDX>), dim3((p.regions + 3) / 4), dim3(256), 0, s, k, p.regions);
  return hipGetLastError();
}

// What the sample may show of a batch that goes by region.  Of keys that come r
// times each in the mean, m sampled keys hold m^2 r / 2n pairs of equal ones, and
// m is chosen for 8 pairs per unit of r (fewer beyond 2^28 operations).  r is
// where one lane per operation becomes as fast: the more bytes of cells there are
// per operation the sooner, later for insert-or-assigns, whose repeats each write,
// and sooner with flags, which the region passes write singly for repeats.  KV64,
// lanes / by region, us:
//   r                                     1          2          4          8         32
//   2^22 insertions, 2^23 cells     297/140    171/121    137/118    114/147     89/148
//     with flags                    301/167    173/167    137/169    117/213     90/215
//     insert-or-assigns             296/146    222/122    194/122    167/146    149/148
//   10^8 insertions, 2^28 cells   5764/2890  4100/2709  3460/3824  2734/3841  2057/3857
//     insert-or-assigns           5765/2938  5239/2750  4984/3826  4614/3815  3350/3872
// One frequent key is told by its share instead: it costs the lanes nothing, and
// the scatter a bucket that is full.  Where the sample sends a batch to the lanes,
// it and the passes that return cost them 20 us of 50 at 2^22 operations, 60 of
// 1500 at 10^8.  Below kSampled bytes of elements there is no sample: of PACKED32
// calls of 2^20 operations it would take 3 us of 55, and save 3 to 10 of 48.
void sample_rule(LoadK &k, OpKind op, uint64_t c) {
  const uint64_t cell = k.A.layout == 0 ? 8 : 16;
  if (k.A.n * cell < kSampled) return;
  const double n = (double)k.A.n, bytes = (double)(cell * c) / n;
  k.per = std::min<uint32_t>(kMostPer, (uint32_t)std::ceil(std::sqrt(16.0 * n) / 1024.0));
  k.slots = 1024;  // at least twice a class's share
  while (k.slots < kSampleSlots && k.slots < 1024 * k.per) k.slots *= 2;
  struct Rule {
    double bytes, least, most;
  };
  const Rule rule = op == OP_INSERT ? (k.A.flags ? Rule{70, 2.5, 4} : Rule{140, 3.3, 8})
                                    : (k.A.flags ? Rule{200, 5, 12} : Rule{600, 5, 40});
  const double r = std::min(rule.most, std::max(rule.least, rule.bytes / bytes));
  const double m = 1024.0 * k.per, pairs = m * m / (2.0 * n) * r;
  k.most_repeated = (uint32_t)std::max(12.0, pairs);
  k.most_repeats = k.most_repeated + (uint32_t)(m / 80.0);
}

}  // namespace

// Where the line lies (one lane per operation against this, us, the faster
// last; both sides of the rule, distinct keys):
//   KV64, 2^26 operations, empty table: c = 8 n 3844 / 2819, c = 4 n 3815 / 2109;
//     2^24: c = 16 n 1.02 times as fast, 32 n 0.71;
//   with n / 4 to n cells used before: c = 4 n 1.25 to 1.36 times, 8 n 0.78;
//   flags, empty: c = 4 n 1.19 to 1.42 times, 8 n 0.97;
//   2^20 operations, empty: c = 4 n 1.26 times (flags 1.09), 8 n 1.10 (0.93);
//   2^19: 1.12 to 0.8 (0.99 to 0.75), too few for its launches;
//   PACKED32, whose cells cost half: 2^22 operations, empty: c = 16 n 1.29 times,
//     32 n 1.08; used before: c = 8 n 1.13, 16 n 0.75.
// So the bytes of cells written (and read, unless empty) per operation decide,
// half as many below 2^21 operations.
bool load_applies(uint64_t n, uint32_t log2c, uint32_t layout, uint64_t used0, bool with_flags) {
  if (n < kMinOps || n >= (1ull << 31) || log2c > 34) return false;
  if (with_flags && n > kMaxFlagged) return false;
  const uint64_t c = 1ull << log2c;
  // at most 3/4 full afterwards, so that few probes leave their region
  if (used0 + n > c / 4 * 3) return false;
  // the batch may hold many keys of a table with more, and a present key costs
  // a lane no more than a lookup (3 * 10^6 insert-or-assigns with flags, half of
  // them present, on 3 * 10^6 of 2^23 cells: 187 us by lanes, 205 here)
  if (used0 > n / 2) return false;
  const uint64_t per_op = (used0 == 0 && !with_flags ? 128 : 64) / (n < 2 * kMinOps ? 2 : 1);
  if ((layout == 0 ? 8 : 16) * c > per_op * n) return false;
  return plan_of(n, log2c, layout, with_flags).ok;
}

size_t load_scratch_bytes(uint64_t n, uint32_t log2c, uint32_t layout, bool with_flags) {
  return plan_of(n, log2c, layout, with_flags).total;
}

hipError_t launch_load(OpKind op, const BulkArgs &a, bool fresh, void *scratch, hipStream_t s) {
  drop_stale_error();
  if ((op != OP_INSERT && !(op == OP_UPSERT && a.up == 0)) || a.kinds || !scratch || a.layout > 1)
    return hipErrorInvalidValue;
  const Plan p = plan_of(a.n, a.log2c, a.layout, a.flags != nullptr);
  if (!p.ok) return hipErrorInvalidValue;
  unsigned char *base = (unsigned char *)scratch;
  LoadK k{};
  k.A = a;
  k.ctl = (LoadCtl *)(base + p.ctl);
  k.n_put_off = (uint32_t *)(base + p.n_put_off);
  k.put_off = (uint16_t *)(base + p.put_off);
  for (int lv = 0; lv < 2; ++lv) {
    k.elem[lv] = base + p.elem[lv];
    k.idx[lv] = (uint32_t *)(base + p.idx[lv]);
    k.cnt[lv] = (uint32_t *)(base + p.cnt[lv]);
    k.cap[lv] = p.cap[lv];
    k.bits[lv] = p.bits[lv];
  }
  k.rbits = p.rbits;
  k.tiles2 = p.tiles2;
  k.fresh = fresh ? 1 : 0;
  sample_rule(k, op, 1ull << a.log2c);
  const bool f = a.flags != nullptr, up = op == OP_UPSERT;
  if (a.layout == 0)
    return up ? (f ? enqueue<0, OP_UPSERT, true>(k, p, s) : enqueue<0, OP_UPSERT, false>(k, p, s))
              : (f ? enqueue<0, OP_INSERT, true>(k, p, s) : enqueue<0, OP_INSERT, false>(k, p, s));
  return up ? (f ? enqueue<1, OP_UPSERT, true>(k, p, s) : enqueue<1, OP_UPSERT, false>(k, p, s))
            : (f ? enqueue<1, OP_INSERT, true>(k, p, s) : enqueue<1, OP_INSERT, false>(k, p, s));
}

}  // namespace lpht
