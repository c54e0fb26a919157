// String keys of liblpht (Sec. 5.7, "Complex Keys").
//
// The table stores references to keys held in a byte pool that the table
// manages.  A cell is two words: the reference word, (signature << 48) |
// pool offset, and the value.  The signature is the low 16 bits of the
// key's 64-bit hash, bits the position (the top log2 c bits) does not use,
// kept in bits of the reference a 48-bit offset leaves free; a probe
// compares signatures first and follows the reference only when they agree.
// Reference words 0 and 1 are the empty cell and the tombstone; pool offsets
// start at 8, so no reference is 0 or 1.
//
// A pool record is a 32-bit length followed by the bytes, rounded up to 8
// bytes.  Records are allocated by bumping a device cursor.  An inserting call
// takes two launches.  The first inserts every absent key by compare-and-swap as
// a claim, a reference to the operation, whose key is read from the call's own
// bytes: equal keys of the call meet it there.  Each claim gets a record, whose
// reference the second puts in the claim's place.  So no operation fences to make
// a record visible (an agent-scope release writes back the XCD's L2), and the
// pool takes one record per inserted key.  Records of erased keys stay in the
// pool until the next migration, which copies only live keys into a new pool (the
// paper reclaims key space when the array is migrated).
//
// The hash is the pair of CRC-32C register updates over the key's bytes with
// the two seeds (Sec. 8.3), the same function as for word keys.

#include <hip/hip_runtime.h>

#include "lpht_device.h"
#include "lpht_str.h"

namespace lpht {

namespace {

constexpr u64 kOffMask = (1ull << 48) - 1;

__device__ __forceinline__ uint32_t crc_byte(const uint32_t (*T)[256], uint32_t r, uint32_t b) {
  return (r >> 8) ^ T[0][(r ^ b) & 0xFFu];
}

// 8 bytes at any alignment (one or two wide loads; never past p + 7).
__device__ __forceinline__ u64 ld8(const uint8_t *p) {
  u64 x;
  __builtin_memcpy(&x, p, 8);
  return x;
}

__device__ __forceinline__ void st8(uint8_t *p, u64 x) { __builtin_memcpy(p, &x, 8); }

// 64-bit hash of bytes s[0..len) (global memory, any alignment).  Eight
// bytes at a time: with the register XORed into their low word, the
// register after them is CRC(0, chunk) (the slicing tables); then the tail
// byte by byte.
__device__ __forceinline__ u64 str_hash(const uint32_t (*T)[256], const uint8_t *s, u64 len, uint32_t seed_hi,
                                        uint32_t seed_lo) {
  uint32_t hi = seed_hi, lo = seed_lo;
  u64 i = 0;
  for (; i + 8 <= len; i += 8) {
    const u64 x = ld8(s + i);
    hi = crc0_u64(T, x ^ hi);
    lo = crc0_u64(T, x ^ lo);
  }
  for (; i < len; ++i) {
    const uint32_t b = s[i];
    hi = crc_byte(T, hi, b);
    lo = crc_byte(T, lo, b);
  }
  return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ u64 rec_bytes(u64 len) { return (4 + len + 7) & ~7ull; }

// Writes the record of s[0..len) at pool offset off (8-aligned).
__device__ __forceinline__ void rec_write(uint8_t *pool, u64 off, const uint8_t *s, u64 len) {
  *(uint32_t *)(pool + off) = (uint32_t)len;
  uint8_t *r = pool + off + 4;
  u64 i = 0;
  for (; i + 8 <= len; i += 8) st8(r + i, ld8(s + i));
  for (; i < len; ++i) r[i] = s[i];
}

// A cell: reference and value.  Plain loads: within a launch a cell only goes
// from empty to a claim (insertions) or from a reference to the tombstone
// (erases), each by compare-and-swap, and a probe that read the cell before
// learns so from its own compare-and-swap.
__device__ __forceinline__ u64x2 ld_cell(const void *cells, u64 p) { return ((const u64x2 *)cells)[p]; }

// Marks a claim among the references: the low 47 bits are the operation's index.
constexpr u64 kClaim = 1ull << 47;

__device__ __forceinline__ bool bytes_equal(const uint8_t *a, const uint8_t *b, u64 len) {
  u64 i = 0;
  for (; i + 8 <= len; i += 8)
    if (ld8(a + i) != ld8(b + i)) return false;
  for (; i < len; ++i)
    if (a[i] != b[i]) return false;
  return true;
}

// Whether the cell's reference word r names the key s[0..len).  Every record
// that a reference names was written by an earlier launch.
template <bool CLAIMS>
__device__ __forceinline__ bool same_key(const StrArgs &a, u64 r, u64 sig, const uint8_t *s, u64 len) {
  if (r == kTomb || (r >> 48) != sig) return false;
  if (CLAIMS && (r & kClaim)) {
    const u64 i = r & (kClaim - 1), o = a.offsets[i];
    return a.offsets[i + 1] - o == len && bytes_equal(a.bytes + o, s, len);
  }
  const uint8_t *rec = a.pool + (r & kOffMask);
  return *(const uint32_t *)rec == (uint32_t)len && bytes_equal(rec + 4, s, len);
}

// Exclusive prefix sum of v over the wavefront's 64 lanes (all active);
// `total` receives the sum.
__device__ __forceinline__ u64 wave_excl_scan(u64 v, u64 &total) {
  const int lane = threadIdx.x & 63;
  u64 x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const u64 y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  total = __shfl(x, 63, 64);
  return x - v;
}

// Looks a key up: the cell that holds it, if any.
struct StrProbe {
  u64 p, r, v;  // r, v: the cell's words
  bool found;
};
__device__ __forceinline__ StrProbe str_probe(const StrArgs &a, const uint32_t (*T)[256], const uint8_t *s, u64 len) {
  const u64 mask = (1ull << a.log2c) - 1, h = str_hash(T, s, len, a.crc_hi, a.crc_lo), sig = h & 0xFFFFull;
  StrProbe q{h >> (64 - a.log2c), kEmpty, 0, false};
  for (u64 step = 0; step <= mask; ++step, q.p = (q.p + 1) & mask) {
    const u64x2 c = ld_cell(a.cells, q.p);
    q.r = c.x;
    q.v = c.y;
    if (q.r == kEmpty) break;
    if (same_key<false>(a, q.r, sig, s, len)) {
      q.found = true;
      break;
    }
  }
  return q;
}

// The value of the present key in cell p.
template <int KIND>
__device__ __forceinline__ void str_update(const StrArgs &a, u64 p, u64 d) {
  if (KIND != kStrUpsert) return;
  u64 *v = (u64 *)a.cells + 2 * p + 1;
  if (a.up == 0)
    __hip_atomic_store(v, d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    add64(v, d);
}

// Finds and erases, one lane each.
template <int KIND>
__global__ void __launch_bounds__(256) k_str_op(StrArgs a) {
  __shared__ uint32_t T[8][256];
  crc_tables_build(T);
  u64 *cells = (u64 *)a.cells;
  const u64 stride = (u64)gridDim.x * blockDim.x;
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += stride) {
    const u64 o0 = a.offsets[i];
    const StrProbe q = str_probe(a, T, a.bytes + o0, a.offsets[i + 1] - o0);
    uint8_t flag = 0;
    u64 out = 0;
    if (q.found) {
      if (KIND == kStrFind) {
        out = q.v;
        flag = 1;
      } else {
        flag = cas64(cells + 2 * q.p, q.r, kTomb) == q.r ? 1 : 0;
      }
    }
    if (a.flags) a.flags[i] = flag;
    if (KIND == kStrFind && a.vals_out) a.vals_out[i] = out;
  }
}

// What the first launch of an inserting call leaves for the second: the
// reference of the record (0: nothing was claimed) and the cell claimed for it.
typedef u64x2 Staged;

// First launch, one lane per operation: absent keys are claimed and their
// records written, present ones updated.  One addition to the pool's cursor per
// workgroup (of 1024: every addition is 12 ns on the one line, 2 * 10^6 operations
// by wavefronts would be 375 us).
//
// Bound: random lines (cell, and record or key for hits) and the latency of each
// key's chain of loads, which one operation per lane and full occupancy hide:
// eight operations per lane, one after the other, with one fence per wavefront
// took 502 us for 2 * 10^6 keys of 8 to 40 bytes in 2^23 cells, the two launches
// 307 us.
template <int KIND>
__global__ void __launch_bounds__(1024, 8) k_str_claim(StrArgs a, Staged *staged) {
  __shared__ uint32_t T[8][256];
  __shared__ u64 s_w[16];
  crc_tables_build(T);
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const u64 mask = (1ull << a.log2c) - 1;
  u64 *cells = (u64 *)a.cells;
  const u64 stride = (u64)gridDim.x * blockDim.x;
  uint32_t err = 0;
  // the bound is uniform over the workgroup, which allocates together
  for (u64 i0 = (u64)blockIdx.x * blockDim.x; i0 < a.n; i0 += stride) {
    const u64 i = i0 + threadIdx.x;
    const uint8_t *s = nullptr;
    u64 len = 0, need = 0, p = 0, sig = 0;
    uint8_t flag = 0xFF;
    if (i < a.n) {
      const u64 o0 = a.offsets[i];
      len = a.offsets[i + 1] - o0;
      s = a.bytes + o0;
      const u64 h = str_hash(T, s, len, a.crc_hi, a.crc_lo);
      sig = h & 0xFFFFull;
      p = h >> (64 - a.log2c);
      for (u64 step = 0; step <= mask; ++step, p = (p + 1) & mask) {
        u64 r = ld_cell(a.cells, p).x;
        if (r == kEmpty) {
          r = cas64(cells + 2 * p, kEmpty, (sig << 48) | kClaim | i);
          if (r == kEmpty) {
            // the value, 0 until now; concurrent insert-or-adds of the key also add
            const u64 d = a.vals ? a.vals[i] : 1;
            if (KIND == kStrInsert || a.up == 0)
              __hip_atomic_store(cells + 2 * p + 1, d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else
              add64(cells + 2 * p + 1, d);
            need = rec_bytes(len);
            flag = 1;
            break;
          }
        }
        if (same_key<true>(a, r, sig, s, len)) {
          str_update<KIND>(a, p, a.vals ? a.vals[i] : 1);
          flag = 0;
          break;
        }
      }
    }
    u64 total;
    u64 off = wave_excl_scan(need, total);
    if (lane == 0) s_w[wave] = total;
    __syncthreads();
    if (threadIdx.x == 0) {
      u64 sum = 0;
      for (uint32_t w = 0; w < 16; ++w) {
        const u64 t = s_w[w];
        s_w[w] = sum;
        sum += t;
      }
      const u64 base = sum ? atomicAdd((unsigned long long *)&a.ctl->pool_used, (unsigned long long)sum) : 0;
      for (uint32_t w = 0; w < 16; ++w) s_w[w] += base;
    }
    __syncthreads();
    off += s_w[wave];
    __syncthreads();  // read before the next round writes it
    if (i >= a.n) continue;
    Staged out = {0, p};
    if (need && off + need <= a.pool_cap) {
      rec_write(a.pool, off, s, len);
      out.x = (sig << 48) | off;
    } else if (need) {
      out.x = kTomb;  // no room in the pool: the claim becomes a tombstone
      flag = 0xFF;
    }
    if (flag == 0xFF) err |= kErrFull;  // no cell, or no room in the pool
    staged[i] = out;
    if (a.flags) a.flags[i] = flag;
  }
  if (err) atomicOr(&a.ctl->err, err);
}

// Second launch: the records' references in the claims' place.
__global__ void __launch_bounds__(256) k_str_publish(StrArgs a, const Staged *staged) {
  const u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const Staged st = staged[i];
  if (st.x) ((u64 *)a.cells)[2 * st.y] = st.x;
}

// Migration: every live key of the old table is copied into the new pool
// (one allocation per wavefront) and inserted into the new (zeroed) table
// with compare-and-swap.
__global__ void __launch_bounds__(256) k_str_migrate(StrMigArgs a) {
  __shared__ uint32_t T[8][256];
  crc_tables_build(T);
  const u64 oc = 1ull << a.log2_old, nmask = (1ull << a.log2_new) - 1;
  const u64 stride = (u64)gridDim.x * blockDim.x;
  uint32_t err = 0;
  for (u64 i0 = (u64)blockIdx.x * blockDim.x; i0 < oc; i0 += stride) {
    const u64 i = i0 + threadIdx.x;
    const u64 r = i < oc ? a.old_cells[2 * i] : kEmpty;
    const bool live = r != kEmpty && r != kTomb;
    const u64 off = r & kOffMask;
    const u64 len = live ? *(const uint32_t *)(a.old_pool + off) : 0;
    const u64 need = live ? rec_bytes(len) : 0;
    u64 total;
    const u64 pre = wave_excl_scan(need, total);
    u64 base = 0;
    if ((threadIdx.x & 63) == 0 && total)
      base = atomicAdd((unsigned long long *)&a.ctl->pool_used, (unsigned long long)total);
    base = __shfl(base, 0, 64);
    if (!live) continue;
    const u64 noff = base + pre;
    if (noff + need > a.new_pool_cap) {
      err |= kErrFull;
      continue;
    }
    const uint8_t *s = a.old_pool + off + 4;
    const u64 h = str_hash(T, s, len, a.crc_hi, a.crc_lo);
    // records are 8-byte aligned: copy whole words
    for (u64 q = 0; q < need; q += 8) *(u64 *)(a.new_pool + noff + q) = *(const u64 *)(a.old_pool + off + q);
    const u64 ref = ((h & 0xFFFFull) << 48) | noff;
    u64 p = h >> (64 - a.log2_new);
    for (u64 step = 0; step <= nmask; ++step, p = (p + 1) & nmask) {
      if (cas64((u64 *)a.new_cells + 2 * p, kEmpty, ref) == kEmpty) {
        a.new_cells[2 * p + 1] = a.old_cells[2 * i + 1];
        break;
      }
    }
  }
  if (err) atomicOr(&a.ctl->err, err);
}

__global__ void __launch_bounds__(256) k_str_recount(const u64 *cells, u64 cap, StrCtl *ctl) {
  const u64 stride = (u64)gridDim.x * blockDim.x;
  long long u = 0, l = 0;
  for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < cap; i += stride) {
    const u64 r = cells[2 * i];
    u += r != kEmpty;
    l += r != kEmpty && r != kTomb;
  }
  u = wave_sum(u);
  l = wave_sum(l);
  if ((threadIdx.x & 63) == 0) {
    if (u) add64(&ctl->used, (u64)u);
    if (l) add64(&ctl->live, (u64)l);
  }
}

__global__ void k_str_ctl(StrCtl *ctl, u64 pool_used, int keep_pool) {
  if (threadIdx.x == 0) {
    ctl->used = 0;
    ctl->live = 0;
    if (!keep_pool) ctl->pool_used = pool_used;
  }
}

uint32_t grid_of(u64 items, uint32_t num_cus) {
  u64 b = (items + 255) / 256;
  const u64 cap = (u64)(num_cus ? num_cus : 1) * 8;
  if (b > cap) b = cap;
  return (uint32_t)(b ? b : 1);
}

}  // namespace

hipError_t launch_str_op(int kind, const StrArgs &a, uint32_t num_cus, hipStream_t s) {
  drop_stale_error();
  const uint32_t g = grid_of(a.n, num_cus);
  switch (kind) {
    case kStrFind: hipLaunchKernelGGL(k_str_op<kStrFind>, dim3(g), dim3(256), 0, s, a); break;
    case kStrErase: hipLaunchKernelGGL(k_str_op<kStrErase>, dim3(g), dim3(256), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_str_insert(int kind, const StrArgs &all, uint64_t slice, void *scratch, uint32_t num_cus, hipStream_t s) {
  drop_stale_error();
  if (kind != kStrInsert && kind != kStrUpsert) return hipErrorInvalidValue;
  if (slice == 0) return hipErrorInvalidValue;
  for (u64 lo = 0; lo < all.n; lo += slice) {
    StrArgs a = all;
    a.n = all.n - lo < slice ? all.n - lo : slice;
    a.offsets = all.offsets + lo;
    a.vals = all.vals ? all.vals + lo : nullptr;
    a.flags = all.flags ? all.flags + lo : nullptr;
    const u64 want = (a.n + 1023) / 1024, most = 2ull * (num_cus ? num_cus : 1);
    const uint32_t grid = (uint32_t)(want < most ? want : most);
    Staged *st = (Staged *)scratch;
    if (kind == kStrInsert)
      hipLaunchKernelGGL(k_str_claim<kStrInsert>, dim3(grid), dim3(1024), 0, s, a, st);
    else
      hipLaunchKernelGGL(k_str_claim<kStrUpsert>, dim3(grid), dim3(1024), 0, s, a, st);
    hipLaunchKernelGGL(k_str_publish, dim3((uint32_t)((a.n + 255) / 256)), dim3(256), 0, s, a, (const Staged *)st);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_str_migrate(const StrMigArgs &a, uint32_t num_cus, hipStream_t s) {
  drop_stale_error();
  hipLaunchKernelGGL(k_str_ctl, dim3(1), dim3(64), 0, s, a.ctl, (u64)8, 0);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_str_migrate, dim3(grid_of(1ull << a.log2_old, num_cus)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_str_recount(const void *cells, uint32_t log2c, StrCtl *ctl, uint32_t num_cus, hipStream_t s) {
  drop_stale_error();
  hipLaunchKernelGGL(k_str_ctl, dim3(1), dim3(64), 0, s, ctl, (u64)0, 1);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_str_recount, dim3(grid_of(1ull << log2c, num_cus)), dim3(256), 0, s, (const u64 *)cells,
                     1ull << log2c, ctl);
  return hipGetLastError();
}

hipError_t launch_str_init(StrCtl *ctl, hipStream_t s) {
  drop_stale_error();
  hipLaunchKernelGGL(k_str_ctl, dim3(1), dim3(64), 0, s, ctl, (u64)8, 0);
  return hipGetLastError();
}

}  // namespace lpht
