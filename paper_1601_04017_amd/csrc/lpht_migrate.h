// Block-parallel cluster migration (Sec. 5.3.1, Lemma 1) by one wavefront
// per block of old cells, shared by the migration kernel (lpht_kernels.hip)
// and the insertion kernel that grows the table while it runs
// (lpht_async.hip).
//
// A wavefront owns old block [d, d + B) and the new range [g d, g (d + B))
// (g = gamma, 1 or 2).  It loads the window [d - H, d + B + H) of old cells
// (H = MIG_HALO) lane-consecutively into registers (the caller prefetches the
// next block's window before working on the current one) and then
//   - stores the window's cells in LDS;
//   - finds the empty cells with ballots, hence the window range [lo, hi) of
//     the clusters that overlap the block, and hashes the keys in it;
//   - places all their elements at once into an image of the new range that
//     holds indices into the window (below);
//   - streams the owned part of the image out as whole cells.
// Elements of the last cluster that land past the owned range are written by
// the next block's wavefront, which sees that cluster as its incoming one; the
// first block's incoming cluster is the one that wraps around the table end.
// Positions are kept unwrapped (old cell x may be negative for block 0).  A
// cluster longer than the halo (or a table without empty cells) sets
// `overflow`; the caller then redoes the whole move another way.
//
// Placement.  Re-inserting a cluster in old-array order gives every element
// the first cell from its home on that no earlier element has.  That is the
// one matching in which every cell prefers the earliest of the elements that
// reach it, and deferred acceptance finds it with the elements proposing in any
// order: an element asks for its home, a cell keeps the smaller index
// (atomic minimum on the image), and whoever is turned away or pushed out asks
// the next cell.  So all lanes place their elements side by side, about 1.3
// LDS atomics each, where one lane per cluster walked it in order (the longest
// of 64 clusters of a block held the wavefront, and with 8 to 10 wavefronts
// per CU nothing hid it).  Elements that do not get their home go on a list that
// the lanes work off without waiting for one another.  KV64 at fill 1/2, blocks
// of 512: doubling 2^26 cells 1.21 -> 0.74 ms (4.3 TB/s), the same size 0.96 ->
// 0.65; blocks of 256: 0.94 -> 0.76 and 0.84 -> 0.52.  (Kept in registers, one
// row of the window after the other: 0.74 and 1.08; all rows in step: 0.97 and
// 1.74, every step issuing an atomic per row for a few lanes.)
#pragma once

#include <type_traits>

#include "lpht_device.h"

namespace lpht {

constexpr int MIG_HALO = 128;
constexpr uint32_t kImgEmpty = 0xFFFFFFFFu;

__host__ __device__ constexpr uint32_t mig_window(uint32_t mb) { return mb + 2 * MIG_HALO; }

// LDS of one wavefront: the window's cells, the image (u32 per new cell) and
// the list of elements still asking (u32, half the window's cells).
__host__ __device__ constexpr size_t mig_wave_lds(uint32_t mb, uint32_t layout, uint32_t gamma) {
  return ((size_t)mig_window(mb) * ((layout == 0 ? 8u : 16u) + 2u) + (size_t)gamma * mig_window(mb) * 4u + 15) & ~(size_t)15;
}
// The scattering form keeps keys and values in registers: the image and the
// list, in whose place each window cell's new slot (u16) is kept afterwards.
__host__ __device__ constexpr size_t mig_wave_lds_scatter(uint32_t mb, uint32_t gamma) {
  return ((size_t)mig_window(mb) * 2u + (size_t)gamma * mig_window(mb) * 4u + 15) & ~(size_t)15;
}

// The window of block b (cells t = lane + 64 q, q < Q, of [b B - H, ...)),
// wrapped modulo the old capacity (mask = capacity - 1).  COH: device-coherent
// loads (agent-scope relaxed atomics), for a table that other wavefronts of
// the same launch wrote.
template <int LAYOUT, int Q, bool COH = false>
__device__ __forceinline__ void mig_load_window(u64 (&nk)[Q], u64 (&nv)[Q], const void *old_cells, u64 mask,
                                                u64 b) {
  constexpr uint32_t mb = 64 * Q - 2 * MIG_HALO;
  const uint32_t lane = threadIdx.x & 63;
  const long long wb = (long long)(b * mb) - MIG_HALO;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const u64 x = (u64)(wb + (long long)(lane + 64 * q)) & mask;
    if (LAYOUT == 0) {
      nk[q] = Cells<0>::word<COH>(old_cells, x);
      nv[q] = 0;
    } else {
      const u64x2 c = Cells<1>::cell<COH>(old_cells, x);
      nk[q] = c.x;
      nv[q] = c.y;
    }
  }
}

// Migrates block `blk` from its window (k, v) into the new table of
// 2^(log2_old + g) cells; `base` is the wavefront's mig_wave_lds(B, LAYOUT,
// 2^g) bytes of LDS (SCATTER: mig_wave_lds_scatter(B, 2^g)).  Returns the
// number of elements written.
//   SCATTER: instead of gathering the owned image from keys and values kept
//     in LDS, each lane stores its own elements that landed in the owned range
//     from its registers and the empty owned cells are zeroed (less LDS, more
//     wavefronts where LDS is short); nothing is written after an overflow.
//   COH: the new cells are written with device-coherent stores (agent-scope
//     relaxed atomics), for readers in the same launch.
template <int LAYOUT, int Q, bool SCATTER = false, bool COH = false>
__device__ __forceinline__ long long mig_block(const u64 (&k)[Q], const u64 (&v)[Q], u64 blk, uint32_t log2_old,
                                               uint32_t g, const uint32_t (*T)[256], uint32_t crc_hi, uint32_t crc_lo,
                                               u64 mul, unsigned char *base, void *new_cells, bool &overflow) {
  constexpr int H = MIG_HALO;
  constexpr uint32_t W = 64 * Q;  // window cells
  constexpr uint32_t mb = W - 2 * H;
  static_assert(H % 64 == 0 && mb % 64 == 0, "window of whole lane rows");
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t gamma = 1u << g;  // 1 or 2
  const uint32_t IW = gamma * W;   // image slots
  typedef typename std::conditional<LAYOUT == 0, u64, u64x2>::type Cell;
  Cell *wcell = (Cell *)base;  // gather only: the window
  uint32_t *img = (uint32_t *)(SCATTER ? base : (unsigned char *)(wcell + W));
  uint32_t *list = img + IW;                     // W / 2 entries
  uint16_t *newpos = (uint16_t *)list;           // scatter only, afterwards: owned slot each element went to
  static_assert(2 * 64 * Q < 0xFFFF, "image slots fit 16 bits");
  const u64 cap = 1ull << log2_old, mask = cap - 1;
  const uint32_t log2_new = log2_old + g;
  long long moved = 0;
  const long long d = (long long)(blk * mb);
  const long long wbase = d - H;  // unwrapped old index of window cell 0
  u64 emp[Q];         // ballot of empty window cells, 64 per word
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const uint32_t t = lane + 64 * q;
    const u64 key = LAYOUT == 0 ? (k[q] & 0xFFFFFFFFull) : k[q];
    if (!SCATTER) {
      if constexpr (LAYOUT == 0)
        wcell[t] = k[q];
      else
        wcell[t] = u64x2{k[q], v[q]};
    }
    emp[q] = __ballot(key == kEmpty);
  }
  for (uint32_t t = lane; t < IW / 4; t += 64)
    ((uint4 *)img)[t] = uint4{kImgEmpty, kImgEmpty, kImgEmpty, kImgEmpty};
  // the window range [lo, hi) of the clusters overlapping the block
  // (cell H - 1 and cell H both non-empty: a cluster comes in from before);
  // every index into emp[] is a constant, so it stays in registers
  int lo = H, hi = H + (int)mb;
  bool skip = false;
  if (!((emp[H / 64 - 1] >> 63) & 1ull) && !(emp[H / 64] & 1ull)) {
    int last = -1;
#pragma unroll
    for (int q = 0; q < H / 64; ++q)
      if (emp[q]) last = 64 * q + 63 - __builtin_clzll(emp[q]);
    if (last < 0) skip = true;
    lo = last + 1;
  }
  if (!((emp[(H + mb) / 64 - 1] >> 63) & 1ull)) {
    int first = -1;
#pragma unroll
    for (int q = Q - 1; q >= 0; --q) {
      if (64 * q < H + (int)mb) break;
      if (emp[q]) first = 64 * q + __builtin_ctzll(emp[q]);
    }
    if (first < 0) skip = true;
    hi = first;
  }
  wave_sync();
  if (skip) {
    overflow = true;
  } else {
    // Only the elements of [lo, hi) are hashed and placed (the halo rows
    // outside it are mostly skipped whole).
    bool bad = false;
    int before = -1;  // the last empty cell of the rows so far
    // Elements that did not get their home are listed (who asks, and for which
    // slot next) and the list worked off by lanes that take the next entry as
    // soon as theirs has settled.
    uint32_t nlist = 0;
    auto work_list = [&]() {
      wave_sync();
      uint32_t next = lane, cur = 0, p = 0;
      bool act = false;
      while (true) {
        if (!act && next < nlist) {
          const uint32_t e = list[next];
          cur = e & 0xFFFFu;
          p = e >> 16;
          act = true;
          next += 64;
        }
        if (!__any(act)) break;
        if (act) {
          if (p >= IW) {
            bad = true;
            act = false;
          } else {
            const uint32_t old = atomicMin(&img[p], cur);
            act = old != kImgEmpty;
            cur = old > cur ? old : cur;  // whoever was pushed out or turned away asks on
            ++p;
          }
        }
      }
      wave_sync();
      nlist = 0;
    };
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const u64 eq = emp[q];
      const int row_before = before;
      if (eq) before = 64 * q + 63 - __builtin_clzll(eq);
      if (64 * q + 63 < lo || 64 * q >= hi) continue;  // the row lies outside [lo, hi)
      const int t = (int)lane + 64 * q;
      const u64 key = LAYOUT == 0 ? (k[q] & 0xFFFFFFFFull) : k[q];
      uint32_t left = 0;
      if (key != kEmpty && key != kTomb && t >= lo && t < hi) {
        // new home, unwrapped consistently with this cell's old position
        const u64 hn = home_of<LAYOUT>(T, key, crc_hi, crc_lo, mul, log2_new);
        // how far the element was displaced in the old table
        const u64 delta = ((u64)(wbase + (long long)t) - (hn >> g)) & mask;
        // image slot of the home; far elements (homes before the window) fail
        // the test below
        const int r = delta < W ? (int)gamma * (t - (int)delta) + (int)(hn & (gamma - 1)) : -1;
        // its cluster's target range begins at gamma times the cluster's start
        const u64 eb = eq & ((1ull << lane) - 1);
        const int start = 1 + (eb ? 64 * q + 63 - __builtin_clzll(eb) : row_before);
        if (r < (int)gamma * start) {
          bad = true;
        } else {
          const uint32_t old = atomicMin(&img[r], (uint32_t)t);
          if (old != kImgEmpty) left = (old > (uint32_t)t ? old : (uint32_t)t) | ((uint32_t)(r + 1) << 16);
        }
      }
      const u64 m = __ballot(left != 0);  // (a slot to ask for is never 0)
      if (m) {
        if (nlist + 64 > W / 2) work_list();
        if (left) list[nlist + (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1))] = left;
        nlist += (uint32_t)__builtin_popcountll(m);
      }
    }
    work_list();
    const u64 dst0 = (u64)d * gamma;
    const uint32_t o0 = gamma * H, n_out = gamma * mb;  // the owned image slots [o0, o0 + n_out)
    auto put = [&](u64 x, u64 kw, u64 vw) {
      if (LAYOUT == 0) {
        if (COH)
          __hip_atomic_store((u64 *)new_cells + x, kw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
          ((u64 *)new_cells)[x] = kw;
      } else if (COH) {
        __hip_atomic_store((u64 *)new_cells + 2 * x, kw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store((u64 *)new_cells + 2 * x + 1, vw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        ((u64x2 *)new_cells)[x] = u64x2{kw, vw};
      }
    };
    if (SCATTER) {
      if (__any(bad)) {
        overflow = true;  // the caller redoes the move; nothing is written
      } else {
        wave_sync();
        for (uint32_t t = lane; t < W / 2; t += 64) ((uint32_t *)newpos)[t] = 0xFFFFFFFFu;
        wave_sync();
        // zeros in the owned cells left empty, then the lane's own elements
        // placed in the owned range
        for (uint32_t t = lane; t < n_out; t += 64) {
          const uint32_t ix = img[o0 + t];
          if (ix == kImgEmpty)
            put(dst0 + t, 0ull, 0ull);
          else
            newpos[ix] = (uint16_t)t;
        }
        wave_sync();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const uint32_t o = newpos[lane + 64 * q];
          if (o >= n_out) continue;
          put(dst0 + o, k[q], v[q]);
          ++moved;
        }
      }
    } else {
      if (bad) overflow = true;
      wave_sync();
      // the owned new cells [g*d, g*(d+B)) = image slots [g*H, g*(H+B))
      for (uint32_t t = lane; t < n_out; t += 64) {
        const uint32_t ix = img[o0 + t];
        const bool e = ix == kImgEmpty;
        const uint32_t j = e ? 0u : ix;
        if constexpr (LAYOUT == 0) {
          const u64 w = wcell[j];
          put(dst0 + t, e ? 0ull : w, 0ull);
        } else {
          const u64x2 w = wcell[j];
          put(dst0 + t, e ? 0ull : w.x, e ? 0ull : w.y);
        }
        moved += !e;
      }
    }
  }
  wave_sync();
  return moved;
}

}  // namespace lpht
