// One operation of a bulk call on the table by a single lane (Algorithm 1 with
// bounded lookahead), shared by the one-lane-per-operation kernels
// (lpht_lane.hip) and the region load (lpht_load.hip).
#pragma once

#include "lpht_device.h"

namespace lpht {

template <int LAYOUT>
__device__ __forceinline__ u64 word_in(const void *a, u64 i) {
  return LAYOUT == 0 ? (u64)((const uint32_t *)a)[i] : ((const u64 *)a)[i];
}

// What a probe looks at: the whole word (PACKED32) or the key, and for finds
// the value too (KV64).
struct Seen {
  u64 w, v;
};

template <int LAYOUT, int OP>
__device__ __forceinline__ Seen look(const void *cells, u64 p) {
  if (LAYOUT == 0) return {Cells<0>::word(cells, p), 0};
  if (OP == OP_FIND) {
    const u64x2 c = Cells<1>::cell(cells, p);
    return {c.x, c.y};
  }
  return {Cells<1>::key(cells, p), 0};
}

template <int LAYOUT>
__device__ __forceinline__ u64 seen_key(u64 w) {
  return LAYOUT == 0 ? (w & 0xFFFFFFFFull) : w;
}

// value := up(value, d) of the present key in cell p
template <int LAYOUT, int UP>
__device__ __forceinline__ void apply_up(void *cells, u64 p, u64 d) {
  if (LAYOUT == 0) {
    if (UP == 1)
      add64((u64 *)cells + p, d << 32);
    else
      ((uint32_t *)cells)[2 * p + 1] = (uint32_t)d;
  } else {
    u64 *v = (u64 *)cells + 2 * p + 1;
    if (UP == 1)
      add64(v, d);
    else
      *v = d;
  }
}

// Ends the operation at cell p, last seen as `s` (its key is k or empty), or
// finds that another operation gave the cell to another key: then false, and
// the probe goes on after p.  A failed compare-and-swap returns the current
// word, which is looked at in place of the cell (the "revisit" of Algorithm 1).
template <int LAYOUT, int OP, int UP>
__device__ __forceinline__ bool settle(void *cells, u64 p, Seen s, u64 k, u64 d, uint8_t &flag, u64 &out) {
  while (true) {
    const u64 ck = seen_key<LAYOUT>(s.w);
    if (ck == k) {
      if (OP == OP_FIND) {
        out = LAYOUT == 0 ? Cells<0>::val_of(s.w) : s.v;
        flag = 1;
      } else if (OP == OP_INSERT) {
        flag = 0;
      } else if (OP == OP_UPSERT || OP == OP_UPDATE) {
        apply_up<LAYOUT, UP>(cells, p, d);
        flag = OP == OP_UPDATE ? 1 : 0;
      } else {
        // the key becomes the tombstone, the value stays
        u64 *w = (u64 *)cells + (LAYOUT == 0 ? p : 2 * p);
        const u64 old = cas64(w, s.w, LAYOUT == 0 ? (s.w & ~0xFFFFFFFFull) | kTomb : kTomb);
        if (old != s.w) {
          s.w = old;
          continue;
        }
        flag = 1;
      }
      return true;
    }
    if (ck != kEmpty) return false;
    if (OP == OP_FIND || OP == OP_UPDATE || OP == OP_ERASE) {
      flag = 0;
      return true;
    }
    u64 *w = (u64 *)cells + (LAYOUT == 0 ? p : 2 * p);
    const u64 old = cas64(w, s.w, LAYOUT == 0 ? (d << 32) | k : k);
    if (old == s.w) {
      // KV64: the claimed cell's value, 0 until now; concurrent insert-or-adds
      // of the same key add to it
      if (LAYOUT == 1) {
        if (OP == OP_UPSERT && UP == 1)
          add64(w + 1, d);
        else
          w[1] = d;
      }
      flag = 1;
      return true;
    }
    s.w = old;
  }
}

// One operation on a non-reserved key.  Returns the flag; finds leave the
// value in `out`.
template <int LAYOUT, int OP, int UP, int W>
__device__ __forceinline__ uint8_t lane_op(const BulkArgs &A, u64 k, u64 d, u64 &out) {
  const u64 mask = (1ull << A.log2c) - 1;
  u64 p = hash_direct<LAYOUT>(k, A.crc_hi, A.crc_lo, A.mul) >> (64 - A.log2c);
  uint8_t flag = 0;
  Seen s = look<LAYOUT, OP>(A.cells, p);
  u64 seen = 1;  // cells passed; more than the mask: every cell holds another key
  bool event = seen_key<LAYOUT>(s.w) == k || seen_key<LAYOUT>(s.w) == kEmpty;
  while (true) {
    if (event && settle<LAYOUT, OP, UP>(A.cells, p, s, k, d, flag, out)) return flag;
    if (seen > mask) break;
    // the next W cells; the first of them that ends the run is looked at
    Seen c[W];
#pragma unroll
    for (int j = 0; j < W; ++j) c[j] = look<LAYOUT, OP>(A.cells, (p + 1 + j) & mask);
    event = false;
    uint32_t at = W - 1;
    s = c[W - 1];
#pragma unroll
    for (int j = W - 1; j >= 0; --j) {
      const u64 ck = seen_key<LAYOUT>(c[j].w);
      if (ck == k || ck == kEmpty) {
        event = true;
        at = j;
        s = c[j];
      }
    }
    // a second look at cells already passed (at the end of a full table)
    // changes nothing: they hold other keys
    p = (p + 1 + at) & mask;
    seen += 1 + at;
  }
  return OP == OP_INSERT || OP == OP_UPSERT ? 0xFF : 0;
}

// ORs the wavefront's error bits into the status block (all lanes call it).
// Bits that are seen set there already stay: one line takes 87 M atomics a
// second, and where reserved keys are frequent every wavefront has some (2^22
// insertions of present keys with one reserved key in 41: 602 -> 33 us).  A stale
// line only means an atomic too many.
__device__ __forceinline__ void lane_errors(DevStatus *st, uint32_t err) {
  const u64 any = __ballot(err != 0);
  if (any) {
    const uint32_t e = (__ballot(err & kErrFull) ? kErrFull : 0) | (__ballot(err & kErrReserved) ? kErrReserved : 0);
    if ((threadIdx.x & 63) == 0 && (st->err & e) != e) atomicOr(&st->err, e);
  }
}

}  // namespace lpht
