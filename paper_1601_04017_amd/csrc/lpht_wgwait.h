// A wait that one wavefront makes for its workgroup.  Not part of the public
// C ABI; the workgroup is a template argument, so that the host tests run this
// code on threads.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define LPHT_WG_FN __device__ __forceinline__
#else
#define LPHT_WG_FN inline
#endif

namespace lpht {

// poll() waits with a bound of its own and returns nonzero, or 0 when the bound
// passed; the leader (a thread of the first wavefront) calls it, and every
// wavefront still in the workgroup gets its result.  *s_word, shared by the
// workgroup, is 0 before the first wait and between waits: wavefronts that
// ended no longer count in barriers, so where the leader's has ended, the others
// pass them alone and read 0, the bound passed.
template <class Workgroup, class Poll>
LPHT_WG_FN uint32_t wg_wait(const Workgroup &wg, uint32_t *s_word, Poll poll) {
  if (wg.leader()) *s_word = poll();
  wg.sync();
  const uint32_t r = *s_word;
  wg.sync();
  if (wg.leader()) *s_word = 0;
  return r;
}

}  // namespace lpht
