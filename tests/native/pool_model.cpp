// The library's memory cache (csrc/lpht_pool.cpp) over a model of the HIP calls
// that it makes.  Memory is numbers; a stream is a count of queued and of done
// work; one other thread's stream may be captured in the global mode, which
// refuses the calls that HIP refuses then, unless the calling thread is in the
// relaxed mode.  Prints "name value" lines for the test to look at.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <set>
#include <thread>

#include "lpht_host.h"

namespace model {

std::recursive_mutex mu;
constexpr uint64_t kTotal = 64ull << 30;  // so the cache's bound is 16 GiB
uint64_t reserved = 0;                    // taken from the device
uint64_t next = 1ull << 32;
struct Mem {
  uint64_t bytes;
  bool pooled;
};
std::map<uint64_t, Mem> live;             // given out
uint64_t pool_held = 0;                   // back in the runtime's pool, still reserved
struct Stream {
  uint64_t queued = 0, done = 0;
};
Stream streams[4];
struct Event {
  Stream *s = nullptr;
  uint64_t at = 0;
};
std::set<Event *> events;
void (*during_alloc)() = nullptr;  // runs while the runtime makes a block
bool capture_elsewhere = false, invalidated = false, refuse_free = false;
uint64_t device_waits = 0, event_waits = 0;
thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;

bool refused() {
  if (!capture_elsewhere || mode == hipStreamCaptureModeRelaxed) return false;
  invalidated = true;
  return true;
}
Stream *of(hipStream_t s) { return s ? (Stream *)s : &streams[0]; }
hipStream_t handle(int i) { return (hipStream_t)&streams[i]; }

hipError_t give(void **p, size_t n, bool pooled) {
  if (reserved + n > kTotal) {
    // the runtime's pool reuses what it holds
    if (!pooled || pool_held < n) return hipErrorOutOfMemory;
    pool_held -= n;
    reserved -= n;
  }
  reserved += n;
  live[next] = {n, pooled};
  *p = (void *)next;
  next += (n + 4095) & ~4095ull;
  return hipSuccess;
}

}  // namespace model

using namespace model;
#define LOCK std::lock_guard<std::recursive_mutex> lk(model::mu)

extern "C" {
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceTotalMem(size_t *b, hipDevice_t) { *b = kTotal; return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m) {
  std::swap(*m, mode);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) {
  *st = hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
  LOCK;
  if (refused()) return hipErrorStreamCaptureUnsupported;
  return give(p, n, false);
}
hipError_t hipFree(void *p) {
  LOCK;
  if (refused()) return hipErrorStreamCaptureUnsupported;
  if (refuse_free) return hipErrorInvalidValue;
  ++device_waits;
  const auto it = live.find((uint64_t)p);
  if (it == live.end()) return hipErrorInvalidValue;
  reserved -= it->second.bytes;
  live.erase(it);
  return hipSuccess;
}
hipError_t hipMemPoolCreate(hipMemPool_t *pool, const hipMemPoolProps *) {
  *pool = (hipMemPool_t)1;
  return hipSuccess;
}
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void *) { return hipSuccess; }
hipError_t hipMemPoolDestroy(hipMemPool_t) { return hipSuccess; }
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) {
  LOCK;
  reserved -= pool_held;
  pool_held = 0;
  return hipSuccess;
}
hipError_t hipMallocFromPoolAsync(void **p, size_t n, hipMemPool_t, hipStream_t) {
  if (during_alloc) during_alloc();
  LOCK;
  return give(p, n, true);
}
hipError_t hipFreeAsync(void *p, hipStream_t) {
  LOCK;
  if (refuse_free) return hipErrorInvalidValue;
  const auto it = live.find((uint64_t)p);
  if (it == live.end() || !it->second.pooled) return hipErrorInvalidValue;
  pool_held += it->second.bytes;
  live.erase(it);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  LOCK;
  Event *x = new Event;
  events.insert(x);
  *e = (hipEvent_t)x;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  LOCK;
  events.erase((Event *)e);
  delete (Event *)e;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  LOCK;
  Event *x = (Event *)e;
  x->s = of(s);
  x->at = x->s->queued;
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  LOCK;
  if (refused()) return hipErrorStreamCaptureUnsupported;
  const Event *x = (Event *)e;
  return x->s->done >= x->at ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  LOCK;
  if (refused()) return hipErrorStreamCaptureUnsupported;
  Event *x = (Event *)e;
  if (x->s->done < x->at) ++event_waits;
  x->s->done = std::max(x->s->done, x->at);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  LOCK;
  if (refused()) return hipErrorStreamCaptureUnsupported;
  of(s)->done = of(s)->queued;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  LOCK;
  if (refused()) return hipErrorStreamCaptureUnsupported;
  for (Stream &s : streams) s.done = s.queued;
  return hipSuccess;
}
}

using lpht::host::pool_alloc;
using lpht::host::pool_free;
using lpht::host::release_pools;

namespace {

constexpr size_t kMiB = 1 << 20, kGiB = 1 << 30;

void show(const char *name, uint64_t v) { std::printf("%s %llu\n", name, (unsigned long long)v); }
void work(int i) { streams[i].queued++; }
void finish(int i) { streams[i].done = streams[i].queued; }

}  // namespace

int main() {
  // another thread's capture: allocations that miss the cache, that look at a
  // block in use, and frees
  {
    void *a = pool_alloc(0, 5 * kMiB, handle(1));
    work(1);
    pool_free(a, handle(1));
    capture_elsewhere = true;
    void *b = pool_alloc(0, 5 * kMiB, handle(2));   // a's block is still in use
    void *c = pool_alloc(0, 900, handle(2));        // a slab
    void *d = pool_alloc(0, 300 * kMiB, handle(2));
    show("capture_allocated", b && c && d);
    for (void *p : {b, c, d}) pool_free(p, handle(2));
    capture_elsewhere = false;
    show("capture_harmed", invalidated);
    finish(1);
  }
  // a block that HIP does not take back stays in the books
  {
    void *a = pool_alloc(0, 20 * kGiB, handle(1));
    refuse_free = true;
    pool_free(a, handle(1));                        // above the bound
    refuse_free = false;
    void *b = pool_alloc(0, 20 * kGiB, handle(1));
    show("kept_block_used_again", a == b);
    pool_free(b, handle(1));
  }
  // the bound: a block still in use when it is freed goes back later
  {
    finish(1);
    void *a = pool_alloc(0, 24 * kGiB, handle(1));
    work(1);
    const uint64_t waits = device_waits + event_waits;
    pool_free(a, handle(1));
    finish(1);
    void *b = pool_alloc(0, 2 * kMiB, handle(2));
    (void)hipMemPoolTrimTo(nullptr, 0);                 // (the runtime's next synchronisation)
    show("reserved_within_bound", reserved <= 17 * kGiB);
    show("waits_over_bound", device_waits + event_waits - waits);
    pool_free(b, handle(2));
  }
  // no memory left: what has completed goes back, without a wait for the device
  // or for an event
  {
    finish(1);
    finish(2);
    void *a = pool_alloc(0, 15 * kGiB, handle(1));
    void *b = pool_alloc(0, 30 * kGiB, handle(1));
    pool_free(a, handle(1));
    const uint64_t waits = device_waits + event_waits;
    void *c = pool_alloc(0, 28 * kGiB, handle(2));
    show("room_made", c != nullptr);
    show("waits_for_room", device_waits + event_waits - waits);
    // a block still in use: waited for where the allocation is in stream order
    work(1);
    pool_free(b, handle(1));
    show("not_in_order", pool_alloc(0, 28 * kGiB, handle(2), false) != nullptr);
    std::thread other([] {
      std::this_thread::sleep_for(std::chrono::milliseconds(20));
      LOCK;
      finish(1);
    });
    void *d = pool_alloc(0, 28 * kGiB, handle(2));
    other.join();
    show("in_order", d != nullptr);
    // the first use never ends: refused in the end
    work(1);
    pool_free(d, handle(1));
    show("never", pool_alloc(0, 30 * kGiB, handle(2)) != nullptr);
    show("waits_at_last", device_waits + event_waits - waits);
    finish(1);
    pool_free(c, handle(2));
  }
  // a release while a block is being made
  {
    static int rc = LPHT_OK;
    during_alloc = [] { std::thread([] { rc = release_pools(); }).join(); };
    void *a = pool_alloc(0, 7 * kMiB, handle(1));
    during_alloc = nullptr;
    show("release_refused", a && rc == LPHT_ERR_INVALID);
    pool_free(a, handle(1));
  }
  show("released", release_pools() == LPHT_OK);
  show("left", live.size());
  show("events_left", events.size());
}
