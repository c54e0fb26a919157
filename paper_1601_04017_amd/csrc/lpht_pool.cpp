// The library's device memory: blocks of every table's cells, status and
// scratch, kept for reuse after they are freed (the paper's user-space memory
// pool, Sec. 7).
//
// Why not the runtime's stream-ordered pool alone: a block freed by an object
// of one pass and asked for by the next went through page mapping again, and
// the next kernel launch waited for it.  Growing a table from 4096 cells with
// 2 * 10^7 keys took 57 ms a pass of which the kernels were 3.5, an insertion of
// 10^7 Zipf keys growing inside the kernel 30 ms of 6; with this cache in front
// of it, and the same kernels, 3.4 and 6.1 ms.
//
// Blocks come from a pool of the runtime (hipMallocFromPoolAsync) in size
// classes and go back to it by hipFreeAsync: hipMalloc is refused, and ruins the
// capture, while any other stream is captured in the global mode, and hipFree
// waits for every stream of the device, a resident kernel's among them.  A freed
// block carries an event recorded on the stream it was freed on, since work
// queued there may still use it (the old table of a migration just enqueued):
//   - an allocation ordered on the same stream takes it at once, behind a
//     stream wait on that event (free of charge in stream order, and right
//     even if the handle has come to name another stream since);
//   - any other allocation takes it only once the event has completed.
// What is cached is bounded by a quarter of the device's memory: beyond that the
// blocks freed longest ago go back, each as soon as a call of the library finds
// its last use completed (the runtime's pool keeps none of it past the next
// synchronisation).  When an allocation fails, all that have completed go back.
// Everything goes back in release_pools.
//
// While a stream is being captured no block of the cache is handed out, since
// a replay would use it at any later time: allocations of a capturing stream
// become nodes of its graph, from a pool of their own, and their frees wait for
// release_pools.  The events' queries are made in the relaxed capture mode, so
// that they pass, and harm nothing, while some other thread captures.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdint>
#include <mutex>
#include <new>
#include <thread>
#include <unordered_map>
#include <vector>

#include "lpht_host.h"

namespace lpht {
namespace host {

bool capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) {
    // the legacy stream while another one is captured: nothing is captured here
    (void)hipGetLastError();
    return false;
  }
  return st != hipStreamCaptureStatusNone;
}

namespace {

constexpr int kMaxDevices = 64;

struct Free {
  void *p;
  hipEvent_t ev;      // null: never used yet
  hipStream_t s;      // the stream it was freed on
  uint64_t seq;       // order of the frees
};

struct Block {
  uint32_t cls;       // size class, or kGraphBlock
  int device;
  bool slab;          // part of a slab: never given back by itself
};
constexpr uint32_t kGraphBlock = ~0u;

struct Device {
  std::unordered_map<uint32_t, std::vector<Free>> free;  // by class, oldest first
  std::vector<void *> slabs;
  uint64_t cached = 0, limit = 0;
  hipMemPool_t pool = nullptr, graph_pool = nullptr;
  // blocks whose event cannot be waited on: given back by release_pools
  std::vector<Free> stuck;
};

std::mutex g_mu;
Device g_dev[kMaxDevices];
std::unordered_map<void *, Block> g_blocks;  // every block the library holds
std::vector<hipEvent_t> g_events;            // spare
uint64_t g_seq = 0;
// blocks handed out by pool_alloc, or being made by it, and not yet given back
// to pool_free
long long g_out = 0;

// Classes: powers of two up to 64 KiB, above that eight steps per power of
// two (at most an eighth is lost).  A class is its size's exponent and eighth.
constexpr uint32_t kSmallLog2 = 16;
constexpr size_t kSlabBytes = 1 << 20;

uint32_t class_of(size_t bytes) {
  uint32_t lg = 9;
  while (lg < kSmallLog2 && ((size_t)1 << lg) < bytes) ++lg;
  if (((size_t)1 << lg) >= bytes) return lg << 3;
  lg = 63 - (uint32_t)__builtin_clzll((unsigned long long)bytes);
  const uint64_t step = 1ull << (lg - 3);
  const uint64_t eighths = (bytes - (1ull << lg) + step - 1) / step;  // 0..8
  return (lg << 3) + (uint32_t)eighths;  // 8 eighths: the next power of two
}

size_t class_bytes(uint32_t cls) {
  const uint32_t lg = cls >> 3;
  return ((size_t)1 << lg) + (size_t)(cls & 7) * (((size_t)1 << lg) >> 3);
}

// A device selected for the calls that go to the current one.
struct OnDevice {
  int before = -1;
  bool ok;
  explicit OnDevice(int device) {
    int cur = -1;
    ok = hipGetDevice(&cur) == hipSuccess;
    if (ok && cur != device) {
      ok = hipSetDevice(device) == hipSuccess;
      if (ok) before = cur;
    }
  }
  ~OnDevice() {
    if (before >= 0) (void)hipSetDevice(before);
  }
};

// The calling thread's HIP calls in the relaxed capture mode.
struct Relaxed {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  bool ok;
  Relaxed() : ok(hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess) {}
  ~Relaxed() {
    if (ok) (void)hipThreadExchangeStreamCaptureMode(&mode);
  }
};

void spare(hipEvent_t ev) {
  if (ev) g_events.push_back(ev);
}

// Takes a free block of the class out of the cache, or null.  `in_order`: the
// block's first use is ordered on s, so one freed on s needs no completion.
void *take(Device &D, uint32_t cls, hipStream_t s, bool in_order) {
  auto it = D.free.find(cls);
  if (it == D.free.end()) return nullptr;
  std::vector<Free> &v = it->second;
  for (int pass = 0; pass < 2; ++pass) {
    for (size_t k = v.size(); k-- > 0;) {
      Free f = v[k];
      const bool same = in_order && f.ev && f.s == s;
      // first pass: blocks that need no query, the last freed first
      if (pass == 0 ? !(same || !f.ev) : (same || !f.ev)) continue;
      hipError_t e = hipSuccess;
      if (f.ev) e = same ? hipStreamWaitEvent(s, f.ev, 0) : hipEventQuery(f.ev);
      if (e == hipErrorNotReady) {
        (void)hipGetLastError();
        continue;
      }
      v.erase(v.begin() + (long)k);
      if (e != hipSuccess) {
        // an event that cannot be waited on (HIP has reported events recorded
        // into a capture this way): the error is the pool's, not the caller's
        (void)hipGetLastError();
        D.stuck.push_back(f);
        D.cached -= class_bytes(cls);
        continue;
      }
      D.cached -= class_bytes(cls);
      spare(f.ev);
      return f.p;
    }
  }
  return nullptr;
}

// Gives cached blocks whose last use has completed back, in stream order on s,
// the one freed longest ago first, until `keep` bytes are left.  Waits for
// nothing.  Returns the bytes given back; `busy`: some block is still in use.
uint64_t give_back(Device &D, uint64_t keep, hipStream_t s, bool *busy = nullptr) {
  struct Ref {
    uint64_t seq;
    uint32_t cls;
  };
  std::vector<Ref> order;
  for (auto &kv : D.free)
    for (const Free &f : kv.second) {
      const auto b = g_blocks.find(f.p);
      if (b != g_blocks.end() && !b->second.slab) order.push_back({f.seq, kv.first});
    }
  std::sort(order.begin(), order.end(), [](const Ref &a, const Ref &b) { return a.seq < b.seq; });
  const uint64_t before = D.cached;
  for (const Ref &r : order) {
    if (D.cached <= keep) break;
    std::vector<Free> &v = D.free[r.cls];
    const auto at = std::find_if(v.begin(), v.end(), [&](const Free &f) { return f.seq == r.seq; });
    if (at == v.end()) continue;
    const hipError_t e = at->ev ? hipEventQuery(at->ev) : hipSuccess;
    if (e != hipSuccess) {
      (void)hipGetLastError();
      if (busy && e == hipErrorNotReady) *busy = true;
      continue;
    }
    if (hipFreeAsync(at->p, s) != hipSuccess) {
      (void)hipGetLastError();  // the block stays where it is
      continue;
    }
    g_blocks.erase(at->p);
    spare(at->ev);
    D.cached -= class_bytes(r.cls);
    v.erase(at);
  }
  return before - D.cached;
}

// The runtime's pool behind one of a device's handles, made at first use.
// keep: it holds freed memory until it is trimmed (a graph's allocations),
// otherwise until the next synchronisation.
hipMemPool_t runtime_pool(hipMemPool_t &slot, int dev, bool keep) {
  if (!slot) {
    hipMemPoolProps props{};
    props.allocType = hipMemAllocationTypePinned;
    props.handleTypes = hipMemHandleTypeNone;
    props.location.type = hipMemLocationTypeDevice;
    props.location.id = dev;
    hipMemPool_t pool = nullptr;
    if (hipMemPoolCreate(&pool, &props) != hipSuccess) return nullptr;
    uint64_t threshold = keep ? ~0ull : 0ull;
    (void)hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &threshold);
    slot = pool;
  }
  return slot;
}

void *graph_alloc(int device, size_t bytes, hipStream_t s) {
  hipMemPool_t pool = runtime_pool(g_dev[device].graph_pool, device, true);
  void *p = nullptr;
  if (!pool || hipMallocFromPoolAsync(&p, bytes, pool, s) != hipSuccess) return nullptr;
  g_blocks[p] = {kGraphBlock, device, true};
  return p;
}

// How long an allocation that found no memory waits for cached blocks still in
// use (a table destroyed just before another one as large is made).
constexpr auto kRoomWait = std::chrono::milliseconds(200);

// `nb` bytes from the runtime's pool, in stream order on s; with the lock held
// by `lk`, given up while the runtime maps memory or a wait goes on.
void *from_runtime(int device, size_t nb, hipStream_t s, bool in_order, std::unique_lock<std::mutex> &lk) {
  Device &D = g_dev[device];
  hipMemPool_t pool = runtime_pool(D.pool, device, false);
  if (!pool) return nullptr;
  const auto attempt = [&]() -> void * {
    void *p = nullptr;
    lk.unlock();
    const hipError_t e = hipMallocFromPoolAsync(&p, nb, pool, s);
    if (e != hipSuccess) (void)hipGetLastError();
    lk.lock();
    return e == hipSuccess ? p : nullptr;
  };
  if (void *p = attempt()) return p;
  const auto until = std::chrono::steady_clock::now() + kRoomWait;
  for (bool first = true;; first = false) {
    bool busy = false;
    const uint64_t given = give_back(D, 0, s, &busy);
    if (first || given) {
      if (hipMemPoolTrimTo(pool, 0) != hipSuccess) (void)hipGetLastError();
      if (void *p = attempt()) return p;
    }
    // (a kernel already running waits for a block that is not in stream order)
    if (!busy || !in_order || std::chrono::steady_clock::now() > until) return nullptr;
    lk.unlock();
    std::this_thread::sleep_for(std::chrono::microseconds(100));
    lk.lock();
  }
}

// A new block (with the lock held by `lk`).
void *fresh(int device, uint32_t cls, hipStream_t s, bool in_order, std::unique_lock<std::mutex> &lk) {
  Device &D = g_dev[device];
  const size_t cb = class_bytes(cls);
  const bool slab = cb <= ((size_t)1 << kSmallLog2);
  const size_t nb = slab ? kSlabBytes : cb;
  void *p = from_runtime(device, nb, s, in_order, lk);
  if (!p) return nullptr;
  if (!slab) {
    g_blocks[p] = {cls, device, false};
    return p;
  }
  // small classes are cut from slabs: one allocation for many status blocks
  D.slabs.push_back(p);
  for (size_t at = 0; at + cb <= nb; at += cb) {
    void *q = (unsigned char *)p + at;
    g_blocks[q] = {cls, device, true};
    if (at) {
      D.free[cls].push_back({q, nullptr, nullptr, ++g_seq});
      D.cached += cb;
    }
  }
  return p;
}

void hold_bound(Device &D, int device, hipStream_t s) {
  if (!D.limit) {
    size_t total = 0;
    if (hipDeviceTotalMem(&total, device) != hipSuccess) (void)hipGetLastError();
    D.limit = std::max<uint64_t>(1ull << 30, total / 4);
  }
  if (D.cached > D.limit) (void)give_back(D, D.limit, s);
}

}  // namespace

void *pool_alloc(int device, size_t bytes, hipStream_t s, bool in_order) try {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  OnDevice on(device);
  if (!on.ok) return nullptr;
  Relaxed relaxed;
  const bool captured = capturing(s);
  std::unique_lock<std::mutex> lk(g_mu);
  Device &D = g_dev[device];
  // counted from here on: the lock is given up on the way, and the pools must
  // not be released meanwhile
  struct Counted {
    bool kept = false;
    Counted() { ++g_out; }
    ~Counted() {
      if (!kept) --g_out;
    }
  } counted;
  void *p = nullptr;
  if (captured) {
    p = graph_alloc(device, bytes, s);
  } else {
    const uint32_t cls = class_of(bytes);
    p = take(D, cls, s, in_order);
    if (!p) p = fresh(device, cls, s, in_order, lk);
    hold_bound(D, device, s);
  }
  counted.kept = p != nullptr;
  return p;
} catch (const std::bad_alloc &) {
  return nullptr;  // host memory for the bookkeeping
}

void pool_free(void *p, hipStream_t s) try {
  if (!p) return;
  Relaxed relaxed;
  Block b;
  hipEvent_t ev = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    const auto it = g_blocks.find(p);
    if (it == g_blocks.end()) return;  // not of this pool
    b = it->second;
    if (!g_events.empty()) {
      ev = g_events.back();
      g_events.pop_back();
    }
  }
  OnDevice on(b.device);
  const bool captured = capturing(s);
  if (!ev && hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
    (void)hipGetLastError();
    ev = nullptr;
  }
  if (!captured && ev && hipEventRecord(ev, s) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipEventDestroy(ev);
    ev = nullptr;
  }
  // freed inside a capture, or outside the capture it was allocated in, or with
  // nothing to wait for: out of use until the pools are released after a device
  // synchronisation
  bool out_of_use = captured || b.cls == kGraphBlock;
  if (!out_of_use && !ev && hipStreamSynchronize(s) != hipSuccess) {
    (void)hipGetLastError();
    out_of_use = true;
  }
  std::lock_guard<std::mutex> lk(g_mu);
  Device &D = g_dev[b.device];
  --g_out;
  if (out_of_use) {
    spare(ev);
    D.stuck.push_back({p, nullptr, s, ++g_seq});
    return;
  }
  D.free[b.cls].push_back({p, ev, s, ++g_seq});
  D.cached += class_bytes(b.cls);
  hold_bound(D, b.device, s);
} catch (const std::bad_alloc &) {
  // no host memory for the bookkeeping: the block is lost to the process
}

int release_pools() try {
  Relaxed relaxed;
  std::lock_guard<std::mutex> lk(g_mu);
  if (g_out != 0) return LPHT_ERR_INVALID;
  int rc = LPHT_OK;
  for (int d = 0; d < kMaxDevices; ++d) {
    Device &D = g_dev[d];
    if (!D.pool && !D.graph_pool) continue;
    OnDevice on(d);
    if (!on.ok || hipDeviceSynchronize() != hipSuccess) {
      rc = LPHT_ERR_DEVICE;
      continue;
    }
    std::vector<Free> all = std::move(D.stuck);
    D.stuck.clear();
    for (auto &kv : D.free) all.insert(all.end(), kv.second.begin(), kv.second.end());
    D.free.clear();
    auto release = [&](void *p, bool graph) {
      if (hipFreeAsync(p, nullptr) == hipSuccess) return;
      (void)hipGetLastError();
      if (!graph) rc = LPHT_ERR_DEVICE;
    };
    for (const Free &f : all) {
      const Block b = g_blocks[f.p];
      // (the slabs' parts go with their slabs)
      if (b.cls == kGraphBlock || !b.slab) release(f.p, b.cls == kGraphBlock);
      g_blocks.erase(f.p);
      if (f.ev && hipEventDestroy(f.ev) != hipSuccess) (void)hipGetLastError();
    }
    for (void *p : D.slabs) release(p, false);
    D.slabs.clear();
    D.cached = 0;
    if (hipDeviceSynchronize() != hipSuccess) rc = LPHT_ERR_DEVICE;
    for (hipMemPool_t *pool : {&D.pool, &D.graph_pool}) {
      if (*pool && (hipMemPoolTrimTo(*pool, 0) != hipSuccess || hipMemPoolDestroy(*pool) != hipSuccess))
        rc = LPHT_ERR_DEVICE;
      *pool = nullptr;
    }
  }
  for (hipEvent_t ev : g_events) (void)hipEventDestroy(ev);
  g_events.clear();
  return rc;
} catch (const std::bad_alloc &) {
  return LPHT_ERR_OOM;
}

void *dev_alloc(lpht_table *t, size_t bytes, hipStream_t s, bool in_order) {
  if (t->cfg.alloc) return t->cfg.alloc(bytes, (void *)s, t->cfg.alloc_ctx);
  return pool_alloc(t->device, bytes, s, in_order);
}

void dev_free(lpht_table *t, void *p, size_t bytes, hipStream_t s) {
  if (!p) return;
  if (t->cfg.free) {
    t->cfg.free(p, bytes, (void *)s, t->cfg.alloc_ctx);
    return;
  }
  pool_free(p, s);
}

}  // namespace host
}  // namespace lpht
