// The serving loop (csrc/lpht_server.cpp) over host memory: tables that only
// count the batches run on them, and copies that fail when told to.  Prints
// "name value" lines for the test to look at.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "lpht_host.h"
#include "lpht_serve.h"

namespace {

std::atomic<int> batches{0}, kernel_arrays{0}, copies{0};
std::atomic<int> fail_kernel{0}, fail_copy{0};  // so many of the next calls
std::atomic<int> array_type{hipMemoryTypeHost}, array_device{0};

bool fails(std::atomic<int> &n) {
  if (n.load() <= 0) return false;
  n--;
  return true;
}

}  // namespace

namespace lpht {
hipError_t launch_serve_copy(const std::vector<ServeSeg> &segs, const std::vector<ServeCount> &counts, hipStream_t) {
  if (segs.empty() && counts.empty()) return hipSuccess;
  if (fails(fail_kernel)) return hipErrorLaunchFailure;
  for (const ServeSeg &g : segs) {
    std::memcpy(g.dst, g.src, g.bytes);
    kernel_arrays++;
  }
  for (const ServeCount &c : counts) c.out[0] = c.out[1] = c.out[2] = 0;
  return hipSuccess;
}
hipError_t launch_persist(uint32_t, const PersistCtl *, const PersistReq *, PersistReq *, PersistDone *, PersistDev *,
                          PersistState *, uint64_t, uint32_t, hipStream_t) {
  return hipErrorNotSupported;
}
hipError_t launch_persist_init(PersistDev *, PersistState *, uint64_t, hipStream_t) { return hipErrorNotSupported; }
namespace host {
uint64_t cell_bytes(uint32_t) { return 16; }
int growth_kind(const lpht_table *, uint64_t) { return 0; }
bool within_fill(const lpht_table *, uint64_t, uint64_t) { return true; }
int grow_before_batch(lpht_table *, uint64_t, hipStream_t) { return LPHT_OK; }
void dev_free(lpht_table *, void *p, size_t, hipStream_t) { std::free(p); }
void *dev_alloc(lpht_table *, size_t n, hipStream_t, bool) { return std::malloc(n); }
BulkArgs make_args(lpht_table *) { return BulkArgs{}; }
}  // namespace host
}  // namespace lpht

extern "C" {
void lpht_config_default(lpht_config *c) { std::memset(c, 0, sizeof(*c)); }
int lpht_create(const lpht_config *c, void *, lpht_table **out) {
  *out = new lpht_table();
  (*out)->cfg = *c;
  (*out)->log2c = c->log2_capacity;
  return LPHT_OK;
}
int lpht_destroy(lpht_table *t, void *) {
  delete t;
  return LPHT_OK;
}
int lpht_batch_create(uint32_t, lpht_batch **out) {
  *out = nullptr;
  return LPHT_OK;
}
int lpht_batch_destroy(lpht_batch *) { return LPHT_OK; }
int lpht_batch_run(lpht_batch *, const lpht_batch_op *, uint32_t, void *) {
  batches++;
  return LPHT_OK;
}

hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  return hipErrorNotSupported;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  if (fails(fail_copy)) return hipErrorInvalidValue;
  std::memcpy(d, s, n);
  copies++;
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *at, const void *p) {
  std::memset(at, 0, sizeof(*at));
  at->type = (hipMemoryType)array_type.load();
  at->device = array_device.load();
  at->devicePointer = (void *)p;
  return hipSuccess;
}
}

int main() {
  const uint32_t cap = 12;
  lpht_server_config cfg{};
  cfg.ntables = 1;
  cfg.layout = LPHT_KV64;
  cfg.log2_capacity = &cap;
  cfg.mode = LPHT_SERVE_WAVES;
  cfg.max_inflight = 4;
  cfg.streams = 1;
  lpht_server *S = nullptr;
  if (lpht_server_create(&cfg, &S) != LPHT_OK) return 1;
  std::vector<uint64_t> keys(100, 7), vals(100);
  std::vector<uint8_t> kinds(100, 0), flags(100);
  const auto serve = [&](const char *name) {
    batches = kernel_arrays = copies = 0;
    lpht_request r{};
    r.n = keys.size();
    r.keys = keys.data();
    r.kinds = kinds.data();
    r.vals_out = vals.data();
    r.flags = flags.data();
    uint64_t ticket = 0;
    lpht_completion c{};
    if (lpht_server_submit(S, &r, &ticket) != LPHT_OK || lpht_server_wait(S, ticket, &c) != LPHT_OK) std::exit(1);
    std::printf("%s.status %d\n%s.batches %d\n%s.kernel_arrays %d\n%s.copies %d\n", name, c.status, name,
                batches.load(), name, kernel_arrays.load(), name, copies.load());
  };
  serve("pinned");
  array_type = hipMemoryTypeDevice;
  serve("device");
  array_device = 1;
  serve("other_device");
  array_device = 0;
  array_type = hipMemoryTypeHost;
  fail_kernel = 1;
  serve("copy_in_refused");
  serve("after_it");
  array_type = hipMemoryTypeUnregistered;
  serve("pageable");
  fail_copy = 1;
  serve("pageable_refused");
  lpht_server_destroy(S);
}
