// Host-only check of the server's host-staged requests (syev3_server.cpp),
// built with g++ under AddressSanitizer and UndefinedBehaviorSanitizer by
// test_server_host.py.  The HIP runtime is replaced by a model: device
// pointers are numbers that are never dereferenced, host allocations are
// entries of a table that the pointer queries answer from, copies and kernel
// launches are recorded and events have completed at once.
//
// Each request must go to the kernel that works on host memory in place
// exactly when its buffers allow it, and be copied otherwise; its launch must
// keep to the server's most workgroups; and the runtime must not be queried
// while the server's lock is held.
#include "syev3_server.cpp"

#include <atomic>
#include <cstdio>
#include <cstdlib>

namespace {

struct Alloc {
  uintptr_t base;
  size_t size;
  hipMemoryType type;
  unsigned flags;
  int device;
  bool managed, same_address;
};
std::vector<Alloc> g_allocs;

struct Seen {
  std::mutex mu;
  std::vector<int> host_launches;  // requests of each launch on host memory
  std::vector<syev3::HostSegment> host;
  int32_t max_blocks = -1;
  std::vector<syev3::Segment> device;
  int to_device = 0, to_host = 0;
} g_seen;

syev3_server* g_server = nullptr;
std::atomic<int> g_queries{0}, g_under_lock{0};

// Whether another thread gets the server's lock (the scheduler holds it for
// moments only).
void query() {
  ++g_queries;
  if (!g_server) return;
  bool got = false;
  std::thread t([&] {
    for (int i = 0; i < 100 && !got; ++i) {
      if (g_server->mu.try_lock()) {
        g_server->mu.unlock();
        got = true;
      } else {
        std::this_thread::sleep_for(std::chrono::milliseconds(1));
      }
    }
  });
  t.join();
  if (!got) ++g_under_lock;
}

const Alloc* find(uintptr_t p) {
  for (const Alloc& a : g_allocs)
    if (p >= a.base && p < a.base + a.size) return &a;
  return nullptr;
}

void record(const syev3::HostTable& t) {
  std::lock_guard<std::mutex> lk(g_seen.mu);
  g_seen.host_launches.push_back(t.nseg);
  for (int i = 0; i < t.nseg; ++i) g_seen.host.push_back(t.seg[i]);
}

}  // namespace

namespace syev3 {
hipError_t launch_segments(const TickTable*, int32_t, hipStream_t) {
  // the table's copy, recorded below, holds the same segments
  return hipSuccess;
}
hipError_t launch_segments_host(const HostTable& t, int32_t max_blocks, hipStream_t) {
  record(t);
  g_seen.max_blocks = max_blocks;
  return hipSuccess;
}
}  // namespace syev3

extern "C" {
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
  static uintptr_t next = (uintptr_t)1 << 44;
  *p = (void*)next;
  next += (n + 4095) / 4096 * 4096;
  return hipSuccess;
}
hipError_t hipFree(void*) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::calloc(1, n);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t)8;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t)8;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t, hipMemcpyKind k, hipStream_t) {
  std::lock_guard<std::mutex> lk(g_seen.mu);
  if (k == hipMemcpyHostToDevice && g_server && dst == g_server->ticks[0].d_table) {
    const syev3::TickTable* t = (const syev3::TickTable*)src;
    for (int i = 0; i < t->nseg; ++i) g_seen.device.push_back(t->seg[i]);
  } else if (k == hipMemcpyHostToDevice) {
    ++g_seen.to_device;
  } else {
    ++g_seen.to_host;
  }
  return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, hipMemcpyKind,
                            hipStream_t) {
  return hipErrorUnknown;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* at, const void* p) {
  query();
  const Alloc* a = find((uintptr_t)p);
  if (!a) return hipErrorInvalidValue;
  at->type = a->type;
  at->device = a->device;
  at->devicePointer = a->same_address ? const_cast<void*>(p) : (char*)const_cast<void*>(p) + 64;
  at->hostPointer = const_cast<void*>(p);
  at->isManaged = a->managed;
  at->allocationFlags = a->flags;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
  query();
  const Alloc* a = find((uintptr_t)p);
  if (!a) return hipErrorInvalidValue;
  *base = (hipDeviceptr_t)a->base;
  *size = a->size;
  return hipSuccess;
}
// ticks are launched directly here
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorUnknown; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorUnknown; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphGetNodes(hipGraph_t, hipGraphNode_t*, size_t*) { return hipErrorUnknown; }
hipError_t hipGraphNodeGetType(hipGraphNode_t, hipGraphNodeType*) { return hipErrorUnknown; }
hipError_t hipGraphKernelNodeGetParams(hipGraphNode_t, hipKernelNodeParams*) {
  return hipErrorUnknown;
}
hipError_t hipGraphExecKernelNodeSetParams(hipGraphExec_t, hipGraphNode_t,
                                           const hipKernelNodeParams*) {
  return hipErrorUnknown;
}
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return hipErrorUnknown;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorUnknown; }
roctx_range_id_t roctxRangeStartA(const char*) { return 0; }
void roctxRangeStop(roctx_range_id_t) {}
}

namespace {

int g_failures = 0;

#define EXPECT(cond, ...)                    \
  do {                                       \
    if (!(cond)) {                           \
      std::fprintf(stderr, __VA_ARGS__);     \
      std::fprintf(stderr, ": %s\n", #cond); \
      ++g_failures;                          \
    }                                        \
  } while (0)

syev3_server* server(int32_t grid_blocks) {
  syev3_server_opts o;
  syev3_server_default_opts(&o);
  o.hbm_budget_bytes = 1 << 30;
  o.max_requests = 256;
  o.max_inflight_ticks = 1;
  o.grid_blocks = grid_blocks;
  o.use_graphs = 0;
  syev3_server* s = nullptr;
  if (syev3_server_create(&o, &s) != SYEV3_OK) std::exit(2);
  return s;
}

void reset() {
  std::lock_guard<std::mutex> lk(g_seen.mu);
  g_seen.host_launches.clear();
  g_seen.host.clear();
  g_seen.device.clear();
  g_seen.to_device = g_seen.to_host = 0;
}

constexpr uintptr_t kBase = (uintptr_t)1 << 32;
constexpr int64_t kN = 1000;
constexpr size_t kA = 48 * kN, kL = 24 * kN, kV = 72 * kN;  // bytes, FP64

// One FP64 request; `direct`: it has to be solved in place.
void request(const char* what, uintptr_t A, uintptr_t lam, uintptr_t V, bool vectors, bool direct,
             int dtype = SYEV3_F64) {
  reset();
  syev3_request_buffers b;
  const int64_t id = syev3_server_acquire(g_server, kN, dtype, vectors, &b);
  EXPECT(id >= 0, "%s", what);
  EXPECT(syev3_server_submit_host(g_server, id, (void*)A, (void*)lam, (void*)V) == SYEV3_OK, "%s",
         what);
  EXPECT(syev3_server_submit_host(g_server, id, (void*)A, (void*)lam, (void*)V) == SYEV3_E_STATE,
         "%s, submitted twice", what);
  EXPECT(syev3_server_wait(g_server, id, 10.0, nullptr) == 1, "%s", what);
  EXPECT(syev3_server_release(g_server, id) == SYEV3_OK, "%s", what);
  EXPECT(syev3_server_submit_host(g_server, id, (void*)A, (void*)lam, (void*)V) == SYEV3_E_STATE,
         "%s, released", what);
  std::lock_guard<std::mutex> lk(g_seen.mu);
  EXPECT(g_seen.host.size() == (size_t)direct && g_seen.device.size() == (size_t)!direct, "%s",
         what);
  EXPECT(g_seen.to_device == (direct ? 0 : 1), "%s", what);
  EXPECT(g_seen.to_host == (direct ? 0 : 1 + (V && vectors)), "%s", what);
  const syev3::Segment* s = direct && g_seen.host.size() == 1 ? &g_seen.host[0].s
                            : !direct && g_seen.device.size() == 1 ? &g_seen.device[0] : nullptr;
  if (!s) return;
  EXPECT(s->A == b.A && s->lambda == b.lambda && s->V == b.V && s->n == kN && s->lda == kN &&
             s->tile_begin == 0 && s->dtype == dtype && s->flags == 0,
         "%s", what);
  if (direct) {
    const syev3::HostSegment& h = g_seen.host[0];
    EXPECT(h.A == (void*)A && h.lambda == (void*)lam &&
               h.V == (vectors ? (void*)V : nullptr),
           "%s", what);
  }
}

}  // namespace

int main() {
  const Alloc pinned{kBase, 1 << 20, hipMemoryTypeHost, hipHostMallocDefault, 0, false, true};
  const uintptr_t A = kBase, L = A + kA, V = L + kL, end = kBase + (1 << 20);
  g_server = server(0);
  g_allocs = {pinned};
  request("pinned", A, L, V, true, true);
  request("pinned, eigenvalues", A, L, 0, false, true);
  request("pinned, vectors kept on the device", A, L, 0, true, true);
  request("pinned, a host V for eigenvalues", A, L, V, false, true);
  request("pinned FP32", A, L, V, true, true, SYEV3_F32_REFINE);
  request("up to the end", end - kA, kBase, kBase + kL, true, true);
  request("the input crosses the end", end - kA + 8, kBase, kBase + kL, true, false);
  request("the eigenvalues cross the end", kBase, end - kL + 8, kBase + kA, true, false);
  request("the vectors cross the end", kBase, kBase + kA, end - kV + 8, true, false);
  request("FP32 up to the end", end - kA / 2, kBase, kBase + kL, true, true, SYEV3_F32_REFINE);
  request("odd input", A + 4, L + 8, V + 8, true, false);
  request("odd eigenvalues", A, L + 4, V + 8, true, false);
  request("odd vectors", A, L, V + 4, true, false);
  request("FP32 on 4 bytes", A + 4, L + 4, V + 4, true, true, SYEV3_F32_REFINE);
  request("eigenvalues over the input", A, A + kA - 8, V, true, false);
  request("vectors over the input", V - 8, A, V + kA - 16, true, false);
  request("vectors over the eigenvalues", A, L, L + kL - 8, true, false);
  request("pageable input", kBase - (1 << 24), L, V, true, false);
  request("pageable eigenvalues", A, kBase - (1 << 24), V, true, false);
  request("pageable vectors", A, L, kBase - (1 << 24), true, false);
  struct {
    const char* what;
    bool direct;
    Alloc a;
  } kinds[] = {
      {"non-coherent", false, {kBase, 1 << 20, hipMemoryTypeHost, hipHostMallocNonCoherent, 0, false, true}},
      {"coherent by flag", true, {kBase, 1 << 20, hipMemoryTypeHost, hipHostMallocCoherent, 0, false, true}},
      {"managed", false, {kBase, 1 << 20, hipMemoryTypeHost, 0, 0, true, true}},
      {"device memory", false, {kBase, 1 << 20, hipMemoryTypeDevice, 0, 0, false, true}},
      {"at another address", false, {kBase, 1 << 20, hipMemoryTypeHost, 0, 0, false, false}},
      {"another device's", false, {kBase, 1 << 20, hipMemoryTypeHost, 0, 1, false, true}},
      {"portable", true, {kBase, 1 << 20, hipMemoryTypeHost, hipHostMallocPortable, 1, false, true}},
  };
  for (const auto& k : kinds) {
    g_allocs = {k.a};
    request(k.what, A, L, V, true, k.direct);
  }
  g_allocs = {pinned};

  // more requests than one launch's table holds, in ticks of any split
  reset();
  std::vector<int64_t> ids;
  for (int i = 0; i < 100; ++i) {
    syev3_request_buffers b;
    ids.push_back(syev3_server_acquire(g_server, 10, SYEV3_F64, 1, &b));
    EXPECT(syev3_server_submit_host(g_server, ids.back(), (void*)(kBase + 10000 * i),
                                    (void*)(kBase + 10000 * i + 480),
                                    (void*)(kBase + 10000 * i + 720)) == SYEV3_OK, "many");
  }
  for (int64_t id : ids) {
    EXPECT(syev3_server_wait(g_server, id, 10.0, nullptr) == 1, "many");
    EXPECT(syev3_server_release(g_server, id) == SYEV3_OK, "many");
  }
  {
    std::lock_guard<std::mutex> lk(g_seen.mu);
    EXPECT(g_seen.host.size() == 100 && g_seen.to_device + g_seen.to_host == 0, "many");
    for (int k : g_seen.host_launches) EXPECT(k >= 1 && k <= syev3::kHostSegments, "many");
  }
  EXPECT(g_seen.max_blocks >= 64, "as many workgroups as the kernel wants");
  EXPECT(g_queries > 0 && g_under_lock == 0, "%d of %d queries under the lock",
         g_under_lock.load(), g_queries.load());
  syev3_server* s = g_server;
  g_server = nullptr;
  syev3_server_destroy(s);

  g_server = server(7);
  request("at most 7 workgroups", A, L, V, true, true);
  EXPECT(g_seen.max_blocks == 7, "at most 7 workgroups, not %d", g_seen.max_blocks);
  s = g_server;
  g_server = nullptr;
  syev3_server_destroy(s);
  std::printf("%d failures\n", g_failures);
  return g_failures != 0;
}
