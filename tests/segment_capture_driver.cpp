// Host-only check of the no-allocation segment call's launches
// (syev3_noalloc.hip), built with g++ under AddressSanitizer and
// UndefinedBehaviorSanitizer by test_segment_capture.py.  The HIP calls that
// it makes are replaced by a model of a stream: eager work is done at once,
// work under capture is recorded and done at each replay.  A "launch" looks
// up every tile's segment in the table it was given, as the segment kernel
// does, and counts the tile at that segment's input; inputs are numbers that
// are never dereferenced.
//
// A captured call must solve exactly its own requests at every replay,
// whatever larger or smaller calls were made since, and an eager call its
// own, in any order of sizes.
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) ((const void*)(x))
#include "syev3_noalloc.hip"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <random>
#include <vector>

namespace {

bool g_capturing = false;
std::vector<std::function<void()>> g_graph;
std::map<uintptr_t, std::vector<int>> g_solved;  // input -> count of each of its tiles
bool g_wild = false;                             // a tile outside every live request

void enqueue(std::function<void()> f) {
  if (g_capturing) g_graph.push_back(std::move(f));
  else f();
}

void solve_tile(const syev3::Segment& s, int64_t tile) {
  const int64_t t = tile - s.tile_begin;
  const auto it = g_solved.find((uintptr_t)s.A);
  if (it == g_solved.end() || t < 0 || t >= (int64_t)it->second.size()) g_wild = true;
  else ++it->second[(size_t)t];
}

template <typename Table>
void run_table(const Table& t, const int64_t* begin) {
  for (int64_t tile = 0; tile < t.total_tiles; ++tile) {
    int n = 0;
    for (int i = 0; i < t.nseg; ++i) n += begin[i] <= tile;
    if (n < 1) g_wild = true;
    else solve_tile(t.seg[n - 1], tile);
  }
}

unsigned char g_device_table[sizeof(syev3::TickTable) +
                             sizeof(int64_t) * syev3::kMaxSegmentsPerTick];

}  // namespace

namespace syev3 {
hipError_t launch_segments(const TickTable* t, int32_t, hipStream_t) {
  enqueue([t] { run_table(*t, table_begins(t)); });
  return hipSuccess;
}
hipError_t launch_segments_inline(const InlineTable& table, int32_t, hipStream_t) {
  enqueue([table] { run_table(table, table.begin); });
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
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = g_device_table;
  return hipSuccess;
}
// pageable host memory: an eager copy reads it before the call returns, a
// captured one at each replay
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) {
  enqueue([=] { std::memcpy(dst, src, n); });
  return hipSuccess;
}
}

namespace {

std::mt19937 g_rng(1);
uintptr_t g_next = 1 << 20;

struct Call {
  syev3::TickTable t;
  std::vector<std::pair<uintptr_t, int>> tiles;  // input, tiles
};

void make(Call& c, int nseg) {
  c.t.nseg = nseg;
  c.t.cap = syev3::kMaxSegmentsPerTick;
  c.t.total_tiles = 0;
  c.tiles.clear();
  for (int i = 0; i < nseg; ++i) {
    const int tiles = 1 + (int)(g_rng() % 4);
    syev3::Segment& s = c.t.seg[i];
    std::memset(&s, 0, sizeof s);
    s.A = (const void*)(g_next += 4096);
    s.n = s.lda = (int64_t)tiles * syev3::kBlock;
    s.tile_begin = c.t.total_tiles;
    c.t.total_tiles += tiles;
    c.tiles.push_back({(uintptr_t)s.A, tiles});
  }
}

// Only c's requests are live: clear their counts.
void live(const Call& c) {
  g_solved.clear();
  g_wild = false;
  for (const auto& q : c.tiles) g_solved[q.first].assign((size_t)q.second, 0);
}

void check(const char* what, int nseg, int other) {
  bool ok = !g_wild;
  for (const auto& q : g_solved)
    for (int k : q.second) ok = ok && k == 1;
  if (ok) return;
  std::fprintf(stderr, "%s of %d requests, then a call of %d: %s\n", what, nseg, other,
               g_wild ? "a tile of no live request" : "a tile not solved once");
  std::exit(1);
}

Call a, b;

}  // namespace

int main() {
  const int sizes[] = {1, 55, 56, 57, 60, 100, 111, 112, 113, 300, 1023, 1024};
  hipStream_t stream = (hipStream_t)8;
  int calls = 0;
  for (int n : sizes) {
    for (int m : sizes) {
      make(a, n);
      live(a);
      if (syev3::launch_segments_noalloc(&a.t, stream) != hipSuccess) return 2;
      check("a call", n, m);
      make(b, m);
      live(b);
      if (syev3::launch_segments_noalloc(&b.t, nullptr) != hipSuccess) return 2;
      check("a call", m, n);
      // captured; then another call on other requests before each replay
      g_graph.clear();
      g_capturing = true;
      if (syev3::launch_segments_noalloc(&a.t, stream) != hipSuccess) return 2;
      g_capturing = false;
      for (int rep = 0; rep < 2; ++rep) {
        live(a);
        for (auto& f : g_graph) f();
        check("a captured call", n, rep ? m : 0);
        live(b);
        if (syev3::launch_segments_noalloc(&b.t, stream) != hipSuccess) return 2;
        check("a call", m, n);
      }
      ++calls;
    }
  }
  std::printf("%d pairs of calls, captured and eager, 0 failures\n", calls);
  return 0;
}
