// syev3_noalloc.hip -- the segment table of syev3_solve_segments_noalloc: a
// fixed array in each GPU's memory instead of one allocated per call or per
// server, for callers that cannot allocate device memory.  Calls of up to
// kInlineSegments segments do not need it: their table is the kernel's
// argument (2.4 us less on the host than the copy and the launch, and no
// copy ahead of the kernel on the stream).
//
// Every device holds its own copy of the array, at its own address, with
// room for the most segments one call accepts, until the process ends.  In
// host code the array's name stands for a host-side shadow, not a device
// address: the address comes from hipGetSymbolAddress, looked up once per
// device with that device current (here, at the entry point's first call on
// the device), and only that address is passed on, to the copy and to the
// segment kernel.
#include <algorithm>
#include <mutex>

#include "syev3_internal.hpp"

namespace syev3 {

constexpr size_t kTableBytes =
    offsetof(TickTable, seg) + (sizeof(Segment) + sizeof(int64_t)) * kMaxSegmentsPerTick;

static __device__ __align__(256) unsigned char scratch[kTableBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch[kMaxDevices] = {};

// Host image of the device table; one call at a time fills it and copies
// from it.
std::mutex g_image_mu;
alignas(16) unsigned char g_image[kTableBytes];

// One workgroup per tile (as a server's ticks), up to 2^24.
int32_t grid_of(int64_t tiles) { return (int32_t)std::min<int64_t>(tiles, (int64_t)1 << 24); }

hipError_t scratch_of_device(int dev, TickTable** out) {
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    int cur = 0;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != dev && (e = hipSetDevice(dev)) != hipSuccess) return e;
    void* ptr = nullptr;
    e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
    if (cur != dev) {
      const hipError_t r = hipSetDevice(cur);
      if (e == hipSuccess) e = r;
    }
    if (e != hipSuccess) return e;
    g_scratch[dev] = ptr;
  }
  *out = (TickTable*)g_scratch[dev];
  return hipSuccess;
}

}  // namespace

// Segments first .. first + count - 1 of the table in one launch whose kernel
// argument they are, their tiles counted from the first one's.
static hipError_t launch_part(const TickTable* host_table, int first, int count,
                              hipStream_t stream) {
  const Segment* seg = host_table->seg + first;
  const int64_t end = first + count < host_table->nseg ? seg[count].tile_begin
                                                       : host_table->total_tiles;
  InlineTable t;
  t.nseg = count;
  t.cap = kInlineSegments;
  t.total_tiles = end - seg[0].tile_begin;
  for (int i = 0; i < count; ++i) {
    t.seg[i] = seg[i];
    t.begin[i] = t.seg[i].tile_begin -= seg[0].tile_begin;
  }
  (void)hipGetLastError();  // launch_segments_inline reads it: drop any stale error
  return launch_segments_inline(t, grid_of(t.total_tiles), stream);
}

hipError_t launch_segments_noalloc(const TickTable* host_table, hipStream_t stream) {
  const int nseg = host_table->nseg;
  hipError_t e;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  // (the default stream cannot be captured)
  if (nseg > kInlineSegments && stream &&
      (e = hipStreamIsCapturing(stream, &capture)) != hipSuccess)
    return e;
  if (nseg <= kInlineSegments || capture != hipStreamCaptureStatusNone) {
    for (int i = 0; i < nseg; i += kInlineSegments) {
      e = launch_part(host_table, i, std::min(nseg - i, kInlineSegments), stream);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  int dev = 0;
  e = stream ? hipStreamGetDevice(stream, &dev) : hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  TickTable* table = nullptr;
  if ((e = scratch_of_device(dev, &table)) != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(g_image_mu);
  TickTable* image = (TickTable*)g_image;
  image->nseg = image->cap = nseg;
  image->total_tiles = host_table->total_tiles;
  std::copy(host_table->seg, host_table->seg + nseg, image->seg);
  int64_t* begins = table_begins(image);
  for (int i = 0; i < nseg; ++i) begins[i] = host_table->seg[i].tile_begin;
  // In stream order: the kernel of an earlier call on this stream has read
  // the table before this copy overwrites it.
  e = hipMemcpyAsync(table, image, tick_table_bytes(nseg), hipMemcpyHostToDevice, stream);
  if (e != hipSuccess) return e;
  (void)hipGetLastError();  // launch_segments reads it: drop any stale error
  return launch_segments(table, grid_of(image->total_tiles), stream);
}

}  // namespace syev3
