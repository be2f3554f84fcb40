// syev3_internal.hpp -- declarations shared by the library's host sources.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "syev3.h"

namespace syev3 {

constexpr int kBlock = 256;  // lanes (matrices) per workgroup: 4 wavefronts

// Plane strides (elements) of the three SoA arrays; unused (0) for AoS.
struct Strides {
  int64_t a, l, v;
};

// Launch the batched solver; arguments already validated (SoA strides
// resolved: each >= n).  Returns the HIP status of the launch.
hipError_t launch_batched(int64_t n, const void* A, Strides ld, int layout,
                          void* lambda, void* V, int dtype, uint32_t flags,
                          int32_t* info, hipStream_t stream);

// One request of a serving tick, as the segment kernel reads it from device
// memory.  Matrices of segment s occupy tiles [tile_begin, tile_begin +
// ceil(n / kBlock)) of the tick's tile space, so no workgroup spans two
// segments.
struct Segment {
  const void* A;  // 6 planes of n, plane stride lda
  void* lambda;   // 3 planes of n, plane stride n
  void* V;        // 9 planes of n, plane stride n; NULL: eigenvalues only
  int64_t n;
  int64_t lda;    // >= n
  int64_t tile_begin;
  int32_t dtype;
  uint32_t flags;
};

// The solver's SoA loads and/or stores with trivial arithmetic (measurement
// aid); mode: SYEV3_PROBE_* bits, at least one of READ and WRITE.
hipError_t launch_stream_probe(int64_t n, const void* A, void* lambda, void* V, int dtype,
                               uint32_t mode, hipStream_t stream);

// A tick's table: header, then the segments in ascending tile_begin order.
// In device memory it has room for `cap` segments and each one's tile_begin
// again, side by side after them (the search for a tile's segment reads 2 KB
// of consecutive memory for 256 segments, not one line per segment).
constexpr int kMaxSegmentsPerTick = SYEV3_SERVER_MAX_SEGMENTS;
struct TickTable {
  int32_t nseg;
  int32_t cap;
  int64_t total_tiles;
  Segment seg[kMaxSegmentsPerTick];
};
// Bytes of a device table with room for `cap` segments.
inline size_t tick_table_bytes(int cap) {
  return offsetof(TickTable, seg) + (sizeof(Segment) + sizeof(int64_t)) * (size_t)cap;
}
// The tile_begins of a device table (or its host image).
template <typename Table>
__host__ __device__ inline auto* table_begins(Table* t) {
  return (decltype(&t->total_tiles))(t->seg + t->cap);
}

// Launch the segment kernel on a table in device memory: grid_blocks
// workgroups stride over the table's tiles.
hipError_t launch_segments(const TickTable* table, int32_t grid_blocks,
                           hipStream_t stream);

// A table small enough to travel as the launch's kernel argument (3600
// bytes), with nothing to copy first.
constexpr int kInlineSegments = 56;
struct InlineTable {
  int32_t nseg;
  int32_t cap;
  int64_t total_tiles;
  int64_t begin[kInlineSegments];
  Segment seg[kInlineSegments];
};
hipError_t launch_segments_inline(const InlineTable& table, int32_t grid_blocks,
                                  hipStream_t stream);

// A request whose input and results are the caller's pinned host memory, in
// planes of n: its matrices are read from there and also stored to s.A, its
// results stored to s.lambda and s.V and, where not NULL, to lambda and V.
struct HostSegment {
  Segment s;  // s.lda == s.n
  const void* A;
  void* lambda;
  void* V;
};
constexpr int kHostSegments = 40;
struct HostTable {
  int32_t nseg;
  int64_t total_tiles;
  int64_t begin[kHostSegments];
  HostSegment seg[kHostSegments];
};
// At most max_blocks workgroups, which stride over the table's tiles.
hipError_t launch_segments_host(const HostTable& table, int32_t max_blocks,
                                hipStream_t stream);

// How many of a server's requests that kernel has been launched on: for tests,
// as its results are those of the copies; not part of the interface.
extern "C" int64_t syev3_server_solved_in_place(syev3_server* s);

// launch_segments for host_table (nseg segments, total_tiles > 0; its cap and what
// follows the segments are not read) with no allocation: as the kernel's
// argument up to kInlineSegments segments (and under capture, in as many
// launches as it takes), else copied into the library's fixed table of the
// stream's device.  That copy is from pageable host memory, which HIP
// completes before returning.
hipError_t launch_segments_noalloc(const TickTable* host_table, hipStream_t stream);

}  // namespace syev3
