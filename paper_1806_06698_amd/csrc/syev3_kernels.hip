// syev3_kernels.hip -- batched 3x3 symmetric eigensolver kernels (gfx950).
//
// One lane per matrix.  Each workgroup handles kBlock = 256 consecutive
// matrices.
//   * SoA: each of the 6 input planes and of the 3 + 9 output planes is read
//     or written by a wavefront as one contiguous 512-byte (FP64) or 256-byte
//     (FP32) run: fully coalesced, no LDS.
//   * AoS: the workgroup's 256 x 6 input block is contiguous in memory; it is
//     read with unit-stride lanes (16 bytes each) into LDS and each lane then
//     picks up its own 6 entries (the transpose).  Outputs go back through
//     LDS the same way, so global stores are unit-stride as well.
// Streams are read and written once; how (workgroup order, non-temporal
// hints, workgroups per compute unit) is chosen per launch, in motion().
#include <algorithm>
#include <type_traits>

#include "syev3_internal.hpp"
#include "syev3_lane.hpp"

namespace syev3 {

// Workgroup order.  The dispatcher deals workgroups to the 8 XCDs in turn,
// so in launch order neighbouring tiles of the batch run on different XCDs.
// In the chunked order each XCD instead takes 2^log2_chunk consecutive tiles
// at a time, over the first `chunked` workgroups (a multiple of 8 chunks, or
// 0 for launch order); the rest keep their own index.
constexpr uint32_t kXcds = 8;
constexpr int kWave = 64;  // gfx950 runs wave64

struct Order {
  uint32_t chunked, log2_chunk;
};

__device__ __forceinline__ uint32_t tile_of_block(uint32_t b, Order o) {
  if (b >= o.chunked) return b;
  const uint32_t x = b % kXcds, slot = b / kXcds;
  const uint32_t in = slot & ((1u << o.log2_chunk) - 1);
  return (((slot >> o.log2_chunk) * kXcds + x) << o.log2_chunk) + in;
}

inline Order chunked_order(int64_t blocks, uint32_t log2_chunk) {
  const int64_t round = (int64_t)kXcds << log2_chunk;
  return Order{(uint32_t)(blocks / round * round), log2_chunk};
}

// NT: with the non-temporal hint.
template <bool NT, typename T>
__device__ __forceinline__ T ld(const T* p) {
  return NT ? __builtin_nontemporal_load(p) : *p;
}
template <bool NT, typename T>
__device__ __forceinline__ void st(T v, T* p) {
  if (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// The element type a form stores: double for FP64, float for both FP32
// forms.
template <int FORM>
using Storage = typename std::conditional<FORM == kFormF64, double, float>::type;

template <typename T>
__device__ __forceinline__ T qnan() {
  return (T)__builtin_nan("");
}

// The 18 plane base addresses of an SoA solve, passed as kernel arguments
// (uniform, held in scalar registers): each array has a plane stride of its
// own, so they may lie anywhere.
template <typename T>
struct Planes {
  const T* a[6];
  T* l[3];
  T* v[9];
};

// T = double: FP64 path.  T = float: FP32 storage with FP64 refinement.
// 64-bit element offsets, for planes of more than 2^32 bytes.  NTL, NTS: the
// loads' and the stores' hint.
template <int FORM, bool VECS, bool INFO, bool NTL, bool NTS>
__global__ __launch_bounds__(kBlock) void k_syev3_soa(int64_t n, Planes<Storage<FORM>> P,
                                                     uint32_t flags, Order order,
                                                     int32_t* __restrict__ info) {
  using T = Storage<FORM>;
  const int64_t i = (int64_t)tile_of_block(blockIdx.x, order) * kBlock + threadIdx.x;
  if (i >= n) return;
  double a[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) a[k] = (double)ld<NTL>(P.a[k] + i);
  double l[3], v[9];
  bool bad;
  const int code = solve3<VECS, FORM>(a, flags, l, v, bad);
#pragma unroll
  for (int j = 0; j < 3; ++j) st<NTS>((T)l[j], P.l[j] + i);
  if (VECS) {
#pragma unroll
    for (int k = 0; k < 9; ++k) st<NTS>((T)v[k], P.v[k] + i);
  }
  if (bad) {  // a NaN or infinite entry: NaN in every output of the matrix
#pragma unroll
    for (int j = 0; j < 3; ++j) st<NTS>(qnan<T>(), P.l[j] + i);
    if (VECS) {
#pragma unroll
      for (int k = 0; k < 9; ++k) st<NTS>(qnan<T>(), P.v[k] + i);
    }
  }
  if (INFO) info[i] = code;
}

// The same with a 32-bit byte offset per lane, for n * sizeof(T) < 2^32:
// loads and stores take the scalar-base addressing form and need no 64-bit
// address arithmetic per lane.
template <int FORM, bool VECS, bool INFO, bool NTL, bool NTS>
__global__ __launch_bounds__(kBlock) void k_syev3_soa32(uint32_t n, Planes<Storage<FORM>> P,
                                                       uint32_t flags, Order order,
                                                       int32_t* __restrict__ info) {
  using T = Storage<FORM>;
  const uint32_t i = tile_of_block(blockIdx.x, order) * (uint32_t)kBlock + threadIdx.x;
  if (i >= n) return;
  const uint32_t off = i * (uint32_t)sizeof(T);  // byte offset within a plane
  double a[6];
#pragma unroll
  for (int k = 0; k < 6; ++k)
    a[k] = (double)ld<NTL>((const T*)((const char*)P.a[k] + off));
  double l[3], v[9];
  bool bad;
  const int code = solve3<VECS, FORM>(a, flags, l, v, bad);
  // The offset is re-defined here (an empty asm emits nothing) so that the
  // stores, past the solve's branches, again see a 32-bit offset and take
  // the scalar-base form rather than a 64-bit address add per store: 12
  // fewer VALU per wavefront, 2.4% faster for the VALU-bound FP32 form.
  uint32_t soff = off;
  asm volatile("" : "+v"(soff));
#pragma unroll
  for (int j = 0; j < 3; ++j) st<NTS>((T)l[j], (T*)((char*)P.l[j] + soff));
  if (VECS) {
#pragma unroll
    for (int k = 0; k < 9; ++k) st<NTS>((T)v[k], (T*)((char*)P.v[k] + soff));
  }
  if (bad) {  // a NaN or infinite entry: NaN in every output of the matrix
#pragma unroll
    for (int j = 0; j < 3; ++j) st<NTS>(qnan<T>(), (T*)((char*)P.l[j] + soff));
    if (VECS) {
#pragma unroll
      for (int k = 0; k < 9; ++k) st<NTS>(qnan<T>(), (T*)((char*)P.v[k] + soff));
    }
  }
  if (INFO) info[i] = code;
}

// Block copies between global memory and the LDS buffer of the AoS kernel:
// 16 bytes per lane when the global address is 16-byte aligned (it is for
// every block when the caller's array is), else one element per lane.
// total elements; lanes t = 0 .. kBlock - 1.  Measured on 2^26 matrices:
// 4% faster in FP64 and 9% in FP32 than element-wide copies.  NT: the loads'
// hint (the stores always have it).
template <bool NT, typename T>
__device__ __forceinline__ void copy_in(T* sm, const T* g, int total, int t) {
  constexpr int W = 16 / sizeof(T);
  typedef T vec __attribute__((ext_vector_type(W)));
  int k0 = 0;
  if (((uintptr_t)g & 15u) == 0) {
    const int nv = total / W;
    for (int k = t; k < nv; k += kBlock) ((vec*)sm)[k] = ld<NT>((const vec*)g + k);
    k0 = nv * W;
  }
  for (int k = k0 + t; k < total; k += kBlock) sm[k] = ld<NT>(g + k);
}

// The same for a full tile, whose size is known at compile time: every lane
// issues all of its loads (or LDS reads) before the first write, so its
// memory requests are in flight together rather than one after another.
// g must be 16-byte aligned.  TOTAL = elements, a multiple of 16 / sizeof(T).
template <bool NT, typename T, int TOTAL>
__device__ __forceinline__ void copy_in_full(T* sm, const T* g, int t) {
  constexpr int W = 16 / sizeof(T);
  constexpr int NV = TOTAL / W;
  constexpr int R = (NV + kBlock - 1) / kBlock;
  static_assert(TOTAL % W == 0, "whole 16-byte vectors");
  typedef T vec __attribute__((ext_vector_type(W)));
  vec x[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int k = t + j * kBlock;
    if (j + 1 < R || k < NV) x[j] = ld<NT>((const vec*)g + k);
  }
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int k = t + j * kBlock;
    if (j + 1 < R || k < NV) ((vec*)sm)[k] = x[j];
  }
}

template <typename T, int TOTAL>
__device__ __forceinline__ void copy_out_full(T* g, const T* sm, int t) {
  constexpr int W = 16 / sizeof(T);
  constexpr int NV = TOTAL / W;
  constexpr int R = (NV + kBlock - 1) / kBlock;
  static_assert(TOTAL % W == 0, "whole 16-byte vectors");
  typedef T vec __attribute__((ext_vector_type(W)));
  vec x[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int k = t + j * kBlock;
    if (j + 1 < R || k < NV) x[j] = ((const vec*)sm)[k];
  }
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int k = t + j * kBlock;
    if (j + 1 < R || k < NV) st<true>(x[j], (vec*)g + k);
  }
}

template <typename T>
__device__ __forceinline__ void copy_out(T* g, const T* sm, int total, int t) {
  constexpr int W = 16 / sizeof(T);
  typedef T vec __attribute__((ext_vector_type(W)));
  int k0 = 0;
  if (((uintptr_t)g & 15u) == 0) {
    const int nv = total / W;
    for (int k = t; k < nv; k += kBlock) st<true>(((const vec*)sm)[k], (vec*)g + k);
    k0 = nv * W;
  }
  for (int k = k0 + t; k < total; k += kBlock) st<true>(sm[k], g + k);
}

template <typename T>
constexpr size_t kAosLds = kBlock * 9 * sizeof(T);

// AoS: IN = 6 (unique entries) or 9 (full row-major matrix, upper triangle
// read).  The whole block is read into LDS before any global store, so the
// full-matrix input may be overwritten by V (in place).  A is therefore not
// __restrict__.  The outputs leave through the same LDS buffer in two
// rounds, lambda and then V, so the buffer holds 9 values per matrix rather
// than 12: 18 KB per workgroup in FP64, which lets 8 waves per SIMD fit in
// the 160 KB of LDS (24 KB allowed only 6).
template <int FORM, int IN, bool VECS, bool INFO, bool NT>
__global__ __launch_bounds__(kBlock) void k_syev3_aos(
    int64_t n, const Storage<FORM>* A, Storage<FORM>* __restrict__ lam, Storage<FORM>* V,
    uint32_t flags, Order order, int32_t* __restrict__ info) {
  using T = Storage<FORM>;
  __shared__ __attribute__((aligned(16))) T sm[kAosLds<T> / sizeof(T)];
  const int64_t base = (int64_t)tile_of_block(blockIdx.x, order) * kBlock;
  const int cnt = (int)((n - base) < kBlock ? (n - base) : kBlock);
  const int t = threadIdx.x;
  const T* Ab = A + base * IN;
  // full tiles of a 16-byte-aligned array take the unrolled copies (every
  // tile but the last, when the caller's arrays are aligned)
  const bool full = cnt == kBlock && ((uintptr_t)A & 15u) == 0 &&
                    ((uintptr_t)lam & 15u) == 0 && (!VECS || ((uintptr_t)V & 15u) == 0);
  if (full) copy_in_full<NT, T, kBlock * IN>(sm, Ab, t);
  else copy_in<NT>(sm, Ab, cnt * IN, t);
  __syncthreads();
  double a[6];
  if (t < cnt) {
    if (IN == 6) {
#pragma unroll
      for (int k = 0; k < 6; ++k) a[k] = (double)sm[6 * t + k];
    } else {
      const T* m = sm + IN * t;
      a[0] = (double)m[0]; a[1] = (double)m[1]; a[2] = (double)m[2];
      a[3] = (double)m[4]; a[4] = (double)m[5]; a[5] = (double)m[8];
    }
  }
  __syncthreads();
  double l[3], v[9];
  bool bad = false;
  if (t < cnt) {
    const int code = solve3<VECS, FORM>(a, flags, l, v, bad);
#pragma unroll
    for (int j = 0; j < 3; ++j) sm[3 * t + j] = (T)l[j];
    if (bad) {  // a NaN or infinite entry: NaN in every output of the matrix
#pragma unroll
      for (int j = 0; j < 3; ++j) sm[3 * t + j] = qnan<T>();
    }
    if (INFO) info[base + t] = code;
  }
  __syncthreads();
  if (full) copy_out_full<T, kBlock * 3>(lam + base * 3, sm, t);
  else copy_out(lam + base * 3, sm, cnt * 3, t);
  if (VECS) {
    __syncthreads();  // every lambda read from LDS before V overwrites it
    if (t < cnt) {
#pragma unroll
      for (int k = 0; k < 9; ++k) sm[9 * t + k] = (T)v[k];
      if (bad) {
#pragma unroll
        for (int k = 0; k < 9; ++k) sm[9 * t + k] = qnan<T>();
      }
    }
    __syncthreads();
    if (full) copy_out_full<T, kBlock * 9>(V + base * 9, sm, t);
    else copy_out(V + base * 9, sm, cnt * 9, t);
  }
}

// How a launch moves its data: the workgroup order, the loads' and the stores'
// non-temporal hints (AoS stores always have theirs), and dynamic LDS the
// kernel does not use, which caps the workgroups a compute unit holds.
struct Motion {
  Order order;
  bool ntl, nts;
  size_t lds;
};

// LDS of a workgroup that lets 3 of them (12 wavefronts) onto a compute unit
// (160 KB) instead of the 8 that the registers allow.
constexpr size_t kLdsFor3 = 52 << 10;
constexpr size_t kLdsFor5 = 32 << 10;  // 5 of them
// An AoS input of at most this much is read with plain loads.
constexpr int64_t kCachedInput = 64 << 20;
// From here (786K matrices, 12 workgroups per compute unit) the cap's extra
// rounds are many enough not to leave compute units idle in the last one.
constexpr int64_t kManyBlocks = 3072;
// FP64 vectors in SoA planes on 128-byte lines store with the hint from here.
constexpr int64_t kHintedStores = 1024;

// The rules, each with both sides measured (us; three sets of buffers in
// turn, N(0,1) matrices):
//  * FP64 with vectors, bound by HBM, caps its workgroups at 3 per compute
//    unit (SoA from kManyBlocks on, AoS from 16384 blocks): fewer wavefronts
//    mix fewer reads into the writes, and 12 per compute unit still cover the
//    solve.  SoA 2^24 393 (cap) against 426, 60 M 1458 against 1602; AoS 2^24
//    390 against 445, full matrices 440 against 520.  Below, the cap costs
//    whole rounds (400,000: 13.2 against 10.4).  Eigenvalues only and FP32
//    storage (72 bytes or less per matrix) need the wavefronts: FP32 vectors
//    2^24 212 without the cap, 286 with it.
//  * AoS FP64 with vectors caps them at 5 from 2560 to 16384 blocks: the
//    stress mix, slower to solve, needs more than 3 (2 M packed matrices 49.5
//    against 52.0; N(0,1) 48.8 either way).  And where its input may be found
//    in the memory-side cache (up to 64 MB: 1.4 M packed matrices, 932 K full
//    ones) it is loaded without the hint.  Mean of N(0,1), stress-mix and SPD
//    matrices over 1 and 4 sets of buffers in turn, against the hint in
//    launch order (from kManyBlocks on with the cap of 3): packed 400,000 9.0
//    against 10.0, 500,000 11.3 against 13.0, 640,000 14.9 against 20.3, 2^20
//    23.6 against 26.7; full 400,000 10.0 against 14.8, 640,000 18.2 against
//    22.7, 900,000 24.5 against 26.5.  The plain loads without the cap: 2^20
//    packed 27.8; with it below 2560 blocks: full 400,000 11.2.  Beyond 64 MB
//    buffers that are not in the cache lose by plain loads (full 2 M
//    matrices, 4 sets: 58.7 against 55.9).
//  * SoA planes that do not all start on a 128-byte line (any odd n, for
//    one): neighbouring wavefronts, and at a tile's edge neighbouring
//    workgroups, share lines.  Non-temporal stores then write partial lines
//    to memory, so loads and stores go through L2 as usual, and chunks of 32
//    tiles keep neighbours on one XCD's L2: FP64 16,777,293 matrices 435
//    against 607 with the hints in launch order (487 without either), 60 M
//    1592 against 2154; FP32 30 M 404 against 585.  FP32 storage does so
//    from 2048 blocks (whole calls: 700,001 11.3 against 14.9, 570,001 10.4
//    against 11.2, 500,003 9.3 either way, 300,489 8.2 against 7.5); three
//    planes of eigenvalues alone lose little to it and keep the hints (FP64
//    30 M 380 against 384).
//  * FP64 vectors below kManyBlocks load without the hint for any planes, as
//    the inputs of such a batch stay in the caches.  Planes off the lines are
//    also stored without it (400,003: 10.4 against 14.8) and take the chunks
//    from 1280 blocks (400,003: 10.4 against 11.5; 300,001: 9.0 against 8.7);
//    planes on the lines are stored with it, in chunks, from kHintedStores on
//    (mean of N(0,1), SPD and stress-mix matrices over 1 and 4 sets of buffers
//    in turn, against no hint: 300,000 7.9 against 9.0, 500,000 12.3 against
//    14.1, 650,000 16.5 against 18.4; with both hints 8.6, 14.4 and 18.7).
//  * Otherwise the hints: FP64 vectors 2^24 393 against 406 without.  The
//    order is launch order (60 M: 1458, in chunks of 256 tiles 1569), but
//    for AoS FP64 vectors chunks of 32 (2^24: 390 against 399; 60 M: 1406
//    against 1475).
//  * Where the plane stride comes within 64 KB of a multiple of 2^29 bytes,
//    all planes meet the same channels at once; how bad that is depends on
//    where the pages of an allocation lie.  FP64 vectors take chunks of 256
//    and load without the hint there.  Mean and worst of six allocations, the
//    first a fresh process's (SPD; N(0,1)): 2^26 1637 and 1678; 1658 and 1665,
//    with the hint 1668 and 1776; 1719 and 1795, in launch order 1727 and
//    1842; 1705 and 1757 (chunks of 64: 1776, of 512 with plain loads 1686;
//    with 2 workgroups per compute unit 1709, with 4 and chunks of 64 1862);
//    2^26 + 4096 1681, with the hint 1682, in launch order 1834; 2^27 3409
//    and 3514, with the hint 3597 and 3862.  Where the multiple is one of
//    2^31 chunks of 32 do better, with the hint or without: 2^28 6776, in
//    chunks of 256 7211 (plain loads 7001), in launch order 7072.
//    FP64 eigenvalues alone take the chunks of 256 (2^26: 761 against 820;
//    2^26 + 4096: 773 against 825; 2^27: 1517 against 1695; but 2^25, 2^28
//    bytes: 410 against 370), and the unrefined FP32 form does at 2^28 bytes
//    (2^26: 908 against 961); the refined one gains nothing from them (912
//    against 918; 1014 against 954 on another device; eigenvalues alone 2^27:
//    1081 against 1080).
template <int FORM, bool VECS>
static Motion motion(int64_t blocks, const void* A, Strides ld, int layout, const void* lambda,
                     const void* V, uint32_t flags) {
  using T = Storage<FORM>;
  constexpr bool kHbmBound = FORM == kFormF64 && VECS;
  const Order launch{0, 0};
  // the slower zero finders are bound by VALU and need the wavefronts
  const bool valu = flags & (kFlagNewton | kFlagPaperBG);
  const bool many = blocks >= kManyBlocks;
  if (layout != 0) {
    if (!kHbmBound) return Motion{launch, true, true, 0};
    const int64_t in_bytes = blocks * kBlock * (layout == 1 ? 6 : 9) * (int64_t)sizeof(T);
    const bool cached = in_bytes <= kCachedInput;
    const size_t lds = blocks >= 16384 ? kLdsFor3 : blocks >= 2560 ? kLdsFor5 : kAosLds<T>;
    return Motion{chunked_order(blocks, 5), !cached, true, valu ? 0 : lds - kAosLds<T>};
  }
  // the planes' distance is within 64 KB of a multiple of 2^log2 bytes
  const auto near = [&](int log2) {
    const uint64_t stride = (uint64_t)(VECS ? ld.v : ld.a) * sizeof(T);
    return ((stride + (1u << 16)) & (((uint64_t)1 << log2) - 1)) <= (1u << 17);
  };
  const bool aliased = FORM != kFormF32R && near(FORM == kFormF64 ? 29 : 28);
  if (!VECS)
    return Motion{FORM == kFormF64 && aliased ? chunked_order(blocks, 8) : launch, true, true, 0};
  const uintptr_t bits = (uintptr_t)A | (uintptr_t)lambda | (uintptr_t)V |
                         (uintptr_t)(ld.a | ld.l | ld.v) * sizeof(T);
  const bool ragged = (bits & 127u) != 0;
  if (kHbmBound ? ragged || !many : ragged && blocks >= 2048)
    return Motion{blocks >= (ragged ? 1280 : kHintedStores) ? chunked_order(blocks, 5) : launch,
                  false, !ragged && blocks >= kHintedStores,
                  kHbmBound && many && !valu ? kLdsFor3 : 0};
  const bool far = kHbmBound && near(31);
  return Motion{aliased ? chunked_order(blocks, far ? 5 : 8) : launch,
                !(kHbmBound && aliased && !far && !valu), true,
                kHbmBound && !valu ? kLdsFor3 : 0};
}

template <int FORM, bool VECS, bool INFO, bool NTL, bool NTS>
static void launch_soa(int64_t n, const void* A, Strides ld, void* lambda, void* V,
                       uint32_t flags, const Motion& m, int32_t* info, dim3 grid, dim3 block,
                       hipStream_t stream) {
  using T = Storage<FORM>;
  Planes<T> P;
  for (int k = 0; k < 6; ++k) P.a[k] = (const T*)A + k * ld.a;
  for (int j = 0; j < 3; ++j) P.l[j] = (T*)lambda + j * ld.l;
  for (int k = 0; k < 9; ++k) P.v[k] = VECS ? (T*)V + k * ld.v : nullptr;
  if ((uint64_t)n * sizeof(T) <= (uint64_t)UINT32_MAX)
    hipLaunchKernelGGL((k_syev3_soa32<FORM, VECS, INFO, NTL, NTS>), grid, block, m.lds, stream,
                       (uint32_t)n, P, flags, m.order, info);
  else
    hipLaunchKernelGGL((k_syev3_soa<FORM, VECS, INFO, NTL, NTS>), grid, block, m.lds, stream, n,
                       P, flags, m.order, info);
}

template <int FORM, bool VECS, bool INFO>
static hipError_t launch_t(int64_t n, const void* A, Strides ld, int layout,
                           void* lambda, void* V, uint32_t flags, int32_t* info,
                           hipStream_t stream) {
  using T = Storage<FORM>;
  const int64_t blocks = (n + kBlock - 1) / kBlock;
  const dim3 grid((unsigned)blocks), block(kBlock);
  const Motion m = motion<FORM, VECS>(blocks, A, ld, layout, lambda, V, flags);
  if (layout == 0) {
    const auto launch = [&](auto ntl, auto nts) {
      launch_soa<FORM, VECS, INFO, decltype(ntl)::value, decltype(nts)::value>(
          n, A, ld, lambda, V, flags, m, info, grid, block, stream);
    };
    using Hint = std::true_type;
    // eigenvalues alone always take both hints, FP32 storage both or neither
    using Plain = std::bool_constant<!VECS>;
    using PlainLoads = std::bool_constant<!(FORM == kFormF64 && VECS)>;
    if (m.ntl) launch(Hint(), Hint());
    else if (m.nts) launch(PlainLoads(), Hint());
    else launch(Plain(), Plain());
  } else {
    // FP64 with vectors alone has plain loads
    constexpr bool kPlain = FORM == kFormF64 && VECS;
    const auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, block, m.lds, stream, n, (const T*)A, (T*)lambda, (T*)V,
                         flags, m.order, info);
    };
    const bool nt = m.ntl || !kPlain;
    if (layout == 1) {
      if (nt) launch(k_syev3_aos<FORM, 6, VECS, INFO, true>);
      else launch(k_syev3_aos<FORM, 6, VECS, INFO, !kPlain>);
    } else {
      if (nt) launch(k_syev3_aos<FORM, 9, VECS, INFO, true>);
      else launch(k_syev3_aos<FORM, 9, VECS, INFO, !kPlain>);
    }
  }
  return hipGetLastError();
}

// A dispatch counts its grid in work-items with 32 bits per dimension, so one
// launch covers at most 2^31 matrices (2^23 workgroups); larger batches are
// solved by consecutive launches on the same stream.  Each matrix is solved
// by its own lane, so the split changes no result.
constexpr int64_t kMaxPerLaunch = (int64_t)1 << 31;

template <int FORM>
static hipError_t launch_dt(int64_t n, const void* A, Strides ld, int layout,
                            void* lambda, void* V, uint32_t flags, int32_t* info,
                            hipStream_t stream) {
  using T = Storage<FORM>;
  // elements per matrix between consecutive matrices: SoA planes are
  // offset as a whole (ld is unchanged), AoS rows are packed
  const int64_t w_in = layout == 0 ? 1 : (layout == 1 ? 6 : 9);
  const int64_t w_lam = layout == 0 ? 1 : 3, w_v = layout == 0 ? 1 : 9;
  for (int64_t s = 0; s < n; s += kMaxPerLaunch) {
    const int64_t m = n - s < kMaxPerLaunch ? n - s : kMaxPerLaunch;
    const T* As = (const T*)A + s * w_in;
    T* ls = (T*)lambda + s * w_lam;
    T* Vs = V ? (T*)V + s * w_v : nullptr;
    int32_t* is = info ? info + s : nullptr;
    hipError_t e;
    if (V) {
      e = info ? launch_t<FORM, true, true>(m, As, ld, layout, ls, Vs, flags, is, stream)
               : launch_t<FORM, true, false>(m, As, ld, layout, ls, Vs, flags, is, stream);
    } else {
      e = info ? launch_t<FORM, false, true>(m, As, ld, layout, ls, Vs, flags, is, stream)
               : launch_t<FORM, false, false>(m, As, ld, layout, ls, Vs, flags, is, stream);
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_batched(int64_t n, const void* A, Strides ld, int layout,
                          void* lambda, void* V, int dtype, uint32_t flags,
                          int32_t* info, hipStream_t stream) {
  if (dtype == kFormF64)
    return launch_dt<kFormF64>(n, A, ld, layout, lambda, V, flags, info, stream);
  if (dtype == kFormF32R)
    return launch_dt<kFormF32R>(n, A, ld, layout, lambda, V, flags, info, stream);
  return launch_dt<kFormF32>(n, A, ld, layout, lambda, V, flags, info, stream);
}

// ---------------------------------------------------------------------------
// Serving: one launch solves every request of a tick.  A tile is kBlock
// matrices of one segment, so each wavefront runs one dtype and one code
// path; the launch has one workgroup per tile unless its grid is capped, in
// which case workgroups stride over the tiles.  Per-matrix arithmetic is
// exactly the batched kernels' (eigenvalues do not depend on whether
// vectors are formed).
// ---------------------------------------------------------------------------
// One tile of segment s: matrices t0 .. t0 + kBlock - 1.  The tile's first
// matrix is folded into the plane bases (uniform, in scalar registers), so
// each lane adds only threadIdx.x elements as a 32-bit byte offset, whatever
// the request's size: every load and store of the solve is a global access
// of a scalar base and that offset, as in the batched SoA kernel (empty asm
// statements keep the bases scalar and the offset 32-bit; only the NaN path
// forms full addresses).  Both forms share one solve, which always forms the
// vectors: a request's type and whether it wants them (V null) are uniform
// branches around the loads and stores.  Plain accesses, as most requests'
// planes share lines (see motion()).  Bound by HBM and the search's latency
// ahead of each tile's loads: 200 requests of 2^U(0,20) matrices (2^24 in
// all, half of them in FP32 storage) 366 us, 4.8 TB/s; 481 us with a solve
// per form, non-temporal accesses, launch order and a search through the
// segments themselves.
template <typename T>
using GlobalT = __attribute__((address_space(1))) T;

// The table's pointers are generic: cast to global memory, else every access
// is a flat one with a 64-bit address per lane.
template <typename T, int N>
__device__ __forceinline__ void load_planes(double (&a)[N], const GlobalT<char>* base,
                                            int64_t pitch, uint32_t off) {
#pragma unroll
  for (int k = 0; k < N; ++k) {
    // each plane's base pinned in scalar registers (else the compiler chains
    // the planes' addresses per lane in 64 bits)
    const GlobalT<char>* p = base + k * pitch;
    asm volatile("" : "+s"(p));
    a[k] = (double)*(const GlobalT<T>*)(p + off);
  }
}

template <typename T, int N>
__device__ __forceinline__ void store_planes(const double (&x)[N], GlobalT<char>* base,
                                             int64_t pitch, uint32_t off) {
#pragma unroll
  for (int k = 0; k < N; ++k) {
    GlobalT<char>* p = base + k * pitch;
    asm volatile("" : "+s"(p));
    *(GlobalT<T>*)(p + off) = (T)x[k];
  }
}

// A host segment's matrices: loaded from its planes in host memory and
// stored, bit for bit, to its planes in device memory.
template <typename T>
__device__ __forceinline__ void load_host_planes(double (&a)[6], const GlobalT<char>* host,
                                                 GlobalT<char>* base, int64_t pitch,
                                                 uint32_t off) {
  T raw[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) raw[k] = *(const GlobalT<T>*)(host + k * pitch + off);
#pragma unroll
  for (int k = 0; k < 6; ++k) *(GlobalT<T>*)(base + k * pitch + off) = raw[k];
#pragma unroll
  for (int k = 0; k < 6; ++k) a[k] = (double)raw[k];
}

// The host memory of a segment that has any.
struct HostSide {
  const void* A;
  void *lambda, *V;
};

template <bool HOST>
__device__ __forceinline__ void solve_segment_tile(const Segment& s, const HostSide& h,
                                                   int64_t t0) {
  const bool f32 = s.dtype != kFormF64;
  const int sh = f32 ? 2 : 3;  // log2 of the element size
  const int64_t pa = s.lda << sh, po = s.n << sh;
  const GlobalT<char>* A = (const GlobalT<char>*)s.A + (t0 << sh);
  GlobalT<char>* L = (GlobalT<char>*)s.lambda + (t0 << sh);
  GlobalT<char>* W = (GlobalT<char>*)s.V + (t0 << sh);
  const bool vecs = s.V != nullptr;
  uint32_t off = threadIdx.x << sh;
  asm volatile("" : "+v"(off));
  double a[6];
  if constexpr (HOST) {
    const GlobalT<char>* hA = (const GlobalT<char>*)h.A + (t0 << sh);
    if (f32) load_host_planes<float>(a, hA, (GlobalT<char>*)A, pa, off);
    else load_host_planes<double>(a, hA, (GlobalT<char>*)A, pa, off);
  } else {
    if (f32) load_planes<float>(a, A, pa, off);
    else load_planes<double>(a, A, pa, off);
  }
  double l[3], v[9];
  bool bad;
  solve3<true, kFormBoth>(a, s.flags, l, v, bad);
  if (bad) {  // a NaN or infinite entry: NaN in every output of the matrix
#pragma unroll
    for (int j = 0; j < 3; ++j) l[j] = qnan<double>();
#pragma unroll
    for (int k = 0; k < 9; ++k) v[k] = qnan<double>();
  }
  uint32_t soff = off;
  asm volatile("" : "+v"(soff));
  const auto store = [&](GlobalT<char>* lam, GlobalT<char>* vec, bool with_vec) {
    if (f32) {
      store_planes<float>(l, lam, po, soff);
      if (with_vec) store_planes<float>(v, vec, po, soff);
    } else {
      store_planes<double>(l, lam, po, soff);
      if (with_vec) store_planes<double>(v, vec, po, soff);
    }
  };
  if constexpr (HOST)
    store((GlobalT<char>*)h.lambda + (t0 << sh), (GlobalT<char>*)h.V + (t0 << sh),
          h.V != nullptr);
  store(L, W, vecs);
}

// The chunked order from here on: 4096 tiles, 200 stress-mix requests of
// 2^U(0,20) matrices (57 K tiles, planes mostly unaligned) 349 us against 367
// in launch order; 1024 requests of 2^U(0,10) (1364 tiles) 9.1 against 8.4.
constexpr int64_t kSegmentsChunkFrom = 4096;

// begin: the segments' first tiles, ascending; LOADS of them per lane and
// round of the search.  solve(i, tile): solves this tile of segment i.
template <int LOADS, typename Begins, typename Solve>
__device__ __forceinline__ void solve_segments(int nseg, int64_t total_tiles, Begins begin,
                                               Solve solve) {
  // A tile's segment is the last whose first tile is at or before it
  // (uniform across the workgroup).  Its index is the count of segments
  // starting at or before the tile, minus one: each lane tests LOADS segments
  // and ballots count them, kRound per round, with the loads in flight
  // together.  A round not all of whose segments start at or before the tile
  // is the last.  A workgroup's tiles ascend, so its next search starts at
  // the round that held this tile's segment.
  constexpr int kRound = LOADS * kWave;
  // with one workgroup per tile, neighbouring tiles on one XCD
  Order order{0, 5};
  if (total_tiles >= kSegmentsChunkFrom && total_tiles <= (int64_t)gridDim.x)
    order.chunked = (uint32_t)total_tiles / (kXcds << 5) * (kXcds << 5);
  int from = 0;  // a multiple of kRound; every segment before it qualifies
  for (int64_t slot = blockIdx.x; slot < total_tiles; slot += gridDim.x) {
    const int64_t tile = order.chunked ? (int64_t)tile_of_block((uint32_t)slot, order) : slot;
    int cnt = from;
    for (int base = from; base < nseg; base += kRound) {
      int64_t tb[LOADS];
#pragma unroll
      for (int u = 0; u < LOADS; ++u) {
        const int j = base + u * kWave + (int)(threadIdx.x % kWave);
        tb[u] = j < nseg ? begin[j] : INT64_MAX;
      }
      int c = 0;
#pragma unroll
      for (int u = 0; u < LOADS; ++u) c += __popcll(__ballot(tb[u] <= tile));
      cnt += c;
      if (c < kRound) break;
    }
    const int lo = cnt - 1;
    from = lo / kRound * kRound;
    solve(lo, tile);
  }
}

// A table's segment, field by field (in scalar registers).
template <typename Seg>
__device__ __forceinline__ Segment read_segment(Seg* g) {
  Segment s;
  s.A = g->A;
  s.lambda = g->lambda;
  s.V = g->V;
  s.n = g->n;
  s.lda = g->lda;
  s.tile_begin = g->tile_begin;
  s.dtype = g->dtype;
  s.flags = g->flags;
  return s;
}

// The server admits the FP64 and the refined FP32 form.
template <bool HOST>
__device__ __forceinline__ void solve_tile_of(const Segment& s, const HostSide& h,
                                              int64_t tile) {
  const int64_t t0 = (tile - s.tile_begin) * kBlock;  // the tile's first matrix
  if (t0 + threadIdx.x < s.n) solve_segment_tile<HOST>(s, h, t0);
}

__global__ __launch_bounds__(kBlock) void k_syev3_segments(const TickTable* __restrict__ t) {
  solve_segments<4>(t->nseg, t->total_tiles, table_begins(t), [&](int i, int64_t tile) {
    solve_tile_of<false>(read_segment(&t->seg[i]), HostSide{}, tile);
  });
}

// The table is the kernel's argument, read where the launch put it (indexed
// as a parameter it could be copied to scratch memory).
__global__ __launch_bounds__(kBlock) void k_syev3_segments_inline(InlineTable) {
  using Arg = const __attribute__((address_space(4))) InlineTable;
  Arg* t = (Arg*)__builtin_amdgcn_kernarg_segment_ptr();
  solve_segments<1>(t->nseg, t->total_tiles, t->begin, [&](int i, int64_t tile) {
    solve_tile_of<false>(read_segment(&t->seg[i]), HostSide{}, tile);
  });
}

// Bound by the host link, whose two directions run at once: one FP64 request
// of 400 K matrices with vectors, 38 MB back, 784 us (49 GB/s; a large copy
// alone reaches 57) against 1116 for a copy in, the solve and two copies
// back; 100 matrices 29 us against 66.  Few workgroups keep the link full,
// and the other compute units free for other ticks' kernels: 2^21 matrices
// 3830 us with 32 of them, 3826 with 128, 3872 with 512, 3976 with 2048;
// 400 K 784, 791, 837, 911.
constexpr int kHostBlocks = 64;

__global__ __launch_bounds__(kBlock) void k_syev3_segments_host(HostTable) {
  using Arg = const __attribute__((address_space(4))) HostTable;
  Arg* t = (Arg*)__builtin_amdgcn_kernarg_segment_ptr();
  // whatever these caches hold of the host's memory may be out of date
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
  solve_segments<1>(t->nseg, t->total_tiles, t->begin, [&](int i, int64_t tile) {
    const HostSide h{t->seg[i].A, t->seg[i].lambda, t->seg[i].V};
    solve_tile_of<true>(read_segment(&t->seg[i].s), h, tile);
  });
}

hipError_t launch_segments(const TickTable* table, int32_t grid_blocks,
                           hipStream_t stream) {
  hipLaunchKernelGGL(k_syev3_segments, dim3((unsigned)grid_blocks), dim3(kBlock), 0,
                     stream, table);
  return hipGetLastError();
}

hipError_t launch_segments_inline(const InlineTable& table, int32_t grid_blocks,
                                  hipStream_t stream) {
  hipLaunchKernelGGL(k_syev3_segments_inline, dim3((unsigned)grid_blocks), dim3(kBlock), 0,
                     stream, table);
  return hipGetLastError();
}

hipError_t launch_segments_host(const HostTable& table, int32_t max_blocks,
                                hipStream_t stream) {
  const int64_t grid =
      std::min<int64_t>(table.total_tiles, std::min<int32_t>(kHostBlocks, max_blocks));
  (void)hipGetLastError();  // read below: drop any stale error
  hipLaunchKernelGGL(k_syev3_segments_host, dim3((unsigned)grid), dim3(kBlock), 0, stream,
                     table);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Streaming probes: the SoA kernel's loads (RD) and/or stores (WR), with a
// sum in place of the solve, in launch order or in the solver's XCD-chunked
// workgroup order.  A read-only probe's one store is taken only for a NaN
// sum, so its loads are kept and it writes nothing for finite input.  RD and
// WR together in launch order is the streaming reference.
// ---------------------------------------------------------------------------
template <typename T, bool VECS, bool RD, bool WR, bool XCD>
__global__ __launch_bounds__(kBlock) void k_stream_reference(int64_t n, const T* __restrict__ A,
                                                             T* __restrict__ lam,
                                                             T* __restrict__ V,
                                                             Order order) {
  const uint32_t b = XCD ? tile_of_block(blockIdx.x, order) : blockIdx.x;
  const int64_t i = (int64_t)b * kBlock + threadIdx.x;
  if (i >= n) return;
  T s = RD ? (T)0 : (T)threadIdx.x;
  if (RD) {
#pragma unroll
    for (int k = 0; k < 6; ++k) s += ld<true>(A + k * n + i);
  }
  if (WR) {
#pragma unroll
    for (int j = 0; j < 3; ++j) st<true>(s * (T)(j + 1), lam + j * n + i);
    if (VECS) {
#pragma unroll
      for (int k = 0; k < 9; ++k) st<true>(s * (T)(k + 4), V + k * n + i);
    }
  } else if (__builtin_isnan(s)) {
    lam[i] = s;
  }
}

template <typename T, bool VECS>
static hipError_t launch_probe_t(int64_t n, const T* A, T* lambda, T* V, uint32_t mode,
                                 hipStream_t stream) {
  const dim3 grid((unsigned)((n + kBlock - 1) / kBlock)), block(kBlock);
  const bool rd = mode & 1u, wr = mode & 2u, xcd = mode & 4u;
  const Order order = chunked_order(grid.x, 8);
#define SYEV3_PROBE_CASE(R, W, X)                                                         \
  if (rd == R && wr == W && xcd == X) {                                                   \
    hipLaunchKernelGGL((k_stream_reference<T, VECS, R, W, X>), grid, block, 0, stream, n, \
                       A, lambda, V, order);                                              \
    return hipGetLastError();                                                             \
  }
  SYEV3_PROBE_CASE(true, true, false)
  SYEV3_PROBE_CASE(true, true, true)
  SYEV3_PROBE_CASE(true, false, false)
  SYEV3_PROBE_CASE(true, false, true)
  SYEV3_PROBE_CASE(false, true, false)
  SYEV3_PROBE_CASE(false, true, true)
#undef SYEV3_PROBE_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_stream_probe(int64_t n, const void* A, void* lambda, void* V, int dtype,
                               uint32_t mode, hipStream_t stream) {
  // the kernel's planes are n apart, so a split batch is not expressible:
  // the probes are for batches one launch can hold
  if (n > kMaxPerLaunch) return hipErrorInvalidValue;
  if (dtype == 0) {
    return V ? launch_probe_t<double, true>(n, (const double*)A, (double*)lambda, (double*)V,
                                            mode, stream)
             : launch_probe_t<double, false>(n, (const double*)A, (double*)lambda, nullptr,
                                             mode, stream);
  }
  return V ? launch_probe_t<float, true>(n, (const float*)A, (float*)lambda, (float*)V, mode,
                                         stream)
           : launch_probe_t<float, false>(n, (const float*)A, (float*)lambda, nullptr, mode,
                                          stream);
}

}  // namespace syev3
