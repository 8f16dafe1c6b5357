// broadcast.hip -- second half of a split column-fused launch.
//
// For the schedules whose distribution phase hands every rank the same
// result (bandwidth-optimal plans of Sec. 7 in either group, and the Ring of
// Sec. 6), the column kernels can store every column's result on rank 0
// alone; the broadcast then copies rank 0's columns to ranks 1, ..., P-1.
// The copy moves the bytes the distribution phase moves, and one more read
// of each column and one fewer write of it than the single fused launch
// (the reducing launch's).  It pays because a launch that reads P streams
// and writes P streams at once interleaves reads and writes across hundreds
// of DRAM rows, while a reducing launch (P reads, one write) and the
// broadcast (one read, P - 1 writes) each stream in one direction.
//
// broadcast_kernel, the tiled copy: tiles as in the reducing launch
// (col_tile_column, device_common.hpp), or 64 consecutive flat columns per
// wave; every wave writes the P - 1 destinations of its columns.  It serves
// the calls the kernel below does not: rank spans under the size rule of
// capi.cpp, and index spaces beyond 32 bits.  Loads and stores are
// nontemporal (NT) or ordinary: from P = 96 ranks, streaming the P - 1
// stores nontemporally at one resident workgroup per CU was 3-4% faster, and
// on flat columns nontemporal stores were 1-11% faster at any P; below
// P = 96 on block tiles, ordinary stores streamed as fast or faster.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>

#include "ar_internal.hpp"
#include "device_common.hpp"

namespace ar {

namespace {

template <typename T, bool NT>
__global__ __launch_bounds__(kBlock) void broadcast_kernel(const ColArgs a) {
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t wave_in_block = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int32_t P = a.P;
  for (uint32_t t = blockIdx.x * uint32_t(kWavesPerBlock) + wave_in_block; t < a.total_tiles;
       t += gridDim.x * uint32_t(kWavesPerBlock)) {
    int64_t e;
    bool live;
    if (a.flat) {
      const uint32_t g = t * uint32_t(kWave) + uint32_t(lane);
      const uint32_t inst = fdiv(g, a.ndiv);
      e = int64_t(inst) * a.stride + int64_t(g - inst * a.ndiv.d);
      live = g < a.flat_cols;
    } else {
      int32_t b;
      live = col_tile_column(a, t, lane, b, e);
    }
    if (live) {
      const T v = ld1<NT>(static_cast<const T*>(a.user[0]) + e);
#pragma unroll 8
      for (int32_t d = 1; d < P; ++d) st1<NT>(static_cast<T*>(a.user[d]) + e, v);
    }
  }
}

// Destination-major copy.  The kernel above writes the P - 1 destinations
// of a column tile at once, so the stores in flight hit P - 1 rank buffers
// (256 MB apart at P = 127, n = 2^26) and HBM writes them at 5.8 TB/s.  Here
// workgroup ids run slice by slice, destination by destination, chunk by
// chunk: the workgroups in flight sweep one destination's buffer in address
// order, and each thread copies 16 bytes once and exits.  A slice's source
// columns are read from HBM once and then from L2 for the other
// destinations: workgroup ids go round-robin over the XCDs, so with C chunks
// per slice a multiple of the XCD count X, workgroup c of a slice runs on
// XCD c mod X for every destination.  The chunk it copies is chunk c
// (interleaved: 1 MB of each slice per XCD, in 4 KB pieces X chunks apart),
// or in XCD regions the ((c mod X) * C / X + c / X)-th (XCD x copies the x-th
// contiguous C / X chunks: 256 KB of each slice).  With C not a multiple of
// X the copy took 1.3x the time, and with 2 MB per XCD 1.4x.
//
// Rank buffers need no common alignment: each destination has its own chunk
// grid, laid on the 128-byte lines of its buffer (its first chunk starts up
// to 31 columns before column 0), so that every store but those of its two
// ends covers whole lines, and the unaligned side is the source's, which L2
// serves.  What bounds the copy is the stores; a store that straddled lines
// wrote each of them twice.  Rows packed back to back at an odd length, 1 GB
// in all, P = 8-127: 6.4-7.6 TB/s, the rate of rows on line boundaries, where
// chunks on a common grid (the same column for every destination) moved
// 5.2-6.8 and the tiled copy, which such calls took before, 2.6-3.3.
//
// All sources are rank 0's row: a chunk has one source whatever the blocks,
// with no look-up of its root.  (With block b's result on rank b, a chunk
// across a block boundary needed two loads and a select per element.)
//
// GAP: instances with a gap between them (stride > n).  The column space is
// then the memory span of a rank's instances, and a 16-byte group that
// touches a gap is copied element by element, which leaves the gap as it is.
//
// A workgroup does little besides its index arithmetic, so that arithmetic
// has no branch before the bounds check and its words lie first and
// together: one load of the kernel's arguments, one of the two rank
// pointers, then the copy.  (With the chunk order behind a branch and the
// words apart, and the second pointer loaded after the check, the copy took
// 2-5% longer.)  LINES = false, every destination on a line boundary, is
// kept for the same reason: its bounds check waits for no pointer.
struct BcastArgs {
  StreamDiv sdiv, cdiv;  // C * P, C (chunks per slice, a multiple of the XCD count X)
  // chunk of workgroup c of a slice: (c & mask) * per_xcd + (c >> shift) --
  // regions: X - 1, C / X, log2 X; interleaved (chunk c itself): 0, 0, 0
  uint32_t mask, per_xcd, shift;
  uint32_t chunks;  // chunks of the longest destination grid
  uint32_t cols;    // columns of a rank's span: (instances - 1) * stride + n
  uint32_t n;       // GAP: instance length
  uint32_t P;
  StreamDiv stdiv;  // GAP: the instance stride
  void* user[kMaxP];
};

__device__ __forceinline__ uint32_t sdiv(uint32_t n, const StreamDiv& d) {
  const uint32_t t = __umulhi(n, d.mul);
  return (t + ((n - t) >> d.s1)) >> d.s2;
}

// 16 bytes at any 4-byte boundary (global memory takes such accesses whole).
typedef int32_t i32x4u __attribute__((ext_vector_type(4), aligned(4)));

// LINES: the chunk grid of a destination starts on a 128-byte line of its
// buffer; else on column 0.
template <bool NT, bool GAP, bool LINES>
__global__ __launch_bounds__(kStreamBlock) void broadcast_stream_kernel(const BcastArgs a) {
  const uint32_t id = blockIdx.x;
  const uint32_t s = sdiv(id, a.sdiv);
  const uint32_t r = id - s * a.sdiv.d;
  const uint32_t y = sdiv(r, a.cdiv);
  const uint32_t c = r - y * a.cdiv.d;  // workgroup c of the slice runs on XCD c mod X
  const uint32_t chunk = s * a.cdiv.d + (c & a.mask) * a.per_xcd + (c >> a.shift);
  int32_t* const row = static_cast<int32_t*>(a.user[y]);
  const int32_t* const row0 = static_cast<const int32_t*>(a.user[0]);
  uint32_t ph = 0;
  if constexpr (LINES) {
    ph = uint32_t(reinterpret_cast<uintptr_t>(row) >> 2) & 31u;
    asm volatile("" ::"s"(row0));  // both pointers are loaded before the check that needs one of them
  }
  // Positions are columns plus ph, so position 0 is the start of a line;
  // positions [ph, cols + ph) hold columns.  What is left of the span from
  // the chunk's start on is compared, not positions past it: near 2^32
  // columns those wrap.
  const uint32_t u0 = chunk * kStreamChunk;
  if ((chunk >= a.chunks) | (y == 0) | (u0 >= a.cols + ph)) return;
  const uint32_t left = a.cols + ph - u0;
  const uint32_t v = threadIdx.x * 4u;
  const int64_t e0 = int64_t(u0) - int64_t(ph);  // the chunk's first column (below 0: the grid's lead)
  int32_t* dst = row + e0 + v;
  const int32_t* src = row0 + e0 + v;
  bool whole = left >= kStreamChunk && u0 >= ph;
  uint32_t i0 = 0;
  if constexpr (GAP) {
    whole = u0 + v >= ph && v + 4u <= left;
    if (whole) {
      const uint32_t m = u0 + v - ph;
      i0 = m - sdiv(m, a.stdiv) * a.stdiv.d;
      whole = i0 + 4u <= a.n;
    }
  }
  if (whole) {
    const i32x4 w = *reinterpret_cast<const i32x4u*>(src);
    if constexpr (NT) __builtin_nontemporal_store(i32x4u(w), reinterpret_cast<i32x4u*>(dst));
    else *reinterpret_cast<i32x4u*>(dst) = w;
    return;
  }
  // the two ends of the span, and groups that touch a gap
#pragma unroll
  for (uint32_t i = 0; i < 4; ++i) {
    bool live = u0 + v + i >= ph && v + i < left;
    if constexpr (GAP) {
      if (live) {
        const uint32_t m = u0 + v + i - ph;
        live = m - sdiv(m, a.stdiv) * a.stdiv.d < a.n;
      }
    }
    if (live) st1<NT>(dst + i, src[i]);
  }
}

// LDS that a workgroup of the copy reserves and does not use in regions
// order, so that four are resident on a CU, where eight fit: with fewer
// stores in flight each XCD's sweep stays in fewer DRAM rows.  P = 127 at 72 MB
// per rank: 7.38 against 7.16 TB/s (rows off the lines 7.19 against 6.79),
// P = 128 at 64 MB 7.37 against 7.15; three a CU: 6.4.  Interleaved chunks
// (one sweep for the whole chip) and copies with gaps ran within 2% either
// way or slower with it.
constexpr uint32_t kCopyLds = 39 * 1024;

void launch_copy(const BcastArgs& a, uint32_t grid, bool nt, bool gap, bool lines, hipStream_t s) {
  const dim3 g(grid), blk(kStreamBlock);
  const uint32_t lds = a.mask != 0 && !gap ? kCopyLds : 0;
#define AR_COPY(GAP, LINES)                                                                               \
  do {                                                                                                    \
    if (nt) hipLaunchKernelGGL((broadcast_stream_kernel<true, GAP, LINES>), g, blk, lds, s, a);             \
    else hipLaunchKernelGGL((broadcast_stream_kernel<false, GAP, LINES>), g, blk, lds, s, a);               \
  } while (0)
  if (gap) AR_COPY(true, true);
  else if (lines) AR_COPY(false, true);
  else AR_COPY(false, false);
#undef AR_COPY
}

// Launches the destination-major copy over a filled-in span, or returns
// false when its grid would reach 2^32 work-items.  The slices of a call are
// evened out and rounded up to the XCD count (a short last slice in regions
// leaves most XCDs idle): at most 1 MB per XCD interleaved, 256 KB in regions
// (at 8-32 MB per rank 1 MB regions ran 3-50% slower; from 64 MB the sizes ran
// within a few percent).
bool launch_dest_major(BcastArgs& a, uint32_t xcds, bool regions, bool gap, bool nt, hipStream_t s) {
  uint32_t shift = 0;
  while ((1u << shift) < xcds) ++shift;
  const bool reg = regions && (1u << shift) == xcds;
  bool lines = false;
  for (uint32_t x = 1; x < a.P; ++x) lines |= reinterpret_cast<uintptr_t>(a.user[x]) % 128 != 0;
  const uint64_t chunks = (uint64_t(a.cols) + (lines ? 31 : 0) + kStreamChunk - 1) / kStreamChunk;
  const uint64_t cmax = (reg ? 64u : 256u) * xcds;
  const uint64_t slices = (chunks + cmax - 1) / cmax;
  const uint64_t C = ((chunks + slices - 1) / slices + xcds - 1) / xcds * xcds;
  const uint64_t grid = (chunks + C - 1) / C * C * a.P;
  if (grid > uint64_t(UINT32_MAX) / kStreamBlock) return false;
  a.chunks = uint32_t(chunks);
  a.cdiv = stream_div(uint32_t(C));
  a.sdiv = stream_div(uint32_t(C) * a.P);
  a.mask = reg ? xcds - 1 : 0;
  a.shift = reg ? shift : 0;
  a.per_xcd = reg ? uint32_t(C) / xcds : 0;
  launch_copy(a, uint32_t(grid), nt, gap, lines, s);
  return true;
}

}  // namespace

constexpr int64_t kCopyRegionsMinBytes = int64_t(16) << 20;

int launch_broadcast_stream(const StreamArgs& a, bool nt, bool /*straddle*/, uint32_t grid, void* stream) {
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  BcastArgs b;
  std::memset(&b, 0, sizeof b);
  b.P = a.P;
  b.cols = a.cols;
  b.n = a.n;
  b.stdiv = StreamDiv{1, 0, 0, 0};
  std::memcpy(b.user, a.user, sizeof b.user);
  // every source on rank 0's row, the order no longer depends on the blocks:
  // unless it is forced, regions above kCopyRegionsMinBytes per rank, whose
  // slices then fill the chip (P = 127 at 256 MB: 4.67-4.70 ms against
  // 4.89-4.96 interleaved; at 18 MB 0.347-0.351 against 0.350-0.355, at 4.5 MB
  // 0.092 against 0.084)
  const bool regions = a.order_forced ? a.regions != 0 : int64_t(a.cols) * 4 > kCopyRegionsMinBytes;
  if (!launch_dest_major(b, 1u << a.xcd_shift, regions, false, nt, s)) {
    // a grid just below 2^32 work-items that the line-aligned grids' extra
    // chunk takes past it: the common grid
    b.chunks = a.chunks;
    b.cdiv = a.cdiv;
    b.sdiv = a.sdiv;
    b.mask = a.regions ? (1u << a.xcd_shift) - 1 : 0;
    b.shift = a.regions ? a.xcd_shift : 0;
    b.per_xcd = a.regions ? a.per_xcd : 0;
    launch_copy(b, grid, nt, false, false, s);
  }
  return int(hipGetLastError());
}

// Rank buffers off 16-byte boundaries, or gaps between the instances: the
// destination-major copy too wherever the size rule of capi.cpp asks for it
// (a.dest_major) and a rank's span fits its 32-bit positions.  With gaps,
// instances that start off 32-byte sectors (a stride that is no multiple of
// 8) or hold fewer than 512 elements take cached stores, which leave the
// parts of a line that different workgroups write to meet in L2, in
// interleaved order: P = 37, 65536 x 106, stride 113: 3.1 TB/s against 2.0
// nontemporal; P = 64, 8192 x 2304, stride 2311: 5.75 against 5.55; strides
// 2328 and 1024 the other way round, 5.5 against 6.2 and 5.25 against 6.0.
int launch_broadcast(const ColArgs& a, int dtype, bool nt, int grid, void* stream) {
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const int64_t span = (a.instances - 1) * a.stride + a.n;
  if (a.dest_major && span <= int64_t(UINT32_MAX) - 2 * kStreamChunk) {
    const bool gap = a.instances > 1 && a.stride != a.n;
    BcastArgs b;
    std::memset(&b, 0, sizeof b);
    b.P = uint32_t(a.P);
    b.cols = uint32_t(span);
    b.n = uint32_t(a.n);
    b.stdiv = stream_div(gap ? uint32_t(a.stride) : 1u);
    std::memcpy(b.user, a.user, sizeof b.user);
    const bool sectors = !gap || (a.stride % 8 == 0 && a.n >= 512);
    if (launch_dest_major(b, a.xcds, a.bcast_regions != 0 && sectors, gap, a.bcast_nt != 0 && sectors, s))
      return int(hipGetLastError());
  }
  const dim3 g(grid), blk(kBlock);
  if (dtype == 0) {
    if (nt) hipLaunchKernelGGL((broadcast_kernel<int32_t, true>), g, blk, a.lds, s, a);
    else hipLaunchKernelGGL((broadcast_kernel<int32_t, false>), g, blk, a.lds, s, a);
  } else {
    if (nt) hipLaunchKernelGGL((broadcast_kernel<float, true>), g, blk, a.lds, s, a);
    else hipLaunchKernelGGL((broadcast_kernel<float, false>), g, blk, a.lds, s, a);
  }
  return int(hipGetLastError());
}

}  // namespace ar
