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
// capi.cpp (copy_call), and index spaces beyond 32 bits.  Loads and stores are
// nontemporal (NT) or ordinary: from P = 96 ranks, streaming the P - 1
// stores nontemporally at one resident workgroup per CU was 3-4% faster, and
// on flat columns nontemporal stores were 1-11% faster at any P; below
// P = 96 on block tiles, ordinary stores streamed as fast or faster.
#include <hip/hip_runtime.h>

#include <cstdint>

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
// contiguous C / X chunks of each slice).  With C not a multiple of X the copy
// took 1.3x the time, and with 2 MB per XCD 1.4x.  The order and C are the
// host's choice (copy_call, capi.cpp).
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
__device__ __forceinline__ uint32_t sdiv(uint32_t n, const StreamDiv& d) {
  const uint32_t t = __umulhi(n, d.mul);
  return (t + ((n - t) >> d.s1)) >> d.s2;
}

// 16 bytes at any 4-byte boundary (global memory takes such accesses whole).
typedef int32_t i32x4u __attribute__((ext_vector_type(4), aligned(4)));

// LINES: the chunk grid of a destination starts on a 128-byte line of its
// buffer; else on column 0.
template <bool NT, bool GAP, bool LINES>
__global__ __launch_bounds__(kStreamBlock) void broadcast_stream_kernel(const CopyArgs a) {
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
// P = 128 at 64 MB 7.37 against 7.15; three a CU: 6.4.  Interleaved chunks (one
// sweep for the whole chip) on the lines keep six: whole calls of 2-16 MiB per
// rank, P = 33-127, took 0.967-1.009 of the time that an earlier copy with more
// index arithmetic per workgroup took, without a cap 0.96-1.03 (100 ranks at 2 MiB 1.03,
// 64 at 5 MiB 1.017).  Off the lines, and with gaps, they ran within 2% either way
// or slower with a cap.
constexpr uint32_t kCopyLds = 39 * 1024, kCopyInterleavedLds = 26 * 1024;

}  // namespace

int launch_copy(const CopyArgs& a, uint32_t grid, bool nt, bool gap, bool lines, void* stream) {
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const dim3 g(grid), blk(kStreamBlock);
  const uint32_t lds = gap ? 0 : a.mask != 0 ? kCopyLds : lines ? 0 : kCopyInterleavedLds;
#define AR_COPY(GAP, LINES)                                                                               \
  do {                                                                                                    \
    if (nt) hipLaunchKernelGGL((broadcast_stream_kernel<true, GAP, LINES>), g, blk, lds, s, a);             \
    else hipLaunchKernelGGL((broadcast_stream_kernel<false, GAP, LINES>), g, blk, lds, s, a);               \
  } while (0)
  if (gap) AR_COPY(true, true);
  else if (lines) AR_COPY(false, true);
  else AR_COPY(false, false);
#undef AR_COPY
  return int(hipGetLastError());
}

int launch_broadcast(const ColArgs& a, int dtype, bool nt, int grid, void* stream) {
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
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
