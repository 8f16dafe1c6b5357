// fused_free.hip -- the fused kernel of int32 plans, whose results do not
// depend on the schedule.
//
// Kolmakov & Zhang, "A Generalization of the Allreduce Operation"
// (arXiv:2004.09362), Sec. 5.4 asks of the combination that it be
// associative and commutative.  On int32 both combinations are exactly that,
// bit for bit (sums wrap modulo 2^32), so every schedule -- any k, either
// group, the Ring -- hands every rank the same value: the combination of the
// P values of a column in any order.  The fp32 kernels rotate ranks by block,
// keep 2^r different sums and tile by block only to reproduce each schedule's
// own rounding (and its choice among signed zeros and NaNs); none of it is
// needed here.  fused_free_kernel walks the columns as they lie in memory,
// V elements per lane, combines the P rows and stores the result to every
// rank, or with `split` to rank 0 alone (the broadcast copies it on).
//
// Bound by HBM (P reads and P writes, or one, of every column; one operation
// per element).  What it measured (int32, MI355X, TB/s of 2 * P * n * 4
// bytes; before: the fp32 plans' kernels), with the choices of free_shape:
//   P = 16, 4096 x 1000 at stride 1024, max, k = 6:  before 3.5
//   P = 127, 65536 x 106, max, k = 12:               before 0.12
// (see the table in free_shape for the widths).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>

#include "ar_internal.hpp"
#include "device_common.hpp"

namespace ar {

namespace {

struct FreeArgs {
  void* user[kMaxP];
  int32_t P, split;
  int64_t n, stride;   // instance length and stride; one span: the whole extent, any stride
  int64_t groups;      // lanes with work: instances * gpi
  int64_t gpi;         // groups of V elements per instance (the last one may hold fewer)
  FastDiv gdiv;        // gpi, for kGaps
};

// How a lane finds its columns: kSpan, one instance (or several without gaps
// between them), lane g at element g * V; kGaps, lane g at group g mod gpi of
// instance g / gpi, 32-bit; kGaps64, the same beyond 2^32 groups.
enum FreeMode { kSpan = 0, kGaps = 1, kGaps64 = 2 };

template <int V>
struct IntVec;
template <>
struct IntVec<1> {
  typedef int32_t U;
};
// at any 4-byte boundary: global memory takes such accesses whole
template <>
struct IntVec<2> {
  typedef int32_t U __attribute__((ext_vector_type(2), aligned(4)));
};
template <>
struct IntVec<4> {
  typedef int32_t U __attribute__((ext_vector_type(4), aligned(4)));
};

template <int V, bool NT>
__device__ __forceinline__ void free_load(int32_t (&x)[V], const int32_t* p) {
  using U = typename IntVec<V>::U;
  U u;
  if constexpr (NT) u = __builtin_nontemporal_load(reinterpret_cast<const U*>(p));
  else u = *reinterpret_cast<const U*>(p);
  if constexpr (V == 1) {
    x[0] = u;
  } else {
#pragma unroll
    for (int i = 0; i < V; ++i) x[i] = u[i];
  }
}

template <int V, bool NT>
__device__ __forceinline__ void free_store(int32_t* p, const int32_t (&x)[V]) {
  using U = typename IntVec<V>::U;
  U u;
  if constexpr (V == 1) {
    u = x[0];
  } else {
#pragma unroll
    for (int i = 0; i < V; ++i) u[i] = x[i];
  }
  if constexpr (NT) __builtin_nontemporal_store(u, reinterpret_cast<U*>(p));
  else *reinterpret_cast<U*>(p) = u;
}

// D: upper bound of P, P itself for EXACT.  Every load has a compile-time
// slot and, unless EXACT, a wave-uniform guard, so all P rows of a lane's
// columns are in flight before the first combination.
template <int D, bool EXACT, int V, int OP, bool NT, int MODE>
__global__ __launch_bounds__(kBlock) void fused_free_kernel(const FreeArgs a) {
  const int32_t P = EXACT ? D : a.P;
  const int64_t nthreads = int64_t(gridDim.x) * kBlock;
  for (int64_t g = int64_t(blockIdx.x) * kBlock + threadIdx.x; g < a.groups; g += nthreads) {
    int64_t e, j = g;
    if constexpr (MODE == kSpan) {
      e = g * V;
    } else {
      int64_t inst;
      if constexpr (MODE == kGaps) {
        const uint32_t q = fdiv(uint32_t(g), a.gdiv);
        inst = q;
      } else {
        inst = g / a.gpi;
      }
      j = g - inst * a.gpi;
      e = inst * a.stride + j * V;
    }
    if (V == 1 || a.n - j * V >= V) {
      int32_t x[D][V];
#pragma unroll
      for (int y = 0; y < D; ++y)
        if (EXACT || y < P) free_load<V, NT>(x[y], static_cast<const int32_t*>(a.user[y]) + e);
#pragma unroll
      for (int y = 1; y < D; ++y)
        if (EXACT || y < P) {
#pragma unroll
          for (int i = 0; i < V; ++i) x[0][i] = comb<OP>(x[0][i], x[y][i]);
        }
      if (a.split) {
        free_store<V, NT>(static_cast<int32_t*>(a.user[0]) + e, x[0]);
      } else {
#pragma unroll
        for (int y = 0; y < D; ++y)
          if (EXACT || y < P) free_store<V, NT>(static_cast<int32_t*>(a.user[y]) + e, x[0]);
      }
    } else {  // the last elements of an instance, fewer than V
      for (int64_t i = 0; i < a.n - j * V; ++i) {
        int32_t acc = static_cast<const int32_t*>(a.user[0])[e + i];
#pragma unroll 8
        for (int y = 1; y < P; ++y) acc = comb<OP>(acc, static_cast<const int32_t*>(a.user[y])[e + i]);
        static_cast<int32_t*>(a.user[0])[e + i] = acc;
        if (!a.split) {
#pragma unroll 8
          for (int y = 1; y < P; ++y) static_cast<int32_t*>(a.user[y])[e + i] = acc;
        }
      }
    }
  }
}

// The launch shape: elements per lane, nontemporal or cached accesses, and
// the LDS each workgroup reserves so that few are resident per CU (kernels
// that stream P rows in and out keep fewer DRAM rows open that way).
struct FreeShape {
  int V;
  bool nt;
  uint32_t lds;
};

// LDS that lets `cap` workgroups fit on a CU (160 KB), 0 for no cap.
constexpr uint32_t free_cap_lds(int cap) { return cap == 0 ? 0u : cap == 1 ? 84u * 1024 : (160u * 1024 / cap - 1024) / 512 * 512; }

// Measured on rows of 2^28 / P columns, TB/s of the bytes moved, on line
// boundaries / one behind the other at an odd length:
//   one launch (P reads, P writes): 16-byte lanes at one or two workgroups a
//     CU, P = 2 6.8 / 6.5 (4-byte lanes 6.2 / 5.8), P = 3 7.0 / 6.4 (6.7 /
//     5.5), P = 5 6.6 / 6.0, P = 8 6.35 / 5.8 (6.4 / 4.7), P = 16 6.5 / 5.6
//     (5.9 / 4.0); 8-byte lanes P = 24 6.0 / 5.3 (5.5 / 4.0), P = 32 6.4 / 5.6
//     (5.7 / 4.2); 4-byte lanes from P = 34, P = 48 5.9 / 5.3, P = 64 5.8 / 5.3,
//     P = 127 5.1 / 4.5 (8-byte lanes 5.4, 5.75, 5.2 / 4.7, 5.2, 4.5);
//   reducing launch (P reads, 1 write): 16-byte lanes at two a CU, P = 8 6.75 /
//     6.7, P = 16 6.7 / 6.6; 8-byte lanes at three, P = 24 6.7 / 6.3, P = 32 6.55 /
//     6.2, P = 48 6.5 / 6.2 and P = 64 6.3 / 5.9 (4-byte lanes 6.6 / 5.8 and 6.5 /
//     5.6); 4-byte lanes P = 127 6.5 / 5.4.
// Rows off the 128-byte lines: a nontemporal access that covers part of a
// line costs the whole line, so only the widest lanes keep them (single
// launches up to P = 8, the reducing launches' reads); the others leave the
// shared lines to meet in L2 (P = 13: 5.2 against 4.0).
FreeShape free_shape(int P, bool split, bool lines, bool big, int64_t n, bool gaps) {
  FreeShape s{};
  s.V = P <= 16 ? 4 : (P <= 33 || (split && !lines && P <= 65)) ? 2 : 1;
  // short instances between gaps: no lane may be left with a part of a group
  // (its elements go one by one)
  if (gaps && n < 4096)
    while (s.V > 1 && n % s.V != 0) s.V /= 2;
  s.nt = big && (lines || (split ? s.V >= 2 : s.V == 4 && P <= 8));
  int cap;
  if (split) cap = P <= 16 ? 2 : 3;
  else if (s.V == 4) cap = P == 2 ? 4 : P <= 4 ? 2 : 1;
  else if (s.V == 2) cap = P <= 4 ? 0 : P <= 16 ? 2 : 1;
  else cap = P <= 6 ? 0 : P <= 16 ? 4 : 2;
  s.lds = free_cap_lds(cap);
  return s;
}

template <int D, bool EXACT, int V>
int launch_free_v(const FreeArgs& a, int op, bool nt, int mode, int grid, uint32_t lds, hipStream_t s) {
  const dim3 g(grid), blk(kBlock);
#define AR_FREE(OP, NT, MODE) \
  hipLaunchKernelGGL((fused_free_kernel<D, EXACT, V, OP, NT, MODE>), g, blk, lds, s, a)
#define AR_FREE_OP(OP)                        \
  do {                                        \
    if (mode == kSpan) {                      \
      if (nt) AR_FREE(OP, true, kSpan);       \
      else AR_FREE(OP, false, kSpan);         \
    } else if (mode == kGaps) {               \
      if (nt) AR_FREE(OP, true, kGaps);       \
      else AR_FREE(OP, false, kGaps);         \
    } else if constexpr (V == 1) {            \
      AR_FREE(OP, false, kGaps64);            \
    } else {                                  \
      return int(hipErrorInvalidValue);       \
    }                                         \
  } while (0)
  if (op == 0) AR_FREE_OP(0);
  else AR_FREE_OP(1);
#undef AR_FREE_OP
#undef AR_FREE
  return int(hipGetLastError());
}

template <int D, bool EXACT, int VMAX>
int launch_free_d(const FreeArgs& a, int V, int op, bool nt, int mode, int grid, uint32_t lds, hipStream_t s) {
  if constexpr (VMAX >= 4)
    if (V == 4) return launch_free_v<D, EXACT, 4>(a, op, nt, mode, grid, lds, s);
  if constexpr (VMAX >= 2)
    if (V == 2) return launch_free_v<D, EXACT, 2>(a, op, nt, mode, grid, lds, s);
  return V == 1 ? launch_free_v<D, EXACT, 1>(a, op, nt, mode, grid, lds, s) : int(hipErrorInvalidValue);
}

int launch_free_p(const FreeArgs& a, int V, int op, bool nt, int mode, int grid, uint32_t lds, hipStream_t s) {
  switch (a.P) {
#define AR_FREE_CASE(PP) \
  case PP: return launch_free_d<PP, true, 4>(a, V, op, nt, mode, grid, lds, s);
    AR_FREE_CASE(2) AR_FREE_CASE(3) AR_FREE_CASE(4) AR_FREE_CASE(5) AR_FREE_CASE(6) AR_FREE_CASE(7) AR_FREE_CASE(8)
    AR_FREE_CASE(9) AR_FREE_CASE(10) AR_FREE_CASE(11) AR_FREE_CASE(12) AR_FREE_CASE(13) AR_FREE_CASE(14)
    AR_FREE_CASE(15) AR_FREE_CASE(16)
#undef AR_FREE_CASE
    default: break;
  }
  switch ((a.P - 2) / 16) {  // P = 17..33, 34..49, ... (the rows after the first in chunks of 16)
    case 0:
    case 1: return launch_free_d<33, false, 2>(a, V, op, nt, mode, grid, lds, s);
    case 2: return launch_free_d<49, false, 2>(a, V, op, nt, mode, grid, lds, s);
    case 3: return launch_free_d<65, false, 2>(a, V, op, nt, mode, grid, lds, s);
    case 4: return launch_free_d<81, false, 1>(a, V, op, nt, mode, grid, lds, s);
    case 5: return launch_free_d<97, false, 1>(a, V, op, nt, mode, grid, lds, s);
    case 6: return launch_free_d<113, false, 1>(a, V, op, nt, mode, grid, lds, s);
    case 7: return launch_free_d<128, false, 1>(a, V, op, nt, mode, grid, lds, s);
    default: return int(hipErrorInvalidValue);
  }
}

}  // namespace

int launch_fused_free(void* const* user, int P, int op, int64_t n, int64_t stride, int64_t instances, bool split,
                      const FusedTuning& tune, void* stream) {
  FreeArgs a;
  std::memset(&a, 0, sizeof a);
  bool lines = true;
  for (int x = 0; x < P; ++x) {
    a.user[x] = user[x];
    lines = lines && reinterpret_cast<uintptr_t>(user[x]) % 128 == 0;
  }
  const bool gaps = instances > 1 && stride != n;
  if (gaps && stride % 32 != 0) lines = false;
  a.P = P;
  a.split = split ? 1 : 0;
  a.n = gaps ? n : instances * n;
  a.stride = stride;
  FreeShape sh = free_shape(P, split, lines, tune.big, n, gaps);
  if (gaps && instances * ((n + sh.V - 1) / sh.V) >= int64_t(UINT32_MAX)) {  // 64-bit division, in one form only
    sh.V = 1;
    sh.nt = false;
  }
  a.gpi = (a.n + sh.V - 1) / sh.V;
  a.groups = (gaps ? instances : 1) * a.gpi;
  const int mode = !gaps ? kSpan : a.groups < int64_t(UINT32_MAX) ? kGaps : kGaps64;
  if (mode == kGaps) a.gdiv = make_fastdiv(uint32_t(a.gpi));
  if (tune.nt >= 0 && mode != kGaps64) sh.nt = tune.nt != 0;
  if (tune.cap_forced) sh.lds = tune.lds;
  const int64_t blocks = (a.groups + kBlock - 1) / kBlock;
  const int grid = int(blocks < 1 ? 1 : blocks > kMaxGrid ? kMaxGrid : blocks);
  return launch_free_p(a, sh.V, op, sh.nt, mode, grid, sh.lds, reinterpret_cast<hipStream_t>(stream));
}

}  // namespace ar
