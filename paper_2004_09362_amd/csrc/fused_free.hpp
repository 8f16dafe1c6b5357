// fused_free.hpp -- the fused kernel of int32 plans, whose results do not
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
// Instantiated for every P = 2..128 in the units that build.py writes.
//
// Bound by HBM (P reads and P writes, or one, of every column; one operation
// per element); the widths, caps and store kinds are chosen in
// free_shape.hpp, with what they measured.
#pragma once

#include "device_common.hpp"

namespace ar {

// All P rows of a lane's columns are loaded before the first combination.
// How a lane finds its columns: without gaps (one instance, or several back
// to back) lane g takes the elements from g * V on; with gaps, group g mod
// gpi of instance g / gpi, in 32 bits where the groups fit.
template <int P, int V, int OP, bool NT>
__global__ __launch_bounds__(kBlock) void fused_free_kernel(const FreeArgs a) {
  for (uint64_t t = blockIdx.x; t < a.blocks; t += gridDim.x) {
    // tbl is a.user (t < 2^62); indexing it by t >> 62 keeps the compiler from
    // hoisting the P rank pointers out of the loop, where they would be
    // spilled to VGPR lanes
    void* const* tbl = a.user + (t >> 62);
    const uint64_t g = t * kBlock + threadIdx.x;
    uint64_t j = g;
    int64_t e = int64_t(g) * V;
    if (a.gaps) {
      const uint64_t inst = a.gaps == 1 ? uint64_t(fdiv(uint32_t(g), a.gdiv)) : g / uint64_t(a.gpi);
      j = g - inst * uint64_t(a.gpi);
      e = int64_t(inst) * a.stride + int64_t(j) * V;
    }
    if (g < uint64_t(a.groups)) {
      const int64_t left = a.n - int64_t(j) * V;  // elements of the instance from the lane's first on
      if (V == 1 || left >= V) {
        int32_t x[P][V];
#pragma unroll
        for (int y = 0; y < P; ++y) ldv<V, NT>(x[y], static_cast<const int32_t*>(tbl[y]) + e);
#pragma unroll
        for (int y = 1; y < P; ++y) {
#pragma unroll
          for (int i = 0; i < V; ++i) x[0][i] = comb<OP>(x[0][i], x[y][i]);
        }
        if (a.split) {
          stv<V, NT>(static_cast<int32_t*>(tbl[0]) + e, x[0]);
        } else {
#pragma unroll
          for (int y = 0; y < P; ++y) stv<V, NT>(static_cast<int32_t*>(tbl[y]) + e, x[0]);
        }
      } else {  // the last elements of an instance, fewer than V
        for (int64_t i = 0; i < left; ++i) {
          int32_t acc = static_cast<const int32_t*>(tbl[0])[e + i];
#pragma unroll 8
          for (int y = 1; y < P; ++y) acc = comb<OP>(acc, static_cast<const int32_t*>(tbl[y])[e + i]);
          static_cast<int32_t*>(tbl[0])[e + i] = acc;
          if (!a.split) {
#pragma unroll 8
            for (int y = 1; y < P; ++y) static_cast<int32_t*>(tbl[y])[e + i] = acc;
          }
        }
      }
    }
  }
}

// Elements per lane that P's instantiations offer: 1, 2 up to 65 ranks, 4 up
// to 16 (a lane holds P * V values).
template <int P, int V>
int launch_free_v(const FreeArgs& a, int op, bool nt, int grid, uint32_t lds, hipStream_t s) {
  const dim3 g(grid), blk(kBlock);
  if (op == 0) {
    if (nt) hipLaunchKernelGGL((fused_free_kernel<P, V, 0, true>), g, blk, lds, s, a);
    else hipLaunchKernelGGL((fused_free_kernel<P, V, 0, false>), g, blk, lds, s, a);
  } else {
    if (nt) hipLaunchKernelGGL((fused_free_kernel<P, V, 1, true>), g, blk, lds, s, a);
    else hipLaunchKernelGGL((fused_free_kernel<P, V, 1, false>), g, blk, lds, s, a);
  }
  return int(hipGetLastError());
}

template <int P>
int launch_free_at(const FreeArgs& a, int V, int op, bool nt, int grid, uint32_t lds, void* stream) {
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  if constexpr (P <= 16)
    if (V == 4) return launch_free_v<P, 4>(a, op, nt, grid, lds, s);
  if constexpr (P <= 65)
    if (V == 2) return launch_free_v<P, 2>(a, op, nt, grid, lds, s);
  return V == 1 ? launch_free_v<P, 1>(a, op, nt, grid, lds, s) : int(hipErrorInvalidValue);
}

}  // namespace ar
