// fused_lo.hip -- the fused latency-optimal kernel for small P.
//
// Kolmakov & Zhang, "A Generalization of the Allreduce Operation"
// (arXiv:2004.09362), Sec. 9.  fused_lo_kernel runs the whole
// latency-optimal schedule for one column of P values held in registers:
// the primed vector R[x] and the starred S[x] of every rank, updated as the
// reduction steps prescribe, then S[x] written to rank x.  The pairs
// combined are exactly those of the step-by-step path, so the results are
// bit-identical, but each input is read once and each output written once
// (2*P*n elements).  The latency-optimal tree of rank x is the same for
// every block, so many small instances form one flat column space with no
// block index: the kernel for many independent small messages (Sec. 1's
// 425-byte average).  fp32 only (int32 plans: fused_free.hip).
//
// Compiled with packed-fp32 instructions disabled; only adds and compares.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "ar_internal.hpp"
#include "device_common.hpp"

namespace ar {

namespace {

constexpr int lo_L(int P) {
  int L = 0;
  while ((1 << L) < P) ++L;
  return L;
}
constexpr int lo_N(int P, int i) {
  int N = P;
  for (int j = 0; j < i; ++j) N -= N / 2;
  return N;
}

// Reduction step I of the latency-optimal schedule on one column: with
// f = floor(N_I/2), every rank receives the primed vector of rank x + f;
// starred sums take it on even N_I, primed sums on every step but the last.
// Before the first odd step S and R hold the same values, and the compiler
// computes their identical combinations once.
template <int P, int I, int OP, typename V>
__device__ __forceinline__ void lo_steps(V (&R)[P], V (&S)[P]) {
  constexpr int L = lo_L(P);
  if constexpr (I < L) {
    constexpr int N = lo_N(P, I);
    constexpr int f = N / 2;
    constexpr bool even = (N % 2) == 0;
    constexpr bool last = (I == L - 1);
    V Rn[P];
#pragma unroll
    for (int x = 0; x < P; ++x) {
      const V recv = R[(x + f) % P];
      if constexpr (even) S[x] = comb<OP>(S[x], recv);
      if constexpr (!last) Rn[x] = comb<OP>(R[x], recv);
    }
    if constexpr (!last) {
#pragma unroll
      for (int x = 0; x < P; ++x) R[x] = Rn[x];
    }
    lo_steps<P, I + 1, OP, V>(R, S);
  }
}

// One lane's V columns from element e on.
template <int P, int OP, int V, bool NT>
__device__ __forceinline__ void lo_cols(const FusedArgs& a, int64_t e) {
  float x[P][V];
#pragma unroll
  for (int y = 0; y < P; ++y) ldv<V, NT>(x[y], static_cast<const float*>(a.user[y]) + e);
#pragma unroll
  for (int i = 0; i < V; ++i) {
    float R[P], S[P];
#pragma unroll
    for (int y = 0; y < P; ++y) R[y] = S[y] = x[y][i];
    lo_steps<P, 0, OP, float>(R, S);
#pragma unroll
    for (int y = 0; y < P; ++y) x[y][i] = S[y];
  }
#pragma unroll
  for (int y = 0; y < P; ++y) stv<V, NT>(static_cast<float*>(a.user[y]) + e, x[y]);
}

// GAPS false: instances back to back, lane g takes the V columns from g * V on
// (a.groups columns in all).  GAPS true: any instance stride, column g is
// element g % n of instance g / n, V = 1; the division in 32 bits (a.ndiv)
// where the columns fit.
template <int P, int OP, int V, bool NT, bool GAPS>
__global__ __launch_bounds__(kBlock) void fused_lo_kernel(const FusedArgs a) {
  const int64_t step = int64_t(gridDim.x) * kBlock * V;
  for (int64_t g = (int64_t(blockIdx.x) * kBlock + threadIdx.x) * V; g < a.groups; g += step) {
    if constexpr (GAPS) {
      const int64_t inst = a.groups <= int64_t(UINT32_MAX) ? int64_t(fdiv(uint32_t(g), a.ndiv)) : g / a.n;
      lo_cols<P, OP, 1, NT>(a, inst * a.stride + (g - inst * a.n));
    } else if (V == 1 || g + V <= a.groups) {
      lo_cols<P, OP, V, NT>(a, g);
    } else {
      for (int64_t i = g; i < a.groups; ++i) lo_cols<P, OP, 1, NT>(a, i);
    }
  }
}

// Columns per lane: four up to three ranks (4-byte lanes leave the memory
// system short of requests: 2^26 elements, P = 2 5.9 / 6.5 TB/s, P = 3 6.7 / 6.7) and
// up to eight where the rows are off the 128-byte lines (P = 3 5.4 / 6.05, P = 5
// 5.15 / 5.8, P = 8 4.6 / 5.8); else one, with which P = 4-12 on the lines streamed
// 4-9% faster.  Accesses off the lines are cached from five ranks up
// (stream_nt's reason).
template <int P, int OP>
int launch_fused_p(const FusedArgs& args, int mode, bool nt, int grid, hipStream_t s) {
  FusedArgs a = args;
  const dim3 blk(kBlock);
  const bool lines = rows_on_lines(a.user, P);
  if (mode == 1) {
    const bool wide = P <= 8 && (!a.tune.big || a.tune.bytes >= kTightCapBytes) &&
                      (P <= 3 || (!lines && (P <= 4 || a.tune.nt != 1)));
    if constexpr (P <= 8) {
      if (wide) {
        constexpr int V = 4;
        const int64_t blocks = (a.groups + kBlock * V - 1) / (kBlock * V);
        const dim3 g(uint32_t(blocks < kMaxGrid ? blocks : kMaxGrid));
        if (!a.tune.cap_forced) a.lds = cap_lds_bytes(a.tune.bytes < kTightCapBytes ? 0 : P == 2 ? 4 : P <= 4 ? 2 : 1);
        if constexpr (P <= 4) {
          if (nt) {
            hipLaunchKernelGGL((fused_lo_kernel<P, OP, V, true, false>), g, blk, a.lds, s, a);
            return int(hipGetLastError());
          }
        }
        hipLaunchKernelGGL((fused_lo_kernel<P, OP, V, false, false>), g, blk, a.lds, s, a);
        return int(hipGetLastError());
      }
    }
    const dim3 g(grid);
    if (lo_nt(a, P, nt)) hipLaunchKernelGGL((fused_lo_kernel<P, OP, 1, true, false>), g, blk, a.lds, s, a);
    else hipLaunchKernelGGL((fused_lo_kernel<P, OP, 1, false, false>), g, blk, a.lds, s, a);
  } else if (mode == 2) {
    if (a.groups <= int64_t(UINT32_MAX)) a.ndiv = make_fastdiv(uint32_t(a.n));
    hipLaunchKernelGGL((fused_lo_kernel<P, OP, 1, false, true>), dim3(grid), blk, a.lds, s, a);
  } else {
    return int(hipErrorInvalidValue);
  }
  return int(hipGetLastError());
}

template <int OP>
int launch_fused_op(const FusedArgs& a, int P, int mode, bool nt, int grid, hipStream_t s) {
  switch (P) {
#define AR_LO_CASE(PP) \
  case PP: return launch_fused_p<PP, OP>(a, mode, nt, grid, s);
    AR_LO_CASE(2) AR_LO_CASE(3) AR_LO_CASE(4) AR_LO_CASE(5) AR_LO_CASE(6) AR_LO_CASE(7) AR_LO_CASE(8)
    AR_LO_CASE(9) AR_LO_CASE(10) AR_LO_CASE(11) AR_LO_CASE(12) AR_LO_CASE(13) AR_LO_CASE(14)
    AR_LO_CASE(15) AR_LO_CASE(16)
#undef AR_LO_CASE
    default: return int(hipErrorInvalidValue);
  }
}

}  // namespace

int launch_fused_lo(const FusedArgs& a, int P, int dtype, int op, int mode, bool nt, int grid, void* stream) {
  if (dtype == 0) return launch_fused_free(a.user, P, op, a.n, a.stride, a.batch, false, a.tune, stream);
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  return op == 0 ? launch_fused_op<0>(a, P, mode, nt, grid, s) : launch_fused_op<1>(a, P, mode, nt, grid, s);
}

}  // namespace ar
