// fused_small.hip -- the fused kernel of small calls at many ranks.
//
// A column-fused wave holds 64 columns of all P ranks: P loads, the whole
// recursion of Secs. 8-9 (up to P (2L - 2) combinations) and P stores in one
// wave's instruction stream.  A call of a few hundred columns fills a few
// waves, which then run that stream alone: at P = 127 and one 425-byte message
// 7.6-9 us, of which HBM needs next to nothing.  Here a workgroup of 16 waves
// takes 16 columns and deals the ranks out over its waves; the primed sums
// pass through LDS, one barrier per step, and every lane carries the primed
// and the starred sums of at most two ranks: 5.7-6 us.  It is bound by latency
// and issue: loads, L times a barrier and an LDS round trip, stores.  (Three
// steps to a barrier, a lane reading seven sums and forming those of its peers,
// took 1 us more, 32 columns to a workgroup, four ranks per lane, 1.1 us.)  Where
// the calls come to it, with both sides measured: small_call (ar_internal.hpp).
//
// The combinations and their operand order are those of mid_steps
// (fused_col.hpp), which with one kept shift are also those of the
// bandwidth-optimal fold.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>

#include "ar_internal.hpp"
#include "device_common.hpp"

namespace ar {

namespace {

constexpr int kSmallBlock = 1024, kSmallWaves = kSmallBlock / kWave;
constexpr int kSmallTile = 16;                                  // columns per workgroup
constexpr int kSmallRanks = kWave / kSmallTile;                 // ranks that a wave covers at a time
constexpr int kSmallSlots = kMaxP / (kSmallRanks * kSmallWaves);  // ranks per lane

struct SmallArgs {
  void* user[kMaxP];
  int64_t stride;
  uint32_t cols;        // columns of all instances
  uint32_t q, m;        // n / P, n % P
  int32_t P, L, split;
  int32_t own;          // 1: every rank's result is its own placement's (r = L)
  FastDiv ndiv, q1div, qdiv;
  uint8_t src[kMaxP];   // placement whose starred sum placement q receives (col_src)
};

template <int OP>
__global__ __launch_bounds__(kSmallBlock) void fused_small_kernel(const SmallArgs a) {
  __shared__ float lds[2][kMaxP * kSmallTile];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int c = lane & (kSmallTile - 1), part = lane / kSmallTile;
  const int P = a.P;
  const uint32_t g = blockIdx.x * uint32_t(kSmallTile) + uint32_t(c);
  const bool live = g < a.cols;
  const uint32_t inst = fdiv(g, a.ndiv);
  const uint32_t i = g - inst * a.ndiv.d;
  const uint32_t longer = a.m * (a.q + 1);  // elements in the blocks of q + 1
  const int b = int(i < longer ? fdiv(i, a.q1div) : a.m + fdiv(i - longer, a.qdiv));
  const int64_t e = int64_t(inst) * a.stride + i;
  // slot s of this lane: rank x0(s) + part, at placement d[s] of the column's
  // block; the rank's address, from four wave-uniform ones
  auto x0 = [&](int s) { return kSmallRanks * (wave + kSmallWaves * s); };
  auto row = [&](int s) {
    const int x = x0(s), last = P - 1;
    float* p0 = static_cast<float*>(a.user[x]);
    float* p1 = static_cast<float*>(a.user[x + 1 < P ? x + 1 : last]);
    float* p2 = static_cast<float*>(a.user[x + 2 < P ? x + 2 : last]);
    float* p3 = static_cast<float*>(a.user[x + 3 < P ? x + 3 : last]);
    return part & 2 ? (part & 1 ? p3 : p2) : (part & 1 ? p1 : p0);
  };
  float R[kSmallSlots], S[kSmallSlots];
  int d[kSmallSlots];
#pragma unroll
  for (int s = 0; s < kSmallSlots; ++s) {
    const int x = x0(s) + part;
    d[s] = x - b + (x < b ? P : 0);
    R[s] = 0.0f;
    if (x0(s) < P) {
      const float* p = row(s);
      if (live && x < P) R[s] = p[e];
    }
  }
#pragma unroll
  for (int s = 0; s < kSmallSlots; ++s) S[s] = R[s];
  int N = P, buf = 0;
  for (int step = 0; step < a.L; ++step) {
    const int f = N / 2;
    const bool even = (N & 1) == 0;
#pragma unroll
    for (int s = 0; s < kSmallSlots; ++s)
      if (x0(s) + part < P) lds[buf][d[s] * kSmallTile + c] = R[s];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < kSmallSlots; ++s) {
      if (x0(s) + part < P) {
        const int from = d[s] + f - (d[s] + f >= P ? P : 0);
        const float recv = lds[buf][from * kSmallTile + c];
        if (even) S[s] = comb<OP>(S[s], recv);
        R[s] = comb<OP>(R[s], recv);  // the last step's primed sum is not used
      }
    }
    N -= f;
    buf ^= 1;
  }
  // rank x receives the starred sum of placement src[d]: its own in
  // latency-optimal plans
  if (!a.own) {
#pragma unroll
    for (int s = 0; s < kSmallSlots; ++s)
      if (x0(s) + part < P) lds[buf][d[s] * kSmallTile + c] = S[s];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < kSmallSlots; ++s)
      if (x0(s) + part < P) S[s] = lds[buf][int(a.src[d[s]]) * kSmallTile + c];
  }
#pragma unroll
  for (int s = 0; s < kSmallSlots; ++s) {
    const int x = x0(s) + part;
    if (x0(s) < P && !(a.split && x0(s) > 0)) {
      float* p = row(s);
      if (live && x < P && !(a.split && x > 0)) p[e] = S[s];
    }
  }
}

}  // namespace

// Cyclic butterfly plans (any r) of fp32.  With a.split only rank 0 receives
// the result (r = 0).
int launch_fused_small(const ColArgs& c, int op, void* stream) {
  SmallArgs a;
  std::memset(&a, 0, sizeof a);
  for (int x = 0; x < c.P; ++x) a.user[x] = c.user[x];
  const int64_t cols = c.n * c.instances;
  if (c.P < 2 || c.P > kMaxP || cols < 1 || cols > int64_t(UINT32_MAX) - kSmallTile) return int(hipErrorInvalidValue);
  a.stride = c.stride;
  a.cols = uint32_t(cols);
  a.q = uint32_t(c.q);
  a.m = uint32_t(c.m);
  a.P = c.P;
  int N[16];  // N_i, the vectors before step i
  for (N[0] = c.P; N[a.L] > 1; ++a.L) N[a.L + 1] = N[a.L] - N[a.L] / 2;
  a.split = c.split;
  a.own = c.r == a.L ? 1 : 0;
  a.ndiv = make_fastdiv(uint32_t(c.n));
  a.q1div = make_fastdiv(a.q + 1);
  a.qdiv = make_fastdiv(a.q > 0 ? a.q : 1);
  // placements [0, w) hold their own sums; the reversed step i delivers
  // placements [max(c_i, held), N_i) from f_i placements back (col_src)
  int held = (1 << c.r) < c.P ? (1 << c.r) : c.P;
  for (int q = 0; q < held; ++q) a.src[q] = uint8_t(q);
  for (int i = a.L - 1; i >= 0; --i) {
    if (N[i] <= held) continue;
    const int f = N[i] / 2, ci = N[i] - f;
    for (int q = ci > held ? ci : held; q < N[i]; ++q) a.src[q] = a.src[q - f];
    held = N[i];
  }
  const dim3 g((a.cols + kSmallTile - 1) / kSmallTile), blk(kSmallBlock);
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  if (op == 0) hipLaunchKernelGGL((fused_small_kernel<0>), g, blk, 0, s, a);
  else hipLaunchKernelGGL((fused_small_kernel<1>), g, blk, 0, s, a);
  return int(hipGetLastError());
}

}  // namespace ar
