// fused_free.hip -- the launch shape of the int32 kernel (fused_free.hpp).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>

#include "ar_internal.hpp"
#include "device_common.hpp"

namespace ar {

namespace {

// The launch shape: elements per lane, nontemporal or cached accesses, and
// the LDS each workgroup reserves so that few are resident per CU (kernels
// that stream P rows in and out keep fewer DRAM rows open that way).
struct FreeShape {
  int V;
  bool nt;
  uint32_t lds;
};

// Measured on calls of 1 GB, TB/s of 2 * P * n * 4 bytes, one launch; in
// brackets the same with 4-byte lanes, nontemporal, at the best cap:
//   rows on 128-byte lines: 16-byte lanes at two workgroups a CU, P = 3 6.6
//     [5.9]; 4-byte lanes, P = 5 6.4, P = 8 6.4, P = 13 6.2 and P = 16 6.4 (wider
//     ones no better: 6.4, 6.45, 6.1, 6.3); 8-byte lanes at one, P = 24 6.1
//     [5.8]; 4-byte lanes at one, P = 64 6.1;
//   rows off the lines, or odd strides: 16-byte lanes, nontemporal, P = 3 6.1
//     [5.6], cached, P = 5 5.8 [5.2], P = 8 5.8 [4.8]; 8-byte lanes, cached, at
//     one, P = 13 5.3 [3.8], P = 24 5.1 [4.0], P = 37 4.7 [3.6]; 4-byte lanes,
//     cached, P = 64 5.3 [3.4], P = 127 4.2 [2.9]: a nontemporal access that
//     covers part of a line costs the whole line, so all but the widest lanes
//     leave the shared lines to meet in L2;
//   instances of 1000 at stride 1024: 16-byte lanes, nontemporal, P = 8 5.5
//     [4.6], P = 16 5.0 [4.3]; 8-byte lanes, P = 24 4.5, P = 64 4.4; 4-byte lanes,
//     cached, P = 127 3.9;
//   reducing launches (P reads, 1 write; a broadcast follows), TB/s of their
//     own bytes, on / off the lines: 8-byte lanes at three, P = 24 6.7 / 6.3,
//     P = 32 6.55 / 6.2, P = 48 6.5 / 6.2; 4-byte lanes P = 64 6.5 / 5.9 (8-byte
//     6.3 / 5.9), P = 127 6.5 / 5.5.
// Calls below kFusedNtThresholdBytes (not `big`) live in the caches: ordinary
// accesses; and below kTightCapBytes the tight caps leave too few waves to
// hide latency behind (P = 8 at 16 MB per rank: 52 us at six workgroups a CU,
// 56 at two; P = 13 at 16 MB: 77 us with 4-byte lanes at four, 85 with 8-byte
// lanes at two).
FreeShape free_shape(int P, bool split, bool lines, const FusedTuning& tune, int64_t n, bool gaps) {
  FreeShape s{};
  const bool tight = tune.bytes >= kTightCapBytes, huge = tune.bytes >= 2 * kTightCapBytes;
  int cap;
  if (split) {
    s.V = P <= 16 ? 4 : (P <= 33 || (!lines && P <= 65)) ? 2 : 1;
    cap = P <= 16 ? 2 : 3;
    s.nt = lines || s.V >= 2;
  } else if (lines && !gaps) {
    s.V = P <= 4 ? (tight || !tune.big ? 4 : 2) : P >= 17 && P <= 37 && (huge || !tune.big) ? 2 : 1;
    if (P <= 4) cap = !tight ? 0 : P == 2 ? 4 : 2;
    else if (P <= 16) cap = P <= 5 ? 0 : P <= 8 ? (huge ? 4 : 6) : (huge ? 3 : 4);
    else cap = huge ? (P <= 64 ? 1 : 0) : s.V == 2 ? 2 : P <= 48 ? 3 : 0;
    s.nt = true;
  } else {
    s.V = P <= 8 || (P <= 16 && lines) ? 4 : P <= 37 || (P <= 65 && gaps) ? 2 : 1;
    // short instances between gaps: no lane may be left with a part of a group
    // (its elements go one by one)
    if (gaps && n < 4096)
      while (s.V > 1 && n % s.V != 0) s.V /= 2;
    if (!tight) cap = P <= 6 ? 0 : P <= 8 ? 6 : P <= 16 ? 4 : 2;
    else if (s.V == 4) cap = P == 2 ? 4 : P <= 4 ? 2 : 1;
    else if (s.V == 2) cap = P <= 4 ? 4 : P <= 8 ? 2 : 1;
    else cap = P <= 6 ? 0 : P <= 16 ? 2 : P <= 64 || gaps ? 1 : 0;
    s.nt = lines ? P <= 65 : s.V == 4 && P <= 4;
  }
  s.nt = s.nt && tune.big != 0;
  s.lds = cap_lds_bytes(cap);
  return s;
}

int launch_free_p(const FreeArgs& a, int P, int V, int op, bool nt, int grid, uint32_t lds, void* stream) {
  switch (P) {
#define AR_FREE_CASE(PP) \
  case PP: return launch_free_at<PP>(a, V, op, nt, grid, lds, stream);
#define AR_FREE_CASE8(B) AR_FREE_CASE(B) AR_FREE_CASE(B + 1) AR_FREE_CASE(B + 2) AR_FREE_CASE(B + 3) \
  AR_FREE_CASE(B + 4) AR_FREE_CASE(B + 5) AR_FREE_CASE(B + 6) AR_FREE_CASE(B + 7)
    AR_FREE_CASE8(2) AR_FREE_CASE8(10) AR_FREE_CASE8(18) AR_FREE_CASE8(26) AR_FREE_CASE8(34) AR_FREE_CASE8(42)
    AR_FREE_CASE8(50) AR_FREE_CASE8(58) AR_FREE_CASE8(66) AR_FREE_CASE8(74) AR_FREE_CASE8(82) AR_FREE_CASE8(90)
    AR_FREE_CASE8(98) AR_FREE_CASE8(106) AR_FREE_CASE8(114) AR_FREE_CASE(122) AR_FREE_CASE(123) AR_FREE_CASE(124)
    AR_FREE_CASE(125) AR_FREE_CASE(126) AR_FREE_CASE(127) AR_FREE_CASE(128)
#undef AR_FREE_CASE8
#undef AR_FREE_CASE
    default: return int(hipErrorInvalidValue);
  }
}

}  // namespace

int launch_fused_free(void* const* user, int P, int op, int64_t n, int64_t stride, int64_t instances, bool split,
                      const FusedTuning& tune, void* stream) {
  FreeArgs a;
  std::memset(&a, 0, sizeof a);
  for (int x = 0; x < P; ++x) a.user[x] = user[x];
  const bool gaps = instances > 1 && stride != n;
  const bool lines = rows_on_lines(user, P) && (!gaps || stride % 32 == 0);
  a.split = split ? 1 : 0;
  a.n = gaps ? n : instances * n;
  a.stride = stride;
  FreeShape sh = free_shape(P, split, lines, tune, n, gaps);
  a.gpi = (a.n + sh.V - 1) / sh.V;
  a.groups = (gaps ? instances : 1) * a.gpi;
  a.gaps = !gaps ? 0 : a.groups + kBlock < int64_t(UINT32_MAX) ? 1 : 2;
  if (a.gaps == 1) a.gdiv = make_fastdiv(uint32_t(a.gpi));
  if (tune.nt >= 0) sh.nt = tune.nt != 0;
  if (tune.cap_forced) sh.lds = tune.lds;
  a.blocks = uint64_t((a.groups + kBlock - 1) / kBlock);
  const int grid = int(a.blocks > uint64_t(kMaxGrid) ? uint64_t(kMaxGrid) : a.blocks);
  return launch_free_p(a, P, sh.V, op, sh.nt, grid, sh.lds, stream);
}

}  // namespace ar
