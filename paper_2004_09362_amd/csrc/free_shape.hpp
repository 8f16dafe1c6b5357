// free_shape.hpp -- the launch shape of the int32 kernel (fused_free.hip), host
// code only.
#pragma once

#include <cstdint>

#include "ar_internal.hpp"

namespace ar {

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
// With gaps a lane's accesses cover parts of lines, except where the gaps are
// multiples of 16 elements, which leave whole half lines.  There launches from 17
// ranks are nontemporal, as are those without gaps (on buffers that alternate beyond
// the caches, nontemporal / cached, P = 24: 80 at stride 96 0.80-0.88, 208 at 224
// 0.80-0.85, 1000 at 1032 0.81-0.91), and up to 16 ranks those from kGapNtBytes (208 at 224
// 0.74-0.83, 1008 at 1024 0.82-0.9, 2304 at 2368 0.85-0.95): one set of buffers, which
// the caches hold to a good part up to 600 MB of traffic, then takes 1.2-1.7 of the
// cached time, below kGapNtBytes up to 1.9.  Other gaps: cached from 17 ranks (88 at 96
// 1.2-1.37, 1000 at 1008 1.02-1.14); up to 16 nontemporal from kGapNtBytes and 512
// elements where every instance starts on a line (1000 at 1024 0.88-0.98), or at four
// ranks and fewer (1000 at 1008 0.94-0.97), else cached (88 at 96 1.07-1.29).
// Calls below kFusedNtThresholdBytes (not `big`) live in the caches: ordinary
// accesses; and below kTightCapBytes the tight caps leave too few waves to
// hide latency behind (P = 8 at 16 MB per rank: 52 us at six workgroups a CU,
// 56 at two; P = 13 at 16 MB: 77 us with 4-byte lanes at four, 85 with 8-byte
// lanes at two).
constexpr int64_t kGapNtBytes = int64_t(256) << 20;
// rows: the rank buffers start on 128-byte lines.  gap: elements between two
// instances, 0 for one instance or none between them.
inline FreeShape free_shape(int P, bool split, bool rows, const FusedTuning& tune, int64_t n, int64_t gap) {
  const bool gaps = gap > 0, lines = rows && (!gaps || (n + gap) % 32 == 0);
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
    if (gaps) {
      const bool large = tune.bytes >= kGapNtBytes;
      if (rows && gap % 16 == 0) s.nt = P >= 17 || large;
      else s.nt = s.nt && P <= 16 && large && n >= 512;
    }
  }
  s.nt = s.nt && tune.big != 0;
  s.lds = cap_lds_bytes(cap);
  return s;
}

}  // namespace ar
