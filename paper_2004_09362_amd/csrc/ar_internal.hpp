// ar_internal.hpp -- types shared by the host plan generator, the C ABI and
// the HIP kernels of libar.so.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

namespace ar {

constexpr int kMaxP = 128;       // largest supported number of ranks
constexpr int kMaxRanges = 8;    // placement ranges per launch
// Largest extent of one rank's buffer, in elements (2^46: 256 TiB of 4-byte
// elements, far above any device's memory), so that every size derived from
// it -- bytes, tiles, products with P -- fits in 64-bit arithmetic.
constexpr int64_t kMaxRankElems = int64_t(1) << 46;
constexpr int kFusedMaxP = 16;   // largest P of the register-resident fused kernel
// P range in which the rank-slot kernel takes shifted max plans as it takes
// sums, nontemporal accesses among them; elsewhere its cached form alone exists
// for them, for batches of short blocks (launch_fused_mid)
constexpr int kRotMaxShiftedMinP = 24, kRotMaxShiftedMaxP = 48;
// Size of the device-resident scratch of ar_execute_noalloc (noalloc.hip):
// the X and Y buffers of a step-wise plan with r > 0 take 2 * P rank
// regions of the call's extent rounded up to 64 elements.
constexpr int64_t kNoAllocScratchBytes = int64_t(64) << 20;

enum Buf : int32_t { kBufNone = -1, kBufU = 0, kBufX = 1, kBufY = 2 };
enum Kind : int32_t { kCopy = 0, kReduce = 1, kReduce2 = 2 };
enum Phase : int32_t { kPhaseReduce = 0, kPhaseDistribute = 1, kPhaseLocal = 2 };
// The group T_P (Sec. 5): cyclic, t_k(x) = x + k mod P, or the group of
// Table 1b for power-of-two P, t_k(x) = x XOR k.  Schedules: the butterfly
// family of Secs. 7-9 (any k in [L, 2L]) or the Ring of Sec. 6.
enum Group : int32_t { kGroupCyclic = 0, kGroupXor = 1 };
enum Sched : int32_t { kSchedButterfly = 0, kSchedRing = 1 };

// Block held at placement p by rank x (h = identity), and the rank a step
// with "delta" pulls from: x - p and x + delta mod P in the cyclic group,
// x XOR p and x XOR delta in the XOR group.
inline int32_t group_block(int32_t group, int32_t x, int32_t p, int32_t P) {
  if (group == kGroupXor) return x ^ p;
  const int32_t b = (x - p) % P;
  return b < 0 ? b + P : b;
}
inline int32_t group_peer(int32_t group, int32_t x, int32_t delta, int32_t P) {
  if (group == kGroupXor) return x ^ delta;
  const int32_t y = (x + delta) % P;
  return y < 0 ? y + P : y;
}

// One range of placements worked on by every rank in a launch.  delta names
// the peer (group_peer); the peer's copy of the same block is its placement
// p + delta (cyclic) or p XOR delta (XOR group).
struct Range {
  int32_t p0, count, kind, delta;
  int32_t dst, own, dst2, own2, src;
};

struct Launch {
  int32_t phase;
  std::vector<Range> ranges;
};

// The schedule and its sizes; built on the host (plan.cpp).
struct Schedule {
  int32_t P = 1, L = 0, k = 0, r = 0, w = 1;
  int32_t group = kGroupCyclic, sched = kSchedButterfly;
  int64_t n = 0;
  std::vector<int32_t> N, f, c;  // N_i, floor(N_i/2), ceil(N_i/2)
  std::vector<Launch> launches;
  int32_t rs_steps = 0, ag_steps = 0;
  bool uses_scratch = false;
  // sizes per instance
  int64_t blocks_pulled_per_rank = 0;
  int64_t combines_per_rank = 0;
  int64_t hbm_blocks = 0;  // block reads + writes per rank, STEPWISE path
};

// Builds the schedule; returns an empty string or the reason it failed.
std::string build_schedule(int32_t P, int64_t n, int32_t k, Schedule* out);
std::string build_schedule_ex(int32_t P, int64_t n, int32_t k, int32_t group, int32_t sched, Schedule* out);

// Verifies that no launch of `s` lets one work item write a location that a
// different work item reads or writes.  Returns "" or a description.
std::string check_hazards(const Schedule& s);

// Balanced partition: block b of n elements over P blocks.
inline int64_t block_off(int64_t n, int32_t P, int32_t b) {
  const int64_t q = n / P, m = n % P;
  return b * q + (b < m ? b : m);
}
inline int64_t block_len(int64_t n, int32_t P, int32_t b) {
  const int64_t q = n / P, m = n % P;
  return q + (b < m ? 1 : 0);
}

// Division of 32-bit numbers by a divisor fixed for a launch: a multiply-high
// and two shifts instead of a division sequence (unsigned division by
// invariant integers, Granlund & Montgomery 1994, "round-up" variant).
struct FastDiv {
  uint32_t d, m, l;  // divisor, magic multiplier, ceil(log2 d)
};

inline FastDiv make_fastdiv(uint32_t d) {
  FastDiv f{d, 0, 0};
  while ((uint64_t(1) << f.l) < d) ++f.l;
  f.m = uint32_t(((uint64_t(1) << 32) * ((uint64_t(1) << f.l) - d)) / d + 1);
  return f;
}

// Host reference of the device quotient (used by the tests).
inline uint32_t fastdiv_host(uint32_t n, const FastDiv& f) {
  if (f.l == 0) return n;
  const uint32_t t = uint32_t((uint64_t(n) * f.m) >> 32);
  return (t + ((n - t) >> 1)) >> (f.l - 1);
}

// ----- device launch interface (kernels.hip) -----

struct DevRange {
  int32_t p0, count, kind, delta;
  int32_t dst, own, dst2, own2, src;
  int32_t first;  // index of the range's first op among the launch's ops
};

struct StepArgs {
  void* user[kMaxP];        // rank buffers
  char* scratch[2];         // X and Y: rank y's region at scratch[i] + y * scratch_rank_stride elements
  int64_t scratch_rank_stride;
  int64_t n, stride;
  int64_t q, m;             // n / P, n % P
  uint32_t total_tiles;     // P * total_ops * batch * tiles_per_seg (< 2^31)
  FastDiv tps, batch, ops;  // tiles per segment, instances, ops per rank
  int32_t P, n_ranges;
  int32_t group;            // kGroupCyclic or kGroupXor
  DevRange ranges[kMaxRanges];
  // Merged runs (step_merged_kernel): the placements p0 .. p0+count-1 of a
  // range touch one run of consecutive blocks of rank x (cyclically), with
  // one peer and one set of buffers, so the range is streamed as one flat
  // space per rank: run_len[i] elements per instance (the whole row when
  // the range covers every placement, else count * ceil(n / P) -- a rank's
  // run is at most that long), batch * run_len[i] columns in all, tiles of
  // 256 columns.  Range i's tiles start at tile_first[i], P * tiles[i] of
  // them (rank-major).
  FastDiv run_len[kMaxRanges], tiles[kMaxRanges];
  uint32_t run_cols[kMaxRanges], tile_first[kMaxRanges];
};

// What the host decided about a fused launch beyond its work, for launchers
// that choose their own shape: nontemporal accesses (0 / 1 by override, -1
// open), whether that is to be nontemporal when open (launches of
// kFusedNtThresholdBytes and more), the bytes the call moves, and an
// overriding occupancy cap.
struct FusedTuning {
  int64_t bytes;
  int32_t nt;
  int32_t big;
  int32_t cap_forced;
  uint32_t lds;  // the overriding cap's LDS
  int32_t layout_forced;  // 1: the column layout is an override's (AR_FUSED_PACKED, AR_FUSED_ROTATE)
};

// Whether every rank buffer starts on a 128-byte line, and whether they all
// start at the same place within one.
inline bool rows_on_lines(void* const* user, int P) {
  for (int x = 0; x < P; ++x)
    if (reinterpret_cast<uintptr_t>(user[x]) % 128 != 0) return false;
  return true;
}
inline bool rows_congruent(void* const* user, int P) {
  for (int x = 1; x < P; ++x)
    if ((reinterpret_cast<uintptr_t>(user[x]) ^ reinterpret_cast<uintptr_t>(user[0])) % 128 != 0) return false;
  return true;
}

// LDS that lets `cap` workgroups fit on a CU (160 KB), 0 for no cap.
constexpr uint32_t cap_lds_bytes(int cap) {
  return cap == 0 ? 0u : cap == 1 ? 84u * 1024 : (160u * 1024 / uint32_t(cap) - 1024) / 512 * 512;
}
// Calls that move less than this run from the caches to a good part: tight
// occupancy caps then leave too few waves to hide latency behind.
constexpr int64_t kTightCapBytes = int64_t(256) << 20;

// lds: dynamic LDS each workgroup reserves without using it, so that fewer
// workgroups are resident per CU (0: no cap); read by the launchers.
struct FusedArgs {
  void* user[kMaxP];
  int64_t n, stride, batch;
  int64_t groups;           // column groups (16-byte mode) or columns (other modes)
  uint32_t lds;
  FusedTuning tune;
  FastDiv ndiv;             // n, for gaps between instances (set by the launcher)
};

// Nontemporal accesses of a latency-optimal launch with one column per lane that
// the host would stream: not off the lines from five ranks up (stream_nt's reason).
// Up to four they are the faster ones there too: P = 2, 140 MB of traffic 27.7 us
// against 30.4 cached, P = 4 28.6 against 29.4.
inline bool lo_nt(const FusedArgs& a, int P, bool nt) {
  return nt && (P <= 4 || a.tune.nt == 1 || rows_on_lines(a.user, P));
}

// Column kernels: wave tile t -> (instance, block, 64 columns of the block).
// The rank table is stored twice over (user[x] == user[x + P]) so that the
// ranks b, b+1, ..., b+P-1 of a rotation are consecutive entries.
struct ColArgs {
  void* user[2 * kMaxP];
  int64_t stride, q, m;     // instance stride, n / P, n % P
  uint32_t total_tiles;     // batch * P * tiles (< 2^31)
  FastDiv tiles, pdiv;      // column tiles per block, P
  int32_t P, r;             // r: distribution steps removed (kept shifts w = min(2^r, P))
  int32_t split;            // 1: store the result to rank 0 only (a broadcast follows)
  uint32_t lds;             // as in FusedArgs
  // Latency-optimal plans (r = L): the tree of every rank is the same for
  // every block, so the kernels may tile the batch * n columns as one flat
  // space (64 per wave, no block index): flat = 1, flat_cols = batch * n
  // (< 2^32 - 64), ndiv = n.
  int32_t flat;
  uint32_t flat_cols;
  FastDiv ndiv;
  // Short blocks (every other plan): with packed = 1 a wave tile covers the
  // same block of ipw instances, lane = j * maxlen + c for column c of
  // instance j of the tile's group; lendiv = maxlen (the longest block),
  // ipw = 64 / maxlen, batch = the number of instances.  Otherwise a tile
  // covers 64 columns of one block of one instance.
  int32_t packed;
  uint32_t ipw, batch;
  FastDiv lendiv;
  // Rank-slot kernel of the cyclic butterfly plans (flat columns, block of
  // each lane from its index i in the instance): the first m blocks hold
  // q + 1 elements (q1div = q + 1), the others q (qdiv = max(q, 1)).
  FastDiv q1div, qdiv;
  int64_t n, instances;  // the call's extent
  FusedTuning tune;
};

// Flat columns lie on the 128-byte lines of every rank's buffer, or on half
// lines (which HBM serves whole): wave rows then cover whole ones.  So they do
// where every gap between instances is a multiple of 16 elements, whatever the
// instances' length.  Block tiles do where the rows are congruent (their tiles are
// laid on the root's lines).  Rank slots, cached over nontemporal, on buffers that
// alternate beyond the caches, 120 MB over all ranks, P = 10-100: 48 at stride 64 1.1-1.25, 128
// at 176 1.22-1.26, 208 at 224 1.1-1.2, 104 at 136 1.02-1.15, 1008 at 1024 0.97-1.1; 104 at 112
// 0.73-0.86, 106 at 128 0.72-0.93, 500 at 512 0.72-0.87, 1000 at 1024 0.83-0.97.
inline bool flat_on_lines(const ColArgs& a) {
  return rows_on_lines(a.user, a.P) && (a.instances == 1 || (a.stride - a.n) % 16 == 0);
}

// Nontemporal accesses of a launch that the host would stream: not off the
// lines, where each access that covers part of a line costs the whole line
// (stores twice over), while ordinary ones meet in L2.  Rows back to back at
// an odd length, one launch, cached / nontemporal, TB/s: P = 8 5.9 / 4.6, P = 13
// 5.3 / 4.1, P = 24 5.0 / 3.8, P = 64 4.8 / 3.3, P = 127 4.3 / 2.8.  Reducing launches (one
// store a column) below 48 ranks keep them: P = 24 5.75 / 5.55, P = 64 5.6 / 5.9;
// so do calls of up to four ranks but those of short instances between gaps:
// P = 4 5.0 / 5.3, 5184 x 1290 at stride 1322 41.7 / 38.4 us; 106 at 113, P = 3 5.1 / 4.2.
inline bool stream_nt(const ColArgs& a, bool nt) {
  if (!nt || a.tune.nt >= 0 || (a.split && a.P < 48)) return nt;
  if (a.P <= 4 && (a.instances == 1 || a.stride == a.n || a.n >= 1024)) return nt;
  return a.packed ? false : a.flat ? flat_on_lines(a) : rows_congruent(a.user, a.P);
}

// The rank-slot kernel's accesses: nontemporal on the lines whatever the size
// (its launches stream short blocks of many instances once), as in reducing
// launches below 48 ranks; AR_FUSED_NT overrides both.
inline bool rot_nt(const ColArgs& a) {
  return a.tune.nt >= 0 ? a.tune.nt != 0 : (a.split && a.P < 48) || flat_on_lines(a);
}

// dtype: 0 int32, 1 float32; op: 0 sum, 1 max.  Returns a hipError_t value.
int launch_step(const StepArgs& a, int dtype, int op, bool vec, bool nt, int grid, void* stream);
// One step as merged runs (a.run_len, a.tiles, ...): each range's blocks of a
// rank streamed as one flat space per instance.
int launch_step_merged(const StepArgs& a, int dtype, int op, bool nt, int grid, void* stream);
// Any int32 plan (fused_free.hip): every rank, or rank 0 with `split`,
// receives the combination of the P values of each column.  The launchers
// below hand their int32 calls to it.
int launch_fused_free(void* const* user, int P, int op, int64_t n, int64_t stride, int64_t instances, bool split,
                      const FusedTuning& tune, void* stream);
// Its kernel's arguments and launcher, one instantiation per P (units written
// by build.py).
struct FreeArgs {
  void* user[kMaxP];
  int32_t split;
  int32_t gaps;        // 0: no gaps between instances; 1: gaps; 2: gaps and 2^32 groups or more
  int64_t n, stride;   // instance length (without gaps the whole span's) and stride
  int64_t groups;      // lanes with work: instances * gpi
  int64_t gpi;         // groups of V elements per instance (the last one may hold fewer)
  uint64_t blocks;     // workgroups with work (the grid's loop)
  FastDiv gdiv;        // gpi
};
template <int P>
int launch_free_at(const FreeArgs& a, int V, int op, bool nt, int grid, uint32_t lds, void* stream);
// Fused latency-optimal kernel; mode 1: one element per lane (contiguous
// instances), 2: any instance stride.
int launch_fused_lo(const FusedArgs& a, int P, int dtype, int op, int mode, bool nt, int grid, void* stream);
// Column-fused kernels, one instantiation per P (units written by build.py):
// bandwidth-optimal (r = 0) and shifted / latency-optimal (r >= 1), and
// their dispatcher over P = 2..128.
template <int P>
int launch_fused_bo(const ColArgs& a, int dtype, int op, bool nt, int grid, void* stream);
template <int P>
int launch_fused_mid(const ColArgs& a, int dtype, int op, bool nt, int grid, void* stream);
int launch_fused_col_any(const ColArgs& a, int P, int dtype, int op, bool nt, int grid, void* stream);
// The same plans, fp32, for calls of up to kSmallCols columns at many ranks
// (fused_small.hip): shifted plans from kSmallShiftedMinP ranks; bandwidth-
// optimal ones, and latency-optimal ones at odd P (whose column kernel needs
// more than a wave's 256 registers), from kSmallMinP.  In a graph of launches,
// us, column kernel / this one, at 106 and 4096 columns: shifted P = 64 5.5 / 4.75
// and 4.8 / 5.4, P = 80 6.5 / 5.3 and 5.9 / 6.0, P = 100 7.4 / 5.5 and 7.1 / 6.4, P = 127
// 8.9 / 6.0 and 9.2 / 7.1; latency-optimal P = 100 4.2 / 5.25, P = 127 7.6 / 5.7 and 8.0 /
// 6.8, P = 128 4.45 / 5.6; bandwidth-optimal (with its broadcast) P = 100 7.6 / 7.3 and
// 8.3 / 8.3, P = 127 8.8 / 7.7 and 9.3 / 9.1; at 8192 columns all the other way round.
constexpr int kSmallShiftedMinP = 80, kSmallMinP = 97;
constexpr int64_t kSmallCols = 4096;
inline bool small_call(const ColArgs& a) {
  const bool lo = (int64_t(1) << a.r) >= a.P;
  const bool ranks = a.r == 0 ? a.P >= kSmallMinP : lo ? a.P >= kSmallMinP && a.P % 2 == 1 : a.P >= kSmallShiftedMinP;
  return ranks && a.n * a.instances <= kSmallCols && a.tune.nt < 0 && !a.tune.cap_forced && !a.tune.layout_forced;
}
int launch_fused_small(const ColArgs& a, int op, void* stream);
// Rank-slot kernel on flat columns (batches of short blocks, sums): the
// cyclic butterfly plans with r < L, or the Ring (ring = true); and its
// dispatcher over P = 2..128.
template <int P>
int launch_fused_rot(const ColArgs& a, int dtype, int op, bool ring, int grid, void* stream);
int launch_fused_rot_any(const ColArgs& a, int P, int dtype, int op, bool ring, int grid, void* stream);
// Column-fused kernels of the other schedules (fused_group.hip): the XOR
// group's Recursive Halving / hybrid / Recursive Doubling for P = 2..128 a
// power of two and any r, and the Ring for any P in 2..128.
int launch_fused_xor(const ColArgs& a, int P, int dtype, int op, bool nt, int grid, void* stream);
int launch_fused_ring(const ColArgs& a, int dtype, int op, bool nt, int grid, void* stream);
// Second half of a split fused launch (broadcast.hip): the results, stored
// on rank 0 by the reducing kernel, copied to the other P - 1 ranks, tiled as
// the reducing launch.
int launch_broadcast(const ColArgs& a, int dtype, bool nt, int grid, void* stream);

// The same copy ordered destination by destination (broadcast.hip), for rank
// buffers of any alignment and instances with or without gaps.  A workgroup
// copies one chunk of kStreamChunk consecutive columns of a rank's span to one
// destination rank, one 16-byte store per thread; ids run slice by slice (C
// chunks per slice), destination by destination, chunk by chunk.
constexpr uint32_t kStreamBlock = 256;  // threads per workgroup, four columns each
constexpr uint32_t kStreamChunk = 4 * kStreamBlock;
// n / d without a branch: t = umulhi(n, mul), (t + ((n - t) >> s1)) >> s2;
// for d = 1, mul = s1 = s2 = 0 (stream_div builds it from a FastDiv).
struct StreamDiv {
  uint32_t d, mul, s1, s2;
};
inline StreamDiv stream_div(uint32_t d) {
  const FastDiv f = make_fastdiv(d);
  return f.l == 0 ? StreamDiv{d, 0, 0, 0} : StreamDiv{d, f.m, 1, f.l - 1};
}
// Host reference of the device quotient (used by the tests).
inline uint32_t stream_div_host(uint32_t n, const StreamDiv& d) {
  const uint32_t t = uint32_t((uint64_t(n) * d.mul) >> 32);
  return (t + ((n - t) >> d.s1)) >> d.s2;
}
// The scalars come first, so that a workgroup reads them in one batch of
// kernel-argument loads before it looks up its two rank pointers.
struct CopyArgs {
  StreamDiv sdiv, cdiv;  // C * P, C (chunks per slice, a multiple of the XCD count X)
  // chunk of workgroup c of a slice: (c & mask) * per_xcd + (c >> shift) --
  // regions: X - 1, C / X, log2 X; interleaved (chunk c itself): 0, 0, 0
  uint32_t mask, per_xcd, shift;
  uint32_t chunks;  // chunks of the longest destination grid
  uint32_t cols;    // columns of a rank's span: (instances - 1) * stride + n
  uint32_t n;       // gap: instance length
  uint32_t P;
  StreamDiv stdiv;  // gap: the instance stride
  void* user[kMaxP];
};
// nt: nontemporal loads and stores.  gap: the span holds gaps between
// instances.  lines: each destination's chunk grid starts on a 128-byte line
// of its buffer; otherwise on column 0.  grid: whole slices of C * P workgroups.
int launch_copy(const CopyArgs& a, uint32_t grid, bool nt, bool gap, bool lines, void* stream);
// Device address of the allocation-free scratch (noalloc.hip) on `device`,
// which must be the current device; looked up on the first call per device.
// Returns a hipError_t value.
int noalloc_scratch(int device, void** ptr);
// Workgroups of a step launch over `total_tiles` wave tiles, and the tile size.
int step_grid(int64_t total_tiles);
int64_t step_tile_elems();

}  // namespace ar
