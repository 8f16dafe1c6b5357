// fused_free.hip -- launches of the int32 kernel (fused_free.hpp), in the shape that
// free_shape.hpp chooses.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>

#include "ar_internal.hpp"
#include "device_common.hpp"
#include "free_shape.hpp"

namespace ar {

namespace {

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
  a.split = split ? 1 : 0;
  a.n = gaps ? n : instances * n;
  a.stride = stride;
  FreeShape sh = free_shape(P, split, rows_on_lines(user, P), tune, n, gaps ? stride - n : 0);
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
