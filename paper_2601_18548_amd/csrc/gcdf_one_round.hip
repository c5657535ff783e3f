// Split-mode query kernels of width 256 as one 8-wave workgroup per compute unit, for
// launches of at most one 64-query tile per compute unit (see one_round).
#define GCDF_ONE_ROUND
#include "gcdf_tile.h"

namespace gcdf {

hipError_t launch_fused_one_round(const DevNet& net, const Job& job, bool pairs, bool want_grad, int num_cu, hipStream_t s) {
  if (net.mode == kBF16X2F16) return launch_m<256, kBF16X2F16, 2, false>(net, job, pairs, want_grad, num_cu, s);
  return launch_m<256, kBF16X2, 2, false>(net, job, pairs, want_grad, num_cu, s);
}

hipError_t launch_fused_sphere_one_round(const DevNet& net, const Job& job, bool pairs, bool want_grad, int num_cu,
                                         hipStream_t s) {
  if (net.mode == kBF16X2F16) return launch_m<256, kBF16X2F16, 2, true>(net, job, pairs, want_grad, num_cu, s);
  return launch_m<256, kBF16X2, 2, true>(net, job, pairs, want_grad, num_cu, s);
}

}  // namespace gcdf
