// Query kernels in 32-query tiles, for sphere obstacles (see narrow_tiles).
#include "gcdf_tile.h"

namespace gcdf {

hipError_t launch_fused_sphere_narrow(const DevNet& net, const Job& job, bool pairs, bool want_grad, int num_cu,
                                      hipStream_t s) {
  if (net.width == 256) return launch_w<256, 1, true>(net, job, pairs, want_grad, num_cu, s);
  return launch_w<512, 1, true>(net, job, pairs, want_grad, num_cu, s);
}

}  // namespace gcdf
