// step_prod2d.hip -- the 2D product rules.
#include "step_kernels.h"

namespace rlbm {

hipError_t launch_prod2d(const LaunchArgs &a) {
  if (a.order == 2) return launch_storage<Stencil<ST_PROD2D, 3>, 2>(a);
  return launch_storage<Stencil<ST_PROD2D, 4>, 3>(a);
}

}  // namespace rlbm
