// step_massive2d.hip -- the massive on-lattice rules in 2D.
#include "step_kernels.h"

namespace rlbm {

hipError_t launch_massive2d(const LaunchArgs &a) {
  if (a.order == 2) return launch_storage<Stencil<ST_MASSIVE2D, 2>, 2>(a);
  return launch_storage<Stencil<ST_MASSIVE2D, 3>, 3>(a);
}

}  // namespace rlbm
