// step_ur2d.hip -- the printed massless rules in 2D.
#include "step_kernels.h"

namespace rlbm {

hipError_t launch_ur2d(const LaunchArgs &a) {
  if (a.order == 2) return launch_storage<Stencil<ST_UR2D, 3>, 2>(a);
  return launch_storage<Stencil<ST_UR2D, 4>, 3>(a);
}

}  // namespace rlbm
