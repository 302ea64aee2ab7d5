// step_prod3d.hip -- the 3D product rules.
#include "step_kernels.h"

namespace rlbm {

hipError_t launch_prod3d(const LaunchArgs &a) {
  if (a.order == 2) return launch_storage<Stencil<ST_PROD3D, 3>, 2>(a);
  return launch_storage<Stencil<ST_PROD3D, 4>, 3>(a);
}

}  // namespace rlbm
