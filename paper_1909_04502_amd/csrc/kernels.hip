// kernels.hip -- dispatch of the step, moments and initial-state launches to the stencil families.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace rlbm {

hipError_t launch(const LaunchArgs &a) {
  switch (a.stencil) {
    case ST_UR2D: return launch_ur2d(a);
    case ST_MASSIVE2D: return launch_massive2d(a);
    case ST_MASSIVE3D: return launch_massive3d(a);
    case ST_UR3D: return launch_ur3d(a);
    case ST_PROD2D: return launch_prod2d(a);
    case ST_PROD3D: return launch_prod3d(a);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace rlbm
