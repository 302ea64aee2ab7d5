// step_onlat3d.hip -- the on-lattice rules in 3D (massive, and the printed massless rule).
#include "step_kernels.h"

namespace rlbm {

hipError_t launch_massive3d(const LaunchArgs &a) { return launch_storage<Stencil<ST_MASSIVE3D, 3>, 3>(a); }
hipError_t launch_ur3d(const LaunchArgs &a) { return launch_storage<Stencil<ST_UR3D, 4>, 3>(a); }

}  // namespace rlbm
