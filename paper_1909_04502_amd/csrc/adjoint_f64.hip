// adjoint_f64.hip -- the reverse step in double storage (HIP, gfx950).
//
// F_t and lam of a site fill the registers, and the tables are read as plain memory here: as scalar loads moved freely
// to the kernel's start they push 454 registers at order 3 and 334 at order 2, against 366 and 250 (two waves per SIMD).
// Per step at 512 x 512: 64 us instead of 71 at order 3, 34 instead of 46 at order 2.  (Float storage with double
// arithmetic is the other way round: 51 instead of 49 us with plain tables.)
#define RLBM_TABLES_PLAIN   // device_math.h
#include "adjoint_step.h"

namespace rlbm {

template <class ST, int N>
static hipError_t launch_step(const AdjointArgs &a) {
  hipLaunchKernelGGL((k_adjoint<ST, N, double, false, double>), adjoint_grid(a), dim3(kAdjBX, kAdjBY, 1), 0, a.stream, a.tb,
                     (const double *)a.state, (const double *)a.lam_in, (double *)a.lam_out, a.tau_field, a.dtau, a.err);
  return hipGetLastError();
}

hipError_t launch_adjoint_step_f64(const AdjointArgs &a) {
  if (a.order == 2) return launch_step<Stencil<ST_PROD2D, 3>, 2>(a);
  return launch_step<Stencil<ST_PROD2D, 4>, 3>(a);
}

}  // namespace rlbm
