// adjoint_step.h -- what the reverse-mode sources share: the sites of a block and the register-resident reverse step
// (HIP device code).
#pragma once
#include <hip/hip_runtime.h>

#include "adjoint_math.h"
#include "kernels.h"

namespace rlbm {

// Site of this thread: kAdjBX x kAdjBY tiles, dealt so that each XCD takes a contiguous band of
// them (the hardware deals consecutive blocks round-robin to the 8 XCDs) and the tap halos of
// neighbouring tiles stay in that XCD's L2 (4-5 % faster than the order as dealt).  The tile
// shape is a constant and the block count follows from the lattice (blockDim and gridDim would be
// vector loads from the dispatch packet that each wave waits for).
constexpr int kAdjBX = 64, kAdjBY = 4;

__device__ __forceinline__ bool site_xyz(CTables *tb, int &x, int &y, int &z) {
  const uint32_t gx = (tb->nx + kAdjBX - 1) / kAdjBX, gy = (tb->ny + kAdjBY - 1) / kAdjBY;
  uint32_t t = blockIdx.x;
  {
    const uint32_t nb = gx * gy * (uint32_t)tb->nz, q = nb / 8, r = nb % 8, k = t % 8, l = t / 8;
    t = k * q + (k < r ? k : r) + l;
  }
  x = (t % gx) * kAdjBX + threadIdx.x;
  y = ((t / gx) % gy) * kAdjBY + threadIdx.y;
  z = t / (gx * gy);
  return x < tb->nx && y < tb->ny;
}

__device__ __forceinline__ int wrap_p(int v, int n) {
  v = v < 0 ? v + n : v;
  return v >= n ? v - n : v;
}

template <class ST, typename S>
__device__ __forceinline__ Offs offs_periodic(CTables *tb, int x, int y, int z) {
  Offs o;
  const uint32_t nx = tb->nx, nxy = (uint32_t)tb->nx * tb->ny;
#pragma unroll
  for (int d = -1; d <= 1; ++d) {
    o.x[d + 1] = (uint32_t)wrap_p(x + d, tb->nx) * (uint32_t)sizeof(S);
    o.y[d + 1] = (uint32_t)wrap_p(y + d, tb->ny) * nx * (uint32_t)sizeof(S);
    o.z[d + 1] = ST::D == 3 ? (uint32_t)wrap_p(z + d, tb->nz) * nxy * (uint32_t)sizeof(S) : 0u;
  }
  return o;
}

template <typename S>
__device__ __forceinline__ double tau_at(CTables *tb, const void *tau_field, int64_t site) {
  return tau_field == nullptr ? tb->tau : (double)((const S *)tau_field)[site];
}

// all writers store the same value: a plain store (a volatile one makes the wave wait for its loads)
__device__ __forceinline__ void set_err(int *err) { *err = 1; }

// lam_t(x) = J_C(F_t(x))^T (S^T lam_{t+1})(x), F_t = S(B_{t-1}); dtau(x) += dL/dtau(x)
template <class ST, int N, typename S, bool DEV, typename A = S>
__global__ void __launch_bounds__(256) k_adjoint(const Tables *__restrict__ tabs, const S *__restrict__ Bprev,
                                                 const S *__restrict__ lam_next, S *__restrict__ lam,
                                                 const void *__restrict__ tau_field, double *__restrict__ dtau,
                                                 int *err) {
  CTables *tb = (CTables *)tabs;
  int x, y, z;
  if (!site_xyz(tb, x, y, z)) return;
  const int64_t sites = tb->sites;
  const int64_t site = ((int64_t)z * tb->ny + y) * tb->nx + x;
  const Offs o = offs_periodic<ST, S>(tb, x, y, z);
  A f[ST::Q], mu[ST::Q];
  pull_prod<ST, S, false, A>(tb, Bprev, sites, o, f);
  pull_prod<ST, S, true, A>(tb, lam_next, sites, o, mu);
  double taub;
  if (!collide_vjp<ST, N, A, DEV>(tb, f, mu, tau_at<S>(tb, tau_field, site), taub)) set_err(err);
  const uint32_t so = (uint32_t)site * (uint32_t)sizeof(S);
#pragma unroll
  for (int i = 0; i < ST::Q; ++i) *(S *)((char *)(lam + (int64_t)i * sites) + so) = (S)f[i];
  if (dtau != nullptr) dtau[site] += taub;
}

inline dim3 adjoint_grid(const AdjointArgs &a) {
  return dim3((unsigned)((long)((a.nx + kAdjBX - 1) / kAdjBX) * ((a.ny + kAdjBY - 1) / kAdjBY) * a.nz), 1, 1);
}

// The reverse step in double storage (adjoint_f64.hip).
hipError_t launch_adjoint_step_f64(const AdjointArgs &a);

}  // namespace rlbm
