// adjoint.hip -- reverse-mode kernels of the RLBM step (HIP, gfx950).
//
// State sequence: B_0 = C(f_0), F_t = S(B_{t-1}), B_t = C(F_t) (S streaming,
// C collision).  Adjoints lam_t = dL/dF_t obey
//   lam_t = J_C(F_t)^T S^T lam_{t+1},   dL/dtau += (dC/dtau)^T S^T lam_{t+1},
// and the loss on the macroscopic fields of F_{T+1} = S(B_T) seeds
// lam_{T+1} = J_macro(F_{T+1})^T g.  Each kernel recomputes the forward
// values of its site from the stored state (no per-site tape is kept).
#include <hip/hip_runtime.h>

#include "adjoint_step.h"

namespace rlbm {

// The same reverse step for float storage and arithmetic, in passes over the shells: the taps of F_t and of
// S^T lam_{t+1}, each pulled once and kept in LDS (its own places: no barrier), with the moments of F_t; the
// reverse of the relaxation and of the equilibrium; and lam_t = mu (1 - Omega) + the terms through n, T and U,
// stored shell by shell.  That fits two waves per SIMD.  All taps of F_t are asked for before the first is
// summed, and those of a shell of lam before the sums of a shell of F_t: left to itself the scheduler waits
// for every load in turn (62 us at 512 x 512).  Order 3 at 512 x 512: 40 us, of which the vector arithmetic
// of four waves per SIMD takes 19; 51 us when each pass pulled its shells again (3590 instead of 2815 vector
// instructions a wave, 455 instead of 221 lines read).  Blocks of one or two rows: 44 and 49 us.
template <class ST, int N, typename S, bool DEV>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8)))
k_adjoint_streamed(const Tables *__restrict__ tabs, const S *__restrict__ Bprev, const S *__restrict__ lam_next,
                   S *__restrict__ lam, const void *__restrict__ tau_field, double *__restrict__ dtau, int *err) {
  CTables *tb = (CTables *)tabs;
  constexpr int D = ST::D, ND = ST::NDIR, NPD = ND / 2, KR = ST::NSHELL;
  using B = BasisDef<D, N>;
  using A = S;
  int x, y, z;
  if (!site_xyz(tb, x, y, z)) return;
  const int64_t sites = tb->sites;
  const int64_t site = ((int64_t)z * tb->ny + y) * tb->nx + x;
  const Offs o = offs_periodic<ST, S>(tb, x, y, z);
  // this thread's F_t and S^T lam_{t+1}, kept in LDS
  __shared__ A fl[ST::Q][kAdjBX * kAdjBY], ml[ST::Q][kAdjBX * kAdjBY];
  const int tid = threadIdx.y * kAdjBX + threadIdx.x;
  // ---- forward recomputation: moments, Landau frame, n, T, equilibrium coefficients ----
  MomAcc<D> acc;
  StageTaps<ST, S> tf[KR], tm[KR];
  const S *fb = Bprev, *lb = lam_next;
#pragma unroll
  for (int j = 0; j < KR; ++j) load_taps<ST, S, false>(fb, sites, o, tf[j]);
  // tau and dtau are asked for with the taps: where there is none, a place in the state instead, unused (a load
  // under a condition would be waited for at once)
  const S tau1 = (tau_field != nullptr ? (const S *)tau_field : Bprev)[site];
  const double dtau0 = (dtau != nullptr ? (const double *)dtau : (const double *)Bprev)[site];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < KR; ++j) {
    load_taps<ST, S, true>(lb, sites, o, tm[j]);
    __builtin_amdgcn_sched_barrier(0);
    A fs[ND];
    stage_interpolate<ST, S, A>(tb, j, tf[j], fs);
    moments_shell<ST, A, ND>(tb, j, fs, 0, acc);
#pragma unroll
    for (int k = 0; k < ND; ++k) fl[j * ND + k][tid] = fs[k];
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int j = 0; j < KR; ++j) {
    A ms[ND];
    stage_interpolate<ST, S, A>(tb, j, tm[j], ms);
#pragma unroll
    for (int k = 0; k < ND; ++k) ml[j * ND + k][tid] = ms[k];
  }
  asm volatile("" ::: "memory");   // they are read back, not kept in registers
  double Nv[D + 1], T[D + 1][D + 1];
  moments_finish<ST, DEV>(tb, acc, Nv, T);
  Macro<D> mac;
  mac.ok = landau_frame<D, 3>(T, mac.eps, mac.U);
  mac.n = lorentz_dot<D>(mac.U, Nv);
  const double m = tb->m;
  mac.ok = temperature_2d(mac.eps / mac.n, m, mac.T) && mac.ok;
  mac.ok = mac.ok && mac.n > 0.0 && mac.eps > 0.0;
  if (!mac.ok) set_err(err);
  const RatiosD rd = ratios_2d_d(m / mac.T);
  double ap[B::NM];
  {
    Ratios rr;
    rr.r0 = rd.r0;
    rr.r2 = rd.r2;
    rr.r3 = rd.r3;
    double Md[B::NM];
    basis_moments<D, N>(mac.n, mac.T, mac.U, rr, Md);
    feq_coefficients<D, N, DEV>(tb, Md, ap);
  }
  const double itau = 1.0 / (tau_field != nullptr ? (double)tau1 : tb->tau);
  const double a0 = mac.U[0] * itau;
  double nU[NPD];
#pragma unroll
  for (int q = 0; q < NPD; ++q) {
    double c0 = 0.0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      const double c = nhat<ST>(2 * q, a);
      if (c != 0.0) c0 += c * mac.U[a + 1];
    }
    nU[q] = c0 * itau;
  }
  // ---- reverse of the relaxation and of the equilibrium evaluation ----
  double a0b = 0.0, nUb[NPD], apb[B::NM];
#pragma unroll
  for (int q = 0; q < NPD; ++q) nUb[q] = 0.0;
#pragma unroll
  for (int k = 0; k < B::NM; ++k) apb[k] = 0.0;
#pragma unroll
  for (int j = 0; j < KR; ++j) {
    A fs[ND], ms[ND];
#pragma unroll
    for (int k = 0; k < ND; ++k) {
      fs[k] = fl[j * ND + k][tid];
      ms[k] = ml[j * ND + k][tid];
    }
    relax_vjp_shell<ST, N, A>(tb, j, fs, ms, ap, a0, nU, a0b, nUb, apb);
  }
  // Omega depends on tau through a0 = U^0 / tau and nU = (n . U) / tau
  double Ub[D + 1];
  Ub[0] = a0b * itau;
  double taub = -a0b * a0;
#pragma unroll
  for (int a = 1; a <= D; ++a) Ub[a] = 0.0;
#pragma unroll
  for (int q = 0; q < NPD; ++q) {
    taub -= nUb[q] * nU[q];
#pragma unroll
    for (int a = 0; a < D; ++a) {
      const double c = nhat<ST>(2 * q, a);
      if (c != 0.0) Ub[a + 1] += c * nUb[q] * itau;
    }
  }
  taub *= itau;
  // ---- reverse of the equilibrium coefficients, EOS, density and Landau frame ----
  double Mb[B::NM];
  coefficients_vjp<D, N>(tb, apb, Mb);
  double nb = 0.0, Tb = 0.0;
  basis_moments_vjp<D, N>(mac.n, mac.T, mac.U, m, rd, Mb, nb, Tb, Ub);
  double Nb[D + 1], Tbar[D + 1][D + 1], Ts[D + 1][D + 1];
  macro_vjp_moments<D>(tb, Nv, T, mac, nb, 0.0, Tb, Ub, Nb, Tbar);
#pragma unroll
  for (int a = 0; a <= D; ++a)
#pragma unroll
    for (int b = 0; b <= D; ++b) Ts[a][b] = 0.5 * (Tbar[a][b] + Tbar[b][a]);
  // ---- lam_t = mu (1 - Omega) + dL/dN^a p^a + dL/dT^ab p^a p^b, shell by shell ----
  asm volatile("" ::: "memory");
  const uint32_t so = (uint32_t)site * (uint32_t)sizeof(S);
  __attribute__((address_space(1))) S *lo = (__attribute__((address_space(1))) S *)lam;
#pragma unroll
  for (int j = 0; j < KR; ++j) {
    A ms[ND], out[ND];
#pragma unroll
    for (int k = 0; k < ND; ++k) ms[k] = ml[j * ND + k][tid];
    const double v = tb->sv[j];
#pragma unroll
    for (int qp = 0; qp < NPD; ++qp) {
      const double b = v * nU[qp];
      out[2 * qp] = (A)((double)ms[2 * qp] * (1.0 - (a0 - b)));
      out[2 * qp + 1] = (A)((double)ms[2 * qp + 1] * (1.0 - (a0 + b)));
    }
    moments_vjp_shell<ST, A, ND>(tb, j, Nb, Ts, out, 0);
#pragma unroll
    for (int k = 0; k < ND; ++k) {
      *(__attribute__((address_space(1))) S *)((__attribute__((address_space(1))) char *)(lo + k * sites) + so) = (S)out[k];
    }
    lo += ND * sites;
    one_after_another(lo);
  }
  if (dtau != nullptr) dtau[site] = dtau0 + taub;
}

// lam_{T+1}(x) = J_macro(F(x))^T g(x), F = S(B); g = (dL/dn, dL/deps, dL/dT, dL/dU)
template <class ST, int N, typename S, bool DEV, typename A = S>
__global__ void __launch_bounds__(256) k_moments_vjp(const Tables *__restrict__ tabs, const S *__restrict__ B,
                                                     FieldPtrs g, S *__restrict__ lam, int *err) {
  CTables *tb = (CTables *)tabs;
  constexpr int D = ST::D;
  int x, y, z;
  if (!site_xyz(tb, x, y, z)) return;
  const int64_t sites = tb->sites;
  const int64_t site = ((int64_t)z * tb->ny + y) * tb->nx + x;
  const Offs o = offs_periodic<ST, S>(tb, x, y, z);
  A f[ST::Q];
  pull_prod<ST, S, false, A>(tb, B, sites, o, f);
  double Nv[D + 1], T[D + 1][D + 1];
  moments_prod<ST, A, DEV>(tb, f, Nv, T);
  Macro<D> mac;
  mac.ok = landau_frame<D, 3>(T, mac.eps, mac.U);
  mac.n = lorentz_dot<D>(mac.U, Nv);
  mac.ok = temperature_2d(mac.eps / mac.n, tb->m, mac.T) && mac.ok && mac.n > 0.0 && mac.eps > 0.0;
  if (!mac.ok) set_err(err);
  double Ub[D + 1];
#pragma unroll
  for (int a = 0; a <= D; ++a) Ub[a] = g.U ? g.U[a * sites + site] : 0.0;
  const double nb = g.n ? g.n[site] : 0.0, eb = g.eps ? g.eps[site] : 0.0, Tb = g.T ? g.T[site] : 0.0;
  A out[ST::Q];
#pragma unroll
  for (int i = 0; i < ST::Q; ++i) out[i] = 0;
  macro_vjp<ST, A>(tb, Nv, T, mac, nb, eb, Tb, Ub, out);
  const uint32_t so = (uint32_t)site * (uint32_t)sizeof(S);
#pragma unroll
  for (int i = 0; i < ST::Q; ++i) *(S *)((char *)(lam + (int64_t)i * sites) + so) = (S)out[i];
}

// Reverse of the initial condition B_0 = C(f_0), f_0 = f^eq(n0, T0, U(u0)) (1 + amp xi):
// du0 (and dn0, dT0 when requested) from lam_1 = dL/dF_1; dtau(x) += dL/dtau(x).
template <class ST, int N, typename S, bool DEV, typename A = S>
__global__ void __launch_bounds__(256) k_init_vjp(const Tables *__restrict__ tabs, const double *__restrict__ n0,
                                                  const double *__restrict__ T0, const double *__restrict__ u0,
                                                  const double *__restrict__ noise, double amp,
                                                  const S *__restrict__ lam1, const void *__restrict__ tau_field,
                                                  double *__restrict__ du0, double *__restrict__ dn0,
                                                  double *__restrict__ dT0, double *__restrict__ dtau, int *err) {
  CTables *tb = (CTables *)tabs;
  constexpr int D = ST::D, Q = ST::Q;
  using B = BasisDef<D, N>;
  int x, y, z;
  if (!site_xyz(tb, x, y, z)) return;
  const int64_t sites = tb->sites;
  const int64_t site = ((int64_t)z * tb->ny + y) * tb->nx + x;
  double U[D + 1], u[D], uu = 0.0;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    u[a] = u0[a * sites + site];
    uu += u[a] * u[a];
  }
  const double gam = 1.0 / sqrt(1.0 - uu);
  U[0] = gam;
#pragma unroll
  for (int a = 0; a < D; ++a) U[a + 1] = gam * u[a];
  const double n = n0[site], T = T0[site];
  const RatiosD rd = ratios_2d_d(tb->m / T);
  Ratios rr;
  rr.r0 = rd.r0;
  rr.r2 = rd.r2;
  rr.r3 = rd.r3;
  double M[B::NM];
  basis_moments<D, N>(n, T, U, rr, M);
  double fe[Q];
  feq_prod<ST, N, double, false>(tb, M, fe);
  A f[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const double sc = noise ? 1.0 + amp * noise[(int64_t)i * sites + site] : 1.0;
    const double fi = fe[i] * sc;
    f[i] = DEV ? (A)(fi - tb->fref[i]) : (A)fi;
  }
  const Offs o = offs_periodic<ST, S>(tb, x, y, z);
  A mu[Q];
  pull_prod<ST, S, true, A>(tb, lam1, sites, o, mu);
  double taub;
  if (!collide_vjp<ST, N, A, DEV>(tb, f, mu, tau_at<S>(tb, tau_field, site), taub)) set_err(err);
  if (dtau != nullptr) dtau[site] += taub;
  // f now holds dL/df_0; through the noise factor to dL/df^eq
  double g[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) g[i] = (double)f[i] * (noise ? 1.0 + amp * noise[(int64_t)i * sites + site] : 1.0);
  double Mb[B::NM];
  feq_vjp<ST, N, double>(tb, g, Mb);
  double nb = 0.0, Tb = 0.0, Ub[D + 1];
#pragma unroll
  for (int a = 0; a <= D; ++a) Ub[a] = 0.0;
  basis_moments_vjp<D, N>(n, T, U, tb->m, rd, Mb, nb, Tb, Ub);
  // U = gamma (1, u):  dL/du_b = gamma Ub^b + gamma^3 u_b (Ub^0 + sum_a Ub^a u_a)
  double s = Ub[0];
#pragma unroll
  for (int a = 0; a < D; ++a) s += Ub[a + 1] * u[a];
  if (du0 != nullptr) {
#pragma unroll
    for (int a = 0; a < D; ++a) du0[a * sites + site] = gam * Ub[a + 1] + gam * gam * gam * u[a] * s;
  }
  if (dn0 != nullptr) dn0[site] = nb;
  if (dT0 != nullptr) dT0[site] = Tb;
}

template <class ST, int N, typename S, bool DEV, typename A = S>
static hipError_t launch_adj_t(const AdjointArgs &a) {
  const dim3 block(kAdjBX, kAdjBY, 1), grid = adjoint_grid(a);
  switch (a.op) {
    case ADJ_STEP:
      // float storage and arithmetic: the streamed kernel (two waves per SIMD); double storage or
      // arithmetic: the register-resident one (at order 3 a block's F_t and lam in double would take
      // 128 KB of LDS, one block per CU, which is what the registers allow too)
      if constexpr (sizeof(S) == 4 && sizeof(A) == 4)
        hipLaunchKernelGGL((k_adjoint_streamed<ST, N, S, DEV>), grid, block, 0, a.stream, a.tb, (const S *)a.state,
                           (const S *)a.lam_in, (S *)a.lam_out, a.tau_field, a.dtau, a.err);
      else if constexpr (sizeof(S) == 8)
        return launch_adjoint_step_f64(a);
      else
        hipLaunchKernelGGL((k_adjoint<ST, N, S, DEV, A>), grid, block, 0, a.stream, a.tb, (const S *)a.state,
                           (const S *)a.lam_in, (S *)a.lam_out, a.tau_field, a.dtau, a.err);
      break;
    case ADJ_MOMENTS:
      hipLaunchKernelGGL((k_moments_vjp<ST, N, S, DEV, A>), grid, block, 0, a.stream, a.tb, (const S *)a.state,
                         a.grads, (S *)a.lam_out, a.err);
      break;
    case ADJ_INIT:
      hipLaunchKernelGGL((k_init_vjp<ST, N, S, DEV, A>), grid, block, 0, a.stream, a.tb, a.n0, a.T0, a.u0, a.noise,
                         a.amp, (const S *)a.lam_in, a.tau_field, a.du0, a.dn0, a.dT0, a.dtau, a.err);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// storage 0: double; 1: float deviations updated in float; 2: float deviations updated in double
template <class ST, int N>
static hipError_t launch_adj_storage(const AdjointArgs &a) {
  if (a.storage == 0) return launch_adj_t<ST, N, double, false>(a);
  if (a.storage == 1) return launch_adj_t<ST, N, float, true>(a);
  return launch_adj_t<ST, N, float, true, double>(a);
}

hipError_t launch_adjoint(const AdjointArgs &a) {
  if (a.stencil != ST_PROD2D) return hipErrorInvalidValue;
  if (a.order == 2) return launch_adj_storage<Stencil<ST_PROD2D, 3>, 2>(a);
  return launch_adj_storage<Stencil<ST_PROD2D, 4>, 3>(a);
}

}  // namespace rlbm
