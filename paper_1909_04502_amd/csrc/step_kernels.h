// step_kernels.h -- HIP kernels of the RLBM update for gfx950 (MI355X) and their launches, one source
// per stencil family (step_*.hip) so that the families compile side by side.
//
// Design (memory-bound: 2 Q words of HBM traffic per site update):
//  * populations in SoA planes f[i][z][y][x]; one thread per site, 64-wide
//    wavefronts along x so every population plane is read and written with
//    fully coalesced 512 B (f64) / 256 B (f32) wavefront accesses;
//  * fused pull-stream + collide: the pre-collision value of population i at
//    x is read from the post-collision planes at the upstream taps (a pure
//    shift on-lattice; bilinear / trilinear interpolation off-lattice, taps
//    and their count fixed at compile time from the direction signs, weights
//    from the per-lattice table); neighbouring taps of a wavefront hit the
//    same cache lines, so the extra taps are served from L1/L2, not HBM;
//  * all constant tables are read through uniform (scalar) loads;
//  * antipodal populations are processed in pairs: sums and differences feed
//    the even / odd halves of the moments and of the projected equilibrium,
//    halving both the moment and the equilibrium arithmetic;
//  * the Landau eigenproblem, equation of state and equilibrium moments are
//    evaluated in double for every storage mode.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include <type_traits>
#include <utility>

#include "device_math.h"
#include "kernels.h"
#include "massive_math.h"
#include "prod_math.h"
#include "stage2d.h"

namespace rlbm {

// Moments of the shifted monomials (p^0 - m) p^e = p^0 p^e - m p^e, in place
// (stencils whose projection rows act on the shifted basis).
template <int D, int N>
__device__ __forceinline__ void shift_basis_moments(double m, double (&M)[BasisDef<D, N>::NM]) {
  constexpr ClassTable<D, N> CL{};
#pragma unroll
  for (int k = 0; k < BasisDef<D, N>::NM; ++k)
    if (CL.partner[k] >= 0) M[k] -= m * M[CL.partner[k]];
}

template <int D>
__device__ __forceinline__ void write_fields(const FieldPtrs &fp, int64_t site, int64_t sites, const Macro<D> &mac) {
  if (fp.n) fp.n[site] = mac.n;
  if (fp.eps) fp.eps[site] = mac.eps;
  if (fp.T) fp.T[site] = mac.T;
  if (fp.U) {
#pragma unroll
    for (int a = 0; a <= D; ++a) fp.U[a * sites + site] = mac.U[a];
  }
}

__device__ __forceinline__ void flag_error(int *err) {
  // all writers store the same value: a benign race, and a plain store (a volatile one would make
  // the wave wait for every load it has in flight)
  *err = 1;
}

template <typename S>
__device__ __forceinline__ double site_tau(CTables *tb, const void *tau_field, int64_t site) {
  // the lattice's tau through a scalar load, chosen by value (a per-site load through a pointer
  // picked between the field and the table would be a vector load the wave waits for)
  const double tau = tb->tau;
  if (tau_field == nullptr) return tau;
  return (double)((const S *)tau_field)[site];
}

// ---------------------------------------------------------------------------
// Kernels
// ---------------------------------------------------------------------------
template <class ST, typename S>
__device__ __forceinline__ Offs make_offs(CTables *tb, int x, int y) {
  Offs o;
  const uint32_t nx = tb->nx;
#pragma unroll
  for (int d = -1; d <= 1; ++d) {
    o.x[d + 1] = (uint32_t)near_site(x + d, tb->nx, tb->open[0]) * (uint32_t)sizeof(S);
    o.y[d + 1] = (uint32_t)near_site(y + d, tb->ny, tb->open[1]) * nx * (uint32_t)sizeof(S);
    o.z[d + 1] = 0u;
  }
  return o;
}

// Integer streaming: population I at the site comes from x - n_I.  The byte
// offsets of the upstream rows are computed once per axis and distance (up to
// ST::RMAX sites), so each population costs one add and one load.
template <class ST, typename S, int R, int... I>
__device__ __forceinline__ void gather_onlat_impl(const S *__restrict__ fin, int64_t sites, const uint32_t (&ox)[2 * R + 1],
                                                  const uint32_t (&oy)[2 * R + 1], S (&f)[ST::Q],
                                                  std::integer_sequence<int, I...>) {
  ((f[I] = *(const S *)((const char *)(fin + (int64_t)I * sites) + (ox[R - ST::dir(I, 0)] + oy[R - ST::dir(I, 1)]))), ...);
}

template <class ST, typename S>
__device__ __forceinline__ void gather_onlat(CTables *tb, const S *__restrict__ fin, int64_t sites,
                                             int x, int y, S (&f)[ST::Q]) {
  constexpr int R = ST::RMAX;
  // byte offsets of the columns x + k - R and the rows y + k - R (k = 0 .. 2R)
  uint32_t ox[2 * R + 1], oy[2 * R + 1];
  const uint32_t nx = tb->nx;
#pragma unroll
  for (int k = 0; k <= 2 * R; ++k) {
    ox[k] = (uint32_t)near_site(x + k - R, tb->nx, tb->open[0]) * (uint32_t)sizeof(S);
    oy[k] = (uint32_t)near_site(y + k - R, tb->ny, tb->open[1]) * nx * (uint32_t)sizeof(S);
  }
  gather_onlat_impl<ST, S, R>(fin, sites, ox, oy, f, std::make_integer_sequence<int, ST::Q>{});
}

// pre-collision populations at the site, in the arithmetic type A (the storage type S, or double
// for float deviations updated in double: product rules)
template <class ST, typename S, typename A = S>
__device__ __forceinline__ void gather(CTables *tb, const S *__restrict__ fin, int64_t sites, int x,
                                       int y, A (&f)[ST::Q]) {
  if constexpr (ST::ONLAT) {
    static_assert(sizeof(A) == sizeof(S), "on-lattice rules compute in their storage type");
    gather_onlat<ST, S>(tb, fin, sites, x, y, f);
  } else {
    const Offs o = make_offs<ST, S>(tb, x, y);
    pull_prod<ST, S, false, A>(tb, fin, sites, o, f);
  }
}

// Collision of one site: f (pre-collision, storage precision; deviations in
// the F32_DEV mode) is replaced by f* in place; returns the macro state of the
// pre-collision populations.  wallT: see site_wall (negative off the walls).
template <class ST, int N, typename S, bool DEV, bool RELAX, bool EXT = false>
__device__ __forceinline__ Macro<ST::D> collide_site(CTables *tb, S (&f)[ST::Q], double tau,
                                                     double wallT = -1.0) {
  if constexpr (ST::ONLAT)
    return collide_massive<ST, N, S, DEV, RELAX, EXT>(tb, f, tau, wallT);
  else
    return collide_prod<ST, N, S, DEV, RELAX, EXT>(tb, f, tau, wallT);
}

// Site of this thread.
__device__ __forceinline__ bool site_coords(CTables *tb, const Tiling &tl, int &x, int &y) {
  int x0, y0;
  tile_origin(tl, x0, y0);
  x = x0 + threadIdx.x;
  y = y0 + threadIdx.y;
  return x < tb->nx && y < tb->ny;
}

// The register kernel: one site per thread, all taps asked for at once.  Where the two states fit the Infinity Cache
// it is bound by the vector instructions a SIMD's waves issue (4 clocks each; order 3 in float 1240 a wave, 8 of 17 us
// at 512 x 512), by the taps' latency before them and by the launch, not by memory.  A fifth of those instructions
// used to move scalars that did not fit the scalar registers (all planes' addresses and all tables at once) and to
// form quotients for the tile's place: see one_after_another, from_here_on and tile_origin.  Per step, before ->
// after: float 512 x 512 19.2 -> 16.4 us, 1024 x 1024 59 -> 52; float with double arithmetic 512 x 512 24.3 -> 19.8;
// double 64 x 64 7.5 -> 5.7, 300 x 301 13.9 -> 12.4; massive order 3 512 x 512 39 -> 34 (a copy of its bytes takes 36);
// massless order 3 512 x 512 38 -> 32.  Past the Infinity Cache the double build, which holds 209 registers instead of
// 153, is 2-3 % slower than it was (1026 x 1026 130 -> 134): the staged kernel is the default there.
template <class ST, int N, typename S, bool DEV, int OCC, bool EXT, bool NT, typename A = S>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OCC > 0 ? OCC : 1, 8))) k_step(const Tables *__restrict__ tabs, const S *__restrict__ fin,
                                              S *__restrict__ fout, const void *__restrict__ tau_field,
                                              FieldPtrs last, int *err, Tiling tl) {
  CTables *tb = (CTables *)tabs;
  int x, y;
  if (!site_coords(tb, tl, x, y)) return;
  const int64_t sites = tb->sites;
  const int64_t site = (int64_t)y * tb->nx + x;
  // asked for with the populations: without a field a place in the state instead, unused (a load under a condition
  // would be waited for at once, with all the others)
  const S tau1 = (tau_field != nullptr ? (const S *)tau_field : fin)[site];
  A f[ST::Q];
  gather<ST, S, A>(tb, fin, sites, x, y, f);
  const double tau = tau_field != nullptr ? (double)tau1 : tb->tau;
  const Macro<ST::D> mac = collide_site<ST, N, A, DEV, true, EXT>(tb, f, tau, EXT ? site_wall(tb, x, y, -1) : -1.0);
  if (!mac.ok) flag_error(err);
  put_pops<NT>(fout, sites, (uint32_t)site * (uint32_t)sizeof(S), f);
  if (last.any) write_fields<ST::D>(last, site, sites, mac);
}

// One 64 x 4 tile per block in the band order, its populations pulled through LDS (stage2d.h).  Bound by
// HBM where the two states do not fit the Infinity Cache: the register kernels fetch every row of a
// window once per wave that reads it, which there costs memory traffic and lines in flight.  Per step,
// order 3: 103 us at 1024 x 1024 in double (5.2 TB/s of what a step has to move, the rate of an ordinary
// copy; a non-temporal one reaches 5.9 in the same layout and 6.9 flat; register kernel 123, windows of 5
// full rows in 16-byte chunks 107), 60 with walls and a force at 700 x 801 (register 76), 119 at
// 1023 x 1025 (132), 371 at 2048 x 2048 in long runs (395 to 413 over the first 22 launches; register 495
// and 507, windows of full rows 394); order 2 at 1025 x 1023 87 (103).
template <class ST, int N, typename S, bool DEV, bool EXT, bool NT, bool WIDE, typename A = S>
__global__ void __launch_bounds__(256) k_step_lds(const Tables *__restrict__ tabs, const S *__restrict__ fin,
                                                  S *__restrict__ fout, const void *__restrict__ tau_field,
                                                  FieldPtrs last, int *err, Tiling tl) {
  CTables *tb = (CTables *)tabs;
  __shared__ __attribute__((aligned(16))) S buf[2 * Stage2D<ST, S>::E];
  int x0, y0;
  tile_origin(tl, x0, y0);
  const int x = x0 + threadIdx.x, y = y0 + threadIdx.y;
  const int64_t sites = tb->sites;
  A f[ST::Q];
  stage_pull<ST, S, A, WIDE>(tb, fin, sites, x0, y0, buf, f);
  if (x >= tb->nx || y >= tb->ny) return;
  const int64_t site = (int64_t)y * tb->nx + x;
  const double tau = site_tau<S>(tb, tau_field, site);
  const Macro<ST::D> mac = collide_site<ST, N, A, DEV, true, EXT>(tb, f, tau, EXT ? site_wall(tb, x, y, -1) : -1.0);
  if (!mac.ok) flag_error(err);
  put_pops<NT>(fout, sites, (uint32_t)site * (uint32_t)sizeof(S), f);
  if (last.any) write_fields<ST::D>(last, site, sites, mac);
}

template <class ST, int N, typename S, bool DEV, typename A = S>
__global__ void __launch_bounds__(256) k_moments(const Tables *__restrict__ tabs, const S *__restrict__ fin,
                                                 FieldPtrs out, int *err, Tiling tl) {
  CTables *tb = (CTables *)tabs;
  int x, y;
  if (!site_coords(tb, tl, x, y)) return;
  const int64_t sites = tb->sites;
  const int64_t site = (int64_t)y * tb->nx + x;
  A f[ST::Q];
  gather<ST, S, A>(tb, fin, sites, x, y, f);
  const Macro<ST::D> mac = collide_site<ST, N, A, DEV, false>(tb, f, 1.0);
  if (!mac.ok) flag_error(err);
  write_fields<ST::D>(out, site, sites, mac);
}

// f(x, 0) = f^eq(n0, T0, U(u0)) (1 + amp xi), then collide; store f*(x, 0).
template <class ST, int N, typename S, bool DEV, typename A = S>
__global__ void __launch_bounds__(256) k_init(const Tables *__restrict__ tabs, const double *__restrict__ n0,
                                              const double *__restrict__ T0, const double *__restrict__ u0,
                                              const double *__restrict__ noise, double amp, S *__restrict__ fout,
                                              const void *__restrict__ tau_field, FieldPtrs fields0, int *err,
                                              Tiling tl) {
  CTables *tb = (CTables *)tabs;
  constexpr int D = ST::D, Q = ST::Q, NP = Q / 2;
  using B = BasisDef<D, N>;
  int x, y;
  if (!site_coords(tb, tl, x, y)) return;
  const int64_t sites = tb->sites;
  const int64_t site = (int64_t)y * tb->nx + x;
  double U[D + 1], uu = 0.0;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    U[a + 1] = u0[a * sites + site];
    uu += U[a + 1] * U[a + 1];
  }
  const double g = 1.0 / sqrt(1.0 - uu);
  U[0] = g;
#pragma unroll
  for (int a = 1; a <= D; ++a) U[a] *= g;
  const double n = n0[site], T = T0[site];
  const Ratios rr = ratios_2d(tb->m / T);
  if (!(uu < 1.0) || !(n > 0.0) || !(T > 0.0)) flag_error(err);
  double M[B::NM];
  basis_moments<D, N>(n, T, U, rr, M);
  if constexpr (ST::SHIFT) shift_basis_moments<D, N>(tb->m, M);
  double fd[Q];
#pragma unroll
  for (int pr = 0; pr < NP; ++pr) {
    double E = 0.0, O = 0.0;
#pragma unroll
    for (int k = 0; k < B::NE; ++k) E += tb->Re[pr][k] * M[k];
#pragma unroll
    for (int k = 0; k < B::NO; ++k) O += tb->Ro[pr][k] * M[B::NE + k];
    fd[2 * pr] = E + O;
    fd[2 * pr + 1] = E - O;
  }
  if constexpr ((Q & 1) != 0) {
    double E = 0.0;
#pragma unroll
    for (int k = 0; k < B::NE; ++k) E += tb->Rrest[k] * M[k];
    fd[Q - 1] = E;
  }
  if (noise != nullptr) {
#pragma unroll
    for (int i = 0; i < Q; ++i) fd[i] *= 1.0 + amp * noise[(int64_t)i * sites + site];
  }
  // the update's form: f, or the deviations f - f^ref (in float, or in double when float deviations
  // are updated in double)
  A f[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) f[i] = DEV ? (A)(fd[i] - tb->fref[i]) : (A)fd[i];
  const double tau = site_tau<S>(tb, tau_field, site);
  const Macro<D> mac = collide_site<ST, N, A, DEV, true, true>(tb, f, tau, site_wall(tb, x, y, -1));
  if (!mac.ok) flag_error(err);
  put_pops<false>(fout, sites, (uint32_t)site * (uint32_t)sizeof(S), f);
  if (fields0.any) write_fields<D>(fields0, site, sites, mac);
}

// ---------------------------------------------------------------------------
// Dispatch
// ---------------------------------------------------------------------------
template <class ST, int N, typename S, bool DEV, typename A = S>
static hipError_t launch_t(const LaunchArgs &a) {
  const Variant vr = kVariants[(a.op == OP_STEP && a.variant >= 0 && a.variant < kNumVariants) ? a.variant : 0];
  const Tiling tl = tiling(a.nx, a.ny, vr.bx, vr.by * vr.bz, vr.xcd != 0);
  const dim3 block(tl.bx, tl.by, 1), grid((unsigned)tl.nb, 1, 1);
  static_assert(ST::D == 2, "the 3D rules: split.hip, split_onlat.hip, split_ur3d.hip");
  switch (a.op) {
    case OP_STEP: {
      // one instantiation per (occupancy target 0, 2 or 4, force/walls, store kind)
      auto go = [&](auto occ, auto ext, auto nt) {
        constexpr int O = decltype(occ)::value;
        constexpr bool E = decltype(ext)::value, T = decltype(nt)::value;
        hipLaunchKernelGGL((k_step<ST, N, S, DEV, O, E, T, A>), grid, block, 0, a.stream, a.tb, (const S *)a.fin,
                           (S *)a.fout, a.tau_field, a.fields, a.err, tl);
      };
      using O0 = std::integral_constant<int, 0>;
      using O2 = std::integral_constant<int, 2>;
      using O4 = std::integral_constant<int, 4>;
      using F = std::false_type;
      using T = std::true_type;
      const bool ext = a.ext;
      if constexpr (!ST::ONLAT) {
        if (vr.lds) {
          const Tiling ltl = tiling(a.nx, a.ny, 64, 4, 1);
          auto launch_lds = [&](auto ext, auto nt, auto wd) {
            constexpr bool E = decltype(ext)::value, T = decltype(nt)::value, W = decltype(wd)::value;
            hipLaunchKernelGGL((k_step_lds<ST, N, S, DEV, E, T, W, A>), dim3((unsigned)ltl.nb, 1, 1), dim3(64, 4, 1), 0,
                               a.stream, a.tb, (const S *)a.fin, (S *)a.fout, a.tau_field, a.fields, a.err, ltl);
          };
          auto lds = [&](auto ext, auto nt) {
            if constexpr (sizeof(S) == 8 && !decltype(ext)::value)
              if (stage_wide(a.fin, a.nx, (int)sizeof(S), a.open_x)) return launch_lds(ext, nt, T{});
            launch_lds(ext, nt, F{});
          };
          if (ext) {
            if (a.nt) lds(T{}, T{});
            else lds(T{}, F{});
          } else {
            if (a.nt) lds(F{}, T{});
            else lds(F{}, F{});
          }
          break;
        }
      }
      if (ext) {
        if (a.nt) go(O0{}, T{}, T{});
        else go(O0{}, T{}, F{});
      } else if (vr.occ == 2) {
        if (a.nt) go(O2{}, F{}, T{});
        else go(O2{}, F{}, F{});
      } else if (vr.occ == 4) {
        if (a.nt) go(O4{}, F{}, T{});
        else go(O4{}, F{}, F{});
      } else {
        if (a.nt) go(O0{}, F{}, T{});
        else go(O0{}, F{}, F{});
      }
      break;
    }
    case OP_MOMENTS:
      hipLaunchKernelGGL((k_moments<ST, N, S, DEV, A>), grid, block, 0, a.stream, a.tb, (const S *)a.fin, a.fields,
                         a.err, tl);
      break;
    case OP_INIT:
      hipLaunchKernelGGL((k_init<ST, N, S, DEV, A>), grid, block, 0, a.stream, a.tb, a.n0, a.T0, a.u0, a.noise,
                         a.amp, (S *)a.fout, a.tau_field, a.fields, a.err, tl);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// storage 0: double; 1: float deviations updated in float; 2: float deviations updated in double
// (product rules)
template <class ST, int N>
static hipError_t launch_storage(const LaunchArgs &a) {
  if (a.storage == 0) return launch_t<ST, N, double, false>(a);
  if (a.storage == 1) return launch_t<ST, N, float, true>(a);
  if constexpr (!ST::ONLAT) return launch_t<ST, N, float, true, double>(a);
  return hipErrorInvalidValue;
}

}  // namespace rlbm
