// split_onlat.hip -- the 143-vector massive rule in 3D, one site's populations spread over the waves of a block
// as in split.hip (HIP, gfx950).
//
// Wave w of a block takes some of the stencil's groups for 64 sites: it loads their populations (one load each:
// integer shifts), adds up their part of the moments, and relaxes and stores them once the state is known.  So
// every population is read once (38 values per lane; the step kernels hold them in registers but for 10 values in
// scratch, 13 with walls and force).  One thread per site could not hold all 143: the double form read 95 of them
// twice and waited for each group's second load, the float form had 188 bytes of scratch per lane, now 44 or 56.
// Bound by memory: 4.8-4.9 TB/s of population traffic at 192^3, where a plain copy of as many bytes reaches 5.7.
// Per step, against one thread per site:
//   192^3 double             3.28 ms    4.02
//   130 x 97 x 83 double     0.56 ms    0.84
//   192^3 float              1.68 ms    1.90
//   40 x 33 x 30 double      0.028 ms   0.034
// (occupancy targets: double 3 waves per SIMD, 2 gives 3.38 ms and 4 spills, 6.9; float 4: 3 spill nothing and are as
// fast on large lattices, but 40 x 33 x 30 takes 21.9 us instead of 17.4)
#define RLBM_TABLES_PLAIN   // device_math.h
#include <hip/hip_runtime.h>

#include "device_math.h"
#include "kernels.h"
#include "massive_math.h"
#include "split_math.h"

namespace rlbm {

// Groups of wave w (NG marks the rest population): about equally many populations each.
template <class ST>
struct WaveGroups;
template <>
struct WaveGroups<Stencil<ST_MASSIVE3D, 3>> {
  static constexpr int W = 4, MAX = 38, PER = 3;
  static constexpr int g[W][PER] = {{3, 4, -1}, {5, 6, 10}, {8, 1, 7}, {9, 0, 2}};
};
// Populations of the e-th group of wave P: the first, and how many; and where they lie among the wave's.
template <class ST>
RLBM_HD constexpr int wg_count(int p, int e) {
  const int g = WaveGroups<ST>::g[p][e];
  return g < 0 ? 0 : (g == ST::NG ? 1 : ST::gcount(g));
}
template <class ST>
RLBM_HD constexpr int wg_first(int p, int e) {
  const int g = WaveGroups<ST>::g[p][e];
  return g < 0 ? 0 : (g == ST::NG ? ST::Q - 1 : ST::gfirst(g));
}
template <class ST>
RLBM_HD constexpr int wg_at(int p, int e) {
  int n = 0;
  for (int i = 0; i < e; ++i) n += wg_count<ST>(p, i);
  return n;
}
template <class ST>
RLBM_HD constexpr bool wg_complete() {
  int n = 0;
  for (int p = 0; p < WaveGroups<ST>::W; ++p) {
    int c = 0;
    for (int e = 0; e < WaveGroups<ST>::PER; ++e) c += wg_count<ST>(p, e);
    if (c > WaveGroups<ST>::MAX) return false;
    n += c;
  }
  return n == ST::Q;
}
static_assert(wg_complete<Stencil<ST_MASSIVE3D, 3>>(), "every group has its wave");

template <class ST, int P, typename S>
__device__ __forceinline__ void load_groups(CTables *tb, const S *__restrict__ fin, int x, int y, int z,
                                            S (&f)[WaveGroups<ST>::MAX]) {
  constexpr int R = ST::RMAX;
  typedef const __attribute__((address_space(1))) char gchar;
  typedef const __attribute__((address_space(1))) S gS;
  uint32_t ox[2 * R + 1], oy[2 * R + 1], oz[2 * R + 1];
  const uint32_t es = sizeof(S), nx = tb->nx, nxy = nx * (uint32_t)tb->ny;
#pragma unroll
  for (int k = 0; k <= 2 * R; ++k) {
    ox[k] = (uint32_t)near_site(x + k - R, tb->nx, tb->open[0]) * es;
    oy[k] = (uint32_t)near_site(y + k - R, tb->ny, tb->open[1]) * nx * es;
    oz[k] = (uint32_t)near_site(z + k - R, tb->nz, tb->open[2]) * nxy * es;
  }
  const int64_t plane = tb->sites * (int64_t)es;
#pragma unroll
  for (int e = 0; e < WaveGroups<ST>::PER; ++e)
#pragma unroll
    for (int n = 0; n < wg_count<ST>(P, e); ++n) {
      const int i = wg_first<ST>(P, e) + n;
      f[wg_at<ST>(P, e) + n] = *(gS *)((gchar *)fin + (int64_t)i * plane +
                                       (ox[R - ST::dir(i, 0)] + oy[R - ST::dir(i, 1)] + oz[R - ST::dir(i, 2)]));
    }
}

// The moments of wave P's populations, to LDS.
template <class ST, int P, typename A, class X>
__device__ __forceinline__ void group_moments(CTables *tb, const A (&f)[WaveGroups<ST>::MAX], int lane,
                                              X &sh) {
  Moments3<A> mom;
#pragma unroll
  for (int e = 0; e < WaveGroups<ST>::PER; ++e) {
    constexpr int NG = ST::NG;
    const int g = WaveGroups<ST>::g[P][e], first = wg_first<ST>(P, e), at = wg_at<ST>(P, e);
    if (g < 0) continue;
    if (g == NG) {   // the rest population
      const double m = tb->m;
      mom.N0 += (A)m * f[at];
      mom.T00 += (A)(m * m) * f[at];
      continue;
    }
    A S0 = 0, Sa[3] = {0, 0, 0}, Sab[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int n = 0; n < wg_count<ST>(P, e); n += 2) {
      const int i = first + n;
      const A s = f[at + n] + f[at + n + 1], d = f[at + n] - f[at + n + 1];
      S0 += s;
      int ab = 0;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const int c = ST::dir(i, a);
        if (c == 1) Sa[a] += d;
        else if (c == -1) Sa[a] -= d;
        else if (c != 0) Sa[a] += (A)c * d;
#pragma unroll
        for (int b = a; b < 3; ++b) {
          const int cc = ST::dir(i, a) * ST::dir(i, b);
          if (cc == 1) Sab[ab] += s;
          else if (cc == -1) Sab[ab] -= s;
          else if (cc != 0) Sab[ab] += (A)cc * s;
          ++ab;
        }
      }
    }
    const A p0 = tab<A>(tb->mgrp[g][0], tb->mgrpf[g][0]), p00 = tab<A>(tb->mgrp[g][1], tb->mgrpf[g][1]);
    const A v = tab<A>(tb->mgrp[g][2], tb->mgrpf[g][2]), p0v = tab<A>(tb->mgrp[g][3], tb->mgrpf[g][3]);
    const A vv = tab<A>(tb->mgrp[g][4], tb->mgrpf[g][4]);
    mom.N0 += p0 * S0;
    mom.T00 += p00 * S0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      mom.Na[a] += v * Sa[a];
      mom.T0a[a] += p0v * Sa[a];
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) mom.Tab[a] += vv * Sab[a];
  }
  put_moments(mom, lane, sh.mom[P]);
}

// Steps 5 and 8 (and the force) of wave P's populations, and their store.
template <class ST, int N, int P, typename S, bool DEV, bool EXT, bool NT, typename A, class X>
__device__ __forceinline__ void relax_groups(CTables *tb, const X &sh, int lane, const A (&f)[WaveGroups<ST>::MAX],
                                             uint32_t site_off, S *__restrict__ fout) {
  constexpr AngTable<3, N> AT{};
  const int64_t sites = tb->sites;
  const A a0 = sh.om[0][lane];
  A ub[3], gv[3] = {0, 0, 0}, cF = 0, gU = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) ub[a] = sh.om[1 + a][lane];
  if constexpr (EXT) {
    cF = sh.om[4][lane];
#pragma unroll
    for (int a = 0; a < 3; ++a) gv[a] = sh.om[5 + a][lane];
    gU = sh.om[8][lane];
  }
  // full equilibrium of population i from its deviation part (float-deviation storage)
  auto full = [&](int i, A e) { return DEV ? e + tab<A>(tb->fref[i], tb->freff[i]) : e; };
  auto put = [&](int i, A v) { put_pop<NT>(fout, sites, site_off, i, (S)v); };
#pragma unroll
  for (int e = 0; e < WaveGroups<ST>::PER; ++e) {
    constexpr int NG = ST::NG;
    const int g = WaveGroups<ST>::g[P][e], first = wg_first<ST>(P, e), at = wg_at<ST>(P, e);
    if (g < 0) continue;
    if (g == NG) {
      const A E = sh.ap[0][lane] * tab<A>(tb->wrest, tb->wrestf);   // the constant monomial is basis entry 0
      A out = f[at] + a0 * (E - f[at]);
      if constexpr (EXT) out -= cF * gU * full(ST::Q - 1, E);
      put(ST::Q - 1, out);
      continue;
    }
    // a' is read again for each group rather than kept in registers across them
    asm volatile("" ::: "memory");
    A ce[20];
#pragma unroll
    for (int q = 0; q < AT.n; ++q) {
      const int l = AT.e[q][0] + AT.e[q][1] + AT.e[q][2];
      A acc = 0;
      if (AT.m0[q] >= 0) acc += sh.ap[AT.m0[q]][lane] * tab<A>(tb->mgrp[g][5 + l], tb->mgrpf[g][5 + l]);
      if (AT.m1[q] >= 0) acc += sh.ap[AT.m1[q]][lane] * tab<A>(tb->mgrp[g][9 + l], tb->mgrpf[g][9 + l]);
      ce[q] = acc;
    }
#pragma unroll
    for (int n = 0; n < wg_count<ST>(P, e); n += 2) {
      const int i = first + n;
      A E = 0, O = 0, b = 0, gn = 0;
#pragma unroll
      for (int q = 0; q < AT.n; ++q) {
        const int c = ipow_dir<ST>(i, AT.e[q][0], AT.e[q][1], AT.e[q][2]);
        if (c == 0) continue;
        const A t = c == 1 ? ce[q] : (c == -1 ? -ce[q] : (A)c * ce[q]);
        if ((AT.e[q][0] + AT.e[q][1] + AT.e[q][2]) & 1) O += t;
        else E += t;
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const int c = ST::dir(i, a);
        if (c == 0) continue;
        b += (A)c * ub[a];
        if constexpr (EXT) gn += (A)c * gv[a];
      }
      const A f0 = f[at + n], f1 = f[at + n + 1];
      A out0 = f0 + (a0 - b) * ((E + O) - f0), out1 = f1 + (a0 + b) * ((E - O) - f1);
      if constexpr (EXT) {   // + (m/T) ((g . v) U^0 - g . U) f^eq
        out0 += cF * (gn - gU) * full(i, E + O);
        out1 += cF * (-gn - gU) * full(i + 1, E - O);
      }
      put(i, out0);
      put(i + 1, out1);
    }
  }
}

// body(std::integral_constant<int, w>) for this wave's w
template <int W, int P = 0, class F>
__device__ __forceinline__ void for_wave(int w, F &&body) {
  if (w == P) body(std::integral_constant<int, P>{});
  else if constexpr (P + 1 < W) for_wave<W, P + 1>(w, body);
}

// The update from wave w's pre-collision populations f on (RELAX = false: the fields alone).
template <class ST, int N, typename S, bool DEV, bool RELAX, bool EXT, bool NT>
__device__ __forceinline__ void onlat_update(CTables *tb, OnlatLds<N, WaveGroups<ST>::W, S> &sh, int w, int lane,
                                             bool live, int x, int y, int z, const S (&f)[WaveGroups<ST>::MAX],
                                             S *__restrict__ fout, const void *__restrict__ tau_field, const FieldPtrs &fields,
                                             int *err) {
  constexpr int W = WaveGroups<ST>::W;
  const uint32_t site = ((uint32_t)z * tb->ny + y) * tb->nx + x;
  for_wave<W>(w, [&](auto p) { group_moments<ST, decltype(p)::value>(tb, f, lane, sh); });
  __syncthreads();
  if (w == (int)((blockIdx.x / 8) % W))
    onlat_state<N, W, S, DEV, RELAX, EXT>(tb, sh, lane, live, x, y, z, site, tau_field, fields, err);
  if constexpr (!RELAX) return;
  __syncthreads();
  split_coefficients<N, W, DEV, S>(tb, w, lane, sh);
  __syncthreads();
  if (!live) return;
  for_wave<W>(w, [&](auto p) {
    relax_groups<ST, N, decltype(p)::value, S, DEV, EXT, NT>(tb, sh, lane, f, site * (uint32_t)sizeof(S), fout);
  });
}

template <class ST, int N, typename S, bool DEV, bool RELAX, bool EXT, bool NT>
__global__ void __launch_bounds__(64 * WaveGroups<ST>::W) __attribute__((amdgpu_waves_per_eu(sizeof(S) == 8 ? 3 : 4, 8)))
k_step_onlat3d(const Tables *__restrict__ tabs, const S *__restrict__ fin, S *__restrict__ fout,
               const void *__restrict__ tau_field, FieldPtrs fields, int *err, SplitTiling tl) {
  CTables *tb = (CTables *)tabs;
  constexpr int W = WaveGroups<ST>::W;
  __shared__ OnlatLds<N, W, S> sh;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int x, y;
  SplitRun run;
  if (!split_site<false>(tb, tl, lane, run, x, y)) return;
  S f[WaveGroups<ST>::MAX];
  for_wave<W>(w, [&](auto p) { load_groups<ST, decltype(p)::value>(tb, fin, x, y, run.z, f); });
  onlat_update<ST, N, S, DEV, RELAX, EXT, NT>(tb, sh, w, lane, lane < run.live, x, y, run.z, f, fout, tau_field, fields, err);
}

// f(x, 0) = f^eq(n0, T0, U(u0)) (1 + amp xi) from the projection rows, then collide; store f*(x, 0).
template <class ST, int N, typename S, bool DEV, bool EXT>
__global__ void __launch_bounds__(64 * WaveGroups<ST>::W) k_init_onlat3d(
    const Tables *__restrict__ tabs, const double *__restrict__ n0, const double *__restrict__ T0, const double *__restrict__ u0,
    const double *__restrict__ noise, double amp, S *__restrict__ fout, const void *__restrict__ tau_field, FieldPtrs fields,
    int *err, SplitTiling tl) {
  CTables *tb = (CTables *)tabs;
  constexpr int W = WaveGroups<ST>::W;
  using B = BasisDef<3, N>;
  __shared__ OnlatLds<N, W, S> sh;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int x, y;
  SplitRun run;
  if (!split_site<false>(tb, tl, lane, run, x, y)) return;
  const bool live = lane < run.live;
  const int64_t sites = tb->sites;
  const uint32_t site = ((uint32_t)run.z * tb->ny + y) * tb->nx + x;
  double M[B::NM];
  if (!first_moments3<N>(tb, n0, T0, u0, site, M) && live) *err = 1;
  if constexpr (ST::SHIFT) {   // moments of (p^0 - m) p^e = p^0 p^e - m p^e
    constexpr ClassTable<3, N> CL{};
#pragma unroll
    for (int k = 0; k < B::NM; ++k)
      if (CL.partner[k] >= 0) M[k] -= tb->m * M[CL.partner[k]];
  }
  S f[WaveGroups<ST>::MAX];
  auto value = [&](int i, double fd) {
    if (noise != nullptr) fd *= 1.0 + amp * noise[(int64_t)i * sites + site];
    return DEV ? (S)(fd - tb->fref[i]) : (S)fd;
  };
  for_wave<W>(w, [&](auto p_) {
    constexpr int P = decltype(p_)::value;
#pragma unroll
    for (int e = 0; e < WaveGroups<ST>::PER; ++e) {
      const int first = wg_first<ST>(P, e), count = wg_count<ST>(P, e), at = wg_at<ST>(P, e);
      if (count == 1) {
        double E = 0.0;
#pragma unroll
        for (int k = 0; k < B::NE; ++k) E += tb->Rrest[k] * M[k];
        f[at] = value(ST::Q - 1, E);
        continue;
      }
#pragma unroll
      for (int n = 0; n < count; n += 2) {
        const int pr = (first + n) / 2;
        double E = 0.0, O = 0.0;
#pragma unroll
        for (int k = 0; k < B::NE; ++k) E += tb->Re[pr][k] * M[k];
#pragma unroll
        for (int k = 0; k < B::NO; ++k) O += tb->Ro[pr][k] * M[B::NE + k];
        f[at + n] = value(first + n, E + O);
        f[at + n + 1] = value(first + n + 1, E - O);
      }
    }
  });
  onlat_update<ST, N, S, DEV, true, EXT, false>(tb, sh, w, lane, live, x, y, run.z, f, fout, tau_field, fields, err);
}

// EXT: the rule is built with force and walls (the massive rule in float storage)
template <class ST, int N, typename S, bool DEV, bool EXT>
static hipError_t launch_onlat_t(const LaunchArgs &a) {
  unsigned nb;
  const SplitTiling tl = split_tiling(a.nx, a.ny, a.nz, nb);
  if (nb == 0) return hipErrorInvalidValue;
  const dim3 grid(nb), block(64 * WaveGroups<ST>::W);
  using T = std::true_type;
  using F = std::false_type;
  auto step = [&](auto relax, auto ext, auto nt) {
    hipLaunchKernelGGL((k_step_onlat3d<ST, N, S, DEV, decltype(relax)::value, decltype(ext)::value, decltype(nt)::value>), grid,
                       block, 0, a.stream, a.tb, (const S *)a.fin, (S *)a.fout, a.tau_field, a.fields, a.err, tl);
  };
  switch (a.op) {
    case OP_STEP:
      if constexpr (EXT) {
        if (a.ext) {
          a.nt ? step(T{}, T{}, T{}) : step(T{}, T{}, F{});
          break;
        }
      }
      a.nt ? step(T{}, F{}, T{}) : step(T{}, F{}, F{});
      break;
    case OP_MOMENTS:
      step(F{}, F{}, F{});
      break;
    case OP_INIT:
      hipLaunchKernelGGL((k_init_onlat3d<ST, N, S, DEV, EXT>), grid, block, 0, a.stream, a.tb, a.n0, a.T0, a.u0, a.noise, a.amp,
                         (S *)a.fout, a.tau_field, a.fields, a.err, tl);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_massive3d(const LaunchArgs &a) {
  using ST = Stencil<ST_MASSIVE3D, 3>;
  if (a.storage == 0) return launch_onlat_t<ST, 3, double, false, false>(a);
  if (a.storage == 1) return launch_onlat_t<ST, 3, float, true, true>(a);
  return hipErrorInvalidValue;
}

}  // namespace rlbm
