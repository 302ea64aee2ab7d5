// split_ur3d.hip -- the printed massless rule in 3D (288 populations), one site's populations spread over the
// waves of a block as in split.hip (HIP, gfx950).
//
// The stencil consists of units of up to four antipodal pairs (a, s b, t c), s, t = +-1, which share |a|, |b|, |c|
// and the group's energy and weight: 33 of four pairs and 6 of two ((5, 4, 0) and its permutations, where one sign
// is none).  Each of eight waves takes five units of 64 sites, loads their populations, adds up their part of the
// moments and, once the state is known, relaxes and stores them.  All waves run the same code on units read from a
// table: the rule's tubes are single rows of a few thousand sites, a block or none per CU, and a step takes as
// long as one block: what counts there is that few instructions have to be fetched (code that spelled out each
// wave's populations was 84 KB, more than an instruction cache holds, and took 57 us a step on 6400 sites) and
// that 288 loads go out at once.  The tube of 6400 takes 13.4 us a step in double (256 registers, two waves per SIMD)
// and 11.0 in float (128 registers and 25 values in scratch; at three waves per SIMD nothing is spilled, but a CU holds
// one block of eight waves instead of two: 10.7, 41 instead of 29 at 40 x 33 x 30 and 325 instead of 268 at
// 128 x 64 x 64).
#define RLBM_TABLES_PLAIN   // device_math.h
#include <hip/hip_runtime.h>

#include "device_math.h"
#include "kernels.h"
#include "massive_math.h"
#include "split_math.h"

namespace rlbm {

namespace {

constexpr int kWaves = 8, kUnits = 5;

struct Unit {
  int g;         // group (energy and weight)
  int n[3];      // a, b, c >= 0
  int pair[4];   // first population of (a, b, c), (a, b, -c), (a, -b, c), (a, -b, -c); -1: none, or the same as another
};

struct UnitTable {
  Unit u[kWaves][kUnits] = {};
  int units = 0, pairs = 0;
  constexpr UnitTable() {
    using ST = Stencil<ST_UR3D, 4>;
    for (int w = 0; w < kWaves; ++w)
      for (int k = 0; k < kUnits; ++k) u[w][k] = Unit{0, {0, 0, 0}, {-1, -1, -1, -1}};
    for (int g = 0; g < ST::NG; ++g) {
      const int first = units;
      for (int i = ST::gfirst(g); i < ST::gfirst(g) + ST::gcount(g); i += 2) {
        int v[3] = {}, m[3] = {};
        for (int a = 0; a < 3; ++a) {
          v[a] = ST::dir(i, a);
          m[a] = v[a] < 0 ? -v[a] : v[a];
        }
        int at = -1;
        for (int k = first; k < units; ++k) {
          const Unit &q = u[k / kUnits][k % kUnits];
          if (q.n[0] == m[0] && q.n[1] == m[1] && q.n[2] == m[2]) at = k;
        }
        if (at < 0) {
          at = units++;
          Unit &q = u[at / kUnits][at % kUnits];
          q.g = g;
          for (int a = 0; a < 3; ++a) q.n[a] = m[a];
        }
        // the first non-zero component is positive
        u[at / kUnits][at % kUnits].pair[(v[1] < 0 ? 2 : 0) + (v[2] < 0 ? 1 : 0)] = i;
        ++pairs;
      }
    }
  }
};
constexpr UnitTable kTable{};
static_assert(kTable.units <= kWaves * kUnits && 2 * kTable.pairs == kUR3DQ, "every pair has its place");
__constant__ UnitTable c_units = kTable;

}  // namespace

// The populations of unit u at the site (x, y, z): f[2 q], f[2 q + 1] of pair q and its opposite; 0 where none.
template <typename S>
__device__ __forceinline__ void load_unit(CTables *tb, const S *__restrict__ fin, const Unit &u, int x, int y,
                                          int z, S (&f)[8]) {
  typedef const __attribute__((address_space(1))) char gchar;
  typedef const __attribute__((address_space(1))) S gS;
  const uint32_t es = sizeof(S), nx = tb->nx, nxy = nx * (uint32_t)tb->ny;
  uint32_t xo[2], yo[2], zo[2];   // at minus and plus the component
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int sg = e ? 1 : -1;
    xo[e] = (uint32_t)near_site(x + sg * u.n[0], tb->nx, tb->open[0]) * es;
    yo[e] = (uint32_t)near_site(y + sg * u.n[1], tb->ny, tb->open[1]) * nx * es;
    zo[e] = (uint32_t)near_site(z + sg * u.n[2], tb->nz, tb->open[2]) * nxy * es;
  }
  const int64_t plane = tb->sites * (int64_t)es;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int sy = q >> 1, sz = q & 1;   // 1: the pair's first member has -b (-c)
    f[2 * q] = f[2 * q + 1] = 0;
    if (u.pair[q] >= 0) {
      gchar *p = (gchar *)fin + (int64_t)u.pair[q] * plane;
      f[2 * q] = *(gS *)(p + (xo[0] + yo[sy] + zo[sz]));
      f[2 * q + 1] = *(gS *)(p + plane + (xo[1] + yo[1 - sy] + zo[1 - sz]));
    }
  }
}

template <typename A>
__device__ __forceinline__ void unit_moments(CTables *tb, const Unit &u, const A (&f)[8], Moments3<A> &mom) {
  const int g = u.g;
  const A a = (A)u.n[0], b = (A)u.n[1], c = (A)u.n[2];
  const A s0 = f[0] + f[1], s1 = f[2] + f[3], s2 = f[4] + f[5], s3 = f[6] + f[7];
  const A d0 = f[0] - f[1], d1 = f[2] - f[3], d2 = f[4] - f[5], d3 = f[6] - f[7];
  const A S0 = (s0 + s1) + (s2 + s3), Sxy = (s0 + s1) - (s2 + s3), Sxz = (s0 - s1) + (s2 - s3), Syz = (s0 - s1) - (s2 - s3);
  const A X = a * ((d0 + d1) + (d2 + d3)), Y = b * ((d0 + d1) - (d2 + d3)), Z = c * ((d0 - d1) + (d2 - d3));
  const A v = tab<A>(tb->mgrp[g][2], tb->mgrpf[g][2]), p0v = tab<A>(tb->mgrp[g][3], tb->mgrpf[g][3]);
  const A vv = tab<A>(tb->mgrp[g][4], tb->mgrpf[g][4]);
  mom.N0 += tab<A>(tb->mgrp[g][0], tb->mgrpf[g][0]) * S0;
  mom.T00 += tab<A>(tb->mgrp[g][1], tb->mgrpf[g][1]) * S0;
  mom.Na[0] += v * X;
  mom.Na[1] += v * Y;
  mom.Na[2] += v * Z;
  mom.T0a[0] += p0v * X;
  mom.T0a[1] += p0v * Y;
  mom.T0a[2] += p0v * Z;
  mom.Tab[0] += vv * ((a * a) * S0);
  mom.Tab[1] += vv * ((a * b) * Sxy);
  mom.Tab[2] += vv * ((a * c) * Sxz);
  mom.Tab[3] += vv * ((b * b) * S0);
  mom.Tab[4] += vv * ((b * c) * Syz);
  mom.Tab[5] += vv * ((c * c) * S0);
}

// Steps 5 and 8 of a unit, and its store.  ce: the group's coefficients of the angular monomials (AngTable order).
template <bool NT, typename S>
__device__ __forceinline__ void relax_unit(const Unit &u, const S (&ce)[20], S a0, const S (&ub)[3], const S (&f)[8],
                                           int64_t sites, uint32_t site_off, S *__restrict__ fout) {
  using A = S;
  const A a = (A)u.n[0], b = (A)u.n[1], c = (A)u.n[2];
  const A aa = a * a, bb = b * b, cc = c * c;
#define CE(x, y, z) ce[ang_index3<3>(x, y, z)]
  const A E = CE(0, 0, 0) + aa * CE(2, 0, 0) + bb * CE(0, 2, 0) + cc * CE(0, 0, 2);
  const A xy = (a * b) * CE(1, 1, 0), xz = (a * c) * CE(1, 0, 1), yz = (b * c) * CE(0, 1, 1);
  const A ox = a * (CE(1, 0, 0) + aa * CE(3, 0, 0) + bb * CE(1, 2, 0) + cc * CE(1, 0, 2));
  const A oy = b * (CE(0, 1, 0) + bb * CE(0, 3, 0) + aa * CE(2, 1, 0) + cc * CE(0, 1, 2));
  const A oz = c * (CE(0, 0, 1) + cc * CE(0, 0, 3) + aa * CE(2, 0, 1) + bb * CE(0, 2, 1));
  const A o3 = (a * b) * (c * CE(1, 1, 1));
#undef CE
  const A bx = a * ub[0], by = b * ub[1], bz = c * ub[2];
  const A ev[4] = {(E + xy) + (xz + yz), (E + xy) - (xz + yz), (E - xy) + (xz - yz), (E - xy) - (xz - yz)};
  const A od[4] = {(ox + oy) + (oz + o3), (ox + oy) - (oz + o3), (ox - oy) + (oz - o3), (ox - oy) - (oz - o3)};
  const A om[4] = {(bx + by) + bz, (bx + by) - bz, (bx - by) + bz, (bx - by) - bz};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (u.pair[q] < 0) continue;
    const A f0 = f[2 * q], f1 = f[2 * q + 1];
    put_pop<NT>(fout, sites, site_off, u.pair[q], f0 + (a0 - om[q]) * ((ev[q] + od[q]) - f0));
    put_pop<NT>(fout, sites, site_off, u.pair[q] + 1, f1 + (a0 + om[q]) * ((ev[q] - od[q]) - f1));
  }
}

// The update from wave w's pre-collision populations f on (RELAX = false: the fields alone).
template <typename S, bool DEV, bool RELAX, bool NT>
__device__ __forceinline__ void ur3d_update(CTables *tb, OnlatLds<3, kWaves, S> &sh, int w, int lane, bool live,
                                            int x, int y, int z, const S (&f)[kUnits][8], S *__restrict__ fout,
                                            const void *__restrict__ tau_field, const FieldPtrs &fields, int *err) {
  constexpr AngTable<3, 3> AT{};
  const uint32_t site = ((uint32_t)z * tb->ny + y) * tb->nx + x;
  Moments3<S> mom;
#pragma unroll
  for (int k = 0; k < kUnits; ++k) unit_moments<S>(tb, c_units.u[w][k], f[k], mom);
  put_moments(mom, lane, sh.mom[w]);
  __syncthreads();
  if (w == (int)((blockIdx.x / 8) % kWaves))
    onlat_state<3, kWaves, S, DEV, RELAX, false>(tb, sh, lane, live, x, y, z, site, tau_field, fields, err);
  if constexpr (!RELAX) return;
  __syncthreads();
  split_coefficients<3, kWaves, DEV, S>(tb, w, lane, sh);
  __syncthreads();
  if (!live) return;
  const S a0 = sh.om[0][lane], ub[3] = {sh.om[1][lane], sh.om[2][lane], sh.om[3][lane]};
  S ce[20];
#pragma unroll
  for (int k = 0; k < kUnits; ++k) {
    const int g = c_units.u[w][k].g;
    asm volatile("" ::: "memory");   // a' is read again where needed rather than kept in registers
    if (k == 0 || g != c_units.u[w][k > 0 ? k - 1 : 0].g) {
#pragma unroll
      for (int q = 0; q < AT.n; ++q) {
        const int l = AT.e[q][0] + AT.e[q][1] + AT.e[q][2];
        S acc = 0;
        if (AT.m0[q] >= 0) acc += sh.ap[AT.m0[q]][lane] * tab<S>(tb->mgrp[g][5 + l], tb->mgrpf[g][5 + l]);
        if (AT.m1[q] >= 0) acc += sh.ap[AT.m1[q]][lane] * tab<S>(tb->mgrp[g][9 + l], tb->mgrpf[g][9 + l]);
        ce[q] = acc;
      }
    }
    relax_unit<NT, S>(c_units.u[w][k], ce, a0, ub, f[k], tb->sites, site * (uint32_t)sizeof(S), fout);
  }
}

template <typename S, bool DEV, bool RELAX, bool NT>
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(sizeof(S) == 8 ? 2 : 4, 8)))
k_step_ur3d(const Tables *__restrict__ tabs, const S *__restrict__ fin, S *__restrict__ fout, const void *__restrict__ tau_field,
            FieldPtrs fields, int *err, SplitTiling tl) {
  CTables *tb = (CTables *)tabs;
  __shared__ OnlatLds<3, kWaves, S> sh;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int x, y;
  SplitRun run;
  if (!split_site<false>(tb, tl, lane, run, x, y)) return;
  S f[kUnits][8];
#pragma unroll
  for (int k = 0; k < kUnits; ++k) load_unit<S>(tb, fin, c_units.u[w][k], x, y, run.z, f[k]);
  ur3d_update<S, DEV, RELAX, NT>(tb, sh, w, lane, lane < run.live, x, y, run.z, f, fout, tau_field, fields, err);
}

// f(x, 0) = f^eq(n0, T0, U(u0)) (1 + amp xi) from the projection rows, then collide; store f*(x, 0).
template <typename S, bool DEV>
__global__ void __launch_bounds__(64 * kWaves) k_init_ur3d(const Tables *__restrict__ tabs, const double *__restrict__ n0,
                                                           const double *__restrict__ T0, const double *__restrict__ u0,
                                                           const double *__restrict__ noise, double amp, S *__restrict__ fout,
                                                           const void *__restrict__ tau_field, FieldPtrs fields, int *err,
                                                           SplitTiling tl) {
  CTables *tb = (CTables *)tabs;
  using B = BasisDef<3, 3>;
  __shared__ OnlatLds<3, kWaves, S> sh;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int x, y;
  SplitRun run;
  if (!split_site<false>(tb, tl, lane, run, x, y)) return;
  const bool live = lane < run.live;
  const int64_t sites = tb->sites;
  const uint32_t site = ((uint32_t)run.z * tb->ny + y) * tb->nx + x;
  double M[B::NM];
  if (!first_moments3<3>(tb, n0, T0, u0, site, M) && live) *err = 1;
  S f[kUnits][8];
#pragma unroll
  for (int k = 0; k < kUnits; ++k)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = c_units.u[w][k].pair[q], pr = i < 0 ? 0 : i / 2;
      double E = 0.0, O = 0.0;
#pragma unroll
      for (int b = 0; b < B::NE; ++b) E += tb->Re[pr][b] * M[b];
#pragma unroll
      for (int b = 0; b < B::NO; ++b) O += tb->Ro[pr][b] * M[B::NE + b];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        double fd = e ? E - O : E + O;
        if (noise != nullptr) fd *= 1.0 + amp * noise[(int64_t)(2 * pr + e) * sites + site];
        f[k][2 * q + e] = i < 0 ? (S)0 : (DEV ? (S)(fd - tb->fref[2 * pr + e]) : (S)fd);
      }
    }
  ur3d_update<S, DEV, true, false>(tb, sh, w, lane, live, x, y, run.z, f, fout, tau_field, fields, err);
}

template <typename S, bool DEV>
static hipError_t launch_ur3d_t(const LaunchArgs &a) {
  unsigned nb;
  const SplitTiling tl = split_tiling(a.nx, a.ny, a.nz, nb);
  if (nb == 0) return hipErrorInvalidValue;
  const dim3 grid(nb), block(64 * kWaves);
  auto step = [&](auto relax, auto nt) {
    hipLaunchKernelGGL((k_step_ur3d<S, DEV, decltype(relax)::value, decltype(nt)::value>), grid, block, 0, a.stream, a.tb,
                       (const S *)a.fin, (S *)a.fout, a.tau_field, a.fields, a.err, tl);
  };
  using T = std::true_type;
  using F = std::false_type;
  switch (a.op) {
    case OP_STEP:
      a.nt ? step(T{}, T{}) : step(T{}, F{});
      break;
    case OP_MOMENTS:
      step(F{}, F{});
      break;
    case OP_INIT:
      hipLaunchKernelGGL((k_init_ur3d<S, DEV>), grid, block, 0, a.stream, a.tb, a.n0, a.T0, a.u0, a.noise, a.amp, (S *)a.fout,
                         a.tau_field, a.fields, a.err, tl);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_ur3d(const LaunchArgs &a) {
  if (a.storage == 0) return launch_ur3d_t<double, false>(a);
  if (a.storage == 1) return launch_ur3d_t<float, true>(a);
  return hipErrorInvalidValue;
}

}  // namespace rlbm
