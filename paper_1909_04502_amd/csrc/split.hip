// split.hip -- the 3D product rules, one site's populations spread over the waves of a block (HIP, gfx950).
//
// A thread that holds all 104 populations of a site needs 220 to 470 registers, which leaves one or two
// waves per SIMD: too few to hide the latency of the taps' loads behind the update's arithmetic.  Here a
// block takes 64 sites (one per lane) and its waves share the populations: wave j pulls shell j (26
// populations), forms that shell's direction sums and, once the macroscopic state is known, relaxes and
// stores that shell.  One wave takes the sums of all shells to the state (the eigen-solve and the equation of
// state), all of them share the projection by parity classes; sums, state and coefficients pass through LDS.
// 123 to 127 (float arithmetic) or 150 to 167 registers per lane and up to 38 KB of LDS per block: four or three
// blocks of four waves per CU, each in another phase, so that loads, arithmetic and stores of different blocks overlap.
//
// What bounds it: the lines a CU's L1 fetches for the taps (195 of 128 bytes per wave in float storage, 52 of
// them its own; L1-to-L2 reads of 690 cycles, 58 to 64 in flight per CU by its counters) and, in double, the
// waves' wait for the one that solves for the state.  Pull and store alone take 1.41 of the step's 1.49 ms at
// 192^3 in float storage and 3.05 of 3.60 ms in double; a copy of the same planes takes 1.17 and 2.35 ms.
// Per step, against the register kernel that this one replaced (64 x 4 sites per block, one site per thread,
// the equation of state in the same form):
//   double 97 x 130 x 83     0.53 ms (3.3 TB/s of population traffic)   0.91
//   double 192^3             3.2 to 3.6 ms (3.7 to 3.3 TB/s)            4.1
//   double 128^3, order 2    0.71 ms                                    2.8
//   float 256^3              4.1 ms (3.4 TB/s)                          4.2
//   float, double arithmetic 256^3   4.6 ms                             6.1
//   float 31 x 40 x 24       0.013 ms                                   0.021
//
// Sites are dealt to blocks in runs of 64 consecutive sites of a slab of kSlab rows (all rows of the
// slab joined end to end, so that rows of any length fill their waves), slab by slab and plane by plane
// inside patches of kSlab rows by kSlab planes, so that the y and z halo rows of the blocks in flight on an
// XCD stay in its L2 (split_tiling: which patches an XCD takes).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_math.h"
#include "kernels.h"
#include "prod_math.h"
#include "split_math.h"

namespace rlbm {

// The update from the pre-collision populations f of this wave's shell w on: state, relaxation, store (RELAX =
// false: the fields alone).
template <class ST, int N, typename S, bool DEV, bool RELAX, bool EXT, bool NT, typename A>
__device__ __forceinline__ void split_update(CTables *tb, SplitLds<N, ST::NSHELL, A> &sh, int w, int lane,
                                             bool live, int x, int y, int z, A (&f)[ST::NDIR], S *__restrict__ fout,
                                             const void *__restrict__ tau_field, const FieldPtrs &fields, int *err) {
  constexpr int ND = ST::NDIR, W = ST::NSHELL;
  const int64_t sites = tb->sites;
  const uint32_t site = ((uint32_t)z * tb->ny + y) * tb->nx + x;
  A s[10];
  shell_sums3<A>(f, s);
#pragma unroll
  for (int q = 0; q < 10; ++q) sh.sums[w][q * 64 + lane] = s[q];
  __syncthreads();
  // the macroscopic state, by one wave (another one in the next block of the XCD, so that the SIMDs share
  // this work)
  if (w == (int)((blockIdx.x / 8) % W)) {
    double Nv[4], T[4][4];
    split_moments<W, A, DEV>(tb, sh.sums, lane, Nv, T);
    Ratios rr;
    const Macro<3> mac = split_state(tb, Nv, T, rr);
    if constexpr (RELAX)
      split_put<EXT, A>(tb, mac, rr, tau_field == nullptr ? tb->tau : (double)((const S *)tau_field)[site],
                        EXT ? site_wall(tb, x, y, z) : -1.0, lane, sh);
    if (!mac.ok && live) *err = 1;
    if (fields.any && live) split_fields(fields, site, sites, mac);
  }
  if constexpr (!RELAX) return;
  __syncthreads();
  split_coefficients<N, W, DEV, A>(tb, w, lane, sh);
  __syncthreads();
  const A vj = tab<A>(tb->sv[w], tb->svf[w]);
  relax_shell3<N, EXT, A>(
      tb, w, [&](int k) { return sh.ap[k][lane]; }, sh.om[0][lane], [&](int q) { return sh.om[1 + q][lane]; },
      [&](int k, A fe, A fk) {   // external force (Sec. 5.4, scheme B): + (m/T) ((g . v) U^0 - g . U) f^eq
        A gn = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const double c = nhat<ST>(k, a);
          if (c != 0.0) gn += (A)c * tab<A>(tb->g[a], tb->gf[a]);
        }
        const int i = w * ND + k;
        return fk + sh.om[14][lane] * (vj * gn * sh.om[15][lane] - sh.om[16][lane]) *
                        (fe + (DEV ? tab<A>(tb->fref[i], tb->freff[i]) : (A)0));
      },
      f);
  if (live) {
    S *out = fout + (int64_t)(w * ND) * sites;
    const uint32_t so = site * (uint32_t)sizeof(S);
#pragma unroll
    for (int k = 0; k < ND; ++k) put_pop<NT>(out, sites, so, k, (S)f[k]);
  }
}

// The step, and (RELAX = false) the fields of the streamed state.
template <class ST, int N, typename S, bool DEV, bool RELAX, bool EXT, bool NT, typename A, bool XCH>
__global__ void __launch_bounds__(64 * ST::NSHELL) __attribute__((amdgpu_waves_per_eu(sizeof(A) == 8 ? 3 : 4, 8)))
k_step_split(const Tables *__restrict__ tabs, const S *__restrict__ fin, S *__restrict__ fout,
             const void *__restrict__ tau_field, FieldPtrs fields, int *err, SplitTiling tl) {
  CTables *tb = (CTables *)tabs;
  static_assert(ST::D == 3 && !ST::ONLAT, "3D product rules");
  constexpr int ND = ST::NDIR, W = ST::NSHELL;
  __shared__ SplitLds<N, W, A> sh;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // this wave's shell
  int x, y;
  SplitRun run;
  if (!split_site<XCH>(tb, tl, lane, run, x, y)) return;
  A f[ND];
  pull_shell3<ST, S, A, XCH>(tb, fin + (int64_t)(w * ND) * tb->sites, tb->sites, w, run, lane, x, y, sh.ex[w], f);
  split_update<ST, N, S, DEV, RELAX, EXT, NT, A>(tb, sh, w, lane, lane < run.live, x, y, run.z, f, fout, tau_field, fields,
                                                 err);
}

// f(x, 0) = f^eq(n0, T0, U(u0)) (1 + amp xi) from the projection rows, then collide; store f*(x, 0).
template <class ST, int N, typename S, bool DEV, typename A>
__global__ void __launch_bounds__(64 * ST::NSHELL) k_init_split(const Tables *__restrict__ tabs, const double *__restrict__ n0,
                                                                const double *__restrict__ T0, const double *__restrict__ u0,
                                                                const double *__restrict__ noise, double amp,
                                                                S *__restrict__ fout, const void *__restrict__ tau_field,
                                                                FieldPtrs fields, int *err, SplitTiling tl) {
  CTables *tb = (CTables *)tabs;
  constexpr int ND = ST::NDIR, W = ST::NSHELL;
  using B = BasisDef<3, N>;
  __shared__ SplitLds<N, W, A> sh;
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
  A f[ND];
#pragma unroll
  for (int q = 0; q < ND / 2; ++q) {
    const int pr = w * (ND / 2) + q;
    double E = 0.0, O = 0.0;
#pragma unroll
    for (int k = 0; k < B::NE; ++k) E += tb->Re[pr][k] * M[k];
#pragma unroll
    for (int k = 0; k < B::NO; ++k) O += tb->Ro[pr][k] * M[B::NE + k];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int i = 2 * pr + e;
      double fd = e ? E - O : E + O;
      if (noise != nullptr) fd *= 1.0 + amp * noise[(int64_t)i * sites + site];
      f[2 * q + e] = DEV ? (A)(fd - tb->fref[i]) : (A)fd;
    }
  }
  split_update<ST, N, S, DEV, true, true, false, A>(tb, sh, w, lane, live, x, y, run.z, f, fout, tau_field, fields, err);
}

template <class ST, int N, typename S, bool DEV, typename A>
static hipError_t launch_split_t(const LaunchArgs &a) {
  unsigned nb;
  const SplitTiling tl = split_tiling(a.nx, a.ny, a.nz, nb);
  if (nb == 0) return hipErrorInvalidValue;
  const dim3 grid(nb), block(64 * ST::NSHELL);
  using T = std::true_type;
  using F = std::false_type;
  auto step = [&](auto relax, auto ext, auto nt) {
    // rows of at least a run's length: upstream sums through LDS
    auto go = [&](auto xch) {
      hipLaunchKernelGGL((k_step_split<ST, N, S, DEV, decltype(relax)::value, decltype(ext)::value, decltype(nt)::value, A,
                                       decltype(xch)::value>),
                         grid, block, 0, a.stream, a.tb, (const S *)a.fin, (S *)a.fout, a.tau_field, a.fields, a.err, tl);
    };
    if (a.nx >= 64) go(T{});
    else go(F{});
  };
  switch (a.op) {
    case OP_STEP:
      if (a.ext) a.nt ? step(T{}, T{}, T{}) : step(T{}, T{}, F{});
      else a.nt ? step(T{}, F{}, T{}) : step(T{}, F{}, F{});
      break;
    case OP_MOMENTS:
      step(F{}, F{}, F{});
      break;
    case OP_INIT:
      hipLaunchKernelGGL((k_init_split<ST, N, S, DEV, A>), grid, block, 0, a.stream, a.tb, a.n0, a.T0, a.u0, a.noise, a.amp,
                         (S *)a.fout, a.tau_field, a.fields, a.err, tl);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <class ST, int N>
static hipError_t launch_split_storage(const LaunchArgs &a) {
  if (a.storage == 0) return launch_split_t<ST, N, double, false, double>(a);
  if (a.storage == 1) return launch_split_t<ST, N, float, true, float>(a);
  return launch_split_t<ST, N, float, true, double>(a);
}

hipError_t launch_prod3d(const LaunchArgs &a) {
  if (a.order == 2) return launch_split_storage<Stencil<ST_PROD3D, 3>, 2>(a);
  return launch_split_storage<Stencil<ST_PROD3D, 4>, 3>(a);
}

}  // namespace rlbm
