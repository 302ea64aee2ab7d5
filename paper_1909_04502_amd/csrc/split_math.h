// split_math.h -- the pieces of the 3D update that the waves of a block share (HIP device code): the sites of
// a block; one shell's pull, direction sums and relaxation of the product rule; the macroscopic state from
// the sums; and the equilibrium's coefficients by parity class.
#pragma once
#include <type_traits>
#include <utility>

#include "kernels.h"
#include "prod_math.h"

namespace rlbm {

// a * b + c in one rounding, written out where a run's end lanes have to form the same value as the others to the last bit
__device__ __forceinline__ double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// The running sum of a column's taps: the first tap starts it, a single tap is the sum.
template <typename A>
__device__ __forceinline__ A tap_sum(bool several, bool first, A wt, A t, A sum) {
  if (!several) return t;
  return first ? wt * t : fmadd(wt, t, sum);
}

// Direction sums of a shell of the 3D rule: s = S0, S^x, S^y, S^z, S^xx, S^xy, S^xz, S^yy, S^yz, S^zz of its
// populations f[0..25].  They come as 3 axis, 6 edge and 4 corner pairs (kDir3D); the edge pairs of a plane and
// the corner pairs enter through their sums and differences, which the components share.
template <typename A>
__device__ __forceinline__ void shell_sums3(const A *f, A (&S)[10]) {
  A s[13], d[13];
#pragma unroll
  for (int q = 0; q < 13; ++q) {
    s[q] = f[2 * q] + f[2 * q + 1];
    d[q] = f[2 * q] - f[2 * q + 1];
  }
  const A h = (A)kInvNorm[2], k = (A)kInvNorm[3], half = (A)0.5, third = (A)(1.0 / 3.0);
  // planes (x, y), (x, z), (y, z)
  const A pxy = s[3] + s[4], mxy = s[3] - s[4], pxz = s[5] + s[6], mxz = s[5] - s[6], pyz = s[7] + s[8],
          myz = s[7] - s[8];
  const A ex = (d[3] + d[4]) + (d[5] + d[6]), ey = (d[3] - d[4]) + (d[7] + d[8]), ez = (d[5] - d[6]) + (d[7] - d[8]);
  // corners (1,1,1), (1,1,-1), (1,-1,1), (-1,1,1)
  const A a = s[9] + s[10], b = s[11] + s[12], c = s[9] - s[10], e = s[11] - s[12];
  const A c0 = a + b;
  const A g = d[9] + d[10], u = d[11] - d[12], cx = g + u, cy = g - u, cz = (d[9] - d[10]) + (d[11] + d[12]);
  S[0] = (((s[0] + s[1]) + s[2]) + ((pxy + pxz) + pyz)) + c0;
  S[1] = fmadd(k, cx, fmadd(h, ex, d[0]));
  S[2] = fmadd(k, cy, fmadd(h, ey, d[1]));
  S[3] = fmadd(k, cz, fmadd(h, ez, d[2]));
  S[4] = fmadd(third, c0, fmadd(half, pxy + pxz, s[0]));
  S[5] = fmadd(third, a - b, half * mxy);
  S[6] = fmadd(third, c + e, half * mxz);
  S[7] = fmadd(third, c0, fmadd(half, pxy + pyz, s[1]));
  S[8] = fmadd(third, c - e, half * myz);
  S[9] = fmadd(third, c0, fmadd(half, pxz + pyz, s[2]));
}

// Sums of the moments over the shells of the 3D rule, shell j with direction sums S.
template <typename A>
struct Moments3 {
  A N0 = 0, T00 = 0, Na[3] = {0, 0, 0}, T0a[3] = {0, 0, 0}, Tab[6] = {0, 0, 0, 0, 0, 0};
  __device__ __forceinline__ void add(CTables *tb, int j, const A (&S)[10]) {
    const A p0 = tab<A>(tb->smom[j][0], tb->smomf[j][0]);
    const A pm = tab<A>(tb->smom[j][1], tb->smomf[j][1]);
    const A p00 = tab<A>(tb->smom[j][2], tb->smomf[j][2]);
    const A p0m = tab<A>(tb->smom[j][3], tb->smomf[j][3]);
    const A pmm = tab<A>(tb->smom[j][4], tb->smomf[j][4]);
    N0 = fmadd(p0, S[0], N0);
    T00 = fmadd(p00, S[0], T00);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      Na[a] = fmadd(pm, S[1 + a], Na[a]);
      T0a[a] = fmadd(p0m, S[1 + a], T0a[a]);
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) Tab[a] = fmadd(pmm, S[4 + a], Tab[a]);
  }
};

// N^a and T^ab in double (the reference's added back for deviations).
template <bool DEV, typename A>
__device__ __forceinline__ void moments_to_state(CTables *tb, const Moments3<A> &mom, double (&Nv)[4],
                                                 double (&T)[4][4]) {
  Nv[0] = mom.N0;
  T[0][0] = mom.T00;
  int ab = 0;
#pragma unroll
  for (int a = 1; a <= 3; ++a) {
    Nv[a] = mom.Na[a - 1];
    T[0][a] = T[a][0] = mom.T0a[a - 1];
#pragma unroll
    for (int b = a; b <= 3; ++b) {
      T[a][b] = T[b][a] = mom.Tab[ab];
      ++ab;
    }
  }
  if constexpr (DEV) {
    int s = 0;
#pragma unroll
    for (int a = 0; a <= 3; ++a) {
      Nv[a] += tb->Nref[a];
#pragma unroll
      for (int b = a; b <= 3; ++b) {
        T[a][b] += tb->Tref[s];
        if (a != b) T[b][a] = T[a][b];
        ++s;
      }
    }
  }
}

// index of the angular monomial n^(ex, ey, ez) in AngTable order (-1: above the order)
template <int N>
RLBM_HD constexpr int ang_index3(int ex, int ey, int ez) {
  constexpr AngTable<3, N> AT{};
  for (int q = 0; q < AT.n; ++q)
    if (AT.e[q][0] == ex && AT.e[q][1] == ey && AT.e[q][2] == ez) return q;
  return -1;
}

// Steps 5 and 8 of shell j of the 3D rule: f <- f + Omega (f^eq - f) on its populations f[0..25], then
// f <- extra(k, f^eq_k, f) (the force term of EXT builds).  With c_e the shell's coefficient of n^e, the even
// and odd parts of f^eq on the direction pairs are formed from the sums that the pairs of an axis, a plane
// and the corners share.  ap(k): a' of basis monomial k; a0 = U^0 / tau; nU(q) = (n_q . U) / tau of pair q.
template <int N, bool EXT, typename A, class Ap, class NU, class Extra>
__device__ __forceinline__ void relax_shell3(CTables *tb, int j, Ap &&ap, A a0, NU &&nU, Extra &&extra,
                                             A *f) {
  constexpr AngTable<3, N> AT{};
  A ce[20];
#pragma unroll
  for (int q = 0; q < AT.n; ++q) {
    const int l = AT.e[q][0] + AT.e[q][1] + AT.e[q][2];
    A acc = 0;
    if (AT.m0[q] >= 0) acc = ap(AT.m0[q]) * tab<A>(tb->sfeq[j][0][l], tb->sfeqf[j][0][l]);
    if (AT.m1[q] >= 0) acc = fmadd(ap(AT.m1[q]), tab<A>(tb->sfeq[j][1][l], tb->sfeqf[j][1][l]), acc);
    ce[q] = acc;
  }
#define CE(x, y, z) ce[ang_index3<N>(x, y, z)]
  const A half = (A)0.5, third = (A)(1.0 / 3.0), h = (A)kInvNorm[2], kk = (A)kInvNorm[3];
  const A v = tab<A>(tb->sv[j], tb->svf[j]);
  auto relax = [&](int q, A wt, A E, A O) {
    const A b = v * nU(q);
    const A f0 = f[2 * q], f1 = f[2 * q + 1], p = E + O, m = E - O;
    f[2 * q] = fmadd(a0 - b, fmadd(wt, p, -f0), f0);
    f[2 * q + 1] = fmadd(a0 + b, fmadd(wt, m, -f1), f1);
    if constexpr (EXT) {
      f[2 * q] = extra(2 * q, wt * p, f[2 * q]);
      f[2 * q + 1] = extra(2 * q + 1, wt * m, f[2 * q + 1]);
    }
  };
  const A c0 = CE(0, 0, 0), xx = CE(2, 0, 0), yy = CE(0, 2, 0), zz = CE(0, 0, 2);
  const A xy = CE(1, 1, 0), xz = CE(1, 0, 1), yz = CE(0, 1, 1);
  const A x1 = CE(1, 0, 0), y1 = CE(0, 1, 0), z1 = CE(0, 0, 1);
  A xxx = 0, xyy = 0, xzz = 0, yxx = 0, yyy = 0, yzz = 0, zxx = 0, zyy = 0, zzz = 0, xyz = 0;
  if constexpr (N >= 3) {
    xxx = CE(3, 0, 0), xyy = CE(1, 2, 0), xzz = CE(1, 0, 2);
    yxx = CE(2, 1, 0), yyy = CE(0, 3, 0), yzz = CE(0, 1, 2);
    zxx = CE(2, 0, 1), zyy = CE(0, 2, 1), zzz = CE(0, 0, 3);
    xyz = CE(1, 1, 1);
  }
#undef CE
  {   // axes
    const A wt = (A)(1.0 / 21.0);
    relax(0, wt, c0 + xx, x1 + xxx);
    relax(1, wt, c0 + yy, y1 + yyy);
    relax(2, wt, c0 + zz, z1 + zzz);
  }
  // edges of a plane (a, b): pairs (1, 1) and (1, -1)
  auto plane = [&](int q, A aa, A bb, A ab, A a1, A aaa, A abb, A b1, A bbb, A baa) {
    const A wt = (A)(4.0 / 105.0);
    const A E = fmadd(half, aa + bb, c0), M = half * ab;
    A oa = a1, ob = b1;
    if constexpr (N >= 3) {
      oa = fmadd(half, aaa + abb, oa);
      ob = fmadd(half, bbb + baa, ob);
    }
    relax(q, wt, E + M, h * (oa + ob));
    relax(q + 1, wt, E - M, h * (oa - ob));
  };
  plane(3, xx, yy, xy, x1, xxx, xyy, y1, yyy, yxx);
  plane(5, xx, zz, xz, x1, xxx, xzz, z1, zzz, zxx);
  plane(7, yy, zz, yz, y1, yyy, yzz, z1, zzz, zyy);
  {   // corners (1,1,1), (1,1,-1), (1,-1,1), (-1,1,1)
    const A wt = (A)(9.0 / 280.0);
    const A E = fmadd(third, (xx + yy) + zz, c0);
    const A bxy = third * xy, bp = third * (xz + yz), bm = third * (xz - yz);
    A ox = x1, oy = y1, oz = z1, o3 = 0;
    if constexpr (N >= 3) {
      ox = fmadd(third, (xxx + xyy) + xzz, ox);
      oy = fmadd(third, (yyy + yxx) + yzz, oy);
      oz = fmadd(third, (zzz + zxx) + zyy, oz);
      o3 = third * xyz;
    }
    const A ep = E + bxy, em = E - bxy, op = ox + oy, om = ox - oy, zp = oz + o3, zm = oz - o3;
    relax(9, wt, ep + bp, kk * (op + zp));
    relax(10, wt, ep - bp, kk * (op - zp));
    relax(11, wt, em + bm, kk * (om + zm));
    relax(12, wt, em - bm, kk * (zm - om));
  }
}

// What the waves of a block exchange, per lane (site), in the order of use.  Wave j's sums lie inside its
// part of `ex`, so no wave overwrites what another still reads; the sums are read, into registers, by the
// wave that then writes the state in their place.
template <int N, int W, typename A>
struct SplitLds {
  union {
    A ex[W][18][66];             // the pull's exchange along x, one part per wave
    A sums[W][18 * 66];          // S0, S^a, S^ab (xx, xy, xz, yy, yz, zz) of each shell, 64 lanes each
    struct {
      double mac[9][64];         // n, T, U^0..U^3, r0, r2, r3 of the site
      A om[17][64];              // U^0 / tau, (n_k . U) / tau of the 13 direction pairs; EXT: m/T, U^0, g . U
      A ap[BasisDef<3, N>::NM][64];  // a' of the equilibrium
    };
  };
};

// The 18 directions with an x component, those of +x first: their places in kDir3D.
struct XDirs {
  int k[18] = {};
  uint32_t yp = 0, yn = 0, zp = 0, zn = 0, kbit[5] = {};   // bit l: of the l-th direction
  constexpr XDirs() {
    int n = 0;
    for (int sgn = 1; sgn >= -1; sgn -= 2)
      for (int q = 0; q < 26; ++q)
        if (kDir3D[q][0] == sgn) {
          k[n] = q;
          yp |= (uint32_t)(kDir3D[q][1] > 0) << n;
          yn |= (uint32_t)(kDir3D[q][1] < 0) << n;
          zp |= (uint32_t)(kDir3D[q][2] > 0) << n;
          zn |= (uint32_t)(kDir3D[q][2] < 0) << n;
          for (int b = 0; b < 5; ++b) kbit[b] |= (uint32_t)((q >> b) & 1) << n;
          ++n;
        }
  }
};
RLBM_HD constexpr int xdir_of(int k) {   // place of direction k among the 18 (-1: no x component)
  constexpr XDirs X{};
  for (int n = 0; n < 18; ++n)
    if (X.k[n] == k) return n;
  return -1;
}

// A run's sites: consecutive in memory, `live` of them, the first at (x0, y0, z).
struct SplitRun {
  int x0, y0, z, live;
  int brk;   // lane of the first site of the second row (64: none; rows of at least 64 sites have one at most)
};

constexpr int kSlab = 8;   // rows of a run's slab, planes of a patch

struct SplitTiling {
  int chunk;    // runs per XCD (0: the XCDs take whole patches in turn)
  int npy;      // slabs along y
  int runs;     // runs of 64 sites per slab plane
  int rows;     // rows per slab
  int planes;   // planes per patch
};

// The tiling of a lattice, and its blocks (0: more than a grid holds).  The XCDs take whole patches in turn, or each
// an eighth of the sequence of patches, whichever leaves the busiest XCD less to do: that is what a step's time
// follows (whole patches against eighths in double: 64 x 48 x 48, whose busiest XCD has 1.11 times the blocks in whole
// patches, 64 against 58 us; 97 x 56 x 56, 1.14 times, 178 against 162; 100 x 72 x 72, 1.09 times, 263 against 252;
// 97 x 100 x 83, 0.97 times, 402 against 420; 100 x 44 x 41, 0.92 times, 104 against 111; the tube of 6400 x 1 x 1, one
// patch, 52 against 14).  From 256 patches on that differs by less than 3 %, which the L2 hits of whole patches outweigh.
inline SplitTiling split_tiling(int nx, int ny, int nz, unsigned &blocks) {
  const int rows = ny < kSlab ? ny : kSlab, planes = nz < kSlab ? nz : kSlab;
  SplitTiling tl{0, (ny + rows - 1) / rows, (int)(((int64_t)rows * nx + 63) / 64), rows, planes};
  const int npz = (nz + planes - 1) / planes;
  const int64_t npatch = (int64_t)tl.npy * npz, per = (int64_t)tl.runs * planes, eighth = (npatch * per + 7) / 8;
  bool whole = true;
  if (npatch < 256) {
    // runs that hold sites: of a plane of the last slab, of a plane of all slabs; and planes of the last patches
    const int64_t last_runs = ((int64_t)(ny - (tl.npy - 1) * rows) * nx + 63) / 64, last_planes = nz - (npz - 1) * planes;
    const int64_t all_runs = (tl.npy - 1) * (int64_t)tl.runs + last_runs;
    auto runs_of = [&](int64_t py) { return py < tl.npy - 1 ? (int64_t)tl.runs : last_runs; };
    auto planes_of = [&](int64_t pz) { return pz < npz - 1 ? (int64_t)planes : last_planes; };
    // and of the first t of the sequence
    auto before = [&](int64_t t) {
      const int64_t p = t / per, w = t % per, pz = p / tl.npy, py = p % tl.npy, z = w / tl.runs, r = w % tl.runs;
      if (p >= npatch) return nz * all_runs;
      const int64_t n = pz * planes * all_runs + planes_of(pz) * py * tl.runs;
      if (z >= planes_of(pz)) return n + planes_of(pz) * runs_of(py);
      return n + z * runs_of(py) + (r < runs_of(py) ? r : runs_of(py));
    };
    int64_t load[8] = {0}, most_whole = 0, most_eighth = 0;
    for (int64_t p = 0; p < npatch; ++p) load[p % 8] += runs_of(p % tl.npy) * planes_of(p / tl.npy);
    for (int k = 0; k < 8; ++k) {
      const int64_t e = before((k + 1) * eighth) - before(k * eighth);
      if (load[k] > most_whole) most_whole = load[k];
      if (e > most_eighth) most_eighth = e;
    }
    whole = most_whole <= most_eighth;
  }
  const int64_t nb = whole ? 8 * ((npatch + 7) / 8) * per : 8 * eighth;
  blocks = nb > 0x7fffffff ? 0u : (unsigned)nb;
  tl.chunk = whole ? 0 : (int)eighth;
  return tl;
}

// The block's run, and the site of this lane (a lane past the run's live sites takes the last of them: its
// loads stay inside the lattice, and it stores nothing).  False where the whole run lies past the lattice.
template <bool XCH>
__device__ __forceinline__ bool split_site(CTables *tb, const SplitTiling &tl, int lane, SplitRun &run,
                                           int &x, int &y) {
  const uint32_t k = blockIdx.x % 8, l = blockIdx.x / 8, per = (uint32_t)(tl.runs * tl.planes);
  const uint32_t t = k * (uint32_t)tl.chunk + l;
  const uint32_t p = tl.chunk ? t / per : (l / per) * 8 + k, w = tl.chunk ? t % per : l % per;
  const int nx = tb->nx, ny = tb->ny;
  run.z = (int)(p / tl.npy) * tl.planes + (int)(w / tl.runs);
  const int y0 = (int)(p % tl.npy) * tl.rows, off0 = (int)(w % tl.runs) * 64;
  if (run.z >= tb->nz) return false;
  const int rows = ny - y0 < tl.rows ? ny - y0 : tl.rows;   // of this slab
  if (off0 >= rows * nx) return false;
  run.live = rows * nx - off0 < 64 ? rows * nx - off0 : 64;
  const int q = off0 / nx;
  run.x0 = off0 - q * nx;
  run.y0 = y0 + q;
  run.brk = nx - run.x0 < 64 ? nx - run.x0 : 64;
  const int at = run.x0 + (lane < run.live ? lane : run.live - 1);
  if constexpr (XCH) {   // one row boundary at most
    x = at >= nx ? at - nx : at;
    y = run.y0 + (at >= nx);
  } else {
    // at / nx by a float quotient, corrected (at < nx + 63; below 128 where nx < 64, else the quotient is 0 or 1)
    int r = (int)((float)at * __builtin_amdgcn_rcpf((float)nx));
    r -= r * nx > at;
    r += at - r * nx >= nx;
    x = at - r * nx;
    y = run.y0 + r;
  }
  return true;
}

__device__ __forceinline__ void split_fields(const FieldPtrs &fp, int64_t site, int64_t sites, const Macro<3> &mac) {
  if (fp.n) fp.n[site] = mac.n;
  if (fp.eps) fp.eps[site] = mac.eps;
  if (fp.T) fp.T[site] = mac.T;
  if (fp.U) {
#pragma unroll
    for (int a = 0; a <= 3; ++a) fp.U[a * sites + site] = mac.U[a];
  }
}

// The directions in groups of at most MAX of the shell's y and z taps.
template <class ST, int MAX>
struct TapGroups {
  static constexpr int kMax = MAX;
  int of[26] = {}, n = 1;
  constexpr TapGroups() {
    int c = 0;
    for (int k = 0; k < 26; ++k) {
      const int w = 1 << ((ST::dir(k, 1) != 0) + (ST::dir(k, 2) != 0));
      if (c + w > MAX) {
        ++n;
        c = 0;
      }
      of[k] = n - 1;
      c += w;
    }
  }
};

template <typename A>
using XExchange = A[18][66];

// Pre-collision populations of shell j (planes from `base` on) at the lane's site (x, y, z): the same
// multilinear sum as pull_prod, along y and z first.  V_k(x), the sum over the y and z taps in the lane's
// own column, comes from one aligned load per tap; the sum upstream in x is V_k of the neighbouring lane,
// read from LDS, where the lanes at the run's ends and at a row boundary find it computed by 18 lanes, one
// per direction with an x component, with the same operations.  So a wave asks for every cache line of a
// plane's row once (74 loads of a row and 50 single lines at the ends, against 124 loads): what bounds the
// pull is the number of lines its CU's L1 has to fetch (split.hip).
// XCH = false (rows shorter than a run, with several row boundaries in it): the upstream sum from loads
// of its own, with the same operations.
// In double storage the taps go in groups of at most 16, the loads of a group before the sums of the group
// before it, which keeps the loads in flight within the registers; float rows, half as long, are all
// asked for at once (at 256^3 in groups 5.4 ms, at once 4.1).
template <class ST, typename S, typename A, bool XCH>
__device__ __forceinline__ void pull_shell3(CTables *tb, const S *__restrict__ base, int64_t sites,
                                            int j, const SplitRun &run, int lane, int x, int y, XExchange<A> &ex,
                                            A (&f)[ST::NDIR]) {
  constexpr int ND = ST::NDIR;
  typedef const __attribute__((address_space(1))) char gchar;
  typedef const __attribute__((address_space(1))) S gS;
  const int nx = tb->nx, ny = tb->ny, nz = tb->nz;
  const uint32_t es = sizeof(S), sx = (uint32_t)nx * es, sxy = sx * (uint32_t)ny;
  const A v = tab<A>(tb->sv[j], tb->svf[j]);
  A mag[4], cm[4];
#pragma unroll
  for (int q = 1; q <= 3; ++q) {
    mag[q] = v * (A)kInvNorm[q];
    cm[q] = (A)1 - mag[q];
  }
  uint32_t yo[3], zo[3];
#pragma unroll
  for (int d = -1; d <= 1; ++d) {
    yo[d + 1] = (uint32_t)near_site(y + d, ny, tb->open[1]) * sx;
    zo[d + 1] = (uint32_t)near_site(run.z + d, nz, tb->open[2]) * sxy;
  }
  // g[k] = the y and z sum of direction k in the column at byte offset xo, for the directions with
  // dir_x = 0 or side (side = 2: all of them)
  auto column = [&](uint32_t xo, auto side_, A(&g)[ND]) {
    constexpr int side = decltype(side_)::value;
    constexpr TapGroups<ST, sizeof(S) == 8 ? 16 : 128> G{};
    uint32_t yx[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) yx[d] = yo[d] + xo;
    S t[2][G.kMax];
    auto load = [&](int gr, S(&tt)[G.kMax]) {
      int m = 0;
#pragma unroll
      for (int k = 0; k < ND; ++k) {
        if (G.of[k] != gr || (side != 2 && ST::dir(k, 0) != side)) continue;
        gchar *plane = (gchar *)base + (int64_t)k * sites * (int64_t)es;
        const int dy = ST::dir(k, 1), dz = ST::dir(k, 2);
#pragma unroll
        for (int tz = 0; tz <= (dz != 0); ++tz)
#pragma unroll
          for (int ty = 0; ty <= (dy != 0); ++ty) tt[m++] = *(gS *)(plane + (yx[1 - ty * dy] + zo[1 - tz * dz]));
      }
    };
    auto sum = [&](int gr, const S(&tt)[G.kMax]) {
      int m = 0;
#pragma unroll
      for (int k = 0; k < ND; ++k) {
        if (G.of[k] != gr || (side != 2 && ST::dir(k, 0) != side)) continue;
        const int dy = ST::dir(k, 1), dz = ST::dir(k, 2), q = (ST::dir(k, 0) != 0) + (dy != 0) + (dz != 0);
        A acc = 0;
#pragma unroll
        for (int tz = 0; tz <= (dz != 0); ++tz)
#pragma unroll
          for (int ty = 0; ty <= (dy != 0); ++ty) {
            A wt = 1;
            if (dy != 0) wt = ty ? mag[q] : cm[q];
            if (dz != 0) wt *= tz ? mag[q] : cm[q];
            acc = tap_sum(dy != 0 || dz != 0, ty == 0 && tz == 0, wt, (A)tt[m++], acc);
          }
        g[k] = acc;
        if constexpr (G.n > 1) asm volatile("" : "+v"(g[k]));   // summed here: its taps' registers are free again
      }
    };
    load(0, t[0]);
#pragma unroll
    for (int gr = 0; gr < G.n; ++gr) {
      if (gr + 1 < G.n) load(gr + 1, t[(gr + 1) & 1]);
      if constexpr (G.n > 1) __builtin_amdgcn_sched_barrier(0);
      sum(gr, t[gr & 1]);
      if constexpr (G.n > 1) __builtin_amdgcn_sched_barrier(0);
    }
  };
  column((uint32_t)x * es, std::integral_constant<int, 2>{}, f);
  if constexpr (!XCH) {
    auto upstream = [&](auto side_) {
      constexpr int side = decltype(side_)::value;
      A up[ND];
      column((uint32_t)near_site(x - side, nx, tb->open[0]) * es, side_, up);
#pragma unroll
      for (int k = 0; k < ND; ++k) {
        if (ST::dir(k, 0) != side) continue;
        const int q = 1 + (ST::dir(k, 1) != 0) + (ST::dir(k, 2) != 0);
        f[k] = fmadd(mag[q], up[k], cm[q] * f[k]);
      }
    };
    upstream(std::integral_constant<int, 1>{});
    upstream(std::integral_constant<int, -1>{});
    return;
  }
  // ---- the same sums at the sites just past the run's ends (slot 0) and past a row boundary inside it
  //      (slot 1), by lane l for the l-th direction with an x component ----
  constexpr XDirs X{};
  if (lane < 18) {
    auto bit = [&](uint32_t m) { return (int)((m >> lane) & 1u); };
    const int k = bit(X.kbit[0]) | bit(X.kbit[1]) << 1 | bit(X.kbit[2]) << 2 | bit(X.kbit[3]) << 3 | bit(X.kbit[4]) << 4;
    const int dy = bit(X.yp) - bit(X.yn), dz = bit(X.zp) - bit(X.zn);
    const bool up = lane < 9;   // +x: upstream is x - 1
    gchar *plane = (gchar *)base + (int64_t)k * sites * (int64_t)es;
    const A mg = (dy != 0 && dz != 0) ? mag[3] : mag[2], cg = (dy != 0 && dz != 0) ? cm[3] : cm[2];
    const uint32_t z0 = zo[1], z1 = dz > 0 ? zo[0] : zo[2];
    auto edge = [&](int xs, int ys) {
      const uint32_t xo = (uint32_t)xs * es;
      const uint32_t y0 = (uint32_t)ys * sx + xo, y1 = (uint32_t)near_site(ys - dy, ny, tb->open[1]) * sx + xo;
      const A t00 = (A) * (gS *)(plane + (y0 + z0));
      A acc = t00;
      if (dy != 0 && dz != 0) {
        const A t10 = (A) * (gS *)(plane + (y1 + z0)), t01 = (A) * (gS *)(plane + (y0 + z1)),
                t11 = (A) * (gS *)(plane + (y1 + z1));
        acc = (cg * cg) * t00;
        acc = fmadd(mg * cg, t10, acc);
        acc = fmadd(cg * mg, t01, acc);
        acc = fmadd(mg * mg, t11, acc);
      } else if (dy != 0 || dz != 0) {
        const A t1 = (A) * (gS *)(plane + (dy != 0 ? y1 + z0 : y0 + z1));
        acc = fmadd(mg, t1, cg * t00);
      }
      return acc;
    };
    const int xl = run.x0 + run.live - 1, yl = run.y0 + (xl >= nx);   // the last live site
    ex[lane][64] = edge(near_site(up ? run.x0 - 1 : (xl >= nx ? xl - nx : xl) + 1, nx, tb->open[0]), up ? run.y0 : yl);
    if (run.brk < run.live) ex[lane][65] = edge(near_site(up ? -1 : nx, nx, tb->open[0]), up ? run.y0 + 1 : run.y0);
  }
#pragma unroll
  for (int k = 0; k < ND; ++k)
    if (ST::dir(k, 0) != 0) ex[xdir_of(k)][lane] = f[k];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int il = lane == 0 ? 64 : (lane == run.brk ? 65 : lane - 1);
  const int ir = lane >= run.live - 1 ? 64 : (lane == run.brk - 1 ? 65 : lane + 1);
#pragma unroll
  for (int k = 0; k < ND; ++k) {
    const int dx = ST::dir(k, 0);
    if (dx == 0) continue;
    const int q = 1 + (ST::dir(k, 1) != 0) + (ST::dir(k, 2) != 0);
    const A up = ex[xdir_of(k)][dx > 0 ? il : ir];
    f[k] = fmadd(mag[q], up, cm[q] * f[k]);
  }
}

// N^a and T^ab of the lane's site from the shells' sums.
template <int W, typename A, bool DEV>
__device__ __forceinline__ void split_moments(CTables *tb, const A (&sums)[W][18 * 66], int lane,
                                              double (&Nv)[4], double (&T)[4][4]) {
  Moments3<A> mom;
#pragma unroll
  for (int j = 0; j < W; ++j) {
    A S[10];
#pragma unroll
    for (int q = 0; q < 10; ++q) S[q] = sums[j][q * 64 + lane];
    mom.add(tb, j, S);
  }
  moments_to_state<DEV>(tb, mom, Nv, T);
}
// Steps 2-4, without the state in LDS.
__device__ __forceinline__ Macro<3> split_state(CTables *tb, const double (&Nv)[4], const double (&T)[4][4],
                                                Ratios &rr) {
  Macro<3> mac;
  mac.ok = landau_frame<3, 3>(T, mac.eps, mac.U);
  mac.n = lorentz_dot<3>(mac.U, Nv);
  const double m = tb->m;
  double r;
  mac.ok = temperature_3d(tb, mac.eps / mac.n, m, mac.T, r) && mac.ok;
  rr = ratios_3d(m / mac.T, r);
  mac.ok = mac.ok && mac.n > 0.0 && mac.eps > 0.0;
  return mac;
}

// The Maxwell-Juettner moments of the initial fields at a site; false where they are not physical.
template <int N>
__device__ __forceinline__ bool first_moments3(CTables *tb, const double *__restrict__ n0,
                                               const double *__restrict__ T0, const double *__restrict__ u0, uint32_t site,
                                               double (&M)[BasisDef<3, N>::NM]) {
  double U[4], uu = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    U[a + 1] = u0[a * tb->sites + site];
    uu += U[a + 1] * U[a + 1];
  }
  const double g = 1.0 / sqrt(1.0 - uu);
  U[0] = g;
#pragma unroll
  for (int a = 1; a <= 3; ++a) U[a] *= g;
  const double n = n0[site], T = T0[site];
  bool inr = true;
  const double r = tb->m == 0.0 ? 0.0 : cheb_r(tb, tb->m / T, inr);
  basis_moments<3, N>(n, T, U, ratios_3d(tb->m / T, r), M);
  return inr && uu < 1.0 && n > 0.0 && T > 0.0;
}

// What the equilibrium is built from, to LDS.
template <class X>
__device__ __forceinline__ void put_state(X &sh, int lane, double n, double T, const double (&U)[4], const Ratios &rr) {
  sh.mac[0][lane] = n;
  sh.mac[1][lane] = T;
#pragma unroll
  for (int a = 0; a <= 3; ++a) sh.mac[2 + a][lane] = U[a];
  sh.mac[6][lane] = rr.r0;
  sh.mac[7][lane] = rr.r2;
  sh.mac[8][lane] = rr.r3;
}

// The state and the ingredients of Omega (and of the force) to LDS, over the sums, which this lane has read.
// A wall site (wallT >= 0, see site_wall) relaxes fully to the equilibrium at rest of its own n and its own or
// the wall's T.
template <bool EXT, typename A, class X>
__device__ __forceinline__ void split_put(CTables *tb, const Macro<3> &mac, const Ratios &rr, double tau,
                                          double wallT, int lane, X &sh) {
  const bool wall = EXT && wallT >= 0.0;
  double Ue[4], Te = mac.T;
  Ratios re = rr;
#pragma unroll
  for (int a = 0; a <= 3; ++a) Ue[a] = wall ? (a == 0 ? 1.0 : 0.0) : mac.U[a];
  if (wall) equilibrium_state<3>(tb, mac, rr, wallT, Te, re);
  const double itau = wall ? 0.0 : 1.0 / tau;
  asm volatile("" ::: "memory");   // the sums are in registers; their place is reused from here on
  put_state(sh, lane, mac.n, Te, Ue, re);
  sh.om[0][lane] = wall ? (A)1 : (A)(mac.U[0] * itau);
#pragma unroll
  for (int q = 0; q < 13; ++q) {
    double acc = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double c = nhat<Stencil<ST_PROD3D, 4>>(2 * q, a);
      if (c != 0.0) acc += c * mac.U[a + 1];
    }
    sh.om[1 + q][lane] = (A)(acc * itau);
  }
  if constexpr (EXT) {   // zero where no force acts
    const bool force = tb->has_force && !wall;
    double gU = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) gU += tb->g[a] * mac.U[a + 1];
    sh.om[14][lane] = force ? (A)(tb->m / mac.T) : (A)0;
    sh.om[15][lane] = (A)mac.U[0];
    sh.om[16][lane] = (A)gU;
  }
}

// a' = Linv^T Linv M' on parity class C (the block of the projection that its monomials span)
template <int N, bool DEV, typename A, int C, class X>
__device__ __forceinline__ void split_class(CTables *tb, int lane, double n, double T,
                                            const double (&U)[4], const Ratios &rr, X &sh) {
  constexpr ClassTable<3, N> CL{};
  constexpr int K = CL.cnt[C];
  if constexpr (K > 0) {
    const double m = tb->m;
    CDouble *lp = tb->LinvP + CL.off[C];
    double mc[K], ak[K];
#pragma unroll
    for (int t = 0; t < K; ++t) {
      const int k = CL.idx[C][t];
      mc[t] = basis_moment<3, N>(k, n, T, U, rr);
      if constexpr (DEV) mc[t] -= tb->Mref[k];
    }
#pragma unroll
    for (int t = 0; t < K; ++t) {
      const int pk = CL.partner[CL.idx[C][t]];
      if (pk >= 0) mc[t] -= m * mc[CL.pos[pk]];
    }
#pragma unroll
    for (int t = 0; t < K; ++t) {
      double acc = 0.0;
#pragma unroll
      for (int u = 0; u <= t; ++u) acc += lp[t * (t + 1) / 2 + u] * mc[u];
      ak[t] = acc;
    }
#pragma unroll
    for (int u = 0; u < K; ++u) {
      double acc = 0.0;
#pragma unroll
      for (int t = u; t < K; ++t) acc += lp[t * (t + 1) / 2 + u] * ak[t];
      sh.ap[CL.idx[C][u]][lane] = (A)acc;
    }
  }
}

// The wave that takes parity class c (0: even, 1, 2, 4: one odd axis, 3, 5, 6: two, 7: three; at N = 3 they
// hold 8, 5, 2 and 1 monomials), of W = 3, 4 or 8 waves.
RLBM_HD constexpr int class_owner(int W, int c) {
  const int bits = (c & 1) + ((c >> 1) & 1) + (c >> 2);
  if (W == 3) return bits == 0 ? 0 : (bits == 1 ? 1 : 2);
  if (W == 4) return c == 0 ? 0 : (c == 1 || c == 3 ? 1 : (c == 2 || c == 5 ? 2 : 3));
  return c;
}

template <int N, int W, bool DEV, typename A, class X, int... C>
__device__ __forceinline__ void split_classes(CTables *tb, int w, int lane, double n, double T,
                                              const double (&U)[4], const Ratios &rr, X &sh,
                                              std::integer_sequence<int, C...>) {
  ((w == class_owner(W, C) ? split_class<N, DEV, A, C>(tb, lane, n, T, U, rr, sh) : (void)0), ...);
}

template <int N, int W, bool DEV, typename A, class X>
__device__ __forceinline__ void split_coefficients(CTables *tb, int w, int lane, X &sh) {
  const double n = sh.mac[0][lane], T = sh.mac[1][lane];
  double U[4];
#pragma unroll
  for (int a = 0; a <= 3; ++a) U[a] = sh.mac[2 + a][lane];
  Ratios rr;
  rr.r0 = sh.mac[6][lane];
  rr.r2 = sh.mac[7][lane];
  rr.r3 = sh.mac[8][lane];
  split_classes<N, W, DEV, A>(tb, w, lane, n, T, U, rr, sh, std::make_integer_sequence<int, 8>{});
}

// ---- on-lattice rules: the waves exchange their part of the moments ----

// What the waves exchange, per lane; the state takes the place of the moments once they are read.
template <int N, int W, typename A>
struct OnlatLds {
  union {
    A mom[W][14][64];                // N^0, T^00, N^a, T^0a, T^ab of each wave's groups
    struct {
      double mac[9][64];             // n, T, U^0..U^3, r0, r2, r3 of the site
      A om[9][64];                   // U^0 / tau, v0 U^a / tau; EXT: m/T, (v0 g^a) U^0, g . U
      A ap[BasisDef<3, N>::NM][64];  // a' of the equilibrium
    };
  };
};

template <typename A>
__device__ __forceinline__ void put_moments(const Moments3<A> &mom, int lane, A (&to)[14][64]) {
  to[0][lane] = mom.N0;
  to[1][lane] = mom.T00;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    to[2 + a][lane] = mom.Na[a];
    to[5 + a][lane] = mom.T0a[a];
  }
#pragma unroll
  for (int a = 0; a < 6; ++a) to[8 + a][lane] = mom.Tab[a];
}

// The state of the lane's site from all waves' moments; fields and flag; and, for the relaxation, what the
// equilibrium and Omega (and the force) are built from, to LDS over the moments.  A wall site: as split_put.
template <int N, int W, typename S, bool DEV, bool RELAX, bool EXT>
__device__ __forceinline__ void onlat_state(CTables *tb, OnlatLds<N, W, S> &sh, int lane, bool live, int x,
                                            int y, int z, uint32_t site, const void *__restrict__ tau_field,
                                            const FieldPtrs &fields, int *err) {
  const int64_t sites = tb->sites;
  double tau = RELAX ? (tau_field == nullptr ? tb->tau : (double)((const S *)tau_field)[site]) : 1.0;
  Moments3<S> mom;
#pragma unroll
  for (int p = 0; p < W; ++p) {
    mom.N0 += sh.mom[p][0][lane];
    mom.T00 += sh.mom[p][1][lane];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      mom.Na[a] += sh.mom[p][2 + a][lane];
      mom.T0a[a] += sh.mom[p][5 + a][lane];
    }
#pragma unroll
    for (int a = 0; a < 6; ++a) mom.Tab[a] += sh.mom[p][8 + a][lane];
  }
  double Nv[4], T[4][4];
  moments_to_state<DEV>(tb, mom, Nv, T);
  Ratios rr;
  const Macro<3> mac = split_state(tb, Nv, T, rr);
  if (!mac.ok && live) *err = 1;
  if (fields.any && live) split_fields(fields, site, sites, mac);
  if constexpr (RELAX) {
    const double wallT = EXT ? site_wall(tb, x, y, z) : -1.0;
    const bool wall = EXT && wallT >= 0.0;
    double Ue[4], Te = mac.T;
    Ratios re = rr;
#pragma unroll
    for (int a = 0; a <= 3; ++a) Ue[a] = wall ? (a == 0 ? 1.0 : 0.0) : mac.U[a];
    if (wall) equilibrium_state<3>(tb, mac, rr, wallT, Te, re);
    if (tb->tau_T != 0.0) tau += tb->tau_T / mac.T;   // step 7: the temperature-dependent part of tau
    const double itau = wall ? 0.0 : 1.0 / tau;
    asm volatile("" ::: "memory");   // the moments are in registers; their place is reused from here on
    put_state(sh, lane, mac.n, Te, Ue, re);
    sh.om[0][lane] = wall ? (S)1 : (S)(mac.U[0] * itau);
#pragma unroll
    for (int a = 0; a < 3; ++a) sh.om[1 + a][lane] = (S)(tb->v0 * mac.U[a + 1] * itau);
    if constexpr (EXT) {   // zero where no force acts
      const bool force = tb->has_force && !wall;
      double gU = 0.0;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        gU += tb->g[a] * mac.U[a + 1];
        sh.om[5 + a][lane] = (S)(tb->v0 * tb->g[a] * mac.U[0]);
      }
      sh.om[4][lane] = force ? (S)(tb->m / mac.T) : (S)0;
      sh.om[8][lane] = (S)gU;
    }
  }
}

}  // namespace rlbm
