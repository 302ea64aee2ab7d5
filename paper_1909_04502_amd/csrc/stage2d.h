// stage2d.h -- LDS-staged pull of the 2D product rules (HIP device code).
//
// A block of 64 x 4 sites stages, one shell at a time, the upstream windows of the shell's 8 planes in
// LDS by direct global-to-LDS loads, which hold no registers while in flight.  A plane's window holds
// only what its direction reads: the tile's 4 rows, a fifth row on the upstream side where n_y != 0, and
// one column element per row on the upstream side where n_x != 0.  Rows are loaded 4 bytes per lane, so
// that any row start and any x extent will do, and lanes address their columns one by one, so that
// periodic and open axes wrap and clamp as in the register kernels (or, WIDE, 16 bytes per lane:
// stage_wide).  Two buffers alternate: the loads of shell j + 1 are in flight while the taps of shell j
// are read from LDS and summed; the block's four waves share each window.  The taps, weights and summation order are those of pull_prod, so the
// populations are the same values to the last bit.
//
// What bounds the pull is the number of cache lines that a CU has in flight on their way to its L1 (some
// 64), so the window is cut to the lines that are needed: 22.5 a plane in double instead of 40 for
// windows of 5 rows of 68 columns in 16-byte chunks.
#pragma once
#include "prod_math.h"

namespace rlbm {

template <class ST, typename S>
struct Stage2D {
  static constexpr int H = (int)sizeof(S) / 4;   // load instructions per window row of 64 elements
  static constexpr int kSide = 8;                // elements kept for the side column, before the rows
  static_assert(ST::D == 2 && !ST::ONLAT && ST::NDIR == 8, "2D product rules: two planes per wave and shell");
  static constexpr bool side(int k) { return ST::dir(k, 0) != 0; }
  static constexpr int rows(int k) { return ST::dir(k, 1) != 0 ? 5 : 4; }
  // first row element of plane k's window in a buffer
  static constexpr int body(int k) {
    int o = 0;
    for (int i = 0; i < k; ++i) o += (side(i) ? kSide : 0) + 64 * rows(i);
    return o + (side(k) ? kSide : 0);
  }
  static constexpr int E = body(7) + 64 * rows(7);   // elements of one buffer
  // 16 bytes per lane: lanes per row, rows per instruction
  static constexpr int LPR = 64 * (int)sizeof(S) / 16, RPI = 64 / LPR;
  static constexpr int row_loads(bool wide, int k) { return wide ? (rows(k) + RPI - 1) / RPI : H * rows(k); }
  static constexpr int min_loads(bool wide) {        // load instructions of a wave per shell, the fewest
    int m = 99;
    for (int w = 0; w < 4; ++w) {
      const int l = row_loads(wide, w) + row_loads(wide, w + 4) + side(w) + side(w + 4);
      m = l < m ? l : m;
    }
    return m;
  }
};

// s_waitcnt vmcnt(N) lgkmcnt(0) (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4 left at its
// maximum, lgkmcnt 11:8): all but the N most recent vector memory loads of this wave, to registers
// or to LDS, and every LDS read of this wave are done
template <int N>
__device__ __forceinline__ void wait_vm_lgkm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4));
}
__device__ __forceinline__ void wait_lgkm() { __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (0x7 << 4)); }

// One direct global-to-LDS load: each active lane l reads the 4 (16) bytes at base + voff and writes
// them to LDS at byte lds + 4 l (16 l) (base and lds wave-uniform; m0 holds the LDS address, and one
// wait state separates its write from the load).  Written as asm so that the compiler does not
// track these loads: it would make every LDS read of the kernel wait for all of them.  The kernel
// waits for them itself (wait_vm_lgkm); they have no register results.
template <bool WIDE>
__device__ __forceinline__ void stage_load(const char *base, uint32_t voff, uint32_t lds) {
  // both uniform operands pass through readfirstlane: the compiler may otherwise hold a uniform
  // value it cannot prove uniform in a vector register, which an "s" operand does not accept
  const uint64_t b = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)((uintptr_t)base >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)base);
  const uint32_t m = __builtin_amdgcn_readfirstlane(lds);
  if constexpr (WIDE)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0" : : "s"(b), "v"(voff), "s"(m)
                 : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %1, %0" : : "s"(b), "v"(voff), "s"(m)
                 : "memory", "m0");
}

// What a wave loads of every shell: planes w and w + 4, from which rows and columns.  Rows and columns
// past the one upstream of the lattice's edge belong to no site; they repeat that one, so every address
// lies inside the plane.
template <class ST, typename S, bool WIDE>
struct StagePlan {
  using L = Stage2D<ST, S>;
  int w;                  // wave of the block (uniform)
  int plane[2], nrow[2];  // uniform
  bool side[2];           // uniform
  int64_t row[2][5];      // byte offsets of the window rows (uniform; 4 bytes per lane)
  uint32_t wide[2][3];    // byte offset of this lane's 16 bytes in the plane, for each of the rows' instructions
  bool wlane[2][3];       // and whether they belong to a window row
  uint32_t lds[2];        // LDS byte offset of the window's first row in a buffer (uniform)
  uint32_t col[L::H];     // byte offset of this lane's 4 bytes in a row
  uint32_t scol[2];       // and in the plane, of this lane's part of the side column
  bool slane[2];          // this lane takes part in the side load

  __device__ __forceinline__ StagePlan(CTables *tb, int x0, int y0) {
    const int nx = tb->nx, ny = tb->ny, openx = tb->open[0], openy = tb->open[1];
    const int lane = threadIdx.x;
    w = __builtin_amdgcn_readfirstlane(threadIdx.y);
#pragma unroll
    for (int h = 0; h < L::H; ++h) {
      const int c = h * (64 / L::H) + lane / L::H;
      col[h] = (uint32_t)near_site(min(x0 + c, nx), nx, openx) * (uint32_t)sizeof(S) + (lane % L::H) * 4u;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      int dx = 0, dy = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (w == k) {
          dx = ST::dir(k + 4 * e, 0);
          dy = ST::dir(k + 4 * e, 1);
          lds[e] = L::body(k + 4 * e) * (uint32_t)sizeof(S);
        }
      plane[e] = w + 4 * e;
      nrow[e] = dy != 0 ? 5 : 4;
      side[e] = dx != 0;
      const int yf = y0 - (dy > 0);   // the window's first row
#pragma unroll
      for (int r = 0; r < 5; ++r)
        row[e][r] = (int64_t)near_site(min(yf + r, ny), ny, openy) * nx * (int64_t)sizeof(S);
#pragma unroll
      for (int n = 0; n < 3; ++n) {
        const int r = n * L::RPI + lane / L::LPR, c = lane % L::LPR * (16 / (int)sizeof(S));
        wide[e][n] = ((uint32_t)near_site(min(yf + r, ny), ny, openy) * (uint32_t)nx +
                      (uint32_t)near_site(min(x0 + c, nx), nx, openx)) * (uint32_t)sizeof(S);
        wlane[e][n] = r < nrow[e];
      }
      const int r = lane / L::H;      // the row of this lane's part of the side column
      const int ys = near_site(min(yf + r, ny), ny, openy), xs = near_site(min(dx > 0 ? x0 - 1 : x0 + 64, nx), nx, openx);
      scol[e] = ((uint32_t)ys * (uint32_t)nx + (uint32_t)xs) * (uint32_t)sizeof(S) + (lane % L::H) * 4u;
      slane[e] = r < nrow[e];
    }
  }

  // the loads of a shell into the buffer at LDS byte buf
  __device__ __forceinline__ void load(const S *__restrict__ fin, int64_t sites, int shell, uint32_t buf) const {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const char *p = (const char *)(fin + (int64_t)(shell * ST::NDIR + plane[e]) * sites);
      if constexpr (WIDE) {
#pragma unroll
        for (int n = 0; n * L::RPI < 5; ++n)
          if (wlane[e][n]) stage_load<true>(p, wide[e][n], buf + lds[e] + (uint32_t)(n * 1024));
      } else {
#pragma unroll
        for (int r = 0; r < 5; ++r) {
          if (r == 4 && nrow[e] == 4) break;
#pragma unroll
          for (int h = 0; h < L::H; ++h)
            stage_load<false>(p + row[e][r], col[h], buf + lds[e] + (uint32_t)(r * 64 * (int)sizeof(S) + h * 256));
        }
      }
      if (side[e] && slane[e]) stage_load<false>(p, scol[e], buf + lds[e] - (uint32_t)(L::kSide * (int)sizeof(S)));
    }
  }
};

// Taps of a shell from its staged windows: the values (read) and their weighted sums (interpolate)
// are separate steps, so that the next shell's loads can be issued between them.
template <class ST, typename S>
struct StageTaps {
  static constexpr int count() {
    int c = 0;
    for (int k = 0; k < ST::NDIR; ++k) c += 1 << ((ST::dir(k, 0) != 0) + (ST::dir(k, 1) != 0));
    return c;
  }
  S v[count()];
};

// Element offsets of this thread's site in a window's row ty (at[.][0]) and ty + 1 (at[.][1]): its left
// neighbour, itself, its right neighbour; the first and last lane find theirs in the side column.
struct StageAt {
  int at[3][2];
  __device__ __forceinline__ StageAt(int side) {
    const int tx = threadIdx.x, ty = threadIdx.y;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      at[1][r] = (ty + r) * 64 + tx;
      at[0][r] = tx == 0 ? ty + r - side : at[1][r] - 1;
      at[2][r] = tx == 63 ? ty + r - side : at[1][r] + 1;
    }
  }
};

template <class ST, typename S>
__device__ __forceinline__ void stage_read(const __attribute__((address_space(3))) S *buf, const StageAt &o,
                                           StageTaps<ST, S> &t) {
  using L = Stage2D<ST, S>;
  int m = 0;
#pragma unroll
  for (int k = 0; k < ST::NDIR; ++k) {
    const int dx = ST::dir(k, 0), dy = ST::dir(k, 1);
    const int z = (dx != 0) + (dy != 0);
#pragma unroll
    for (int tap = 0; tap < (1 << z); ++tap) {
      int bit = 0, ox = 0, oy = 0;
      if (dx != 0) {
        const int c = (tap >> bit++) & 1;
        ox = dx > 0 ? (c ? 0 : -1) : (c ? 1 : 0);
      }
      if (dy != 0) {
        const int c = (tap >> bit++) & 1;
        oy = dy > 0 ? (c ? 0 : -1) : (c ? 1 : 0);
      }
      t.v[m++] = buf[L::body(k) + o.at[ox + 1][dy > 0 ? oy + 1 : oy]];
    }
  }
}

template <class ST, typename S, typename A>
__device__ __forceinline__ void stage_interpolate(CTables *tb, int j, const StageTaps<ST, S> &t,
                                                  A (&fs)[ST::NDIR]) {
  const A v = tab<A>(tb->sv[j], tb->svf[j]);
  A pw[3][3];
#pragma unroll
  for (int z = 1; z <= 2; ++z) {
    const A mag = v * (A)kInvNorm[z];
    const A cm = (A)1 - mag;
#pragma unroll
    for (int nf = 0; nf <= z; ++nf) {
      A r = 1;
#pragma unroll
      for (int q = 0; q < nf; ++q) r *= mag;
#pragma unroll
      for (int q = nf; q < z; ++q) r *= cm;
      pw[z][nf] = r;
    }
  }
  int m = 0;
#pragma unroll
  for (int k = 0; k < ST::NDIR; ++k) {
    const int dx = ST::dir(k, 0), dy = ST::dir(k, 1);
    const int z = (dx != 0) + (dy != 0);
    A acc = 0;
#pragma unroll
    for (int tap = 0; tap < (1 << z); ++tap) {
      int bit = 0, nfar = 0;
      if (dx != 0) nfar += dx > 0 ? !((tap >> bit++) & 1) : ((tap >> bit++) & 1);
      if (dy != 0) nfar += dy > 0 ? !((tap >> bit++) & 1) : ((tap >> bit++) & 1);
      acc += pw[z][nfar] * (A)t.v[m++];
    }
    fs[k] = acc;
  }
}

// The taps of a shell's populations at a site, from global memory; TRANSPOSE mirrors them as pull_prod does.
// stage_interpolate sums them.  fin: the shell's first plane; moved on to the next shell's.
template <class ST, typename S, bool TRANSPOSE>
__device__ __forceinline__ void load_taps(const S *&fin, int64_t sites, const Offs &o, StageTaps<ST, S> &t) {
  typedef const __attribute__((address_space(1))) char gchar;
  int m = 0;
#pragma unroll
  for (int k = 0; k < ST::NDIR; ++k) {
    gchar *plane = (gchar *)fin + k * sites * (int64_t)sizeof(S);
    const int dx = ST::dir(k, 0), dy = ST::dir(k, 1);
    const int z = (dx != 0) + (dy != 0);
#pragma unroll
    for (int tap = 0; tap < (1 << z); ++tap) {
      int bit = 0, ox = 0, oy = 0;
      if (dx != 0) {
        const int c = (tap >> bit++) & 1;
        ox = dx > 0 ? (c ? 0 : -1) : (c ? 1 : 0);
      }
      if (dy != 0) {
        const int c = (tap >> bit++) & 1;
        oy = dy > 0 ? (c ? 0 : -1) : (c ? 1 : 0);
      }
      if (TRANSPOSE) {
        ox = -ox;
        oy = -oy;
      }
      const uint32_t off = o.x[ox + 1] + o.y[oy + 1];
      t.v[m++] = *(const __attribute__((address_space(1))) S *)(plane + off);
    }
  }
  fin += ST::NDIR * sites;
  one_after_another(fin);
}

// pull_prod with the loads of a shell asked for before the sums of the shell before it.
template <class ST, typename S, typename A>
__device__ __forceinline__ void pull_ahead(CTables *tb, const S *fin, int64_t sites, const Offs &o, A (&f)[ST::Q]) {
  constexpr int KR = ST::NSHELL;
  StageTaps<ST, S> t[2];
  load_taps<ST, S, false>(fin, sites, o, t[0]);
#pragma unroll
  for (int j = 0; j < KR; ++j) {
    if (j + 1 < KR) load_taps<ST, S, false>(fin, sites, o, t[(j + 1) & 1]);
    __builtin_amdgcn_sched_barrier(0);
    A fs[ST::NDIR];
    stage_interpolate<ST, S, A>(tb, j, t[j & 1], fs);
#pragma unroll
    for (int k = 0; k < ST::NDIR; ++k) {
      asm volatile("" : "+v"(fs[k]));   // summed here: its taps' registers are free again
      f[j * ST::NDIR + k] = fs[k];
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The pre-collision populations of this thread's site (x0 + threadIdx.x, y0 + threadIdx.y) of a 64 x 4
// tile.  Called by all threads of the block, also those of sites past the lattice's edge: they take part
// in the loads and barriers, and their populations are not those of a site.  No vector memory access of
// the caller may be in flight.
template <class ST, typename S, typename A, bool WIDE>
__device__ __forceinline__ void stage_pull(CTables *tb, const S *__restrict__ fin, int64_t sites, int x0,
                                           int y0, S *buf, A (&f)[ST::Q]) {
  using L = Stage2D<ST, S>;
  constexpr int KR = ST::NSHELL;
  static_assert(KR >= 2, "two shells in flight");
  typedef __attribute__((address_space(3))) S lds_t;
  const uint32_t lds = (uint32_t)(uintptr_t)(lds_t *)buf;   // LDS byte address of the buffers
  const StagePlan<ST, S, WIDE> plan(tb, x0, y0);
  plan.load(fin, sites, 0, lds);
  plan.load(fin, sites, 1, lds + L::E * (int)sizeof(S));
  const StageAt at(L::kSide);
#pragma unroll
  for (int j = 0; j < KR; ++j) {
    // shell j has landed in this wave's part of its buffer once at most the loads of shell j + 1
    // are in flight (no other vector memory access is issued before the last shell; the fewest that a
    // wave of the block has of a shell); the barrier extends that to the whole block
    if (j + 1 < KR) wait_vm_lgkm<L::min_loads(WIDE)>();
    else wait_vm_lgkm<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    StageTaps<ST, S> taps;
    stage_read<ST, S>((const lds_t *)buf + (j & 1) * L::E, at, taps);
    if (j + 2 < KR) {
      // every wave has read shell j before its buffer is refilled with shell j + 2, whose loads
      // then overlap the interpolation and shell j + 1
      wait_lgkm();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      plan.load(fin, sites, j + 2, lds + (j & 1) * L::E * (int)sizeof(S));
    }
    A fs[ST::NDIR];
    stage_interpolate<ST, S, A>(tb, j, taps, fs);
    // the shell's sums are formed here, before the next barrier, so that its taps do not stay live
    // in registers across the later shells (the compiler would otherwise sink every sum to the end)
#pragma unroll
    for (int k = 0; k < ST::NDIR; ++k) {
      asm volatile("" : "+v"(fs[k]));
      f[j * ST::NDIR + k] = fs[k];
    }
  }
}

// Rows may be loaded 16 bytes per lane: every row of every plane starts on 16 bytes and every chunk of 16 lies inside
// the lattice or past its edge as a whole (an open x axis repeats its last site, so no chunk may lie past it).
// Taken in double storage without walls and force, where a wave then issues 7 loads a shell instead of 20.  That is
// all it gives: in time the two forms are even (2048 x 2048 371.4 and 371.5 us, 1024 x 1024 102.6 and 103.3,
// 3000 x 1500 466 and 465); in float storage and with walls the 4-byte loads are ahead (float 2048 x 2048 210 against
// 211.6 us, walls at 1024 x 1024 106.7 against 107.5).
inline bool stage_wide(const void *fin, int nx, int elem, bool openx) {
  return (uintptr_t)fin % 16 == 0 && nx * elem % 16 == 0 && (!openx || nx % 64 == 0);
}

}  // namespace rlbm
