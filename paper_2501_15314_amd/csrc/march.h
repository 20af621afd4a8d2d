// Plane-marching stencil kernels on the red/black split layout.
//
// A workgroup owns a tile of BY rows (axis 1) x 2*BX in-row indices m
// (axis 2, two per thread, accessed as 2-vectors) and marches over a chunk of
// planes along axis 0 (Geo::mbx, mby, mch, mch3).  The x-neighbours of a cell come from a
// register window over three planes, the y- and z-neighbours from an LDS copy
// of the current plane with a one-cell halo.  BX divides hn2/2 and BY divides
// n1, so no workgroup is partial and every halo cell is loaded.
//
// These kernels move bytes: at 256^3 in float32 a pressure half sweep moves
// 101 MB, near the 5 to 6 TB/s that reads and writes of such sets reach.  To
// stay at that they have to spend few instructions per plane, since a wave has
// one vector and one scalar issue slot in four cycles: what is fixed along a
// march (halo positions, stencil diagonals and their reciprocals) is found
// before it, the parity of a plane is an index into two sets of records, the
// register window moves by renaming over four unrolled planes, plane offsets
// are scalar and advance by addition, no load is under a condition, and LDS is
// double buffered, which leaves one barrier per plane.  Per wave and plane a
// pressure half sweep takes about 30 vector instructions (81 and, for its
// setup, 246 per chunk when every plane found its own halo and diagonals), the
// Laplacian about 100 (232, two IEEE divisions per colour and cell pair among
// them).  At 256^3 float32, before and after, us: half sweep 20.4 / 19.3, first
// sweep 31.3 / 21.9, restriction 24.6 / 20.0, prolongation 23.8 / 15.2,
// Laplacian 33.5 / 24.7 (5.2, 4.6, 5.4, 4.9, 5.4 TB/s); float64: 41.0 / 37.8,
// 43.2 / 38.9, 41.1 / 39.8, 39.3 / 31.7, 51.5 / 51.6; at 128^3 float32, where
// the grids are small and setup counts: 6.7 / 5.5, 8.9 / 7.1, 7.5 / 5.0,
// 7.3 / 5.3, 10.3 / 7.5; momentum half sweep at 256^3 float32 66.2 / 65.9, its
// first sweep 108 / 76.5.
#pragma once
#include <hip/hip_ext.h>

#include <type_traits>

#include "internal.h"

namespace ibs {

constexpr int MARCH_CH = 8;       // most planes per workgroup
constexpr int MARCH_TILE = 1104;  // >= max (BY+2)(2BX+2) over BX*BY <= 256

struct MarchShape {
  int bx, by;
  dim3 grid, block;
};

// ncomp stacks independent component grids along grid.z.
inline MarchShape march_shape(const Geo &g, int ncomp) {
  MarchShape s;
  s.bx = g.mbx;
  s.by = g.mby;
  s.block = dim3(s.bx, s.by, 1);
  const int len = ncomp == 3 ? g.mch3 : g.mch;
  int nch = (g.n0 + len - 1) / len;
  s.grid = dim3(g.hn2 / (2 * s.bx), g.n1 / s.by, nch * ncomp);
  return s;
}

template <typename T>
struct V2 {
  T x, y;
};
// Element and 2-vector access at a byte offset from a pointer that is the same
// for the whole workgroup: the offset is 32 bits wide (one plane of one colour
// is far below 4 GiB), so an access needs one address register and no 64-bit
// arithmetic per lane.
template <typename S>
__device__ __forceinline__ S ldo(const S *p, unsigned off) {
  return *(const S *)((const char *)p + off);
}
template <typename R, typename S>
__device__ __forceinline__ V2<R> ld2(const S *p, unsigned off = 0) {
  V2<R> v;
  const char *q = (const char *)p + off;
  if (sizeof(S) == 4) {
    float2 f = *(const float2 *)q;
    v.x = (R)f.x;
    v.y = (R)f.y;
  } else {
    double2 f = *(const double2 *)q;
    v.x = (R)f.x;
    v.y = (R)f.y;
  }
  return v;
}
template <typename T>
__device__ __forceinline__ void st2(T *p, unsigned off, T a, T b) {
  char *q = (char *)p + off;
  if (sizeof(T) == 4) {
    *(float2 *)q = make_float2((float)a, (float)b);
  } else {
    *(double2 *)q = make_double2((double)a, (double)b);
  }
}

// a / d for a divisor whose correctly rounded reciprocal r = 1 / d is at hand:
// one fused remainder step gives the correctly rounded quotient (Markstein's
// theorem; a and the quotient normal numbers), the same bits as the division
// at 3 operations instead of about 10.  Infinite quotients, whose remainder is
// infinite or NaN, stay infinite.
template <typename T>
__device__ __forceinline__ T div_by(T a, T d, T r) {
  const T q = a * r, e = fma(-q, d, a);
  return __builtin_isfinite(e) ? fma(e, r, q) : q;
}

// Coordinate wrap for periodic axes; -1 if outside a wall box.
__device__ __forceinline__ int mwrap(int i, int n, int bc) {
  if (i < 0) return bc ? -1 : i + n;
  if (i >= n) return bc ? -1 : i - n;
  return i;
}

// Tile coordinates of this workgroup.  The dispatcher deals consecutive
// workgroups round-robin to the 8 XCDs; with `xcd` set, each XCD walks all
// row tiles of one plane chunk (grid.z) in turn while the other XCDs take the
// seven chunks beside it, so the tiles that share halo rows run on one XCD at
// the same time and those re-reads hit its L2.  Measured, this pays on the
// three-component momentum grids and on the Laplacian of the S~ product, and
// costs time on the single-component multigrid levels, which keep the plain
// order.
struct MarchBlock {
  int x, y, z;
};
__device__ __forceinline__ MarchBlock march_block(bool xcd) {
  const unsigned gx = gridDim.x, gxy = gx * gridDim.y;
  MarchBlock mb;
  if (xcd && gridDim.z % 8 == 0) {
    const unsigned b = blockIdx.x + gx * (blockIdx.y + gridDim.y * blockIdx.z);
    const unsigned slot = b / 8, rem = slot % gxy;
    mb.x = rem % gx;
    mb.y = rem / gx;
    mb.z = (slot / gxy) * 8 + b % 8;
  } else {
    mb.x = blockIdx.x;
    mb.y = blockIdx.y;
    mb.z = blockIdx.z;
  }
  return mb;
}

// Per-block geometry of a march.
struct MarchPos {
  int tx, ty, m0, j, i0, i1, comp;
};
// len: planes per workgroup
__device__ __forceinline__ MarchPos march_pos(const Geo &g, int len, bool xcd) {
  MarchPos p;
  const MarchBlock mb = march_block(xcd);
  p.tx = threadIdx.x;
  p.ty = threadIdx.y;
  p.m0 = 2 * (mb.x * blockDim.x + threadIdx.x);
  p.j = mb.y * blockDim.y + threadIdx.y;
  int nch = (g.n0 + len - 1) / len;
  p.comp = mb.z / nch;
  int ch = mb.z - p.comp * nch;
  p.i0 = ch * len;
  p.i1 = min(p.i0 + len, g.n0);
  return p;
}

// The halo of a plane tile (rows ty = -1 and BY, columns m = -1 and 2 BX) by
// position: the threads of the tile's first and last row each bring the pair
// of cells beyond their own, those of its first and last column one cell.
// What does not change along the march -- offsets, LDS slots, whether the
// cells lie outside a wall box (they are 0: `zero` stores that once for both
// LDS buffers) -- is found here, without a division.  BY >= 2 (n1 is even and
// so is BY); a tile one pair wide (BX == 1: rows of 4 cells, or whose quarter is
// a prime above 64) has both columns at one thread, which brings the right one
// too, in kernels of their own (THIN; loaded where it is used, the cell costs the
// float64 momentum solve on 64 x 64 x 268 cells 30 us of 915).  Every thread loads: those
// that bring nothing share an address of their row, so that the loads are not
// under a condition (the compiler waits for all outstanding loads where a
// conditional one may or may not be among them, which serialises the march).
struct MarchEdge {
  int rslot, cslot;   // LDS slots of the row pair and the column cell, -1: none
  int jr, mr, mc;     // row and in-row index of the pair, in-row index of the column cell
  int mt, tslot;      // in-row index and slot of the right column cell of a thin tile
};
template <bool THIN, class Z>
__device__ __forceinline__ MarchEdge march_edge(const Geo &g, const MarchPos &p, int BX, int BY, Z zero) {
  MarchEdge e;
  const int W2 = 2 * BX + 2;
  const bool lastr = p.ty == BY - 1, lastc = !THIN && p.tx == BX - 1;
  e.rslot = e.cslot = e.tslot = -1;
  e.jr = THIN ? p.j - p.ty : p.j;  // in a thin tile the first row's for all, or each lane's would be a transaction
  e.mr = e.mc = e.mt = p.m0 - 2 * p.tx;
  if (p.ty == 0 || lastr) {
    const int jj = mwrap(lastr ? p.j + 1 : p.j - 1, g.n1, g.bc1);
    const int slot = (lastr ? BY + 1 : 0) * W2 + 2 * p.tx + 1;
    if (jj >= 0) {
      e.jr = jj;
      e.mr = p.m0;
      e.rslot = slot;
    } else {
      zero(slot);
      zero(slot + 1);
    }
  }
  if (p.tx == 0 || lastc) {
    const int mm = mwrap(lastc ? p.m0 + 2 : p.m0 - 1, g.hn2, g.bc2);
    const int slot = (p.ty + 1) * W2 + (lastc ? 2 * BX + 1 : 0);
    if (mm >= 0) {
      e.mc = mm;
      e.cslot = slot;
    } else {
      zero(slot);
    }
  }
  if (THIN) {
    const int mm = mwrap(p.m0 + 2, g.hn2, g.bc2), slot = (p.ty + 1) * W2 + 3;
    if (mm >= 0) {
      e.mt = mm;
      e.tslot = slot;
    } else {
      zero(slot);
    }
  }
  return e;
}

// Stencil diagonal of cell (jj, kk), the part of axes 1 and 2 (fixed along a
// march along axis 0) and the part of axis 0 (per plane).  Pressure
// Laplacian: the number of missing neighbours (the cell has 6 - di - djk);
// momentum operator on component d: the 7-point diagonal count in units of
// 1/h^2 (di + djk) with the tangential wall ghosts.
__device__ __forceinline__ int diag_jk(const Geo &g, int jj, int kk, bool helm, int d) {
  const int e1 = (jj == 0) + (jj == g.n1 - 1), e2 = (kk == 0) + (kk == g.n2 - 1);
  if (!helm) return (g.bc1 ? e1 : 0) + (g.bc2 ? e2 : 0);
  return 4 + (g.bc1 && d != 1 ? wall_ghost_diag(g.bc1) * e1 : 0) + (g.bc2 && d != 2 ? wall_ghost_diag(g.bc2) * e2 : 0);
}
// a normal wall face of momentum component d (held at 0), axes 1 and 2
__device__ __forceinline__ bool wall_jk(const Geo &g, int jj, int kk, int d) {
  return d == 1 ? (g.bc1 && jj == 0) : (d == 2 ? (g.bc2 && kk == 0) : false);
}

// Where a march stands: element offsets, from the start of a colour plane
// array, of the plane being computed, of the next one (the last one again at
// the end of the chunk) and of the one after it (wrapped; the nearest one
// outside a wall box).  All scalar and advanced by additions: with the vector
// work of a plane down to a few tens of instructions, multiplying each offset
// out again would cost as much.
struct MarchOff {
  long long cur, nxt, win;
  long long P, wrap;
  int last, n0;
};
__device__ __forceinline__ long long march_win(const MarchOff &o, int i, long long at) {
  return i + 1 < o.n0 ? at + o.P : o.wrap;
}
__device__ __forceinline__ MarchOff march_off(const Geo &g, int i0, int i1) {
  MarchOff o;
  o.P = (long long)g.n1 * g.hn2;
  o.wrap = g.bc0 ? (g.n0 - 1) * o.P : 0;
  o.last = i1 - 1;
  o.n0 = g.n0;
  o.cur = o.nxt = i0 * o.P;
  o.win = march_win(o, i0, o.nxt);
  return o;
}
// to plane i: nxt and win become those of plane i + 1
__device__ __forceinline__ void march_next(MarchOff &o, int i) {
  o.cur = o.nxt;
  if (i < o.last) {
    o.nxt += o.P;
    o.win = march_win(o, i + 1, o.nxt);
  }
}
// offset of the plane before i0
__device__ __forceinline__ long long march_prev(const Geo &g, const MarchOff &o, int i0) {
  return i0 > 0 ? o.cur - o.P : (g.bc0 ? 0 : (g.n0 - 1) * o.P);
}

// What a cell's update needs besides the field values, found once per march
// for the planes inside the grid (the planes at a wall of axis 0 form it anew
// from the packed diagonal counts): `inv` = 1 / number of neighbours for the
// pressure; the divisor a0 + nu/h^2 diag, its reciprocal and the wall flag for
// the momentum operator.
template <typename T>
struct CellRec {
  T inv, den;
  bool wall;
};

// One red-black half sweep of colour `color` on the component grids of x.
//   SW_POISSON: x_c = (h^2 b_c + sum of neighbours) / (number of neighbours)
//               (Gauss-Seidel for L = G^T G);
//   SW_FIRST:   the first pressure sweep from x = 0, colour 1: the colour-0
//               values h^2 b / nnb are formed on the fly from b (and stored),
//               then the colour-1 update as above;
//   SW_HELM:    SOR for A = a0 - nu Delta_h on velocity component `comp`:
//               x_c += omega ((b_c + nu/h^2 sum) / (a0 + nu/h^2 diag) - x_c),
//               wall faces untouched.  Neighbours outside a wall box are 0
//               (normal walls hold 0, tangential ghosts enter the diagonal:
//               -u on a no-slip wall, +u on a free-slip wall).
//   SW_HFIRST:  the first SOR sweep of SW_HELM from x = 0, colour 1: the
//               colour-0 values omega b / (a0 + nu/h^2 diag) are formed on
//               the fly from b (and stored), then the colour-1 update; one
//               pass replaces clearing x and two half sweeps.
//   SW_FIRST1:  SW_FIRST without storing the colour-0 values, for a cycle
//               whose next half sweep recomputes colour 0 from colour 1
//               (a Gauss-Seidel update never reads the old value of its
//               own colour).
enum { SW_POISSON = 0, SW_FIRST = 1, SW_HELM = 2, SW_HFIRST = 3, SW_FIRST1 = 4 };

template <typename T, typename TB, int MODE, bool THIN>
__global__ void __launch_bounds__(256) k_sweep(Geo g, T *x, const TB *b, int color, double h2, double a0,
                                               double nuh2, double omega) {
  constexpr bool FIRSTM = MODE == SW_FIRST || MODE == SW_HFIRST || MODE == SW_FIRST1;
  constexpr bool HELMM = MODE == SW_HELM || MODE == SW_HFIRST;
  __shared__ T tile[2][MARCH_TILE];
  const MarchPos p = march_pos(g, HELMM ? g.mch3 : g.mch, HELMM);
  const int BX = blockDim.x, BY = blockDim.y, W2 = 2 * BX + 2;
  const int d = p.comp, c = FIRSTM ? 1 : color;
  const long long N = 2 * g.half;
  T *own = x + d * N + (long long)c * g.half;
  T *oth = x + d * N + (long long)(1 - c) * g.half;
  const TB *bown = b + d * N + (long long)c * g.half;
  // the other colour: in the first-sweep modes it is formed from the
  // right-hand side (the loads fetch that raw, oxf turns it into the value)
  using TO = typename std::conditional<FIRSTM, TB, T>::type;
  const TO *osrc = FIRSTM ? (const TO *)(b + d * N + (long long)(1 - c) * g.half) : (const TO *)oth;
  const unsigned rw = p.j * g.hn2 + p.m0;  // this thread's two cells within a plane
  const T th2 = (T)h2, ta0 = (T)a0, tnu = (T)nuh2, tom = (T)omega;
  const MarchEdge e = march_edge<THIN>(g, p, BX, BY, [&](int q) { tile[0][q] = tile[1][q] = T(0); });
  const unsigned eoff = (unsigned)(e.jr * g.hn2 + e.mr) * sizeof(TO), coff = (unsigned)(p.j * g.hn2 + e.mc) * sizeof(TO),
                 toff = (unsigned)(p.j * g.hn2 + e.mt) * sizeof(TO);

  // Own cells at plane i have k = 2 m + s, s = (c + i + j) & 1; the
  // other-colour cells of the same row 1 - s, those of the rows beside it s.
  // Index 0 holds for the plane i0 and every second one after it.
  const int s0 = (c + p.i0 + p.j) & 1;
  auto rec = [&](int diag, bool wall) {
    CellRec<T> r;
    if (HELMM) {
      r.den = fma(tnu, (T)diag, ta0);
      r.inv = T(1) / r.den;
    } else {
      r.den = T(0);
      r.inv = inv_nn<T>(6 - diag);
    }
    r.wall = wall;
    return r;
  };
  const int di0 = HELMM ? 2 : 0;
  CellRec<T> ro[2][2], rr[2][2], rc[2], rt[2];  // own row (either colour), row pair, column cells
  unsigned pk = 0, pkr = 0, pkc = 0, pkt = 0;    // their counts of axes 1 and 2, 4 bits each
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int s = f ? 1 - s0 : s0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int k = 2 * (p.m0 + u) + s;
      const int dg = diag_jk(g, p.j, k, HELMM, d);
      pk |= (unsigned)dg << (8 * f + 4 * u);
      ro[f][u] = rec(di0 + dg, HELMM && wall_jk(g, p.j, k, d));
      if (FIRSTM) {
        const int dr = diag_jk(g, e.jr, k, HELMM, d);
        pkr |= (unsigned)dr << (8 * f + 4 * u);
        rr[f][u] = rec(di0 + dr, HELMM && wall_jk(g, e.jr, k, d));
      }
    }
    if (FIRSTM) {
      const int k = 2 * e.mc + s;
      const int dc = diag_jk(g, p.j, k, HELMM, d);
      pkc |= (unsigned)dc << (4 * f);
      rc[f] = rec(di0 + dc, HELMM && wall_jk(g, p.j, k, d));
      if (THIN) {
        const int kt = 2 * e.mt + s;
        const int dt = diag_jk(g, p.j, kt, HELMM, d);
        pkt |= (unsigned)dt << (4 * f);
        rt[f] = rec(di0 + dt, HELMM && wall_jk(g, p.j, kt, d));
      }
    }
  }
  // planes at a wall of axis 0: where the tabulated records do not hold (e0,
  // e1), past which there is no plane (z0, z1), wall faces of component 0
  const bool diw = HELMM ? g.bc0 && d != 0 : g.bc0 != 0;
  const int e0 = diw ? 0 : -2, e1 = diw ? g.n0 - 1 : -2, z0 = g.bc0 ? 0 : -2, z1 = g.bc0 ? g.n0 - 1 : -2;
  const int wf0 = HELMM && d == 0 && g.bc0 ? 0 : -2;
  const int die = HELMM ? 2 + wall_ghost_diag(g.bc0) : 1;
  struct Pair {
    CellRec<T> r[2];
  };
  // the records of a pair at plane i: as tabulated, or anew
  auto at_plane = [&](int i, const CellRec<T> *r, unsigned packed, int sh) {
    Pair q;
    q.r[0] = r[0];
    q.r[1] = r[1];
    if (i == e0 || i == e1) {
      q.r[0] = rec(die + ((packed >> sh) & 15), r[0].wall);
      q.r[1] = rec(die + ((packed >> (sh + 4)) & 15), r[1].wall);
    }
    if (HELMM && i == wf0) q.r[0].wall = q.r[1].wall = true;
    return q;
  };
  // a colour-0 value of a first sweep from its right-hand side
  auto oxf = [&](T bv, const CellRec<T> &r) -> T {
    if (!HELMM) return pc_first(th2, bv, r.inv);
    const T v = tom * div_by(bv, r.den, r.inv);
    return r.wall ? T(0) : v;
  };
  MarchOff at = march_off(g, p.i0, p.i1);
  // the colour-0 pair of plane i (in the grid) in the first-sweep modes; f: index of its records
  auto owin = [&](int i, V2<T> v, int f) -> V2<T> {
    if (FIRSTM) {
      const Pair q = at_plane(i, ro[f], pk, 8 * f);
      v.x = oxf(v.x, q.r[0]);
      v.y = oxf(v.y, q.r[1]);
    }
    return v;
  };
  struct Ops {
    V2<T> hr, b, x, w;  // halo row pair, own right-hand side and value, other colour at the next plane
    T hc, ht;           // halo column cells
  };
  auto fetch = [&](Ops &o) {
    o.hr = ld2<T>(osrc + at.nxt, eoff);
    o.hc = (T)ldo(osrc + at.nxt, coff);
    if (THIN) o.ht = (T)ldo(osrc + at.nxt, toff);
    o.b = ld2<T>(bown + at.nxt, rw * (unsigned)sizeof(TB));
    if (MODE == SW_HELM) o.x = ld2<T>((const T *)own + at.nxt, rw * (unsigned)sizeof(T));
    o.w = ld2<T>(osrc + at.win, rw * (unsigned)sizeof(TO));
  };
  // Plane i from the other colour at planes i - 1 and i (wp, wc) and the
  // operands o; leaves that of plane i + 1 in wn.  The operands of plane i + 1
  // are loaded into on before anything is computed.  f: index of the records
  // of the own colour at plane i, and of the LDS buffer (two of them, so one
  // barrier per plane is enough).
  auto step = [&](int i, int f, const V2<T> &wp, const V2<T> &wc, V2<T> &wn, const Ops &o, Ops &on) {
    march_next(at, i);
    fetch(on);
    T *t = tile[f];
    T *trow = t + (p.ty + 1) * W2 + 2 * p.tx;
    trow[1] = wc.x;
    trow[2] = wc.y;
    V2<T> hr = o.hr;
    T hc = o.hc, ht = THIN ? o.ht : T(0);
    if (FIRSTM) {
      const Pair qr = at_plane(i, rr[f], pkr, 8 * f), qc = at_plane(i, rc, pkc, 0);
      hr.x = oxf(hr.x, qr.r[0]);
      hr.y = oxf(hr.y, qr.r[1]);
      hc = oxf(hc, qc.r[1 - f]);
      if (THIN) ht = oxf(ht, at_plane(i, rt, pkt, 0).r[1 - f]);
    }
    if (e.rslot >= 0) {
      t[e.rslot] = hr.x;
      t[e.rslot + 1] = hr.y;
    }
    if (e.cslot >= 0) t[e.cslot] = hc;
    const int s = f ? 1 - s0 : s0;
    if (THIN && e.tslot >= 0) t[e.tslot] = ht;
    __syncthreads();
    wn = i == z1 ? V2<T>{T(0), T(0)} : owin(i + 1 < g.n0 ? i + 1 : 0, o.w, f);
    const Pair q = at_plane(i, ro[f], pk, 8 * f);
    T out[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const T sum = (u ? wp.y : wp.x) + (u ? wn.y : wn.x) + trow[u + 1 - W2] + trow[u + 1 + W2] + trow[u + s] +
                    trow[u + 1 + s];
      const T bv = u ? o.b.y : o.b.x;
      const CellRec<T> &r = q.r[u];
      if (!HELMM) {
        out[u] = pc_relax(th2, bv, sum, r.inv);
      } else {
        const T xv = MODE == SW_HELM ? (u ? o.x.y : o.x.x) : T(0);
        const T gs = div_by<T>(fma(tnu, sum, bv), r.den, r.inv);
        out[u] = r.wall ? xv : fma(tom, gs - xv, xv);
      }
    }
    st2(own + at.cur, rw * (unsigned)sizeof(T), out[0], out[1]);
    if (MODE == SW_FIRST || MODE == SW_HFIRST) st2(oth + at.cur, rw * (unsigned)sizeof(T), wc.x, wc.y);
  };
  // the other colour's records at plane i0 are those of index 1
  const V2<T> lp = ld2<T>(osrc + march_prev(g, at, p.i0), rw * (unsigned)sizeof(TO));
  const V2<T> lc = ld2<T>(osrc + at.cur, rw * (unsigned)sizeof(TO));
  Ops oa, ob;
  fetch(oa);
  V2<T> w0 = p.i0 == z0 ? V2<T>{T(0), T(0)} : owin(p.i0 > 0 ? p.i0 - 1 : g.n0 - 1, lp, 0), w1 = owin(p.i0, lc, 1), w2, w3;
  // four planes per turn, so that the window moves by renaming
  for (int i = p.i0;;) {
    step(i, 0, w0, w1, w2, oa, ob);
    if (++i >= p.i1) break;
    step(i, 1, w1, w2, w3, ob, oa);
    if (++i >= p.i1) break;
    step(i, 0, w2, w3, w0, oa, ob);
    if (++i >= p.i1) break;
    step(i, 1, w3, w0, w1, ob, oa);
    if (++i >= p.i1) break;
  }
}

template <typename T, typename TB, int MODE>
hipError_t sweep_launch(const MarchShape &M, const Geo &g, T *x, const TB *b, int color, double a0, double nuh2,
                        double omega, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (M.bx == 1)
    hipExtLaunchKernelGGL((k_sweep<T, TB, MODE, true>), M.grid, M.block, 0, s, e0, e1, 0, g, x, b, color, g.h2, a0, nuh2,
                          omega);
  else
    hipExtLaunchKernelGGL((k_sweep<T, TB, MODE, false>), M.grid, M.block, 0, s, e0, e1, 0, g, x, b, color, g.h2, a0, nuh2,
                          omega);
  return hipGetLastError();
}

// Operators on both colours at once: every thread owns the four cells of
// row (i, j) stored at in-row indices m0, m0+1 of both colour planes.
//   AP_LAP:    y = L x  (x of type T, y double) for the pressure Laplacian;
//   AP_HRESID: r = b - A x on velocity component `comp` (x, b double; r of
//              type TR), plus per-block partial sums of r^2 into part.
enum { AP_LAP = 0, AP_HRESID = 1 };

template <typename T, typename TR, int MODE, bool THIN>
__global__ void __launch_bounds__(256) k_apply2(Geo g, const T *x, const double *b, TR *out, double a0, double nuh2,
                                                double *part) {
  constexpr bool HELMM = MODE == AP_HRESID;
  constexpr int NB = sizeof(T) == 4 ? 2 : 1;  // LDS buffers: two spare a barrier, but in float64 cost residency
  __shared__ T tile[NB][2][MARCH_TILE];       // [buffer][colour]
  __shared__ double red[4];
  const MarchPos p = march_pos(g, HELMM ? g.mch3 : g.mch, true);  // chunk-per-XCD order (L z at 256^3: 46.2 -> 42.9 us)
  const int BX = blockDim.x, BY = blockDim.y, W2 = 2 * BX + 2;
  const int d = p.comp;
  const long long N = 2 * g.half;
  const T *xg = x + d * N;
  const double *bg = b ? b + d * N : nullptr;
  TR *og = out + d * N;
  const unsigned rw = p.j * g.hn2 + p.m0;  // this thread's cells within a plane
  const MarchEdge e = march_edge<THIN>(g, p, BX, BY, [&](int q) {
#pragma unroll
    for (int z = 0; z < NB; ++z) tile[z][0][q] = tile[z][1][q] = T(0);
  });
  const unsigned eoff = (unsigned)(e.jr * g.hn2 + e.mr) * sizeof(T), coff = (unsigned)(p.j * g.hn2 + e.mc) * sizeof(T),
                 toff = (unsigned)(p.j * g.hn2 + e.mt) * sizeof(T);
  // coefficient of the cell itself, inside the grid: for parity index f and
  // cell u (the cells of colour 0 at plane i0 have k = 2 m + s0)
  const int s0 = (p.i0 + p.j) & 1, di0 = HELMM ? 2 : 0;
  const double rh2 = 1.0 / g.h2;
  auto coef = [&](int diag) { return HELMM ? fma(nuh2, (double)diag, a0) : (double)(6 - diag); };
  double ca[2][2];
  bool wl[2][2];
  unsigned pk = 0;
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int k = 2 * (p.m0 + u) + (f ? 1 - s0 : s0);
      const int dg = diag_jk(g, p.j, k, HELMM, d);
      pk |= (unsigned)dg << (8 * f + 4 * u);
      ca[f][u] = coef(di0 + dg);
      wl[f][u] = HELMM && wall_jk(g, p.j, k, d);
    }
  struct Win {
    V2<T> q[2];
  };
  MarchOff at = march_off(g, p.i0, p.i1);
  auto win_ld = [&](long long off) {
    Win r;
#pragma unroll
    for (int q = 0; q < 2; ++q) r.q[q] = ld2<T>(xg + q * g.half + off, rw * (unsigned)sizeof(T));
    return r;
  };
  Win none;
  none.q[0] = none.q[1] = V2<T>{T(0), T(0)};
  const bool diw = HELMM ? g.bc0 && d != 0 : g.bc0 != 0;
  const int e0 = diw ? 0 : -2, e1 = diw ? g.n0 - 1 : -2, z0 = g.bc0 ? 0 : -2, z1 = g.bc0 ? g.n0 - 1 : -2;
  const int wf0 = HELMM && d == 0 && g.bc0 ? 0 : -2;
  const int die = HELMM ? 2 + wall_ghost_diag(g.bc0) : 1;
  struct Ops {
    V2<T> hr[2];
    T hc[2], ht[2];
    V2<double> b[2];
    Win w;
  };
  auto fetch = [&](Ops &o) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const T *xp = xg + q * g.half + at.nxt;
      o.hr[q] = ld2<T>(xp, eoff);
      o.hc[q] = ldo(xp, coff);
      if (THIN) o.ht[q] = ldo(xp, toff);
      if (MODE == AP_HRESID) o.b[q] = ld2<double>(bg + q * g.half + at.nxt, rw * (unsigned)sizeof(double));
    }
    o.w = win_ld(at.win);
  };
  double acc = 0.0;
  // as in k_sweep; f: parity index of colour 0 at plane i, and the LDS buffer
  auto step = [&](int i, int f, const Win &wp, const Win &wc, Win &wn, const Ops &o, Ops &on) {
    march_next(at, i);
    fetch(on);
    const int rowb = (p.ty + 1) * W2 + 2 * p.tx;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      T *t = tile[f % NB][q];
      t[rowb + 1] = wc.q[q].x;
      t[rowb + 2] = wc.q[q].y;
      if (e.rslot >= 0) {
        t[e.rslot] = o.hr[q].x;
        t[e.rslot + 1] = o.hr[q].y;
      }
      if (e.cslot >= 0) t[e.cslot] = o.hc[q];
      if (THIN && e.tslot >= 0) t[e.tslot] = o.ht[q];
    }
    __syncthreads();
    wn = i == z1 ? none : o.w;
    const bool edge = i == e0 || i == e1;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int fq = f ^ q;
      const T *trow = tile[f % NB][1 - q] + rowb;
      const int s = fq ? 1 - s0 : s0;
      double r[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const double sum = (double)(u ? wp.q[1 - q].y : wp.q[1 - q].x) + (double)(u ? wn.q[1 - q].y : wn.q[1 - q].x) +
                           (double)trow[u + 1 - W2] + (double)trow[u + 1 + W2] + (double)trow[u + s] +
                           (double)trow[u + 1 + s];
        const double xv = (double)(u ? wc.q[q].y : wc.q[q].x);
        double cc = ca[fq][u];
        if (edge) cc = coef(die + ((pk >> (8 * fq + 4 * u)) & 15));
        if (MODE == AP_LAP) {
          r[u] = div_by<double>(fma(cc, xv, -sum), g.h2, rh2);
        } else {
          const bool wall = i == wf0 || wl[fq][u];
          const double rv = (u ? o.b[q].y : o.b[q].x) - fma(cc, xv, -mul_rn(nuh2, sum));
          r[u] = wall ? 0.0 : rv;
          acc = fma(r[u], r[u], acc);
        }
      }
      st2(og + q * g.half + at.cur, rw * (unsigned)sizeof(TR), (TR)r[0], (TR)r[1]);
    }
    if (NB == 1) __syncthreads();
  };
  Win w0 = win_ld(march_prev(g, at, p.i0)), w1 = win_ld(at.cur), w2, w3;
  Ops oa, ob;
  fetch(oa);
  if (p.i0 == z0) w0 = none;
  for (int i = p.i0;;) {
    step(i, 0, w0, w1, w2, oa, ob);
    if (++i >= p.i1) break;
    step(i, 1, w1, w2, w3, ob, oa);
    if (++i >= p.i1) break;
    step(i, 0, w2, w3, w0, oa, ob);
    if (++i >= p.i1) break;
    step(i, 1, w3, w0, w1, ob, oa);
    if (++i >= p.i1) break;
  }
  if (MODE == AP_HRESID) {
    const int tid = threadIdx.x + blockDim.x * threadIdx.y;
    acc = wave_sum(acc);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) {
      double t = 0.0;
      const int nw = (blockDim.x * blockDim.y + 63) / 64;
      for (int w = 0; w < nw; ++w) t += red[w];
      part[blockIdx.x + (long long)gridDim.x * (blockIdx.y + (long long)gridDim.y * blockIdx.z)] = t;
    }
  }
}

}  // namespace ibs
