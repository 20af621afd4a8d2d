// Geometric multigrid V-cycle for the pressure Laplacian L = G^T G, used as
// the preconditioner M^-1 ~ L^+ of the Schur Krylov solve.  The paper applies
// an exact fast-diagonalisation solve of L once per iteration (Sec. 4.2) and
// names a multigrid V-cycle as its linear-time replacement (Sec. 7).
//
// Cycle: red-black Gauss-Seidel smoothing (pre: red then black, post: black
// then red, so the cycle is symmetric), residual restricted by averaging the
// eight children, trilinear cell-centred prolongation, coarse operators
// rediscretised on 2h, and a single-workgroup kernel that runs V-cycles on
// the coarsest grids entirely in LDS.  Kernels are templated on the working
// precision T (float or double) and on the right-hand-side type TB.
#include <hip/hip_ext.h>

#include <algorithm>

#include "internal.h"
#include "march.h"

namespace ibs {

// Coarse right-hand side: the average of the fine residual over the eight
// children.  The last half sweep relaxed the black cells, whose residual is
// therefore zero; only the four red children contribute: in fine planes 2I
// and 2I+1, rows 2J and 2J+1, each at in-row index K of the red plane.
//
// Plane march over the fine grid like the sweeps (register window of black
// planes along axis 0, LDS tile of the current black plane): a thread forms
// the residuals of its two red cells (in-row m0, m0+1 = coarse K, K+1),
// sums them over the plane pair, and the pair of rows is combined through
// LDS; the even-row thread writes the two coarse values (one per colour).
// The chunk of planes per workgroup is even, so a pair never splits.
__host__ __device__ inline int restrict_chunk(const Geo &gf) { return gf.mch < 2 ? 2 : gf.mch; }

template <typename T, typename TB, bool THIN>
__global__ void __launch_bounds__(256) k_restrict(Geo gf, const T *xf, const TB *bf, Geo gc, T *bc) {
  __shared__ T tile[2][MARCH_TILE];
  __shared__ T pair[256][2];
  const int BX = blockDim.x, BY = blockDim.y, W2 = 2 * BX + 2;
  MarchPos p;
  p.tx = threadIdx.x;
  p.ty = threadIdx.y;
  p.m0 = 2 * (blockIdx.x * BX + p.tx);
  p.j = blockIdx.y * BY + p.ty;
  const int tid = p.tx + BX * p.ty, len = restrict_chunk(gf);
  p.i0 = blockIdx.z * len;
  p.i1 = min(p.i0 + len, gf.n0);
  const T *red = xf, *blk = xf + gf.half;
  const long long PC = (long long)gc.n1 * gc.hn2;
  MarchOff at = march_off(gf, p.i0, p.i1);
  const unsigned rw = p.j * gf.hn2 + p.m0;
  // coarse row J at in-row index K / 2 (K = m0 is even): the same place in both colour planes
  const unsigned cw = (unsigned)((p.j >> 1) * gc.hn2 + (p.m0 >> 1)) * sizeof(T);
  const MarchEdge e = march_edge<THIN>(gf, p, BX, BY, [&](int q) { tile[0][q] = tile[1][q] = T(0); });
  const unsigned eoff = (unsigned)(e.jr * gf.hn2 + e.mr) * sizeof(T), coff = (unsigned)(p.j * gf.hn2 + e.mc) * sizeof(T),
                 toff = (unsigned)(p.j * gf.hn2 + e.mt) * sizeof(T);
  const T ih2 = (T)(1.0 / gf.h2);
  // number of neighbours inside the grid, for the parities of even (i0) and odd planes
  const int s0 = p.j & 1;
  T nt[2][2];
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int u = 0; u < 2; ++u) nt[f][u] = (T)(6 - diag_jk(gf, p.j, 2 * (p.m0 + u) + (f ? 1 - s0 : s0), false, 0));
  const int z0 = gf.bc0 ? 0 : -2, z1 = gf.bc0 ? gf.n0 - 1 : -2;  // planes at a wall of axis 0
  struct Ops {
    V2<T> hr, x, b, w;
    T hc, ht;
  };
  auto fetch = [&](Ops &o) {
    const T *bp = blk + at.nxt;
    o.hr = ld2<T>(bp, eoff);
    o.hc = ldo(bp, coff);
    if (THIN) o.ht = ldo(bp, toff);
    o.x = ld2<T>(red + at.nxt, rw * (unsigned)sizeof(T));
    o.b = ld2<T>(bf + at.nxt, rw * (unsigned)sizeof(TB));
    o.w = ld2<T>(blk + at.win, rw * (unsigned)sizeof(T));
  };
  T acc[2] = {T(0), T(0)};
  // the coarse values of the plane pair that ends at plane i: this row and,
  // from LDS, its partner (written by odd rows, read after the next barrier)
  auto emit = [&](int i) {
    if (p.ty & 1) return;
    const T v0 = (acc[0] + pair[tid + BX][0]) * (T)0.125;
    const T v1 = (acc[1] + pair[tid + BX][1]) * (T)0.125;
    const int I = i >> 1;
    const bool odd = (I + (p.j >> 1)) & 1;  // colour of (I, J, K)
    T *o = bc + I * PC;
    *(T *)((char *)o + cw) = odd ? v1 : v0;
    *(T *)((char *)(o + gc.half) + cw) = odd ? v0 : v1;
  };
  // plane i (f = i & 1): as in k_sweep
  auto step = [&](int i, int f, const V2<T> &wp, const V2<T> &wc, V2<T> &wn, const Ops &o, Ops &on) {
    march_next(at, i);
    fetch(on);
    T *t = tile[f];
    T *trow = t + (p.ty + 1) * W2 + 2 * p.tx;
    trow[1] = wc.x;
    trow[2] = wc.y;
    if (e.rslot >= 0) {
      t[e.rslot] = o.hr.x;
      t[e.rslot + 1] = o.hr.y;
    }
    if (e.cslot >= 0) t[e.cslot] = o.hc;
    if (THIN && e.tslot >= 0) t[e.tslot] = o.ht;
    __syncthreads();
    wn = i == z1 ? V2<T>{T(0), T(0)} : o.w;
    if (f == 0) {
      if (i > p.i0) emit(i - 1);
      acc[0] = acc[1] = T(0);
    }
    const int s = f ? 1 - s0 : s0;
    const bool edge = i == z0 || i == z1;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const T sum = (u ? wp.y : wp.x) + (u ? wn.y : wn.x) + trow[u + 1 - W2] + trow[u + 1 + W2] + trow[u + s] +
                    trow[u + 1 + s];
      const T nn = edge ? nt[f][u] - T(1) : nt[f][u];
      acc[u] += pc_resid(u ? o.b.y : o.b.x, u ? o.x.y : o.x.x, sum, nn, ih2);
    }
    if (f == 1 && (p.ty & 1)) {
      pair[tid][0] = acc[0];
      pair[tid][1] = acc[1];
    }
  };
  V2<T> w0 = ld2<T>(blk + march_prev(gf, at, p.i0), rw * (unsigned)sizeof(T));
  V2<T> w1 = ld2<T>(blk + at.cur, rw * (unsigned)sizeof(T)), w2, w3;
  Ops oa, ob;
  fetch(oa);
  if (p.i0 == z0) w0 = V2<T>{T(0), T(0)};
  for (int i = p.i0;;) {  // i0 and i1 are even
    step(i, 0, w0, w1, w2, oa, ob);
    step(i + 1, 1, w1, w2, w3, ob, oa);
    if ((i += 2) >= p.i1) break;
    step(i, 0, w2, w3, w0, oa, ob);
    step(i + 1, 1, w3, w0, w1, ob, oa);
    if ((i += 2) >= p.i1) break;
  }
  __syncthreads();
  emit(p.i1 - 1);
}

// x_f += P x_c on the red fine cells only (the following black half sweep
// overwrites the black cells without reading them).  P is trilinear
// cell-centred interpolation: per axis weight 3/4 on the parent and 1/4 on
// the parent's neighbour on the child's side (past a wall the parent itself,
// periodic axes wrap).
//
// Plane march over the fine grid: a thread owns the red cells at in-row
// m0, m0+1 of fine row (i, j).  A coarse plane serves four fine planes, two of
// each parity; its blend over axes 2 and 1 is formed once per parity when the
// plane enters the march (plane_blend: from rows J (parent) and Jo at the four
// coarse K = m0-1 .. m0+2) and kept, so that a fine plane takes one blend of
// two kept values per cell.  The next coarse plane and the fine rows of the
// next pair of planes are loaded before a pair is computed.
template <typename T>
__global__ void __launch_bounds__(256) k_prolong(Geo gf, T *xf, Geo gc, const T *xc) {
  const int BX = blockDim.x, BY = blockDim.y;
  const int m0 = 2 * (blockIdx.x * BX + threadIdx.x), j = blockIdx.y * BY + threadIdx.y;
  const int len = gf.mch;
  const int i0 = blockIdx.z * len, i1 = min(i0 + len, gf.n0);
  const int J = j >> 1, Jn = J + ((j & 1) ? 1 : -1), Jw = mwrap(Jn, gc.n1, gc.bc1);
  const int rows[2] = {J, Jw < 0 ? J : Jw};  // past a wall the parent itself
  int Kq[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int K = m0 - 1 + q, Kw = mwrap(K, gc.n2, gc.bc2);
    Kq[q] = Kw >= 0 ? Kw : (K < 0 ? 0 : gc.n2 - 1);
  }
  // byte offsets of the eight coarse values within an even plane; on an odd
  // plane the other colour holds the cell
  long long off[2][2][4];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = (rows[r] + Kq[q]) & 1;
      const long long e = (long long)rows[r] * gc.hn2 + (Kq[q] >> 1);
      off[0][r][q] = (e + c * gc.half) * (long long)sizeof(T);
      off[1][r][q] = (e + (1 - c) * gc.half) * (long long)sizeof(T);
    }
  struct Raw {
    T v[2][4];
  };
  auto load_plane = [&](int I) {
    Raw w;
    const int Iw = mwrap(I, gc.n0, gc.bc0), P = Iw >= 0 ? Iw : (I < 0 ? 0 : gc.n0 - 1);
    const char *base = (const char *)(xc + (long long)P * gc.n1 * gc.hn2);
    if (P & 1) {
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) w.v[r][q] = *(const T *)(base + off[1][r][q]);
    } else {
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) w.v[r][q] = *(const T *)(base + off[0][r][q]);
    }
    return w;
  };
  // fine red cells at plane i: k = 2 (m0 + u) + s, s = (i + j) & 1; parent
  // K = m0 + u (slot u + 1), neighbour K - 1 (slot u, s = 0) or K + 1 (slot u + 2)
  struct Blend {
    T even[2], odd[2];  // at even and odd fine planes
  };
  auto plane_blend = [&](const Raw &w) {
    Blend z;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const T lo = blend34(blend34(w.v[0][u + 1], w.v[0][u]), blend34(w.v[1][u + 1], w.v[1][u]));
      const T hi = blend34(blend34(w.v[0][u + 1], w.v[0][u + 2]), blend34(w.v[1][u + 1], w.v[1][u + 2]));
      z.even[u] = (j & 1) ? hi : lo;
      z.odd[u] = (j & 1) ? lo : hi;
    }
    return z;
  };
  const long long P = (long long)gf.n1 * gf.hn2;
  const unsigned rw = (unsigned)(j * gf.hn2 + m0) * sizeof(T);
  auto xload = [&](int i) { return ld2<T>(xf + i * P, rw); };
  // fine plane i between the coarse planes lo and hi; the parent is hi for even i
  auto even = [&](int i, const V2<T> &xv, const Blend &lo, const Blend &hi) {
    st2<T>(xf + i * P, rw, xv.x + fma(T(0.75), hi.even[0], T(0.25) * lo.even[0]),
           xv.y + fma(T(0.75), hi.even[1], T(0.25) * lo.even[1]));
  };
  auto odd = [&](int i, const V2<T> &xv, const Blend &lo, const Blend &hi) {
    st2<T>(xf + i * P, rw, xv.x + fma(T(0.25), hi.odd[0], T(0.75) * lo.odd[0]),
           xv.y + fma(T(0.25), hi.odd[1], T(0.75) * lo.odd[1]));
  };
  int i = i0, I = (i0 - 1) >> 1;  // the fine plane i lies between the coarse planes I and I + 1
  V2<T> x0 = xload(i0), x1 = x0;
  const Raw ra = load_plane(I), rb = load_plane(I + 1);
  Blend lo = plane_blend(ra), hi = plane_blend(rb);
  if (i & 1) {
    odd(i, x0, lo, hi);
    if (++i >= i1) return;
    x0 = xload(i);
  }
  if (i + 1 < i1) x1 = xload(i + 1);
  Raw rn = load_plane(I + 2);
  for (;;) {  // i even, between lo and hi; i + 1 lies between hi and plane I + 2
    const V2<T> c0 = x0, c1 = x1;
    const Blend nw = plane_blend(rn);
    const bool two = i + 1 < i1;
    if (i + 2 < i1) {
      x0 = xload(i + 2);
      if (i + 3 < i1) {
        x1 = xload(i + 3);
        rn = load_plane(I + 3);
      }
    }
    even(i, c0, lo, hi);
    if (two) odd(i + 1, c1, hi, nw);
    if ((i += 2) >= i1) return;
    ++I;
    lo = hi;
    hi = nw;
  }
}

// The first black half sweep from x = 0 and the red one after it in one pass:
// from the right-hand side alone, only the red values are stored (the next
// half sweep forms the black ones anew from them).  The two SW_FIRST1 and
// SW_POISSON passes it replaces write the black values and read them and half
// of the right-hand side back: 201 MB at 256^3 in float32 against 101 MB.
//
// A workgroup owns whole rows (no halo along axis 2) of which the first and
// last are a halo whose black values it computes but whose red ones it does not
// store (the first red values of the row beyond are formed by those threads from
// a load of their own), and marches over a
// chunk of planes with the black values one plane ahead of the red ones: at
// plane k it forms black(k) from the first red values r0(k - 1 .. k + 1) and
// red(k - 1) from black(k - 2 .. k); neighbours along axis 0 are in registers,
// the others in LDS (two buffers, one barrier per plane).  A cell outside a
// wall box has a reciprocal count of 0 and so stays 0.
//
// Bounded by bytes on a large level: at 384^3 it moves 465 MB of HBM traffic at
// 5.7 TB/s, where 340 MB are what it asks for -- a workgroup of 8 rows stores 6,
// and its first and last row bring one more row each from beyond.  On a level
// that the last-level cache holds, by the latency of a plane's loads (two planes
// ahead) and its barrier with two workgroups of 8 wavefronts on a compute unit.
// float32, before (both passes) and after, us: 128^3 12.5 / 10.1, 256^3 41.2 / 29.9,
// 384^3 136 / 82.
// In float64 its registers leave half the wavefronts or spill (256^3: 76.7
// before, 75.6 one plane ahead, 192 two ahead), so that form keeps two passes.
// With a float64 right-hand side the float32 form holds it two planes ahead only
// with spills, which pay in workgroups of more than 512 threads: a cycle with this
// pass less one with the two separate ones, one and two planes ahead, us:
// 256 x 256 x 64 -0.8 / +1.7, 256^3 -5.9 / -4.3, rows of 384 -4.3 / -23.9, of 512
// -22.7 / -44.0.
// Chunks of 16 planes in one and a third rounds of workgroups took 34.4 us at
// 256^3, and neighbouring row tiles on one XCD no less than spread ones.
struct First2Shape {
  int bx, rows, chunk;
  dim3 grid;
};
constexpr int FIRST2_WAVES = 16;  // wavefronts on a compute unit (its registers)
// Whole rows of at most 256 entries per colour, and enough rows that a
// workgroup's wrap at most once.
bool mg_first2_fits(const Geo &g) {
  return g.hn2 % 2 == 0 && g.hn2 <= 256 && g.n1 >= 16 && g.n0 >= 4 && g.half < (1LL << 31);  // 32-bit byte offsets on the coarse grid
}
// pairs: a workgroup's stored rows and planes are whole pairs
static First2Shape first2_shape(const Geo &g, bool pairs) {
  First2Shape s;
  s.bx = g.hn2 / 2;
  s.rows = 512 / s.bx;
  if (s.rows < 8) s.rows = 8;
  if (s.rows > 16) s.rows = 16;
  if (pairs) s.rows &= ~1;
  const int ty = (g.n1 + s.rows - 3) / (s.rows - 2);
  // one round of workgroups on the 256 compute units, if that leaves them a
  // few planes each: the planes before and after a chunk are computed again
  // (the wavefronts of a workgroup go round the four SIMDs, so five take the
  // room of eight: 256 x 256 x 80 cells with 15 wavefronts on a compute unit
  // counted on 98.5 us a cycle, with 10 82.0; the passes one by one 91.6)
  int waves = (s.bx * s.rows + 63) / 64;
  if (waves > 4) waves = (waves + 3) & ~3;
  const int slots = 256 * (FIRST2_WAVES / waves), nch = slots / ty > 0 ? slots / ty : 1;
  s.chunk = (g.n0 + nch - 1) / nch;
  if (s.chunk < 2) s.chunk = 2;
  if (pairs) s.chunk = (s.chunk + 1) & ~1;
  s.grid = dim3(ty, (g.n0 + s.chunk - 1) / s.chunk);
  return s;
}

template <typename T, typename TB, int NT>
__global__ void __launch_bounds__(NT, 4) k_first2(Geo g, T *x, const TB *b, double h2, int chunk) {
  // planes that operands are loaded ahead of their use
  constexpr int AH = sizeof(TB) == 4 || NT > 512 ? 2 : 1;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int BX = blockDim.x, rows = blockDim.y, W = g.hn2 + 2, TS = rows * W;
  T *lds = (T *)lds_raw;  // [buffer][red, black][rows][W]
  const int mz = blockIdx.y;
  const int tx = threadIdx.x, ty = threadIdx.y, m0 = 2 * tx;
  const int j0 = blockIdx.x * (rows - 2), ju = j0 - 1 + ty, jw = mwrap(ju, g.n1, g.bc1);
  const bool in = jw >= 0 && jw < g.n1;  // a row far past the last one wraps no more: unused
  const int j = in ? jw : 0;
  const bool store = ty > 0 && ty < rows - 1 && ju < g.n1;
  const int i0 = mz * chunk, i1 = min(i0 + chunk, g.n0);
  const long long P = (long long)g.n1 * g.hn2;
  const unsigned rw = j * g.hn2 + m0;
  const T th2 = (T)h2;
  const TB *br = b, *bk = b + g.half;
  // reciprocal counts of the thread's cells by parity of k, inside the grid
  const int s0 = (i0 + ju) & 1;  // parity of the red cells at plane i0
  T inv[2][2];
  unsigned pk = 0;
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int dg = diag_jk(g, j, 2 * (m0 + u) + (f ? 1 - s0 : s0), false, 0);
      pk |= (unsigned)dg << (8 * f + 4 * u);
      inv[f][u] = in ? inv_nn<T>(6 - dg) : T(0);
    }
  // the row beyond the halo rows, whose red cells have the parity of the own black ones
  const int jeu = ty == 0 ? ju - 1 : (ty == rows - 1 ? ju + 1 : ju), jew = mwrap(jeu, g.n1, g.bc1);
  const bool ein = jew >= 0 && jew < g.n1;
  const int je = ein ? jew : 0;
  const unsigned ew = je * g.hn2 + m0;
  T inve[2][2];
  unsigned pke = 0;
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int dg = diag_jk(g, je, 2 * (m0 + u) + (f ? 1 - s0 : s0), false, 0);
      pke |= (unsigned)dg << (8 * f + 4 * u);
      inve[f][u] = ein ? inv_nn<T>(6 - dg) : T(0);
    }
  // counts of parity index f at plane i: as tabulated, one less at a wall of
  // axis 0, 0 outside (near, known to the compiler: the plane may be such)
  auto counts = [&](auto near, int i, int f, const T (&tab)[2][2], unsigned packed, bool inside, T (&c)[2]) {
    c[0] = tab[f][0];
    c[1] = tab[f][1];
    if (decltype(near)::value && g.bc0 && (i <= 0 || i >= g.n0 - 1)) {
      const bool out = !inside || i < 0 || i >= g.n0;
      c[0] = out ? T(0) : inv_nn<T>(5 - (int)((packed >> (8 * f)) & 15));
      c[1] = out ? T(0) : inv_nn<T>(5 - (int)((packed >> (8 * f + 4)) & 15));
    }
  };
  auto count = [&](auto near, int i, int f, T (&c)[2]) { counts(near, i, f, inv, pk, in, c); };
  auto plane = [&](int i) {  // a plane's offset; past a wall the nearest plane, whose counts are 0
    if (i < 0) i = g.bc0 ? 0 : i + g.n0;
    if (i >= g.n0) i = g.bc0 ? g.n0 - 1 : i - g.n0;
    return i * P;
  };
  auto ldr = [&](long long o) { return ld2<T>(br + o, rw * (unsigned)sizeof(TB)); };
  auto lde = [&](long long o) { return ld2<T>(br + o, ew * (unsigned)sizeof(TB)); };
  auto ldk = [&](long long o) { return ld2<T>(bk + o, rw * (unsigned)sizeof(TB)); };
  // offsets of the planes k + AH and k + AH + 1, and of k, advanced by addition
  long long o2 = plane(i0 - 1 + AH), o3 = plane(i0 + AH), ok = (i0 - 2) * P;
  auto first = [&](V2<T> v, const T (&c)[2]) { return V2<T>{pc_first(th2, v.x, c[0]), pc_first(th2, v.y, c[1])}; };
  // a pair into an LDS plane, with the row's ends (periodic: the other end)
  auto put = [&](T *t, const V2<T> &v) {
    T *r = t + ty * W + m0;
    r[1] = v.x;
    r[2] = v.y;
    if (tx == 0) t[ty * W + g.hn2 + 1] = g.bc2 ? T(0) : v.x;
    if (tx == BX - 1) t[ty * W] = g.bc2 ? T(0) : v.y;
  };
  const bool first_row = ty == 0, last_row = ty == rows - 1;
  const int up = first_row ? 0 : -W, dn = last_row ? 0 : W;
  // relaxed pair: prev, next along axis 0, the LDS plane t (e in place of the
  // row beyond the halo rows), parity s of its cells
  auto relax = [&](const V2<T> &p, const V2<T> &n, const T *t, const V2<T> &e, int s, const V2<T> &bv, const T (&c)[2]) {
    const T *r = t + ty * W + m0;
    const T ux = first_row ? e.x : r[1 + up], uy = first_row ? e.y : r[2 + up];
    const T dx = last_row ? e.x : r[1 + dn], dy = last_row ? e.y : r[2 + dn];
    const T sx = p.x + n.x + ux + dx + r[s] + r[1 + s];
    const T sy = p.y + n.y + uy + dy + r[1 + s] + r[2 + s];
    return V2<T>{pc_relax(th2, bv.x, sx, c[0]), pc_relax(th2, bv.y, sy, c[1])};
  };
  // Plane k (parity index f of the black cells there, which is that of the red
  // ones at k - 1 and k + 1).  Operands are loaded AH planes before their use
  // (few waves fit a compute unit): q holds b_red of plane k at k & 7, bb and be
  // b_black and the red right-hand side of the row beyond at k & 3; r0 and kk the
  // first red and the black values at k & 3.  All indices are known to the
  // compiler, eight planes per turn, so everything stays in registers.
  V2<T> q[8], bb[4], be[4], r0[4], kk[4];
  auto body = [&](auto near, int k, int u, int f, T *R) {
    T *K = R + TS;
    T c[2], ck[2];
    count(near, k + 1, f, c);
    r0[(u + 1) & 3] = first(q[(u + 1) & 7], c);
    const int s = f ? 1 - s0 : s0;  // parity of the cells of index f
    count(near, k, f, ck);
    counts(near, k, f, inve, pke, ein, c);
    const V2<T> e = first(be[u & 3], c);
    kk[u & 3] = relax(r0[(u + 3) & 3], r0[(u + 1) & 3], R, e, s, bb[u & 3], ck);
    if (k > i0) {
      count(near, k - 1, f, c);
      const V2<T> v = relax(kk[(u + 2) & 3], kk[u & 3], K, e, s, q[(u + 7) & 7], c);
      if (store) st2<T>(x + ok - P, rw * (unsigned)sizeof(T), v.x, v.y);
    }
  };
  auto step = [&](int k, int u, int f) {
    q[(u + AH + 1) & 7] = ldr(o3);
    bb[(u + AH) & 3] = ldk(o2);
    be[(u + AH) & 3] = lde(o2);
    o2 = o3;
    const int nx = k + AH + 2;
    if (nx == (g.bc0 ? 0 : g.n0)) o3 = 0;
    else if (nx > 0 && nx < g.n0 + (g.bc0 ? 0 : 8)) o3 += P;
    ok += P;
    T *R = lds + (f ? 2 * TS : 0);
    put(R, r0[u & 3]);
    put(R + TS, kk[(u + 3) & 3]);
    __syncthreads();
    if (g.bc0 && (k <= 1 || k >= g.n0 - 2)) body(std::true_type{}, k, u, f, R);
    else body(std::false_type{}, k, u, f, R);
  };
  // before the march, which starts at plane i0 - 1 (u = 0; its black values are
  // the first needed): parity index 0 is that of the red cells at i0, so of
  // those at i0 - 2 and of the black ones at i0 - 1
  T c[2];
  const V2<T> qm = ldr(plane(i0 - 2));
  q[0] = ldr(plane(i0 - 1));
  q[1] = ldr(plane(i0));
  bb[0] = ldk(plane(i0 - 1));
  be[0] = lde(plane(i0 - 1));
  if (AH == 2) {
    q[2] = ldr(plane(i0 + 1));
    bb[1] = ldk(plane(i0));
    be[1] = lde(plane(i0));
  }
  kk[2] = kk[3] = V2<T>{T(0), T(0)};
  count(std::true_type{}, i0 - 2, 0, c);
  r0[3] = first(qm, c);
  count(std::true_type{}, i0 - 1, 1, c);
  r0[0] = first(q[0], c);
  for (int k = i0 - 1;;) {
    step(k, 0, 0);
    if (++k > i1) break;
    step(k, 1, 1);
    if (++k > i1) break;
    step(k, 2, 0);
    if (++k > i1) break;
    step(k, 3, 1);
    if (++k > i1) break;
    step(k, 4, 0);
    if (++k > i1) break;
    step(k, 5, 1);
    if (++k > i1) break;
    step(k, 6, 0);
    if (++k > i1) break;
    step(k, 7, 1);
    if (++k > i1) break;
  }
}

// Prolongation and the black half sweep after it in one pass: the red values
// x + P x_c are formed on the way (the arithmetic of k_prolong) and not stored,
// since the red half sweep that follows relaxes them from the black ones.  The
// two passes move 75 + 101 MB at 256^3 in float32, this one 109.
//
// The march of k_first2: whole rows, of which the first and last only serve
// their neighbours; a chunk starts at an even plane, so the parity of the plane
// is that of its place in the unrolled loop, and every second plane brings the
// blend of one more coarse plane.
//
// Bounded as k_first2: 151 MB counted for 109 at 256^3, 6.0 TB/s; 471 for 368 at
// 384^3, 6.4.  Both passes before and this one after, float32, us: 256^3 34.5 / 25.2,
// 384^3 115 / 73, 128^3 10.6 / 10.2.
template <typename T, typename TB, int NT>
__global__ void __launch_bounds__(NT, 4) k_prolong_black(Geo g, T *x, const TB *b, Geo gc, const T *xc, double h2,
                                                         int chunk) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int BX = blockDim.x, rows = blockDim.y, W = g.hn2 + 2, TS = rows * W;
  T *lds = (T *)lds_raw;  // [buffer][rows][W]
  const int tx = threadIdx.x, ty = threadIdx.y, m0 = 2 * tx;
  const int ju = blockIdx.x * (rows - 2) - 1 + ty, jw = mwrap(ju, g.n1, g.bc1);
  const bool in = jw >= 0 && jw < g.n1;
  const int j = in ? jw : 0;
  const bool store = ty > 0 && ty < rows - 1 && ju < g.n1;
  const int i0 = blockIdx.y * chunk, i1 = min(i0 + chunk, g.n0);
  const long long P = (long long)g.n1 * g.hn2, PC = (long long)gc.n1 * gc.hn2;
  const unsigned rw = j * g.hn2 + m0;
  const T th2 = (T)h2;
  const TB *bk = b + g.half;
  T *xk = x + g.half;
  // black cells at plane i0 have parity s0
  const int s0 = (1 + i0 + j) & 1;
  T inv[2][2];
  unsigned pk = 0;
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int dg = diag_jk(g, j, 2 * (m0 + u) + (f ? 1 - s0 : s0), false, 0);
      pk |= (unsigned)dg << (8 * f + 4 * u);
      inv[f][u] = inv_nn<T>(6 - dg);
    }
  // the eight coarse values of a row's pair, as in k_prolong: byte offsets in
  // even and odd coarse planes
  const int J = j >> 1, Jw = mwrap(J + ((j & 1) ? 1 : -1), gc.n1, gc.bc1);
  const int cr[2] = {J, Jw < 0 ? J : Jw};
  unsigned off[2][2][4];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int K = m0 - 1 + q, Kw = mwrap(K, gc.n2, gc.bc2), Kq = Kw >= 0 ? Kw : (K < 0 ? 0 : gc.n2 - 1);
      const long long e = (long long)cr[r] * gc.hn2 + (Kq >> 1);
      const int c = (cr[r] + Kq) & 1;
      off[0][r][q] = (unsigned)((e + c * gc.half) * sizeof(T));
      off[1][r][q] = (unsigned)((e + (1 - c) * gc.half) * sizeof(T));
    }
  struct Raw {
    T v[2][4];
  };
  struct Blend {
    T even[2], odd[2];
  };
  auto load_plane = [&](int I) {
    Raw w;
    const int Iw = mwrap(I, gc.n0, gc.bc0), p = Iw >= 0 ? Iw : (I < 0 ? 0 : gc.n0 - 1);
    const T *base = xc + p * PC;
    const bool odd = p & 1;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) w.v[r][q] = ldo(base, odd ? off[1][r][q] : off[0][r][q]);
    return w;
  };
  auto plane_blend = [&](const Raw &w) {
    Blend z;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const T lo = blend34(blend34(w.v[0][u + 1], w.v[0][u]), blend34(w.v[1][u + 1], w.v[1][u]));
      const T hi = blend34(blend34(w.v[0][u + 1], w.v[0][u + 2]), blend34(w.v[1][u + 1], w.v[1][u + 2]));
      z.even[u] = (j & 1) ? hi : lo;
      z.odd[u] = (j & 1) ? lo : hi;
    }
    return z;
  };
  auto plane = [&](int i) {  // a plane's offset; past a wall the nearest one
    if (i < 0) i = g.bc0 ? 0 : i + g.n0;
    if (i >= g.n0) i = g.bc0 ? g.n0 - 1 : i - g.n0;
    return i * P;
  };
  // red values of plane i between the coarse planes lo and hi; 0 outside the grid
  auto red = [&](int i, auto odd, const V2<T> &xv, const Blend &lo, const Blend &hi) {
    constexpr bool O = decltype(odd)::value;
    const T wl = O ? T(0.75) : T(0.25), wh = O ? T(0.25) : T(0.75);
    const T px = fma(wh, O ? hi.odd[0] : hi.even[0], wl * (O ? lo.odd[0] : lo.even[0]));
    const T py = fma(wh, O ? hi.odd[1] : hi.even[1], wl * (O ? lo.odd[1] : lo.even[1]));
    const bool out = !in || (g.bc0 && (i < 0 || i >= g.n0));
    return V2<T>{out ? T(0) : xv.x + px, out ? T(0) : xv.y + py};
  };
  auto ldx = [&](long long o) { return ld2<T>((const T *)x + o, rw * (unsigned)sizeof(T)); };
  auto ldk = [&](long long o) { return ld2<T>(bk + o, rw * (unsigned)sizeof(TB)); };
  auto put = [&](T *t, const V2<T> &v) {
    T *r = t + ty * W + m0;
    r[1] = v.x;
    r[2] = v.y;
    if (tx == 0) t[ty * W + g.hn2 + 1] = g.bc2 ? T(0) : v.x;
    if (tx == BX - 1) t[ty * W] = g.bc2 ? T(0) : v.y;
  };
  const int up = ty == 0 ? 0 : -W, dn = ty == rows - 1 ? 0 : W;  // beyond the first and last row: not used
  // plane k at place u: r(k + 1) from xr(k + 1), loaded two planes ago, then the
  // black values from r(k - 1 .. k + 1); all indices known to the compiler
  V2<T> r[4], xr[4], bb[4];
  Blend bl[4];
  Raw raw;
  long long o2 = plane(i0 + 2), o3 = plane(i0 + 3), ok = (i0 - 1) * P;
  auto step = [&](int k, int u, int f, auto odd) {
    xr[(u + 3) & 3] = ldx(o3);
    bb[(u + 2) & 3] = ldk(o2);
    o2 = o3;
    const int nx = k + 4;
    if (nx == (g.bc0 ? 0 : g.n0)) o3 = 0;
    else if (nx < g.n0 + (g.bc0 ? 0 : 8)) o3 += P;
    ok += P;
    T *t = lds + (f ? TS : 0);
    put(t, r[u & 3]);
    __syncthreads();
    if (!f) {  // k even: k + 1 lies between the coarse planes k / 2 and k / 2 + 1
      bl[(u / 2 + 1) & 3] = plane_blend(raw);
      raw = load_plane(k / 2 + 2);
    }
    r[(u + 1) & 3] = red(k + 1, odd, xr[(u + 1) & 3], bl[(u / 2) & 3], bl[(u / 2 + 1) & 3]);
    const V2<T> &p = r[(u + 3) & 3], &n = r[(u + 1) & 3];
    T c0 = inv[f][0], c1 = inv[f][1];
    if (g.bc0 && (k == 0 || k == g.n0 - 1)) {
      c0 = inv_nn<T>(5 - (int)((pk >> (8 * f)) & 15));
      c1 = inv_nn<T>(5 - (int)((pk >> (8 * f + 4)) & 15));
    }
    const int s = f ? 1 - s0 : s0;
    const T *q = t + ty * W + m0;
    const T sx = p.x + n.x + q[1 + up] + q[1 + dn] + q[s] + q[1 + s];
    const T sy = p.y + n.y + q[2 + up] + q[2 + dn] + q[1 + s] + q[2 + s];
    if (store)
      st2<T>(xk + ok, rw * (unsigned)sizeof(T), pc_relax(th2, bb[u & 3].x, sx, c0), pc_relax(th2, bb[u & 3].y, sy, c1));
  };
  {
    const int I = i0 / 2;
    const Raw ra = load_plane(I - 1), rb = load_plane(I);
    const V2<T> xm = ldx(plane(i0 - 1)), x0 = ldx(plane(i0));
    xr[1] = ldx(plane(i0 + 1));
    bb[0] = ldk(plane(i0));
    raw = load_plane(I + 1);
    xr[2] = ldx(o2);
    bb[1] = ldk(plane(i0 + 1));
    const Blend lo = plane_blend(ra);
    bl[0] = plane_blend(rb);
    r[3] = red(i0 - 1, std::true_type{}, xm, lo, bl[0]);
    r[0] = red(i0, std::false_type{}, x0, lo, bl[0]);
  }
  for (int k = i0;;) {
    step(k, 0, 0, std::true_type{});
    if (++k >= i1) break;
    step(k, 1, 1, std::false_type{});
    if (++k >= i1) break;
    step(k, 2, 0, std::true_type{});
    if (++k >= i1) break;
    step(k, 3, 1, std::false_type{});
    if (++k >= i1) break;
    step(k, 4, 0, std::true_type{});
    if (++k >= i1) break;
    step(k, 5, 1, std::false_type{});
    if (++k >= i1) break;
    step(k, 6, 0, std::true_type{});
    if (++k >= i1) break;
    step(k, 7, 1, std::false_type{});
    if (++k >= i1) break;
  }
}

// The last black half sweep of the descent and the restriction in one pass: the
// black values feed the red residuals and are not stored, since the ascent
// relaxes them anew from the red ones.  The two passes move 101 + 109 MB at
// 256^3 in float32, this one 109.
//
// The march of k_first2 with the red values loaded: at plane k it forms
// black(k), then the residuals of the red cells at k - 1, summed over pairs of
// planes and, through LDS, pairs of rows (a workgroup stores whole pairs: its
// stored rows and its chunk start at even places and are even in number, which
// takes a row off a workgroup of 9, 11, 13 or 15).
//
// Bounded as k_first2, and it reads most of all, three arrays with their halo rows:
// 180 MB counted for 109 at 256^3, 5.8 TB/s; 535 for 368 at 384^3, 6.1.  Both
// passes before and this one after, float32, us: 256^3 39.3 / 31.2, 384^3 141 / 88,
// 128^3 10.2 / 10.3.
template <typename T, typename TB, int NT>
__global__ void __launch_bounds__(NT, 4) k_black_restrict(Geo g, const T *x, const TB *b, Geo gc, T *bc, double h2,
                                                          int chunk) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int BX = blockDim.x, rows = blockDim.y, W = g.hn2 + 2, TS = rows * W;
  T *lds = (T *)lds_raw;        // [buffer][red, black][rows][W]
  T *pair = lds + 4 * TS;       // [rows][BX][2]
  const int tx = threadIdx.x, ty = threadIdx.y, m0 = 2 * tx;
  const int ju = blockIdx.x * (rows - 2) - 1 + ty, jw = mwrap(ju, g.n1, g.bc1);
  const bool in = jw >= 0 && jw < g.n1;
  const int j = in ? jw : 0;
  const bool store = ty > 0 && ty < rows - 1 && ju < g.n1;
  const int i0 = blockIdx.y * chunk, i1 = min(i0 + chunk, g.n0);
  const long long P = (long long)g.n1 * g.hn2, PC = (long long)gc.n1 * gc.hn2;
  const unsigned rw = j * g.hn2 + m0, cw = (unsigned)((j >> 1) * gc.hn2 + (m0 >> 1)) * sizeof(T);
  const T th2 = (T)h2, ih2 = (T)(1.0 / g.h2);
  const TB *bk = b + g.half;
  const int s0 = (i0 + j) & 1;  // parity of the red cells at plane i0
  // by parity of k: reciprocal counts (0 outside the grid) and counts
  T inv[2][2], nn[2][2];
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int dg = diag_jk(g, j, 2 * (m0 + u) + (f ? 1 - s0 : s0), false, 0);
      inv[f][u] = in ? inv_nn<T>(6 - dg) : T(0);
      nn[f][u] = (T)(6 - dg);
    }
  // the row beyond a halo row
  const int jeu = ty == 0 ? ju - 1 : (ty == rows - 1 ? ju + 1 : ju), jew = mwrap(jeu, g.n1, g.bc1);
  const bool ein = jew >= 0 && jew < g.n1;
  const unsigned ew = (ein ? jew : 0) * g.hn2 + m0;
  auto plane = [&](int i) {  // a plane's offset; past a wall the nearest one
    if (i < 0) i = g.bc0 ? 0 : i + g.n0;
    if (i >= g.n0) i = g.bc0 ? g.n0 - 1 : i - g.n0;
    return i * P;
  };
  auto outside = [&](int i) { return g.bc0 && (i < 0 || i >= g.n0); };
  auto ldx = [&](long long o) { return ld2<T>(x + o, rw * (unsigned)sizeof(T)); };
  auto lde = [&](long long o) { return ld2<T>(x + o, ew * (unsigned)sizeof(T)); };
  auto ldr = [&](long long o) { return ld2<T>(b + o, rw * (unsigned)sizeof(TB)); };
  auto ldk = [&](long long o) { return ld2<T>(bk + o, rw * (unsigned)sizeof(TB)); };
  auto put = [&](T *t, const V2<T> &v) {
    T *r = t + ty * W + m0;
    r[1] = v.x;
    r[2] = v.y;
    if (tx == 0) t[ty * W + g.hn2 + 1] = g.bc2 ? T(0) : v.x;
    if (tx == BX - 1) t[ty * W] = g.bc2 ? T(0) : v.y;
  };
  const bool first_row = ty == 0, last_row = ty == rows - 1;
  const int up = first_row ? 0 : -W, dn = last_row ? 0 : W;
  auto sums = [&](const V2<T> &p, const V2<T> &n, const T *t, const V2<T> &e, int s) {
    const T *r = t + ty * W + m0;
    const T ux = first_row ? e.x : r[1 + up], uy = first_row ? e.y : r[2 + up];
    const T dx = last_row ? e.x : r[1 + dn], dy = last_row ? e.y : r[2 + dn];
    return V2<T>{p.x + n.x + ux + dx + r[s] + r[1 + s], p.y + n.y + uy + dy + r[1 + s] + r[2 + s]};
  };
  // as in k_first2; xr: red values of plane k at k & 7, br: b_red of plane k - 1
  // and bb, be: b_black and the row beyond of plane k, all at k & 3
  V2<T> xr[8], br[4], bb[4], be[4], kk[4];
  T acc[2] = {T(0), T(0)};
  long long o1 = plane(i0), o2 = plane(i0 + 1), o3 = plane(i0 + 2);
  // the coarse values of the plane pair that ends at plane i: rows of even place
  // (odd ty) add their partner's sums
  auto emit = [&](int i) {
    if (!store || !(ty & 1)) return;
    const T *q = pair + ((ty + 1) * BX + tx) * 2;
    const T v0 = (acc[0] + q[0]) * (T)0.125, v1 = (acc[1] + q[1]) * (T)0.125;
    const int I = i >> 1;
    const bool odd = (I + (j >> 1)) & 1;  // colour of (I, J, K)
    T *o = bc + I * PC;
    *(T *)((char *)o + cw) = odd ? v1 : v0;
    *(T *)((char *)(o + gc.half) + cw) = odd ? v0 : v1;
  };
  // k = i0 - 1 + u (mod 8); f: parity index of the black cells at k, and the buffer
  auto step = [&](int k, int u, int f) {
    xr[(u + 3) & 7] = ldx(o3);
    bb[(u + 2) & 3] = ldk(o2);
    be[(u + 2) & 3] = lde(o2);
    br[(u + 2) & 3] = ldr(o1);
    o1 = o2;
    o2 = o3;
    const int nx = k + 4;
    if (nx == (g.bc0 ? 0 : g.n0)) o3 = 0;
    else if (nx > 0 && nx < g.n0 + (g.bc0 ? 0 : 8)) o3 += P;
    T *R = lds + (f ? 2 * TS : 0), *K = R + TS;
    V2<T> &xn = xr[(u + 1) & 7];
    if (outside(k + 1) || !in) xn = V2<T>{T(0), T(0)};
    put(R, xr[u & 7]);
    put(K, kk[(u + 3) & 3]);
    __syncthreads();
    const int s = f ? 1 - s0 : s0;
    if (!f) {  // plane k - 1 is even and starts a pair; the one that ended at k - 2 has its partners' sums in LDS
      if (k > i0 + 1) emit(k - 2);
      acc[0] = acc[1] = T(0);
    }
    V2<T> e = be[u & 3];
    if (!ein || outside(k)) e = V2<T>{T(0), T(0)};
    T c0 = inv[f][0], c1 = inv[f][1];
    if (g.bc0 && (k <= 0 || k >= g.n0 - 1)) {
      const bool out = !in || outside(k);
      c0 = out ? T(0) : inv_nn<T>((int)nn[f][0] - 1);
      c1 = out ? T(0) : inv_nn<T>((int)nn[f][1] - 1);
    }
    const V2<T> sb = sums(xr[(u + 7) & 7], xn, R, e, s);
    kk[u & 3] = V2<T>{pc_relax(th2, bb[u & 3].x, sb.x, c0), pc_relax(th2, bb[u & 3].y, sb.y, c1)};
    if (k > i0) {
      const V2<T> sr = sums(kk[(u + 2) & 3], kk[u & 3], K, e, s), xv = xr[(u + 7) & 7], bv = br[u & 3];
      const bool wall = g.bc0 && (k - 1 == 0 || k == g.n0);
      const T n0 = wall ? nn[f][0] - T(1) : nn[f][0], n1 = wall ? nn[f][1] - T(1) : nn[f][1];
      acc[0] += pc_resid(bv.x, xv.x, sr.x, n0, ih2);
      acc[1] += pc_resid(bv.y, xv.y, sr.y, n1, ih2);
      if (f && store && !(ty & 1)) {  // plane k - 1 ends a pair
        T *q = pair + (ty * BX + tx) * 2;
        q[0] = acc[0];
        q[1] = acc[1];
      }
    }
  };
  // before the march, which starts at plane i0 - 1 (u = 0, black parity index 0)
  {
    V2<T> xm = ldx(plane(i0 - 2)), xc = ldx(plane(i0 - 1));
    xr[1] = ldx(plane(i0));
    bb[0] = ldk(plane(i0 - 1));
    be[0] = lde(plane(i0 - 1));
    br[0] = ldr(plane(i0 - 2));
    xr[2] = ldx(plane(i0 + 1));
    bb[1] = ldk(plane(i0));
    be[1] = lde(plane(i0));
    br[1] = ldr(plane(i0 - 1));
    if (outside(i0 - 2) || !in) xm = V2<T>{T(0), T(0)};
    if (outside(i0 - 1) || !in) xc = V2<T>{T(0), T(0)};
    xr[7] = xm;
    xr[0] = xc;
    kk[2] = kk[3] = V2<T>{T(0), T(0)};
  }
  for (int k = i0 - 1;;) {
    step(k, 0, 0);
    if (++k > i1) break;
    step(k, 1, 1);
    if (++k > i1) break;
    step(k, 2, 0);
    if (++k > i1) break;
    step(k, 3, 1);
    if (++k > i1) break;
    step(k, 4, 0);
    if (++k > i1) break;
    step(k, 5, 1);
    if (++k > i1) break;
    step(k, 6, 0);
    if (++k > i1) break;
    step(k, 7, 1);
    if (++k > i1) break;
  }
  __syncthreads();
  emit(i1 - 1);
}

template <typename TB>
hipError_t mg_smooth_first2(const Geo &g, float *x, const TB *b, hipStream_t s) {
  if (!mg_first2_fits(g)) return hipErrorInvalidValue;
  const First2Shape f = first2_shape(g, false);
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
  const size_t lds = 4 * sizeof(float) * f.rows * (g.hn2 + 2);
  const dim3 block(f.bx, f.rows);
  if (f.bx * f.rows <= 512)
    hipExtLaunchKernelGGL((k_first2<float, TB, 512>), f.grid, block, lds, s, e0, e1, 0, g, x, b, g.h2, f.chunk);
  else
    hipExtLaunchKernelGGL((k_first2<float, TB, 1024>), f.grid, block, lds, s, e0, e1, 0, g, x, b, g.h2, f.chunk);
  return hipGetLastError();
}
template <typename TB>
hipError_t mg_prolong_black(const Geo &g, float *x, const TB *b, const Geo &gc, const float *xc, hipStream_t s) {
  if (!mg_first2_fits(g)) return hipErrorInvalidValue;
  First2Shape f = first2_shape(g, false);
  f.chunk = (f.chunk + 1) & ~1;  // chunks start at even planes
  f.grid.y = (g.n0 + f.chunk - 1) / f.chunk;
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
  const size_t lds = 2 * sizeof(float) * f.rows * (g.hn2 + 2);
  const dim3 block(f.bx, f.rows);
  if (f.bx * f.rows <= 512)
    hipExtLaunchKernelGGL((k_prolong_black<float, TB, 512>), f.grid, block, lds, s, e0, e1, 0, g, x, b, gc, xc, g.h2,
                          f.chunk);
  else
    hipExtLaunchKernelGGL((k_prolong_black<float, TB, 1024>), f.grid, block, lds, s, e0, e1, 0, g, x, b, gc, xc, g.h2,
                          f.chunk);
  return hipGetLastError();
}
template hipError_t mg_prolong_black<float>(const Geo &, float *, const float *, const Geo &, const float *, hipStream_t);
template hipError_t mg_prolong_black<double>(const Geo &, float *, const double *, const Geo &, const float *, hipStream_t);
template <typename TB>
hipError_t mg_black_restrict(const Geo &g, const float *x, const TB *b, const Geo &gc, float *bc, hipStream_t s) {
  if (!mg_first2_fits(g)) return hipErrorInvalidValue;
  const First2Shape f = first2_shape(g, true);
  // pairs of planes and rows stay inside one workgroup
  if (g.n0 % 2 || g.n1 % 2 || f.rows % 2 || f.chunk % 2) return hipErrorInvalidValue;
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
  const size_t lds = sizeof(float) * f.rows * (4 * (g.hn2 + 2) + 2 * f.bx);
  const dim3 block(f.bx, f.rows);
  if (f.bx * f.rows <= 512)
    hipExtLaunchKernelGGL((k_black_restrict<float, TB, 512>), f.grid, block, lds, s, e0, e1, 0, g, x, b, gc, bc, g.h2,
                          f.chunk);
  else
    hipExtLaunchKernelGGL((k_black_restrict<float, TB, 1024>), f.grid, block, lds, s, e0, e1, 0, g, x, b, gc, bc, g.h2,
                          f.chunk);
  return hipGetLastError();
}
template hipError_t mg_black_restrict<float>(const Geo &, const float *, const float *, const Geo &, float *, hipStream_t);
template hipError_t mg_black_restrict<double>(const Geo &, const float *, const double *, const Geo &, float *, hipStream_t);
template hipError_t mg_smooth_first2<float>(const Geo &, float *, const float *, hipStream_t);
template hipError_t mg_smooth_first2<double>(const Geo &, float *, const double *, hipStream_t);

template <typename T, typename TB>
hipError_t mg_smooth_first(const Geo &g, T *x, const TB *b, bool store_red, hipStream_t s) {
  MarchShape M = march_shape(g, 1);
  // launched with the events of an enclosing ProbeExt, if any (as the three below)
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
  if (store_red) return sweep_launch<T, TB, SW_FIRST>(M, g, x, b, 1, 0.0, 0.0, 1.0, s, e0, e1);
  return sweep_launch<T, TB, SW_FIRST1>(M, g, x, b, 1, 0.0, 0.0, 1.0, s, e0, e1);
}
template <typename T, typename TB>
hipError_t mg_smooth(const Geo &g, T *x, const TB *b, int color, hipStream_t s) {
  MarchShape M = march_shape(g, 1);
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
  return sweep_launch<T, TB, SW_POISSON>(M, g, x, b, color, 0.0, 0.0, 1.0, s, e0, e1);
}

template <typename T, typename TB>
hipError_t mg_restrict(const Geo &gf, const T *xf, const TB *bf, const Geo &gc, T *bc, hipStream_t s) {
  MarchShape M = march_shape(gf, 1);
  const int len = restrict_chunk(gf);
  M.grid.z = (gf.n0 + len - 1) / len;
  // pairs of planes and rows stay inside one workgroup
  if (gf.n0 % 2 || M.block.y % 2 || len % 2) return hipErrorInvalidValue;
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
  if (M.bx == 1)
    hipExtLaunchKernelGGL((k_restrict<T, TB, true>), M.grid, M.block, 0, s, e0, e1, 0, gf, xf, bf, gc, bc);
  else
    hipExtLaunchKernelGGL((k_restrict<T, TB, false>), M.grid, M.block, 0, s, e0, e1, 0, gf, xf, bf, gc, bc);
  return hipGetLastError();
}
template <typename T>
hipError_t mg_prolong(const Geo &gf, T *xf, const Geo &gc, const T *xc, hipStream_t s) {
  MarchShape M = march_shape(gf, 1);
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
  hipExtLaunchKernelGGL(k_prolong<T>, M.grid, M.block, 0, s, e0, e1, 0, gf, xf, gc, xc);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Tile levels.  On the small levels of the cycle a launch costs more than the
// work it carries (a few microseconds whatever the grid), and the march
// kernels above spend seven launches per level.  A tile level takes two: one
// workgroup per 8^3 tile loads its tile with a halo into LDS and runs the
// tile's whole descent (pre-smoothing, residual, restriction: k_tile_down) or
// whole ascent (prolongation, post-smoothing: k_tile_up), recomputing the
// halo cells that neighbouring tiles own.  A half sweep is exact on a box one
// cell smaller on every side than the box whose values it reads, so the box
// shrinks by one cell per half sweep and a halo of two cells per sweep
// suffices.  Every cell takes the operations of k_sweep, k_restrict and
// k_prolong in the same order (pc_first, pc_relax, pc_resid, blend34), so a
// tile level gives the bits of the march kernels.
//
// Region coordinates r of a tile at grid origin o with halo H stand for the
// unwrapped grid coordinate u = o - H + r.  A wall axis has no cells outside
// [0, n) (their LDS slots hold 0, which a neighbour sum then adds as the
// missing neighbour); a periodic axis wraps.  Origins and halos are even and n
// is even, so the colour of a cell is the parity of r0 + r1 + r2.
//
// Layout.  The region holds each colour by itself, row by row like the grid:
// (r0, r1) a row of 8 entries per colour, cells r2 = 2 m + parity.  Along axis
// 2 the halo is 4 whatever the sweeps, which puts every pair of entries on an
// even in-row index of the grid.  A thread owns half a row, 4 entries of both
// colours, for the whole kernel: their right-hand sides, values and reciprocal
// neighbour counts (0 for a cell outside the grid) stay in registers, and
// from LDS it reads four vectors and one value per half sweep, on consecutive
// addresses for consecutive threads.  No cell is tested: what the rows' ends
// hold beyond the halo's reach is wrong but never used.
//
// Bounded by latency where the tiles are fewer than the compute units (32^3),
// else by vector instructions and LDS.  Against one thread per cell column,
// every cell testing box, walls and count for itself and reading its six
// neighbours and b from LDS: descent at 64^3 10.5 -> 6.4 us, at 32^3 6.9 ->
// 4.3 (float64 13.1 -> 8.6, 8.1 -> 4.7), ascent 7.7 -> 6.3 and 6.1 -> 5.0 (8.7
// -> 8.4, 6.1 -> 5.9).
constexpr int TL_TS = 8;  // tile edge in cells
constexpr int TL_H2 = 4;  // halo along axis 2
constexpr int TL_ROW = (TL_TS + 2 * TL_H2) / 2;                                         // entries of a row per colour
__host__ __device__ constexpr int tile_edge(int sweeps) { return TL_TS + 4 * sweeps; }  // region edge, axes 0 and 1
__host__ __device__ constexpr int tile_threads(int R) { return 2 * R * R; }

struct TileAxes {
  int o[3], n[3], bc[3];
  __device__ __forceinline__ bool inside(int a, int u) const { return (unsigned)u < (unsigned)n[a] || !bc[a]; }
  // the grid coordinate of an unwrapped u in [-n, 2n) (tile_edges_fit); inside
  // a wall box u is its own
  __device__ __forceinline__ int wrap(int a, int u) const {
    return u + (u < 0 ? n[a] : 0) - (u >= n[a] ? n[a] : 0);
  }
  // neighbours that a wall removes along axis a
  __device__ __forceinline__ int walls(int a, int u) const {
    return (bc[a] != 0) * ((u == 0) + (u == n[a] - 1));
  }
};
// the tile of this workgroup on grid g (or the matching block of the coarse
// grid gc, whose origin is half the fine one)
__device__ __forceinline__ TileAxes tile_axes(const Geo &g, int scale) {
  TileAxes t;
  const int t1 = (g.n1 + TL_TS - 1) / TL_TS, t2 = (g.n2 + TL_TS - 1) / TL_TS, b = blockIdx.x;
  const int tile[3] = {b / (t1 * t2), (b / t2) % t1, b % t2};
  t.n[0] = g.n0 / scale; t.n[1] = g.n1 / scale; t.n[2] = g.n2 / scale;
  t.bc[0] = g.bc0; t.bc[1] = g.bc1; t.bc[2] = g.bc2;
#pragma unroll
  for (int a = 0; a < 3; ++a) t.o[a] = tile[a] * TL_TS / scale;
  return t;
}

template <typename T>
struct alignas(16) Quad {
  T v[4];
};

// A thread's half row of the region: its place, the offsets of its two pairs
// of entries in a colour plane of the grid, and what its cells share.
template <typename T, int R>
struct TileRow {
  int r0, r1, h, par;  // par: (r0 + r1) & 1
  int q;               // LDS slot of its first entry
  int nn01;            // neighbours that axes 0 and 1 leave
  bool live;           // the row lies in the grid
  bool tile;           // its tile cells (two entries per colour) are the tile's own
  long long off[2];
  T inv[2][4];  // 1 / neighbours per colour and entry, 0 outside the grid

  __device__ __forceinline__ bool box(int lo) const {
    return live && r0 >= lo && r0 < R - lo && r1 >= lo && r1 < R - lo;
  }
  // unwrapped axis-2 coordinate of entry e of colour c
  __device__ __forceinline__ int u2(const TileAxes &ax, int c, int e) const {
    return ax.o[2] - TL_H2 + 2 * (4 * h + e) + ((c + par) & 1);
  }
};
template <typename T, int R>
__device__ __forceinline__ TileRow<T, R> tile_row(const Geo &g, const TileAxes &ax) {
  constexpr int H = (R - TL_TS) / 2;
  TileRow<T, R> w;
  const int tid = threadIdx.x, row = tid >> 1;
  w.h = tid & 1;
  w.r0 = row / R;
  w.r1 = row - w.r0 * R;
  w.par = (w.r0 + w.r1) & 1;
  w.q = TL_ROW * row + 4 * w.h;
  const int u0 = ax.o[0] - H + w.r0, u1 = ax.o[1] - H + w.r1;
  w.live = ax.inside(0, u0) && ax.inside(1, u1);
  w.tile = w.r0 >= H && w.r0 < H + TL_TS && w.r1 >= H && w.r1 < H + TL_TS && u0 < ax.n[0] && u1 < ax.n[1] &&
           ax.o[2] + 4 * w.h < ax.n[2];
  w.nn01 = 6 - ax.walls(0, u0) - ax.walls(1, u1);
  // outside a wall box (nothing used there) the first row, the first pair
  const long long line = w.live ? ((long long)ax.wrap(0, u0) * g.n1 + ax.wrap(1, u1)) * g.hn2 : 0;
#pragma unroll
  for (int z = 0; z < 2; ++z) {
    const int m = (ax.o[2] - TL_H2) / 2 + 4 * w.h + 2 * z;
    const int mw = m + (m < 0 ? g.hn2 : 0) - (m >= g.hn2 ? g.hn2 : 0);
    w.off[z] = line + (ax.inside(2, 2 * m) ? mw : 0);
  }
  const T i0 = w.live ? inv_nn<T>(w.nn01) : T(0);
  const bool edge = ax.bc[2] && (ax.o[2] == 0 || ax.o[2] + TL_TS + TL_H2 >= ax.n[2]);
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) w.inv[c][e] = i0;
  if (edge) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int u2 = w.u2(ax, c, e);
        w.inv[c][e] = w.live && ax.inside(2, u2) ? inv_nn<T>(w.nn01 - ax.walls(2, u2)) : T(0);
      }
  }
  return w;
}
// the four entries of one colour from the grid (p: that colour's plane)
template <typename T, typename S>
__device__ __forceinline__ Quad<T> tile_load(const S *p, const long long off[2]) {
  const V2<T> a = ld2<T>(p + off[0]), b = ld2<T>(p + off[1]);
  return Quad<T>{{a.x, a.y, b.x, b.y}};
}
// the sums of the neighbours of the thread's four cells of colour c: own row's
// other-colour entries from registers, the rows beside and the one entry
// beyond from LDS (o: the other colour)
template <typename T, int R>
__device__ __forceinline__ Quad<T> tile_sums(const T *o, const TileRow<T, R> &w, int c, const Quad<T> &x) {
  const Quad<T> xm = *(const Quad<T> *)(o + w.q - TL_ROW * R), xp = *(const Quad<T> *)(o + w.q + TL_ROW * R);
  const Quad<T> ym = *(const Quad<T> *)(o + w.q - TL_ROW), yp = *(const Quad<T> *)(o + w.q + TL_ROW);
  const bool s = (c + w.par) & 1;
  const T far = o[w.q + (s ? 4 : -1)];
  const T z[5] = {s ? x.v[0] : far, s ? x.v[1] : x.v[0], s ? x.v[2] : x.v[1], s ? x.v[3] : x.v[2], s ? far : x.v[3]};
  Quad<T> r;
#pragma unroll
  for (int e = 0; e < 4; ++e) r.v[e] = xm.v[e] + xp.v[e] + ym.v[e] + yp.v[e] + z[e] + z[e + 1];
  return r;
}
// one red-black half sweep of colour c over the rows of the box [lo, R - lo)^2
template <typename T, int R>
__device__ __forceinline__ void tile_sweep(T (*sx)[TL_ROW * R * R], const TileRow<T, R> &w, int c, int lo,
                                           const Quad<T> b[2], Quad<T> x[2], T th2) {
  if (w.box(lo)) {
    const Quad<T> sum = tile_sums<T, R>(sx[1 - c], w, c, x[1 - c]);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[c].v[e] = pc_relax(th2, b[c].v[e], sum.v[e], w.inv[c][e]);
    *(Quad<T> *)(sx[c] + w.q) = x[c];
  }
  __syncthreads();
}
// the tile's own cells of both colours: two entries of each half row
template <typename T, int R>
__device__ __forceinline__ void tile_store(const Geo &g, const TileRow<T, R> &w, const Quad<T> x[2], T *out) {
  if (!w.tile) return;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    T *p = out + c * g.half + (w.h ? w.off[0] : w.off[1]);
    st2<T>(p, 0, w.h ? x[c].v[0] : x[c].v[2], w.h ? x[c].v[1] : x[c].v[3]);
  }
}

// Descent of one tile: PRE red-black sweeps from x = 0 (red then black), x of
// the tile's cells written, and the coarse right-hand side of the tile's
// coarse cells: the average of the residuals of the four red children (the
// black ones were relaxed last and have none).  The halo is 2 PRE: the first
// red values need only their own b, every later half sweep shrinks the box.
template <typename T, typename TB, int PRE>
__global__ void __launch_bounds__(tile_threads(tile_edge(PRE))) k_tile_down(Geo g, T *x, const TB *b, Geo gc, T *bc) {
  constexpr int R = tile_edge(PRE), H = 2 * PRE, TC = TL_TS / 2;
  __shared__ __attribute__((aligned(16))) T sx[2][TL_ROW * R * R];
  __shared__ __attribute__((aligned(16))) T rs[TL_TS * TL_TS * TC];  // red residuals [row][coarse K]
  const TileAxes ax = tile_axes(g, 1);
  const TileRow<T, R> w = tile_row<T, R>(g, ax);
  const int tid = threadIdx.x;
  const T th2 = (T)g.h2, ih2 = (T)(1.0 / g.h2);
  Quad<T> bb[2], xx[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) bb[c] = tile_load<T>(b + c * g.half, w.off);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    xx[0].v[e] = w.inv[0][e] != T(0) ? pc_first(th2, bb[0].v[e], w.inv[0][e]) : T(0);
    xx[1].v[e] = T(0);
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) *(Quad<T> *)(sx[c] + w.q) = xx[c];
  __syncthreads();
  tile_sweep<T, R>(sx, w, 1, 1, bb, xx, th2);
  if (PRE == 2) {
    tile_sweep<T, R>(sx, w, 0, 2, bb, xx, th2);
    tile_sweep<T, R>(sx, w, 1, 3, bb, xx, th2);
  }
  tile_store<T, R>(g, w, xx, x);
  // the red residuals of the tile's rows; a row's red cell at entry m is the
  // child of coarse K = m - TL_H2 / 2 there
  if (w.tile) {
    const Quad<T> sum = tile_sums<T, R>(sx[1], w, 0, xx[1]);
    T r[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      r[e] = pc_resid(bb[0].v[e], xx[0].v[e], sum.v[e], (T)(w.nn01 - ax.walls(2, w.u2(ax, 0, e))), ih2);
    T *p = rs + ((w.r0 - H) * TL_TS + w.r1 - H) * TC + 2 * w.h;
    st2<T>(p, 0, w.h ? r[0] : r[2], w.h ? r[1] : r[3]);
  }
  __syncthreads();
  // coarse cell (C0, C1, C2) of the tile: the residuals of its four rows,
  // added plane by plane per row, then the two rows, as k_restrict does
  if (tid < TC * TC * TC) {
    const int C2 = tid % TC, C1 = (tid / TC) % TC, C0 = tid / (TC * TC);
    const T *p = rs + (2 * C0 * TL_TS + 2 * C1) * TC + C2;
    const T a0 = p[0] + p[TL_TS * TC], a1 = p[TC] + p[TL_TS * TC + TC];
    const int I = ax.o[0] / 2 + C0, J = ax.o[1] / 2 + C1, K = ax.o[2] / 2 + C2;
    if (I < gc.n0 && J < gc.n1 && K < gc.n2) bc[sidx(gc, I, J, K)] = (a0 + a1) * (T)0.125;
  }
}

// Ascent of one tile: x = xin + P x_c on the red cells (trilinear
// cell-centred, as k_prolong: per axis 3/4 on the parent, 1/4 on the
// parent's neighbour on the child's side, the parent itself past a wall),
// then POST sweeps black then red, and the tile's cells written to xout.
// xout is not xin: neighbouring tiles still read the halo's old values.  The
// halo is 2 POST; the coarse block spans the parents and their neighbours of
// the whole region, past a wall the nearest cell (the parent itself).
template <typename T, typename TB, int POST>
__global__ void __launch_bounds__(tile_threads(tile_edge(POST))) k_tile_up(Geo g, const T *xin, T *xout, const TB *b,
                                                                            Geo gc, const T *xc) {
  constexpr int R = tile_edge(POST), H = 2 * POST, NT = tile_threads(R);
  constexpr int RC = R / 2 + 2, RK = TL_ROW + 2, RKP = 12;  // coarse block: RC x RC rows of RK, RKP apart
  constexpr int NC = (RC * RC * RK + NT - 1) / NT;
  __shared__ __attribute__((aligned(16))) T sx[2][TL_ROW * R * R];
  __shared__ __attribute__((aligned(16))) T sc[RC * RC * RKP];
  const TileAxes ax = tile_axes(g, 1), cx = tile_axes(g, 2);
  const TileRow<T, R> w = tile_row<T, R>(g, ax);
  const int tid = threadIdx.x;
  const T th2 = (T)g.h2;
  // the coarse block, b and the red x: every load issued before the first is used
  T cl[NC];
#pragma unroll
  for (int t = 0; t < NC; ++t) {
    const int e = min(tid + t * NT, RC * RC * RK - 1), row = e / RK, c2 = e - row * RK, c0 = row / RC, c1 = row - c0 * RC;
    auto at = [&](int a, int u) {
      const int v = cx.bc[a] ? min(max(u, 0), cx.n[a] - 1) : cx.wrap(a, u);
      return v;
    };
    cl[t] = xc[sidx(gc, at(0, cx.o[0] - H / 2 - 1 + c0), at(1, cx.o[1] - H / 2 - 1 + c1),
                    at(2, cx.o[2] - TL_H2 / 2 - 1 + c2))];
  }
  Quad<T> bb[2], xx[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) bb[c] = tile_load<T>(b + c * g.half, w.off);
  xx[0] = tile_load<T>(xin, w.off);
#pragma unroll
  for (int t = 0; t < NC; ++t) {
    const int e = tid + t * NT, row = e / RK;
    if (e < RC * RC * RK) sc[row * RKP + (e - row * RK)] = cl[t];
  }
  __syncthreads();
  // prolongation onto the red cells of the half row: coarse planes
  // (u0 - 1) >> 1 and the next with weights by the parity of u0 (that of r0),
  // rows J and Jo; entry m has the parent K = m, its neighbour on the side of
  // the cell's parity (block slots m + 1 and m or m + 2)
  {
    const bool o0 = w.r0 & 1, o1 = w.r1 & 1, o2 = w.par;
    const int lo = (w.r0 + 1) >> 1, J = (w.r1 >> 1) + 1, Jo = o1 ? J + 1 : J - 1;
    const T wlo = o0 ? (T)0.75 : (T)0.25, whi = (T)1 - wlo;
    T acc[4];
#pragma unroll
    for (int pl = 0; pl < 2; ++pl) {
      T zz[2][4];
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        const T *p = sc + ((lo + pl) * RC + (y ? Jo : J)) * RKP + 4 * w.h;
        const Quad<T> a = *(const Quad<T> *)p;
        const T a4 = p[4], a5 = p[5];
        zz[y][0] = blend34(a.v[1], o2 ? a.v[2] : a.v[0]);
        zz[y][1] = blend34(a.v[2], o2 ? a.v[3] : a.v[1]);
        zz[y][2] = blend34(a.v[3], o2 ? a4 : a.v[2]);
        zz[y][3] = blend34(a4, o2 ? a5 : a.v[3]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const T z = blend34(zz[0][e], zz[1][e]);
        acc[e] = pl ? fma(whi, z, acc[e]) : wlo * z;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      xx[0].v[e] = w.inv[0][e] != T(0) ? xx[0].v[e] + acc[e] : T(0);
      xx[1].v[e] = T(0);
    }
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) *(Quad<T> *)(sx[c] + w.q) = xx[c];
  __syncthreads();
  tile_sweep<T, R>(sx, w, 1, 1, bb, xx, th2);
  tile_sweep<T, R>(sx, w, 0, 2, bb, xx, th2);
  if (POST == 2) {
    tile_sweep<T, R>(sx, w, 1, 3, bb, xx, th2);
    tile_sweep<T, R>(sx, w, 0, 4, bb, xx, th2);
  }
  tile_store<T, R>(g, w, xx, xout);
}

// Edges that the tiles take.  The last tiles of an axis may be cut (they store
// only what lies in the grid); along axis 2 the cut must not split a pair of
// entries, and neither the region nor its coarse block, which reach 12 and 7
// cells past the origin of the last tile, may wrap past a second period: 10
// cells are too few.
bool tile_edges_fit(int n0, int n1, int n2) {
  auto rows = [](int n) { return n % 2 == 0 && n >= 8 && n != 10; };
  return rows(n0) && rows(n1) && n2 % 4 == 0 && n2 >= 8;
}
bool tile_level_fits(const Geo &g, const Geo &gc, int pre, int post) {
  return tile_edges_fit(g.n0, g.n1, g.n2) && gc.n0 * 2 == g.n0 && gc.n1 * 2 == g.n1 && gc.n2 * 2 == g.n2 &&
         (pre == 1 || pre == 2) && (post == 1 || post == 2);
}
static unsigned tile_count(const Geo &g) {
  auto cut = [](int n) { return (unsigned)((n + TL_TS - 1) / TL_TS); };
  return cut(g.n0) * cut(g.n1) * cut(g.n2);
}

template <typename T, typename TB>
hipError_t mg_tile_down(const Geo &g, T *x, const TB *b, const Geo &gc, T *bc, int pre, hipStream_t s) {
  if (!tile_level_fits(g, gc, pre, 1)) return hipErrorInvalidValue;
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
  if (pre == 2)
    hipExtLaunchKernelGGL((k_tile_down<T, TB, 2>), dim3(tile_count(g)), dim3(tile_threads(tile_edge(2))), 0, s, e0,
                          e1, 0, g, x, b, gc, bc);
  else
    hipExtLaunchKernelGGL((k_tile_down<T, TB, 1>), dim3(tile_count(g)), dim3(tile_threads(tile_edge(1))), 0, s, e0,
                          e1, 0, g, x, b, gc, bc);
  return hipGetLastError();
}
template <typename T, typename TB>
hipError_t mg_tile_up(const Geo &g, const T *xin, T *xout, const TB *b, const Geo &gc, const T *xc, int post,
                      hipStream_t s) {
  if (!tile_level_fits(g, gc, 1, post) || xin == xout) return hipErrorInvalidValue;
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
  if (post == 2)
    hipExtLaunchKernelGGL((k_tile_up<T, TB, 2>), dim3(tile_count(g)), dim3(tile_threads(tile_edge(2))), 0, s, e0,
                          e1, 0, g, xin, xout, b, gc, xc);
  else
    hipExtLaunchKernelGGL((k_tile_up<T, TB, 1>), dim3(tile_count(g)), dim3(tile_threads(tile_edge(1))), 0, s, e0,
                          e1, 0, g, xin, xout, b, gc, xc);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Coarse-grid kernel: one workgroup, the whole coarse hierarchy in LDS
// (natural layout).  Projects the right-hand side to mean zero (L is
// singular on constants), then runs `cycles` V-cycles with `sweeps` red-black
// sweeps per level and `bottom` sweeps on the smallest grid.
constexpr int COARSE_MAX = 4096;                 // cells of the coarse grid
constexpr int COARSE_CAP = 4096 + 512 + 64 + 8 + 8;
constexpr int COARSE_THREADS = 1024;
constexpr int COARSE_MAXLEV = 8;
int coarse_max_cells() { return COARSE_MAX; }

struct LvlDim { int n0, n1, n2, off, l1, l2, pow2; };

__device__ __forceinline__ void lds_decode(const LvlDim &d, int e, int &i, int &j, int &k) {
  if (d.pow2) {
    k = e & (d.n2 - 1);
    j = (e >> d.l2) & (d.n1 - 1);
    i = e >> (d.l1 + d.l2);
  } else {
    k = e % d.n2;
    int r = e / d.n2;
    j = r % d.n1;
    i = r / d.n1;
  }
}

template <typename T>
__device__ __forceinline__ T lds_nb(const T *x, LvlDim d, int bc0, int bc1, int bc2, int i, int j, int k, int &nn) {
  T s = T(0);
  int t;
  nn = 0;
  t = nbr(i, -1, d.n0, bc0); if (t >= 0) { s += x[d.off + (t * d.n1 + j) * d.n2 + k]; ++nn; }
  t = nbr(i, 1, d.n0, bc0);  if (t >= 0) { s += x[d.off + (t * d.n1 + j) * d.n2 + k]; ++nn; }
  t = nbr(j, -1, d.n1, bc1); if (t >= 0) { s += x[d.off + (i * d.n1 + t) * d.n2 + k]; ++nn; }
  t = nbr(j, 1, d.n1, bc1);  if (t >= 0) { s += x[d.off + (i * d.n1 + t) * d.n2 + k]; ++nn; }
  t = nbr(k, -1, d.n2, bc2); if (t >= 0) { s += x[d.off + (i * d.n1 + j) * d.n2 + t]; ++nn; }
  t = nbr(k, 1, d.n2, bc2);  if (t >= 0) { s += x[d.off + (i * d.n1 + j) * d.n2 + t]; ++nn; }
  return s;
}

// Sync of the threads that take part in a coarse-kernel phase: the whole
// workgroup, or only wavefront 0 for levels small enough for one wavefront
// (its LDS operations complete in program order, so a compiler-level fence
// between phases suffices).
__device__ __forceinline__ void phase_sync(bool one_wave) {
  if (one_wave) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  } else {
    __syncthreads();
  }
}

// One red-black half sweep over the cells of colour `color` only (the
// in-row index of a colour-c cell of row (i, j) is k = 2 kh + ((i+j+c) & 1);
// every level has an even n2).
template <typename T>
__device__ void lds_smooth(T *x, const T *b, LvlDim d, int bc0, int bc1, int bc2, T h2, int color, int nthr) {
  const int hn2 = d.n2 >> 1;
  const int nc = d.n0 * d.n1 * hn2;
  for (int e = threadIdx.x; e < nc; e += nthr) {
    int kh, r, i, j;
    if (d.pow2) {
      kh = e & (hn2 - 1);
      r = e >> (d.l2 - 1);
      j = r & (d.n1 - 1);
      i = r >> d.l1;
    } else {
      kh = e % hn2;
      r = e / hn2;
      j = r % d.n1;
      i = r / d.n1;
    }
    const int k = 2 * kh + ((i + j + color) & 1);
    int nn;
    T s = lds_nb(x, d, bc0, bc1, bc2, i, j, k, nn);
    const int q = d.off + (i * d.n1 + j) * d.n2 + k;
    x[q] = (h2 * b[q] + s) * inv_nn<T>(nn);
  }
}

template <typename T>
__device__ __forceinline__ T lds_resid(const T *x, const T *b, LvlDim d, int bc0, int bc1, int bc2, T ih2, int i,
                                       int j, int k) {
  int nn;
  T s = lds_nb(x, d, bc0, bc1, bc2, i, j, k, nn);
  int e = d.off + (i * d.n1 + j) * d.n2 + k;
  return b[e] - ((T)nn * x[e] - s) * ih2;
}

template <typename T>
__device__ double block_sum(double v, double *red) {
  v = wave_sum(v);
  int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  if (l == 0) red[w] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0) {
    for (int q = 0; q < COARSE_THREADS / 64; ++q) t += red[q];
    red[COARSE_THREADS / 64] = t;
  }
  __syncthreads();
  t = red[COARSE_THREADS / 64];
  __syncthreads();
  return t;
}

__device__ __forceinline__ int coarse_partner(int C, int odd, int nc, int bc) {
  int o = C + (odd ? 1 : -1);
  if (o < 0 || o >= nc) o = bc ? C : (o < 0 ? o + nc : o - nc);
  return o;
}

template <typename T, typename TB>
__global__ void __launch_bounds__(COARSE_THREADS) k_coarse(Geo g, const TB *bin, T *xout, int cycles, int sweeps,
                                                           int bottom) {
  __shared__ T sx[COARSE_CAP];
  __shared__ T sb[COARSE_CAP];
  __shared__ double red[COARSE_THREADS / 64 + 1];
  __shared__ LvlDim dims[COARSE_MAXLEV];
  __shared__ int s_nl;
  if (threadIdx.x == 0) {
    int nl = 1;
    dims[0].n0 = g.n0; dims[0].n1 = g.n1; dims[0].n2 = g.n2; dims[0].off = 0;
    while (nl < COARSE_MAXLEV) {
      LvlDim q = dims[nl - 1];
      if ((q.n0 & 1) || (q.n1 & 1) || (q.n2 & 1) || q.n0 < 4 || q.n1 < 4 || q.n2 < 4) break;
      LvlDim nx;
      nx.n0 = q.n0 / 2; nx.n1 = q.n1 / 2; nx.n2 = q.n2 / 2;
      nx.off = q.off + q.n0 * q.n1 * q.n2;
      dims[nl] = nx;
      ++nl;
    }
    for (int l = 0; l < nl; ++l) {
      LvlDim &q = dims[l];
      bool p2 = !(q.n0 & (q.n0 - 1)) && !(q.n1 & (q.n1 - 1)) && !(q.n2 & (q.n2 - 1));
      q.pow2 = p2;
      q.l1 = 31 - __clz(q.n1);
      q.l2 = 31 - __clz(q.n2);
    }
    s_nl = nl;
  }
  __syncthreads();
  const int nl = s_nl;
  const int bc0 = g.bc0, bc1 = g.bc1, bc2 = g.bc2;
  const int nc0 = g.n0 * g.n1 * g.n2;
  // load b (split layout -> natural) and project it to mean zero
  double loc = 0.0;
  for (int e = threadIdx.x; e < nc0; e += COARSE_THREADS) {
    int k = e % g.n2, r = e / g.n2, j = r % g.n1, i = r / g.n1;
    T v = (T)bin[sidx(g, i, j, k)];
    sb[e] = v;
    sx[e] = T(0);
    loc += (double)v;
  }
  double mean = block_sum<T>(loc, red) / (double)nc0;
  for (int e = threadIdx.x; e < nc0; e += COARSE_THREADS) sb[e] -= (T)mean;
  __syncthreads();

  // levels of at most 2 x 64 cells run on wavefront 0 alone
  auto small = [&](const LvlDim &q) { return q.n0 * q.n1 * q.n2 <= 128; };
  for (int cyc = 0; cyc < cycles; ++cyc) {
    T h = (T)g.h;
    for (int l = 0; l + 1 < nl; ++l) {
      const LvlDim f = dims[l], c = dims[l + 1];
      const bool one = small(f);
      const int nthr = one ? 64 : COARSE_THREADS;
      if (!one || threadIdx.x < 64) {
        T h2 = h * h;
        for (int s = 0; s < sweeps; ++s) {
          lds_smooth(sx, sb, f, bc0, bc1, bc2, h2, 0, nthr);
          phase_sync(one);
          lds_smooth(sx, sb, f, bc0, bc1, bc2, h2, 1, nthr);
          phase_sync(one);
        }
        int ncc = c.n0 * c.n1 * c.n2;
        T ih2 = T(1) / h2;
        for (int e = threadIdx.x; e < ncc; e += nthr) {
          int i, j, k;
          lds_decode(c, e, i, j, k);
          T acc = T(0);
          for (int q = 0; q < 8; ++q)
            acc += lds_resid(sx, sb, f, bc0, bc1, bc2, ih2, 2 * i + (q >> 2), 2 * j + ((q >> 1) & 1), 2 * k + (q & 1));
          sb[c.off + e] = acc * (T)0.125;
          sx[c.off + e] = T(0);
        }
      }
      if (one) phase_sync(true);
      else __syncthreads();
      h = h * (T)2;
    }
    {
      const LvlDim f = dims[nl - 1];
      const bool one = small(f);
      const int nthr = one ? 64 : COARSE_THREADS;
      if (!one || threadIdx.x < 64) {
        T h2 = h * h;
        for (int s = 0; s < bottom; ++s) {
          lds_smooth(sx, sb, f, bc0, bc1, bc2, h2, 0, nthr);
          phase_sync(one);
          lds_smooth(sx, sb, f, bc0, bc1, bc2, h2, 1, nthr);
          phase_sync(one);
        }
      }
    }
    for (int l = nl - 2; l >= 0; --l) {
      h = h * (T)0.5;
      const LvlDim f = dims[l], c = dims[l + 1];
      const bool one = small(f);
      const int nthr = one ? 64 : COARSE_THREADS;
      // the coarse level was written by all threads (large) or wavefront 0
      if (!small(c) || !one) __syncthreads();
      if (!one || threadIdx.x < 64) {
        int ncf = f.n0 * f.n1 * f.n2;
        for (int e = threadIdx.x; e < ncf; e += nthr) {
          int i, j, k;
          lds_decode(f, e, i, j, k);
          int I0 = i >> 1, J0 = j >> 1, K0 = k >> 1;
          int I1 = coarse_partner(I0, i & 1, c.n0, bc0);
          int J1 = coarse_partner(J0, j & 1, c.n1, bc1);
          int K1 = coarse_partner(K0, k & 1, c.n2, bc2);
          const T *xc = sx + c.off;
#define XC(a, b, cc) xc[((a) * c.n1 + (b)) * c.n2 + (cc)]
          T v0 = (T)0.75 * XC(I0, J0, K0) + (T)0.25 * XC(I1, J0, K0);
          T v1 = (T)0.75 * XC(I0, J1, K0) + (T)0.25 * XC(I1, J1, K0);
          T v2 = (T)0.75 * XC(I0, J0, K1) + (T)0.25 * XC(I1, J0, K1);
          T v3 = (T)0.75 * XC(I0, J1, K1) + (T)0.25 * XC(I1, J1, K1);
#undef XC
          T w0 = (T)0.75 * v0 + (T)0.25 * v1;
          T w1 = (T)0.75 * v2 + (T)0.25 * v3;
          sx[f.off + e] += (T)0.75 * w0 + (T)0.25 * w1;
        }
        phase_sync(one);
        T h2 = h * h;
        for (int s = 0; s < sweeps; ++s) {
          lds_smooth(sx, sb, f, bc0, bc1, bc2, h2, 1, nthr);
          phase_sync(one);
          lds_smooth(sx, sb, f, bc0, bc1, bc2, h2, 0, nthr);
          phase_sync(one);
        }
      }
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < nc0; e += COARSE_THREADS) {
    int k = e % g.n2, r = e / g.n2, j = r % g.n1, i = r / g.n1;
    xout[sidx(g, i, j, k)] = sx[e];
  }
}

template <typename T, typename TB>
hipError_t mg_coarse(const Geo &gc, const TB *b, T *x, int cycles, int sweeps, hipStream_t s) {
  if ((long long)gc.n0 * gc.n1 * gc.n2 > COARSE_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_coarse<T, TB>), dim3(1), dim3(COARSE_THREADS), 0, s, gc, b, x, cycles, sweeps, 8);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Exact coarse-grid solve by fast diagonalisation (the direct method of
// Sec. 4.2, here on the coarsest multigrid grid): the rediscretised
// Laplacian of a box with a per-axis boundary type is a Kronecker sum
// L = L0 (+) L1 (+) L2 of 1-D operators with known orthonormal eigenvectors
// Q_a and eigenvalues lam_a, so
//     x = (Q0 x Q1 x Q2) diag(1 / (lam0_i + lam1_j + lam2_k)) (Q0 x Q1 x Q2)^T b,
// the constant mode (all eigenvalues zero) dropped (the pseudo-inverse).
// One workgroup keeps the grid in LDS and applies the six 1-D transforms.
constexpr int FD_MAXN = 32;
constexpr int FD_CELLS = 4096;
constexpr int FD_THREADS = 1024;

// Lines along an axis of n elements are read as pairs and kept an odd number of
// pairs apart, which spreads them over the LDS banks; a grid of at most 4096
// cells with at most 32 along an axis fills at most FD_PAD places in every
// such layout (4 x 32 x 32 cells 6144, 3 x 32 x 32 cells 6144).
constexpr int FD_PAD = 6144;
__host__ __device__ constexpr int fd_line(int n) { return (((n + 1) / 2) | 1) * 2; }

// Eigenvectors Q_a[m][t] (cell m, mode t) of the three axes rounded to T, by
// rows along either index and with zeros past the end of a row, and the
// eigenvalues.
template <typename T>
struct alignas(16) FdBasis {
  T row[2][3][FD_MAXN * fd_line(FD_MAXN)];  // [0]: by mode, over cells; [1]: by cell, over modes
  T lam[3][FD_MAXN];
  __device__ __forceinline__ void load(const Geo &g, const double *p, int tid, int nthr) {
    const int n[3] = {g.n0, g.n1, g.n2};
    const int q1 = n[0] * n[0], q2 = q1 + n[1] * n[1], q3 = q2 + n[2] * n[2], all = q3 + n[0] + n[1] + n[2];
    for (int t = tid; t < all; t += nthr) {
      const T v = (T)p[t];
      if (t < q3) {
        const int a = t < q1 ? 0 : (t < q2 ? 1 : 2), na = a == 0 ? n[0] : (a == 1 ? n[1] : n[2]);
        const int q = t - (a == 0 ? 0 : (a == 1 ? q1 : q2)), r = q / na, c = q - r * na, l = fd_line(na);
        row[0][a][c * l + r] = v;
        row[1][a][r * l + c] = v;
        if (na & 1) {  // the last pair's second weight
          if (r == na - 1) row[0][a][c * l + na] = T(0);
          if (c == na - 1) row[1][a][r * l + na] = T(0);
        }
      } else {
        const int q = t - q3, a = q < n[0] ? 0 : (q < n[0] + n[1] ? 1 : 2);
        lam[a][q - (a == 0 ? 0 : (a == 1 ? n[0] : n[0] + n[1]))] = v;
      }
    }
  }
};
// The places of one element in the three layouts with lines along axis a: of
// the line and of the element.
struct FdPlace {
  int line[3], at[3], i[3];
};
__device__ __forceinline__ FdPlace fd_place(const Geo &g, int e) {
  FdPlace p;
  const int r = e / g.n2;
  p.i[2] = e - r * g.n2;
  p.i[0] = r / g.n1;
  p.i[1] = r - p.i[0] * g.n1;
  p.line[0] = (p.i[1] * g.n2 + p.i[2]) * fd_line(g.n0);
  p.line[1] = (p.i[0] * g.n2 + p.i[2]) * fd_line(g.n1);
  p.line[2] = (p.i[0] * g.n1 + p.i[1]) * fd_line(g.n2);
#pragma unroll
  for (int a = 0; a < 3; ++a) p.at[a] = p.line[a] + p.i[a];
  return p;
}
// The grid in A (elements at at[2]) to x, element tid + u nthr in v[u], by way
// of A and B (whose places past a line's end hold finite values).  The six 1-D
// transforms: forward along axes 2, 1, 0, the last divided by the sums of the
// eigenvalues, backward along 0, 1, 2; each leaves its result in lines along
// the axis of the next.
template <typename T, int EPT>
__device__ __forceinline__ void fd_solve(const Geo &g, const FdBasis<T> &fb, T *A, T *B, const FdPlace (&pl)[EPT], int nc,
                                         int tid, int nthr, T (&v)[EPT]) {
  typedef T Pair __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int p = 0; p < 6; ++p) {
    const int a = p < 3 ? 2 - p : p - 3, w = p < 2 ? 1 - p : (p < 4 ? p - 2 : 2);  // axes of this pass and the next
    const int na = a == 0 ? g.n0 : (a == 1 ? g.n1 : g.n2), np = (na + 1) / 2;
    const T *rows = p < 3 ? fb.row[0][a] : fb.row[1][a];
    const T *in = p & 1 ? B : A;
    T *o = p & 1 ? A : B;
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
      if (tid + u * nthr < nc) {
        const int ia = a == 0 ? pl[u].i[0] : (a == 1 ? pl[u].i[1] : pl[u].i[2]);
        const Pair *M = (const Pair *)(rows + ia * fd_line(na));
        const Pair *x = (const Pair *)(in + (a == 0 ? pl[u].line[0] : (a == 1 ? pl[u].line[1] : pl[u].line[2])));
        T acc = T(0);
#pragma unroll 4
        for (int t = 0; t < np; ++t) {
          const Pair m = M[t], z = x[t];
          acc = fma(m.x, z.x, acc);
          acc = fma(m.y, z.y, acc);
        }
        if (p == 2) {
          const T d = fb.lam[0][pl[u].i[0]] + fb.lam[1][pl[u].i[1]] + fb.lam[2][pl[u].i[2]];
          acc = d > T(0) ? acc / d : T(0);
        }
        if (p < 5) o[w == 0 ? pl[u].at[0] : (w == 1 ? pl[u].at[1] : pl[u].at[2])] = acc;
        v[u] = acc;
      }
    }
    if (p < 5) __syncthreads();
  }
}

template <typename T, typename TB>
__global__ void __launch_bounds__(FD_THREADS) k_coarse_fd(Geo g, const TB *bin, T *xout, const double *fd) {
  __shared__ __attribute__((aligned(16))) T bufA[FD_PAD];
  __shared__ __attribute__((aligned(16))) T bufB[FD_PAD];
  __shared__ FdBasis<T> basis;
  constexpr int EPT = FD_CELLS / FD_THREADS;
  const int nc = g.n0 * g.n1 * g.n2, tid = threadIdx.x;
  FdPlace pl[EPT];
  T v[EPT];
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    pl[u] = fd_place(g, min(tid + u * FD_THREADS, nc - 1));
    v[u] = (T)bin[sidx(g, pl[u].i[0], pl[u].i[1], pl[u].i[2])];
  }
  basis.load(g, fd, tid, FD_THREADS);
  for (int q = tid; q < FD_PAD; q += FD_THREADS) bufA[q] = bufB[q] = T(0);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < EPT; ++u)
    if (tid + u * FD_THREADS < nc) bufA[pl[u].at[2]] = v[u];
  __syncthreads();
  fd_solve<T, EPT>(g, basis, bufA, bufB, pl, nc, tid, FD_THREADS, v);
#pragma unroll
  for (int u = 0; u < EPT; ++u)
    if (tid + u * FD_THREADS < nc) xout[sidx(g, pl[u].i[0], pl[u].i[1], pl[u].i[2])] = v[u];
}

template <typename T, typename TB>
hipError_t mg_coarse_fd(const Geo &gc, const TB *b, T *x, const double *fd, hipStream_t s) {
  if ((long long)gc.n0 * gc.n1 * gc.n2 > FD_CELLS || gc.n0 > FD_MAXN || gc.n1 > FD_MAXN || gc.n2 > FD_MAXN)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_coarse_fd<T, TB>), dim3(1), dim3(FD_THREADS), 0, s, gc, b, x, fd);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The last two levels of the V-cycle in one workgroup: a fine grid of at most
// SUB_FINE cells (natural layout in LDS) and its coarsest grid, solved exactly
// by fast diagonalisation.  The same cycle as the grid-wide levels: from
// x = 0, `pre` red-black pairs (the first one is the sweep from zero), the
// residual averaged over the eight children, the exact coarse solve (constant
// mode dropped), trilinear prolongation, `post` black-red pairs.  One launch
// replaces the eight of the two levels, which are bound by latency.
//
// Layout as in the tile kernels: a thread owns four entries of a row in both
// colours (rows of n2 / 2 entries per colour, in quads), with right-hand side,
// values and reciprocal neighbour counts in registers; a half sweep reads four
// vectors and one value from LDS.  A neighbour past a wall is a row of zeros.
//
// Bounded by the latency of its phases on one compute unit: 7.1 us inside the
// kernel in float32 on 16^3 cells (2.0 until the right-hand side is there, 0.25
// a half sweep, 0.7 residual, 0.4 restriction, 1.6 coarse solve, 0.8
// prolongation), and the launch.  Before, each cell went by 16-bit index
// tables read from memory and its six neighbours one by one, and the coarse
// lines met in the same LDS banks: 13.2 -> 8.2 us, in float64 14.0 -> 10.8;
// the coarse solve by itself on 10 x 12 x 14 cells in float64 14.6 -> 9.1.
constexpr int SUB_FINE = 4096;
constexpr int SUB_COARSE = SUB_FINE / 8;
constexpr int SUB_PAD = 2 * SUB_COARSE;  // lines of 1 or 3 elements take twice their places
constexpr int SUB_THREADS = 1024;
// per colour: rows of quads (n2 / 2 is even, so a row of two entries fills half
// of its quad and the rows take at most twice the colour's cells) and zeros
constexpr int SUB_ROWS = SUB_FINE + 4;

template <typename T, typename TB, int NT>
__global__ void __launch_bounds__(NT) k_subcycle(Geo gf, Geo gc, const TB *bin, T *xout, const double *fd,
                                                          int pre, int post) {
  __shared__ __attribute__((aligned(16))) T sx[2][SUB_ROWS];
  __shared__ __attribute__((aligned(16))) T fa[SUB_PAD], fb[SUB_PAD];
  __shared__ FdBasis<T> basis;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int quads = (gf.hn2 + 3) / 4, RS = 4 * quads, rows = gf.n0 * gf.n1, zero = rows * RS;
  const int nc = gc.n0 * gc.n1 * gc.n2;
  // the thread's quad: entries m0 .. m0 + cnt - 1 of row (i, j)
  const int row = tid / quads, m0 = 4 * (tid - row * quads), i = row / gf.n1, j = row - i * gf.n1;
  const bool live = row < rows;
  const int cnt = min(gf.hn2 - m0, 4);  // 2 or 4
  const int q = row * RS + m0;
  const long long g0 = live ? (long long)row * gf.hn2 + m0 : 0;
  const long long off[2] = {g0, cnt == 4 ? g0 + 2 : g0};
  Quad<T> bb[2], xx[2], inv[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) bb[c] = tile_load<T>(bin + c * gf.half, off);
  basis.load(gc, fd, tid, nthr);
  for (int e = tid; e < SUB_PAD; e += nthr) fa[e] = fb[e] = T(0);
  // LDS offsets of the neighbouring quads and of the entries beside the quad
  auto line = [&](int a, int b) { return a < 0 || b < 0 ? zero : (a * gf.n1 + b) * RS + m0; };
  const int im = mwrap(i - 1, gf.n0, gf.bc0), ip = mwrap(i + 1, gf.n0, gf.bc0);
  const int jm = mwrap(j - 1, gf.n1, gf.bc1), jp = mwrap(j + 1, gf.n1, gf.bc1);
  const int ml = mwrap(m0 - 1, gf.hn2, gf.bc2), mr = mwrap(m0 + cnt, gf.hn2, gf.bc2);
  const int qxm = line(im, j), qxp = line(ip, j), qym = line(i, jm), qyp = line(i, jp);
  const int ql = ml < 0 ? zero : row * RS + ml, qr = mr < 0 ? zero : row * RS + mr;
  const int nn01 = 2 + (im >= 0) + (ip >= 0) + (jm >= 0) + (jp >= 0), par = (i + j) & 1;
  auto nn = [&](int c, int e) {  // neighbours of entry e of colour c
    const int k = 2 * (m0 + e) + ((c + par) & 1);
    return gf.bc2 ? nn01 - (k == 0) - (k == gf.n2 - 1) : nn01;
  };
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) inv[c].v[e] = live && e < cnt ? inv_nn<T>(nn(c, e)) : T(0);
  const T h2 = (T)(gf.h * gf.h), ih2 = T(1) / h2;
  auto put = [&](int c, const Quad<T> &v) {
    if (live) *(Quad<T> *)(sx[c] + q) = v;
  };
  auto sums = [&](int c, const Quad<T> &x) {
    const T *o = sx[1 - c];
    const Quad<T> xm = *(const Quad<T> *)(o + qxm), xp = *(const Quad<T> *)(o + qxp);
    const Quad<T> ym = *(const Quad<T> *)(o + qym), yp = *(const Quad<T> *)(o + qyp);
    const bool s = (c + par) & 1;
    const T far = o[s ? qr : ql];
    const T x2 = cnt == 2 ? far : x.v[2];  // entry 1 of a half quad meets the row's end
    const T z0 = s ? x.v[0] : far, z1 = s ? x.v[1] : x.v[0], z2 = s ? x2 : x.v[1], z3 = s ? x.v[3] : x.v[2],
            z4 = s ? far : x.v[3];
    Quad<T> r;
    r.v[0] = xm.v[0] + xp.v[0] + ym.v[0] + yp.v[0] + z0 + z1;
    r.v[1] = xm.v[1] + xp.v[1] + ym.v[1] + yp.v[1] + z1 + z2;
    r.v[2] = xm.v[2] + xp.v[2] + ym.v[2] + yp.v[2] + z2 + z3;
    r.v[3] = xm.v[3] + xp.v[3] + ym.v[3] + yp.v[3] + z3 + z4;
    return r;
  };
  // one half sweep over colour c (the operations of lds_smooth)
  auto smooth = [&](int c) {
    if (live) {
      const Quad<T> sum = sums(c, xx[1 - c]);
#pragma unroll
      for (int e = 0; e < 4; ++e) xx[c].v[e] = pc_relax(h2, bb[c].v[e], sum.v[e], inv[c].v[e]);
      put(c, xx[c]);
    }
    __syncthreads();
  };
  // the first half sweep from x = 0
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    xx[0].v[e] = pre > 0 ? pc_first(h2, bb[0].v[e], inv[0].v[e]) : T(0);
    xx[1].v[e] = T(0);
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    put(c, xx[c]);
    if (tid < 4) sx[c][zero + tid] = T(0);
  }
  __syncthreads();
  for (int p = 0; p < pre; ++p) {
    if (p) smooth(0);
    smooth(1);
  }
  // residual of every fine cell (as lds_resid), left in place of x, then the
  // average over the eight children of each coarse cell
  {
    Quad<T> r[2];
    if (live) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const Quad<T> sum = sums(c, xx[1 - c]);
#pragma unroll
        for (int e = 0; e < 4; ++e) r[c].v[e] = pc_resid(bb[c].v[e], xx[c].v[e], sum.v[e], (T)nn(c, e), ih2);
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 2; ++c) put(c, r[c]);
  }
  __syncthreads();
  const FdPlace pl[1] = {fd_place(gc, min(tid, nc - 1))};
  if (tid < nc) {
    T acc = T(0);
#pragma unroll
    for (int z = 0; z < 8; ++z) {
      const int di = z >> 2, dj = (z >> 1) & 1, dk = z & 1;
      acc += sx[(di + dj + dk) & 1][((2 * pl[0].i[0] + di) * gf.n1 + 2 * pl[0].i[1] + dj) * RS + pl[0].i[2]];
    }
    fa[pl[0].at[2]] = acc * (T)0.125;
  }
  __syncthreads();
  // the exact coarse solution, in natural order into fa
  T xc[1];
  fd_solve<T, 1>(gc, basis, fa, fb, pl, nc, tid, nthr, xc);
  if (tid < nc) fa[tid] = xc[0];
  __syncthreads();
  // trilinear prolongation onto the red cells (axis 0, then 1, then 2), and
  // onto the black ones if no sweep follows, which would relax them first
  {
    auto partner = [](int C, int odd, int n, int bc) {
      const int o = C + (odd ? 1 : -1);
      return o >= 0 && o < n ? o : (bc ? C : (o < 0 ? o + n : o - n));
    };
    const int I0 = live ? i >> 1 : 0, J0 = live ? j >> 1 : 0;
    const int I1 = partner(I0, i & 1, gc.n0, gc.bc0), J1 = partner(J0, j & 1, gc.n1, gc.bc1);
    const T *p00 = fa + (I0 * gc.n1 + J0) * gc.n2, *p10 = fa + (I1 * gc.n1 + J0) * gc.n2;
    const T *p01 = fa + (I0 * gc.n1 + J1) * gc.n2, *p11 = fa + (I1 * gc.n1 + J1) * gc.n2;
    auto prolong = [&](int c) {
      const bool s = (c + par) & 1;
      // entry e: parent K = m0 + e, its neighbour K - 1 (s = 0) or K + 1
      T w[5];
#pragma unroll
      for (int t = 0; t < 5; ++t) {
        const int k = m0 + t - (s ? 0 : 1);
        const int kw = k < 0 ? (gc.bc2 ? 0 : gc.n2 - 1) : (k < gc.n2 ? k : (gc.bc2 || k > gc.n2 ? gc.n2 - 1 : 0));
        w[t] = blend34(blend34(p00[kw], p10[kw]), blend34(p01[kw], p11[kw]));
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const T near = s ? w[e] : w[e + 1], far = s ? w[e + 1] : w[e];
        xx[c].v[e] += blend34(near, far);
      }
      put(c, xx[c]);
    };
    prolong(0);
    if (post == 0) prolong(1);
  }
  __syncthreads();
  for (int p = 0; p < post; ++p) {
    smooth(1);
    smooth(0);
  }
  if (live) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      T *o = xout + c * gf.half;
      st2<T>(o + off[0], 0, xx[c].v[0], xx[c].v[1]);
      if (cnt == 4) st2<T>(o + off[1], 0, xx[c].v[2], xx[c].v[3]);
    }
  }
}

bool subcycle_fits(const Geo &gf, const Geo &gc) {
  const long long nf = (long long)gf.n0 * gf.n1 * gf.n2;
  return nf <= SUB_FINE && gf.n2 % 4 == 0 && gc.n0 <= FD_MAXN && gc.n1 <= FD_MAXN && gc.n2 <= FD_MAXN && gc.n0 * 2 == gf.n0 &&
         gc.n1 * 2 == gf.n1 && gc.n2 * 2 == gf.n2;
}

template <typename T, typename TB>
hipError_t mg_subcycle(const Geo &gf, const Geo &gc, const TB *b, T *x, const double *fd, int pre, int post,
                       hipStream_t s) {
  if (!subcycle_fits(gf, gc)) return hipErrorInvalidValue;
  // a thread per quad of a row, and per coarse cell
  const int need = std::max(gf.n0 * gf.n1 * ((gf.hn2 + 3) / 4), gc.n0 * gc.n1 * gc.n2), nthr = (need + 63) / 64 * 64;
  if (nthr > SUB_THREADS) return hipErrorInvalidValue;
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
  // half the threads leave the registers that the float64 kernel wants
  if (nthr <= SUB_THREADS / 2)
    hipExtLaunchKernelGGL((k_subcycle<T, TB, SUB_THREADS / 2>), dim3(1), dim3(nthr), 0, s, e0, e1, 0, gf, gc, b, x, fd,
                          pre, post);
  else
    hipExtLaunchKernelGGL((k_subcycle<T, TB, SUB_THREADS>), dim3(1), dim3(nthr), 0, s, e0, e1, 0, gf, gc, b, x, fd, pre,
                          post);
  return hipGetLastError();
}

// Packed eigen-decompositions of the three 1-D Laplacians of a coarse grid
// (host): Q0 (n0 x n0), Q1, Q2 row-major with the eigenvectors as columns,
// then lam0, lam1, lam2.  No-slip axes: cell-centred Neumann operator,
// eigenvectors cos(pi k (i + 1/2) / n), eigenvalues (4/h^2) sin^2(pi k / 2n).
// Periodic axes: the constant, cos / sin(2 pi k i / n) pairs and, for even n,
// (-1)^i, eigenvalues (4/h^2) sin^2(pi k / n).
int coarse_fd_size(const int n[3]) { return n[0] * n[0] + n[1] * n[1] + n[2] * n[2] + n[0] + n[1] + n[2]; }
void coarse_fd_build(const int n[3], const int bc[3], double h, double *out) {
  const double pi = 3.14159265358979323846;
  double *q = out;
  double *l = out + n[0] * n[0] + n[1] * n[1] + n[2] * n[2];
  for (int a = 0; a < 3; ++a) {
    const int na = n[a];
    const double c = 4.0 / (h * h);
    for (int col = 0; col < na; ++col) {
      double lamv;
      for (int i = 0; i < na; ++i) {
        double v;
        if (bc[a]) {
          const double nrm = col == 0 ? sqrt((double)na) : sqrt(0.5 * na);
          v = cos(pi * col * (i + 0.5) / na) / nrm;
        } else if (col == 0) {
          v = 1.0 / sqrt((double)na);
        } else if ((na % 2 == 0) && col == na - 1) {
          v = ((i & 1) ? -1.0 : 1.0) / sqrt((double)na);
        } else {
          const int k = (col + 1) / 2;  // columns 1, 2 -> k = 1 (cos, sin), 3, 4 -> k = 2 ...
          const double th = 2.0 * pi * k * i / na;
          v = ((col & 1) ? cos(th) : sin(th)) / sqrt(0.5 * na);
        }
        q[i * na + col] = v;
      }
      if (bc[a]) {
        const double sn = sin(pi * col / (2.0 * na));
        lamv = c * sn * sn;
      } else if (col == 0) {
        lamv = 0.0;
      } else if ((na % 2 == 0) && col == na - 1) {
        lamv = c;
      } else {
        const int k = (col + 1) / 2;
        const double sn = sin(pi * k / na);
        lamv = c * sn * sn;
      }
      l[col] = lamv;
    }
    q += na * na;
    l += na;
  }
}

#define INST(T, TB)                                                                                    \
  template hipError_t mg_smooth_first<T, TB>(const Geo &, T *, const TB *, bool, hipStream_t);        \
  template hipError_t mg_smooth<T, TB>(const Geo &, T *, const TB *, int, hipStream_t);               \
  template hipError_t mg_restrict<T, TB>(const Geo &, const T *, const TB *, const Geo &, T *,         \
                                         hipStream_t);                                                 \
  template hipError_t mg_coarse<T, TB>(const Geo &, const TB *, T *, int, int, hipStream_t);                   \
  template hipError_t mg_coarse_fd<T, TB>(const Geo &, const TB *, T *, const double *, hipStream_t);   \
  template hipError_t mg_subcycle<T, TB>(const Geo &, const Geo &, const TB *, T *, const double *, int, int, \
                                         hipStream_t);                                               \
  template hipError_t mg_tile_down<T, TB>(const Geo &, T *, const TB *, const Geo &, T *, int, hipStream_t);   \
  template hipError_t mg_tile_up<T, TB>(const Geo &, const T *, T *, const TB *, const Geo &, const T *, int, \
                                        hipStream_t);
INST(float, float)
INST(float, double)
INST(double, double)
#undef INST
template hipError_t mg_prolong<float>(const Geo &, float *, const Geo &, const float *, hipStream_t);
template hipError_t mg_prolong<double>(const Geo &, double *, const Geo &, const double *, hipStream_t);

}  // namespace ibs
