// The coupling term of S~ = L + c^-1 B^T B on the matrix cores: interpolation
// of a cell field's gradient to the points (W^T G z), spreading of a point
// vector followed by the divergence (D W q), and the two fused for the
// product D W W^T G z, in which the point values never leave the chip.
//
// A point of tile T (cells 4T..4T+3 per axis) only reaches the 8^3 cells
// 4T-2 .. 4T+5 per axis, its region, whichever staggering a component has.
// One workgroup per non-empty point tile stages the region and, 64 points at
// a time, the 1-D weights of its points laid out over the region's positions
// (zero outside a support).  Over these dense rows both directions are
// contractions:
//
//   interpolation:  q_p = -sum_jk (wy wz Td, dy wz Tw, wy dz Tw),
//     Tw[jk] = sum_i wx_p[i] z[i][jk], Td[jk] = sum_i dx_p[i] z[i][jk],
//     two matrix products (64 jk) x (8 i) x (16 points), the rest 15
//     multiply-adds per four rows and two cross-lane sums;
//   spreading:      F[ij][k] = sum_p (q0 dx[i] wy[j] + q1 wx[i] dy[j]) wz[k] + (q2 wx[i] wy[j]) dz[k],
//     a matrix product (64 ij) x (2 terms of each point) x (8 k).
//
// w are the centre weights of an axis and d[t] = w_face[t+1] - w_face[t] the
// differences of its face weights: summation by parts moves the difference
// of z (of the spread forces) from the faces to the weights.  z enters
// relative to one cell of the region, so that a sum rounds at the size of
// z's variation over the region, below the rounding that z itself carries.
//
// A point is handled once, by its own tile; a tile with more than 64 points
// is split over several workgroups (k_couple_items).  The regions of
// neighbouring tiles overlap: every workgroup writes its region's sums to a
// buffer of its own, and k_region_add adds to each cell the regions that
// hold it (those of two tiles per axis), in a fixed order.  No atomics; every
// sum has a fixed order, so results repeat bitwise.
//
// Bound by load latency and instruction issue, not bytes: 144000 points in a
// 256^3 grid (about 25 MB) take 36 us for the product and 13 us for the
// region sums, 300 points in 32^3 5.9 + 4.6 us; from the touch lists, which
// stage a point about six times, 22 + 57 us (32 + 68 us and 7.3 + 6.7 us
// when this kernel was written, before the list kernels got faster).  Points
// are split into workgroups of 64 and not looped over: 55 us with one
// workgroup per tile.  Points scattered through a volume go to the touch lists
// (couple_pays).
#include <hip/hip_ext.h>

#include "internal.h"

namespace ibs {

constexpr int CR = 8;                 // region edge
constexpr int CR3 = CR * CR * CR;     // region cells
constexpr int CRS = CR * CR + 16;     // LDS stride between region planes: four planes read by a wavefront fall on different banks
constexpr int CPTS = 64;              // most points of a workgroup
// a staged point: per axis eight pairs (centre weight, face-weight
// difference), padded so that the 16 points that a wavefront reads together
// start on different banks.  Along axes 0 and 1 a lane's four positions
// hi, 2 + hi, 4 + hi, 6 + hi are adjacent (pair_at).
constexpr int CAX = 2 * CR;
constexpr int CPS = 3 * CAX + 2;
__device__ __forceinline__ int pair_at(int axis, int t) { return axis < 2 ? 4 * (t & 1) + (t >> 1) : t; }

// 16 x 16 x 4 float64 matrix product of one wavefront: lane l holds A[l % 16][l / 16]
// and B[l / 16][l % 16]; accumulator element r of lane l is D[row][l % 16]
// with row = (l / 16) + 4 r.  The rows stand for 16 positions (hi, lo) of a
// region plane pair: lane group g and element r for hi = g / 2,
// lo = 4 (g % 2) + r.
typedef double V4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ V4 mac(double a, double b, V4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int row_group(int row) { return row & 3; }
__device__ __forceinline__ int row_elem(int row) { return row >> 2; }
struct alignas(16) Pair {
  double w, d;
};

enum { CP_PRODUCT = 0, CP_INTERP = 1, CP_SPREAD = 2 };

// The workgroups' work: at most CPTS points of one tile each, tiles in index
// order, a tile's points cut into even shares of whole 16-point groups.
// item = (tile, first point, end, 0); parts[tile] = (first item, count), set
// for the listed tiles (the others hold count 0).  One workgroup; the item
// count is written to *total.
__global__ void __launch_bounds__(SCAN1_T) k_couple_items(int n, const int *tiles, const int *tstart, int4 *items,
                                                          int2 *parts, int *total) {
  const int sum = block_scan(
      n,
      [&](int q) {
        const int t = tiles[q];
        return (tstart[t + 1] - tstart[t] + CPTS - 1) / CPTS;
      },
      [&](int q, int nc, int f) {
        const int t = tiles[q], s0 = tstart[t], s1 = tstart[t + 1];
        const int share = ((s1 - s0 + nc - 1) / nc + 15) & ~15;
        for (int c = 0; c < nc; ++c)
          items[f + c] = make_int4(t, min(s0 + c * share, s1), min(s0 + (c + 1) * share, s1), 0);
        parts[t] = make_int2(f, nc);
      });
  if (threadIdx.x == 0) *total = sum;
}
hipError_t couple_items(int n, const int *tiles, const int *tstart, int4 *items, int2 *parts, int *total,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_couple_items, dim3(1), dim3(SCAN1_T), 0, s, n, tiles, tstart, items, parts, total);
  return hipGetLastError();
}
long long couple_max_items(long long K, long long ntiles) { return (K < ntiles ? K : ntiles) + K / CPTS; }
// The region buffer holds at most CBATCH items (64 MiB); a product over more
// items (surfaces through that many tiles) runs in batches of as many.
constexpr int CBATCH = 16384;
size_t couple_region_bytes(long long K, long long ntiles) {
  const long long m = couple_max_items(K, ntiles);
  return sizeof(double) * CR3 * (size_t)(m < CBATCH ? m : CBATCH);
}

// Whether these kernels beat the touch-list ones on a placement of K points in
// `tiles` point tiles, cut into `items` workgroups, whose supports reach
// `active` tiles.  They pay for every workgroup whatever its points (a region
// staged, written and read back) and for the active tiles once a batch; the
// lists for every active tile more, and for the pairs of point and tile.  The
// costs in ns are a fit to products of a large grid; measured, these kernels and
// the lists, us: spheres of 144000 points in 256^3 cells 49 / 79; scattered
// points in 64^3 cells, 1000 16.2 / 17.9, 20000 34.8 / 32.1, 100000 48 / 65; in
// 128^3, 10000 79 / 103, 100000 253 / 169, 1000000 388 / 531; in 256^3, 10000 158 /
// 232, 100000 (six batches) 2102 / 883, 1000000 (16) 5899 / 1454.
bool couple_pays(long long K, long long tiles, long long items, long long active) {
  const long long batches = items > 0 ? (items + CBATCH - 1) / CBATCH : 1;
  const double here = 6.3 * items + 0.12 * K + (0.8 + 1.1 * (batches - 1)) * active;
  const double lists = 1.55 * tiles + 0.4 * K + 2.75 * active;
  return here <= lists;
}

//   CP_PRODUCT: region = D W W^T G z (times h), z a cell field
//   CP_INTERP:  out = alpha W^T G z + beta y
//   CP_SPREAD:  region = D W q (times h)
template <int KER, int MODE>
__global__ void __launch_bounds__(256, 4)
k_couple(Geo g, double ih, int nt1, int nt2, int nitems, const int4 *__restrict__ items,
         const double *X, const double *z, const double *q, double *region, double alpha, const double *y, double beta, double *out) {
  constexpr int W = KerWidth<KER>::W;
  __shared__ double reg[MODE == CP_SPREAD ? 1 : CR * CRS];
  __shared__ __align__(16) double wts[CPTS * CPS];
  __shared__ __align__(16) double qs[CPTS][4];  // q0, q1, 0, q2: the factors of the two terms
  static_assert(4 * CR3 <= CPTS * CPS, "the four wavefronts' region sums must fit the weight buffer");
  static_assert(CAX % 4 == 0 && CPS % 2 == 0, "pairs are read two at a time");
  // consecutive workgroups go round-robin to the 8 XCDs: each takes a
  // contiguous eighth of the items, so that neighbouring regions meet in its L2
  const int per = (nitems + 7) >> 3, it = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (it >= nitems) return;
  const int4 item = items[it];
  const int tile = item.x, s0 = item.y, np = item.z - item.y, np16 = (np + 15) & ~15;
  const int T2 = tile % nt2, rt = tile / nt2, T1 = rt % nt1, T0 = rt / nt1;
  const int org[3] = {4 * T0 - 2, 4 * T1 - 2, 4 * T2 - 2};
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, lg = lane >> 4, ln = lane & 15;
  // staging task of this thread: axis sa of point sp
  const int sp = tid / 3, sa = tid - 3 * sp;
  const double xs = sp < np ? X[3 * s0 + tid] : 0.0;
  double qv = 0.0;
  if (MODE == CP_SPREAD) qv = sp < np ? q[3 * s0 + tid] : 0.0;
  double zv[CR3 / 256];
  if (MODE != CP_SPREAD) {
    // the region: two rows of eight z cells per 16 lanes; cells outside a
    // wall box hold 0 (no support reaches them).  A region reaches at most
    // two cells past the grid.  Offsets inside a colour plane are 32-bit (a
    // plane of 2^31 cells would need more memory than the card has).
    const int lj = (tid >> 3) & 7, lk = tid & 7;
    int j = org[1] + lj, k = org[2] + lk;
    bool okjk = true;
    if (g.bc1) okjk = (unsigned)j < (unsigned)g.n1;
    else j += (j < 0 ? g.n1 : 0) - (j >= g.n1 ? g.n1 : 0);
    if (g.bc2) okjk = okjk && (unsigned)k < (unsigned)g.n2;
    else k += (k < 0 ? g.n2 : 0) - (k >= g.n2 ? g.n2 : 0);
    const unsigned ojk = (unsigned)j * (unsigned)g.hn2 + (unsigned)(k >> 1), plane = (unsigned)(g.n1 * g.hn2);
#pragma unroll
    for (int u = 0; u < CR3 / 256; ++u) {
      int i = org[0] + wave + 4 * u;  // the same for a whole wavefront
      bool ok = okjk;
      if (g.bc0) ok = ok && (unsigned)i < (unsigned)g.n0;
      else i += (i < 0 ? g.n0 : 0) - (i >= g.n0 ? g.n0 : 0);
      const double *zc = z + (((i + j + k) & 1) ? g.half : 0);
      zv[u] = ok ? zc[(unsigned)i * plane + ojk] : 0.0;
    }
  }
  if (sp < np16) {
    Pair *pr = (Pair *)(wts + sp * CPS + sa * CAX);
#pragma unroll
    for (int t = 0; t < CR; ++t) pr[t] = Pair{0.0, 0.0};
    if (sa == 2) pr[CR] = Pair{0.0, 0.0};  // the row's padding: the z weight of lanes past the region
    if (MODE == CP_SPREAD) qs[sp][sa == 2 ? 3 : sa] = qv;
    if (sp < np) {
      double wf[4], wc[4];
      const int n = sa == 0 ? g.n0 : (sa == 1 ? g.n1 : g.n2), bc = sa == 0 ? g.bc0 : (sa == 1 ? g.bc1 : g.bc2);
      const int o = sa == 0 ? org[0] : (sa == 1 ? org[1] : org[2]);
      const int f0 = axis_weights<KER>(xs, ih, true, wf);
      int lf = f0 - o, lc = axis_weights<KER>(xs, ih, false, wc) - o;
      // a periodic image puts the support into the region; the limits are
      // those of the tile's points (and keep every store inside the row)
      if (!bc && (unsigned)lf > 8u - W) lf = wrapi(lf, n);
      if (!bc && (unsigned)lc > 8u - W) lc = wrapi(lc, n);
      lf = min(max(lf, 1), CR - W);
      lc = min(max(lc, 0), CR - W);
      // a wall face (index 0 along a wall axis) carries no gradient
#pragma unroll
      for (int t = 0; t < W; ++t)
        if (MODE != CP_SPREAD && bc && f0 + t == 0) wf[t] = 0.0;
      double before = 0.0;
#pragma unroll
      for (int t = 0; t < W; ++t) {
        pr[pair_at(sa, lc + t)].w = wc[t];
        pr[pair_at(sa, lf - 1 + t)].d = wf[t] - before;
        before = wf[t];
      }
      pr[pair_at(sa, lf - 1 + W)].d = -before;
    }
  }
  if (MODE != CP_SPREAD) {
#pragma unroll
    for (int u = 0; u < CR3 / 256; ++u) {
      const int e = tid + 256 * u;
      reg[(e >> 6) * CRS + (e & 63)] = zv[u];
    }
  }
  if (tid < CPTS) qs[tid][2] = 0.0;
  __syncthreads();
  // the positions of this lane's matrix rows: A operands row ln
  const int ahi = row_group(ln) >> 1, alo = 4 * (row_group(ln) & 1) + row_elem(ln);
  V4 F[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) F[mt] = V4{0, 0, 0, 0};
  // 16 points per wavefront
  const int p0 = 16 * wave;
  if (p0 < np) {
    if (MODE != CP_SPREAD) {
      const Pair *px = (const Pair *)(wts + (p0 + ln) * CPS);
      const Pair *py = px + CAX / 2 + 4 * (lg >> 1), *pz = px + CAX + 4 * (lg & 1);
      const Pair x0 = px[pair_at(0, lg)], x1 = px[pair_at(0, 4 + lg)];
      Pair zw[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) zw[r] = pz[r];
      const double ref = reg[3 * CRS + 3 * CR + 3];  // a cell of the tile itself
      double qd[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        // rows (2 mt + ahi, alo) of planes lg and 4 + lg
        const int e0 = lg * CRS + (2 * mt + ahi) * CR + alo;
        const double z0 = reg[e0] - ref, z1 = reg[e0 + 4 * CRS] - ref;
        V4 Tw = V4{0, 0, 0, 0}, Td = V4{0, 0, 0, 0};
        Tw = mac(z0, x0.w, Tw);
        Td = mac(z0, x0.d, Td);
        Tw = mac(z1, x1.w, Tw);
        Td = mac(z1, x1.d, Td);
        double sd = zw[0].w * Td[0], sw = zw[0].w * Tw[0], sz = zw[0].d * Tw[0];
#pragma unroll
        for (int r = 1; r < 4; ++r) {
          sd = fma(zw[r].w, Td[r], sd);
          sw = fma(zw[r].w, Tw[r], sw);
          sz = fma(zw[r].d, Tw[r], sz);
        }
        const Pair wy = py[mt];
        qd[0] = fma(wy.w, sd, qd[0]);
        qd[1] = fma(wy.d, sw, qd[1]);
        qd[2] = fma(wy.w, sz, qd[2]);
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        qd[d] += __shfl_xor(qd[d], 16, 64);
        qd[d] += __shfl_xor(qd[d], 32, 64);
        qd[d] *= -ih;
      }
      if (lg < 3) {
        const double v = lg == 0 ? qd[0] : (lg == 1 ? qd[1] : qd[2]);
        if (MODE == CP_INTERP) {
          if (p0 + ln < np) {
            const long long o = 3LL * (s0 + p0 + ln) + lg;
            out[o] = alpha * v + (y ? beta * y[o] : 0.0);
          }
        } else {
          qs[p0 + ln][lg == 2 ? 3 : lg] = v;  // 0 for the padding points, whose rows are 0
        }
      }
      // read below by other lanes of this wavefront only
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (MODE != CP_INTERP) {
      // two points and both terms per product: lane group lg holds term
      // lg % 2 of point lg / 2; an odd last point pairs with a padding row
      const int term = lg & 1, pts = min(16, np - p0);
      const double *row = wts + (p0 + (lg >> 1)) * CPS, *rz = row + 2 * CAX + (ln < 8 ? 2 * ln + term : CAX);
      const Pair *px = (const Pair *)row + 4 * ahi, *py = (const Pair *)(row + CAX) + pair_at(1, alo);
      const Pair *pq = (const Pair *)&qs[p0 + (lg >> 1)][0] + term;
#pragma unroll
      for (int s = 0; s < 16; s += 2) {
        if (s >= pts) break;
        const Pair wy = py[s * (CPS / 2)], qq = pq[2 * s];
        // A = d_x (q0 w_y) + w_x (q1 d_y) for the first term, w_x (q2 w_y) for the second
        const double u = qq.w * wy.w, v = qq.d * (term ? wy.w : wy.d), bz = rz[s * CPS];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
          const Pair wx = px[s * (CPS / 2) + mt];
          F[mt] = mac(fma(wx.d, u, wx.w * v), bz, F[mt]);
        }
      }
    }
  }
  if (MODE != CP_INTERP) {
    __syncthreads();
    double *part = wts;
    if (ln < 8 && p0 < np) {
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          part[wave * CR3 + (2 * mt + (lg >> 1)) * CR * CR + (4 * (lg & 1) + r) * CR + ln] = F[mt][r];
    }
    __syncthreads();
    double *dst = region + (long long)it * CR3;
#pragma unroll
    for (int u = 0; u < CR3 / 256; ++u) {
      const int e = tid + 256 * u;
      double v = part[e];
      for (int w = 1; 16 * w < np; ++w) v += part[w * CR3 + e];
      dst[e] = v;
    }
  }
}

// out += alpha times the region sums, on the active tiles: along an axis
// a cell c = 0..3 of tile T lies in the regions of T (at c + 2) and of T - 1
// (at c + 6, c < 2) or T + 1 (at c - 2, c >= 2); tiles without points and
// past a wall have none.  One wavefront per tile.
__global__ void __launch_bounds__(256) k_region_add(Geo g, int nt0, int nt1, int nt2, int lo, int hi, int nactive,
                                                    const int *__restrict__ active, const int2 *__restrict__ parts,
                                                    const double *__restrict__ region, double alpha, double *__restrict__ out) {
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tile = w < nactive ? active[w] : -1;
  if (tile < 0) return;  // a hole of the launch order
  const int c[3] = {lane >> 4, (lane >> 2) & 3, lane & 3};
  const int t[3] = {tile / (nt1 * nt2), (tile / nt2) % nt1, tile % nt2};
  const int nt[3] = {nt0, nt1, nt2}, bc[3] = {g.bc0, g.bc1, g.bc2};
  const long long e = sidx(g, 4 * t[0] + c[0], 4 * t[1] + c[1], 4 * t[2] + c[2]);
  const double old = out[e];
  int tn[3][2], at[3][2];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    int v = c[a] < 2 ? t[a] - 1 : t[a] + 1;
    if ((unsigned)v >= (unsigned)nt[a]) v = bc[a] ? -1 : (v < 0 ? v + nt[a] : v - nt[a]);
    tn[a][0] = t[a];
    at[a][0] = c[a] + 2;
    tn[a][1] = v;
    at[a][1] = c[a] < 2 ? c[a] + 6 : c[a] - 2;
  }
  int2 pt[8];
#pragma unroll
  for (int o = 0; o < 8; ++o) {
    const int a0 = tn[0][o >> 2], a1 = tn[1][(o >> 1) & 1], a2 = tn[2][o & 1];
    const int2 p = (a0 | a1 | a2) >= 0 ? parts[(a0 * nt1 + a1) * nt2 + a2] : make_int2(0, 0);
    // the tile's items of this batch, [lo, hi)
    const int f = max(p.x, lo);
    pt[o] = make_int2(f - lo, min(p.x + p.y, hi) - f);
  }
  // each tile's first two regions are loaded before any is added
  double v[8], v1[8];
  const double *src[8];
#pragma unroll
  for (int o = 0; o < 8; ++o) {
    src[o] = region + (long long)pt[o].x * CR3 + at[0][o >> 2] * CR * CR + at[1][(o >> 1) & 1] * CR + at[2][o & 1];
    v[o] = pt[o].y > 0 ? src[o][0] : 0.0;
    v1[o] = pt[o].y > 1 ? src[o][CR3] : 0.0;
  }
  double sum = 0.0;
#pragma unroll
  for (int o = 0; o < 8; ++o) {
    v[o] += v1[o];
    for (int m = 2; m < pt[o].y; ++m) v[o] += src[o][(long long)m * CR3];
    sum += v[o];
  }
  out[e] = old + alpha * sum;
}

// items [lo, hi) of one batch (all of them for an interpolation)
template <int MODE>
static void launch_couple(const Geo &g, const Coupling &c, int lo, int hi, const double *z, const double *q, double alpha,
                          const double *y, double beta, double *out, hipStream_t s) {
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
  const dim3 gr(8 * ((hi - lo + 7) / 8)), bl(256);
  if (c.ker == KER_PESKIN4)
    hipExtLaunchKernelGGL((k_couple<KER_PESKIN4, MODE>), gr, bl, 0, s, e0, e1, 0, g, 1.0 / g.h, c.nt1, c.nt2, hi - lo,
                          c.items + lo, c.X, z, q, c.region, alpha, y, beta, out);
  else
    hipExtLaunchKernelGGL((k_couple<KER_ROMA3, MODE>), gr, bl, 0, s, e0, e1, 0, g, 1.0 / g.h, c.nt1, c.nt2, hi - lo,
                          c.items + lo, c.X, z, q, c.region, alpha, y, beta, out);
}
static void launch_region_add(const Geo &g, const Coupling &c, int lo, int hi, double alpha, double *out,
                              hipStream_t s) {
  // the active tiles' cells read and written
  ProbeExt probe_(PR_BAND_DIV, s, (double)probe_band_cells() * 2 * sizeof(double));
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
  hipExtLaunchKernelGGL(k_region_add, dim3((c.nactive + 3) / 4), dim3(256), 0, s, e0, e1, 0, g, c.nt0, c.nt1, c.nt2, lo,
                        hi, c.nactive, c.active, c.parts, c.region, alpha / g.h, out);
}

hipError_t couple_product(const Geo &g, const Coupling &c, const double *z, double alpha, double *w, hipStream_t s) {
  for (int lo = 0; lo < c.nitems; lo += CBATCH) {
    const int hi = c.nitems - lo < CBATCH ? c.nitems : lo + CBATCH;
    {
      // positions and the cells of the support band read
      ProbeExt probe_(PR_INTERP_GRAD, s, (double)probe_points() * 24 + (double)probe_band_cells() * sizeof(double));
      launch_couple<CP_PRODUCT>(g, c, lo, hi, z, nullptr, 0.0, nullptr, 0.0, nullptr, s);
    }
    launch_region_add(g, c, lo, hi, alpha, w, s);
  }
  return hipGetLastError();
}
hipError_t couple_interp(const Geo &g, const Coupling &c, const double *z, double alpha, const double *y, double beta,
                         double *out, hipStream_t s) {
  if (c.nitems == 0) return hipSuccess;
  // positions read, results written (and y read), the cells of the support band
  ProbeExt probe_(PR_INTERP_GRAD, s,
                  (double)probe_points() * (y ? 72 : 48) + (double)probe_band_cells() * sizeof(double));
  launch_couple<CP_INTERP>(g, c, 0, c.nitems, z, nullptr, alpha, y, beta, out, s);
  return hipGetLastError();
}

hipError_t couple_spread(const Geo &g, const Coupling &c, const double *q, double alpha, double *out, hipStream_t s) {
  for (int lo = 0; lo < c.nitems; lo += CBATCH) {
    const int hi = c.nitems - lo < CBATCH ? c.nitems : lo + CBATCH;
    launch_couple<CP_SPREAD>(g, c, lo, hi, nullptr, q, 0.0, nullptr, 0.0, nullptr, s);
    launch_region_add(g, c, lo, hi, alpha, out, s);
  }
  return hipGetLastError();
}

}  // namespace ibs
