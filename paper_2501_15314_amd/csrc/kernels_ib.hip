// Lagrangian-point kernels: placement of the body points, binning into 4^3-
// cell tiles, interpolation W^T (paper Sec. 2.3, eq. interpolation) and
// spreading W (eq. regularization), optionally followed by the divergence
// (B^T = D W, eq. modified_poisson).
//
// Determinism.  No floating-point atomics are used.  Points are sorted into
// tiles in canonical order (tile, original index).  Interpolation reduces
// each point's stencil in a fixed butterfly order.  Spreading is done per
// active tile by one workgroup from the tile's touch list, whose points have
// a fixed order: eight half-wavefronts add every eighth of them into registers,
// a lane to its own columns of faces, and the eight partial sums of a face are
// added in order, so every grid value is summed in the same order on every run.
#include <hip/hip_ext.h>

#include "internal.h"

namespace ibs {

static int nblk(long long n, int bs) { return (int)((n + bs - 1) / bs); }

__global__ void k_points(Geo g, int K, const BodyDev *bodies, const int *body_of, const double *off,
                         double *X, double *U, int *tile, int nt0, int nt1, int nt2) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= K) return;
  const BodyDev &b = bodies[body_of[k]];
  double o0 = off[3 * k], o1 = off[3 * k + 1], o2 = off[3 * k + 2];
  double l0 = b.R[0] * o0 + b.R[1] * o1 + b.R[2] * o2;
  double l1 = b.R[3] * o0 + b.R[4] * o1 + b.R[5] * o2;
  double l2 = b.R[6] * o0 + b.R[7] * o1 + b.R[8] * o2;
  double x0 = b.c[0] + l0, x1 = b.c[1] + l1, x2 = b.c[2] + l2;
  X[3 * k] = x0; X[3 * k + 1] = x1; X[3 * k + 2] = x2;
  // U = u_s + omega x L~
  U[3 * k] = b.v[0] + (b.w[1] * l2 - b.w[2] * l1);
  U[3 * k + 1] = b.v[1] + (b.w[2] * l0 - b.w[0] * l2);
  U[3 * k + 2] = b.v[2] + (b.w[0] * l1 - b.w[1] * l0);
  double ih = 1.0 / g.h;
  int c0 = (int)floor(x0 * ih), c1 = (int)floor(x1 * ih), c2 = (int)floor(x2 * ih);
  c0 = g.bc0 ? min(max(c0, 0), g.n0 - 1) : wrapi(c0, g.n0);
  c1 = g.bc1 ? min(max(c1, 0), g.n1 - 1) : wrapi(c1, g.n1);
  c2 = g.bc2 ? min(max(c2, 0), g.n2 - 1) : wrapi(c2, g.n2);
  tile[k] = ((c0 >> 2) * nt1 + (c1 >> 2)) * nt2 + (c2 >> 2);
}
hipError_t points_place(const Geo &g, int K, const BodyDev *bodies, const int *body_of, const double *off,
                        double *X, double *U, int *tile, int nt0, int nt1, int nt2, hipStream_t s) {
  if (K == 0) return hipSuccess;
  hipLaunchKernelGGL(k_points, dim3(nblk(K, 256)), dim3(256), 0, s, g, K, bodies, body_of, off, X, U, tile,
                     nt0, nt1, nt2);
  return hipGetLastError();
}

__global__ void k_count(int K, const int *tile, int *counts) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < K) atomicAdd(&counts[tile[k]], 1);
}
hipError_t bin_count(int K, const int *tile, int *counts, hipStream_t s) {
  if (K == 0) return hipSuccess;
  hipLaunchKernelGGL(k_count, dim3(nblk(K, 256)), dim3(256), 0, s, K, tile, counts);
  return hipGetLastError();
}

// ---- exclusive scan: 1024 items per block, then the block totals ----------
constexpr int SCAN_T = 256, SCAN_ITEMS = 4, SCAN_CHUNK = SCAN_T * SCAN_ITEMS;

__device__ int block_excl_scan(int v, int *sh) {
  int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int o = 1; o < SCAN_T; o <<= 1) {
    int a = t >= o ? sh[t - o] : 0;
    __syncthreads();
    sh[t] += a;
    __syncthreads();
  }
  int incl = sh[t];
  int tot = sh[SCAN_T - 1];
  __syncthreads();
  sh[SCAN_T] = tot;
  return incl - v;
}

__global__ void k_scan1(const int *in, int *out, int n, int *bsum) {
  __shared__ int sh[SCAN_T + 1];
  long long base = (long long)blockIdx.x * SCAN_CHUNK + threadIdx.x * SCAN_ITEMS;
  int v[SCAN_ITEMS], s = 0;
  for (int q = 0; q < SCAN_ITEMS; ++q) {
    long long i = base + q;
    v[q] = i < n ? in[i] : 0;
    s += v[q];
  }
  int ex = block_excl_scan(s, sh);
  for (int q = 0; q < SCAN_ITEMS; ++q) {
    long long i = base + q;
    if (i < n) out[i] = ex;
    ex += v[q];
  }
  if (threadIdx.x == 0) bsum[blockIdx.x] = sh[SCAN_T];
}
// single block: exclusive scan of the block sums in place (any count), total at bsum[nb]
__global__ void k_scan2(int *bsum, int nb) {
  __shared__ int sh[SCAN_T + 1];
  int carry = 0;
  for (int base = 0; base < nb; base += SCAN_T) {
    int i = base + threadIdx.x;
    int v = i < nb ? bsum[i] : 0;
    int ex = block_excl_scan(v, sh);
    int tot = sh[SCAN_T];
    if (i < nb) bsum[i] = ex + carry;
    carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) bsum[nb] = carry;
}
__global__ void k_scan3(int *out, int n, const int *bsum, int nb) {
  long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] += bsum[i / SCAN_CHUNK];
  if (i == 0) out[n] = bsum[nb];
}
// The whole scan in one workgroup, 4096 items a pass: a pass takes about two
// microseconds, the three launches above about eight together, so up to two
// passes (the tile counts of grids up to 80^3).
constexpr int SCAN1_MAX = 2 * 4 * SCAN1_T;
__global__ void __launch_bounds__(SCAN1_T) k_scan_one(const int *in, int *out, int n) {
  const int total = block_scan(n, [&](int i) { return in[i]; }, [&](int i, int, int ex) { out[i] = ex; });
  if (threadIdx.x == 0) out[n] = total;
}
hipError_t scan_exclusive(const int *in, int *out, int n, int *tmp, hipStream_t s) {
  if (n <= SCAN1_MAX) {
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(SCAN1_T), 0, s, in, out, n);
    return hipGetLastError();
  }
  int nb = nblk(n, SCAN_CHUNK);
  hipLaunchKernelGGL(k_scan1, dim3(nb), dim3(SCAN_T), 0, s, in, out, n, tmp);
  hipLaunchKernelGGL(k_scan2, dim3(1), dim3(SCAN_T), 0, s, tmp, nb);
  hipLaunchKernelGGL(k_scan3, dim3(nblk(n, 256)), dim3(256), 0, s, out, n, tmp, nb);
  return hipGetLastError();
}

__global__ void k_scatter(int K, const int *tile, const int *start, int *fillc, int *perm_tmp) {
  int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= K) return;
  int t = tile[k];
  perm_tmp[start[t] + atomicAdd(&fillc[t], 1)] = k;
}
hipError_t bin_scatter(int K, const int *tile, const int *start, int *fillc, int *perm_tmp, hipStream_t s) {
  if (K == 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter, dim3(nblk(K, 256)), dim3(256), 0, s, K, tile, start, fillc, perm_tmp);
  return hipGetLastError();
}

// Canonical order inside each tile: rank by original index.
__global__ void k_canon(int K, const int *tile, const int *start, const int *perm_tmp, int *perm) {
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= K) return;
  int k = perm_tmp[q];
  int t = tile[k];
  int s0 = start[t], s1 = start[t + 1];
  int r = 0;
  for (int p = s0; p < s1; ++p) r += perm_tmp[p] < k;
  perm[s0 + r] = k;
}
hipError_t bin_canon(int K, const int *tile, const int *start, const int *perm_tmp, int *perm, hipStream_t s) {
  if (K == 0) return hipSuccess;
  hipLaunchKernelGGL(k_canon, dim3(nblk(K, 256)), dim3(256), 0, s, K, tile, start, perm_tmp, perm);
  return hipGetLastError();
}

__global__ void k_compact(int n, const int *flags, const int *pos, int *list) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n && flags[t]) list[pos[t]] = t;
}
hipError_t compact(int n, const int *flags, const int *pos, int *list, hipStream_t s) {
  hipLaunchKernelGGL(k_compact, dim3(nblk(n, 256)), dim3(256), 0, s, n, flags, pos, list);
  return hipGetLastError();
}

__global__ void k_gather3(int K, const int *perm, const double *src, double *dst) {
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= 3 * K) return;
  int s = q / 3, d = q - 3 * s;
  dst[q] = src[3 * perm[s] + d];
}
__global__ void k_scatter3(int K, const int *perm, const double *src, double *dst) {
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= 3 * K) return;
  int s = q / 3, d = q - 3 * s;
  dst[3 * perm[s] + d] = src[q];
}
__global__ void k_scale3(int n, const double *x, double a, const double *y, double b, double *out) {
  int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  out[q] = a * x[q] + (y ? b * y[q] : 0.0);
}
hipError_t gather3(int K, const int *perm, const double *src, double *dst, hipStream_t s) {
  if (K == 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather3, dim3(nblk(3LL * K, 256)), dim3(256), 0, s, K, perm, src, dst);
  return hipGetLastError();
}
hipError_t scatter3(int K, const int *perm, const double *src, double *dst, hipStream_t s) {
  if (K == 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter3, dim3(nblk(3LL * K, 256)), dim3(256), 0, s, K, perm, src, dst);
  return hipGetLastError();
}
hipError_t scale3(int K, const double *x, double alpha, const double *y, double beta, double *out,
                  hipStream_t s) {
  if (K == 0) return hipSuccess;
  hipLaunchKernelGGL(k_scale3, dim3(nblk(3LL * K, 256)), dim3(256), 0, s, 3 * K, x, alpha, y, beta, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Interpolation from a non-empty point tile, by one workgroup or several
// (grid.y: workgroup y takes the chunks y, y + grid.y, ... of IPTS points).
// The points of tile T (cells 4T..4T+3 per axis) only reach nodes 4T-2 .. 4T+5
// per axis, so a workgroup first stages that 8^3 region of the source in LDS
// (MODE 0: the three face fields; MODE 1: the cell field, whose face gradients
// are formed from LDS) together with the 1-D weights of its points (face and
// centre nodes per axis), then gathers every point's stencil from LDS: 16 lanes
// per point (node offsets (a, b)), z nodes summed in order, the 16 partial sums
// reduced by a fixed butterfly.
//
// Bounded by vector instructions (144000 points at 256^3): a support always
// lies in the region -- the staging sees to that, once per point and axis -- so
// the gather tests nothing, reads weights and neighbouring nodes as vectors
// from LDS, takes the wrap around a periodic axis only where it is one, and the
// butterfly stays in the vector registers: 84 vector and 17 LDS instructions
// per four points where there were 168 and 56.  In float32, before and after:
// 144000 points in 2144 tiles 24.2 / 13.9 us; 9000 points in 160 tiles, cut
// into several workgroups each, 20.7 / 4.9 us.
constexpr int IREG = 8;   // region width per axis
// region stride between x planes: 2 more than IREG^2, so the 16 lanes of a
// point (x offsets a, y offsets b) fall on 16 distinct LDS banks
constexpr int IRS = IREG * IREG + 2;
constexpr int IPTS = 32;  // points staged per pass

// v + v of the lane N places on in its row of 16
template <int N>
__device__ __forceinline__ float ror16_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, true));
}
template <int N>
__device__ __forceinline__ double ror16_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + N, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + N, 0xf, 0xf, true);
  return v + __hiloint2double(hi, lo);
}
// Sum over each row of 16 lanes, in the order of a butterfly over lane
// distances 8, 4, 2, 1: after the step of distance d the partial sums repeat
// with period d, so a rotation by d meets the same value as an exchange.
template <typename TA>
__device__ __forceinline__ TA sum16(TA v) {
  return ror16_add<1>(ror16_add<2>(ror16_add<4>(ror16_add<8>(v))));
}

template <int KER, int MODE, typename T, typename TA>
__global__ void __launch_bounds__(256) k_interp(Geo g, int nt1, int nt2, const int *tiles, const int *tstart,
                                                const double *X, const T *src, double alpha, const double *y,
                                                double beta, double *out) {
  constexpr int W = KerWidth<KER>::W;
  constexpr int NC = MODE == 0 ? 3 : 1;
  // TA: the arithmetic type (float64, or float32 for the gradient of a
  // float32 cell field in the float32 Krylov cycle, weights rounded to it)
  __shared__ TA reg[NC][IREG * IRS];
  __shared__ __attribute__((aligned(16))) TA pw[IPTS][3][2][4];  // [point][axis][face/centre][node]
  __shared__ int pb[IPTS][3][2];  // start of the support along the axis, as an offset into the region
  const int tile = tiles[blockIdx.x];
  if (tile < 0) return;  // a hole of the launch order
  const int s0 = tstart[tile] + IPTS * blockIdx.y, s1 = tstart[tile + 1];
  if (s0 >= s1) return;  // fewer chunks than workgroups
  const int T2 = tile % nt2, r = tile / nt2, T1 = r % nt1, T0 = r / nt1;
  const int o0 = 4 * T0 - 2, o1 = 4 * T1 - 2, o2 = 4 * T2 - 2;  // region origin
  const long long N = 2 * g.half;
  // this thread's staging task: point pt, axis ax, staggering st; the
  // coordinate of the first chunk is loaded before the region, so that both
  // loads are in flight together
  static_assert(6 * IPTS <= 256, "one staging task per thread");
  const int spt = threadIdx.x / 6, srem = threadIdx.x - 6 * spt, ax = srem >> 1, st = srem & 1;
  double xv = spt < IPTS && s0 + spt < s1 ? X[3 * (s0 + spt) + ax] : 0.0;
#pragma unroll
  for (int e0 = 0; e0 < IREG * IREG * IREG; e0 += 256) {
    const int e = e0 + threadIdx.x, li = e / (IREG * IREG), lj = (e / IREG) % IREG, lk = e % IREG;
    int i = o0 + li, j = o1 + lj, k = o2 + lk;  // within one period of the grid (n >= 16)
    bool ok = true;
    if (g.bc0) ok = ok && (unsigned)i < (unsigned)g.n0;
    else i += (i < 0 ? g.n0 : 0) - (i >= g.n0 ? g.n0 : 0);
    if (g.bc1) ok = ok && (unsigned)j < (unsigned)g.n1;
    else j += (j < 0 ? g.n1 : 0) - (j >= g.n1 ? g.n1 : 0);
    if (g.bc2) ok = ok && (unsigned)k < (unsigned)g.n2;
    else k += (k < 0 ? g.n2 : 0) - (k >= g.n2 ? g.n2 : 0);
    const long long at = ok ? sidx(g, i, j, k) : 0;
#pragma unroll
    for (int comp = 0; comp < NC; ++comp) {
      const TA v = (TA)src[comp * N + at];
      reg[comp][li * IRS + lj * IREG + lk] = ok ? v : TA(0);
    }
  }
  const int lane = threadIdx.x & 15;
  // node offsets of this lane; a 3-point kernel leaves lanes without nodes,
  // which read the last one with weight 0
  const int ta = min(lane >> 2, W - 1), tb = min(lane & 3, W - 1);
  const bool idle = (lane >> 2) >= W || (lane & 3) >= W;
  const int lofs = ta * IRS + tb * IREG;
  const double ih = 1.0 / g.h;
  const TA tih = (TA)ih;
  const int org = ax == 0 ? o0 : (ax == 1 ? o1 : o2);
  const int na = ax == 0 ? g.n0 : (ax == 1 ? g.n1 : g.n2);
  const bool wall = (ax == 0 ? g.bc0 : (ax == 1 ? g.bc1 : g.bc2)) != 0;
  const int stride = ax == 0 ? IRS : (ax == 1 ? IREG : 1);
  for (int c0 = s0; c0 < s1; c0 += IPTS * gridDim.y) {
    const int np = min(IPTS, s1 - c0);
    if (c0 != s0) {
      __syncthreads();
      if (spt < np) xv = X[3 * (c0 + spt) + ax];
    }
    if (spt < np) {
      TA wv[4];
      const int i0 = axis_weights<KER, TA>(xv, ih, st == 0, wv);
      // a wall face (index 0 along a wall axis) carries no gradient: zero its weight
      if (MODE == 1 && st == 0 && wall) {
#pragma unroll
        for (int t = 0; t < 4; ++t) wv[t] = i0 + t == 0 ? TA(0) : wv[t];
      }
      int l0 = i0 - org;
      if (!wall && (unsigned)l0 >= IREG) l0 = wrapi(l0 + na / 2, na) - na / 2;
      // a face difference (MODE 1) also reads the node below the support
      constexpr int hi = IREG - W;
      const int lo = MODE == 1 && st == 0 ? 1 : 0;
      if (l0 < lo || l0 > hi) {
        // a point outside its tile (beyond a wall): the nodes that the region
        // holds keep their weights, the others carry nothing
        const int lc = min(max(l0, lo), hi), sh = lc - l0;
        TA nw[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          TA v = TA(0);
#pragma unroll
          for (int q = 0; q < W; ++q) v = t + sh == q ? wv[q] : v;
          nw[t] = v;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) wv[t] = nw[t];
        l0 = lc;
      }
      pb[spt][ax][st] = l0 * stride;
#pragma unroll
      for (int t = 0; t < 4; ++t) pw[spt][ax][st][t] = wv[t];
    }
    __syncthreads();
    for (int pt = threadIdx.x >> 4; pt < np; pt += 16) {
      TA acc[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int sx = d == 0 ? 0 : 1, sy = d == 1 ? 0 : 1, sz = d == 2 ? 0 : 1;
        const TA *R = reg[MODE == 0 ? d : 0] + pb[pt][0][sx] + pb[pt][1][sy] + pb[pt][2][sz] + lofs;
        const TA *wz = pw[pt][2][sz];
        const TA wab = idle ? TA(0) : pw[pt][0][sx][ta] * pw[pt][1][sy][tb];
        TA s = TA(0);
#pragma unroll
        for (int c = 0; c < W; ++c) {
          const TA v = MODE == 0 ? R[c] : (R[c] - R[c - (d == 0 ? IRS : (d == 1 ? IREG : 1))]) * tih;
          s = fma(wab * wz[c], v, s);
        }
        acc[d] = sum16(s);
      }
      if (lane < 3) {
        const long long o = 3LL * (c0 + pt) + lane;
        const double v = (double)(lane == 0 ? acc[0] : (lane == 1 ? acc[1] : acc[2]));
        out[o] = fma(alpha, v, y ? beta * y[o] : 0.0);
      }
    }
  }
}
// Workgroups per point tile: enough for two rounds of the chip's 1024 resident
// ones where tiles are few, without splitting where the tiles fill it.
static dim3 interp_grid(int ntiles) {
  int parts = 2048 / ntiles;
  parts = parts < 1 ? 1 : (parts > 8 ? 8 : parts);
  return dim3(ntiles, parts);
}

template <typename T>
hipError_t interp_grad(int ker, const Geo &g, int nt1, int nt2, int ntiles_nz, const int *tiles, const int *tstart,
                       const double *X, const T *z, double alpha, const double *y, double beta, double *out,
                       hipStream_t s, bool f32) {
  // positions read, results written (and y read), the cells of the support band (T each)
  ProbeExt probe_(PR_INTERP_GRAD, s,
                    (double)probe_points() * (beta != 0.0 ? 72 : 48) + (double)probe_band_cells() * sizeof(T));
  if (ntiles_nz == 0) return hipSuccess;
  if (f32 && sizeof(T) != sizeof(float)) return hipErrorInvalidValue;
  dim3 gr = interp_grid(ntiles_nz), bl(256);
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
#define INTERP(K_, A_)                                                                                             \
  hipExtLaunchKernelGGL((k_interp<K_, 1, T, A_>), gr, bl, 0, s, e0, e1, 0, g, nt1, nt2, tiles, tstart, X, z, alpha, y, \
                        beta, out)
  if (ker == KER_PESKIN4) {
    if (f32) INTERP(KER_PESKIN4, float);
    else INTERP(KER_PESKIN4, double);
  } else {
    if (f32) INTERP(KER_ROMA3, float);
    else INTERP(KER_ROMA3, double);
  }
#undef INTERP
  return hipGetLastError();
}
template hipError_t interp_grad<float>(int, const Geo &, int, int, int, const int *, const int *, const double *,
                                       const float *, double, const double *, double, double *, hipStream_t, bool);
template hipError_t interp_grad<double>(int, const Geo &, int, int, int, const int *, const int *, const double *,
                                        const double *, double, const double *, double, double *, hipStream_t, bool);

hipError_t interp_face(int ker, const Geo &g, int nt1, int nt2, int ntiles_nz, const int *tiles, const int *tstart,
                       const double *X, const double *u3, double alpha, const double *y, double beta, double *out,
                       hipStream_t s) {
  // positions read, results written (and y read), three face components of the support band
  ProbeScope probe_(PR_INTERP_FACE, s,
                    (double)probe_points() * (beta != 0.0 ? 72 : 48) + (double)probe_band_cells() * 3 * 8);
  if (ntiles_nz == 0) return hipSuccess;
  dim3 gr = interp_grid(ntiles_nz), bl(256);
  if (ker == KER_PESKIN4)
    hipLaunchKernelGGL((k_interp<KER_PESKIN4, 0, double, double>), gr, bl, 0, s, g, nt1, nt2, tiles, tstart, X, u3, alpha,
                       y, beta, out);
  else
    hipLaunchKernelGGL((k_interp<KER_ROMA3, 0, double, double>), gr, bl, 0, s, g, nt1, nt2, tiles, tstart, X, u3, alpha, y,
                       beta, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Touch lists.  Tile T owns the cells 4T..4T+3 per axis; for velocity
// component d its face box also holds the upper face 4T+4 along d (needed by
// the divergence of its last cell).  A point touches T when its support meets
// that box for some component.  Lists are built once per placement: count
// per tile, scan, then fill per tile.

// Range of tiles touched along one axis (union over the components).
template <int KER>
__device__ __forceinline__ void touch_range(double x, double ih, int &lo, int &hi) {
  constexpr int W = KerWidth<KER>::W;
  double s;
  int f0 = support_start<KER>(x, ih, true, s);   // face nodes along this axis
  int c0 = support_start<KER>(x, ih, false, s);  // centre nodes
  auto fdiv = [](int a) { return a >= 0 ? a / 4 : -((-a + 3) / 4); };
  lo = min(fdiv(f0 - 1), fdiv(c0));
  hi = max(fdiv(f0 + W - 1), fdiv(c0 + W - 1));
}

// Touch lists built tile by tile, without atomics: the 64 lanes of a
// wavefront walk the points of the neighbouring point tiles of tile t (home
// tiles within one tile along each axis, wrapped on periodic axes; a point's
// support never reaches further) in a fixed order (neighbour offsets in
// lexicographic order, sorted points within a tile) and keep those whose
// support touches t.  PASS 0 writes the count of every tile; PASS 1 writes the
// lists of the active tiles by ordered wavefront compaction, so every list
// has the same order on every run.
template <int KER, int PASS>
__global__ void __launch_bounds__(256) k_touch_tile(Geo g, int nt0, int nt1, int nt2, int ntl, const int *ntl_dev,
                                                    const int *tiles, const int *tstart, const double *X,
                                                    int *counts, const int *lstart, int *list) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int w = blockIdx.x * 4 + wave;
  if (w >= ntl || (ntl_dev && w >= *ntl_dev)) return;
  const int t = tiles ? tiles[w] : w;
  const int nt[3] = {nt0, nt1, nt2}, bc[3] = {g.bc0, g.bc1, g.bc2};
  const int tc[3] = {t / (nt1 * nt2), (t / nt2) % nt1, t % nt2};
  int nb[3][3], nn[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    nn[a] = 0;
    for (int sft = -1; sft <= 1; ++sft) {
      int v = tc[a] + sft;
      if (v < 0 || v >= nt[a]) {
        if (bc[a]) continue;
        v = wrapi(v, nt[a]);
      }
      bool dup = false;
      for (int q = 0; q < nn[a]; ++q) dup = dup || nb[a][q] == v;
      if (!dup) nb[a][nn[a]++] = v;
    }
  }
  const double ih = 1.0 / g.h;
  const unsigned long long below = (1ull << lane) - 1ull;
  const int base = PASS ? lstart[t] : 0;
  int cnt = 0;
  for (int q0 = 0; q0 < nn[0]; ++q0)
    for (int q1 = 0; q1 < nn[1]; ++q1)
      for (int q2 = 0; q2 < nn[2]; ++q2) {
        const int n = (nb[0][q0] * nt1 + nb[1][q1]) * nt2 + nb[2][q2];
        const int p0 = tstart[n], p1 = tstart[n + 1];
        for (int pb = p0; pb < p1; pb += 64) {
          const int p = pb + lane;
          bool hit = false;
          if (p < p1) {
            hit = true;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
              int lo, hi;
              touch_range<KER>(X[3 * p + a], ih, lo, hi);
              bool in = false;
              for (int v = lo; v <= hi; ++v) {
                int u = v;
                if (u < 0 || u >= nt[a]) {
                  if (bc[a]) continue;
                  u = wrapi(u, nt[a]);
                }
                in = in || u == tc[a];
              }
              hit = hit && in;
            }
          }
          const unsigned long long m = __ballot(hit);
          if (PASS == 1 && hit) list[base + cnt + __popcll(m & below)] = p;
          cnt += __popcll(m);
        }
      }
  if (PASS == 0 && lane == 0) counts[t] = cnt;
}

hipError_t touch_tiles(int ker, const Geo &g, int nt0, int nt1, int nt2, int ntl, const int *ntl_dev,
                       const int *tiles, const int *tstart, const double *X, int *counts, const int *lstart,
                       int *list, hipStream_t s) {
  if (ntl == 0) return hipSuccess;
  const dim3 gr((ntl + 3) / 4), bl(256);
  if (list == nullptr) {
    if (ker == KER_PESKIN4)
      hipLaunchKernelGGL((k_touch_tile<KER_PESKIN4, 0>), gr, bl, 0, s, g, nt0, nt1, nt2, ntl, ntl_dev, tiles,
                         tstart, X, counts, lstart, list);
    else
      hipLaunchKernelGGL((k_touch_tile<KER_ROMA3, 0>), gr, bl, 0, s, g, nt0, nt1, nt2, ntl, ntl_dev, tiles, tstart,
                         X, counts, lstart, list);
  } else {
    if (ker == KER_PESKIN4)
      hipLaunchKernelGGL((k_touch_tile<KER_PESKIN4, 1>), gr, bl, 0, s, g, nt0, nt1, nt2, ntl, ntl_dev, tiles,
                         tstart, X, counts, lstart, list);
    else
      hipLaunchKernelGGL((k_touch_tile<KER_ROMA3, 1>), gr, bl, 0, s, g, nt0, nt1, nt2, ntl, ntl_dev, tiles, tstart,
                         X, counts, lstart, list);
  }
  return hipGetLastError();
}

// Flag the tiles within one tile (per axis, wrapped on periodic axes) of the
// n non-empty point tiles: the only tiles a point's support can reach.  Every
// writer stores the same value 1.
__global__ void k_mark_near(Geo g, int nt0, int nt1, int nt2, int n, const int *nz, int *flags) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= 27 * n) return;
  const int t = nz[q / 27], o = q % 27;
  const int nt[3] = {nt0, nt1, nt2}, bc[3] = {g.bc0, g.bc1, g.bc2};
  const int tc[3] = {t / (nt1 * nt2), (t / nt2) % nt1, t % nt2};
  const int off[3] = {o / 9 - 1, (o / 3) % 3 - 1, o % 3 - 1};
  int v[3];
  for (int a = 0; a < 3; ++a) {
    v[a] = tc[a] + off[a];
    if (v[a] < 0 || v[a] >= nt[a]) {
      if (bc[a]) return;
      v[a] = wrapi(v[a], nt[a]);
    }
  }
  flags[(v[0] * nt1 + v[1]) * nt2 + v[2]] = 1;
}
hipError_t mark_near(const Geo &g, int nt0, int nt1, int nt2, int n, const int *nz, int *flags, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_mark_near, dim3(nblk(27LL * n, 256)), dim3(256), 0, s, g, nt0, nt1, nt2, n, nz, flags);
  return hipGetLastError();
}

// Launch order of a tile list (one workgroup, counting sort).  The
// dispatcher deals consecutive workgroups round-robin to the 8 XCDs, each
// with its own L2: the list (in tile-index order, i.e. spatially sorted) is
// cut into ORD_X contiguous chunks and chunk c is dealt to the workgroups
// c, c + 8, c + 16, ..., so the neighbouring tiles that share points and
// halo cells run on one XCD and find them in its L2.  Within a chunk the
// tiles go in order of decreasing list length (the workgroups with the most
// work start first, which shortens the tail).  out has ORD_X * ceil(n /
// ORD_X) entries; -1 marks the holes of a short last chunk (those
// workgroups exit).  Each tile's result does not depend on the order, which
// within a length bucket is arbitrary.
constexpr int ORD_T = 1024, ORD_B = 256, ORD_X = 8;
__global__ void __launch_bounds__(ORD_T) k_order_active(int n, const int *active, const int *lstart, int *out) {
  __shared__ int cnt[ORD_X * ORD_B], base[ORD_X * ORD_B];
  const int t = threadIdx.x;
  const int cs = (n + ORD_X - 1) / ORD_X;
  for (int b = t; b < ORD_X * ORD_B; b += ORD_T) cnt[b] = 0;
  for (int i = t; i < ORD_X * cs; i += ORD_T) out[i] = -1;
  __syncthreads();
  auto key = [&](int i) {
    const int a = active[i];
    return (i / cs) * ORD_B + ORD_B - 1 - min(lstart[a + 1] - lstart[a], ORD_B - 1);
  };
  for (int i = t; i < n; i += ORD_T) atomicAdd(&cnt[key(i)], 1);
  __syncthreads();
  if (t < ORD_X) {
    int acc = 0;  // position within chunk t
    for (int b = 0; b < ORD_B; ++b) {
      base[t * ORD_B + b] = acc;
      acc += cnt[t * ORD_B + b];
    }
  }
  __syncthreads();
  for (int i = t; i < n; i += ORD_T) out[atomicAdd(&base[key(i)], 1) * ORD_X + i / cs] = active[i];
}
int order_launch_count(int n) { return ORD_X * ((n + ORD_X - 1) / ORD_X); }
hipError_t order_active(int n, const int *active, const int *lstart, int *out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_order_active, dim3(1), dim3(ORD_T), 0, s, n, active, lstart, out);
  return hipGetLastError();
}

__global__ void k_positive(int n, const int *counts, int *flags, int2 *clear) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  flags[t] = counts[t] > 0;
  if (clear) clear[t] = make_int2(0, 0);
}
hipError_t positive_flags(int n, const int *counts, int *flags, hipStream_t s, int2 *clear) {
  hipLaunchKernelGGL(k_positive, dim3(nblk(n, 256)), dim3(256), 0, s, n, counts, flags, clear);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Spreading on one active tile from its touch list.
//
// Staging: a chunk of listed points at a time, one task per (point, axis)
// computing the face- and centre-node weights of that axis (one square root
// each) and laying them out over the tile's own positions along the axis: 5
// face and 4 centre positions, zero outside the point's support, once for all
// three components.  The weights get to their positions by a shift in two
// selections (by one, then by 0, +-2 or +-4 positions).
//
// Accumulation: lane l < 30 of every half-wavefront owns two neighbouring
// z-columns (same x, consecutive y) of a face box (component 0: 5 x 4
// columns of 4 faces, component 1: 4 x 5 columns of 4 faces, component 2:
// 4 x 4 columns of 5 faces).  Half-wavefront h (0..7) adds the listed points
// h, h+8, h+16, ... in list order into registers, with no branch:
// q_d w_x[ci] w_y[cj] times the five z weights of the column (zeros add
// nothing); the x and z weights serve both columns, so a lane reads 9 LDS
// values per point for 10 products.  The eight partial sums of a face are
// added in a fixed order, so every grid value is summed in the same order
// on every run.
//
// PIPE: three further wavefronts stage the next chunk while four accumulate
// the current one (two LDS buffers, one barrier per chunk).  Otherwise the
// four stage a chunk, then accumulate it: twice the workgroups per compute
// unit, each slower.
//
// Bounded by vector instructions and LDS reads about equally.  With each
// weight stored once per axis, at its position, for all components (it was
// selected, multiplied and stored for each), 1.3 million pairs of point and
// tile at 256^3 take 21.5 instead of 24.0 million vector instructions and 11.3
// instead of 13.1 million LDS cycles: 39.2 -> 35.6 us in float32, 67.7 -> 60.1
// in float64; with PIPE, 81000 pairs in 392 tiles at 64^3, 22.3 -> 15.0 and
// 26.5 -> 19.2 us.  What is left are the products with the zeros around the
// supports (five in six); skipping them would cost more selections.
constexpr int BAND_ACC = 256, BAND_PIPE = 192;  // accumulating threads, further ones of PIPE
// Values per point: for each axis the 5 face positions, the value q of the
// component, two unused, and from BAND_C the 4 centre positions, each group on
// a 16-byte boundary.  The two points that a wavefront reads at once are four
// apart, 16 modulo 32 values, and so fall on distinct LDS banks.
constexpr int BAND_Q = 5, BAND_C = 8, BAND_AX = 12, BAND_WS = 3 * BAND_AX;

template <typename TA>
struct alignas(16) Vec4 {
  TA v[4];
};

// v[i] = w[i - d] for the N positions i, 0 outside w[0..3]
template <int N, typename TA>
__device__ __forceinline__ void band_positions(const TA w[4], int d, TA v[N]) {
  const bool odd = d & 1;
  const int e = d >> 1;
  TA c[5];  // w shifted by d & 1
  c[0] = odd ? TA(0) : w[0];
#pragma unroll
  for (int t = 1; t < 4; ++t) c[t] = odd ? w[t - 1] : w[t];
  c[4] = odd ? w[3] : TA(0);
#pragma unroll
  for (int t = 0; t < N; ++t) {
    TA x = e == 0 ? c[t] : TA(0);
#pragma unroll
    for (int u = -2; u <= 2; ++u)
      if (u != 0 && t - 2 * u >= 0 && t - 2 * u < 5) x = e == u ? c[t - 2 * u] : x;
    v[t] = x;
  }
}

template <int KER, bool DIV, bool PIPE, typename TA, typename TO>
__global__ void __launch_bounds__(BAND_ACC + (PIPE ? BAND_PIPE : 0))
    k_band(Geo g, int nt1, int nt2, const int *active, const int *lstart, const int *list, const double *X,
           const double *q, double alpha, TO *out) {
  // TA: the weights' and sums' type (float64, or float32 for the S~ products
  // of the float32 Krylov cycle).  BAND_CH listed points per chunk: a multiple
  // of the 8 half-wavefronts that leaves LDS for four (PIPE) or eight
  // workgroups on a compute unit
  constexpr int BAND_CH = 64;
  // after the last chunk the same LDS holds the per-half-wavefront face sums part[8][3][80]
  static_assert(8 * 3 * 80 <= (PIPE ? 2 : 1) * BAND_CH * BAND_WS, "face sums must fit the weight buffers");
  __shared__ __attribute__((aligned(16))) TA wts[(PIPE ? 2 : 1) * BAND_CH * BAND_WS + 4];  // + room for a fifth z position
  TA(*part)[3][80] = reinterpret_cast<TA(*)[3][80]>(wts);
  const int tile = active[blockIdx.x];
  if (tile < 0) return;  // a hole of the launch order
  const int T2 = tile % nt2, r = tile / nt2, T1 = r % nt1, T0 = r / nt1;
  const int tid = threadIdx.x;
  const int s0 = lstart[tile], s1 = lstart[tile + 1];
  const double ih = 1.0 / g.h;
  const int nchunk = (s1 - s0 + BAND_CH - 1) / BAND_CH;
  // Staging task: axis a of listed point cand of every chunk, and the point's
  // value q_a.  Its operands are loaded one chunk ahead and its list entry two
  // chunks ahead (the load of a position depends on it).
  static_assert(3 * BAND_CH <= BAND_PIPE && BAND_PIPE <= BAND_ACC, "one staging task per thread");
  const int task = PIPE ? tid - BAND_ACC : tid, cand = task / 3, a = task - 3 * cand;
  const bool stager = task >= 0 && cand < BAND_CH;
  const int orga = a == 0 ? 4 * T0 : (a == 1 ? 4 * T1 : 4 * T2), na = a == 0 ? g.n0 : (a == 1 ? g.n1 : g.n2);
  const bool per = (a == 0 ? g.bc0 : (a == 1 ? g.bc1 : g.bc2)) == 0;
  int p_cur = -1, p_nxt = -1;
  double xa = 0.0, qa = 0.0;
  auto entry = [&](int k) {
    const int c = s0 + k * BAND_CH + cand;
    return (stager && c < s1) ? list[c] : -1;
  };
  auto operands = [&](int p) {
    const int pc = p >= 0 ? p : 0;  // every list here is non-empty, so point 0 exists
    xa = X[3 * pc + a];
    qa = q[3 * pc + a];
  };
  auto stage_first = [&]() {
    p_cur = entry(0);
    operands(p_cur);
    p_nxt = entry(1);
  };
  // chunk k into the LDS buffer
  auto stage = [&](int k, TA *buf) {
    if (p_cur >= 0) {
      TA wf[4], wc[4], F[5], C[4];
      int lf = axis_weights<KER, TA>(xa, ih, true, wf) - orga;
      int lc = axis_weights<KER, TA>(xa, ih, false, wc) - orga;
      // periodic image of the support start in [-4, n - 4): every offset
      // that reaches the box (-3 .. its last position) keeps its value,
      // and no image of another can reach it, for any n >= 16
      if (per && (lf < -4 || lf >= na - 4)) lf = wrapi(lf + 4, na) - 4;
      if (per && (lc < -4 || lc >= na - 4)) lc = wrapi(lc + 4, na) - 4;
      band_positions<5>(wf, lf, F);
      band_positions<4>(wc, lc, C);
      TA *row = buf + cand * BAND_WS + BAND_AX * a;
#pragma unroll
      for (int t = 0; t < 5; ++t) row[t] = F[t];
      row[BAND_Q] = (TA)qa;
#pragma unroll
      for (int t = 0; t < 4; ++t) row[BAND_C + t] = C[t];
    }
    p_cur = p_nxt;
    operands(p_cur);
    p_nxt = entry(k + 2);
  };
  // Accumulation: each half-wavefront takes every 8th listed point; lane hl
  // of a half owns, for component cd, the x position ci and the two y
  // positions cj0, cj0 + 1 (the second absent at the odd end of a 5-wide box)
  // of a pair of face columns, nf faces along z: 30 of the 32 lanes.
  const int wv = tid >> 6, lane = tid & 63, hl = lane & 31;
  const int slot = wv + 4 * (lane >> 5);
  const int cd = hl < 10 ? 0 : (hl < 22 ? 1 : 2);
  const int cl = hl - (cd == 0 ? 0 : (cd == 1 ? 10 : 22));
  const int cli = cd == 1 ? cl / 3 : cl / 2;  // column pairs along y: 2, 3, 2
  const int cby = cd == 1 ? 5 : 4;            // columns along y in this component's box
  const int ci = min(cli, 4), cj0 = 2 * (cl - (cd == 1 ? 3 : 2) * cli);
  const bool has1 = cj0 + 1 < cby;
  const int nf = cd == 2 ? 5 : 4;
  const bool owner = hl < 30;
  // this lane's weights in a point's row: x position ci, first y position, z positions
  const int wxo = (cd == 0 ? 0 : BAND_C) + ci, wyo = BAND_AX + (cd == 1 ? 0 : BAND_C) + cj0,
            wzo = 2 * BAND_AX + (cd == 2 ? 0 : BAND_C), wqo = BAND_AX * cd + BAND_Q;
  TA acc0[5] = {TA(0), TA(0), TA(0), TA(0), TA(0)}, acc1[5] = {TA(0), TA(0), TA(0), TA(0), TA(0)};
  auto accumulate = [&](int k, const TA *buf) {
    const int nc = min(BAND_CH, s1 - s0 - k * BAND_CH);
#pragma unroll 2
    for (int c = slot; c < nc; c += 8) {
      const TA *W = buf + c * BAND_WS;
      const TA wx = W[wxo] * W[wqo];
      const TA wab0 = wx * W[wyo];
      // without a second column (has1 false), and at a fifth z position
      // that the component has not, the lane reads what lies behind, for
      // sums that are never stored
      const TA wab1 = wx * W[wyo + 1];
      TA wz[5];
      *(Vec4<TA> *)wz = *(const Vec4<TA> *)(W + wzo);
      wz[4] = W[wzo + 4];
#pragma unroll
      for (int fk = 0; fk < 5; ++fk) {
        acc0[fk] += wab0 * wz[fk];
        acc1[fk] += wab1 * wz[fk];
      }
    }
  };
  if (PIPE) {
    if (tid >= BAND_ACC) {
      stage_first();
      for (int k = 0; k < nchunk; ++k) {
        stage(k, wts + (k & 1) * (BAND_CH * BAND_WS));
        __syncthreads();  // chunk k is staged, and chunk k - 1 accumulated
      }
    } else {
      for (int k = 0; k < nchunk; ++k) {
        __syncthreads();
        accumulate(k, wts + (k & 1) * (BAND_CH * BAND_WS));
      }
    }
    __syncthreads();
  } else {
    stage_first();
    for (int k = 0; k < nchunk; ++k) {
      stage(k, wts);
      __syncthreads();
      accumulate(k, wts);
      __syncthreads();
    }
  }
  if (tid < BAND_ACC && owner) {
    // face box index: (ci * by + cj) * bz + fk with by = 4 or 5, bz = 4 or 5
    const int bz = cd == 2 ? 5 : 4;
#pragma unroll
    for (int fk = 0; fk < 5; ++fk) {
      if (fk < nf) {
        part[slot][cd][(ci * cby + cj0) * bz + fk] = acc0[fk];
        if (has1) part[slot][cd][(ci * cby + cj0 + 1) * bz + fk] = acc1[fk];
      }
    }
  }
  __syncthreads();
  const long long N = 2 * g.half;
  // the eight partial sums of each face, in order; left in part[0]
  if (tid < 240) {
    TA *f0 = &part[0][0][0] + tid, f = *f0;
#pragma unroll
    for (int h = 1; h < 8; ++h) f += f0[240 * h];
    *f0 = f;
  }
  __syncthreads();
  auto face = [&](int d, int idx) { return part[0][d][idx]; };
  if (DIV) {
    if (tid < 64) {
      int ci2 = tid >> 4, cj2 = (tid >> 2) & 3, ck = tid & 3;
      TA dv = TA(0);
      dv += face(0, ((ci2 + 1) * 4 + cj2) * 4 + ck) - face(0, (ci2 * 4 + cj2) * 4 + ck);
      dv += face(1, (ci2 * 5 + cj2 + 1) * 4 + ck) - face(1, (ci2 * 5 + cj2) * 4 + ck);
      dv += face(2, (ci2 * 4 + cj2) * 5 + ck + 1) - face(2, (ci2 * 4 + cj2) * 5 + ck);
      int gi = 4 * T0 + ci2, gj = 4 * T1 + cj2, gk = 4 * T2 + ck;
      const long long o = sidx(g, gi, gj, gk);
      out[o] = (TO)((double)out[o] + alpha * (double)dv * ih);
    }
  } else {
    if (tid < 192) {
      int d = tid >> 6, t = tid & 63;
      int fi = t >> 4, fj = (t >> 2) & 3, fk = t & 3;
      int by = 4 + (d == 1), bz = 4 + (d == 2);
      int gi = 4 * T0 + fi, gj = 4 * T1 + fj, gk = 4 * T2 + fk;
      const long long o = d * N + sidx(g, gi, gj, gk);
      out[o] = (TO)((double)out[o] + alpha * (double)face(d, (fi * by + fj) * bz + fk));
    }
  }
}

// PIPE up to the tiles that are resident at once, four workgroups on each of
// 256 compute units; beyond that throughput counts.  Without and with, by the
// same staging: 392 tiles 20.6 and 15.7 us, 4456 tiles 40.8 and 51.6 us.
constexpr int BAND_PIPE_TILES = 1024;

template <typename TO>
static hipError_t band_launch(int ker, bool div, const Geo &g, int nt1, int nt2, int nactive, const int *active,
                              const int *lstart, const int *list, const double *X, const double *q, double alpha,
                              TO *out, hipStream_t s, bool f32) {
  // positions and values read, the active tiles' cells (div) or faces read and written
  ProbeExt probe_(div ? PR_BAND_DIV : PR_BAND_FACE, s,
                    (double)probe_points() * 48 + (double)probe_band_cells() * (div ? 1 : 3) * 2 * sizeof(TO));
  if (nactive == 0) return hipSuccess;
  const bool pipe = nactive <= BAND_PIPE_TILES;
  const dim3 gr(nactive), bl(BAND_ACC + (pipe ? BAND_PIPE : 0));
  hipEvent_t e0, e1;
  probe_ext_take(&e0, &e1);
#define BAND(K_, D_, A_)                                                                                        \
  do {                                                                                                          \
    if (pipe)                                                                                                   \
      hipExtLaunchKernelGGL((k_band<K_, D_, true, A_, TO>), gr, bl, 0, s, e0, e1, 0, g, nt1, nt2, active,       \
                            lstart, list, X, q, alpha, out);                                                    \
    else                                                                                                        \
      hipExtLaunchKernelGGL((k_band<K_, D_, false, A_, TO>), gr, bl, 0, s, e0, e1, 0, g, nt1, nt2, active,      \
                            lstart, list, X, q, alpha, out);                                                    \
  } while (0)
  if (f32) {
    if (!div) return hipErrorInvalidValue;  // float32 sums serve the S~ products only
    if (ker == KER_PESKIN4) BAND(KER_PESKIN4, true, float);
    else BAND(KER_ROMA3, true, float);
  } else if constexpr (sizeof(TO) == sizeof(double)) {
    if (ker == KER_PESKIN4) {
      if (div) BAND(KER_PESKIN4, true, double);
      else BAND(KER_PESKIN4, false, double);
    } else {
      if (div) BAND(KER_ROMA3, true, double);
      else BAND(KER_ROMA3, false, double);
    }
  } else {
    return hipErrorInvalidValue;  // a float32 output takes float32 sums
  }
#undef BAND
  return hipGetLastError();
}
hipError_t band_apply(int ker, bool div, const Geo &g, int nt1, int nt2, int nactive, const int *active,
                      const int *lstart, const int *list, const double *X, const double *q, double alpha,
                      double *out, hipStream_t s, bool f32) {
  return band_launch(ker, div, g, nt1, nt2, nactive, active, lstart, list, X, q, alpha, out, s, f32);
}
hipError_t band_apply(int ker, bool div, const Geo &g, int nt1, int nt2, int nactive, const int *active,
                      const int *lstart, const int *list, const double *X, const double *q, double alpha,
                      float *out, hipStream_t s, bool f32) {
  return band_launch(ker, div, g, nt1, nt2, nactive, active, lstart, list, X, q, alpha, out, s, f32);
}

}  // namespace ibs
