// Exact pseudo-inverse of the pressure Laplacian by fast diagonalisation in
// float64: the direct solve of paper Sec. 4.2 (Lynch et al.), which factors
// L once and applies L^-1 exactly in every Krylov iteration.
//
// L = Lx (x) I (x) I + I (x) Ly (x) I + I (x) I (x) Lz is a Kronecker sum of
// 1-D second-difference matrices, each diagonalised by an orthonormal
// eigenbasis Q_a with eigenvalues lambda_a.  So
//     L^+ v = Q diag(1 / (lx + ly + lz)) Q^T v,   Q = Qx (x) Qy (x) Qz,
// with the constant mode (all three eigenvalues zero) mapped to zero.  Q^T v
// and Q w are three mode products each: the n x n matrix applied along one
// axis of the n0 x n1 x n2 array.
//
// The bases are taken about the middle of the axis (walls: the DCT-II
// vectors; periodic: cosines and sines of 2 pi k (i + 1/2) / n), so that every
// vector is even or odd under i -> n - 1 - i, n/2 of each.  With the sums and
// differences of the mirrored entries a product of size n is two of size
// n/2, half the multiplications: the even modes see in[m] + in[n-1-m], the
// odd ones in[m] - in[n-1-m], and back, out[m] and out[n-1-m] are the sum and
// the difference of the even and the odd part.  A transformed axis holds its
// even modes first.  The products are dense matrix products in float64 on the
// matrix cores (n N flops each, 6 n N per application).
#include <math.h>

#include <vector>

#include "internal.h"

namespace ibs {

constexpr int MP_Q = 32;   // output tile: 32 entries of either half x 64 lines
constexpr int MP_L = 64;
constexpr int MP_K = 8;    // summation step
constexpr int MP_SM = 48;  // LDS stride of a step's matrix rows, and of its rows of lines: rows kk and kk + 1
constexpr int MP_SX = 80;  //   of a wavefront's operand on different banks
constexpr int MP_SZ = 10;  // LDS stride of the lines of a step along the contiguous axis

typedef double V4 __attribute__((ext_vector_type(4)));

// Mode product along one axis of an array viewed as [P][n][R], h = n / 2:
//   forward:  out[p][q], out[p][h + q] = sum_{m < h} A_even[m][q] (in[m] + in[n-1-m]), A_odd[m][q] (in[m] - in[n-1-m])
//   back:     out[p][m], out[p][n-1-m] = E +- O,  E = sum_{q < h} A_even[q][m] in[q],  O = sum A_odd[q][m] in[h + q]
// A: the even half matrix, then the odd one, h x h row-major.
// MP_F_ROW, MP_B_ROW: an axis above the contiguous one (R > 1).  MP_F_Z,
// MP_B_Z: the contiguous axis (R == 1; a line is the row in[p][0..n), the tile
// runs over 64 of them), read from (forward) or written to (back) the
// red/black split layout, so that an application starts and ends there
// without conversion passes.  With lx (x transform only, P == 1) the result
// is scaled by 1 / (lx[k] + ly[j] + lz[i]) for line r = j n2 + i, and the
// all-zero mode set to 0.
//
// Four wavefronts, each 16 entries of both halves x 32 lines as 2 x 2 matrix
// products of 16 x 16 x 4 (v_mfma_f64_16x16x4: lane l holds A[l % 16][l / 16],
// B[l / 16][l % 16] and D[l / 16 + 4 r][l % 16]); the next step's operands are
// loaded while a step is computed, into the other half of the LDS.  Along
// the contiguous axis the lines are the product's rows, so that the stores
// run along the transformed index.  The workgroups of a line tile follow each
// other on one XCD and find its lines in that XCD's L2.
//
// Bound by memory and its latency (a product reads and writes the grid): at
// 128 x 128 x 192 a product along 128 cells takes 15 to 17 us (50 MB, 3.1
// TB/s; the matrix cores are busy 5 us), one along the contiguous 192 cells
// 22; with the unfolded n x n matrices 23 and 30, on the vector units 38 and
// 56 with two more layout passes.  Summation steps loaded two ahead: 24.5 us
// where one ahead takes 23.
enum { MP_F_ROW = 0, MP_B_ROW = 1, MP_F_Z = 2, MP_B_Z = 3 };

template <int MODE>
__global__ void __launch_bounds__(256, 4) k_mode(const double *__restrict__ A, const double *__restrict__ in,
                                                 double *__restrict__ out, int n, int nk, long long ntiles,
                                                 long long P, long long R, const double *__restrict__ lx,
                                                 const double *__restrict__ ly, const double *__restrict__ lz, int n1,
                                                 int n2, long long half) {
  constexpr bool Z = MODE == MP_F_Z || MODE == MP_B_Z, FWD = MODE == MP_F_ROW || MODE == MP_F_Z;
  __shared__ __align__(16) double Ms[2][2][MP_K * MP_SM];                     // [half][sum index][entry]
  __shared__ __align__(16) double Xs[2][2][Z ? MP_L * MP_SZ : MP_K * MP_SX];  // [half][line][sum index] or [sum index][line]
  const int h = n >> 1;
  // block -> (line tile, entry tile): consecutive blocks go round-robin to the
  // 8 XCDs, so an XCD takes the nk entry tiles of one line tile in turn
  const long long slot = blockIdx.x >> 3, lt = (slot / nk) * 8 + (blockIdx.x & 7);
  if (lt >= ntiles) return;
  const int k0 = (int)(slot % nk) * MP_Q;
  const long long rt = (R + MP_L - 1) / MP_L;                           // line tiles of one p
  const long long p = Z ? 0 : lt / rt, l0 = (Z ? lt : lt % rt) * MP_L;  // first line (r, or p along the contiguous axis)
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int lg = lane >> 4, ln = lane & 15;
  const int wk = 16 * (wave & 1), wl = 32 * (wave >> 1);  // this wavefront's corner of the tile
  // loads of one step: a pair of matrix entries (row mr, columns mc of half
  // mh) and two pairs of lines' values: row mr and its partner (the mirrored
  // row, or that of the odd half) at lines c, or along the contiguous axis
  // entries zm and their partners of line zl
  const int mr = tid >> 5, mh = (tid >> 4) & 1, mc = 2 * (tid & 15), c = 2 * (tid & 31);
  const int zl = tid >> 2, zm = 2 * (tid & 3);
  const double *mp = A + (long long)mh * h * h + (long long)mr * h + k0 + mc, *xa, *xb;
  bool okx, swap = false;
  if (!Z) {
    okx = l0 + c < R;
    xa = in + (p * n + mr) * R + l0 + c;
    xb = in + (p * n + (FWD ? n - 1 - mr : h + mr)) * R + l0 + c;
  } else {
    const long long line = l0 + zl;
    okx = line < P;
    if (FWD) {
      // entries zm (even), zm + 1 of row line = (i, j), one of each colour;
      // their partners n - 1 - zm (odd), n - 2 - zm
      const int i = (int)(line / n1), j = (int)(line - (long long)i * n1);
      swap = (i + j) & 1;
      xa = in + line * h + (zm >> 1);
      xb = in + line * h + ((n - 2 - zm) >> 1);
    } else {
      xa = in + line * n + zm;
      xb = xa + h;
    }
  }
  // a tile inside the arrays, whole steps: no masks
  const bool full = h % MP_K == 0 && k0 + MP_Q <= h && l0 + MP_L <= (Z ? P : R);
  double2 mreg, ea, eb;
  auto pair = [&](const double *x) -> double2 {
    if (MODE != MP_F_Z) return *(const double2 *)x;
    const double red = x[0], blk = x[half];
    return swap ? make_double2(blk, red) : make_double2(red, blk);
  };
  auto load = [&](int m0) {  // the step that follows the last one loaded
    if (full) {
      mreg = *(const double2 *)mp;
      ea = pair(xa);
      eb = pair(xb);
    } else {
      mreg = ea = eb = make_double2(0.0, 0.0);
      if (m0 + mr < h && k0 + mc < h) mreg = *(const double2 *)mp;
      if (okx && m0 + (Z ? zm : mr) < h) {
        ea = pair(xa);
        eb = pair(xb);
      }
    }
    mp += (long long)MP_K * h;
    const long long step = Z ? (FWD ? MP_K / 2 : MP_K) : MP_K * R;
    xa += step;
    xb += FWD ? -step : step;
  };
  auto store = [&](int b) {
    *(double2 *)&Ms[b][mh][mr * MP_SM + mc] = mreg;
    double2 e = ea, o = eb;
    if (MODE == MP_F_ROW) {
      e = make_double2(ea.x + eb.x, ea.y + eb.y);
      o = make_double2(ea.x - eb.x, ea.y - eb.y);
    } else if (MODE == MP_F_Z) {  // eb holds (n - 2 - m, n - 1 - m)
      e = make_double2(ea.x + eb.y, ea.y + eb.x);
      o = make_double2(ea.x - eb.y, ea.y - eb.x);
    }
    const int at = Z ? zl * MP_SZ + zm : mr * MP_SX + c;
    *(double2 *)&Xs[b][0][at] = e;
    *(double2 *)&Xs[b][1][at] = o;
  };
  V4 acc[2][2];  // [half][line tile]
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[q][j] = V4{0, 0, 0, 0};
  const bool active = k0 + wk < h;
  load(0);
  store(0);
  __syncthreads();
  int b = 0;
  for (int m0 = 0; m0 < h; m0 += MP_K, b ^= 1) {
    const bool more = m0 + MP_K < h;
    if (more) load(m0 + MP_K);
    if (active) {
#pragma unroll
      for (int s = 0; s < MP_K; s += 4)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const double mk = Ms[b][q][(s + lg) * MP_SM + wk + ln];
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int l = wl + 16 * j + ln;
            const double x = Z ? Xs[b][q][l * MP_SZ + s + lg] : Xs[b][q][(s + lg) * MP_SX + l];
            acc[q][j] = Z ? __builtin_amdgcn_mfma_f64_16x16x4f64(x, mk, acc[q][j], 0, 0, 0)
                          : __builtin_amdgcn_mfma_f64_16x16x4f64(mk, x, acc[q][j], 0, 0, 0);
          }
        }
    }
    if (more) {
      store(b ^ 1);
      __syncthreads();
    }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = k0 + wk + (Z ? ln : lg + 4 * r);
      const long long line = l0 + wl + 16 * j + (Z ? lg + 4 * r : ln);
      if (k >= h || line >= (Z ? P : R)) continue;
      double v0 = acc[0][j][r], v1 = acc[1][j][r];
      int k1 = h + k;
      if (!FWD) {
        const double e = v0;
        v0 = e + v1;
        v1 = e - v1;
        k1 = n - 1 - k;
      }
      if (MODE == MP_B_Z) {
        const int gi = (int)(line / n1), gj = (int)(line - (long long)gi * n1);
        double *row = out + line * h;
        row[((gi + gj + k) & 1) * half + (k >> 1)] = v0;
        row[((gi + gj + k1) & 1) * half + (k1 >> 1)] = v1;
      } else if (Z) {
        out[line * n + k] = v0;
        out[line * n + k1] = v1;
      } else {
        if (FWD && lx) {
          const int jj = (int)(line / n2), ii = (int)(line - (long long)jj * n2);
          const double lyz = ly[jj] + lz[ii], lam0 = lx[k] + lyz, lam1 = lx[k1] + lyz;
          v0 = lam0 > 0.0 ? v0 / lam0 : 0.0;
          v1 = lam1 > 0.0 ? v1 / lam1 : 0.0;
        }
        out[(p * n + k) * R + line] = v0;
        out[(p * n + k1) * R + line] = v1;
      }
    }
}

namespace {
template <int MODE>
hipError_t mode(const Geo &g, const double *A, const double *in, double *out, int n, long long P, long long R,
                const double *lx, const double *ly, const double *lz, hipStream_t s) {
  constexpr bool Z = MODE == MP_F_Z || MODE == MP_B_Z;
  const long long tiles = Z ? (P + MP_L - 1) / MP_L : P * ((R + MP_L - 1) / MP_L);
  const int nk = (n / 2 + MP_Q - 1) / MP_Q;
  // the pair loads and the halves: every axis is a multiple of 4
  if (n % 4 || (!Z && R % 4)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_mode<MODE>, dim3((unsigned)(8 * ((tiles + 7) / 8) * nk)), dim3(256), 0, s, A, in, out, n, nk, tiles,
                     P, R, lx, ly, lz, g.n1, g.n2, g.half);
  return hipGetLastError();
}
}  // namespace

size_t fdx_blob_doubles(const int n[3]) {
  return (size_t)n[0] * n[0] + (size_t)n[1] * n[1] + (size_t)n[2] * n[2] + n[0] + n[1] + n[2];
}

// blob: per axis the forward halves A[m][q] (even, odd) and the back ones
// A[q][m], h x h each; then the eigenvalues lx, ly, lz, even modes first.
void fdx_blob_build(const int n[3], const int bc[3], double h, double *blob) {
  const double pi = 3.14159265358979323846, c = 4.0 / (h * h);
  double *lam = blob + (size_t)n[0] * n[0] + (size_t)n[1] * n[1] + (size_t)n[2] * n[2];
  for (int a = 0; a < 3; ++a) {
    const int na = n[a], ha = na / 2;
    const size_t hh = (size_t)ha * ha;
    // a table of one period of the cosine: every argument is a multiple of pi / (2 na)
    std::vector<double> tab(4 * (size_t)na);
    for (int t = 0; t < 4 * na; ++t) tab[t] = cos(pi * t / (2.0 * na));
    for (int odd = 0; odd < 2; ++odd)
      for (int q = 0; q < ha; ++q) {
        // walls: mode 2 q + odd, argument pi mode (i + 1/2) / n; periodic:
        // cos of mode q, sin of mode q + 1, argument 2 pi mode (i + 1/2) / n
        const long long mode = bc[a] ? 2 * q + odd : q + odd;
        const bool flat = bc[a] ? mode == 0 : (mode == 0 || 2 * mode == na);
        const double nrm = 1.0 / sqrt(flat ? (double)na : 0.5 * na);
        for (int m = 0; m < ha; ++m) {
          const long long t = bc[a] ? mode * (2 * m + 1) : 2 * mode * (2 * m + 1) - (odd ? na : 0);  // sin x = cos(x - pi / 2)
          const double v = tab[(size_t)(((t % (4LL * na)) + 4LL * na) % (4LL * na))] * nrm;
          blob[odd * hh + (size_t)m * ha + q] = v;
          blob[(2 + odd) * hh + (size_t)q * ha + m] = v;
        }
        const double sn = sin(pi * mode / (bc[a] ? 2.0 * na : (double)na));
        lam[odd * ha + q] = c * sn * sn;
      }
    blob += (size_t)na * na;
    lam += na;
  }
}

hipError_t fdx_precond(const Geo &g, const double *v, double *z, double *w1, double *w2, const double *blob,
                       hipStream_t s) {
  const int n0 = g.n0, n1 = g.n1, n2 = g.n2;
  const size_t s0 = (size_t)n0 * n0, s1 = (size_t)n1 * n1, s2 = (size_t)n2 * n2;
  const double *fx = blob, *fy = fx + s0, *fz = fy + s1;  // forward; the back halves follow at half of each
  const double *bx = fx + s0 / 2, *by = fy + s1 / 2, *bz = fz + s2 / 2;
  const double *lx = fz + s2, *ly = lx + n0, *lz = ly + n1;
  const long long rows = (long long)n0 * n1, plane = (long long)n1 * n2;
  const double *no = nullptr;
  hipError_t e;
  // forward: z, y, then x with the division by the eigenvalues; back: x, y, z
  if ((e = mode<MP_F_Z>(g, fz, v, w2, n2, rows, 1, no, no, no, s))) return e;
  if ((e = mode<MP_F_ROW>(g, fy, w2, w1, n1, n0, n2, no, no, no, s))) return e;
  if ((e = mode<MP_F_ROW>(g, fx, w1, w2, n0, 1, plane, lx, ly, lz, s))) return e;
  if ((e = mode<MP_B_ROW>(g, bx, w2, w1, n0, 1, plane, no, no, no, s))) return e;
  if ((e = mode<MP_B_ROW>(g, by, w1, w2, n1, n0, n2, no, no, no, s))) return e;
  return mode<MP_B_Z>(g, bz, w2, z, n2, rows, 1, no, no, no, s);
}

}  // namespace ibs
