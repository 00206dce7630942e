// The smoothed covariance of complete common-grid data as an operator: its
// products with a block of vectors are formed without the P x P covariance
// ever being stored (Section 3.2's blockwise processing, Section 3.4's
// products of the covariance with the projection matrix).
//
// With every curve observed at every node, the pair weights of eq. 2.4 are one
// constant off the diagonal p = q and zero on it, and the pair sums are
// G = (Y^T Y - diag) / (P(P-1)). Write Z_{i,0} for curve i filtered by the
// product taps K and Z_{i,k} for the taps K u_k (u_k = m / H_k along
// coordinate k, H_k = h_k (M_k - 1)), and W_e(x) = sum_m K(m) (m/H)^e for the
// 1-D window sums at x. Where the s- and t-windows of a covariance node share
// no grid node (|s_k - t_k| > 2 R_k for some k), no diagonal pair enters the
// window: the weight moments are a tensor product and the local-linear
// intercept has a closed form, which factors over the two ends:
//   b0(s,t) = (1/n) sum_i [ L_i(s) L_i(t) - B_i(s) B_i(t) ]
//   B_i(x) = (A(x) Z_{i,0}(x) - sum_k (a_k/v_k) Z_{i,k}(x)) / S(x),
//   L_i(x) = Z_{i,0}(x) / S(x) + B_i(x)   (curve i's own local-linear smooth),
// with a_k = W_1/W_0, v_k = W_2/W_0 - a_k^2 at x_k, A = sum_k a_k^2/v_k and
// S = prod_k W_0(x_k). Away from the band |s - t|_inf <= 2R the smoothed
// covariance therefore has rank at most 2n + 1 (with the mean term) and
//   Gamma X = (1/n) (L (L^T X) - B (B^T X)) - mu (mu^T X) + Delta X,
// where Delta is nonzero on the band only: there the (2d+1)-moment system is
// solved per node with the diagonal pairs removed,
//   weight moments   = prod_k W(s_k) W(t_k) - prod_k E_k(s_k, t_k),
//   response moments = (1/n) [ sum_i Z_a(s) Z_b(t) - sum_p f(p; s,t) Y2(p) ],
// (E_k the 1-D sums over shared nodes of K(p-s)K(p-t) times powers of u and
// v, Y2(p) = sum_i Y_ip^2, f the product of the per-coordinate factors), and
// Delta = b0_band - b0_closed form. Delta is either recomputed in every
// product (tile by tile, nothing of the covariance kept) or formed once and
// kept in tile blocks (the band only). Everything is FP64.
//
// d = 1 (k_band): band tiles of 64 nodes; one workgroup per s-tile visits the
// t-tiles within reach of the band. d = 2 and 3 (k_band_mfma): one workgroup per
// 32 s-nodes (4 x 8 of the last two coordinates), t-blocks of 4 x 4 nodes; per
// pair of blocks of 16 nodes:
//   1. the 2d+1 response moments of the full pair sums as FP64 matrix
//      products over the curves;
//   2. the diagonal correction, coordinate by coordinate: summed over p_0 ahead
//      of the products (k_hsum), over p_1 per workgroup and t-tile, over p_2 per
//      lane;
//   3. Delta from the first row of the inverse of the weight-moment matrix.
//      That row depends on the two nodes' positions only, and coordinate by
//      coordinate on t_k - s_k alone where both lie R_k or more from the border:
//      the operator tabulates it for every combination of the coordinates' pair
//      classes (k_wtab);
//   4. Delta times the t-rows of X added to the s-rows' outputs (or the block
//      stored). Of two mirrored blocks one is formed; k_band_turned applies the
//      transposes.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <utility>
#include <vector>

#include "common.hpp"
#include "covop.hpp"
#include "wls.hpp"

namespace fpca {
namespace {

constexpr int BT = 512;  // band kernel threads
constexpr int NC = 16;   // curves per staged chunk
constexpr int ZP = 66;   // padded row of 64 nodes in LDS

struct CovGeo {
  int d;
  int M[3];
  int R[3];
  int64_t stride[3];
  int64_t P;
  int n;
  double inv_n;
  const double *K[3];  // K(m), m = -R..R
  const double *U[3];  // m / H
  const double *W[3];  // W[x*3 + e]
  const double *E[3];  // E[(x*(4R+1) + delta + 2R)*6 + ab], ab: 00 10 01 20 11 02
  int tb[3], nt[3], span[3];
  int nslot;
  double H[3];  // h_k (M_k - 1)
  // d >= 2: pair classes of every coordinate (cls[(x * (4R + 1) + delta + 2R)]:
  // 2 * class + 1 if the class is met mirrored), their numbers, the table of
  // first rows of the inverse weight-moment matrices (8 doubles per combination
  // of classes, the last coordinate's fastest), and per node of a coordinate
  // 1 / W_0, a^2 / v and a / v
  const int *cls[3];
  int ncls[3];
  const double *rows;
  const double *nd[3];
};

template <int d>
constexpr int tile_ext() {
  return d == 1 ? 64 : (d == 2 ? 8 : 4);
}

// ------------------------------------------------------------------ set-up
__global__ void k_transpose(int64_t n, int64_t P, const double *__restrict__ Y, double *__restrict__ Yn) {
  __shared__ double t[32][33];
  const int64_t p0 = int64_t(blockIdx.x) * 32, i0 = int64_t(blockIdx.y) * 32;
  for (int r = threadIdx.y; r < 32; r += 8) {
    const int64_t i = i0 + r, p = p0 + threadIdx.x;
    t[r][threadIdx.x] = (i < n && p < P) ? Y[i * P + p] : 0.0;
  }
  __syncthreads();
  for (int r = threadIdx.y; r < 32; r += 8) {
    const int64_t p = p0 + r, i = i0 + threadIdx.x;
    if (p < P && i < n) Yn[p * n + i] = t[threadIdx.x][r];
  }
}

__global__ void k_sq(int64_t P, int n, const double *__restrict__ Yn, double *__restrict__ Y2) {
  const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (p >= P) return;
  double s = 0.0;
  for (int i = 0; i < n; ++i) {
    const double v = Yn[p * n + i];
    s = fma(v, v, s);
  }
  Y2[p] = s;
}

struct FilterMap {
  int nmap;
  int fo[4], fi[4], e[4];
};

// One 1-D pass along coordinate k of node-major arrays [P][F][n]: map j of
// blockIdx.y takes family fi through the taps K (e = 0) or K u (e = 1) into
// family fo.
__global__ void k_filter(CovGeo g, int k, const double *__restrict__ in, int Fin, double *__restrict__ out,
                         int Fout, FilterMap fm) {
  const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int n = g.n;
  if (idx >= g.P * n) return;
  const int j = blockIdx.y;
  const int64_t p = idx / n;
  const int i = int(idx - p * n);
  const int64_t st = g.stride[k];
  const int R = g.R[k];
  const int xk = int((p / st) % g.M[k]);
  const int lo = -min(R, xk), hi = min(R, g.M[k] - 1 - xk);
  const int fi = fm.fi[j], fo = fm.fo[j];
  const bool wu = fm.e[j] != 0;
  const double *Kk = g.K[k], *Uk = g.U[k];
  double acc = 0.0;
  for (int m = lo; m <= hi; ++m) {
    const double w = wu ? Kk[m + R] * Uk[m + R] : Kk[m + R];
    acc = fma(w, in[((p + int64_t(m) * st) * Fin + fi) * n + i], acc);
  }
  out[(p * Fout + fo) * n + i] = acc;
}

// L and B of every curve at every node from the filtered families.
__global__ void k_lr_prep(CovGeo g, const double *__restrict__ Zn, double *__restrict__ Ln, double *__restrict__ Bn) {
  const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int n = g.n;
  if (idx >= g.P * n) return;
  const int64_t p = idx / n;
  const int i = int(idx - p * n);
  const int F = g.d + 1;
  double S = 1.0, A = 0.0, bsum = 0.0;
  for (int k = 0; k < g.d; ++k) {
    const int x = int((p / g.stride[k]) % g.M[k]);
    const double w0 = g.W[k][x * 3], w1 = g.W[k][x * 3 + 1], w2 = g.W[k][x * 3 + 2];
    const double a = w1 / w0, v = w2 / w0 - a * a;
    S *= w0;
    A += a * a / v;
    bsum += (a / v) * Zn[(p * F + 1 + k) * n + i];
  }
  const double z0 = Zn[(p * F) * n + i];
  const double B = (A * z0 - bsum) / S;
  Ln[p * n + i] = z0 / S + B;
  Bn[p * n + i] = B;
}

// ------------------------------------------------------------------ low rank
// Partial products over 64 rows: part[blk][i][c] = sum_t L[t][i] X[t][c],
// part[blk][n + i][c] likewise with B, part[blk][2n][c] = sum_t mu[t] X[t][c].
__global__ __launch_bounds__(256) void k_lr_partial(CovGeo g, int r, const double *__restrict__ X,
                                                    const double *__restrict__ Ln, const double *__restrict__ Bn,
                                                    const double *__restrict__ mu, double *__restrict__ part) {
  __shared__ double Xs[64][64];
  __shared__ double ms[64];
  const int n = g.n;
  const int64_t blk = blockIdx.x, row0 = blk * 64;
  const int nrows = int(min<int64_t>(64, g.P - row0));
  for (int e = threadIdx.x; e < 64 * 64; e += 256) {
    const int t = e >> 6, c = e & 63;
    Xs[t][c] = (t < nrows && c < r) ? X[(row0 + t) * r + c] : 0.0;
  }
  if (threadIdx.x < 64) ms[threadIdx.x] = threadIdx.x < nrows ? mu[row0 + threadIdx.x] : 0.0;
  __syncthreads();
  const int il = threadIdx.x & 63, cq = threadIdx.x >> 6;
  const int i = blockIdx.y * 64 + il;
  const int64_t base = blk * (2 * int64_t(n) + 1);
  if (i < n) {
    double u[16], v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) u[j] = v[j] = 0.0;
    for (int t = 0; t < nrows; ++t) {
      const double l = Ln[(row0 + t) * n + i], b = Bn[(row0 + t) * n + i];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const double x = Xs[t][cq + 4 * j];
        u[j] = fma(l, x, u[j]);
        v[j] = fma(b, x, v[j]);
      }
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int c = cq + 4 * j;
      if (c < r) {
        part[(base + i) * 64 + c] = u[j];
        part[(base + n + i) * 64 + c] = v[j];
      }
    }
  }
  if (blockIdx.y == 0 && threadIdx.x < r) {
    double s = 0.0;
    for (int t = 0; t < nrows; ++t) s = fma(ms[t], Xs[t][threadIdx.x], s);
    part[(base + 2 * n) * 64 + threadIdx.x] = s;
  }
}

// tot[j][c] = sum over the row blocks of part[b][j][c]: one workgroup per row
// j; thread (group g, column c) adds blocks g, g + 4, ... (eight loads in
// flight), then the four groups are added in order.
__global__ __launch_bounds__(256) void k_lr_reduce(int64_t nblk, int rows, int r, const double *__restrict__ part,
                                                   double *__restrict__ tot) {
  __shared__ double gs[4][64];
  const int j = blockIdx.x, c = threadIdx.x & 63, g = threadIdx.x >> 6;
  double s = 0.0;
  if (c < r) {
    int64_t b = g;
    for (; b + 28 < nblk; b += 32) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[((b + 4 * u) * rows + j) * 64 + c];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; b < nblk; b += 4) s += part[(b * rows + j) * 64 + c];
  }
  gs[g][c] = s;
  __syncthreads();
  if (g == 0 && c < r) tot[int64_t(j) * 64 + c] = ((gs[0][c] + gs[1][c]) + gs[2][c]) + gs[3][c];
}

// out[s][c] = (1/n) sum_i (L[s][i] U[i][c] - B[s][i] V[i][c]) - mu[s] m[c]
__global__ __launch_bounds__(256) void k_lr_out(CovGeo g, int r, const double *__restrict__ Ln,
                                                const double *__restrict__ Bn, const double *__restrict__ mu,
                                                const double *__restrict__ tot, double *__restrict__ out) {
  __shared__ double Us[32][64], Vs[32][64];
  __shared__ double Ls[64][33], Bs[64][33];
  const int n = g.n;
  const int64_t row0 = int64_t(blockIdx.x) * 64;
  const int nrows = int(min<int64_t>(64, g.P - row0));
  const int sl = threadIdx.x >> 2, cq = threadIdx.x & 3;
  double acc[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) acc[j] = 0.0;
  for (int i0 = 0; i0 < n; i0 += 32) {
    __syncthreads();
    for (int e = threadIdx.x; e < 32 * 64; e += 256) {
      const int ii = e >> 6, c = e & 63;
      const bool ok = i0 + ii < n && c < r;
      Us[ii][c] = ok ? tot[int64_t(i0 + ii) * 64 + c] : 0.0;
      Vs[ii][c] = ok ? tot[int64_t(n + i0 + ii) * 64 + c] : 0.0;
    }
    for (int e = threadIdx.x; e < 64 * 32; e += 256) {
      const int t = e >> 5, ii = e & 31;
      const bool ok = t < nrows && i0 + ii < n;
      Ls[t][ii] = ok ? Ln[(row0 + t) * n + i0 + ii] : 0.0;
      Bs[t][ii] = ok ? Bn[(row0 + t) * n + i0 + ii] : 0.0;
    }
    __syncthreads();
    for (int ii = 0; ii < 32; ++ii) {
      const double l = Ls[sl][ii], b = Bs[sl][ii];
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[j] = fma(l, Us[ii][cq + 4 * j], fma(-b, Vs[ii][cq + 4 * j], acc[j]));
    }
  }
  if (sl < nrows) {
    const double m = mu[row0 + sl];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int c = cq + 4 * j;
      if (c < r) out[(row0 + sl) * r + c] = acc[j] * g.inv_n - m * tot[int64_t(2 * n) * 64 + c];
    }
  }
}

// ------------------------------------------------------------------ band
// Per-coordinate exponent index of each weight moment (S0, S1[D], S2 upper
// triangle row by row) for D = 2d coordinates s_0..s_{d-1}, t_0..t_{d-1}:
// 0 = (0,0), 1 = (1,0), 2 = (0,1), 3 = (2,0), 4 = (1,1), 5 = (0,2) as powers of
// (u_k, v_k).
template <int d>
__device__ constexpr int mom_ab(int q, int k) {
  constexpr int D = 2 * d;
  if (q == 0) return 0;
  if (q <= D) {
    const int j = q - 1;
    return (j % d == k) ? (j < d ? 1 : 2) : 0;
  }
  int idx = q - 1 - D;
  int j = 0;
  while (idx >= D - j) {
    idx -= D - j;
    ++j;
  }
  const int l = j + idx;
  const int kj = j % d, kl = l % d;
  const bool sj = j < d, sl = l < d;
  if (kj == kl) {
    if (kj != k) return 0;
    if (j == l) return sj ? 3 : 5;
    return 4;
  }
  if (k == kj) return sj ? 1 : 2;
  if (k == kl) return sl ? 1 : 2;
  return 0;
}

// m[q] = prod_k P_k[ab(q,k)] - prod_k E_k[ab(q,k)] with every index fixed at
// compile time (the per-coordinate factors stay in registers).
template <int d, int q>
__device__ inline double weight_moment(const double (&Pk)[3][6], const double (&Ek)[3][6]) {
  constexpr int a0 = mom_ab<d>(q, 0);
  constexpr int a1 = d > 1 ? mom_ab<d>(q, 1) : 0;
  constexpr int a2 = d > 2 ? mom_ab<d>(q, 2) : 0;
  double pp = Pk[0][a0], ee = Ek[0][a0];
  if constexpr (d > 1) {
    pp *= Pk[1][a1];
    ee *= Ek[1][a1];
  }
  if constexpr (d > 2) {
    pp *= Pk[2][a2];
    ee *= Ek[2][a2];
  }
  return pp - ee;
}

template <int d, int... q>
__device__ inline void fill_weight_moments(const double (&Pk)[3][6], const double (&Ek)[3][6], double *m,
                                           std::integer_sequence<int, q...>) {
  ((m[q] = weight_moment<d, q>(Pk, Ek)), ...);
}

struct BandArgs {
  CovGeo g;
  const double *Zn;
  const double *Y2;
  const double *X;  // fused product: P x r
  int r;
  double *out;
  double *band;  // stored blocks
  const double *Hs;  // d >= 2: Y2 summed over p_0 (k_hsum) for s_0 from hs0 on; Y2 itself for d = 2
  int hs0;
  int c0, nc;        // d >= 2: columns of X of this launch
  // d >= 2: the units of s-nodes of this launch, lo .. lo + cnt - 1: s_0 for d = 3,
  // tiles of four s_1 for d = 2. Half of the pairs formed: the distances of this
  // launch, and the blocks of Delta formed (TurnedGeo).
  int lo, cnt, i0, ni;
  double *delta;
};

// Local node li of a tile (coordinate d-1 fastest) and its grid coordinates.
template <int d>
__device__ inline void tile_node(int li, const int *lo, const CovGeo &g, int *x, bool *ok, int64_t *p) {
  constexpr int TB = tile_ext<d>();
  int rem = li;
  bool v = true;
  int64_t q = 0;
#pragma unroll
  for (int k = d - 1; k >= 0; --k) {
    x[k] = lo[k] + rem % TB;
    rem /= TB;
    v = v && x[k] < g.M[k];
    q += int64_t(x[k]) * g.stride[k];
  }
  *ok = v;
  *p = q;
}

// The per-coordinate products of window sums and the shared-node sums of the
// pair (s, t) of coordinate k.
__device__ inline void pair_factors(const CovGeo &g, int k, int xs, int xt, double (&P)[6], double (&E)[6]) {
  const int R2 = 2 * g.R[k];
  const double *Wk = g.W[k];
  const double ws0 = Wk[xs * 3], ws1 = Wk[xs * 3 + 1], ws2 = Wk[xs * 3 + 2];
  const double wt0 = Wk[xt * 3], wt1 = Wk[xt * 3 + 1], wt2 = Wk[xt * 3 + 2];
  P[0] = ws0 * wt0;
  P[1] = ws1 * wt0;
  P[2] = ws0 * wt1;
  P[3] = ws2 * wt0;
  P[4] = ws1 * wt1;
  P[5] = ws0 * wt2;
  const int dc = min(max(xt - xs, -R2), R2);
  const double *Er = &g.E[k][(int64_t(xs) * (2 * R2 + 1) + dc + R2) * 6];
#pragma unroll
  for (int j = 0; j < 6; ++j) E[j] = Er[j];
}

constexpr int ZH = 34;  // padded row of the 32 t-nodes of a half tile

// d = 1. Per s-tile: every t-tile within reach of the band, each in two halves
// of 32 t-nodes (4 nodes per thread keep the FP64 solve within the registers).
constexpr int B1_UN = 2 * NC * (ZP + ZH) > 64 * 33 + 32 * 64 ? 2 * NC * (ZP + ZH) : 64 * 33 + 32 * 64;
constexpr int B1_LDS = B1_UN + 4096;  // curve chunks | Delta and X tiles, then the Y2 box

template <bool STORE>
__global__ __launch_bounds__(BT) void k_band(BandArgs A) {
  constexpr int d = 1, NT = 3, NS = 6;
  extern __shared__ double sm[];
  double *Zs = sm;                // [2][NC][ZP]: the 64 s-nodes
  double *Zt = sm + 2 * NC * ZP;  // [2][NC][ZH]: the 32 t-nodes of the half
  double *Dl = sm;                // [64][33]
  double *Xl = sm + 64 * 33;      // [32][64]
  double *Yb = sm + B1_UN;        // Y2 box

  const CovGeo &g = A.g;
  const int n = g.n, M = g.M[0], R = g.R[0];
  const int tid = threadIdx.x;
  const int a = tid >> 4, b = tid & 15;  // s-locals 2a, 2a+1; t-locals 32 hh + 2b, + 1
  const int s0 = int(blockIdx.x) * 64;
  const int ro = tid >> 3, cg = tid & 7;  // fused product: s-row and column group
  double acco[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acco[j] = 0.0;

  for (int o = 0; o < g.nslot; ++o) {
    const int c = int(blockIdx.x) + o - g.span[0];
    if (c < 0 || c >= g.nt[0]) continue;  // uniform across the workgroup
    const int t0 = c * 64;
    __syncthreads();  // readers of the previous tile pair's tables are done
    // Y2 over the nodes shared by some s- and t-window of the tile pair
    const int plo = max(max(s0, t0) - R, 0);
    const int np = min(min(s0, t0) + 63 + R, M - 1) - plo + 1;
    for (int e = tid; e < np; e += BT) Yb[e] = A.Y2[plo + e];

    for (int hh = 0; hh < 2; ++hh) {
      // ---- 1. response moments of the full pair sums
      double acc[2][2][NT];
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int q = 0; q < NT; ++q) acc[x][y][q] = 0.0;
      for (int i0 = 0; i0 < n; i0 += NC) {
        __syncthreads();
        constexpr int ps = 2 * NC * 64, pt = 2 * NC * 32;
        for (int e = tid; e < ps + pt; e += BT) {
          const bool side = e >= ps;
          const int rem = side ? e - ps : e;
          const int node = rem / (2 * NC);
          const int fi = rem - node * (2 * NC);
          const int f = fi / NC, ii = fi - f * NC;
          const int x = side ? t0 + 32 * hh + node : s0 + node;
          const double v = x < M && i0 + ii < n ? A.Zn[(int64_t(x) * 2 + f) * n + i0 + ii] : 0.0;
          if (side)
            Zt[(f * NC + ii) * ZH + node] = v;
          else
            Zs[(f * NC + ii) * ZP + node] = v;
        }
        __syncthreads();
#pragma unroll 2
        for (int ii = 0; ii < NC; ++ii) {
          double zs[2][2], zt[2][2];
#pragma unroll
          for (int f = 0; f < 2; ++f) {
            const double2 s2 = *reinterpret_cast<const double2 *>(&Zs[(f * NC + ii) * ZP + 2 * a]);
            const double2 t2 = *reinterpret_cast<const double2 *>(&Zt[(f * NC + ii) * ZH + 2 * b]);
            zs[0][f] = s2.x;
            zs[1][f] = s2.y;
            zt[0][f] = t2.x;
            zt[1][f] = t2.y;
          }
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) {
              acc[x][y][0] = fma(zs[x][0], zt[y][0], acc[x][y][0]);
              acc[x][y][1] = fma(zs[x][1], zt[y][0], acc[x][y][1]);
              acc[x][y][2] = fma(zs[x][0], zt[y][1], acc[x][y][2]);
            }
        }
      }

      double delta[2][2];
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const int s = s0 + 2 * a + x, t = t0 + 32 * hh + 2 * b + y;
          const int xs = min(s, M - 1), xt = min(t, M - 1);
          // closed-form (tensor-product) intercept from the full moments
          const double *Wk = g.W[0];
          const double as = Wk[xs * 3 + 1] / Wk[xs * 3], vs = Wk[xs * 3 + 2] / Wk[xs * 3] - as * as;
          const double at = Wk[xt * 3 + 1] / Wk[xt * 3], vt = Wk[xt * 3 + 2] / Wk[xt * 3] - at * at;
          const double fac = 1.0 + (as * as / vs + at * at / vt);
          const double lin = (as / vs) * acc[x][y][1] + (at / vt) * acc[x][y][2];
          const double low = (acc[x][y][0] * fac - lin) * g.inv_n / (Wk[xs * 3] * Wk[xt * 3]);
          // ---- 2. diagonal correction: subtract sum_p f(p; s,t) Y2(p) from acc
          const double *K0 = g.K[0], *U0 = g.U[0];
          const int lo = max(max(s, t) - R, 0), hi = min(min(s, t) + R, M - 1);
          double c0 = 0.0, c1 = 0.0, c2 = 0.0;
          for (int p = lo; p <= hi; ++p) {
            const double kk = K0[p - s + R] * K0[p - t + R] * Yb[p - plo];
            c0 += kk;
            c1 = fma(kk, U0[p - s + R], c1);
            c2 = fma(kk, U0[p - t + R], c2);
          }
          // ---- 3. weight moments, the solve and Delta
          double dv = 0.0;
          if (s < M && t < M && t - s >= -2 * R && t - s <= 2 * R) {
            double Pk[3][6], Ek[3][6], m[NS + NT];
            pair_factors(g, 0, xs, xt, Pk[0], Ek[0]);
            fill_weight_moments<d>(Pk, Ek, m, std::make_integer_sequence<int, NS>{});
            m[NS] = (acc[x][y][0] - c0) * g.inv_n;
            m[NS + 1] = (acc[x][y][1] - c1) * g.inv_n;
            m[NS + 2] = (acc[x][y][2] - c2) * g.inv_n;
            int8_t st;
            dv = wls_b0<2>(m, &st) - low;
          }
          delta[x][y] = dv;
          // one element's solve at a time: no interleaving of their registers
          __builtin_amdgcn_sched_barrier(0);
        }

      // ---- 4. output
      if constexpr (STORE) {
        double *blk = A.band + (int64_t(blockIdx.x) * g.nslot + o) * 4096;
#pragma unroll
        for (int x = 0; x < 2; ++x)
          *reinterpret_cast<double2 *>(&blk[(2 * a + x) * 64 + 32 * hh + 2 * b]) =
              make_double2(delta[x][0], delta[x][1]);
      } else {
        __syncthreads();  // all readers of the curve chunks are done
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y) Dl[(2 * a + x) * 33 + 2 * b + y] = delta[x][y];
        for (int e = tid; e < 32 * 64; e += BT) {
          const int t = e >> 6, cc = e & 63;
          const int tn = t0 + 32 * hh + t;
          Xl[e] = (tn < M && cc < A.r) ? A.X[int64_t(tn) * A.r + cc] : 0.0;
        }
        __syncthreads();
        for (int t = 0; t < 32; ++t) {
          const double dd = Dl[ro * 33 + t];
#pragma unroll
          for (int j = 0; j < 8; ++j) acco[j] = fma(dd, Xl[t * 64 + cg + 8 * j], acco[j]);
        }
      }
    }
  }
  if constexpr (!STORE) {
    if (s0 + ro < M) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int cc = cg + 8 * j;
        if (cc < A.r) A.out[int64_t(s0 + ro) * A.r + cc] += acco[j];
      }
    }
  }
}

// ------------------------------------------------------------------ d = 2, 3
typedef double f64x4 __attribute__((ext_vector_type(4)));

// First row of the inverse of the (D+1) x (D+1) weight-moment matrix, with
// wls_b0's factorization and status rule: b0 = sum_q w_q T_q. FALLBACK gives
// (1/S0, 0, ..), EMPTY NaN.
template <int D>
__device__ inline void wls_weights(const double *m, double (&w)[D + 1]) {
  constexpr int n = D + 1;
  double A[n][n];
  const double S0 = m[0];
  A[0][0] = S0;
  int q = 1 + D;
#pragma unroll
  for (int k = 0; k < D; ++k) A[1 + k][0] = m[1 + k];
#pragma unroll
  for (int k = 0; k < D; ++k)
#pragma unroll
    for (int l = k; l < D; ++l) A[1 + l][1 + k] = m[q++];
  bool ok = true;
#pragma unroll
  for (int i = 1; i < n; ++i) ok = ok && (A[i][i] > 0.0);
#pragma unroll
  for (int j = 0; j < n; ++j) {
    double dj = A[j][j];
#pragma unroll
    for (int k = 0; k < j; ++k) dj -= A[j][k] * (A[j][k] * A[k][k]);
    ok = ok && (dj >= 1e-10 * A[j][j]);
    const double inv = 1.0 / dj;
#pragma unroll
    for (int i = j + 1; i < n; ++i) {
      double v = A[i][j];
#pragma unroll
      for (int k = 0; k < j; ++k) v -= A[i][k] * (A[j][k] * A[k][k]);
      A[i][j] = v * inv;
    }
    A[j][j] = dj;
  }
  if (!(S0 > 0.0) || !ok) {
    w[0] = S0 > 0.0 ? 1.0 / S0 : __builtin_nan("");
#pragma unroll
    for (int i = 1; i < n; ++i) w[i] = S0 > 0.0 ? 0.0 : __builtin_nan("");
    return;
  }
  // L z = e_0, then L^T w = D^-1 z
  w[0] = 1.0;
#pragma unroll
  for (int i = 1; i < n; ++i) {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < i; ++k) v -= A[i][k] * w[k];
    w[i] = v;
  }
#pragma unroll
  for (int i = n - 1; i >= 0; --i) {
    double v = w[i] / A[i][i];
#pragma unroll
    for (int k = i + 1; k < n; ++k) v -= A[k][i] * w[k];
    w[i] = v;
  }
}

template <int d>
__device__ inline void pair_weights(const CovGeo &g, const int (&xs)[3], const int (&xt)[3], double (&w)[2 * d + 1]) {
  constexpr int D = 2 * d, NS = 1 + D + D * (D + 1) / 2;
  double Pk[3][6], Ek[3][6], m[NS];
#pragma unroll
  for (int k = 0; k < d; ++k) pair_factors(g, k, xs[k], xt[k], Pk[k], Ek[k]);
  fill_weight_moments<d>(Pk, Ek, m, std::make_integer_sequence<int, NS>{});
  wls_weights<D>(m, w);
}

// The table of rows: thread e takes the combination of classes e. rep[k][c]: the
// class's own pair of nodes, as s * (4R + 1) + delta + 2R, or -1 where no pair of
// the grid has that class (the row is not read then).
template <int d>
__global__ __launch_bounds__(64) void k_wtab(CovGeo g, int64_t count, const int *__restrict__ r0,
                                             const int *__restrict__ r1, const int *__restrict__ r2,
                                             double *__restrict__ tab) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= count) return;
  int xs[3] = {0, 0, 0}, xt[3] = {0, 0, 0};
  int64_t rem = e;
  bool have = true;
#pragma unroll
  for (int k = d - 1; k >= 0; --k) {
    const int wd = 4 * g.R[k] + 1;
    const int c = (k == 0 ? r0 : (k == 1 ? r1 : r2))[int(rem % g.ncls[k])];
    rem /= g.ncls[k];
    have = have && c >= 0;
    xs[k] = max(c, 0) / wd;
    xt[k] = xs[k] + max(c, 2 * g.R[k]) % wd - 2 * g.R[k];
  }
  if (!have) return;
  double w[2 * d + 1];
  pair_weights<d>(g, xs, xt, w);
#pragma unroll
  for (int q = 0; q < 2 * d + 1; ++q) tab[e * 8 + q] = w[q];
}

// d = 3: Y2 summed over p_0 with the factors of (s_0, t_0 = s_0 + delta), s_0 from
// lo on: H[((s_0 - lo) (4R_0 + 1) + delta + 2 R_0)][ab][p_1 p_2], ab: K K, K K u, K K v.
__global__ __launch_bounds__(256) void k_hsum(CovGeo g, int lo, const double *__restrict__ Y2, double *__restrict__ H) {
  const int64_t plane = int64_t(g.M[1]) * g.M[2];
  const int64_t nb = (plane + 255) / 256, pair = blockIdx.x / nb;
  const int64_t p = (blockIdx.x % nb) * 256 + threadIdx.x;
  if (p >= plane) return;
  const int R = g.R[0], wd = 4 * R + 1;
  const int s = lo + int(pair / wd), t = s + int(pair % wd) - 2 * R;
  double h0 = 0.0, h1 = 0.0, h2 = 0.0;
  if (t >= 0 && t < g.M[0])
    for (int q = max(max(s, t) - R, 0); q <= min(min(s, t) + R, g.M[0] - 1); ++q) {
      const double f = g.K[0][q - s + R] * g.K[0][q - t + R] * Y2[q * plane + p];
      h0 += f;
      h1 = fma(f, g.U[0][q - s + R], h1);
      h2 = fma(f, g.U[0][q - t + R], h2);
    }
  double *o = H + pair * 3 * plane + p;
  o[0] = h0;
  o[plane] = h1;
  o[2 * plane] = h2;
}

// Node-major curves [P][F][n] to blocks of 4 x 4 nodes of the last two
// coordinates, [block][f][curve / 2][node][curve % 2] (missing nodes and the odd
// curve 0): a wavefront's operands are then whole cache lines, where sixteen
// nodes' rows are sixteen lines per quarter wavefront (64^3 nodes, n = 100, one
// product: 282 -> 239 ms).
__global__ __launch_bounds__(256) void k_retile(CovGeo g, const double *__restrict__ Zn, double *__restrict__ Zt) {
  constexpr int KB = 128;
  __shared__ double t[16][KB + 1];
  const int d = g.d, F = d + 1, f = blockIdx.y, n = g.n, nk2 = (n + 1) / 2;
  const int M1 = g.M[d - 2], M2 = g.M[d - 1], nT1 = (M1 + 3) / 4, nT2 = (M2 + 3) / 4;
  const int64_t ti = blockIdx.x;
  const int T2 = int(ti % nT2), T1 = int(ti / nT2 % nT1);
  const int64_t x0 = ti / nT2 / nT1;
  for (int k0 = 0; k0 < n; k0 += KB) {
    __syncthreads();
    for (int e = threadIdx.x; e < 16 * KB; e += 256) {
      const int k = e % KB, nd = e / KB, x1 = 4 * T1 + nd / 4, x2 = 4 * T2 + nd % 4;
      const int64_t p = (x0 * M1 + x1) * M2 + x2;
      t[nd][k] = x1 < M1 && x2 < M2 && k0 + k < n ? Zn[(p * F + f) * n + k0 + k] : 0.0;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 16 * KB; e += 256) {
      const int q = e >> 5, i = e & 31;
      if (k0 / 2 + q < nk2) Zt[((ti * F + f) * nk2 + k0 / 2 + q) * 32 + i] = t[i >> 1][2 * q + (i & 1)];
    }
  }
}

constexpr int MT = 512;     // threads: 8 wavefronts
constexpr int MKC = 104;    // curves per LDS chunk
template <int d>
constexpr int mfma_nv() { return 2 * d - 1; }  // H2 variants
inline size_t band_mfma_lds(int d, int n, int R2, int ncb) {
  const size_t kp = size_t(std::min(MKC, (n + 7) / 8 * 8));
  const size_t z = size_t(d + 1) * kp * 32, red = size_t(8) * ncb * 256;
  return (std::max(z, red) + 2 * size_t(8 + 2 * R2) * (2 * d - 1) * 16) * 8;
}

// Half of the pairs. Delta is symmetric, so of the blocks (s, t) and (t, s) one is
// formed where they lie apart in s_0, or in the tile of s_1: with an even distance
// t - s the one with t > s, with an odd one that with t < s (every s has as many t
// then). A launch takes the distances half_dt(i), i0 <= i < i0 + ni, of coordinate 0
// (d = 2: 0) and leaves its blocks, 16 s x 16 t each, at [distance][s-unit][block of
// s][tile distance in coordinate 1][in coordinate 2]; k_band_turned applies the
// transposes.
struct TurnedGeo {
  int T1h, T2h, T2n;  // reach in tiles; distances in coordinate 2
  int nk;             // distances in coordinate 1, at most
  int nT1, nT2, nB2;  // tiles of the coordinates; blocks of s in coordinate 2 (pairs of them)
};
__host__ __device__ inline TurnedGeo turned_geo(const int *M, const int *R, int d) {
  TurnedGeo t;
  t.T1h = (2 * R[d - 2] + 3) / 4;
  t.T2h = (2 * R[d - 1] + 3) / 4;
  t.T2n = 2 * t.T2h + 1;
  t.nk = d == 3 ? 2 * t.T1h + 1 : t.T1h;
  t.nT1 = (M[d - 2] + 3) / 4;
  t.nT2 = (M[d - 1] + 3) / 4;
  t.nB2 = (M[d - 1] + 7) / 8 * 2;
  return t;
}
__host__ __device__ inline int half_dt(int i) { return i % 2 == 0 ? i : -i; }
// Tile distance in coordinate 1 to its place (T1h of them at dt = 0), and back.
__device__ inline int turned_k(const TurnedGeo &t, int dt, int d1) {
  return dt ? d1 + t.T1h : (d1 > 0 ? d1 / 2 - 1 : t.T1h / 2 + (-d1 - 1) / 2);
}
__device__ inline int turned_d1(const TurnedGeo &t, int dt, int k) {
  return dt ? k - t.T1h : (k < t.T1h / 2 ? 2 * (k + 1) : -(2 * (k - t.T1h / 2) + 1));
}
// The block's place: u the s-unit within the launch (all of its distances count
// on: (i - i0) cnt + unit), S1 (d = 3) and S2 the tiles of s.
template <int d>
__device__ inline int64_t turned_slot(const TurnedGeo &t, int u, int S1, int S2, int k, int d2) {
  const int64_t blk = d == 3 ? (int64_t(u) * t.nT1 + S1) * t.nB2 + S2 : int64_t(u) * t.nB2 + S2;
  return ((blk * t.nk + k) * t.T2n + d2 + t.T2h) * 256;
}

// One workgroup per s-set (s_0; 4 of s_1; 8 of s_2): two blocks of 16 s-nodes,
// whose filtered curves stay in LDS. Steps over (t_0; 4 of t_1); each wavefront
// takes 4 of t_2, so a block of 16 t-nodes, against one of the s-blocks (both at
// once need twice the accumulators, which then spill: 334 against 282 ms at that
// stage). The FP64 matrix products D[t][s] = Zt Zs^T run over the curves in steps
// of eight (lane group g takes curves 2g and 2g + 1 of the eight, one 16-byte
// read per t-node), Zt straight from memory, double buffered in registers. Lane
// (g, l) of a result holds s-node l and the t-nodes (t_1 = v, t_2 = g), v = 0..3,
// which is the operand layout of the product with X that follows: Delta never
// leaves the registers. 64^3 nodes, R = 6, n = 100, r = 16: 230 ms, of which the
// matrix instructions issue for 79 ms (7 of 64 cycles per 4 curves and 256 pairs);
// the rest is the latency of two wavefronts per SIMD: the diagonal terms (about
// 50 ms), the rows of weights (50 ms, a gather of 64 rows per instruction) and
// curves missed in L2. With the responses on the vector units from LDS, the
// diagonal terms by LDS passes with barriers and a solve per pair: 1166 ms.
// HALF: half of the pairs (TurnedGeo), Delta's blocks also left in memory. All pairs 230 ms (above), half of them and k_band_turned 114;
// d = 2, 100^2 nodes, R = 6, n = 100, r = 20: 486 and 343 us.
// TAB: the rows of weights come from the operator's table; without the memory for
// it each is solved where it is needed (a solve per pair, with spills: all pairs at
// 64^3, k_hsum for one s_0 at a time, 589 ms; d = 2, 100^2 nodes, R = 28: 4.5 for 1.9).
template <int d, int NCB, bool STORE, bool HALF, bool TAB>
__global__ __launch_bounds__(MT) void k_band_mfma(BandArgs A) {
  constexpr int F = d + 1, NT = 2 * d + 1, NV = mfma_nv<d>();
  constexpr int k1 = d - 2, k2 = d - 1;
  extern __shared__ double sm[];
  const CovGeo &g = A.g;
  const int n = g.n, R1 = g.R[k1], R2 = g.R[k2], M1 = g.M[k1], M2 = g.M[k2];
  const int R0 = d == 3 ? g.R[0] : 0, M0 = d == 3 ? g.M[0] : 1;
  const int kp = min(MKC, (n + 7) / 8 * 8);
  const int nch = (n + MKC - 1) / MKC;
  const int hw = 8 + 2 * R2;  // p_2 span of the s-set
  double *Zs = sm;            // [F][kp][32], the halves of a row swapped where curve / 2 is odd
  const int zsz = max(F * kp * 32, 8 * NCB * 256);
  double *H2 = sm + zsz;      // [2][hw][NV][16 (s_1, t_1)]
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 15, gq = (tid & 63) >> 4;
  // s-set of this workgroup; consecutive workgroups of an XCD are neighbours
  int s0 = 0, s1a, s2a;
  {
    const int n1 = (M1 + 3) / 4, n2 = (M2 + 7) / 8;
    const int nwg = int(gridDim.x), per = nwg / 8;
    int id = int(blockIdx.x);
    if (id < per * 8) id = (id % 8) * per + id / 8;
    s2a = (id % n2) * 8;
    id /= n2;
    if constexpr (d == 3) {
      s1a = (id % n1) * 4;
      s0 = A.lo + id / n1;
    } else {
      s1a = (A.lo + id) * 4;
    }
  }
  const int64_t st0 = d == 3 ? g.stride[0] : 0, st1 = g.stride[k1];
  auto node_of = [&](int x0, int x1, int x2) { return int64_t(x0) * st0 + int64_t(x1) * st1 + x2; };
  // this wavefront's s-block and this lane's s-node
  const int sb = wave & 1;
  const int xs1 = s1a + (l >> 2), xs2 = s2a + 4 * sb + (l & 3);
  const bool sok = xs1 < M1 && xs2 < M2;
  const int xs1c = min(xs1, M1 - 1), xs2c = min(xs2, M2 - 1);
  double sq[2 + d];
  {
    const double *n1 = g.nd[k1] + xs1c * 3, *n2 = g.nd[k2] + xs2c * 3;
    sq[0] = n1[0] * n2[0];
    sq[1] = n1[1] + n2[1];
    sq[2 + k1] = n1[2];
    sq[2 + k2] = n2[2];
    if constexpr (d == 3) {
      const double *n0 = g.nd[0] + s0 * 3;
      sq[0] *= n0[0];
      sq[1] += n0[1];
      sq[2] = n0[2];
    }
  }
  const int nT1 = (M1 + 3) / 4, nT2 = (M2 + 3) / 4, nk2 = (n + 1) / 2;
  auto load_zs = [&](int ch) {
    const int q0 = ch * (MKC / 2), kp2 = kp / 2;
    const int64_t ti = (int64_t(s0) * nT1 + s1a / 4) * nT2 + s2a / 4;
    for (int e = tid; e < 2 * F * kp2 * 32; e += MT) {
      const int i = e & 31, r = e >> 5, q = r % kp2, fb = r / kp2, f = fb % F, b = fb / F;
      const bool ok = s2a / 4 + b < nT2 && q0 + q < nk2;
      const double v = ok ? A.Zn[(((ti + b) * F + f) * nk2 + q0 + q) * 32 + i] : 0.0;
      Zs[(f * kp + 2 * q + (i & 1)) * 32 + ((16 * b + (i >> 1)) ^ (16 * (q & 1)))] = v;
    }
  };
  if (nch == 1) load_zs(0);
  f64x4 oacc[NCB];
#pragma unroll
  for (int c = 0; c < NCB; ++c) oacc[c] = f64x4{0.0, 0.0, 0.0, 0.0};

  const int t0lo = d == 3 ? max(0, s0 - 2 * R0) : 0, t0hi = d == 3 ? min(M0 - 1, s0 + 2 * R0) : 0;
  const TurnedGeo tg = turned_geo(g.M, g.R, d);
  // the t-tiles of coordinate 1 in an order by their number modulo the reach, so
  // that the workgroups of an XCD, whose reaches overlap, take the same tile at
  // about the same time and find its curves in their L2
  const int T1h = (2 * R1 + 3) / 4, T1n = 2 * T1h + 1, T1lo = s1a / 4 - T1h;
  const int T2lo = max(0, s2a - 2 * R2) / 4, T2hi = min(M2 - 1, s2a + 7 + 2 * R2) / 4;
  const int p2lo = max(s2a - R2, 0), np2 = min(s2a + 7 + R2, M2 - 1) - p2lo + 1;
  const int64_t plane = int64_t(M1) * M2;
  const double iH1 = 1.0 / g.H[k1], iH2 = 1.0 / g.H[k2];
  // this lane's place in the product over p_2: its value for lane (t_2; s_1, s_2) is in lane (s_1; t_2, s_2)
  const int perm = (((tid >> 2) & 3) * 16 + ((tid >> 4) & 3) * 4 + (tid & 3)) * 4;
  int buf = 0;
  for (int i = HALF ? A.i0 : t0lo; i < (HALF ? A.i0 + A.ni : t0hi + 1); ++i) {
    const int dt = HALF ? half_dt(i) : 0, t0 = HALF ? s0 + dt : i;
    if (HALF && (t0 < 0 || t0 >= M0)) continue;
    for (int k = 0; k < T1n; ++k) {
      int T1 = k - (T1lo % T1n + T1n) % T1n;
      T1 = T1lo + (T1 < 0 ? T1 + T1n : T1);
      const int t1a = 4 * T1;
      if (T1 < 0 || t1a >= M1) continue;
      if (HALF && dt == 0 && t1a != s1a && (((t1a + s1a) & 4) == 0) != (t1a > s1a)) continue;  // formed as (t, s)
      const bool turned = HALF && (dt != 0 || t1a != s1a);
      // ---- the diagonal terms summed over p_0 and p_1
      double *Hb = H2 + buf * hw * NV * 16;
      buf ^= 1;
      const bool any = min(s1a, t1a) + 3 + R1 >= max(s1a, t1a) - R1;  // some shared p_1
      if (any) {
        const double *Hg = d == 3 ? A.Hs + int64_t((s0 - A.hs0) * (4 * R0 + 1) + t0 - s0 + 2 * R0) * 3 * plane : A.Hs;
        // rows s_1 + 4 t_1 (lane l of the first operand), columns p_2: one
        // variant and 16 columns per task
        const int ct = (np2 + 15) / 16;
        const int lo = max(max(s1a, t1a) - R1, 0), hi = min(min(s1a, t1a) + 3 + R1, M1 - 1);
        const int s1 = s1a + (l & 3), t1 = t1a + (l >> 2);
        const int plo = max(s1, t1) - R1, phi = min(s1, t1) + R1;
        for (int task = wave; task < NV * ct; task += 8) {
          const int v = task % NV, col = 16 * (task / NV) + l;
          const double *y = Hg + (v < 3 ? 0 : v - 2) * plane + p2lo + min(col, np2 - 1);
          f64x4 h = {0.0, 0.0, 0.0, 0.0};
          for (int p4 = lo; p4 <= hi; p4 += 4) {
            const int p = p4 + gq;
            const double us = double(p - s1) * iH1, vt = double(p - t1) * iH1;
            const bool in = p <= hi && p >= plo && p <= phi;
            double f = in ? fmax(1.0 - us * us, 0.0) * fmax(1.0 - vt * vt, 0.0) : 0.0;
            if (v == 1) f *= us;
            if (v == 2) f *= vt;
            h = __builtin_amdgcn_mfma_f64_16x16x4f64(f, y[int64_t(min(p, hi)) * M2], h, 0, 0, 0);
          }
          if (col < np2) {
#pragma unroll
            for (int i = 0; i < 4; ++i) Hb[(col * NV + v) * 16 + gq + 4 * i] = h[i];
          }
        }
      }
      __syncthreads();
      for (int T20 = T2lo; T20 <= T2hi; T20 += 4) {
        const int T2 = T20 + (wave >> 1);
        const int t2a = 4 * T2, s2b = s2a + 4 * sb;
        const bool work = T2 <= T2hi && t2a - (s2b + 3) <= 2 * R2 && s2b - (t2a + 3) <= 2 * R2;
        if (nch == 1 && !work) continue;
        f64x4 acc[NT];
#pragma unroll
        for (int q = 0; q < NT; ++q) acc[q] = f64x4{0.0, 0.0, 0.0, 0.0};
        // pair classes and the t-nodes' factors, requested ahead of the products
        const int xt2 = t2a + gq, xt2c = min(xt2, M2 - 1);
        int c1[4] = {0, 0, 0, 0};
#pragma unroll
        for (int v = 0; TAB && v < 4; ++v)
          c1[v] = g.cls[k1][xs1c * (4 * R1 + 1) + min(max(min(t1a + v, M1 - 1) - xs1c, -2 * R1), 2 * R1) + 2 * R1];
        const int c2 = !TAB ? 0 : g.cls[k2][xs2c * (4 * R2 + 1) + min(max(xt2c - xs2c, -2 * R2), 2 * R2) + 2 * R2];
        const double *n2 = g.nd[k2] + xt2c * 3;
        const double tS2 = n2[0], tA2 = n2[1], tB2 = n2[2];
        const int64_t tt = (int64_t(t0) * nT1 + T1) * nT2 + T2;
        for (int ch = 0; ch < nch; ++ch) {
          if (nch > 1) {
            __syncthreads();
            load_zs(ch);
            __syncthreads();
          }
          if (!work) continue;
          const int cn = min(MKC, n - ch * MKC);
          const double2 *zt = reinterpret_cast<const double2 *>(A.Zn) + (tt * F * nk2 + ch * (MKC / 2) + gq) * 16 + l;
          const int left = nk2 - ch * (MKC / 2) - gq;  // pairs of curves from this lane's first on
          auto fetch = [&](int k, double2 (&v)[F]) {
#pragma unroll
            for (int f = 0; f < F; ++f)
              v[f] = k / 2 < left ? zt[(int64_t(f) * nk2 + k / 2) * 16] : make_double2(0.0, 0.0);
          };
          const double *zs = Zs + 2 * gq * 32 + ((16 * sb + l) ^ (16 * (gq & 1)));
          auto mult = [&](int k, const double2 (&v)[F]) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              double z[F], a[F];
#pragma unroll
              for (int f = 0; f < F; ++f) {
                z[f] = zs[(f * kp + k + u) * 32];
                a[f] = u ? v[f].y : v[f].x;
              }
              acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0], z[0], acc[0], 0, 0, 0);
#pragma unroll
              for (int q = 0; q < d; ++q) {
                acc[1 + q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0], z[1 + q], acc[1 + q], 0, 0, 0);
                acc[1 + d + q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1 + q], z[0], acc[1 + d + q], 0, 0, 0);
              }
            }
          };
          double2 va[F], vb[F];
          fetch(0, va);
          for (int k = 0; k < cn; k += 16) {
            fetch(k + 8, vb);
            mult(k, va);
            if (k + 8 >= cn) break;
            fetch(k + 16, va);
            mult(k + 8, vb);
          }
        }
        if (!work) continue;
        const int c0 = d == 3 && TAB ? g.cls[0][s0 * (4 * R0 + 1) + t0 - s0 + 2 * R0] : 0;
        const double sg0 = c0 & 1 ? -1.0 : 1.0;
        double low[4], w[4][NT];
        bool inb[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int xt1 = t1a + v;
          inb[v] = sok && xt1 < M1 && xt2 < M2 && abs(xt2 - xs2) <= 2 * R2 && abs(xt1 - xs1) <= 2 * R1;
          if constexpr (TAB) {
            // pairs outside the band or the grid read the row of some class; their Delta is 0
            const int64_t e = (int64_t(d == 3 ? c0 >> 1 : 0) * g.ncls[k1] + (max(c1[v], 0) >> 1)) * g.ncls[k2] +
                              (max(c2, 0) >> 1);
            const double *row = g.rows + (inb[v] ? e : 0) * 8;
#pragma unroll
            for (int q = 0; q < NT; ++q) w[v][q] = row[q];
          } else {
            int xs[3] = {s0, xs1c, xs2c}, xt[3] = {t0, min(xt1, M1 - 1), xt2c};
            if constexpr (d == 2) {
              xs[0] = xs1c, xs[1] = xs2c;
              xt[0] = min(xt1, M1 - 1), xt[1] = xt2c;
            }
            pair_weights<d>(g, xs, xt, w[v]);
            // one solve at a time: no interleaving of their registers
            __builtin_amdgcn_sched_barrier(0);
          }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double *n1 = g.nd[k1] + min(t1a + v, M1 - 1) * 3;
          double tS = n1[0] * tS2, tA = n1[1] + tA2;
          double x = sq[2 + k1] * acc[1 + k1][v] + n1[2] * acc[1 + d + k1][v] +
                     sq[2 + k2] * acc[1 + k2][v] + tB2 * acc[1 + d + k2][v];
          if constexpr (d == 3) {
            const double *n0 = g.nd[0] + t0 * 3;
            tS *= n0[0];
            tA += n0[1];
            x += sq[2] * acc[1][v] + n0[2] * acc[1 + d][v];
          }
          low[v] = (acc[0][v] * (1.0 + (sq[1] + tA)) - x) * g.inv_n * (sq[0] * tS);
        }
        // ---- 2. the diagonal terms summed over p_2, a matrix product of the
        // sums over p_0 and p_1 (rows s_1 + 4 t_1) with the factors of
        // coordinate 2 (columns s_2 + 4 t_2, here in lane l)
        if (any) {
          const int sc = s2b + (l & 3), tc = t2a + (l >> 2);
          const int lo = max(max(s2b, t2a) - R2, 0), hi = min(min(s2b, t2a) + 3 + R2, M2 - 1);
          const int plo = max(sc, tc) - R2, phi = min(sc, tc) + R2;
          f64x4 cr[NT];
#pragma unroll
          for (int q = 0; q < NT; ++q) cr[q] = f64x4{0.0, 0.0, 0.0, 0.0};
          for (int p4 = lo; p4 <= hi; p4 += 4) {
            const int p = p4 + gq;
            const double us = double(p - sc) * iH2, vt = double(p - tc) * iH2;
            const bool in = p <= hi && p >= plo && p <= phi;
            const double f = in ? fmax(1.0 - us * us, 0.0) * fmax(1.0 - vt * vt, 0.0) : 0.0;
            const double *hp = Hb + (min(p, hi) - p2lo) * NV * 16 + l;
            const double h0 = hp[0], h1 = hp[16], h2 = hp[32];
            cr[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(h0, f, cr[0], 0, 0, 0);
            cr[1 + k1] = __builtin_amdgcn_mfma_f64_16x16x4f64(h1, f, cr[1 + k1], 0, 0, 0);
            cr[1 + d + k1] = __builtin_amdgcn_mfma_f64_16x16x4f64(h2, f, cr[1 + d + k1], 0, 0, 0);
            cr[1 + k2] = __builtin_amdgcn_mfma_f64_16x16x4f64(h0, f * us, cr[1 + k2], 0, 0, 0);
            cr[1 + d + k2] = __builtin_amdgcn_mfma_f64_16x16x4f64(h0, f * vt, cr[1 + d + k2], 0, 0, 0);
            if constexpr (d == 3) {
              cr[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(hp[48], f, cr[1], 0, 0, 0);
              cr[1 + d] = __builtin_amdgcn_mfma_f64_16x16x4f64(hp[64], f, cr[1 + d], 0, 0, 0);
            }
          }
#pragma unroll
          for (int q = 0; q < NT; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const double c = cr[q][v];
              acc[q][v] -= __hiloint2double(__builtin_amdgcn_ds_bpermute(perm, __double2hiint(c)),
                                               __builtin_amdgcn_ds_bpermute(perm, __double2loint(c)));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // ---- 3. Delta
        double delta[4];
        const double sg2 = c2 & 1 ? -1.0 : 1.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double sg1 = c1[v] & 1 ? -1.0 : 1.0;
          double dv = w[v][0] * acc[0][v];
          dv = fma(sg1, w[v][1 + k1] * acc[1 + k1][v] + w[v][1 + d + k1] * acc[1 + d + k1][v], dv);
          dv = fma(sg2, w[v][1 + k2] * acc[1 + k2][v] + w[v][1 + d + k2] * acc[1 + d + k2][v], dv);
          if constexpr (d == 3) dv = fma(sg0, w[v][1] * acc[1][v] + w[v][1 + d] * acc[1 + d][v], dv);
          delta[v] = inb[v] ? dv * g.inv_n - low[v] : 0.0;
        }
        // ---- 4. output
        if constexpr (STORE) {
          constexpr int TB = tile_ext<d>();
          if (sok) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int xt1 = t1a + v;
              if (xt1 >= M1 || xt2 >= M2) continue;
              const int a1 = xs1 / TB, a2 = xs2 / TB;
              int64_t tile = int64_t(a1) * g.nt[k2] + a2;
              int slot = (xt1 / TB - a1 + g.span[k1]) * (2 * g.span[k2] + 1) + (xt2 / TB - a2 + g.span[k2]);
              int sl = (xs1 % TB) * TB + xs2 % TB, tl = (xt1 % TB) * TB + xt2 % TB;
              if constexpr (d == 3) {
                const int a0 = s0 / TB;
                tile += int64_t(a0) * g.nt[1] * g.nt[2];
                slot += (t0 / TB - a0 + g.span[0]) * (2 * g.span[1] + 1) * (2 * g.span[2] + 1);
                sl += (s0 % TB) * TB * TB;
                tl += (t0 % TB) * TB * TB;
              }
              A.band[((tile * g.nslot + slot) * 64 + sl) * 64 + tl] = delta[v];
            }
          }
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int xt1 = t1a + v;
            const bool tok = xt1 < M1 && xt2 < M2;
            const int64_t q = node_of(t0, min(xt1, M1 - 1), min(xt2, M2 - 1));
#pragma unroll
            for (int c = 0; c < NCB; ++c) {
              const int col = 16 * c + l;
              const double xv = A.X[q * A.r + A.c0 + min(col, A.nc - 1)];
              oacc[c] =
                  __builtin_amdgcn_mfma_f64_16x16x4f64(tok && col < A.nc ? xv : 0.0, delta[v], oacc[c], 0, 0, 0);
            }
          }
          if (turned)
            *reinterpret_cast<f64x4 *>(A.delta +
                                       turned_slot<d>(tg, (i - A.i0) * A.cnt + (d == 3 ? s0 : s1a / 4) - A.lo, s1a / 4,
                                                      s2a / 4 + sb, turned_k(tg, dt, T1 - s1a / 4), T2 - s2a / 4 - sb) +
                                       l * 16 + 4 * gq) = f64x4{delta[0], delta[1], delta[2], delta[3]};
        }
      }
    }
  }
  if constexpr (!STORE) {
    // the wavefronts' sums added in order: [wave / 2][s-block][c][row (column of X)][s]
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NCB; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) sm[((wave * NCB + c) * 16 + gq + 4 * v) * 16 + l] = oacc[c][v];
    __syncthreads();
    for (int e = tid; e < 2 * NCB * 256; e += MT) {
      const int col = e % (NCB * 16), sn = e / (NCB * 16);  // column of X, s-node 0..31
      const int b = sn >> 4, c = col >> 4;
      const int x1 = s1a + ((sn >> 2) & 3), x2 = s2a + 4 * b + (sn & 3);
      double v = 0.0;
#pragma unroll
      for (int w = 0; w < 4; ++w) v += sm[(((2 * w + b) * NCB + c) * 16 + (col & 15)) * 16 + (sn & 15)];
      if (x1 < M1 && x2 < M2 && col < A.nc) A.out[node_of(s0, x1, x2) * A.r + A.c0 + col] += v;
    }
  }
}

// The transposes of the blocks of Delta that a launch of k_band_mfma has left,
// times X at their s-nodes, added to the t-nodes' outputs. One workgroup per block
// of 16 t-nodes; its four wavefronts take every fourth of the blocks that have it
// for their t, and their sums are added in order: products repeat bit for bit
// (added with FP64 atomics by k_band_mfma itself, one product at 64^3 took 130 ms,
// now 114, and the order was the scheduler's). Bound by the reading of Delta, 2 KB per block.
template <int d, int NCB>
__global__ __launch_bounds__(256) void k_band_turned(BandArgs A, int tlo) {
  __shared__ double red[4][16 * NCB][17];
  const CovGeo &g = A.g;
  const int M1 = g.M[d - 2], M2 = g.M[d - 1];
  const int64_t st0 = d == 3 ? g.stride[0] : 0, st1 = g.stride[d - 2];
  const TurnedGeo tg = turned_geo(g.M, g.R, d);
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 15, gq = (tid & 63) >> 4;
  int id = int(blockIdx.x);
  const int T2 = id % tg.nT2;
  id /= tg.nT2;
  const int T1 = d == 3 ? id % tg.nT1 : tlo + id, t0 = d == 3 ? tlo + id / tg.nT1 : 0;
  f64x4 acc[NCB];
#pragma unroll
  for (int c = 0; c < NCB; ++c) acc[c] = f64x4{0.0, 0.0, 0.0, 0.0};
  for (int e = wave; e < A.ni * tg.nk * tg.T2n; e += 4) {
    const int i = e / (tg.nk * tg.T2n), k = e / tg.T2n % tg.nk, d2 = e % tg.T2n - tg.T2h;
    const int dist = half_dt(A.i0 + i), s0 = t0 - dist;
    if (dist == 0 && k >= tg.T1h) continue;
    const int S1 = T1 - turned_d1(tg, dist, k), S2 = T2 - d2, su = d == 3 ? s0 : S1;
    if (S1 < 0 || S1 >= tg.nT1 || S2 < 0 || S2 >= tg.nT2 || su < A.lo || su >= A.lo + A.cnt) continue;
    const double *dl = A.delta + turned_slot<d>(tg, i * A.cnt + su - A.lo, S1, S2, k, d2) + l;
    double dt[4], x[4][NCB];
#pragma unroll
    for (int j = 0; j < 4; ++j) dt[j] = dl[(4 * j + gq) * 16];
    // lane group gq of step j: s-node 4 j + gq, so (s_1 = j, s_2 = gq) of its block
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int x1 = 4 * S1 + j, x2 = 4 * S2 + gq;
      const double *row = A.X + (int64_t(s0) * st0 + int64_t(min(x1, M1 - 1)) * st1 + min(x2, M2 - 1)) * A.r + A.c0;
#pragma unroll
      for (int c = 0; c < NCB; ++c) {
        const int col = 16 * c + l;
        const double v = row[min(col, A.nc - 1)];
        x[j][c] = x1 < M1 && x2 < M2 && col < A.nc ? v : 0.0;
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int c = 0; c < NCB; ++c) acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[j][c], dt[j], acc[c], 0, 0, 0);
  }
#pragma unroll
  for (int c = 0; c < NCB; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][16 * c + gq + 4 * v][l] = acc[c][v];
  __syncthreads();
  // t-node i of a block: t_1 = i % 4, t_2 = i / 4
  for (int e = tid; e < 256 * NCB; e += 256) {
    const int col = e % (16 * NCB), i = e / (16 * NCB);
    const int y1 = 4 * T1 + (i & 3), y2 = 4 * T2 + (i >> 2);
    if (y1 >= M1 || y2 >= M2 || col >= A.nc) continue;
    A.out[(int64_t(t0) * st0 + int64_t(y1) * st1 + y2) * A.r + A.c0 + col] +=
        (red[0][col][i] + red[1][col][i]) + (red[2][col][i] + red[3][col][i]);
  }
}

__global__ void k_zero_f64(double *p, int64_t n) {
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
    p[i] = 0.0;
}

// Product with the stored band blocks.
template <int d>
__global__ __launch_bounds__(BT) void k_band_apply(BandArgs A) {
  constexpr int TB = tile_ext<d>();
  extern __shared__ double sm[];
  double *Dl = sm;            // [64][65]
  double *Xl = sm + 64 * 65;  // [64][64]
  __shared__ long long sidx[64], tidx[64];
  __shared__ int sok[64], tok[64];
  const CovGeo &g = A.g;
  const int tid = threadIdx.x;
  int sa[3] = {0, 0, 0}, s0[3] = {0, 0, 0};
  {
    int64_t rem = blockIdx.x;
#pragma unroll
    for (int k = d - 1; k >= 0; --k) {
      sa[k] = int(rem % g.nt[k]);
      rem /= g.nt[k];
      s0[k] = sa[k] * TB;
    }
  }
  if (tid < 64) {
    int x[3];
    bool ok;
    int64_t p;
    tile_node<d>(tid, s0, g, x, &ok, &p);
    sok[tid] = ok;
    sidx[tid] = ok ? p : 0;
  }
  const int ro = tid >> 3, cg = tid & 7;
  double acco[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acco[j] = 0.0;
  for (int o = 0; o < g.nslot; ++o) {
    int t0[3] = {0, 0, 0};
    bool inside = true;
    {
      int rem = o;
#pragma unroll
      for (int k = d - 1; k >= 0; --k) {
        const int w = 2 * g.span[k] + 1;
        const int c = sa[k] + rem % w - g.span[k];
        rem /= w;
        inside = inside && c >= 0 && c < g.nt[k];
        t0[k] = c * TB;
      }
    }
    if (!inside) continue;
    __syncthreads();
    if (tid < 64) {
      int x[3];
      bool ok;
      int64_t p;
      tile_node<d>(tid, t0, g, x, &ok, &p);
      tok[tid] = ok;
      tidx[tid] = ok ? p : 0;
    }
    const double *blk = A.band + (int64_t(blockIdx.x) * g.nslot + o) * 4096;
    for (int e = tid; e < 4096; e += BT) Dl[(e >> 6) * 65 + (e & 63)] = blk[e];
    __syncthreads();
    for (int e = tid; e < 64 * 64; e += BT) {
      const int t = e >> 6, c = e & 63;
      Xl[e] = (tok[t] && c < A.r) ? A.X[tidx[t] * A.r + c] : 0.0;
    }
    __syncthreads();
    for (int t = 0; t < 64; ++t) {
      const double dd = Dl[ro * 65 + t];
#pragma unroll
      for (int j = 0; j < 8; ++j) acco[j] = fma(dd, Xl[t * 64 + cg + 8 * j], acco[j]);
    }
  }
  if (sok[ro]) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int c = cg + 8 * j;
      if (c < A.r) A.out[sidx[ro] * A.r + c] += acco[j];
    }
  }
}

// ------------------------------------------------------------------ host
CovGeo make_geo(const fpca_covop_s *op) {
  CovGeo g{};
  g.d = op->d;
  int64_t st = 1;
  for (int k = 2; k >= 0; --k) {
    g.M[k] = k < op->d ? op->M[k] : 1;
    g.R[k] = k < op->d ? op->R[k] : 0;
  }
  for (int k = op->d - 1; k >= 0; --k) {
    g.stride[k] = st;
    st *= op->M[k];
  }
  g.P = op->P;
  g.n = int(op->n);
  g.inv_n = 1.0 / double(op->n);
  for (int k = 0; k < op->d; ++k) {
    g.K[k] = op->tab + op->tab_K[k];
    g.U[k] = op->tab + op->tab_U[k];
    g.W[k] = op->tab + op->tab_W[k];
    g.E[k] = op->tab + op->tab_E[k];
    g.tb[k] = op->tb[k];
    g.nt[k] = op->nt[k];
    g.span[k] = op->span[k];
    g.H[k] = op->H[k];
    g.cls[k] = op->cls[k];
    g.ncls[k] = op->ncls[k];
    g.nd[k] = op->tab + op->tab_nd[k];
  }
  g.rows = op->rows;
  g.nslot = op->nslot;
  return g;
}

void free_op(fpca_covop_s *op) {
  for (void *p : {static_cast<void *>(op->mem), static_cast<void *>(op->Zn), static_cast<void *>(op->tables),
                  static_cast<void *>(op->hsum), static_cast<void *>(op->delta), static_cast<void *>(op->band)})
    if (p) (void)hipFree(p);
  delete op;
}

// Memory that an operator can do without: taken where it is at most half of what is
// free, so that the calls which follow find theirs.
bool optional_alloc(fpca_context *ctx, void **p, size_t bytes) {
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
    (void)hipGetLastError();
    free_b = 0;
  }
  *p = nullptr;
  return bytes <= free_b / 2 && scratch_malloc(ctx, p, bytes) == hipSuccess;
}

unsigned nb256(int64_t n) { return unsigned((n + 255) / 256); }

BandArgs band_args(const fpca_covop_s *op, const double *X, int r, double *out) {
  BandArgs A{};
  A.g = make_geo(op);
  A.Zn = op->Zn;
  A.Y2 = op->Y2;
  A.X = X;
  A.r = r;
  A.out = out;
  A.band = op->band;
  A.Hs = op->d == 3 ? op->hsum : op->Y2;
  A.lo = A.hs0 = A.i0 = A.ni = 0;
  return A;
}

template <bool STORE>
int launch_band1(fpca_covop_s *op, const double *X, int r, double *out) {
  const BandArgs A = band_args(op, X, r, out);
  FPCA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_band<STORE>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, B1_LDS * 8));
  hipLaunchKernelGGL((k_band<STORE>), dim3(unsigned(op->n_stiles)), dim3(BT), B1_LDS * 8, op->ctx->stream, A);
  FPCA_LAUNCH_CHECK("covop band");
  return FPCA_OK;
}

template <int d, int NCB, bool STORE, bool HALF, bool TAB>
int launch_band_mfma(fpca_covop_s *op, const BandArgs &A) {
  const size_t lds = band_mfma_lds(d, int(op->n), op->R[d - 1], NCB);
  const int64_t nwg = A.cnt * (d == 3 ? int64_t((op->M[1] + 3) / 4) : 1) * ((op->M[d - 1] + 7) / 8);
  if (nwg > 0x7fffffffLL) return set_error(FPCA_ERR_UNSUPPORTED, "covariance operator: too many nodes");
  FPCA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_band_mfma<d, NCB, STORE, HALF, TAB>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
  hipLaunchKernelGGL((k_band_mfma<d, NCB, STORE, HALF, TAB>), dim3(unsigned(nwg)), dim3(MT), lds, op->ctx->stream, A);
  FPCA_LAUNCH_CHECK("covop band");
  return FPCA_OK;
}

// Units of s-nodes (see BandArgs) of the whole grid.
template <int d>
int band_units(const fpca_covop_s *op) {
  return d == 3 ? op->M[0] : (op->M[0] + 3) / 4;
}

// Blocks of Delta per unit and distance, in bytes.
template <int d>
size_t turned_unit_bytes(const fpca_covop_s *op) {
  const TurnedGeo t = turned_geo(op->M, op->R, d);
  return size_t(d == 3 ? t.nT1 : 1) * t.nB2 * t.nk * t.T2n * 256 * 8;
}
// Workgroups of k_band_mfma per unit, and the distances of coordinate 0.
template <int d>
int64_t unit_wgs(const fpca_covop_s *op) {
  return (d == 3 ? int64_t((op->M[1] + 3) / 4) : 1) * ((op->M[d - 1] + 7) / 8);
}
template <int d>
int half_dists(const fpca_covop_s *op) {
  return d == 3 ? std::min(2 * op->R[0], op->M[0] - 1) + 1 : 1;
}

// All pairs of the launch's units.
template <int d, int NCB, bool STORE>
int launch_all(fpca_covop_s *op, const BandArgs &A) {
  return op->rows ? launch_band_mfma<d, NCB, STORE, false, true>(op, A)
                  : launch_band_mfma<d, NCB, STORE, false, false>(op, A);
}

// Half of the pairs with s in the units A.lo .. A.lo + A.cnt - 1, and their
// transposes: all units and as many distances at a time as there is memory for, or
// one distance and a share of the units.
template <int d, int NCB>
int launch_turned(fpca_covop_s *op, BandArgs A) {
  const TurnedGeo tg = turned_geo(op->M, op->R, d);
  const int units = band_units<d>(op), dists = half_dists<d>(op), ulo = A.lo, uhi = A.lo + A.cnt;
  A.delta = op->delta;
  auto launch = [&]() -> int {
    if (int rc = launch_band_mfma<d, NCB, false, true, true>(op, A)) return rc;
    // the units of t-nodes that the launch's s-nodes reach
    int tlo = 0, tcnt = units;
    if (d == 2) {
      tlo = std::max(0, A.lo - tg.T1h);
      tcnt = std::min(tg.nT1, A.lo + A.cnt + tg.T1h) - tlo;
    } else if (A.ni == 1) {
      tlo = A.lo + half_dt(A.i0);
      tcnt = A.cnt;
    }
    const int64_t nwg = int64_t(tcnt) * (d == 3 ? tg.nT1 : 1) * tg.nT2;
    hipLaunchKernelGGL((k_band_turned<d, NCB>), dim3(unsigned(nwg)), dim3(256), 0, op->ctx->stream, A, tlo);
    FPCA_LAUNCH_CHECK("covop band turned");
    return FPCA_OK;
  };
  for (A.i0 = 0; A.i0 < dists; A.i0 += A.ni) {
    A.ni = std::min(op->delta_dists, dists - A.i0);
    const int dt = half_dt(A.i0);
    const int lo = A.ni == 1 ? std::max(ulo, -dt) : ulo, hi = A.ni == 1 ? std::min(uhi, units - std::max(0, dt)) : uhi;
    if (lo >= hi) continue;
    const int parts = (hi - lo + op->delta_units - 1) / op->delta_units;
    for (int u = 0; u < parts; ++u) {
      A.lo = lo + int(int64_t(hi - lo) * u / parts);
      A.cnt = lo + int(int64_t(hi - lo) * (u + 1) / parts) - A.lo;
      if (int rc = launch()) return rc;
    }
  }
  return FPCA_OK;
}

// k_hsum for cnt s_0 from lo on.
int launch_hsum(fpca_covop_s *op, const CovGeo &g, int lo, int cnt) {
  const int64_t nwg = int64_t(nb256(int64_t(op->M[1]) * op->M[2])) * cnt * (4 * op->R[0] + 1);
  if (nwg > 0x7fffffffLL) return set_error(FPCA_ERR_UNSUPPORTED, "covariance operator: too many nodes");
  hipLaunchKernelGGL(k_hsum, dim3(unsigned(nwg)), dim3(256), 0, op->ctx->stream, g, lo, op->Y2, op->hsum);
  FPCA_LAUNCH_CHECK("covop hsum");
  return FPCA_OK;
}

// d >= 2: at most 32 columns of X per launch (their sums stay in registers). Where
// the sums of k_hsum do not fit for all s_0, they are formed for hs_planes at a time.
template <int d>
int launch_band(fpca_covop_s *op, bool store, const double *X, int r, double *out) {
  BandArgs A = band_args(op, X, r, out);
  const int units = band_units<d>(op), step = d == 3 ? op->hs_planes : units;
  if (store) {
    const int64_t n = op->n_stiles * op->nslot * 4096;
    hipLaunchKernelGGL(k_zero_f64, dim3(unsigned(std::min<int64_t>((n + 255) / 256, 65536))), dim3(256), 0,
                       op->ctx->stream, op->band, n);
    FPCA_LAUNCH_CHECK("covop band zero");
  }
  for (int u = 0; u < units; u += step) {
    A.lo = A.hs0 = u;
    A.cnt = std::min(step, units - u);
    if (step < units)
      if (int rc = launch_hsum(op, A.g, A.lo, A.cnt)) return rc;
    if (store) {
      if (int rc = launch_all<d, 1, true>(op, A)) return rc;
      continue;
    }
    for (A.c0 = 0; A.c0 < r; A.c0 += 32) {
      A.nc = std::min(32, r - A.c0);
      const bool one = A.nc <= 16;
      if (int rc = op->delta ? (one ? launch_turned<d, 1>(op, A) : launch_turned<d, 2>(op, A))
                             : (one ? launch_all<d, 1, false>(op, A) : launch_all<d, 2, false>(op, A)))
        return rc;
    }
  }
  return FPCA_OK;
}

// Memory for Delta's blocks, up to 512 MB for d = 3 (64^3 nodes, R = 6, one product:
// 120 ms with 256, 114 with 512, 113 with 1024) and 1024 MB for d = 2 (100^2 nodes,
// R = 28: 3.2 ms with 256, 2.3 with 512, 1.9 with 1024). Where all units' blocks fit, as many
// distances as do go into a launch. Otherwise a launch takes one distance and so
// many units that its workgroups, one per CU at a time, fill whole rounds of the
// CUs. Without the memory, or where a launch would leave half of the CUs without
// work (all pairs are formed in about the same time then), products form all pairs.
template <int d>
void reserve_delta(fpca_covop_s *op) {
  const size_t unit = turned_unit_bytes<d>(op);
  const int units = band_units<d>(op);
  const int64_t wgs = unit_wgs<d>(op), cus = op->ctx->num_cus;
  if (!op->rows) return;
  for (size_t budget = size_t(d == 3 ? 512 : 1024) << 20; budget >= unit; budget /= 2) {
    int64_t u = std::min<int64_t>(units, int64_t(budget / unit)), dists = 1;
    if (u == units)
      dists = std::min<int64_t>(half_dists<d>(op), int64_t(budget / unit) / units);
    else if (u * wgs >= cus)
      u = u * wgs / cus * cus / wgs;
    else if (2 * u * wgs < cus)
      return;
    void *p = nullptr;
    if (optional_alloc(op->ctx, &p, unit * size_t(u * dists))) {
      op->delta = static_cast<double *>(p);
      op->delta_units = int(u);
      op->delta_dists = int(dists);
      return;
    }
  }
}

template <int d>
int launch_band_apply(fpca_covop_s *op, const double *X, int r, double *out) {
  BandArgs A{};
  A.g = make_geo(op);
  A.X = X;
  A.r = r;
  A.out = out;
  A.band = op->band;
  const size_t lds = size_t(64 * 65 + 64 * 64) * 8;
  FPCA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_band_apply<d>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)));
  hipLaunchKernelGGL((k_band_apply<d>), dim3(unsigned(op->n_stiles)), dim3(BT), lds, op->ctx->stream, A);
  FPCA_LAUNCH_CHECK("covop band apply");
  return FPCA_OK;
}

int band_dispatch(fpca_covop_s *op, bool store, const double *X, int r, double *out) {
  switch (op->d) {
    case 1: return store ? launch_band1<true>(op, X, r, out) : launch_band1<false>(op, X, r, out);
    case 2: return launch_band<2>(op, store, X, r, out);
    default: return launch_band<3>(op, store, X, r, out);
  }
}

}  // namespace

int covop_apply_internal(fpca_covop_s *op, int r, const double *X, double *out) {
  fpca_context *ctx = op->ctx;
  const CovGeo g = make_geo(op);
  const int rows = int(2 * op->n + 1);
  hipLaunchKernelGGL(k_lr_partial, dim3(unsigned(op->lr_blocks), unsigned((op->n + 63) / 64)), dim3(256), 0,
                     ctx->stream, g, r, X, op->Ln, op->Bn, op->mu, op->lr_part);
  FPCA_LAUNCH_CHECK("covop lr partial");
  hipLaunchKernelGGL(k_lr_reduce, dim3(unsigned(rows)), dim3(256), 0, ctx->stream, op->lr_blocks, rows, r,
                     op->lr_part, op->lr_tot);
  FPCA_LAUNCH_CHECK("covop lr reduce");
  hipLaunchKernelGGL(k_lr_out, dim3(unsigned((op->P + 63) / 64)), dim3(256), 0, ctx->stream, g, r, op->Ln, op->Bn,
                     op->mu, op->lr_tot, out);
  FPCA_LAUNCH_CHECK("covop lr out");
  if (op->mode == FPCA_COVOP_STORE_BAND) {
    switch (op->d) {
      case 1: return launch_band_apply<1>(op, X, r, out);
      case 2: return launch_band_apply<2>(op, X, r, out);
      default: return launch_band_apply<3>(op, X, r, out);
    }
  }
  return band_dispatch(op, false, X, r, out);
}

}  // namespace fpca

using namespace fpca;

extern "C" int fpca_covop_create(fpca_handle ctx, const fpca_grid *grid, int64_t n, const double *Y,
                                 const double *mu, const double *bandwidth, int mode, fpca_covop *op_out) {
  if (int rc = check_handle(ctx)) return rc;
  int64_t P;
  if (int rc = check_grid(grid, &P)) return rc;
  if (!op_out) return set_error(FPCA_ERR_INVALID_ARG, "op is required");
  *op_out = nullptr;
  if (!Y || !mu || !bandwidth) return set_error(FPCA_ERR_INVALID_ARG, "Y, mu and bandwidth are required");
  if (grid->mask) return set_error(FPCA_ERR_UNSUPPORTED, "the covariance operator takes the full rectangle only");
  if (n < 1 || n > (int64_t(1) << 20)) return set_error(FPCA_ERR_INVALID_ARG, "need 1 <= n <= 2^20");
  if (mode != FPCA_COVOP_RECOMPUTE && mode != FPCA_COVOP_STORE_BAND)
    return set_error(FPCA_ERR_INVALID_ARG, "bad mode %d", mode);
  const int d = grid->d;
  const int rmax = d == 3 ? 6 : (d == 2 ? 28 : 2016);
  auto *op = new fpca_covop_s();
  op->ctx = ctx;
  op->d = d;
  op->P = P;
  op->n = n;
  op->mode = mode;
  std::vector<double> htab;
  for (int k = 0; k < d; ++k) {
    const int M = grid->M[k];
    const double h = bandwidth[k];
    if (!(h > 0.0) || !std::isfinite(h)) {
      delete op;
      return set_error(FPCA_ERR_INVALID_ARG, "bandwidths must be positive and finite");
    }
    const double H = h * double(M - 1);
    const int R = std::min(int(std::floor(H)), M - 1);
    if (R < 1 || R > rmax) {
      delete op;
      return set_error(FPCA_ERR_UNSUPPORTED, "coordinate %d: window of %d grid steps (need 1..%d)", k, R, rmax);
    }
    op->M[k] = M;
    op->R[k] = R;
    op->H[k] = H;
    // taps, window sums and shared-node sums
    std::vector<double> K(2 * R + 1), U(2 * R + 1);
    for (int m = -R; m <= R; ++m) {
      const double u = double(m) / H;
      K[m + R] = std::fabs(u) < 1.0 ? 1.0 - u * u : 0.0;
      U[m + R] = u;
    }
    std::vector<double> W(size_t(M) * 3), E(size_t(M) * (4 * R + 1) * 6, 0.0);
    for (int x = 0; x < M; ++x) {
      double w0 = 0, w1 = 0, w2 = 0;
      for (int m = -std::min(R, x); m <= std::min(R, M - 1 - x); ++m) {
        w0 += K[m + R];
        w1 += K[m + R] * U[m + R];
        w2 += K[m + R] * U[m + R] * U[m + R];
      }
      W[x * 3] = w0;
      W[x * 3 + 1] = w1;
      W[x * 3 + 2] = w2;
      const double a = w1 / w0, v = w2 / w0 - a * a;
      if (!(w0 > 0.0) || !(v >= 1e-8 * (w2 / w0))) {
        delete op;
        return set_error(FPCA_ERR_UNSUPPORTED, "coordinate %d: degenerate window at node %d", k, x);
      }
      for (int dl = -2 * R; dl <= 2 * R; ++dl) {
        const int t = x + dl;
        if (t < 0 || t >= M) continue;
        double e[6] = {0, 0, 0, 0, 0, 0};
        for (int p = std::max(std::max(x, t) - R, 0); p <= std::min(std::min(x, t) + R, M - 1); ++p) {
          const double kk = K[p - x + R] * K[p - t + R], us = U[p - x + R], vt = U[p - t + R];
          e[0] += kk;
          e[1] += kk * us;
          e[2] += kk * vt;
          e[3] += kk * us * us;
          e[4] += kk * us * vt;
          e[5] += kk * vt * vt;
        }
        for (int j = 0; j < 6; ++j) E[(size_t(x) * (4 * R + 1) + dl + 2 * R) * 6 + j] = e[j];
      }
    }
    op->tab_K[k] = int64_t(htab.size());
    htab.insert(htab.end(), K.begin(), K.end());
    op->tab_U[k] = int64_t(htab.size());
    htab.insert(htab.end(), U.begin(), U.end());
    op->tab_W[k] = int64_t(htab.size());
    htab.insert(htab.end(), W.begin(), W.end());
    op->tab_E[k] = int64_t(htab.size());
    htab.insert(htab.end(), E.begin(), E.end());
    op->tab_nd[k] = int64_t(htab.size());
    for (int x = 0; x < M; ++x) {
      const double a = W[x * 3 + 1] / W[x * 3], v = W[x * 3 + 2] / W[x * 3] - a * a;
      htab.insert(htab.end(), {1.0 / W[x * 3], a * a / v, a / v});
    }
    const int TB = d == 1 ? 64 : (d == 2 ? 8 : 4);
    op->tb[k] = TB;
    op->nt[k] = (M + TB - 1) / TB;
    op->span[k] = (2 * R + TB - 1) / TB;
  }
  op->n_stiles = 1;
  op->nslot = 1;
  for (int k = 0; k < d; ++k) {
    op->n_stiles *= op->nt[k];
    op->nslot *= 2 * op->span[k] + 1;
  }
  op->lr_blocks = (P + 63) / 64;
  // d >= 2: pair classes of every coordinate: one per offset for the pairs R
  // or more from the border, then one per pair (s, t) near the left border;
  // pairs near the right border alone are those mirrored (u and v change sign,
  // and with them the entries of the row that go with them). The rows' number
  // depends on the windows, not on the curves: R = 6 on d = 3 up to 175 classes per
  // coordinate, 343 MB; R = 28 on d = 2 up to 3277, 687 MB.
  std::vector<int> itab;
  int64_t cls_off[3] = {0, 0, 0}, rep_off[3] = {0, 0, 0}, nrows = 0;
  if (d >= 2) {
    nrows = 1;
    for (int k = 0; k < d; ++k) {
      const int M = op->M[k], R = op->R[k], wd = 4 * R + 1;
      std::vector<int> rep(wd, -1), cls(size_t(M) * wd, 0);
      for (int x = 0; x < M; ++x)
        for (int j = 0; j < wd; ++j) {
          const int t = x + j - 2 * R;
          if (t < 0 || t >= M) continue;
          if (std::min(x, t) >= R && std::max(x, t) <= M - 1 - R) {
            rep[j] = x * wd + j;
            cls[size_t(x) * wd + j] = 2 * j;
          } else if (std::min(x, t) < R) {
            cls[size_t(x) * wd + j] = 2 * int(rep.size());
            rep.push_back(x * wd + j);
          }
        }
      for (int x = 0; x < M; ++x)
        for (int j = 0; j < wd; ++j) {
          const int t = x + j - 2 * R;
          if (t < 0 || t >= M || std::min(x, t) < R || std::max(x, t) <= M - 1 - R) continue;
          cls[size_t(x) * wd + j] = cls[size_t(M - 1 - x) * wd + (4 * R - j)] + 1;
        }
      cls_off[k] = int64_t(itab.size());
      itab.insert(itab.end(), cls.begin(), cls.end());
      rep_off[k] = int64_t(itab.size());
      itab.insert(itab.end(), rep.begin(), rep.end());
      op->ncls[k] = int(rep.size());
      nrows *= op->ncls[k];
    }
  }
  const int F = d + 1;
  // filtered curves: node-major for d = 1, in blocks of 16 nodes above
  const int64_t nblk16 = d == 1 ? 0 : (d == 3 ? op->M[0] : 1) * int64_t((op->M[d - 2] + 3) / 4) * ((op->M[d - 1] + 3) / 4);
  const size_t zn_n = d == 1 ? size_t(P) * F * n : size_t(nblk16) * F * size_t((n + 1) / 2) * 32;
  const size_t lr_n = size_t(op->lr_blocks) * (2 * n + 1) * 64;
  const size_t bytes_zn = carve_bytes(zn_n, 8), bytes_pfn = d == 1 ? 0 : carve_bytes(size_t(P) * F * n, 8);
  const size_t bytes_main = 2 * carve_bytes(size_t(P) * n, 8) + 2 * carve_bytes(P, 8) + carve_bytes(htab.size(), 8) +
                            carve_bytes(lr_n, 8) + carve_bytes(size_t(2 * n + 1) * 64, 8);
  const size_t bytes_band =
      mode == FPCA_COVOP_STORE_BAND ? carve_bytes(size_t(op->n_stiles) * op->nslot * 4096, 8) : 0;
  const size_t bytes_rows = carve_bytes(size_t(nrows) * 8, 8), bytes_tables = carve_bytes(itab.size(), 4) + bytes_rows;
  // k_hsum's sums of one s_0
  const size_t bytes_plane = d == 3 ? size_t(4 * op->R[0] + 1) * 3 * op->M[1] * op->M[2] * 8 : 0;
  double *pfn = nullptr;  // node-major filtered curves, until they are in blocks
  auto fail = [&](int rc) {
    if (pfn) (void)hipFree(pfn);
    free_op(op);
    return rc;
  };
  if (int rc = set_device(ctx)) return fail(rc);
  {
    // the band's blocks follow once the node-major curves are gone
    size_t free_b = 0, total_b = 0;
    const size_t need = bytes_main + bytes_zn + std::max(bytes_pfn, bytes_band + bytes_plane);
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) return fail(set_error(FPCA_ERR_DEVICE, "hipMemGetInfo failed"));
    if (need > free_b)
      return fail(set_error(FPCA_ERR_WORKSPACE, "covariance operator needs %zu bytes, %zu free", need, free_b));
  }
  auto device_alloc = [&](auto **p, size_t bytes) {
    if (hipMalloc(reinterpret_cast<void **>(p), bytes) == hipSuccess) return true;
    *p = nullptr;
    (void)hipGetLastError();
    return false;
  };
  if (!device_alloc(&op->mem, bytes_main) || !device_alloc(&op->Zn, bytes_zn) || (d >= 2 && !device_alloc(&pfn, bytes_pfn)))
    return fail(set_error(FPCA_ERR_WORKSPACE, "hipMalloc failed"));
  Carver cv{op->mem, 0, bytes_main};
  op->Ln = cv.take<double>(size_t(P) * n);
  op->Bn = cv.take<double>(size_t(P) * n);
  op->Y2 = cv.take<double>(P);
  op->mu = cv.take<double>(P);
  op->tab = cv.take<double>(htab.size());
  op->lr_part = cv.take<double>(lr_n);
  op->lr_tot = cv.take<double>(size_t(2 * n + 1) * 64);
  hipStream_t s = ctx->stream;
  if (hipMemcpyAsync(op->tab, htab.data(), htab.size() * 8, hipMemcpyHostToDevice, s) != hipSuccess ||
      hipMemcpyAsync(op->mu, mu, size_t(P) * 8, hipMemcpyDeviceToDevice, s) != hipSuccess)
    return fail(set_error(FPCA_ERR_DEVICE, "copy failed"));
  // the transposed curves take the place of the products' partial sums (which are
  // larger); the passes alternate between pfn and the operator's block, and the
  // curves end in the latter
  double *Yn = op->lr_part, *last = d == 1 ? op->Zn : pfn, *tmp = op->Zn;
  CovGeo g = make_geo(op);
  int rc = FPCA_OK;
  do {
    hipLaunchKernelGGL(k_transpose, dim3(unsigned((P + 31) / 32), unsigned((n + 31) / 32)), dim3(32, 8), 0, s, n, P,
                       Y, Yn);
    if (hipGetLastError() != hipSuccess) {
      rc = set_error(FPCA_ERR_DEVICE, "transpose launch failed");
      break;
    }
    hipLaunchKernelGGL(k_sq, dim3(nb256(P)), dim3(256), 0, s, P, int(n), Yn, op->Y2);
    // separable passes, last coordinate first; the last pass lands in `last`
    const double *in = Yn;
    int Fin = 1;
    for (int pass = 0; pass < d && rc == FPCA_OK; ++pass) {
      const int k = d - 1 - pass;
      double *dst = ((d - 1 - pass) % 2 == 0) ? last : tmp;
      FilterMap fm{};
      fm.nmap = 0;
      fm.fo[fm.nmap] = 0, fm.fi[fm.nmap] = 0, fm.e[fm.nmap] = 0, ++fm.nmap;
      fm.fo[fm.nmap] = k + 1, fm.fi[fm.nmap] = 0, fm.e[fm.nmap] = 1, ++fm.nmap;
      for (int j = k + 1; j < d; ++j) fm.fo[fm.nmap] = j + 1, fm.fi[fm.nmap] = j + 1, fm.e[fm.nmap] = 0, ++fm.nmap;
      hipLaunchKernelGGL(k_filter, dim3(nb256(P * n), unsigned(fm.nmap)), dim3(256), 0, s, g, k, in, Fin, dst, F, fm);
      if (hipGetLastError() != hipSuccess) rc = set_error(FPCA_ERR_DEVICE, "filter launch failed");
      in = dst;
      Fin = F;
    }
    if (rc != FPCA_OK) break;
    hipLaunchKernelGGL(k_lr_prep, dim3(nb256(P * n)), dim3(256), 0, s, g, last, op->Ln, op->Bn);
    if (d >= 2) hipLaunchKernelGGL(k_retile, dim3(unsigned(nblk16), unsigned(F)), dim3(256), 0, s, g, last, op->Zn);
    if (hipGetLastError() != hipSuccess) rc = set_error(FPCA_ERR_DEVICE, "prep launch failed");
  } while (false);
  // pfn, the host's tables and the caller's Y are done with once the stream is
  const hipError_t e1 = hipStreamSynchronize(s);
  if (pfn) (void)hipFree(pfn);
  pfn = nullptr;
  if (rc != FPCA_OK) return fail(rc);
  if (e1 != hipSuccess) return fail(hip_fail(e1, "covariance operator set-up"));
  if (bytes_band && !device_alloc(&op->band, bytes_band))
    return fail(set_error(FPCA_ERR_WORKSPACE, "hipMalloc of the band failed"));
  if (d >= 2) {
    // The table of rows and k_hsum's sums of all s_0 are held where they fit; else
    // the rows are solved for and the sums formed for fewer s_0 at a time.
    if (d == 3) {
      op->hs_planes = op->M[0];
      while (op->hs_planes > 1 &&
             !optional_alloc(ctx, reinterpret_cast<void **>(&op->hsum), bytes_plane * op->hs_planes))
        op->hs_planes = (op->hs_planes + 1) / 2;
      if (!op->hsum && !device_alloc(&op->hsum, bytes_plane))
        return fail(set_error(FPCA_ERR_WORKSPACE, "hipMalloc failed"));
      if (op->hs_planes == op->M[0]) rc = launch_hsum(op, g, 0, op->M[0]);
    }
    if (rc == FPCA_OK && optional_alloc(ctx, reinterpret_cast<void **>(&op->tables), bytes_tables)) {
      double *rows = reinterpret_cast<double *>(op->tables);
      const int *ditab = reinterpret_cast<const int *>(op->tables + bytes_rows);
      if (hipMemcpyAsync(op->tables + bytes_rows, itab.data(), itab.size() * 4, hipMemcpyHostToDevice, s) != hipSuccess)
        return fail(set_error(FPCA_ERR_DEVICE, "copy failed"));
      for (int k = 0; k < d; ++k) op->cls[k] = ditab + cls_off[k];
      op->rows = rows;
      g = make_geo(op);
      const int *rp[3] = {ditab + rep_off[0], ditab + rep_off[1], ditab + rep_off[2]};
      const dim3 wg(unsigned((nrows + 63) / 64));
      if (d == 2)
        hipLaunchKernelGGL(k_wtab<2>, wg, dim3(64), 0, s, g, nrows, rp[0], rp[1], rp[2], rows);
      else
        hipLaunchKernelGGL(k_wtab<3>, wg, dim3(64), 0, s, g, nrows, rp[0], rp[1], rp[2], rows);
      if (hipGetLastError() != hipSuccess) rc = set_error(FPCA_ERR_DEVICE, "table launch failed");
    }
  }
  if (rc == FPCA_OK && mode == FPCA_COVOP_STORE_BAND) rc = band_dispatch(op, true, nullptr, 0, nullptr);
  const hipError_t e2 = hipStreamSynchronize(s);
  if (rc != FPCA_OK) return fail(rc);
  if (e2 != hipSuccess) return fail(hip_fail(e2, "covariance operator set-up"));
  if (mode == FPCA_COVOP_STORE_BAND) {
    // products read the band and the low-rank part only
    for (auto **p : {&op->Zn, &op->hsum}) {
      if (*p) (void)hipFree(*p);
      *p = nullptr;
    }
    if (op->tables) (void)hipFree(op->tables);
    op->tables = nullptr;
    op->rows = nullptr;
    for (int k = 0; k < 3; ++k) op->cls[k] = nullptr;
  } else if (d == 2) {
    reserve_delta<2>(op);
  } else if (d == 3) {
    reserve_delta<3>(op);
  }
  *op_out = op;
  return FPCA_OK;
}

extern "C" int fpca_covop_apply(fpca_covop op, int r, const double *X, double *out) {
  if (!op) return set_error(FPCA_ERR_INVALID_ARG, "null operator");
  if (int rc = check_handle(op->ctx)) return rc;
  if (r < 1 || r > 64) return set_error(FPCA_ERR_INVALID_ARG, "need 1 <= r <= 64");
  if (!X || !out) return set_error(FPCA_ERR_INVALID_ARG, "X and out are required");
  if (int rc = set_device(op->ctx)) return rc;
  return covop_apply_internal(op, r, X, out);
}

extern "C" int fpca_covop_destroy(fpca_covop op) {
  if (!op) return FPCA_OK;
  if (op->ctx) (void)hipSetDevice(op->ctx->device);
  if (op->ctx && op->ctx->stream) (void)hipStreamSynchronize(op->ctx->stream);
  free_op(op);
  return FPCA_OK;
}
