// Covariance smoother for general pair weights (eq. 2.4 on the 2d-dimensional
// grid, any C; d = 2 and 3) in three kernels, and its cross-validation scores.
//
// The moments of the local-linear fit factor over the 2d coordinates, so they
// are formed by 1-D passes with the taps (1-u^2) u^e, e = 0..2, in FP64:
//   t-coordinates   C with t-degree <= 2, G with t-degree <= 1: 9 arrays for
//                   d = 2, 14 for d = 3 (X);
//   s_d .. s_2      14 and 27 arrays (Y);
//   s_1             the final moments of a block of nodes, into LDS, then one
//                   lane per node solves its system (wls_b0).
// d = 2: k_stage_ts2 forms Y of one (s_1, t_1) straight from C and G (the window
// of t_1 read from L2, everything else in LDS), then k_stage_w. d = 3: k_stage_t3
// (X), k_stage_s3 (Y of a range of t-columns), k_stage_w on that range.
// In the passes over lines a thread holds a whole line of at most N values in
// registers and forms all its outputs from them: an input is read once, no index
// is computed per tap and no tap is multiplied outside the window; taps have the
// same index in every lane and come through scalar loads. Between passes a line
// changes direction through LDS. N (16, 24, 32, 40) is the longest coordinate
// rounded up.
//
// Bound: the FP64 arrays between the kernels, 112 bytes written per node for
// d = 2, 112 and 216 for d = 3.
// C and G are symmetric, so cross-validation needs the nodes s_1 <= t_1 only: the
// stages skip the rows and columns that no such node reads.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

#include "common.hpp"
#include "staged.hpp"
#include "wls.hpp"

namespace fpca {
namespace {

// Columns per stage-W workgroup and MB of Y at a time (d = 3, N = 16): 16^6 nodes,
// 20 CV jobs: 43 ms; 8 columns 45; 128 MB 45, 256 MB 45, all of Y (3.6 GB) 49.
constexpr int QBW = 16;
constexpr int YCHUNK = 512;
// Jobs per launch (blockIdx.z). 80 jobs, 1 / 4 / 8 / 16 per launch: 16^2 nodes 2.36,
// 0.94, 0.69 and 0.56 ms, 24^2 3.78, 2.20, 1.92 and 1.93, 32^2 9.4, 8.6, 8.3 and 8.1 (16:
// twice the kernel arguments).
constexpr int SB_MAX = 8;
constexpr int SC_TILE = 32;  // score tile
constexpr int SC_WG = 2048;   // score workgroups per job, at most

struct SJob {
  const void *Ca, *Cb, *Ga, *Gb, *Qf, *Gf, *Cf;
  double c0;
  double h[3];
  int R[3];
  double *taps;  // [coordinate][e][TAPW], centred
  double *X, *Y;
  void *b0;  // P x P of T
  double *part;
};
struct SBatch {
  int M[3];
  int P, PR;  // nodes, s-positions per s_1 index
  int cv;
  const uint8_t *mask;
  int8_t *status;
  SJob j[SB_MAX];
};

constexpr int NMAX = 40;  // longest coordinate
constexpr int TAPC = NMAX + 2;     // centre of a tap table
constexpr int TAPW = 2 * TAPC + 1;
typedef const __attribute__((address_space(4))) double CTap;
__device__ inline CTap *taps_of(const SJob &jb, int k, int e) { return (CTap *)(jb.taps + (k * 3 + e) * TAPW + TAPC); }

__global__ void k_staged_taps(SBatch b, int d) {
  const SJob &jb = b.j[blockIdx.z];
  const int k = blockIdx.y;
  for (int i = threadIdx.x; i < 3 * TAPW; i += blockDim.x) {
    const int e = i / TAPW, m = i % TAPW - TAPC;
    const double u = double(m) / (jb.h[k] * double(b.M[k] - 1));
    const double K = fabs(u) < 1.0 ? 1.0 - u * u : 0.0;
    jb.taps[(k * 3 + e) * TAPW + m + TAPC] = K * (e == 0 ? 1.0 : (e == 1 ? u : u * u));
  }
}

// Adds the taps k and -k, k = K .. R, to out[o] = sum over k of t[k] v[O0 + o + k]
// (v zero outside 0 .. N - 1); k <= R holds for every lane or for none. (p0, m0)
// and (p1, m1): the taps of K and K + 1, requested two steps ahead (the table
// reaches NMAX + 2).
template <int K, int N, int O0, int NO>
__device__ inline void line_taps(const double (&v)[N], CTap *t, int R, double (&out)[NO], double p0, double m0, double p1,
                                 double m1) {
  if constexpr (K < N) {
    if (K > R) return;
    const double p2 = t[K + 2], m2 = t[-K - 2];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
      if (O0 + o + K < N) out[o] = fma(p0, v[O0 + o + K < N ? O0 + o + K : 0], out[o]);
      if (O0 + o - K >= 0) out[o] = fma(m0, v[O0 + o - K >= 0 ? O0 + o - K : 0], out[o]);
    }
    line_taps<K + 1, N, O0, NO>(v, t, R, out, p1, m1, p2, m2);
  }
}

// The outputs of a line, st(x, value) for x < n, in two halves for N > 16.
template <int N, int O0 = 0, typename ST>
__device__ inline void line_out(const double (&v)[N], CTap *t, int R, int n, ST st) {
  constexpr int NO = N <= 16 ? N : N / 2;
  const double c = t[0], p1 = t[1], m1 = t[-1], p2 = t[2], m2 = t[-2];
  double out[NO];
#pragma unroll
  for (int o = 0; o < NO; ++o) out[o] = c * v[O0 + o];
  line_taps<1, N, O0, NO>(v, t, R, out, p1, m1, p2, m2);
#pragma unroll
  for (int o = 0; o < NO; ++o)
    if (O0 + o < n) st(O0 + o, out[o]);
  if constexpr (O0 + NO < N) line_out<N, O0 + NO>(v, t, R, n, st);
}

template <int N, typename LD>
__device__ inline void line_load(double (&v)[N], int n, LD ld) {
#pragma unroll
  for (int x = 0; x < N; ++x) v[x] = x < n ? ld(x) : 0.0;
}

// The array x of X: family, t-degree and the first of its arrays of Y.
template <int d>
__device__ inline void x_array(int x, int &fam, int &deg, int &y0) {
  int i = 0, y = 0;
  fam = deg = y0 = 0;
  for (int f = 0; f < 2; ++f) {
    const int md = 2 - f;
    for (int e3 = 0; e3 <= (d == 3 ? md : 0); ++e3)
      for (int e2 = 0; e2 <= md - e3; ++e2)
        for (int e1 = 0; e1 <= md - e3 - e2; ++e1) {
          const int dg = e1 + e2 + e3, left = md - dg;
          if (i == x) {
            fam = f;
            deg = dg;
            y0 = y;
          }
          ++i;
          y += d == 2 ? left + 1 : (left + 1) * (left + 2) / 2;
        }
  }
}

// ------------------------------------------------------------------ d = 2
// Workgroup (t_1 = blockIdx.x, s_1 = blockIdx.y, family = blockIdx.z % 2: C or
// G): the M_2 x M_2 nodes (s_2, t_2).
//   1. the t_1 sums at every (s_2, t_2) with the family's 3 or 2 taps;
//   2. t_2 lines of those arrays to the 6 or 3 arrays X;
//   3. s_2 lines of X to the 10 or 4 arrays Y.
// The families apart: 51 KB of LDS and several workgroups per CU, whose phases
// overlap (both together, 76 KB, ran one per CU: 72 against 47 us for 32^4 nodes, R = 2).
// Whole s-rows per workgroup with X in memory between two kernels: 69 us.
template <typename T, int N>
__global__ __launch_bounds__(256) void k_stage_ts2(SBatch b) {
  extern __shared__ double lds[];  // [6][M2][S], the first arrays of it in step 1
  const SJob &jb = b.j[blockIdx.z >> 1];
  const int fam = blockIdx.z & 1;
  const int M1 = b.M[0], M2 = b.M[1], P = b.P, S = M2 | 1, tid = threadIdx.x;
  const int t1 = blockIdx.x, s1 = blockIdx.y, R1 = jb.R[0];
  if (b.cv && s1 > t1 + R1) return;  // no node s_1 <= t_1 reads it
  const int A = M2 * S;
  {
    const T *Wa = static_cast<const T *>(fam ? jb.Ga : jb.Ca), *Wb = static_cast<const T *>(fam ? jb.Gb : jb.Cb);
    CTap *k0 = taps_of(jb, 0, 0), *k1 = taps_of(jb, 0, 1), *k2 = taps_of(jb, 0, 2);
    const int lo = max(-R1, -t1), hi = min(R1, M1 - 1 - t1);
    // WA, WB: whether the family W = Wa - Wb has its arrays (no Wa: c0 off the
    // diagonal); UB rows of the window requested at once
    auto sums = [&](auto wa, auto wb) {
      constexpr bool WA = decltype(wa)::value, WB = decltype(wb)::value;
      constexpr int UB = 8;
      for (int e = tid; e < M2 * M2; e += 256) {
        const int s2 = e / M2, t2 = e - s2 * M2, p = s1 * M2 + s2;
        const int64_t base = int64_t(p) * P + t1 * M2 + t2;
        double a0 = 0.0, a1 = 0.0, a2 = 0.0;
        for (int k = lo; k <= hi; k += UB) {
          T va[UB], vb[UB];
#pragma unroll
          for (int u = 0; u < UB; ++u) {
            const int64_t i = base + min(k + u, hi) * M2;
            if constexpr (WA) va[u] = Wa[i];
            if constexpr (WB) vb[u] = Wb[i];
          }
#pragma unroll
          for (int u = 0; u < UB; ++u) {
            if (k + u > hi) break;  // the same for every lane
            double w;
            if constexpr (WA)
              w = double(va[u]);
            else
              w = (t1 + k + u) * M2 + t2 == p ? 0.0 : jb.c0;
            if constexpr (WB) w -= double(vb[u]);
            a0 = fma(k0[k + u], w, a0);
            a1 = fma(k1[k + u], w, a1);
            if (!fam) a2 = fma(k2[k + u], w, a2);
          }
        }
        double *o = lds + s2 * S + t2;
        o[0] = a0;
        o[A] = a1;
        if (!fam) o[2 * A] = a2;
      }
    };
    if (!Wa)
      sums(std::false_type(), std::false_type());
    else if (!Wb)
      sums(std::true_type(), std::false_type());
    else
      sums(std::true_type(), std::true_type());
  }
  const int md = 2 - fam;
  __syncthreads();
  {
    // line (e1, s_2): the array with t_1 exponent e1 gives e_2 = 0 .. md - e1
    const int e1 = tid / M2, s2 = tid - e1 * M2;
    const bool on = e1 <= md;
    double v[N];
    if (on) line_load<N>(v, M2, [&](int x) { return lds[e1 * A + s2 * S + x]; });
    __syncthreads();  // X overwrites the lines
    for (int e2 = 0; e2 <= md; ++e2) {
      if (on && e2 <= md - e1) {
        // X of (e_2, e_1) in the order of x_array
        const int x = fam ? 2 * e2 + e1 : (e2 == 0 ? e1 : (e2 == 1 ? 3 + e1 : 5));
        double *o = lds + x * A + s2 * S;
        line_out<N>(v, taps_of(jb, 1, e2), jb.R[1], M2, [&](int i, double val) { o[i] = val; });
      }
    }
  }
  __syncthreads();
  {
    const int x = tid / M2, t2 = tid - x * M2;
    if (x < (fam ? 3 : 6)) {
      int f, deg, y0;
      x_array<2>(x + 6 * fam, f, deg, y0);
      double v[N];
      line_load<N>(v, M2, [&](int i) { return lds[x * A + i * S + t2]; });
      double *Y = jb.Y + int64_t(s1) * M2 * P + t1 * M2 + t2;
      const int64_t PP = int64_t(P) * P;
      for (int e = 0; e <= md; ++e) {
        if (e <= md - deg) {
          double *Ye = Y + (y0 + e) * PP;
          line_out<N>(v, taps_of(jb, 1, e), jb.R[1], M2, [&](int i, double val) { Ye[int64_t(i) * P] = val; });
        }
      }
    }
  }
}

// ------------------------------------------------------------------ d = 3
// X of one s-row per workgroup, the t-block in LDS between passes; the threads
// cover the lines of each pass (M_1 M_2, M_1 M_3, M_2 M_3 of them). With N = 16 a
// thread has one t_3 line at most and keeps it for all three exponents.
template <typename T, int N>
__global__ __launch_bounds__(256) void k_stage_t3(SBatch b) {
  extern __shared__ double lds[];
  const SJob &jb = b.j[blockIdx.z];
  const int M1 = b.M[0], M2 = b.M[1], M3 = b.M[2], P = b.P, p = blockIdx.x;
  const int64_t PP = int64_t(P) * P;
  const int S3 = M3 | 1;  // odd row length: the t_3 lines of neighbouring threads meet different banks
  double *B1 = lds, *B2 = lds + M1 * M2 * S3;
  // cross-validation reads X at t_1 >= s_1 - R_1 only; those need t_1 >= s_1 - 2 R_1
  const int x1 = b.cv ? max(0, p / b.PR - jb.R[0]) : 0, i1 = b.cv ? max(0, x1 - jb.R[0]) : 0;
  int xi = 0;
  for (int fam = 0; fam < 2; ++fam) {
    const T *A = static_cast<const T *>(fam == 0 ? jb.Ca : jb.Ga), *B = static_cast<const T *>(fam == 0 ? jb.Cb : jb.Gb);
    const int md = 2 - fam;
    double v[N];
    for (int e3 = 0; e3 <= md; ++e3) {
      for (int l = threadIdx.x + i1 * M2; l < M1 * M2; l += 256) {
        if (N > 16 || e3 == 0) {
          const int64_t base = int64_t(p) * P + l * M3;
          const int diag = p - l * M3;
          if (!A)
            line_load<N>(v, M3, [&](int x) { return x == diag ? 0.0 : jb.c0; });
          else if (B)
            line_load<N>(v, M3, [&](int x) { return double(A[base + x]) - double(B[base + x]); });
          else
            line_load<N>(v, M3, [&](int x) { return double(A[base + x]); });
        }
        line_out<N>(v, taps_of(jb, 2, e3), jb.R[2], M3, [&](int x, double o) { B1[l * S3 + x] = o; });
      }
      __syncthreads();
      for (int e2 = 0; e2 <= md - e3; ++e2) {
        for (int l = threadIdx.x + i1 * M3; l < M1 * M3; l += 256) {
          const int t1 = l / M3, t3 = l - t1 * M3;
          double w[N];
          line_load<N>(w, M2, [&](int x) { return B1[(t1 * M2 + x) * S3 + t3]; });
          line_out<N>(w, taps_of(jb, 1, e2), jb.R[1], M2, [&](int x, double o) { B2[(t1 * M2 + x) * S3 + t3] = o; });
        }
        __syncthreads();
        for (int l = threadIdx.x; l < M2 * M3; l += 256) {
          const int t2 = l / M3, t3 = l - t2 * M3;
          double w[N];
          line_load<N>(w, M1, [&](int x) { return x >= i1 ? B2[(x * M2 + t2) * S3 + t3] : 0.0; });
          for (int e1 = 0; e1 <= md - e3 - e2; ++e1) {
            double *X = jb.X + (xi + e1) * PP + int64_t(p) * P + l;
            line_out<N>(w, taps_of(jb, 0, e1), jb.R[0], M1, [&](int x, double o) {
              if (x >= x1) X[int64_t(x) * M2 * M3] = o;
            });
          }
        }
        xi += md - e3 - e2 + 1;
        __syncthreads();
      }
    }
  }
}

// Y of the columns qlo .. qlo + nc - 1: a workgroup takes an s_1 index, 16 t
// columns and one array of X: thread (s_2, column) passes the s_3 line, then (s_3, column) the s_2 line.
constexpr int QS = 16;
template <int N>
__global__ __launch_bounds__(256) void k_stage_s3(SBatch b, int nx, int qlo, int nc) {
  extern __shared__ double lds[];  // [s_2][s_3][QS]
  const SJob &jb = b.j[int(blockIdx.z) / nx];
  const int x = int(blockIdx.z) % nx;
  const int M2 = b.M[1], M3 = b.M[2], P = b.P, a1 = blockIdx.y;
  const int64_t PP = int64_t(P) * P, YS = int64_t(P) * nc;
  const int q0 = qlo + int(blockIdx.x) * QS, c = threadIdx.x % QS, q = q0 + c;
  if (b.cv && a1 > min(q0 + QS - 1, P - 1) / b.PR + jb.R[0]) return;
  int fam, deg, y0;
  x_array<3>(x, fam, deg, y0);
  const int md = 2 - fam - deg;
  const double *X = jb.X + x * PP + int64_t(a1) * b.PR * P + min(q, P - 1);
  double *Y = jb.Y + int64_t(a1) * b.PR * nc + q - qlo;
  for (int e3 = 0; e3 <= md; ++e3) {
    if (e3) __syncthreads();
    for (int s2 = threadIdx.x / QS; s2 < M2; s2 += 256 / QS) {
      double v[N];
      line_load<N>(v, M3, [&](int s) { return X[int64_t(s2 * M3 + s) * P]; });
      line_out<N>(v, taps_of(jb, 2, e3), jb.R[2], M3, [&](int s, double o) { lds[(s2 * M3 + s) * QS + c] = o; });
    }
    __syncthreads();
    for (int s3 = threadIdx.x / QS; s3 < M3; s3 += 256 / QS) {
      double w[N];
      line_load<N>(w, M2, [&](int s) { return lds[(s * M3 + s3) * QS + c]; });
      for (int e2 = 0; e2 <= md - e3; ++e2) {
        double *Ye = Y + (y0 + e2) * YS;
        if (q < qlo + nc)
          line_out<N>(w, taps_of(jb, 1, e2), jb.R[1], M2, [&](int s, double o) { Ye[int64_t(s * M3 + s3) * nc] = o; });
      }
    }
    y0 += md - e3 + 1;
  }
}

// ------------------------------------------------------------------ stage W
// Array y of Y: degree left for s_1, and the final moments it gives.
struct YInfo {
  signed char nj[27];
  signed char mom[27][3];
};

// Workgroup (position r of the s-coordinates other than s_1, QB t columns of
// qlo .. qlo + nc - 1): thread (y, column) passes the s_1 line of array y, its
// outputs land in LDS as final moments, then one lane per node solves. (Several
// positions per workgroup with the next one's lines requested ahead need
// registers that cost a resident workgroup: slower.)
template <typename T, int d, int N, int QB, int NTH>
__global__ __launch_bounds__(NTH) void k_stage_w(SBatch b, YInfo yi, int qlo, int nc) {
  constexpr int D = 2 * d, NM = 2 + 2 * D + D * (D + 1) / 2, NY = d == 2 ? 14 : 27;
  static_assert(NY * QB <= NTH, "one line per thread");
  extern __shared__ double F[];  // [NM][M1 * QB + pad]
  const SJob &jb = b.j[blockIdx.z];
  const int M1 = b.M[0], P = b.P, PR = b.PR, qhi = qlo + nc;
  const int FS = M1 * QB + QB;
  const int r = blockIdx.y, q0 = qlo + int(blockIdx.x) * QB;
  // cross-validation: outputs s_1 <= the last t_1 of the columns, from rows below n_in
  const int n_out = b.cv ? min(M1, min(q0 + QB - 1, qhi - 1) / PR + 1) : M1;
  const int n_in = min(M1, n_out + jb.R[0]);
  {
    const int y = threadIdx.x / QB, c = threadIdx.x % QB;
    if (y < NY) {
      const double *Y = jb.Y + y * (int64_t(P) * nc) + int64_t(r) * nc + min(q0 + c, qhi - 1) - qlo;
      double v[N];
      line_load<N>(v, n_in, [&](int s) { return Y[int64_t(s) * PR * nc]; });
      for (int e = 0; e < 3; ++e) {
        if (e >= yi.nj[y]) break;
        double *f = F + yi.mom[y][e] * FS + c;
        line_out<N>(v, taps_of(jb, 0, e), jb.R[0], n_out, [&](int s, double o) { f[s * QB] = o; });
      }
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < n_out * QB; e += NTH) {
    const int a1 = e / QB, c = e % QB;
    if (q0 + c >= qhi) continue;
    double m[NM];
#pragma unroll
    for (int i = 0; i < NM; ++i) m[i] = F[i * FS + e];
    int8_t st;
    const int64_t o = (int64_t(a1) * PR + r) * P + q0 + c;
    static_cast<T *>(jb.b0)[o] = T(wls_b0<D>(m, &st));
    if (!b.cv && b.status) b.status[o] = st;
  }
}

// ------------------------------------------------------------------ score
// sum Q_f - 2 G_f g + C_f g^2 over all nodes, g(p, q) = b0(min, max) (the fit at
// (q, p) is the fit at (p, q) up to rounding), 0 outside the mask and where b0 is
// NaN (an empty window). Tile pairs (I, J), I <= J; one FP64 partial per workgroup.
template <typename T>
__global__ __launch_bounds__(256) void k_staged_score(SBatch b, int npairs) {
  __shared__ double A[SC_TILE][SC_TILE + 1];
  __shared__ double red[4];
  const SJob &jb = b.j[blockIdx.z];
  const int P = b.P, nt = (P + SC_TILE - 1) / SC_TILE;
  const T *Gh = static_cast<const T *>(jb.b0), *Q = static_cast<const T *>(jb.Qf);
  const T *G = static_cast<const T *>(jb.Gf), *C = static_cast<const T *>(jb.Cf);
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  double s = 0.0;
  for (int t = blockIdx.x; t < npairs; t += gridDim.x) {
    int id = t, I = 0;
    while (id >= nt - I) {
      id -= nt - I;
      ++I;
    }
    const int r0 = I * SC_TILE, c0 = (I + id) * SC_TILE;
    double qv[8], gv[8], cv[8];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int rr = ty + 8 * u;
      const bool ia = r0 + rr < P && c0 + tx < P, ib = id > 0 && c0 + rr < P && r0 + tx < P;
      const int64_t o1 = ia ? int64_t(r0 + rr) * P + c0 + tx : 0, o2 = ib ? int64_t(c0 + rr) * P + r0 + tx : 0;
      A[rr][tx] = ia ? double(Gh[o1]) : 0.0;
      qv[u] = ia ? double(Q[o1]) : 0.0;
      gv[u] = ia ? double(G[o1]) : 0.0;
      cv[u] = ia ? double(C[o1]) : 0.0;
      qv[4 + u] = ib ? double(Q[o2]) : 0.0;
      gv[4 + u] = ib ? double(G[o2]) : 0.0;
      cv[4 + u] = ib ? double(C[o2]) : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int rr = ty + 8 * u;
      double g = id > 0 || rr <= tx ? A[rr][tx] : A[tx][rr];
      if (b.mask && r0 + rr < P && c0 + tx < P && (!b.mask[r0 + rr] || !b.mask[c0 + tx])) g = 0.0;
      if (g != g) g = 0.0;
      s += qv[u] - 2.0 * gv[u] * g + cv[u] * g * g;
      // (c0 + rr, r0 + tx): the node (r0 + tx, c0 + rr) of this tile. Not on a
      // diagonal tile, where half of those nodes are never written: weights of
      // zero do not make up for an infinity in them
      if (id == 0) continue;
      double g2 = A[tx][rr];
      if (b.mask && c0 + rr < P && r0 + tx < P && (!b.mask[c0 + rr] || !b.mask[r0 + tx])) g2 = 0.0;
      if (g2 != g2) g2 = 0.0;
      s += qv[4 + u] - 2.0 * gv[4 + u] * g2 + cv[4 + u] * g2 * g2;
    }
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) jb.part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ __launch_bounds__(64) void k_staged_finish(const double *__restrict__ part, int n,
                                                      double *__restrict__ scores) {
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 64) s += part[int64_t(blockIdx.x) * n + i];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (threadIdx.x == 0) scores[blockIdx.x] = s;
}

// ------------------------------------------------------------------ host
// Moment index in the order S0, S1[D], S2 (upper triangle by rows), T0, T1[D] of
// the exponents e over (s_1 .. s_d, t_1 .. t_d).
int moment_of(int D, int fam, const int *e) {
  int c[2] = {-1, -1}, deg = 0;
  for (int k = 0; k < D; ++k)
    for (int r = 0; r < e[k]; ++r) c[deg++] = k;
  const int NC = 1 + D + D * (D + 1) / 2;
  if (fam == 1) return deg == 0 ? NC : NC + 1 + c[0];
  if (deg == 0) return 0;
  if (deg == 1) return 1 + c[0];
  int idx = 1 + D;
  for (int r = 0; r < c[0]; ++r) idx += D - r;
  return idx + c[1] - c[0];
}

YInfo make_yinfo(int d) {
  YInfo yi;
  std::memset(&yi, 0, sizeof(yi));
  int y = 0;
  for (int f = 0; f < 2; ++f) {
    const int md = 2 - f;
    for (int t3 = 0; t3 <= (d == 3 ? md : 0); ++t3)
      for (int t2 = 0; t2 <= md - t3; ++t2)
        for (int t1 = 0; t1 <= md - t3 - t2; ++t1) {
          const int left = md - t1 - t2 - t3;
          for (int s3 = 0; s3 <= (d == 3 ? left : 0); ++s3)
            for (int s2 = 0; s2 <= left - s3; ++s2) {
              yi.nj[y] = (signed char)(left - s3 - s2 + 1);
              for (int s1 = 0; s1 <= left - s3 - s2; ++s1) {
                const int e2[4] = {s1, s2, t1, t2}, e3[6] = {s1, s2, s3, t1, t2, t3};
                yi.mom[y][s1] = (signed char)moment_of(2 * d, f, d == 2 ? e2 : e3);
              }
              ++y;
            }
        }
  }
  return yi;
}

struct Shape {
  int d, M[3], P, PR, N, nx, ny;
  int nc;  // t-columns of Y at a time
};
Shape shape_of(const fpca_grid *g) {
  Shape s{};
  s.d = g->d;
  s.P = 1;
  int mx = 1;
  for (int k = 0; k < 3; ++k) {
    s.M[k] = k < g->d ? g->M[k] : 1;
    s.P *= s.M[k];
    mx = std::max(mx, s.M[k]);
  }
  s.PR = s.P / s.M[0];
  s.N = mx <= 16 ? 16 : (mx + 7) / 8 * 8;
  s.nx = g->d == 2 ? 0 : 14;
  s.ny = g->d == 2 ? 14 : 27;
  s.nc = s.P;
  if (g->d == 3) s.nc = int(std::min<int64_t>(s.P, std::max<int64_t>(QS, (int64_t(YCHUNK) << 20) / (8 * s.ny * s.P) / QS * QS)));
  return s;
}

size_t job_bytes(const Shape &s, size_t elem, bool cv) {
  const size_t PP = size_t(s.P) * s.P;
  return carve_bytes(size_t(s.nx) * PP, 8) + carve_bytes(size_t(s.ny) * s.P * s.nc, 8) + (cv ? carve_bytes(PP, elem) : 0) +
         carve_bytes(9 * TAPW, 8);
}

// The attribute belongs to the process: always the same value, so that threads with
// grids of different sizes do not lower it for each other.
template <typename K>
int want_lds(K kernel, size_t lds) {
  if (lds > 64 * 1024)
    FPCA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 160 * 1024));
  return FPCA_OK;
}

// The three stages of the batch's nb jobs.
template <typename T, int N>
int launch_stages(fpca_context *ctx, const Shape &s, const SBatch &b, int nb) {
  hipStream_t st = ctx->stream;
  hipLaunchKernelGGL(k_staged_taps, dim3(1, unsigned(s.d), unsigned(nb)), dim3(256), 0, st, b, s.d);
  FPCA_LAUNCH_CHECK("staged taps");
  const YInfo yi = make_yinfo(s.d);
  if (s.d == 2) {
    const size_t lds = size_t(6) * s.M[1] * (s.M[1] | 1) * 8;
    if (int rc = want_lds(&k_stage_ts2<T, N>, lds)) return rc;
    hipLaunchKernelGGL((k_stage_ts2<T, N>), dim3(unsigned(s.M[0]), unsigned(s.M[0]), unsigned(2 * nb)), dim3(256),
                       lds, st, b);
    FPCA_LAUNCH_CHECK("staged TS");
    constexpr int QB = 8;
    const size_t ldw = size_t(20) * (s.M[0] + 1) * QB * 8;
    if (int rc = want_lds(&k_stage_w<T, 2, N, QB, 128>, ldw)) return rc;
    hipLaunchKernelGGL((k_stage_w<T, 2, N, QB, 128>), dim3(unsigned((s.P + QB - 1) / QB), unsigned(s.PR), unsigned(nb)),
                       dim3(128), ldw, st, b, yi, 0, s.P);
    FPCA_LAUNCH_CHECK("staged W");
    return FPCA_OK;
  }
  const size_t lds = size_t(2) * s.M[0] * s.M[1] * (s.M[2] | 1) * 8;
  if (int rc = want_lds(&k_stage_t3<T, N>, lds)) return rc;
  hipLaunchKernelGGL((k_stage_t3<T, N>), dim3(unsigned(s.P), 1, unsigned(nb)), dim3(256), lds, st, b);
  FPCA_LAUNCH_CHECK("staged T");
  const size_t lsd = size_t(s.M[1]) * s.M[2] * QS * 8;
  if (int rc = want_lds(&k_stage_s3<N>, lsd)) return rc;
  // Y of nc columns at a time: part of it is still in the 256 MB Infinity Cache
  // when the second kernel reads it
  for (int qlo = 0; qlo < s.P; qlo += s.nc) {
    const int nc = std::min(s.nc, s.P - qlo);
    hipLaunchKernelGGL((k_stage_s3<N>), dim3(unsigned((nc + QS - 1) / QS), unsigned(s.M[0]), unsigned(nb * s.nx)),
                       dim3(256), lsd, st, b, s.nx, qlo, nc);
    FPCA_LAUNCH_CHECK("staged S");
    // the final moments of M_1 x QB nodes sit in LDS
    constexpr int QB = N == 16 ? QBW : 8, NTH = (27 * QB + 63) / 64 * 64;
    const size_t ldw = size_t(35) * (s.M[0] + 1) * QB * 8;
    if (int rc = want_lds(&k_stage_w<T, 3, N, QB, NTH>, ldw)) return rc;
    hipLaunchKernelGGL((k_stage_w<T, 3, N, QB, NTH>), dim3(unsigned((nc + QB - 1) / QB), unsigned(s.PR), unsigned(nb)),
                       dim3(NTH), ldw, st, b, yi, qlo, nc);
    FPCA_LAUNCH_CHECK("staged W");
  }
  return FPCA_OK;
}

template <typename T>
int launch_any(fpca_context *ctx, const Shape &s, const SBatch &b, int nb) {
  if (s.N == 16) return launch_stages<T, 16>(ctx, s, b, nb);
  if (s.N == 24) return launch_stages<T, 24>(ctx, s, b, nb);
  if (s.N == 32) return launch_stages<T, 32>(ctx, s, b, nb);
  return launch_stages<T, 40>(ctx, s, b, nb);
}

void fill_job(const Shape &s, const StagedJob &in, SJob *o) {
  o->Ca = in.Ca;
  o->Cb = in.Cb;
  o->Ga = in.Ga;
  o->Gb = in.Gb;
  o->Qf = in.Qf;
  o->Gf = in.Gf;
  o->Cf = in.Cf;
  o->c0 = in.c0;
  for (int k = 0; k < 3; ++k) {
    o->h[k] = k < s.d ? in.h[k] : 1.0;
    o->R[k] = k < s.d ? int(std::min(std::floor(in.h[k] * double(s.M[k] - 1)), double(s.M[k] - 1))) : 0;
  }
}

SBatch make_batch(const Shape &s, const fpca_grid *grid, bool cv) {
  SBatch b;
  std::memset(&b, 0, sizeof(b));
  for (int k = 0; k < 3; ++k) b.M[k] = s.M[k];
  b.P = s.P;
  b.PR = s.PR;
  b.cv = cv ? 1 : 0;
  b.mask = grid->mask;
  return b;
}

}  // namespace

bool staged_supported(const fpca_grid *g) {
  if (g->d != 2 && g->d != 3) return false;
  int64_t P = 1;
  for (int k = 0; k < g->d; ++k) {
    if (g->M[k] > NMAX) return false;
    P *= g->M[k];
  }
  // d = 3: stage S keeps M_2 M_3 x 16 values in LDS (stage T two t-blocks, at most 96 KB)
  return P <= 4096 && (g->d == 2 || int64_t(g->M[1]) * g->M[2] * QS * 8 <= 160 * 1024);
}

template <typename T>
int staged_smooth(fpca_context *ctx, const fpca_grid *grid, const StagedJob &job, T *out, int8_t *status) {
  const Shape s = shape_of(grid);
  const size_t PP = size_t(s.P) * s.P;
  if (int rc = ws_reserve(ctx, job_bytes(s, sizeof(T), false))) return rc;
  Carver cw{static_cast<char *>(ctx->ws), 0, ctx->ws_size};
  SBatch b = make_batch(s, grid, false);
  b.status = status;
  fill_job(s, job, &b.j[0]);
  b.j[0].X = cw.take<double>(size_t(s.nx) * PP);
  b.j[0].Y = cw.take<double>(size_t(s.ny) * s.P * s.nc);
  b.j[0].taps = cw.take<double>(9 * TAPW);
  b.j[0].b0 = out;
  return launch_any<T>(ctx, s, b, 1);
}

template <typename T>
int staged_scores(fpca_context *ctx, const fpca_grid *grid, const std::vector<StagedJob> &jobs, double *scores) {
  const Shape s = shape_of(grid);
  const size_t PP = size_t(s.P) * s.P, per = job_bytes(s, sizeof(T), true), J = jobs.size();
  // score workgroups per job, by the grid: many jobs on a small one need little
  const int nt = (s.P + SC_TILE - 1) / SC_TILE, npairs = nt * (nt + 1) / 2, nsc = std::min(npairs, SC_WG);
  const size_t bytes_part = carve_bytes(J * nsc, 8);
  // 1 GB of moments at most: 32^2 nodes eight jobs, 40^2 three (40 jobs 10.5 ms; 10.1 with
  // eight), 16^3 one (20 jobs 43.5 ms; 42.1 with four)
  int nb_max = int(std::max<size_t>(1, std::min<size_t>({size_t(SB_MAX), J, (size_t(1) << 30) / per})));
  while (nb_max > 1 && !ws_room(ctx, bytes_part + nb_max * per)) --nb_max;  // a scratch limit: fewer jobs at a time
  if (int rc = ws_reserve(ctx, bytes_part + nb_max * per)) return rc;
  Carver cw{static_cast<char *>(ctx->ws), 0, ctx->ws_size};
  double *part = cw.take<double>(J * nsc);
  SBatch b = make_batch(s, grid, true);
  for (int i = 0; i < nb_max; ++i) {
    b.j[i].X = cw.take<double>(size_t(s.nx) * PP);
    b.j[i].Y = cw.take<double>(size_t(s.ny) * s.P * s.nc);
    b.j[i].b0 = cw.take<T>(PP);
    b.j[i].taps = cw.take<double>(9 * TAPW);
  }
  for (size_t j0 = 0; j0 < J; j0 += nb_max) {
    const int nb = int(std::min<size_t>(nb_max, J - j0));
    for (int i = 0; i < nb; ++i) {
      fill_job(s, jobs[j0 + i], &b.j[i]);
      b.j[i].part = part + (j0 + i) * nsc;
    }
    if (int rc = launch_any<T>(ctx, s, b, nb)) return rc;
    hipLaunchKernelGGL(k_staged_score<T>, dim3(unsigned(nsc), 1, unsigned(nb)), dim3(256), 0, ctx->stream, b, npairs);
    FPCA_LAUNCH_CHECK("staged score");
  }
  hipLaunchKernelGGL(k_staged_finish, dim3(unsigned(J)), dim3(64), 0, ctx->stream, part, nsc, scores);
  FPCA_LAUNCH_CHECK("staged finish");
  return FPCA_OK;
}

template int staged_smooth<float>(fpca_context *, const fpca_grid *, const StagedJob &, float *, int8_t *);
template int staged_smooth<double>(fpca_context *, const fpca_grid *, const StagedJob &, double *, int8_t *);
template int staged_scores<float>(fpca_context *, const fpca_grid *, const std::vector<StagedJob> &, double *);
template int staged_scores<double>(fpca_context *, const fpca_grid *, const std::vector<StagedJob> &, double *);

}  // namespace fpca
