// Device side of the stiff path: a Rosenbrock method, one trajectory per
// lane, for stiff systems (the paper's library pairs its explicit kernels
// with a Rosenbrock kernel, Sections "Adaptive explicit Runge-Kutta methods"
// and "Discussion"; it does not give the method).
//
// The method is Rodas4 (Hairer & Wanner 1996, Sec. IV.7; order 4, embedded
// order 3, stiffly accurate), in its transformed variables, which need no
// products with the Jacobian:
//   (1/(h gamma) I - J) u_i = f(y + sum_{j<i} a_ij u_j) + (1/h) sum_{j<i} c_ij u_j
//   y+ = y + sum_j m_j u_j,   error estimate e = u_s,   J = df/dy(y)
// for autonomous right-hand sides.  One LU factorisation with partial
// pivoting per attempt, six triangular solves.  Step control is the explicit
// path's (eq:errnorm, eq:controller with nu = 4); output times are landed on:
// a step that would pass the next output time is shortened to end there.
//
// A lone wavefront issues one instruction at a time, dependent or not, so the
// kernel's time is its instruction count: the matrix is factored and
// substituted over its structural entries only (LuPattern), and everything a
// lane needs lives in VGPRs, indexed by compile-time constants.  Measured
// with the full 8 x 8 factorisation before it: HIRES, 100,003 trajectories
// with 16 outputs, 4.41 -> 2.09 ms, 10^6 final states 22.4 -> 12.0 ms;
// Robertson, 100,000 with 16 outputs, 0.552 -> 0.473 ms.
// Reciprocals (of the pivots, h and h gamma, and the error scales) use the
// hardware reciprocal refined by Newton steps instead of IEEE division.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "gs_kernels.hpp"

namespace gs {

// Rodas4 in transformed variables: gamma, a_ij, c_ij (below the diagonal),
// m_j.  The error weights are (0, ..., 0, 1).
struct Rodas4 {
  static constexpr int S = 6, ORDER = 4;
  static constexpr double GAMMA = 0.25;
  __host__ __device__ static constexpr double A(int i, int j) {
    constexpr double a[6][6] = {
        {0, 0, 0, 0, 0, 0},
        {1.544, 0, 0, 0, 0, 0},
        {0.9466785280815826, 0.2557011698983284, 0, 0, 0, 0},
        {3.314825187068521, 2.896124015972201, 0.9986419139977817, 0, 0, 0},
        {1.221224509226641, 6.019134481288629, 12.53708332932087, -0.6878860361058950, 0, 0},
        {1.221224509226641, 6.019134481288629, 12.53708332932087, -0.6878860361058950, 1.0, 0}};
    return a[i][j];
  }
  __host__ __device__ static constexpr double C(int i, int j) {
    constexpr double c[6][6] = {
        {0, 0, 0, 0, 0, 0},
        {-5.6688, 0, 0, 0, 0, 0},
        {-2.430093356833875, -0.2063599157091915, 0, 0, 0, 0},
        {-0.1073529058151375, -9.594562251023355, -20.47028614809616, 0, 0, 0},
        {7.496443313967647, -10.24680431464352, -33.99990352819905, 11.70890893206160, 0, 0},
        {8.083246795921522, -7.981132988064893, -31.52159432874371, 16.31930543123136,
         -6.058818238834054, 0}};
    return c[i][j];
  }
  __host__ __device__ static constexpr double M(int j) {
    constexpr double m[6] = {1.221224509226641, 6.019134481288629, 12.53708332932087,
                             -0.6878860361058950, 1.0, 1.0};
    return m[j];
  }
};

template <>
struct OutlinePow<Rodas4> {
  static constexpr bool value = true;
};

// ---------------------------------------------------------------------------
// Stiff mass-action kinetics (this library's own networks, with the same
// structure as the classic problems below).  f and the hand-written Jacobian.
//
// Kin3: y = (a, b, c), theta = (k1, k2, k3):
//   a -> b (k1 a),  b + c -> 2c (k2 b c),  c -> a (k3 c)
struct Kin3 {
  static constexpr int D = 3, P = 3;
  // Wavefronts per SIMD the register budget allows (167 registers).
  static constexpr int WAVES_PER_EU = 3;
  // Entries of jac() that are not structurally zero, one bit per column.
  static constexpr unsigned JROW[D] = {0x05, 0x07, 0x06};
  static constexpr unsigned PIVOT_COLS = 0x0;  // columns dominant for y >= 0: no exchanges
  template <class T>
  struct ParT {
    T k1, k2, k3;
  };
  using Par = ParT<double>;
  template <class T>
  __device__ static ParT<T> prep(const T (&th)[P]) {
    return ParT<T>{th[0], th[1], th[2]};
  }
  template <class T>
  __device__ static void f(double, const T (&y)[D], const ParT<T>& p, T (&dy)[D]) {
    const T r1 = p.k1 * y[0], r2 = p.k2 * y[1] * y[2], r3 = p.k3 * y[2];
    dy[0] = r3 - r1;
    dy[1] = r1 - r2;
    dy[2] = r2 - r3;
  }
  __device__ static void jac(const double (&y)[D], const Par& p, double (&J)[D][D]) {
    const double k2b = p.k2 * y[1], k2c = p.k2 * y[2];
    J[0][0] = -p.k1;
    J[0][1] = 0.0;
    J[0][2] = p.k3;
    J[1][0] = p.k1;
    J[1][1] = -k2c;
    J[1][2] = -k2b;
    J[2][0] = 0.0;
    J[2][1] = k2c;
    J[2][2] = k2b - p.k3;
  }
};

// Kin8: y1..y8, theta = (k1..k10, s, k12):
//   y1 <-> y2 (k1, k2), y2 -> y3 (k3), y3 <-> y4 (k4, k5),
//   y4 + y5 <-> y6 (k6, k7), y6 -> y7 (k8), y7 -> y8 (k9), y8 -> y1 (k10),
//   source -> y5 (s), y5 -> sink (k12)
struct Kin8 {
  static constexpr int D = 8, P = 12;
  static constexpr int WAVES_PER_EU = 2;
  // Entries of jac() that are not structurally zero, one bit per column.
  static constexpr unsigned JROW[D] = {0x83, 0x03, 0x0e, 0x3c, 0x38, 0x38, 0x60, 0xc0};
  static constexpr unsigned PIVOT_COLS = 0x0;  // columns dominant for y >= 0: no exchanges
  template <class T>
  struct ParT {
    T k[P];
  };
  using Par = ParT<double>;
  template <class T>
  __device__ static ParT<T> prep(const T (&th)[P]) {
    ParT<T> p;
#pragma unroll
    for (int i = 0; i < P; ++i) p.k[i] = th[i];
    return p;
  }
  template <class T>
  __device__ static void f(double, const T (&y)[D], const ParT<T>& p, T (&dy)[D]) {
    const T r1 = p.k[0] * y[0], r2 = p.k[1] * y[1], r3 = p.k[2] * y[1], r4 = p.k[3] * y[2];
    const T r5 = p.k[4] * y[3], r6 = p.k[5] * y[3] * y[4], r7 = p.k[6] * y[5];
    const T r8 = p.k[7] * y[5], r9 = p.k[8] * y[6], r10 = p.k[9] * y[7];
    const T r12 = p.k[11] * y[4];
    dy[0] = r2 - r1 + r10;
    dy[1] = r1 - r2 - r3;
    dy[2] = r3 - r4 + r5;
    dy[3] = r4 - r5 - r6 + r7;
    dy[4] = r7 - r6 + p.k[10] - r12;
    dy[5] = r6 - r7 - r8;
    dy[6] = r8 - r9;
    dy[7] = r9 - r10;
  }
  __device__ static void jac(const double (&y)[D], const Par& p, double (&J)[D][D]) {
#pragma unroll
    for (int r = 0; r < D; ++r)
#pragma unroll
      for (int c = 0; c < D; ++c) J[r][c] = 0.0;
    const double k6y4 = p.k[5] * y[3], k6y5 = p.k[5] * y[4];
    J[0][0] = -p.k[0];
    J[0][1] = p.k[1];
    J[0][7] = p.k[9];
    J[1][0] = p.k[0];
    J[1][1] = -(p.k[1] + p.k[2]);
    J[2][1] = p.k[2];
    J[2][2] = -p.k[3];
    J[2][3] = p.k[4];
    J[3][2] = p.k[3];
    J[3][3] = -(p.k[4] + k6y5);
    J[3][4] = -k6y4;
    J[3][5] = p.k[6];
    J[4][3] = -k6y5;
    J[4][4] = -(k6y4 + p.k[11]);
    J[4][5] = p.k[6];
    J[5][3] = k6y5;
    J[5][4] = k6y4;
    J[5][5] = -(p.k[6] + p.k[7]);
    J[6][5] = p.k[7];
    J[6][6] = -p.k[8];
    J[7][6] = p.k[8];
    J[7][7] = -p.k[9];
  }
};

// ---------------------------------------------------------------------------
// The two classic stiff chemistry problems the paper names with its
// Rosenbrock kernel (Discussion: Robertson 1966; Schaefer 1975), in their
// standard form (Hairer & Wanner 1996, Sec. IV.1, IV.10) with the rate
// constants as per-trajectory parameters.
//
// Rober: y = (y1, y2, y3), theta = (k1, k2, k3), nominal (0.04, 3e7, 1e4):
//   y1' = -k1 y1 + k3 y2 y3,  y2' = k1 y1 - k3 y2 y3 - k2 y2^2,  y3' = k2 y2^2
struct Rober {
  static constexpr int D = 3, P = 3;
  static constexpr int WAVES_PER_EU = 3;
  // Entries of jac() that are not structurally zero, one bit per column.
  static constexpr unsigned JROW[D] = {0x07, 0x07, 0x02};
  static constexpr unsigned PIVOT_COLS = 0x0;  // columns dominant for y >= 0: no exchanges
  template <class T>
  struct ParT {
    T k1, k2, k3;
  };
  using Par = ParT<double>;
  template <class T>
  __device__ static ParT<T> prep(const T (&th)[P]) {
    return ParT<T>{th[0], th[1], th[2]};
  }
  template <class T>
  __device__ static void f(double, const T (&y)[D], const ParT<T>& p, T (&dy)[D]) {
    const T r1 = p.k1 * y[0], r2 = p.k2 * y[1] * y[1], r3 = p.k3 * y[1] * y[2];
    dy[0] = r3 - r1;
    dy[1] = r1 - r3 - r2;
    dy[2] = r2;
  }
  __device__ static void jac(const double (&y)[D], const Par& p, double (&J)[D][D]) {
    const double k3y2 = p.k3 * y[1], k3y3 = p.k3 * y[2], k2y2 = 2.0 * p.k2 * y[1];
    J[0][0] = -p.k1;
    J[0][1] = k3y3;
    J[0][2] = k3y2;
    J[1][0] = p.k1;
    J[1][1] = -k3y3 - k2y2;
    J[1][2] = -k3y2;
    J[2][0] = 0.0;
    J[2][1] = k2y2;
    J[2][2] = 0.0;
  }
};

// Hires: y1..y8, theta = (a, b, c, s, d, e, kf, g), nominal (1.71, 0.43, 8.32,
// 0.0007, 0.035, 1.12, 280, 0.69); the problem's other constants are the sums
// 8.75 = c + b, 10.03 = c + a, 1.745 = a + d, 1.81 = e + g:
//   y1' = -a y1 + b y2 + c y3 + s        y5' = -(a + d) y5 + b y6 + b y7
//   y2' =  a y1 - (c + b) y2             y6' = -kf y6 y8 + g y4 + a y5 - b y6 + g y7
//   y3' = -(c + a) y3 + b y4 + d y5      y7' =  kf y6 y8 - (e + g) y7
//   y4' =  c y2 + a y3 - e y4            y8' = -kf y6 y8 + (e + g) y7
struct Hires {
  static constexpr int D = 8, P = 8;
  // Two wavefronts, with the state between attempts partly in scratch: 10^6
  // final states 12.0 ms (one wavefront, no spills: 14.3).
  static constexpr int WAVES_PER_EU = 2;
  // Entries of jac() that are not structurally zero, one bit per column.
  static constexpr unsigned JROW[D] = {0x07, 0x03, 0x1c, 0x0e, 0x70, 0xf8, 0xe0, 0xe0};
  // Columns at which the factorisation exchanges rows itself.  Column k of
  // 1/(h gamma) I - J is diagonally dominant at 0, 1, 2 and 4 while the
  // concentrations are positive; at 3 the dominance needs e >= b + g, which
  // half of a perturbed ensemble breaks, and an exchange there unsettles 5
  // and 6.  (Exchanges at every column: 2.54 against 2.09 ms.)
  static constexpr unsigned PIVOT_COLS = 0x68;
  template <class T>
  struct ParT {
    T a, b, c, s, d, e, kf, g, cb, ca, ad, eg;
  };
  using Par = ParT<double>;
  template <class T>
  __device__ static ParT<T> prep(const T (&th)[P]) {
    ParT<T> p;
    p.a = th[0];
    p.b = th[1];
    p.c = th[2];
    p.s = th[3];
    p.d = th[4];
    p.e = th[5];
    p.kf = th[6];
    p.g = th[7];
    p.cb = p.c + p.b;
    p.ca = p.c + p.a;
    p.ad = p.a + p.d;
    p.eg = p.e + p.g;
    return p;
  }
  template <class T>
  __device__ static void f(double, const T (&y)[D], const ParT<T>& p, T (&dy)[D]) {
    const T r = p.kf * y[5] * y[7];
    dy[0] = -p.a * y[0] + p.b * y[1] + p.c * y[2] + p.s;
    dy[1] = p.a * y[0] - p.cb * y[1];
    dy[2] = -p.ca * y[2] + p.b * y[3] + p.d * y[4];
    dy[3] = p.c * y[1] + p.a * y[2] - p.e * y[3];
    dy[4] = -p.ad * y[4] + p.b * y[5] + p.b * y[6];
    dy[5] = -r + p.g * y[3] + p.a * y[4] - p.b * y[5] + p.g * y[6];
    dy[6] = r - p.eg * y[6];
    dy[7] = -r + p.eg * y[6];
  }
  __device__ static void jac(const double (&y)[D], const Par& p, double (&J)[D][D]) {
#pragma unroll
    for (int r = 0; r < D; ++r)
#pragma unroll
      for (int c = 0; c < D; ++c) J[r][c] = 0.0;
    const double ky8 = p.kf * y[7], ky6 = p.kf * y[5];
    J[0][0] = -p.a;
    J[0][1] = p.b;
    J[0][2] = p.c;
    J[1][0] = p.a;
    J[1][1] = -p.cb;
    J[2][2] = -p.ca;
    J[2][3] = p.b;
    J[2][4] = p.d;
    J[3][1] = p.c;
    J[3][2] = p.a;
    J[3][3] = -p.e;
    J[4][4] = -p.ad;
    J[4][5] = p.b;
    J[4][6] = p.b;
    J[5][3] = p.g;
    J[5][4] = p.a;
    J[5][5] = -ky8 - p.b;
    J[5][6] = p.g;
    J[5][7] = -ky6;
    J[6][5] = ky8;
    J[6][6] = -p.eg;
    J[6][7] = ky6;
    J[7][5] = -ky8;
    J[7][6] = p.eg;
    J[7][7] = -ky6;
  }
};

// ---------------------------------------------------------------------------
// Which entries of the LU factors of (1/(h gamma)) I - J can be non-zero when
// rows are exchanged at the columns of PIVOT_COLS only: J's own, the diagonal
// and the fill of the elimination; at a column of PIVOT_COLS every row that
// has an entry there may become the pivot row, so all of them take the union
// of their entries (the row-merge structure of George & Ng 1985).  HIRES
// keeps 31 of its 64 entries (15 multiply-adds to factor instead of 140, 23
// to substitute instead of 56), kin8 28.
template <class F>
struct LuPattern {
  bool nz[F::D][F::D];
  constexpr LuPattern() : nz{} {
    constexpr int D = F::D;
    for (int r = 0; r < D; ++r)
      for (int c = 0; c < D; ++c) nz[r][c] = r == c || ((F::JROW[r] >> c) & 1u) != 0;
    for (int k = 0; k < D; ++k) {
      const bool merge = ((F::PIVOT_COLS >> k) & 1u) != 0;
      for (int c = k; c < D; ++c) {
        bool any = nz[k][c];
        if (merge)
          for (int r = k; r < D; ++r) any = any || (nz[r][k] && nz[r][c]);
        for (int r = k; r < D; ++r)
          if (nz[r][k] && (merge || r > k)) nz[r][c] = nz[r][c] || any;
      }
    }
  }
};
template <class F>
__host__ __device__ constexpr bool lu_nz(int r, int c) {
  constexpr LuPattern<F> pat{};
  return pat.nz[r][c];
}
// Row exchanges at column k are carried out by lu_factor.
template <class F>
__host__ __device__ constexpr bool lu_pivots(int k) {
  return ((F::PIVOT_COLS >> k) & 1u) != 0;
}

// LU factorisation with partial pivoting (the first row of largest |entry|
// in the column), in place over the entries of LuPattern: the rows of the
// not yet eliminated part are exchanged, multipliers stay below the diagonal
// in the order they were computed, reciprocals of the pivots in inv,
// sw[r][k] says that step k exchanged rows k and r.  The operations left out
// are products with exact zeros, so the factors have the bits of the full
// factorisation.  `lost` says that a column outside PIVOT_COLS needed an
// exchange, which invalidates the factors.  False if a pivot is zero or not
// finite.
template <class F>
__device__ __forceinline__ bool lu_factor(double (&M)[F::D][F::D], bool (&sw)[F::D][F::D],
                                          double (&inv)[F::D], bool& lost) {
  constexpr int D = F::D;
  bool ok = true;
  lost = false;
  sfor<D>([&](auto K) {
    constexpr int k = decltype(K)::value;
    double best = fabs(M[k][k]);
    if constexpr (lu_pivots<F>(k)) {
      int p = k;
      sfor<D - k - 1>([&](auto R) {
        constexpr int r = k + 1 + decltype(R)::value;
        if constexpr (lu_nz<F>(r, k)) {
          const double a = fabs(M[r][k]);
          p = a > best ? r : p;
          best = a > best ? a : best;
        }
      });
      sfor<D - k - 1>([&](auto R) {
        constexpr int r = k + 1 + decltype(R)::value;
        if constexpr (lu_nz<F>(r, k)) sw[r][k] = p == r;
      });
      // The exchange runs under a per-lane branch: a wavefront in which no
      // lane pivots at this column skips it.
      if (p != k) {
        sfor<D - k - 1>([&](auto R) {
          constexpr int r = k + 1 + decltype(R)::value;
          if constexpr (lu_nz<F>(r, k)) {
            sfor<D - k>([&](auto C) {
              constexpr int c = k + decltype(C)::value;
              if constexpr (lu_nz<F>(k, c)) {
                const double a = M[k][c], b = M[r][c];
                M[k][c] = sw[r][k] ? b : a;
                M[r][c] = sw[r][k] ? a : b;
              }
            });
          }
        });
      }
    }
    ok = ok & (best > 0.0) & ((best - best) == 0.0);  // false for NaN and infinity
    inv[k] = fast_rcp(M[k][k]);
    sfor<D - k - 1>([&](auto R) {
      constexpr int r = k + 1 + decltype(R)::value;
      if constexpr (lu_nz<F>(r, k)) {
        if constexpr (!lu_pivots<F>(k)) lost = lost | (fabs(M[r][k]) > best);
        const double l = M[r][k] * inv[k];
        M[r][k] = l;
        sfor<D - k - 1>([&](auto C) {
          constexpr int c = k + 1 + decltype(C)::value;
          if constexpr (lu_nz<F>(k, c)) M[r][c] = fma(-l, M[k][c], M[r][c]);
        });
      }
    });
  });
  return ok;
}

// x <- M^{-1} x with the factors of lu_factor, its row exchanges applied as
// the substitution reaches them.  Substitution runs column by column, so the
// updates of one step are independent of each other.
template <class F>
__device__ __forceinline__ void lu_solve(const double (&M)[F::D][F::D],
                                         const bool (&sw)[F::D][F::D],
                                         const double (&inv)[F::D], double (&x)[F::D]) {
  constexpr int D = F::D;
  sfor<D - 1>([&](auto K) {
    constexpr int k = decltype(K)::value;
    if constexpr (lu_pivots<F>(k)) {
      sfor<D - k - 1>([&](auto R) {
        constexpr int r = k + 1 + decltype(R)::value;
        if constexpr (lu_nz<F>(r, k)) {
          const double a = x[k], b = x[r];
          x[k] = sw[r][k] ? b : a;
          x[r] = sw[r][k] ? a : b;
        }
      });
    }
    sfor<D - k - 1>([&](auto R) {
      constexpr int r = k + 1 + decltype(R)::value;
      if constexpr (lu_nz<F>(r, k)) x[r] = fma(-M[r][k], x[k], x[r]);
    });
  });
  rfor<D>([&](auto C) {
    constexpr int c = decltype(C)::value;
    x[c] *= inv[c];
    sfor<c>([&](auto R) {
      constexpr int r = decltype(R)::value;
      if constexpr (lu_nz<F>(r, c)) x[r] = fma(-M[r][c], x[c], x[r]);
    });
  });
}

// The stages of an attempt of length h from y with f0 = f(y): solve(x)
// replaces x by M^{-1} x; y+ in yn, the error estimate (the last stage) in
// err.
template <class F, class Solve>
__device__ __forceinline__ void rodas_stages(const Inputs<F>& in, double t, double h,
                                             const double (&y)[F::D], const double (&f0)[F::D],
                                             double (&yn)[F::D], double (&err)[F::D],
                                             Solve&& solve) {
  using TB = Rodas4;
  constexpr int D = F::D, S = TB::S;
  const double ih = fast_rcp(h);
  double u[S][D];
  sfor<S>([&](auto I) {
    constexpr int i = decltype(I)::value;
    double x[D];
    if constexpr (i == 0) {
#pragma unroll
      for (int c = 0; c < D; ++c) x[c] = f0[c];
    } else {
      double Y[D];
#pragma unroll
      for (int c = 0; c < D; ++c) {
        double acc = y[c], cu = 0.0;
        sfor<i>([&](auto J) {
          constexpr int j = decltype(J)::value;
          acc = fma(TB::A(i, j), u[j][c], acc);
          cu = fma(TB::C(i, j), u[j][c], cu);
        });
        Y[c] = acc;
        x[c] = cu;
      }
      double fy[D];
      F::f(t, Y, in.par, fy);
#pragma unroll
      for (int c = 0; c < D; ++c) x[c] = fma(ih, x[c], fy[c]);
    }
    solve(x);
#pragma unroll
    for (int c = 0; c < D; ++c) u[i][c] = x[c];
  });
#pragma unroll
  for (int c = 0; c < D; ++c) {
    double acc = y[c];
    sfor<S>([&](auto J) {
      constexpr int j = decltype(J)::value;
      acc = fma(TB::M(j), u[j][c], acc);
    });
    yn[c] = acc;
    err[c] = u[S - 1][c];
  }
}

// An attempt whose matrix needs a row exchange outside PIVOT_COLS: the full
// matrix, factored with partial pivoting over all rows.  Matrix, pivot rows
// and right-hand side are indexed at run time and live in scratch memory:
// the path is rare, and so it adds next to nothing to the register budget of
// the kernel that holds it.  False if a pivot is zero or not finite.
template <class F>
__device__ __forceinline__ bool rodas_pivoted(const Inputs<F>& in, double t, double h, double ig,
                                              const double (&y)[F::D], const double (&f0)[F::D],
                                              double (&yn)[F::D], double (&err)[F::D]) {
  constexpr int D = F::D;
  double M[D][D], inv[D], b[D];
  int piv[D];
  F::jac(y, in.par, M);
#pragma unroll
  for (int r = 0; r < D; ++r)
#pragma unroll
    for (int c = 0; c < D; ++c) M[r][c] = (r == c ? ig : 0.0) - M[r][c];
  bool ok = true;
#pragma clang loop unroll(disable)
  for (int k = 0; k < D; ++k) {
    int p = k;
    double best = fabs(M[k][k]);
#pragma clang loop unroll(disable)
    for (int r = k + 1; r < D; ++r) {
      const double a = fabs(M[r][k]);
      p = a > best ? r : p;
      best = a > best ? a : best;
    }
    piv[k] = p;
#pragma clang loop unroll(disable)
    for (int c = 0; c < D; ++c) {
      const double a = M[k][c];
      M[k][c] = M[p][c];
      M[p][c] = a;
    }
    ok = ok && best > 0.0 && (best - best) == 0.0;
    inv[k] = fast_rcp(M[k][k]);
#pragma clang loop unroll(disable)
    for (int r = k + 1; r < D; ++r) {
      const double l = M[r][k] * inv[k];
      M[r][k] = l;
#pragma clang loop unroll(disable)
      for (int c = k + 1; c < D; ++c) M[r][c] = fma(-l, M[k][c], M[r][c]);
    }
  }
  rodas_stages<F>(in, t, h, y, f0, yn, err, [&](double (&x)[D]) {
#pragma unroll
    for (int c = 0; c < D; ++c) b[c] = x[c];
#pragma clang loop unroll(disable)
    for (int k = 0; k < D; ++k) {
      const double a = b[k];
      b[k] = b[piv[k]];
      b[piv[k]] = a;
    }
#pragma clang loop unroll(disable)
    for (int c = 0; c < D - 1; ++c)
#pragma clang loop unroll(disable)
      for (int r = c + 1; r < D; ++r) b[r] = fma(-M[r][c], b[c], b[r]);
#pragma clang loop unroll(disable)
    for (int c = D - 1; c >= 0; --c) {
      b[c] *= inv[c];
#pragma clang loop unroll(disable)
      for (int r = 0; r < c; ++r) b[r] = fma(-M[r][c], b[c], b[r]);
    }
#pragma unroll
    for (int c = 0; c < D; ++c) x[c] = b[c];
  });
  return ok;
}

// One Rodas4 attempt of length h from y with f0 = f(y).  Returns the squared
// error norm (NaN if the matrix could not be factored) and y+ in yn.
template <class F>
__device__ __forceinline__ double rodas_attempt(const Inputs<F>& in, double t, double h,
                                                const double (&y)[F::D],
                                                const double (&f0)[F::D],
                                                double (&yn)[F::D]) {
  constexpr int D = F::D;
  const double ig = fast_rcp(h * Rodas4::GAMMA);
  double inv[D], err[D];
  bool ok, lost;
  {
    double M[D][D];
    F::jac(y, in.par, M);
#pragma unroll
    for (int r = 0; r < D; ++r)
#pragma unroll
      for (int c = 0; c < D; ++c) M[r][c] = r == c ? ig - M[r][c] : -M[r][c];
    bool sw[D][D];
    ok = lu_factor<F>(M, sw, inv, lost);
    if (!lost)
      rodas_stages<F>(in, t, h, y, f0, yn, err,
                      [&](double (&x)[D]) { lu_solve<F>(M, sw, inv, x); });
  }
  if (lost) ok = rodas_pivoted<F>(in, t, h, ig, y, f0, yn, err);
  double sq = 0.0;
#pragma unroll
  for (int c = 0; c < D; ++c) {
    const double sc = fma(in.rtol, max_abs(y[c], yn[c]), in.atol);
    const double r = err[c] * fast_rcp1(sc);
    sq = fma(r, r, sq);
  }
  const double en2 = sq * (1.0 / D);
  return ok ? en2 : __builtin_nan("");
}

// Persistent stiff solve, organised like the explicit forward kernel: an
// outer loop retires and refills lanes, an inner loop runs attempts of the
// live lanes until enough of them have finished for a refill (`refill` idle
// lanes, one atomic for all of them: a ballot and a prefix count in
// wave-uniform code), so retirement, the loads and the starting step of new
// trajectories are shared by many lanes instead of stalling the wave once per
// lane (leaving the inner loop at every finished lane: HIRES, 250,000 final
// states, 4.66 against 3.50 ms).  Static mode gives each lane one trajectory.
template <class F>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(F::WAVES_PER_EU)))
stiff_kernel(Params P) {
  using TB = Rodas4;
  constexpr int D = F::D;
  const int64_t n = P.n;
  const int lane = threadIdx.x & 63;
  int64_t idx = 0;
  bool live = false;
  bool queue_empty = P.sched_static != 0;  // wave-uniform
  Inputs<F> in;
  double y[D], f0[D];
  double t = 0.0, h = 0.0;
  double t_stop = 0.0;  // the next output time, or t1 after the last (in a register)
  int32_t nacc = 0, nrej = 0, nanrun = 0, kk = 0;

  auto store_node = [&](int q, const double (&v)[D]) {
#pragma unroll
    for (int c = 0; c < D; ++c) P.y_out[((int64_t)c * P.K + q) * n + idx] = v[c];
  };
  auto finish = [&](int32_t st) {
    for (int q = kk; q < P.K; ++q) {
#pragma unroll
      for (int c = 0; c < D; ++c) P.y_out[((int64_t)c * P.K + q) * n + idx] = __builtin_nan("");
    }
#pragma unroll
    for (int c = 0; c < D; ++c) P.y_final[(int64_t)c * n + idx] = y[c];
    P.n_acc[idx] = nacc;
    P.n_rej[idx] = nrej;
    P.status[idx] = st;
    live = false;
  };
  // Take trajectory i: load, validate, nodes at t0, first evaluation,
  // starting step.  Trajectories with nothing to integrate finish here.
  auto start = [&](int64_t i) {
    idx = i;
    live = true;
    nacc = nrej = nanrun = kk = 0;
    load_inputs<F>(P, i, in, y);
    t = in.t0;
    bool fin = true;
#pragma unroll
    for (int c = 0; c < D; ++c) fin = fin && (y[c] - y[c]) == 0.0;
    if (!inputs_valid<F>(P, i, in)) {
      finish(ST_BAD_INPUT);
      return;
    }
    while (kk < P.K && node_time(P, kk, i) <= in.t0) store_node(kk++, y);
    t_stop = kk < P.K ? node_time(P, kk, i) : in.t1;
    if (!fin) {
      finish(ST_NONFINITE);
      return;
    }
    if (!(in.t1 > in.t0)) {
      finish(ST_OK);
      return;
    }
    F::f(t, y, in.par, f0);
    h = P.h0 > 0.0 ? dmin(P.h0, in.t1 - in.t0) : initial_step<TB, F>(in, y, f0);
  };

  if (P.sched_static) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g < n) start(g);
  }
  for (;;) {
    if (!queue_empty) {
      const uint64_t idle = __ballot(!live);
      const int nidle = __popcll(idle);
      if (nidle >= P.refill) {
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(P.counters, (unsigned long long)nidle);
        base = first_lane(base);
        if (base + (unsigned long long)nidle >= (unsigned long long)n) queue_empty = true;
        if (!live) {
          const unsigned long long pos = base + __popcll(idle & lanemask_lt());
          if (pos < (unsigned long long)n) {
            const int64_t id = P.order ? P.order[pos] : (int64_t)pos;
            if (id >= 0 && id < n) start(id);  // a bad permutation entry is skipped
          }
        }
      }
    }
    if (__ballot(live) == 0) {
      if (queue_empty) break;
      continue;
    }
    int32_t st = -1;  // status once this lane's trajectory has finished
    // A finished lane waits in the inner loop until enough lanes are idle for
    // a refill (all of them once the queue is empty), so the retirement and
    // everything around the inner loop run once per refill, not per lane.
    const int held = __popcll(__ballot(!live));
    const int leave_at = queue_empty ? 64 : P.refill;
    for (;;) {
      if (live && st < 0) {
        if ((uint32_t)nacc + (uint32_t)nrej >= P.max_attempts) {
          st = ST_MAX_STEPS;
        } else {
          const double stop = t_stop;
          double hh = h;
          bool land = false;
          if (t + hh >= stop) {
            hh = stop - t;
            land = true;
          }
          double yn[D];
          const double en2 = rodas_attempt<F>(in, t, hh, y, f0, yn);
          const bool finite = (en2 - en2) == 0.0;
          const double factor = step_factor<TB>(P, en2, 1.0, finite);
          bool done = false;
          if (finite && en2 <= 1.0) {
            ++nacc;
            t = land ? stop : t + hh;
            bool yfin = true;
#pragma unroll
            for (int c = 0; c < D; ++c) {
              y[c] = yn[c];
              yfin = yfin && (yn[c] - yn[c]) == 0.0;
            }
            if (!yfin) {
              st = ST_NONFINITE;
            } else {
              while (kk < P.K && t_stop <= t) {
                store_node(kk++, y);
                t_stop = kk < P.K ? node_time(P, kk, idx) : in.t1;
              }
              F::f(t, y, in.par, f0);
              nanrun = 0;
              done = t >= in.t1;
            }
          } else {
            ++nrej;
            nanrun = finite ? 0 : nanrun + 1;
            if (nanrun >= 50) st = ST_NONFINITE;
          }
          h = hh * factor;
          if (done)
            st = ST_OK;
          else if (st < 0 && underflow(h, t))
            st = ST_DT_UNDERFLOW;
        }
      }
      const int done = __popcll(__ballot(live && st >= 0));
      if (done > 0 && held + done >= leave_at) break;
    }
    if (live && st >= 0) finish(st);
  }
}

// f of a stiff right-hand side at m points (SoA, point index fastest).
template <class F>
__global__ void __launch_bounds__(256) stiff_rhs_kernel(int64_t m, const double* y,
                                                        const double* theta, double* f) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  double yv[F::D], th[F::P], fv[F::D];
#pragma unroll
  for (int c = 0; c < F::D; ++c) yv[c] = y[(int64_t)c * m + i];
#pragma unroll
  for (int c = 0; c < F::P; ++c) th[c] = theta[(int64_t)c * m + i];
  F::f(0.0, yv, F::prep(th), fv);
#pragma unroll
  for (int c = 0; c < F::D; ++c) f[(int64_t)c * m + i] = fv[c];
}

}  // namespace gs
