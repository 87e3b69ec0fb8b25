// dg_tables.hpp -- the 1D reference operators as compile-time constants.
//
// n Gauss-Lobatto nodes and n Gauss points on [0,1] and the matrices built on
// them, evaluated by constexpr functions: with the loops over table entries
// unrolled the entries become literals of the instructions (FP32) or scalar
// moves (FP64).  Read from memory through the scalar cache instead, every
// phase of an apply issues its own table loads and waits for them together
// with its LDS traffic, because both count on the same counter.
#pragma once

#include "dg_internal.hpp"

namespace dg {

template <typename T>
struct KTables {
  T M[kMaxN * kMaxN], S[kMaxN * kMaxN];
  T d0[kMaxN], d1[kMaxN];
  EvenOdd<T> eM, eS, eB, eBt, eDg, eDgt, eC;
};

namespace ctab {

// Legendre polynomial P_m and its first two derivatives at x (three-term recurrence)
struct Leg {
  double p, d, dd;
};
constexpr Leg legendre(int m, double x) {
  double p0 = 1.0, p1 = x, d0 = 0.0, d1 = 1.0, e0 = 0.0, e1 = 0.0;
  if (m == 0) return {p0, d0, e0};
  for (int k = 2; k <= m; ++k) {
    const double a = (2.0 * k - 1.0) / k, b = (k - 1.0) / k;
    const double p2 = a * x * p1 - b * p0, d2 = a * (p1 + x * d1) - b * d0, e2 = a * (2.0 * d1 + x * e1) - b * e0;
    p0 = p1; p1 = p2;
    d0 = d1; d1 = d2;
    e0 = e1; e1 = e2;
  }
  return {p1, d1, e1};
}

struct Nodes {
  double x[kMaxN] = {};
  double w[kMaxN] = {};
};
// Roots of P_m (DERIV = false) or P'_m (true) in (-1, 1), ascending: Newton's
// method on the deflated polynomial from the right end, polished without
// deflation, and made symmetric.
template <bool DERIV>
constexpr Nodes roots(int m) {
  Nodes r;
  const int cnt = DERIV ? m - 1 : m;
  for (int k = 0; k < cnt; ++k) {
    double x = 1.0;
    for (int it = 0; it < 60; ++it) {
      const Leg l = legendre(m, x);
      const double f = DERIV ? l.d : l.p, g = DERIV ? l.dd : l.d;
      double s = 0.0;
      for (int j = 0; j < k; ++j) s += 1.0 / (x - r.x[cnt - 1 - j]);
      x -= f / (g - f * s);
    }
    for (int it = 0; it < 3; ++it) {
      const Leg l = legendre(m, x);
      x -= DERIV ? l.d / l.dd : l.p / l.d;
    }
    r.x[cnt - 1 - k] = x;
  }
  for (int k = 0; k < cnt / 2; ++k) {
    const double a = 0.5 * (r.x[cnt - 1 - k] - r.x[k]);
    r.x[k] = -a;
    r.x[cnt - 1 - k] = a;
  }
  if (cnt & 1) r.x[cnt / 2] = 0.0;
  return r;
}
// n Gauss points and weights, n Gauss-Lobatto nodes, on [0,1]
constexpr Nodes gauss(int n) {
  Nodes r = roots<false>(n);
  for (int i = 0; i < n; ++i) {
    const Leg l = legendre(n, r.x[i]);
    r.w[i] = 1.0 / ((1.0 - r.x[i] * r.x[i]) * l.d * l.d);  // half of the weight on [-1,1]
    r.x[i] = 0.5 * (1.0 + r.x[i]);
  }
  return r;
}
constexpr Nodes lobatto(int n) {
  const Nodes in = roots<true>(n - 1);
  Nodes r;
  r.x[0] = 0.0;
  for (int i = 1; i < n - 1; ++i) r.x[i] = 0.5 * (1.0 + in.x[i - 1]);
  r.x[n - 1] = 1.0;
  return r;
}

// Lagrange basis function i on the nodes xs and its derivative at x, by products
constexpr double lagrange(int n, const double* xs, int i, double x) {
  double v = 1.0;
  for (int j = 0; j < n; ++j)
    if (j != i) v *= (x - xs[j]) / (xs[i] - xs[j]);
  return v;
}
constexpr double lagrange_d(int n, const double* xs, int i, double x) {
  double s = 0.0;
  for (int m = 0; m < n; ++m) {
    if (m == i) continue;
    double v = 1.0 / (xs[i] - xs[m]);
    for (int j = 0; j < n; ++j)
      if (j != i && j != m) v *= (x - xs[j]) / (xs[i] - xs[j]);
    s += v;
  }
  return s;
}

struct Mat {
  double a[kMaxN][kMaxN] = {};
};
// a with its centro-symmetry (SIGN +1) or -antisymmetry (-1), and where SYM its
// symmetry, exact to the last bit: equal entries are then one constant
constexpr Mat centro(int n, const Mat& m, double sign, bool sym) {
  Mat r;
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) {
      r.a[i][j] = 0.5 * (m.a[i][j] + sign * m.a[n - 1 - i][n - 1 - j]);
      if (sym) r.a[i][j] = 0.5 * (r.a[i][j] + 0.5 * (m.a[j][i] + sign * m.a[n - 1 - j][n - 1 - i]));
    }
  return r;
}
template <typename T>
constexpr void even_odd(int n, const Mat& A, EvenOdd<T>& eo) {
  const int h = n / 2;
  for (int i = 0; i < h; ++i) {
    for (int j = 0; j < h; ++j) {
      eo.E[i * kMaxH + j] = (T)(0.5 * (A.a[i][j] + A.a[i][n - 1 - j]));
      eo.O[i * kMaxH + j] = (T)(0.5 * (A.a[i][j] - A.a[i][n - 1 - j]));
    }
    if (n & 1) {
      eo.C[i] = (T)A.a[i][h];
      eo.R[i] = (T)A.a[h][i];
    }
  }
  if (n & 1) eo.mm = (T)A.a[h][h];
}
template <typename T>
constexpr void store(int n, const Mat& A, T (&out)[kMaxN * kMaxN]) {
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) out[i * kMaxN + j] = (T)A.a[i][j];
}

template <int N, typename T>
constexpr KTables<T> make() {
  KTables<T> t{};
  const Nodes g = gauss(N), l = lobatto(N);
  Mat B, Bt, D, Dg, Dgt, M, S, C;
  for (int q = 0; q < N; ++q)
    for (int i = 0; i < N; ++i) {
      B.a[q][i] = Bt.a[i][q] = lagrange(N, l.x, i, g.x[q]);
      D.a[q][i] = lagrange_d(N, l.x, i, g.x[q]);
      Dg.a[q][i] = Dgt.a[i][q] = lagrange_d(N, g.x, i, g.x[q]);
    }
  for (int i = 0; i < N; ++i)
    for (int j = 0; j < N; ++j)
      for (int q = 0; q < N; ++q) {
        M.a[i][j] += g.w[q] * B.a[q][i] * B.a[q][j];
        S.a[i][j] += g.w[q] * D.a[q][i] * D.a[q][j];
        C.a[i][j] += g.w[q] * B.a[q][i] * D.a[q][j];
      }
  M = centro(N, M, 1.0, true);
  S = centro(N, S, 1.0, true);
  B = centro(N, B, 1.0, false);
  Bt = centro(N, Bt, 1.0, false);
  Dg = centro(N, Dg, -1.0, false);
  Dgt = centro(N, Dgt, -1.0, false);
  C = centro(N, C, -1.0, false);
  store(N, M, t.M);
  store(N, S, t.S);
  for (int i = 0; i < N; ++i) {
    t.d0[i] = (T)lagrange_d(N, l.x, i, 0.0);
    t.d1[N - 1 - i] = -t.d0[i];
  }
  even_odd(N, M, t.eM);
  even_odd(N, S, t.eS);
  even_odd(N, B, t.eB);
  even_odd(N, Bt, t.eBt);
  even_odd(N, Dg, t.eDg);
  even_odd(N, Dgt, t.eDgt);
  even_odd(N, C, t.eC);
  return t;
}

}  // namespace ctab

}  // namespace dg
