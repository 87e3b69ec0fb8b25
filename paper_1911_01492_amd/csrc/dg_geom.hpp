// dg_geom.hpp -- trilinear element maps on the device.
//
// Element e = ex + nx (ey + ny ez) has the 8 corner vertices
// (ex + c0, ey + c1, ez + c2), corner index c = c0 + 2 c1 + 4 c2, of the
// (nx+1)(ny+1)(nz+1) vertex grid (x-index fastest); without a vertex array
// the grid is uniform, vertex (i, j, l) at (i/nx, j/ny, l/nz).
#pragma once

#include "dg_internal.hpp"

namespace dg {

// 1 / x and sqrt(x) from the hardware approximation, to within an ulp and without
// the scaling steps of the full-range functions: 1 / x by Newton's method, sqrt(x)
// by Goldschmidt's iteration (residuals by fused multiply-add).
// recip: x and 1 / x normal.  root: x zero or normal; in FP64 subnormal too (rsqf
// flushes them, rsq does not).
__device__ __forceinline__ float recip(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.0f), r);
}
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}
// 1 / det J of a trilinear element: in FP32 through 2^24 det, which is normal
// wherever 1 / det is finite, and finite wherever the squares of the areas are
// (det^2 is about the product of the areas, so det < 2^96)
__device__ __forceinline__ float recip_det(float x) { return 0x1p24f * recip(0x1p24f * x); }
__device__ __forceinline__ double recip_det(double x) { return recip(x); }
__device__ __forceinline__ float root(float x) {
  const float y = __builtin_amdgcn_rsqf(fmaxf(x, 0x1p-126f)), g = x * y;
  return fmaf(fmaf(-g, g, x), 0.5f * y, g);
}
__device__ __forceinline__ double root(double x) {
  const double y = __builtin_amdgcn_rsq(fmax(x, 0x1p-1022));
  double g = x * y, h = 0.5 * y;
  const double r = fma(-g, h, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  return fma(fma(-g, g, x), h, g);
}

// J[a][d] = d x_a / d xi_d, written with the edge vectors of the corner cube:
// dF/dxi_0 = (1-xi_1)(1-xi_2)(X1-X0) + xi_1(1-xi_2)(X3-X2) + (1-xi_1)xi_2(X5-X4) + xi_1 xi_2 (X7-X6)
// and cyclically for the other two directions.
template <typename T>
__device__ __forceinline__ void trilinear_jacobian(const T (&X)[8][3], const T (&xi)[3], T (&J)[3][3]) {
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int b = 1 << d;
    const int o1 = (d == 0) ? 1 : 0, o2 = (d == 2) ? 1 : 2;  // the other two axes
    const T s1 = xi[o1], s2 = xi[o2];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      T acc = T(0);
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        if (c & b) continue;  // edge from corner c to c + b
        const T w = (((c >> o1) & 1) ? s1 : T(1) - s1) * (((c >> o2) & 1) ? s2 : T(1) - s2);
        acc += w * (X[c + b][a] - X[c][a]);
      }
      J[a][d] = acc;
    }
  }
}

// J at the points of one line along xi_2 (xi_0, xi_1 fixed).  In the sum of
// trilinear_jacobian the column along xi_2 depends on xi_0, xi_1 only and the
// other two columns are affine in xi_2, so after this set-up (the edge
// vectors of the corner cube combined once per line) each point costs six
// multiply-adds: J[.][0] = p0 + xi_2 d0, J[.][1] = p1 + xi_2 d1, J[.][2] = c2.
template <typename T>
struct JacZLine {
  T p0[3], d0[3], p1[3], d1[3], c2[3];
  __device__ __forceinline__ JacZLine(const T (&X)[8][3], T x0, T x1) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      // edges along xi_0 from corners 0, 2, 4, 6 (weights in xi_1, xi_2)
      const T lo0 = (T(1) - x1) * (X[1][a] - X[0][a]) + x1 * (X[3][a] - X[2][a]);
      const T hi0 = (T(1) - x1) * (X[5][a] - X[4][a]) + x1 * (X[7][a] - X[6][a]);
      p0[a] = lo0;
      d0[a] = hi0 - lo0;
      // edges along xi_1 from corners 0, 1, 4, 5 (weights in xi_0, xi_2)
      const T lo1 = (T(1) - x0) * (X[2][a] - X[0][a]) + x0 * (X[3][a] - X[1][a]);
      const T hi1 = (T(1) - x0) * (X[6][a] - X[4][a]) + x0 * (X[7][a] - X[5][a]);
      p1[a] = lo1;
      d1[a] = hi1 - lo1;
      // edges along xi_2 from corners 0..3 (weights in xi_0, xi_1)
      c2[a] = (T(1) - x1) * ((T(1) - x0) * (X[4][a] - X[0][a]) + x0 * (X[5][a] - X[1][a])) +
              x1 * ((T(1) - x0) * (X[6][a] - X[2][a]) + x0 * (X[7][a] - X[3][a]));
    }
  }
  __device__ __forceinline__ void at(T x2, T (&J)[3][3]) const {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      J[a][0] = p0[a] + x2 * d0[a];
      J[a][1] = p1[a] + x2 * d1[a];
      J[a][2] = c2[a];
    }
  }
};

// J at the point (xi_A, xi_B) = (ta, tb) of the face xi_D = s (s = 0 or 1),
// A < B the tangential axes.  On the face the weights of trilinear_jacobian
// that carry the factor xi_D or 1 - xi_D are 0 or 1: the tangential columns
// keep the two edges of the face itself, the normal column all four edges
// along D.
template <int D, typename T>
__device__ __forceinline__ void face_jacobian(const T (&X)[8][3], int s, T ta, T tb, T (&J)[3][3]) {
  constexpr int A = D == 0 ? 1 : 0, B = D == 2 ? 1 : 2;
  constexpr int BD = 1 << D, BA = 1 << A, BB = 1 << B;
  const int c0 = s ? BD : 0;  // the face's first corner
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    J[r][D] = (T(1) - tb) * ((T(1) - ta) * (X[BD][r] - X[0][r]) + ta * (X[BA + BD][r] - X[BA][r])) +
              tb * ((T(1) - ta) * (X[BB + BD][r] - X[BB][r]) + ta * (X[BA + BB + BD][r] - X[BA + BB][r]));
    J[r][A] = (T(1) - tb) * (X[c0 + BA][r] - X[c0][r]) + tb * (X[c0 + BB + BA][r] - X[c0 + BB][r]);
    J[r][B] = (T(1) - ta) * (X[c0 + BB][r] - X[c0][r]) + ta * (X[c0 + BA + BB][r] - X[c0 + BA][r]);
  }
}

template <typename TC>
struct V3 {
  TC x, y, z;
};
template <typename TC>
__device__ __forceinline__ V3<TC> cross(const V3<TC>& a, const V3<TC>& b) {
  return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
template <typename TC>
__device__ __forceinline__ TC dot(const V3<TC>& a, const V3<TC>& b) {
  return a.x * b.x + a.y * b.y + a.z * b.z;
}
template <typename TC>
__device__ __forceinline__ V3<TC> lin(const V3<TC>& a, TC t, const V3<TC>& b) {
  return {a.x + t * b.x, a.y + t * b.y, a.z + t * b.z};
}
template <typename TC>
__device__ __forceinline__ V3<TC> operator-(const V3<TC>& a, const V3<TC>& b) {
  return {a.x - b.x, a.y - b.y, a.z - b.z};
}

// Tangential axes of a face with normal axis D: B the one of smaller stride (x, or
// y where x is the normal), A the other.
__device__ __forceinline__ int axis_b(int D) { return D == 0 ? 1 : 0; }
__device__ __forceinline__ int axis_a(int D) { return D == 2 ? 1 : 2; }

// J of one side on the line xi_A = ta of its face xi_D = s: the column along B is
// constant (jb, times odd), those along A and D are affine in xi_B.  odd: -1
// where (D, A, B) is an odd permutation, so that ja x jb is the row D of adj J,
// jb x jd the row A and odd jd x ja the row B.
template <typename TC>
struct FaceLine {
  V3<TC> jb, ap, aq, dp, dq;
  __device__ __forceinline__ FaceLine(const TC* X, int D, int s, TC ta) {
    const int A = axis_a(D), B = axis_b(D);
    auto corner = [&](int cd, int ca, int cb) {
      const TC* c = X + 3 * ((cd << D) | (ca << A) | (cb << B));
      return V3<TC>{c[0], c[1], c[2]};
    };
    const TC sg = s ? TC(-1) : TC(1), odd = D == 1 ? TC(1) : TC(-1);
    auto edge = [&](const V3<TC>& p, const V3<TC>& q) {  // along D
      return V3<TC>{sg * (q.x - p.x), sg * (q.y - p.y), sg * (q.z - p.z)};
    };
    const V3<TC> f00 = corner(s, 0, 0), f10 = corner(s, 1, 0), f01 = corner(s, 0, 1), f11 = corner(s, 1, 1);
    const V3<TC> e00 = edge(f00, corner(1 - s, 0, 0)), e10 = edge(f10, corner(1 - s, 1, 0));
    const V3<TC> e01 = edge(f01, corner(1 - s, 0, 1)), e11 = edge(f11, corner(1 - s, 1, 1));
    const V3<TC> b0 = f01 - f00, b1 = lin(b0, ta, (f11 - f10) - b0);
    jb = {odd * b1.x, odd * b1.y, odd * b1.z};
    ap = f10 - f00;
    aq = (f11 - f01) - ap;
    dp = lin(e00, ta, e10 - e00);
    dq = lin(e01, ta, e11 - e01) - dp;
  }
};

template <typename T>
__device__ __forceinline__ T det3(const T (&J)[3][3]) {
  return J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) - J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) +
         J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]);
}

// adjugate: adj(J) = det(J) J^{-1}
template <typename T>
__device__ __forceinline__ void adj3(const T (&J)[3][3], T (&A)[3][3]) {
  A[0][0] = J[1][1] * J[2][2] - J[1][2] * J[2][1];
  A[0][1] = J[0][2] * J[2][1] - J[0][1] * J[2][2];
  A[0][2] = J[0][1] * J[1][2] - J[0][2] * J[1][1];
  A[1][0] = J[1][2] * J[2][0] - J[1][0] * J[2][2];
  A[1][1] = J[0][0] * J[2][2] - J[0][2] * J[2][0];
  A[1][2] = J[0][2] * J[1][0] - J[0][0] * J[1][2];
  A[2][0] = J[1][0] * J[2][1] - J[1][1] * J[2][0];
  A[2][1] = J[0][1] * J[2][0] - J[0][0] * J[2][1];
  A[2][2] = J[0][0] * J[1][1] - J[0][1] * J[1][0];
}

}  // namespace dg
