// tables_driver.cpp -- test driver: the 1D operators that the kernels hold as
// constants (ctab::make) against those that dg_setup builds (build_tables), entry
// by entry, FP64 and FP32, on the CPU.
#include "dg_api.hip"
#include "dg_tables.hpp"

#include <cstdio>

using namespace dg;

static int fails = 0;
static double worst = 0.0;

template <typename T>
static double largest(const T* a, int rows, int cols, int stride) {
  double m = 0.0;
  for (int i = 0; i < rows; ++i)
    for (int j = 0; j < cols; ++j) m = std::fmax(m, std::fabs((double)a[i * stride + j]));
  return m;
}
// |a - b| against the largest entry amax of the operator, in units of its roundoff
template <typename T>
static void same(const char* what, int n, const T* a, const T* b, int rows, int cols, int stride, double tol, double amax) {
  const double u = sizeof(T) == 8 ? 0x1p-53 : 0x1p-24;
  for (int i = 0; i < rows; ++i)
    for (int j = 0; j < cols; ++j) {
      const double d = std::fabs((double)a[i * stride + j] - (double)b[i * stride + j]);
      worst = std::fmax(worst, d / (amax * u) / tol);
      if (!(d <= tol * u * amax)) {
        ++fails;
        std::printf("n=%d %s [%d][%d] (%d bytes): %.17g %.17g\n", n, what, i, j, (int)sizeof(T), (double)a[i * stride + j],
                    (double)b[i * stride + j]);
      }
    }
}
template <typename T>
static void same_eo(const char* what, int n, const EvenOdd<T>& a, const EvenOdd<T>& b, double tol) {
  const int h = n / 2;
  double amax = std::fmax(largest(a.E, h, h, kMaxH), largest(a.O, h, h, kMaxH));
  if (n & 1) amax = std::fmax(amax, std::fmax(largest(a.C, 1, h, kMaxH), std::fmax(largest(a.R, 1, h, kMaxH), std::fabs((double)a.mm))));
  same(what, n, a.E, b.E, h, h, kMaxH, tol, amax);
  same(what, n, a.O, b.O, h, h, kMaxH, tol, amax);
  if (n & 1) {
    same(what, n, a.C, b.C, 1, h, kMaxH, tol, amax);
    same(what, n, a.R, b.R, 1, h, kMaxH, tol, amax);
    same(what, n, &a.mm, &b.mm, 1, 1, 1, tol, amax);
  }
}
template <typename T>
static void compare(int n, const Tables<T>& a, const KTables<T>& b, double tol) {
  same("M", n, a.M, b.M, n, n, kMaxN, tol, largest(a.M, n, n, kMaxN));
  same("S", n, a.S, b.S, n, n, kMaxN, tol, largest(a.S, n, n, kMaxN));
  same("d0", n, a.d0, b.d0, 1, n, kMaxN, tol, largest(a.d0, 1, n, kMaxN));
  same("d1", n, a.d1, b.d1, 1, n, kMaxN, tol, largest(a.d1, 1, n, kMaxN));
  same_eo("M", n, a.eM, b.eM, tol);
  same_eo("S", n, a.eS, b.eS, tol);
  same_eo("B", n, a.eB, b.eB, tol);
  same_eo("Bt", n, a.eBt, b.eBt, tol);
  same_eo("Dg", n, a.eDg, b.eDg, tol);
  same_eo("Dgt", n, a.eDgt, b.eDgt, tol);
  same_eo("C", n, a.eC, b.eC, tol);
}
template <int N>
static void degree() {
  static Tables<double> t;
  static Tables<float> f;
  static constexpr KTables<double> kt = ctab::make<N, double>();
  static constexpr KTables<float> kf = ctab::make<N, float>();
  if (!build_tables(N, t)) {
    ++fails;
    return;
  }
  tables_to_f32(t, f);
  // FP64: sums of up to 3 n products of entries that are themselves quotients of
  // 2 n factors, by two routes: 16 n^2 units.  FP32: the FP64 values rounded once,
  // to neighbouring numbers at most.
  compare(N, t, kt, 16.0 * N * N);
  compare(N, f, kf, 2.0);
}

int main() {
  degree<2>();
  degree<3>();
  degree<4>();
  degree<5>();
  degree<6>();
  degree<7>();
  degree<8>();
  if (fails) std::printf("tables: %d failures\n", fails);
  else std::printf("tables: ok (%.3f of the tolerance at most)\n", worst);
  return fails != 0;
}
