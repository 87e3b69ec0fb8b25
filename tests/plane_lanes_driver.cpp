// plane_lanes_driver.cpp -- test driver: the lanes of the register-plane apply
// over every small mesh, on the CPU.  Each plane of each element is stored by
// exactly one lane, and that lane's lower and upper neighbours along x and y
// (from the lane beside it in its 16-lane row, or from the plane that a rim
// lane loads) are the mesh's, or absent on a Dirichlet boundary.
#include <cstdio>
#include <vector>
#include "dg_plane_lanes.hpp"

using namespace dg;

static int fails = 0;

template <int N>
static void mesh(int nx, int ny, bool periodic) {
  constexpr int BY = plane_by(N);
  std::vector<int> stored(nx * ny * N, 0);
  auto bad = [&](const char* what, const PlaneLane& p) {
    if (++fails <= 20)
      std::printf("n=%d %dx%d %s element (%d, %d): %s\n", N, nx, ny, periodic ? "periodic" : "dirichlet", p.cx, p.cy, what);
  };
  for (int ty = 0; ty * BY < ny; ++ty)
    for (int tx = 0; tx * 4 < nx; ++tx) {
      PlaneLane L[64];
      for (int l = 0; l < 64; ++l) L[l] = plane_lane<N>(nx, ny, periodic, tx, ty, l);
      for (int l = 0; l < 64; ++l) {
        const PlaneLane& p = L[l];
        if (p.cx < 0 || p.cx >= nx || p.cy < 0 || p.cy >= ny) bad("outside the mesh", p);
        const int e = p.cx + nx * p.cy;
        if (p.okX && (e + p.dX < 0 || e + p.dX >= nx * ny)) bad("x-neighbour outside the mesh", p);
        if (p.okY && (e + p.dY < 0 || e + p.dY >= nx * ny)) bad("y-neighbour outside the mesh", p);
        // the rows that exchange planes hold the same element
        const int mate = N == 2 ? l ^ 16 : l & 15;
        if (p.cx != L[mate].cx || p.cy != L[mate].cy) bad("rows of different elements", p);
        if (!p.act) continue;
        const int row = l >> 4;
        ++stored[e * N + (N == 2 ? row & 1 : row)];
        // the neighbour each side is given: an element, -1 absent, -2 another side's data or nothing
        auto side = [&](bool rim, bool other, bool ok, int d, int lane) {
          if (rim) return !ok ? -1 : other ? -2 : e + d;
          return lane < 0 || lane > 15 ? -2 : L[(l & ~15) + lane].cx + nx * L[(l & ~15) + lane].cy;
        };
        const int r = l & 15;
        const int xl = p.cx > 0 ? e - 1 : periodic ? e + nx - 1 : -1, xh = p.cx < nx - 1 ? e + 1 : periodic ? e + 1 - nx : -1;
        const int yl = p.cy > 0 ? e - nx : periodic ? e + nx * (ny - 1) : -1,
                  yh = p.cy < ny - 1 ? e + nx : periodic ? e - nx * (ny - 1) : -1;
        if (side(p.rimXL, false, p.okX, p.dX, r - 1) != xl || p.hasXL != (xl >= 0)) bad("lower neighbour along x", p);
        if (side(p.rimXH, p.rimXL, p.okX, p.dX, r + 1) != xh || p.hasXH != (xh >= 0)) bad("upper neighbour along x", p);
        if (side(p.rimYL, false, p.okY, p.dY, r - 4) != yl || p.hasYL != (yl >= 0)) bad("lower neighbour along y", p);
        if (side(p.rimYH, p.rimYL, p.okY, p.dY, r + 4) != yh || p.hasYH != (yh >= 0)) bad("upper neighbour along y", p);
      }
    }
  for (int i = 0; i < nx * ny * N; ++i)
    if (stored[i] != 1) {
      PlaneLane p{};
      p.cx = i / N % nx;
      p.cy = i / N / nx;
      bad("not stored exactly once", p);
    }
}

// the rule at ordinary meshes and at flat ones (the line kernel's bricks overhang less along y)
static void rule(bool want, int n, int prec, int nx, int ny, int nz) {
  if (use_planes(n, prec, nx, ny, nz) != want) {
    ++fails;
    std::printf("rule: n=%d prec=%d %dx%dx%d\n", n, prec, nx, ny, nz);
  }
}

int main() {
  for (int p = 0; p < 4; ++p) rule(p < 3, 2, p, 50, 50, 50);
  for (int n = 5; n <= 8; ++n) rule(false, n, 1, 100, 100, 100);
  rule(true, 2, 0, 160, 9, 160);
  rule(true, 2, 0, 4, 200, 200);
  rule(true, 2, 0, 200, 200, 3);
  rule(false, 2, 0, 159, 4, 159);
  rule(true, 2, 0, 448, 4, 448);
  rule(true, 3, 0, 97, 97, 97);
  rule(false, 3, 0, 343, 6, 343);
  rule(true, 3, 1, 50, 50, 50);
  rule(false, 3, 2, 159, 6, 159);
  rule(true, 3, 2, 259, 6, 259);
  rule(false, 4, 0, 100, 100, 100);
  rule(true, 4, 1, 48, 48, 48);
  rule(true, 4, 2, 36, 36, 36);
  rule(false, 4, 1, 776, 1, 776);
  rule(false, 4, 2, 225, 1, 225);
  rule(false, 4, 1, 148, 6, 148);
  rule(true, 4, 1, 317, 6, 317);
  for (int nx = 1; nx <= 17; ++nx)
    for (int ny = 1; ny <= 33; ++ny)
      for (int b = 0; b < 2; ++b) {
        mesh<2>(nx, ny, b);
        mesh<3>(nx, ny, b);
        mesh<4>(nx, ny, b);
      }
  std::printf(fails ? "plane lanes: %d failures\n" : "plane lanes: ok\n", fails);
  return fails != 0;
}
