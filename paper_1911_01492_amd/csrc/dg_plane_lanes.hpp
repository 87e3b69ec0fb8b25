// dg_plane_lanes.hpp -- which meshes k_apply_planes (dg_planes.hpp) is used
// for, which element a lane of it holds, whether it stores it, and where its x-
// and y-neighbours come from.  Plain integer logic, for the host too.
#pragma once

#include <hip/hip_runtime.h>

#include "dg_lines.hpp"

namespace dg {

__host__ __device__ constexpr int plane_by(int n) { return n == 2 ? 8 : 4; }  // elements of a wave's tile along y (4 along x)

// Where that kernel is the faster one: large enough meshes, by type (the
// crossings lie between these sizes, line kernel vs this, us): n = 2, 40^3 8.1
// vs 7.9-8.2, 50^3 9.1-12.4 vs 7.9-10.2; n = 3, FP32 / BF16 33^3 9.3 vs 9.2-9.6,
// 42^3 13-14 vs 12.4, FP64 53^3 33.3 vs 33.9, 97^3 211 vs 178; n = 4, FP32 31^3
// 10.2 vs 10.8, 40^3 17.3 vs 16.2-17.8, 57^3 46 vs 42, BF16 31^3 9.5 vs 9.2,
// 40^3 15.7 vs 13.6.
// On meshes flat along y its tiles (8 elements along y at n = 2, 4 above) overhang
// more than the line kernel's bricks (4, 3, 2). With q the elements of its tiles per
// element of the bricks (up to 2), the crossing moves up by a power of q from where
// q costs more than the kernel gains; this / line kernel in time on both sides: n =
// 2 FP64 q = 1.33 106 x 9 x 106 0.88, q = 2 159 x 4 x 159 1.05, 236 x 4 x 236 0.98;
// n = 3 FP32 q = 1.33 119 x 5 x 119 1.02, 225 x 5 x 225 0.88, BF16 159 x 6 x 159
// 1.09, 259 x 6 x 259 0.89, FP64 q = 1.11 154 x 17 x 154 1.05, q = 1.14 184 x 21 x
// 184 1.01-1.04, q = 1.33 343 x 6 x 343 1.19; n = 4 FP32 q = 1.2 106 x 9 x 106 1.11,
// 184 x 9 x 184 0.99, q = 1.33 225 x 6 x 225 1.04, 317 x 6 x 317 0.93, q = 2 776 x 1
// x 776 1.36, BF16 q = 1.2 86 x 9 x 86 1.07, 142 x 10 x 142 0.95, q = 1.33 184 x 6 x
// 184 1.06, 317 x 6 x 317 0.91.
inline bool use_planes(int n, int prec, int nx, int ny, int nz) {
  struct Rule {
    double from, q0;  // elements at q <= q0, times (q / q0)^power above
    int power;
  };
  constexpr Rule rules[3][3] = {{{100000, 1.34, 2}, {100000, 1.34, 2}, {100000, 1.34, 2}},  // [n - 2][prec]
                                {{400000, 1.07, 10}, {70000, 1.14, 7}, {70000, 1.14, 7}},
                                {{1e300, 1.0, 0}, {100000, 1.05, 6}, {40000, 1.05, 8}}};
  if (n < 2 || n > 4 || prec < 0 || prec > 2) return false;
  const Rule& r = rules[n - 2][prec];
  auto up = [](int a, int b) { return (double)((a + b - 1) / b) * b; };
  const double q = up(ny, plane_by(n)) * nz / (up(ny, tile_y(n)) * up(nz, tile_z(n)));
  double E = (double)nx * ny * nz;
  if (q > r.q0)
    for (int i = 0; i < r.power; ++i) E *= r.q0 / q;
  return E >= r.from;
}

// A wave's tile is 4 elements along x and plane_by(n) along y, in 4 x 4 blocks
// of lanes: lane = lx + 4 ly + 16 row, the rows being the element's planes
// (n = 2: two rows per block, the second block above the first in y).  The last
// tile along an axis is moved back inside the mesh, and so is the second block
// (n = 2) of a mesh narrower than the tile; an element that two tiles or
// blocks then hold is stored by the first of them.  So the mesh's last element
// is the first of a block (lx or ly = 0) only where it is the only one.
struct PlaneLane {
  int cx, cy;         // the element (x, y); the lanes past a mesh narrower than a block hold its last one
  bool act;           // this lane's element is stored
  bool hasXL, hasXH, hasYL, hasYH;    // the element has that neighbour
  // The rim lanes: their low (first lane of the block) or high neighbour (last
  // lane, or the mesh's last element) is not beside them.  Each loads one plane
  // per axis, the neighbour dX (dY) elements away where okX (okY).  Both sides
  // fall on one lane only where the axis has one element and no wrap, so that
  // neither neighbour exists.
  bool rimXL, rimXH, rimYL, rimYH, okX, okY;
  int dX, dY;
};

// tx, ty: the wave's tile
template <int N>
__host__ __device__ __forceinline__ PlaneLane plane_lane(int nx, int ny, bool periodic, int tx, int ty, int lane) {
  constexpr int BY = plane_by(N);
  PlaneLane p;
  const int row = lane >> 4, lx = lane & 3, ly = (lane >> 2) & 3;
  const int x0 = tx * 4, y0 = ty * BY, up = N == 2 ? row >> 1 : 0;
  const int ux = (x0 < nx - 4 ? x0 : nx < 4 ? 0 : nx - 4) + lx;
  const int yb = ny >= 8 || ny < 4 ? 4 : ny - 4;  // of the second block, from the first one
  const int uy = (y0 < ny - BY ? y0 : ny < BY ? 0 : ny - BY) + ly + yb * up;
  p.cx = ux < nx ? ux : nx - 1;
  p.cy = uy < ny ? uy : ny - 1;
  // An axis of one element with periodic wrap: all four lanes along it hold
  // that element, and the shifts give an inner lane itself as both neighbours.
  const bool selfX = nx == 1 && periodic, selfY = ny == 1 && periodic;
  p.act = (selfX ? lx == 1 : ux >= x0 && ux < nx) && (selfY ? uy == 1 : uy >= y0 + (ny < BY ? 4 * up : 0) && uy < ny) && (N != 3 || row < 3);
  p.hasXL = p.cx > 0 || periodic;
  p.hasXH = p.cx < nx - 1 || periodic;
  p.hasYL = p.cy > 0 || periodic;
  p.hasYH = p.cy < ny - 1 || periodic;
  p.rimXL = lx == 0;
  p.rimXH = !selfX && (lx == 3 || p.cx == nx - 1);
  p.rimYL = ly == 0;
  p.rimYH = !selfY && (ly == 3 || p.cy == ny - 1);
  p.dX = p.rimXL ? (p.cx > 0 ? -1 : nx - 1) : (p.cx < nx - 1 ? 1 : 1 - nx);
  p.dY = (p.rimYL ? (p.cy > 0 ? -1 : ny - 1) : (p.cy < ny - 1 ? 1 : 1 - ny)) * nx;
  p.okX = p.rimXL ? p.hasXL : p.rimXH && p.hasXH;
  p.okY = p.rimYL ? p.hasYL : p.rimYH && p.hasYH;
  return p;
}

}  // namespace dg
