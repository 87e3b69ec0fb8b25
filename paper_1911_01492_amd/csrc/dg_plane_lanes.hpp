// dg_plane_lanes.hpp -- which element a lane of k_apply_planes (dg_planes.hpp)
// holds, whether it stores it, and where its x- and y-neighbours come from.
// Plain integer logic, for the host too.
#pragma once

#include <hip/hip_runtime.h>

namespace dg {

__host__ __device__ constexpr int plane_by(int n) { return n == 2 ? 8 : 4; }  // elements of a wave's tile along y (4 along x)

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
