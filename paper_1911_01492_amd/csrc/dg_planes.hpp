// dg_planes.hpp -- sum-factorised SWIPDG apply y = A x on affine
// (axis-parallel box) elements for n = 2, 3, 4 nodes per direction, with whole
// element planes in registers.
//
// The operator is the Kronecker sum of the line kernel of dg_affine.hip,
//     y = M_z P1 + L_z P2,   P1 = M_y (L_x x) + L_y (M_x x),   P2 = M_y M_x x,
// M the 1D mass, L_d the 1D DG operator along d (volume stiffness and the two
// faces normal to d; L_y and L_z act on mass-applied lines, so their face terms
// read the neighbour's mass-applied trace and normal derivative).
//
// A lane owns one (x, y) plane of an element (n^2 values), a wave 4 x 4
// elements (x, y) of one layer: lane = ex + 4 ey + 16 i3, so the contractions
// along x and y need no exchange at all, the face scalars of x- and
// y-neighbours inside the wave come by DPP row shifts of 1 and 4 lanes, and the
// planes of the four 16-lane rows turn into z-lines by 4 x 4 transposes of
// rows and registers (v_permlane32_swap, v_permlane16_swap).  No LDS, no
// barrier.  (n = 3 leaves the fourth row idle; at n = 2 rows 2 and 3 hold a
// second 4 x 4 block of elements, next in y.)  The lanes on the rim of the
// 4 x 4 block load the plane of their neighbour outside it and reduce it
// to the same face scalars (dg_plane_lanes.hpp).  A wave walks LZ layers upwards: the z-face data
// of the layer below stays in registers, and a layer is finished when the
// next one's lower trace is known (below the first and above the last layer
// only P2 is formed).
//
// Against the line kernel this takes 30-40% fewer VALU instructions per DOF, no
// LDS traffic and a third of the cache accesses; at two to four waves per SIMD
// (110 VGPRs at n = 2 in FP64, 136 at n = 4 in FP32) it is bound by its own
// instruction stream and load latency (79^3 Q1 FP64: VALU busy 48%, address unit 63%,
// waiting 53%).  Line kernel before it -> this, us: 146^3 Q1 FP64 198 -> 148, FP32
// 119 -> 61, BF16 128 -> 50; 97^3 Q2 FP64 160 -> 148, FP32 123 -> 71, BF16 134 -> 73;
// 73^3 Q3 FP32 79 -> 63, BF16 83 -> 55.  In FP64 at n = 4 the planes take all 256 VGPRs
// and it ties with the line kernel (149 vs 152), so it is not built there.
// Part of the translation unit dg_affine.hip.
#pragma once

#include "dg_internal.hpp"
#include "dg_kernels.hpp"
#include "dg_lines.hpp"
#include "dg_plane_lanes.hpp"
#include "dg_tables.hpp"

namespace dg {

// value of the lane D lanes below (SHR) or above (!SHR) in the 16-lane row
// (zero past the row's end: the callers replace the rim lanes' values)
template <int CTRL>
__device__ __forceinline__ float row_shift(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double row_shift(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
constexpr int kRowShl = 0x100, kRowShr = 0x110;  // + distance

// rows 2, 3 of a <-> rows 0, 1 of b
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
// rows 1, 3 of a <-> rows 0, 2 of b
__device__ __forceinline__ void swap16(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
template <int N>
__device__ __forceinline__ void transpose_words(uint32_t (&w)[4]) {
  if constexpr (N > 2) {
    swap32(w[0], w[2]);
    swap32(w[1], w[3]);
  }
  swap16(w[0], w[1]);
  if constexpr (N > 2) swap16(w[2], w[3]);
}
// r[i] of row j <-> r[j] of row i, for the N registers and the element's N rows
template <int N>
__device__ __forceinline__ void transpose_rows(float (&r)[N]) {
  uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < N; ++i) w[i] = __float_as_uint(r[i]);
  transpose_words<N>(w);
#pragma unroll
  for (int i = 0; i < N; ++i) r[i] = __uint_as_float(w[i]);
}
template <int N>
__device__ __forceinline__ void transpose_rows(double (&r)[N]) {
  uint32_t lo[4] = {0, 0, 0, 0}, hi[4] = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < N; ++i) {
    lo[i] = (uint32_t)__double2loint(r[i]);
    hi[i] = (uint32_t)__double2hiint(r[i]);
  }
  transpose_words<N>(lo);
  transpose_words<N>(hi);
#pragma unroll
  for (int i = 0; i < N; ++i) r[i] = __hiloint2double((int)hi[i], (int)lo[i]);
}

// Face terms of the line operator (see line_op_s), one side each, added to b.
// upper: this element is T^-; u1, g1 its trace and raw normal derivative,
// UH, GHr the neighbour's (zero without one).
template <int N, typename TC, typename TT>
__device__ __forceinline__ void upper_face(const TT& T, TC u1, TC g1, TC UH, TC GHr, bool has, TC G, TC ih, TC sig,
                                           TC At, TC (&b)[N]) {
  const TC J = u1 - UH, GAi = At * G * ih, aP = sig * G * (has ? TC(2) : TC(1));
  b[N - 1] += At * aP * J - GAi * (g1 + GHr);
  const TC cj = GAi * J;
#pragma unroll
  for (int i = 0; i < N; ++i) b[i] -= cj * T.d1[i];
}
template <int N, typename TC, typename TT>
__device__ __forceinline__ void lower_face(const TT& T, TC u0, TC g0, TC UL, TC GLr, bool has, TC G, TC ih, TC sig,
                                           TC At, TC (&b)[N]) {
  const TC J = UL - u0, GAi = At * G * ih, aP = sig * G * (has ? TC(2) : TC(1));
  b[0] += GAi * (g0 + GLr) - At * aP * J;
  const TC cj = GAi * J;
#pragma unroll
  for (int i = 0; i < N; ++i) b[i] -= cj * T.d0[i];
}

// zeros read in place of a neighbour's plane where there is none
__device__ const uint4 kZeroPlane[8] = {};

// one plane: n^2 consecutive values
template <int N, typename TC, typename TIN>
__device__ __forceinline__ void load_plane(const TIN* __restrict__ p, TC (&u)[N][N]) {
#pragma unroll
  for (int j = 0; j < N; ++j)
#pragma unroll
    for (int i = 0; i < N; ++i) u[j][i] = load_as<TC, TIN>(p + j * N + i);
}
// ok ? p : zeros, both in global memory
template <typename TIN>
__device__ __forceinline__ const TIN* or_zeros(bool ok, const TIN* p) {
  typedef const __attribute__((address_space(1))) TIN* G;
  return (const TIN*)(ok ? (G)p : (G)(const TIN*)kZeroPlane);
}

// P2 = M_y M_x u in place
template <int N, typename TC, typename TT>
__device__ __forceinline__ void mass_plane(const TT& T, TC (&u)[N][N]) {
#pragma unroll
  for (int j = 0; j < N; ++j) {
    TC a[N];
    mass_line<N, TC, false>(T, u[j], a);
#pragma unroll
    for (int i = 0; i < N; ++i) u[j][i] = a[i];
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    TC c[N], a[N];
#pragma unroll
    for (int j = 0; j < N; ++j) c[j] = u[j][i];
    mass_line<N, TC, false>(T, c, a);
#pragma unroll
    for (int j = 0; j < N; ++j) u[j][i] = a[j];
  }
}
// plane (y, x) at z = row -> plane (z, x) at y = row
template <int N, typename TC>
__device__ __forceinline__ void turn_plane(TC (&u)[N][N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    TC c[N];
#pragma unroll
    for (int j = 0; j < N; ++j) c[j] = u[j][i];
    transpose_rows<N>(c);
#pragma unroll
    for (int j = 0; j < N; ++j) u[j][i] = c[j];
  }
}

// Origin of logical tile t of the 4 x BY x lz tiles: slabs of CY tile rows
// along y, x fastest inside a slab, then y, then z (see brick_origin).
__device__ __forceinline__ void plane_tile(int t, int ntx, int nty, int ntz, int (&o)[3]) {
  const int CY = max(1, min(nty, 96 / ntx));
  const int slab = ntx * CY * ntz;
  const int g = t / slab, r = t - g * slab;
  const int cy = min(CY, nty - g * CY);
  const int bx = r % ntx, q = r / ntx;
  o[0] = bx;
  o[1] = g * CY + q % cy;
  o[2] = q / cy;
}

// sel ? a : b
template <typename TC>
__device__ __forceinline__ TC pick(bool sel, TC a, TC b) {
  return sel ? a : b;
}

template <int N, typename TIN, typename TOUT, typename TC, bool DOT>
__global__ __launch_bounds__(kBlock, 2) void k_apply_planes(
    MeshArgs<TC> m, const TIN* __restrict__ x, TOUT* __restrict__ y, double* partials, const int* skip, int lz) {
  constexpr int NN = N * N, N3 = NN * N, BY = plane_by(N);
  static_assert(NN * sizeof(TIN) <= sizeof(kZeroPlane), "the zero plane");
  constexpr KTables<TC> T = ctab::make<N, TC>();
  __shared__ double red[kBlock / 64];
  if (skip != nullptr && *skip) return;
  x += (size_t)blockIdx.y * (size_t)m.E * N3;  // vector blockIdx.y of a multi-vector apply
  y += (size_t)blockIdx.y * (size_t)m.E * N3;
  const int ntx = (m.nx + 3) / 4, nty = (m.ny + BY - 1) / BY, ntz = (m.nz + lz - 1) / lz;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tile = (int)xcd_remap(blockIdx.x, gridDim.x) * (kBlock / 64) + wave;
  double part = 0.0;
  if (tile < ntx * nty * ntz) {
    int o[3];
    plane_tile(tile, ntx, nty, ntz, o);
    const PlaneLane p = plane_lane<N>(m.nx, m.ny, m.periodic != 0, o[0], o[1], lane);
    const int row = lane >> 4, z0 = o[2] * lz, z1 = min(z0 + lz, m.nz);
    const int r3 = N == 2 ? row & 1 : (N == 3 ? min(row, 2) : row);  // z of the lane's plane, y of its turned plane
    const bool act = p.act, hasXL = p.hasXL, hasXH = p.hasXH, hasYL = p.hasYL, hasYH = p.hasYH;
    const bool rimXL = p.rimXL, rimXH = p.rimXH, rimYL = p.rimYL, rimYH = p.rimYH, okX = p.okX, okY = p.okY;
    const int64_t sz = (int64_t)m.nx * m.ny * N3, dX = (int64_t)p.dX * N3, dY = (int64_t)p.dY * N3;
    const int64_t e0 = p.cx + (int64_t)m.nx * p.cy, ez = (int64_t)m.nx * m.ny;
    const TIN* px = x + e0 * N3 + r3 * NN;  // the lane's plane in layer 0

    TC up[N], gp[N];  // z-face scalars (trace, derivative) of the layer below at its upper face
    TC yp[N][N];      // the layer in progress: all but its upper z-face
    TC Gz = TC(0);    // its face coefficient there
    // upper z-face of layer z from the lower scalars of the layer above, and y
    auto finish = [&](int z, const TC (&u0)[N], const TC (&g0)[N], bool has) {
      const int64_t eb = (e0 + z * ez) * N3 + r3 * N;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        TC b[N];
#pragma unroll
        for (int k = 0; k < N; ++k) b[k] = yp[k][i];
        upper_face<N, TC>(T, up[i], gp[i], u0[i], g0[i], has, Gz, m.ih[2], m.sg[2], m.At[2], b);
#pragma unroll
        for (int k = 0; k < N; ++k) yp[k][i] = b[k];
      }
      if (act) {
        TOUT* py = y + eb;
        const TIN* pd = x + eb;
#pragma unroll
        for (int k = 0; k < N; ++k)
#pragma unroll
          for (int i = 0; i < N; ++i) {
            const TOUT v = (TOUT)yp[k][i];
            __builtin_nontemporal_store(v, py + k * NN + i);
            if (DOT) part += (double)load_as<TC, TIN>(pd + k * NN + i) * (double)v;
          }
      }
    };
#pragma unroll
    for (int i = 0; i < N; ++i) up[i] = gp[i] = TC(0);
    if (z0 > 0 || m.periodic) {
      TC u[N][N];
      load_plane<N, TC, TIN>(px + (z0 > 0 ? z0 - 1 : m.nz - 1) * sz, u);
      mass_plane<N, TC>(T, u);
      turn_plane<N, TC>(u);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        up[i] = u[N - 1][i];
#pragma unroll
        for (int k = 0; k < N; ++k) gp[i] += T.d1[k] * u[k][i];
      }
    }
    // The loop's first address decides 3-4% here (instruction fetch): with this no-op
    // it is 4 past a multiple of 8, 58^3 Q3 BF16 35.5 -> 34.0 us, 84^3 78.7 -> 75.9.
    if constexpr (N == 4 && sizeof(TIN) == 2 && !DOT) asm volatile("s_nop 0");
    for (int z = z0; z < z1; ++z) {
      const TIN* pz = px + z * sz;
      const int64_t e = e0 + z * ez;
      TC u[N][N], s[N][N], hu[N], hg[N], ku[N], kg[N];  // rim scalars along x; along y, mass-applied
      {
        TC xh[N][N], yh[N][N];
        load_plane<N, TC, TIN>(or_zeros(okX, pz + dX), xh);
        load_plane<N, TC, TIN>(or_zeros(okY, pz + dY), yh);
        load_plane<N, TC, TIN>(pz, u);
#pragma unroll
        for (int j = 0; j < N; ++j) {
          hu[j] = pick(rimXL, xh[j][N - 1], xh[j][0]);
          hg[j] = TC(0);
#pragma unroll
          for (int i = 0; i < N; ++i) hg[j] += pick<TC>(rimXL, T.d1[i], T.d0[i]) * xh[j][i];
        }
        TC a[N], b[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
          a[i] = pick(rimYL, yh[N - 1][i], yh[0][i]);
          b[i] = TC(0);
#pragma unroll
          for (int j = 0; j < N; ++j) b[i] += pick<TC>(rimYL, T.d1[j], T.d0[j]) * yh[j][i];
        }
        mass_line<N, TC, false>(T, a, ku);
        mass_line<N, TC, false>(T, b, kg);
      }
      const TC K = m.K[e];
      // ---- s = L_x u, u <- M_x u
      {
        const TC GL_ = m.G[6 * e], GH_ = m.G[6 * e + 1];
#pragma unroll
        for (int j = 0; j < N; ++j) {
          const TC a0 = dot_end<N, TC, 0>(T, u[j]), a1 = dot_end<N, TC, 1>(T, u[j]);
          const TC UL = pick(rimXL, hu[j], row_shift<kRowShr + 1>(u[j][N - 1]));
          const TC GL = pick(rimXL, hg[j], row_shift<kRowShr + 1>(a1));
          const TC UH = pick(rimXH, hu[j], row_shift<kRowShl + 1>(u[j][0]));
          const TC GH = pick(rimXH, hg[j], row_shift<kRowShl + 1>(a0));
          line_op_s<N, TC, false>(T, u[j], a0, a1, UL, GL, UH, GH, hasXL, hasXH, GL_, GH_, K * m.vs[0], m.ih[0],
                                  m.sg[0], m.At[0], s[j]);
          TC a[N];
          mass_line<N, TC, false>(T, u[j], a);
#pragma unroll
          for (int i = 0; i < N; ++i) u[j][i] = a[i];
        }
      }
      // ---- s <- P1 = M_y s + L_y u (+ the reaction on P2), u <- P2 = M_y u
      {
        const TC GL_ = m.G[6 * e + 2], GH_ = m.G[6 * e + 3];
        const TC cr = m.R ? m.R[e] * m.vol : TC(0);
#pragma unroll
        for (int i = 0; i < N; ++i) {
          TC c[N], b[N], p[N], q[N], a0 = TC(0), a1 = TC(0);
#pragma unroll
          for (int j = 0; j < N; ++j) {
            c[j] = u[j][i];
            q[j] = s[j][i];
            a0 += T.d0[j] * c[j];
            a1 += T.d1[j] * c[j];
          }
          const TC UL = pick(rimYL, ku[i], row_shift<kRowShr + 4>(c[N - 1]));
          const TC GL = pick(rimYL, kg[i], row_shift<kRowShr + 4>(a1));
          const TC UH = pick(rimYH, ku[i], row_shift<kRowShl + 4>(c[0]));
          const TC GH = pick(rimYH, kg[i], row_shift<kRowShl + 4>(a0));
          line_op_s<N, TC, false>(T, c, a0, a1, UL, GL, UH, GH, hasYL, hasYH, GL_, GH_, K * m.vs[1], m.ih[1], m.sg[1],
                                  m.At[1], b);
          mass_line<N, TC, false>(T, q, p);
          mass_line<N, TC, false>(T, c, q);
#pragma unroll
          for (int j = 0; j < N; ++j) {
            s[j][i] = p[j] + b[j] + cr * q[j];
            u[j][i] = q[j];
          }
        }
      }
      turn_plane<N, TC>(u);
      turn_plane<N, TC>(s);
      // ---- z: finish the layer below with the own lower face scalars, begin this one
      TC g0[N];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        g0[i] = TC(0);
#pragma unroll
        for (int k = 0; k < N; ++k) g0[i] += T.d0[k] * u[k][i];
      }
      if (z > z0) finish(z - 1, u[0], g0, true);
      const TC GL_ = m.G[6 * e + 4];
      const bool hasL = z > 0 || m.periodic;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        TC c[N], q[N], b[N], p[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
          c[k] = u[k][i];
          q[k] = s[k][i];
        }
        mass_line<N, TC, false>(T, q, p);
        sym_line<N, TC>(T.S, T.eS, c, b);
#pragma unroll
        for (int k = 0; k < N; ++k) b[k] = p[k] + K * m.vs[2] * b[k];
        lower_face<N, TC>(T, c[0], g0[i], up[i], gp[i], hasL, GL_, m.ih[2], m.sg[2], m.At[2], b);
#pragma unroll
        for (int k = 0; k < N; ++k) yp[k][i] = b[k];
        up[i] = c[N - 1];
        gp[i] = dot_end<N, TC, 1>(T, c);
      }
      Gz = m.G[6 * e + 5];
    }
    const bool above = z1 < m.nz || m.periodic;
    TC u0[N], g0[N];
#pragma unroll
    for (int i = 0; i < N; ++i) u0[i] = g0[i] = TC(0);
    if (above) {
      TC u[N][N];
      load_plane<N, TC, TIN>(px + (z1 < m.nz ? z1 : 0) * sz, u);
      mass_plane<N, TC>(T, u);
      turn_plane<N, TC>(u);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        u0[i] = u[0][i];
#pragma unroll
        for (int k = 0; k < N; ++k) g0[i] += T.d0[k] * u[k][i];
      }
    }
    finish(z1 - 1, u0, g0, above);
  }
  if (DOT) {
    const double mine[1] = {block_sum<kBlock>(part, red)};
    store_partials<1>(mine, partials, blockIdx.x);
  }
}

// ---------------------------------------------------------------- launchers
// Layers per wave.  Each wave also forms P2 of the layers below and above its
// own (about a third of a layer's work each), which favours many layers; but
// fewer than about 3000 waves leave the 1024 SIMDs short of work: 63^3 Q1 FP64
// 14.2 / 12.1 / 13.0 us at 1 / 2 / 4 layers (8064 waves at one), 42^3 Q2 FP32
// 12.4 / 12.7 / 15.6 (5082), 73^3 Q3 FP32 88.7 / 77.7 / 75.3 (26353); 8 layers
// gain nothing more (83.8).
static int plane_layers(int n, int nx, int ny, int nz) {
  const int64_t cols = (int64_t)((nx + 3) / 4) * ((ny + plane_by(n) - 1) / plane_by(n));
  int lz = 4;
  while (lz > 1 && cols * ((nz + lz - 1) / lz) < 3000) lz >>= 1;
  return lz < nz ? lz : nz;
}
// blocks (and block partials) of the kernel
static int64_t plane_blocks(int n, int nx, int ny, int nz) {
  const int lz = plane_layers(n, nx, ny, nz);
  const int64_t t = (int64_t)((nx + 3) / 4) * ((ny + plane_by(n) - 1) / plane_by(n)) * ((nz + lz - 1) / lz);
  return (t + kBlock / 64 - 1) / (kBlock / 64);
}

template <int N, typename TIN, typename TOUT, typename TC>
static hipError_t run_planes(const MeshArgs<TC>& m, int dot, const void* x, void* y, double* partials,
                             const int* skip, hipStream_t s, int nrhs) {
  const int lz = plane_layers(N, m.nx, m.ny, m.nz);
  const dim3 grid((unsigned)plane_blocks(N, m.nx, m.ny, m.nz), (unsigned)nrhs);
  if (dot)
    hipLaunchKernelGGL((k_apply_planes<N, TIN, TOUT, TC, true>), grid, dim3(kBlock), 0, s, m, (const TIN*)x, (TOUT*)y,
                       partials, skip, lz);
  else
    hipLaunchKernelGGL((k_apply_planes<N, TIN, TOUT, TC, false>), grid, dim3(kBlock), 0, s, m, (const TIN*)x, (TOUT*)y,
                       partials, skip, lz);
  return hipGetLastError();
}
template <int N>
static hipError_t run_planes_prec(int prec, int dot, const MeshArgs<double>& m64, const MeshArgs<float>& m32,
                                  const void* x, void* y, double* partials, const int* skip, hipStream_t s, int nrhs) {
  switch (prec) {
    case 0:
      if constexpr (N < 4) return run_planes<N, double, double, double>(m64, dot, x, y, partials, skip, s, nrhs);
      break;
    case 1: return run_planes<N, float, float, float>(m32, dot, x, y, partials, skip, s, nrhs);
    case 2: return run_planes<N, uint16_t, float, float>(m32, dot, x, y, partials, skip, s, nrhs);
  }
  return hipErrorInvalidValue;
}
// y = A x as launch_apply_affine, for the meshes that use_planes names: partials
// only, nrhs vectors as the second grid dimension
static hipError_t launch_apply_planes(int n, int prec, int dot, const MeshArgs<double>& m64, const MeshArgs<float>& m32,
                                      const void* x, void* y, double* partials, const int* skip, hipStream_t s,
                                      int nrhs = 1) {
  switch (n) {
    case 2: return run_planes_prec<2>(prec, dot, m64, m32, x, y, partials, skip, s, nrhs);
    case 3: return run_planes_prec<3>(prec, dot, m64, m32, x, y, partials, skip, s, nrhs);
    case 4: return run_planes_prec<4>(prec, dot, m64, m32, x, y, partials, skip, s, nrhs);
  }
  return hipErrorInvalidValue;
}

}  // namespace dg
