// dg_geom.hip -- element geometry helpers: trilinear element maps, volume
// quadrature points and the load vector b_i = int f phi_i (Sec. 4.1, right
// hand side l_h), for affine and trilinear meshes.
#include "dg_internal.hpp"
#include "dg_kernels.hpp"
#include "dg_geom.hpp"
#include "dg_lines.hpp"
#include "dg_faces.hpp"

namespace dg {

// coordinate a of corner q (bit 0: +x, bit 1: +y, bit 2: +z) of the element at (cx, cy, cz)
__device__ __forceinline__ double corner_coord(const MeshArgs<double>& m, int cx, int cy, int cz, int q, int a) {
  const int v[3] = {cx + (q & 1), cy + ((q >> 1) & 1), cz + ((q >> 2) & 1)};
  if (m.vert) return m.vert[3 * (v[0] + (int64_t)(m.nx + 1) * (v[1] + (int64_t)(m.ny + 1) * v[2])) + a];
  return a == 0 ? v[0] * m.hx : (a == 1 ? v[1] * m.hy : v[2] * m.hz);
}

// x = sum_c X_c prod_d (c_d ? xi_d : 1 - xi_d) at the Gauss points, one thread
// per x-row of n points: along it a coordinate is p + xi_0 d, p and d bilinear
// in (xi_1, xi_2).  The rows are collected in LDS and leave as one contiguous
// run, two values per lane (the kernel is bound by its 24 bytes per point).
// (24^3 Q5, 72 MB: one thread per point and 24-byte strides 31 us, one thread per
// coordinate 24, this 15)
template <int N>
__global__ __launch_bounds__(kBlock) void k_quad_points(MeshArgs<double> m, double* __restrict__ xq) {
  constexpr int NN = N * N, R = 3 * N, RS = R | 1, EPB = elems_per_block(N);
  typedef double pair_t __attribute__((ext_vector_type(2), aligned(8)));
  __shared__ double sX[EPB * 24], sO[EPB * NN * RS];
  const int64_t e0 = (int64_t)blockIdx.x * EPB;
  const int ne = (int)(m.E - e0 < EPB ? m.E - e0 : EPB), tid = threadIdx.x;
  for (int i = tid; i < ne * 24; i += kBlock) {
    const int64_t e = e0 + i / 24;
    const int ex = (int)(e % m.nx), ey = (int)((e / m.nx) % m.ny), ez = (int)(e / ((int64_t)m.nx * m.ny));
    sX[i] = corner_coord(m, ex, ey, ez, (i % 24) / 3, i % 3);  // 3 corner + coordinate
  }
  __syncthreads();
  const Tables<double>& T = *m.tab;
  if (tid < ne * NN) {
    const int el = tid / NN, t = tid - el * NN;
    const double x1 = T.gx[t % N], x2 = T.gx[t / N], y1 = 1.0 - x1, y2 = 1.0 - x2;
    double* o = sO + tid * RS;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double* X = sX + el * 24 + a;
      const double p = y2 * (y1 * X[0] + x1 * X[6]) + x2 * (y1 * X[12] + x1 * X[18]);
      const double r = y2 * (y1 * X[3] + x1 * X[9]) + x2 * (y1 * X[15] + x1 * X[21]);
#pragma unroll
      for (int i = 0; i < N; ++i) o[3 * i + a] = (1.0 - T.gx[i]) * p + T.gx[i] * r;
    }
  }
  __syncthreads();
  double* out = xq + e0 * (NN * R);
  const int tot = ne * NN * R;
  for (int j = 2 * tid; j < tot; j += 2 * kBlock) {
    const int r0 = j / R, r1 = (j + 1) / R;
    if (j + 1 < tot) {
      pair_t v;
      v.x = sO[j + r0 * (RS - R)];
      v.y = sO[j + 1 + r1 * (RS - R)];
      *(pair_t*)(out + j) = v;
    } else {
      out[j] = sO[j + r0 * (RS - R)];
    }
  }
}

// b_i = sum_q w_q |det J_q| f_q B_{q1 i1} B_{q2 i2} B_{q3 i3} by sum
// factorisation, n^2 threads per element: the z-line of w |det J| f is formed
// from the line's Jacobian and contracted along z in registers, then along y
// and x through one LDS tile; b leaves as z-lines, whose lanes are adjacent
// in memory.  Summing all n^3 points per DOF took 84 us at 24^3 Q5,
// this 15 us (48 MB moved).
template <int N>
__global__ __launch_bounds__(kBlock) void k_load_vector(MeshArgs<double> m, const double* __restrict__ fq,
                                                        double* __restrict__ b) {
  constexpr int NN = N * N, N3 = NN * N, EPB = elems_per_block(N), PE = Lay<N, double>::PE;
  constexpr bool ELEM = 64 % NN == 0;  // an element's threads lie in one wavefront
  __shared__ double sA[EPB * PE], sX[EPB][8][3];
  const Tables<double>& T = *m.tab;
  const int tid = threadIdx.x, el = tid / NN, t = tid % NN, t1 = t % N, t2 = t / N;
  const int64_t e = (int64_t)blockIdx.x * EPB + el;
  const bool act = (el < EPB) && (e < m.E);
  const int le = act ? el : 0;
  double* A = sA + le * PE;
  double f[N], v[N];
  if (act) {
    const int ex = (int)(e % m.nx), ey = (int)((e / m.nx) % m.ny), ez = (int)(e / ((int64_t)m.nx * m.ny));
    glb_get<N, 2, double, double>(fq, e, t1, t2, f);
    for (int q = t; q < 24; q += NN) sX[le][q / 3][q % 3] = corner_coord(m, ex, ey, ez, q / 3, q % 3);
  }
  lds_sync<ELEM>();
  if (act) {
    const JacZLine<double> jz(sX[le], T.gx[t1], T.gx[t2]);
    const double w12 = T.gw[t1] * T.gw[t2];
#pragma unroll
    for (int q = 0; q < N; ++q) {
      double J[3][3];
      jz.at(T.gx[q], J);
      f[q] *= w12 * T.gw[q] * fabs(det3(J));
    }
    contract_eo<N, double, 1>(T.eBt, f, v);
    lds_put<N, 2>(A, t1, t2, v);
  }
  lds_sync<ELEM>();
  if (act) {
    lds_get<N, 1>(A, t1, t2, f);
    contract_eo<N, double, 1>(T.eBt, f, v);
    lds_put<N, 1>(A, t1, t2, v);
  }
  lds_sync<ELEM>();
  if (act) {
    lds_get<N, 0>(A, t1, t2, f);
    contract_eo<N, double, 1>(T.eBt, f, v);
    lds_put<N, 0>(A, t1, t2, v);
  }
  lds_sync<ELEM>();
  if (act) {
    lds_get<N, 2>(A, t1, t2, v);
    double* pb = b + e * N3;
#pragma unroll
    for (int i = 0; i < N; ++i) pb[lidx<N, 2>(t1, t2, i)] = v[i];
  }
}

template <int N>
static hipError_t run_qp(const MeshArgs<double>& m, double* xq, hipStream_t s) {
  hipLaunchKernelGGL((k_quad_points<N>), dim3((unsigned)element_blocks(N, m.E)), dim3(kBlock), 0, s, m, xq);
  return hipGetLastError();
}
template <int N>
static hipError_t run_lv(const MeshArgs<double>& m, const double* fq, double* b, hipStream_t s) {
  hipLaunchKernelGGL((k_load_vector<N>), dim3((unsigned)element_blocks(N, m.E)), dim3(kBlock), 0, s, m, fq, b);
  return hipGetLastError();
}

hipError_t launch_quad_points(int n, const MeshArgs<double>& m, double* xq, hipStream_t s) {
  switch (n) {
    case 2: return run_qp<2>(m, xq, s);
    case 3: return run_qp<3>(m, xq, s);
    case 4: return run_qp<4>(m, xq, s);
    case 5: return run_qp<5>(m, xq, s);
    case 6: return run_qp<6>(m, xq, s);
    case 7: return run_qp<7>(m, xq, s);
    case 8: return run_qp<8>(m, xq, s);
  }
  return hipErrorInvalidValue;
}
hipError_t launch_load_vector(int n, const MeshArgs<double>& m, const double* fq, double* b,
                              hipStream_t s) {
  switch (n) {
    case 2: return run_lv<2>(m, fq, b, s);
    case 3: return run_lv<3>(m, fq, b, s);
    case 4: return run_lv<4>(m, fq, b, s);
    case 5: return run_lv<5>(m, fq, b, s);
    case 6: return run_lv<6>(m, fq, b, s);
    case 7: return run_lv<7>(m, fq, b, s);
    case 8: return run_lv<8>(m, fq, b, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace dg
