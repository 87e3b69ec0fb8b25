// dg_trilinear.hip -- SWIPDG apply on trilinear hexahedra (curved meshes,
// "problem C" with multilinear geometries of Sec. 3.3), Jacobians computed
// on the fly at every volume and face quadrature point.
//
// Volume (sum factorisation through the Gauss points):
//   v    = (B (x) B (x) B) u                      interpolation GLL -> Gauss
//   gr_d = Dg along axis d applied to v            reference gradient
//   g    = G_q gr,  G_q = w_q K |det J| J^{-1} J^{-T} = w_q K adj(J) adj(J)^T / |det J|
//   y    = (B^T (x) B^T (x) B^T) (sum_d Dg_d^T g_d + c w_q |det J| v)
// (the last term is the optional reaction, c = 0 without it)
// Faces: k_tri_faces (dg_trifaces.hpp) runs first and leaves every element its
// six faces' rows in the workspace; they join the transposed contractions of
// the volume part along the lines of their axis, so they cost no exchange of
// their own.
//
// The discrete form is symmetric, so the transposed apply evaluates the same
// kernel.
#include "dg_internal.hpp"
#include "dg_kernels.hpp"
#include "dg_lines.hpp"
#include "dg_geom.hpp"
#include "dg_trifaces.hpp"

namespace dg {

// Synchronisation of the n^2 threads of one element: every exchange through
// LDS in these kernels stays inside one element (its tiles, face buffers and
// corner slots).  When n^2 divides 64 an element lies inside one wavefront,
// whose lanes execute together and whose LDS operations complete in order, so
// only the compiler has to be kept from moving LDS accesses across this
// point; otherwise the element may span two wavefronts and the workgroup
// barrier is used.
template <int N>
__device__ __forceinline__ void elem_sync() {
  if constexpr (64 % (N * N) == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// coordinate a of corner c (bit 0: +x, bit 1: +y, bit 2: +z) of the element
// at grid position (cx, cy, cz) (the callers know it: no index division)
template <typename TC>
__device__ __forceinline__ void corner_at(const MeshArgs<TC>& m, int cx, int cy, int cz, int c, int a, TC& out) {
  const int vx = cx + (c & 1), vy = cy + ((c >> 1) & 1), vz = cz + ((c >> 2) & 1);
  const int64_t v = vx + (int64_t)(m.nx + 1) * (vy + (int64_t)(m.ny + 1) * vz);
  out = m.vert[3 * v + a];
}

// The two faces normal to axis D, added to the thread's line t along D
template <int N, int D, typename TC>
__device__ __forceinline__ void add_faces(const MeshArgs<TC>& m, const Tables<TC>& T, int64_t e, int t, TC (&o)[N]) {
  constexpr int NN = N * N;
  const int64_t at = (e * 3 + D) * (2 * NN) + t;
  const TC ol = m.fb[at], zl = m.fb[at + NN], ou = m.fbu[at], zu = m.fbu[at + NN];
#pragma unroll
  for (int i = 0; i < N; ++i) o[i] += T.d0[i] * zl + T.d1[i] * zu;
  o[0] += ol;
  o[N - 1] += ou;
}

// Volume part of the trilinear apply for the thread's element: the element
// tile C receives (B^T (x) B^T (x) B^T)(sum_d Dg_d^T g_d + c w |det J| v) of
// the input x (see the file header), with coefficient K (and the reaction
// coefficients of m, if any); (ex, ey, ez): the element's grid position.
// Xs: the element's corner slot in LDS (filled here).  All threads of the
// block call this (it synchronises).
// FACES: the element's face terms, left in m.fb by k_tri_faces, join on the way.
template <int N, typename TC, typename TIN, bool AFF = false, bool FACES = false>
__device__ void tri_volume(const MeshArgs<TC>& m, const Tables<TC>& T, const TIN* __restrict__ x, int64_t e,
                           int ex, int ey, int ez, bool act, int t, int t1, int t2, TC K, TC (&Xs)[8][3], TC* A,
                           TC* B, TC* C) {
  constexpr int NN = N * N;
  if (act) {
    TC uz[N];
    for (int q = t; q < 24; q += NN) corner_at(m, ex, ey, ez, q / 3, q % 3, Xs[q / 3][q % 3]);
    glb_get<N, 2, TC, TIN>(x, e, t1, t2, uz);
    TC a[N];
    contract_eo<N, TC, 1>(T.eB, uz, a);  // phase Z: interpolate along z
    lds_put<N, 2>(A, t1, t2, a);
  }
  elem_sync<N>();
  const TC (&X)[8][3] = Xs;
  if (act) {  // phase Y
    TC a[N], b[N];
    lds_get<N, 1>(A, t1, t2, a);
    contract_eo<N, TC, 1>(T.eB, a, b);
    lds_put<N, 1>(B, t1, t2, b);
  }
  elem_sync<N>();
  if (act) {  // phase X: v and d/dxi_0
    TC a[N], v[N], d1[N];
    lds_get<N, 0>(B, t1, t2, a);
    contract_eo<N, TC, 1>(T.eB, a, v);
    contract_eo<N, TC, -1>(T.eDg, v, d1);
    lds_put<N, 0>(A, t1, t2, v);
    lds_put<N, 0>(C, t1, t2, d1);
  }
  elem_sync<N>();
  if (act) {  // phase Y': d/dxi_1
    TC v[N], d2[N];
    lds_get<N, 1>(A, t1, t2, v);
    contract_eo<N, TC, -1>(T.eDg, v, d2);
    lds_put<N, 1>(B, t1, t2, d2);
  }
  elem_sync<N>();
  if (act) {  // phase Z': d/dxi_2, geometry, g = G gr, Dg_z^T g_2
    TC d1[N], d2[N], d3[N], wz[N], v[N];
    lds_get<N, 2>(A, t1, t2, v);
    contract_eo<N, TC, -1>(T.eDg, v, d3);
    lds_get<N, 2>(C, t1, t2, d1);
    lds_get<N, 2>(B, t1, t2, d2);
    const TC wq12 = T.gw[t1] * T.gw[t2] * K;
    const TC cw12 = m.R ? m.R[e] * T.gw[t1] * T.gw[t2] : TC(0);  // reaction weight
    TC G0[3][3], dJ0 = TC(1);
    if (AFF) {  // parallelepiped: adj adj^T / |det J| and |det J| are the same at every point
      const TC xi[3] = {TC(0.5), TC(0.5), TC(0.5)};
      TC J[3][3], Aj[3][3];
      trilinear_jacobian(X, xi, J);
      adj3(J, Aj);
      dJ0 = fabs(det3(J));
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int cc = r; cc < 3; ++cc) {
          G0[r][cc] = (Aj[r][0] * Aj[cc][0] + Aj[r][1] * Aj[cc][1] + Aj[r][2] * Aj[cc][2]) / dJ0;
          G0[cc][r] = G0[r][cc];
        }
    }
    const JacZLine<TC> jz(X, T.gx[t1], T.gx[t2]);  // unused (and dropped) for AFF
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const TC a1 = d1[q], a2 = d2[q], a3 = d3[q];  // G gr in place of gr
      if (AFF) {
        const TC c = wq12 * T.gw[q];
        v[q] *= cw12 * T.gw[q] * dJ0;  // reaction c w |det J| u at the point
        d1[q] = c * (G0[0][0] * a1 + G0[0][1] * a2 + G0[0][2] * a3);
        d2[q] = c * (G0[1][0] * a1 + G0[1][1] * a2 + G0[1][2] * a3);
        d3[q] = c * (G0[2][0] * a1 + G0[2][1] * a2 + G0[2][2] * a3);
      } else {
        TC J[3][3], Aj[3][3];
        jz.at(T.gx[q], J);
        adj3(J, Aj);
        // det J from the adjugate's first row
        const TC dJ = fabs(J[0][0] * Aj[0][0] + J[1][0] * Aj[0][1] + J[2][0] * Aj[0][2]);
        const TC c = wq12 * T.gw[q] * recip_det(dJ);
        v[q] *= cw12 * T.gw[q] * dJ;  // reaction c w |det J| u at the point
        if constexpr (N <= 5 && sizeof(TC) == 8) {
          // G gr with G formed: more operations, but at most 128 registers (four waves per SIMD)
          TC Gm[3][3];
#pragma unroll
          for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int cc = r; cc < 3; ++cc)
              Gm[r][cc] = Gm[cc][r] = c * (Aj[r][0] * Aj[cc][0] + Aj[r][1] * Aj[cc][1] + Aj[r][2] * Aj[cc][2]);
          d1[q] = Gm[0][0] * a1 + Gm[0][1] * a2 + Gm[0][2] * a3;
          d2[q] = Gm[1][0] * a1 + Gm[1][1] * a2 + Gm[1][2] * a3;
          d3[q] = Gm[2][0] * a1 + Gm[2][1] * a2 + Gm[2][2] * a3;
        } else {  // c adj (adj^T gr)
          TC h[3];
#pragma unroll
          for (int r = 0; r < 3; ++r) h[r] = c * (Aj[0][r] * a1 + Aj[1][r] * a2 + Aj[2][r] * a3);
          d1[q] = Aj[0][0] * h[0] + Aj[0][1] * h[1] + Aj[0][2] * h[2];
          d2[q] = Aj[1][0] * h[0] + Aj[1][1] * h[1] + Aj[1][2] * h[2];
          d3[q] = Aj[2][0] * h[0] + Aj[2][1] * h[1] + Aj[2][2] * h[2];
        }
      }
    }
    contract_eo<N, TC, -1>(T.eDgt, d3, wz);
#pragma unroll
    for (int q = 0; q < N; ++q) wz[q] += v[q];
    lds_put<N, 2>(A, t1, t2, wz);
    lds_put<N, 2>(C, t1, t2, d1);
    lds_put<N, 2>(B, t1, t2, d2);
  }
  elem_sync<N>();
  if (act) {  // phase Y'': += Dg_y^T g_1
    TC g2[N], w[N], r[N];
    lds_get<N, 1>(B, t1, t2, g2);
    lds_get<N, 1>(A, t1, t2, w);
    contract_eo<N, TC, -1>(T.eDgt, g2, r);
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] += r[i];
    lds_put<N, 1>(A, t1, t2, w);
  }
  elem_sync<N>();
  if (act) {  // phase X'': += Dg_x^T g_0, then B_x^T
    TC g1[N], w[N], r[N], o[N];
    lds_get<N, 0>(C, t1, t2, g1);
    lds_get<N, 0>(A, t1, t2, w);
    contract_eo<N, TC, -1>(T.eDgt, g1, r);
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] += r[i];
    contract_eo<N, TC, 1>(T.eBt, w, o);
    if (FACES) add_faces<N, 0>(m, T, e, t, o);
    lds_put<N, 0>(A, t1, t2, o);
  }
  elem_sync<N>();
  if (act) {  // phase Y''': B_y^T
    TC w[N], o[N];
    lds_get<N, 1>(A, t1, t2, w);
    contract_eo<N, TC, 1>(T.eBt, w, o);
    if (FACES) add_faces<N, 1>(m, T, e, t, o);
    lds_put<N, 1>(A, t1, t2, o);
  }
  elem_sync<N>();
  if (act) {  // phase Z''': B_z^T -> accumulator C
    TC w[N], o[N];
    lds_get<N, 2>(A, t1, t2, w);
    contract_eo<N, TC, 1>(T.eBt, w, o);
    if (FACES) add_faces<N, 2>(m, T, e, t, o);
    lds_put<N, 2>(C, t1, t2, o);
  }
}

// Threads per block of the apply: 128 at n = 8, where the tiles of FP64 (13.8 KB
// per element) let only two blocks of 256 reside on a CU, but five of 128
__host__ __device__ constexpr int tri_block(int n) { return n == 8 ? 128 : kBlock; }

// Waves per SIMD asked of the register allocator, as many as LDS leaves room
// for: FP64 four up to n = 5 (at most 128 registers; 58^3 Q4 284 us with three,
// 247 with four) and three above; FP32 five from n = 6 on.
__host__ __device__ constexpr int tri_min_waves(int n, int bytes) {
  return bytes == 8 ? (n <= 5 ? 4 : 3) : (n >= 6 ? 5 : 1);
}

// Volume part of the apply and the face rows of k_tri_faces.  DOT: block
// partials of <x, y> for the CG.  48^3 Q7 in FP64, back to back: 495 us, 1.6 GB
// (3.2 TB/s), 63% of the cycles issue vector instructions (blocks of 256: 557 us; with
// the gradient's metric formed at every point and IEEE division 532 us).
template <int N, typename TIN, typename TOUT, typename TC, bool AFF, bool DOT>
__global__ __launch_bounds__(tri_block(N)) __attribute__((amdgpu_waves_per_eu(tri_min_waves(N, sizeof(TC))))) void k_apply_trilinear(
    MeshArgs<TC> m, const TIN* __restrict__ x, TOUT* __restrict__ y, double* partials, const int* skip) {
  constexpr int NN = N * N, N3 = NN * N, BLK = tri_block(N), EPB = BLK / NN, PE = Lay<N, TC>::PE;
  __shared__ TC sA[EPB * PE], sB[EPB * PE], sC[EPB * PE];
  __shared__ TC sX[EPB][8][3];
  __shared__ double red[BLK / 64];
  if (skip != nullptr && *skip) return;
  const Tables<TC>& T = *m.tab;
  const int64_t blk = xcd_remap(blockIdx.x, gridDim.x);
  const int tid = threadIdx.x, el = tid / NN, t = tid % NN, t1 = t % N, t2 = t / N;
  const int64_t e = blk * EPB + el;
  const bool act = (el < EPB) && (e < m.E);
  const int le = act ? el : 0;
  int ex = 0, ey = 0, ez = 0;
  TC K = TC(1);
  if (act) {
    ex = (int)(e % m.nx);
    ey = (int)((e / m.nx) % m.ny);
    ez = (int)(e / ((int64_t)m.nx * m.ny));
    K = m.K[e];
  }
  tri_volume<N, TC, TIN, AFF, true>(m, T, x, e, ex, ey, ez, act, t, t1, t2, K, sX[le], sA + le * PE, sB + le * PE,
                                    sC + le * PE);
  double part = 0.0;
  if (act) {  // the thread's own line: no exchange since it was written
    TC o[N], uz[N];
    lds_get<N, 2>(sC + le * PE, t1, t2, o);
    if (DOT) glb_get<N, 2, TC, TIN>(x, e, t1, t2, uz);
    TOUT* py = y + e * N3;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const TOUT v = (TOUT)o[i];
      __builtin_nontemporal_store(v, &py[lidx<N, 2>(t1, t2, i)]);
      if (DOT) part += (double)uz[i] * (double)v;
    }
  }
  if (DOT) {
    const double mine[1] = {block_sum<BLK>(part, red)};
    store_partials<1>(mine, partials, blockIdx.x);
  }
}

// ---------------------------------------------------------------- dA / dtheta
// Per element T, with u and v: parts[7 T] = u_T . (volume form of T with
// K = 1) v_T here, and from k_tri_faces the whole form of a face with unit
// coefficient, u . (rows of both sides) v: parts[7 T + 2 + 2 d] of the upper
// face (d, 1), parts[7 T + 1 + 2 d] of a lower face on a Dirichlet boundary.
// The reaction term does not depend on theta and is left out.
// 23 x 18 x 21 Q4: 13 us here and 25 us for the faces; 85 us with every face
// evaluated from both of its elements, by points, in one kernel.
template <int N>
__global__ __launch_bounds__(kBlock) void k_dA_parts_trilinear(MeshArgs<double> m, const double* __restrict__ u,
                                                               const double* __restrict__ v,
                                                               double* __restrict__ parts) {
  constexpr int NN = N * N, EPB = elems_per_block(N), PE = Lay<N, double>::PE;
  __shared__ double sA[EPB * PE], sB[EPB * PE], sC[EPB * PE];
  __shared__ double sX[EPB][8][3];
  const Tables<double>& T = *m.tab;
  const int tid = threadIdx.x, el = tid / NN, t = tid % NN, t1 = t % N, t2 = t / N;
  const int64_t e = (int64_t)blockIdx.x * EPB + el;
  const bool act = (el < EPB) && (e < m.E);
  const int le = act ? el : 0;
  double* C = sC + le * PE;
  int ex = 0, ey = 0, ez = 0;
  if (act) {
    ex = (int)(e % m.nx);
    ey = (int)((e / m.nx) % m.ny);
    ez = (int)(e / ((int64_t)m.nx * m.ny));
  }
  MeshArgs<double> m1 = m;
  m1.R = nullptr;
  tri_volume<N, double, double>(m1, T, v, e, ex, ey, ez, act, t, t1, t2, 1.0, sX[le], sA + le * PE, sB + le * PE, C);
  // u_T . C: the lines' sums, added in thread order by the element's first thread
  double* sRed = sB + le * PE;  // no longer read (act) by the volume part's last phase
  if (act) {
    double uz[N], c[N], p = 0.0;
    glb_get<N, 2, double, double>(u, e, t1, t2, uz);
    lds_get<N, 2>(C, t1, t2, c);
#pragma unroll
    for (int i = 0; i < N; ++i) p += uz[i] * c[i];
    sRed[t] = p;
  }
  elem_sync<N>();
  if (act && t == 0) {
    double s = 0.0;
    for (int j = 0; j < NN; ++j) s += sRed[j];
    parts[7 * e] = s;
  }
}

// g_T = K_T parts[T][0] + sum over faces (d, s) of dgamma/dtheta_T times the
// whole unit-coefficient face form (of a lower interior face: the neighbour's
// part of its upper face).
// dgamma/dtheta_T = gamma K_N / (K_T + K_N) on interior faces, K_T on boundary faces.
__global__ __launch_bounds__(256) void k_dA_combine_trilinear(MeshArgs<double> m, const double* __restrict__ parts,
                                                              double* __restrict__ g) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= m.E) return;
  const int ex = (int)(e % m.nx), ey = (int)((e / m.nx) % m.ny), ez = (int)(e / ((int64_t)m.nx * m.ny));
  const double K = m.K[e];
  double acc = K * parts[7 * e];
  for (int d = 0; d < 3; ++d)
    for (int s = 0; s < 2; ++s) {
      int64_t nb;
      if (d == 0) nb = neighbour<0>(m, ex, ey, ez, s);
      else if (d == 1) nb = neighbour<1>(m, ex, ey, ez, s);
      else nb = neighbour<2>(m, ex, ey, ez, s);
      if (nb < 0) {
        acc += K * parts[7 * e + 1 + 2 * d + s];
      } else {
        const double Kn = m.K[nb];
        const double gam = 2.0 * K * Kn / (K + Kn);
        acc += gam * Kn / (K + Kn) * parts[7 * (s ? e : nb) + 2 + 2 * d];
      }
    }
  g[e] = acc;
}

// ---------------------------------------------------------------- diagonal
// diag(A)_i = a(phi_i, phi_i) by sum factorisation: phi_i is a product of 1D
// basis functions, so every term of the quadrature of a(phi_i, phi_i) is a
// point factor times a product of one 1D table entry per axis, with the
// tables of products BB, BD, DD of basis values and derivatives:
//   volume  sum_q sum_{r<=s} (2 - [r=s]) G_rs(q) T_x T_y T_z,  T_a = DD on the
//           axis r = s, BD on the two axes r != s, BB elsewhere (+ c w |det J| BB BB BB)
//   face    (end layer along D only, where phi_i != 0)
//           w (sigma gamma |N| -+ gamma l'(end) c_D) BB BB -+ w gamma (c_a BD BB + c_b BB BD),
//           c = adj(J) N / det J the conormal; on a Dirichlet face gamma -> K
//           and the flux terms twice, outward.
// n^2 threads per element as in the apply: the six factors of a z-line are
// formed from the line's Jacobian and contracted along z in registers, then
// along y and x through LDS, grouped by their x table.  The face factors are
// formed by points and contracted by whole lines with uniform tables.  Summing
// all n^3 points for every DOF instead (6 n^3 multiply-adds per DOF) took 144 ms
// against 0.93 ms on 48^3 Q7, and 1102 against 28 us on 23 x 18 x 21 Q4 (43 us
// with the face contractions by points, a lane reading its own table row), both
// inverses written in the same pass.  Vector instructions bound it.
// The three point factors of the face normal to D on side s at the thread's
// point (t1, t2) = (A, B): F0 (BB BB), F1 (BD along A), F2 (BD along B), n^2 each.
template <int N, int D>
__device__ __forceinline__ void diag_face(const MeshArgs<double>& m, const Tables<double>& T, int64_t e, int ex, int ey,
                                          int ez, const double (&X)[8][3], int t1, int t2, double* F, int s) {
  constexpr int A = D == 0 ? 1 : 0, B = D == 2 ? 1 : 2;
  const int t = t1 + N * t2;
  const int end = s ? N - 1 : 0;
  const int nD = D == 0 ? m.nx : (D == 1 ? m.ny : m.nz), c = D == 0 ? ex : (D == 1 ? ey : ez);
  const bool has = m.periodic || (s ? c < nD - 1 : c > 0);
  const bool self = m.periodic && nD == 1;  // one element along D, periodic
  const double w = T.gw[t1] * T.gw[t2], G = m.G[6 * e + 2 * D + s];
  double J[3][3], Aj[3][3];
  face_jacobian<D>(X, s, T.gx[t1], T.gx[t2], J);
  adj3(J, Aj);
  const double idet = recip(J[0][D] * Aj[D][0] + J[1][D] * Aj[D][1] + J[2][D] * Aj[D][2]);
  // N dS is row D of adj J (of the upper side's on the element's own face)
  double Nv[3] = {Aj[D][0], Aj[D][1], Aj[D][2]}, cDo = 0.0;
  if (self) {
    double Jo[3][3], Ao[3][3];
    face_jacobian<D>(X, 1 - s, T.gx[t1], T.gx[t2], Jo);
    adj3(Jo, Ao);
    if (s == 0) {
#pragma unroll
      for (int r = 0; r < 3; ++r) Nv[r] = Ao[D][r];
    }
    // the other side of the face: its normal derivative at the end node (its trace there is zero)
    cDo = (Ao[D][0] * Nv[0] + Ao[D][1] * Nv[1] + Ao[D][2] * Nv[2]) / det3(Jo) * (s ? T.d0 : T.d1)[end];
  }
  const double NN2 = Nv[0] * Nv[0] + Nv[1] * Nv[1] + Nv[2] * Nv[2];
  const double pen = (D == 0 ? m.sg[0] : (D == 1 ? m.sg[1] : m.sg[2])) * G * (has ? 2.0 : 1.0);
  // [phi] = phi on the upper face, -phi on the lower; on a Dirichlet face both
  // flux terms, outward normal: 2 G in either case
  const double fl = s ? -2.0 * G : 2.0 * G, wf = w * fl * idet;
  const double cD = self ? Aj[D][0] * Nv[0] + Aj[D][1] * Nv[1] + Aj[D][2] * Nv[2] : NN2;
  F[t] = w * (pen * root(NN2) + fl * ((s ? T.d1 : T.d0)[end] * cD * idet + cDo));
  F[N * N + t] = wf * (Aj[A][0] * Nv[0] + Aj[A][1] * Nv[1] + Aj[A][2] * Nv[2]);
  F[2 * N * N + t] = wf * (Aj[B][0] * Nv[0] + Aj[B][1] * Nv[1] + Aj[B][2] * Nv[2]);
}

template <int N>
__global__ __launch_bounds__(kBlock) void k_diag_trilinear(MeshArgs<double> m, DiagOut out, const int* run) {
  constexpr int NN = N * N, N3 = NN * N, EPB = elems_per_block(N), PE = Lay<N, double>::PE;
  // three tiles; the point factors of the six faces (18 n^2) follow the first
  constexpr int TE = 3 * PE > PE + 18 * NN ? 3 * PE : PE + 18 * NN;
  __shared__ double sT[EPB * TE];
  __shared__ double sX[EPB][8][3];
  if (run != nullptr && *run == 0) return;
  const Tables<double>& T = *m.tab;
  // the product tables, through an address derived anew at each use (all of them
  // do not fit in scalar registers at once)
  auto tabs = [&]() -> const Tables<double>& {
    uint64_t a = (uint64_t)m.tab;
    asm volatile("" : "+s"(a));
    typedef const __attribute__((address_space(4))) Tables<double>* ConstTab;
    return *(const Tables<double>*)(ConstTab)a;
  };
  const int tid = threadIdx.x, el = tid / NN, t = tid % NN, t1 = t % N, t2 = t / N;
  const int64_t e = (int64_t)blockIdx.x * EPB + el;
  const bool act = (el < EPB) && (e < m.E);
  const int le = act ? el : 0;
  double* A = sT + le * TE;
  double* B = A + PE;
  double* C = B + PE;
  int ex = 0, ey = 0, ez = 0;
  double K = 1.0;
  if (act) {
    ex = (int)(e % m.nx);
    ey = (int)((e / m.nx) % m.ny);
    ez = (int)(e / ((int64_t)m.nx * m.ny));
    K = m.K[e];
    for (int q = t; q < 24; q += NN) corner_at(m, ex, ey, ez, q / 3, q % 3, sX[le][q / 3][q % 3]);
  }
  elem_sync<N>();
  const double(&X)[8][3] = sX[le];
  // z-lines contracted along z: a00, a01, a11 with BB, a02, a12 with BD (the
  // factors 2 of the mixed terms here), a22 with DD joined by the reaction
  double a00[N], a01[N], a02[N], a11[N], a12[N], a22[N];
  if (act) {
    const JacZLine<double> jz(X, T.gx[t1], T.gx[t2]);
    const double wq = T.gw[t1] * T.gw[t2] * K, cw = m.R ? m.R[e] * T.gw[t1] * T.gw[t2] : 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i) a00[i] = a01[i] = a02[i] = a11[i] = a12[i] = a22[i] = 0.0;
#pragma unroll
    for (int q = 0; q < N; ++q) {
      double J[3][3], Aj[3][3];
      jz.at(T.gx[q], J);
      adj3(J, Aj);
      const double dJ = fabs(J[0][0] * Aj[0][0] + J[1][0] * Aj[0][1] + J[2][0] * Aj[0][2]);
      const double c = wq * T.gw[q] * recip(dJ), cr = cw * T.gw[q] * dJ;
      auto G = [&](int r, int s2) { return c * (Aj[r][0] * Aj[s2][0] + Aj[r][1] * Aj[s2][1] + Aj[r][2] * Aj[s2][2]); };
      const double g00 = G(0, 0), g01 = 2.0 * G(0, 1), g02 = 2.0 * G(0, 2), g11 = G(1, 1), g12 = 2.0 * G(1, 2),
                   g22 = G(2, 2);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const double bb = T.BB[q * kMaxN + i], bd = T.BD[q * kMaxN + i], dd = T.DD[q * kMaxN + i];
        a00[i] += bb * g00;
        a01[i] += bb * g01;
        a11[i] += bb * g11;
        a02[i] += bd * g02;
        a12[i] += bd * g12;
        a22[i] += dd * g22 + bb * cr;
      }
    }
  }
  double acc[N], v[N], w[N];
  // x table DD: a00 (y: BB)
  if (act) lds_put<N, 2>(A, t1, t2, a00);
  elem_sync<N>();
  if (act) {
    lds_get<N, 1>(A, t1, t2, v);
    prod_line<N, false>(tabs().BB, v, w);
    lds_put<N, 1>(A, t1, t2, w);
  }
  elem_sync<N>();
  if (act) {
    lds_get<N, 0>(A, t1, t2, v);
    prod_line<N, false>(tabs().DD, v, acc);
  }
  elem_sync<N>();
  // x table BD: a01 (y: BD) + a02 (y: BB)
  if (act) {
    lds_put<N, 2>(A, t1, t2, a01);
    lds_put<N, 2>(B, t1, t2, a02);
  }
  elem_sync<N>();
  if (act) {
    lds_get<N, 1>(A, t1, t2, v);
    prod_line<N, false>(tabs().BD, v, w);
    lds_get<N, 1>(B, t1, t2, v);
    prod_line<N, true>(tabs().BB, v, w);
    lds_put<N, 1>(A, t1, t2, w);
  }
  elem_sync<N>();
  if (act) {
    lds_get<N, 0>(A, t1, t2, v);
    prod_line<N, true>(tabs().BD, v, acc);
  }
  elem_sync<N>();
  // x table BB: a11 (y: DD) + a12 (y: BD) + a22 (y: BB)
  if (act) {
    lds_put<N, 2>(A, t1, t2, a11);
    lds_put<N, 2>(B, t1, t2, a12);
    lds_put<N, 2>(C, t1, t2, a22);
  }
  elem_sync<N>();
  if (act) {
    lds_get<N, 1>(A, t1, t2, v);
    prod_line<N, false>(tabs().DD, v, w);
    lds_get<N, 1>(B, t1, t2, v);
    prod_line<N, true>(tabs().BD, v, w);
    lds_get<N, 1>(C, t1, t2, v);
    prod_line<N, true>(tabs().BB, v, w);
    lds_put<N, 1>(A, t1, t2, w);
  }
  elem_sync<N>();
  if (act) {
    lds_get<N, 0>(A, t1, t2, v);
    prod_line<N, true>(tabs().BB, v, acc);
    lds_put<N, 0>(A, t1, t2, acc);  // the thread's own x-line
  }
  elem_sync<N>();
  // faces: the point factors, then 6 n lines along A and 6 n along B with
  // uniform tables; entry (t1, t2) of row r of face f = 2 D + s at (3 f + r) n^2 + t
  double* F = A + PE;
  if (act) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      diag_face<N, 0>(m, T, e, ex, ey, ez, X, t1, t2, F + 3 * s * NN, s);
      __builtin_amdgcn_sched_barrier(0);  // face by face: fewer registers
      diag_face<N, 1>(m, T, e, ex, ey, ez, X, t1, t2, F + (6 + 3 * s) * NN, s);
      __builtin_amdgcn_sched_barrier(0);
      diag_face<N, 2>(m, T, e, ex, ey, ez, X, t1, t2, F + (12 + 3 * s) * NN, s);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  elem_sync<N>();
  if (act) {
#pragma unroll 1
    for (int q = t; q < 6 * N; q += NN) {  // along A: BB F0 + BD F1 to row 0, BB F2 to row 1
      double* R = F + q / N * (3 * NN) + q % N * N;
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] = R[i];
      prod_line<N, false>(tabs().BB, v, w);
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] = R[NN + i];
      prod_line<N, true>(tabs().BD, v, w);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        R[i] = w[i];
        v[i] = R[2 * NN + i];
      }
      prod_line<N, false>(tabs().BB, v, w);
#pragma unroll
      for (int i = 0; i < N; ++i) R[NN + i] = w[i];
    }
  }
  elem_sync<N>();
  if (act) {
#pragma unroll 1
    for (int q = t; q < 6 * N; q += NN) {  // along B: BB row 0 + BD row 1 to row 2
      double* R = F + q / N * (3 * NN) + q % N;
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] = R[i * N];
      prod_line<N, false>(tabs().BB, v, w);
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] = R[NN + i * N];
      prod_line<N, true>(tabs().BD, v, w);
#pragma unroll
      for (int i = 0; i < N; ++i) R[2 * NN + i * N] = w[i];
    }
  }
  elem_sync<N>();
  if (act) {  // along x: the thread's own x-line (t1, t2) = (y, z)
    A[lds_idx<N, 0, double>(t1, t2, 0)] += F[2 * NN + t];
    A[lds_idx<N, 0, double>(t1, t2, N - 1)] += F[5 * NN + t];
  }
  elem_sync<N>();
  if (act) {
    lds_get<N, 2>(A, t1, t2, v);
    if (t2 == 0) {  // along y: the layers y = 0 and y = n - 1
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] += F[8 * NN + t1 + N * i];
    }
    if (t2 == N - 1) {
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] += F[11 * NN + t1 + N * i];
    }
    v[0] += F[14 * NN + t];  // along z
    v[N - 1] += F[17 * NN + t];
#pragma unroll
    for (int i = 0; i < N; ++i) out.put(e * N3 + lidx<N, 2>(t1, t2, i), v[i]);
  }
}

// ---------------------------------------------------------------- launchers
int64_t tri_apply_blocks(int n, int64_t E) {
  const int epb = tri_block(n) / (n * n);
  return (E + epb - 1) / epb;
}

template <int N, typename TIN, typename TOUT, typename TC, bool DOT>
static hipError_t run_tri(const MeshArgs<TC>& m, const void* x, void* y, double* partials, CgState* st, int par,
                          const int* skip, hipStream_t s) {
  const int64_t nb = tri_apply_blocks(N, m.E);
  if (m.affg)
    hipLaunchKernelGGL((k_apply_trilinear<N, TIN, TOUT, TC, true, DOT>), dim3((unsigned)nb), dim3(tri_block(N)), 0, s, m,
                       (const TIN*)x, (TOUT*)y, partials, skip);
  else
    hipLaunchKernelGGL((k_apply_trilinear<N, TIN, TOUT, TC, false, DOT>), dim3((unsigned)nb), dim3(tri_block(N)), 0, s, m,
                       (const TIN*)x, (TOUT*)y, partials, skip);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !DOT || st == nullptr) return e;  // st == nullptr: partials only
  return launch_finish_dot(partials, nb, st, par, s);
}

template <int N, bool DOT>
static hipError_t run_tri_prec(int prec, const MeshArgs<double>& m64, const MeshArgs<float>& m32, const void* x,
                               void* y, double* partials, CgState* st, int par, const int* skip, hipStream_t s) {
  switch (prec) {
    case 0: return run_tri<N, double, double, double, DOT>(m64, x, y, partials, st, par, skip, s);
    case 1: return run_tri<N, float, float, float, DOT>(m32, x, y, partials, st, par, skip, s);
    case 2: return run_tri<N, uint16_t, float, float, DOT>(m32, x, y, partials, st, par, skip, s);
  }
  return hipErrorInvalidValue;
}

template <int N>
static hipError_t run_tri_n(int prec, int dot, const MeshArgs<double>& m64, const MeshArgs<float>& m32,
                            const void* x, void* y, double* partials, CgState* st, int par, const int* skip,
                            hipStream_t s) {
  const hipError_t e = launch_tri_faces(N, prec, m64, m32, x, skip, s);
  if (e != hipSuccess) return e;
  if (dot) return run_tri_prec<N, true>(prec, m64, m32, x, y, partials, st, par, skip, s);
  return run_tri_prec<N, false>(prec, m64, m32, x, y, partials, st, par, skip, s);
}

hipError_t launch_apply_trilinear(int n, int prec, int trans, int dot, const MeshArgs<double>& m64,
                                  const MeshArgs<float>& m32, const void* x, void* y, double* partials,
                                  CgState* st, int par, const int* skip, hipStream_t s) {
  (void)trans;  // symmetric form: A^T x is evaluated by the same kernel
  switch (n) {
    case 2: return run_tri_n<2>(prec, dot, m64, m32, x, y, partials, st, par, skip, s);
    case 3: return run_tri_n<3>(prec, dot, m64, m32, x, y, partials, st, par, skip, s);
    case 4: return run_tri_n<4>(prec, dot, m64, m32, x, y, partials, st, par, skip, s);
    case 5: return run_tri_n<5>(prec, dot, m64, m32, x, y, partials, st, par, skip, s);
    case 6: return run_tri_n<6>(prec, dot, m64, m32, x, y, partials, st, par, skip, s);
    case 7: return run_tri_n<7>(prec, dot, m64, m32, x, y, partials, st, par, skip, s);
    case 8: return run_tri_n<8>(prec, dot, m64, m32, x, y, partials, st, par, skip, s);
  }
  return hipErrorInvalidValue;
}

template <int N>
static hipError_t run_tri_diag(const MeshArgs<double>& m, const DiagOut& d, const int* run, hipStream_t s) {
  hipLaunchKernelGGL((k_diag_trilinear<N>), dim3((unsigned)element_blocks(N, m.E)), dim3(kBlock), 0, s, m, d, run);
  return hipGetLastError();
}
template <int N>
static hipError_t run_dA_tri(const MeshArgs<double>& m, const double* u, const double* v, double* parts, double* g,
                             hipStream_t s) {
  const int64_t nb = element_blocks(N, m.E);
  hipError_t e = launch_tri_faces_dA(N, m, u, v, parts, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_dA_parts_trilinear<N>), dim3((unsigned)nb), dim3(kBlock), 0, s, m, u, v, parts);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_dA_combine_trilinear, dim3((unsigned)((m.E + 255) / 256)), dim3(256), 0, s, m, parts, g);
  return hipGetLastError();
}

hipError_t launch_dA_trilinear(int n, const MeshArgs<double>& m, const double* u, const double* v, double* parts,
                               double* g, hipStream_t s) {
  switch (n) {
    case 2: return run_dA_tri<2>(m, u, v, parts, g, s);
    case 3: return run_dA_tri<3>(m, u, v, parts, g, s);
    case 4: return run_dA_tri<4>(m, u, v, parts, g, s);
    case 5: return run_dA_tri<5>(m, u, v, parts, g, s);
    case 6: return run_dA_tri<6>(m, u, v, parts, g, s);
    case 7: return run_dA_tri<7>(m, u, v, parts, g, s);
    case 8: return run_dA_tri<8>(m, u, v, parts, g, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_diag_trilinear(int n, const MeshArgs<double>& m, const DiagOut& d, const int* run, hipStream_t s) {
  switch (n) {
    case 2: return run_tri_diag<2>(m, d, run, s);
    case 3: return run_tri_diag<3>(m, d, run, s);
    case 4: return run_tri_diag<4>(m, d, run, s);
    case 5: return run_tri_diag<5>(m, d, run, s);
    case 6: return run_tri_diag<6>(m, d, run, s);
    case 7: return run_tri_diag<7>(m, d, run, s);
    case 8: return run_tri_diag<8>(m, d, run, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace dg
