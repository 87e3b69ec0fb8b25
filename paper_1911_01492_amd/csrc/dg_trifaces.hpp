// dg_trifaces.hpp -- face terms of the trilinear apply: the first of its two
// kernels (the second, in dg_trilinear.hip, adds them to the volume part), and
// of the sensitivity dA/dtheta.
//
// Every face is evaluated once, an interior one by its lower element T^-.  With
// the trace u and the raw normal derivative g of a side on the n x n face
// nodes, v = B B u, (ga, gb) = tangential derivatives, gd = B B g at the Gauss
// points, N = n dS of T^-, c_r = adj(J)_r . N / det J of the side, the face form
// (Sec. 4.1) gives at every point, with J = v^- - v^+, F = sum of c . (gd, ga, gb)
// over the two sides and G the face coefficient (gamma / 2 inside, K on a
// Dirichlet face, where T^+ is absent),
//     P^- = w (sigma gamma |N| J - G F) = -P^+,   R^+- = -w G J c^+-,
// and the rows of a side are  out = (B B)^T (P + Dg_a^T Ra + Dg_b^T Rb)  on the
// face nodes plus  z = (B B)^T Rd  times the normal derivatives l_i'(end) along
// the line behind each.  They go to the face buffer of the workspace in the
// basis in which the volume kernel holds its lines of that axis: Gauss points
// in both directions for axis 0, x projected for axis 1, both for axis 2.
//
// A wave evaluates F = 64 / (2 n) faces of one axis with no barrier: a lane owns
// one side and one line of n points in each of the four contractions, all in
// registers with the tables uniform; only the turn of the lines goes through
// LDS.  The sides of a face are neighbouring lanes and exchange N, v and F by
// DPP.
//
// With one thread per face point instead (each output a dot product of n LDS
// values with a table row of the thread's own, in one kernel with the volume
// part) an apply of 48^3 Q7 took 1500 us; with this kernel 945 us back to back (1090
// in a run of a few applies: faces 516, volume 587), against 450 us for its
// arithmetic (581 flop per DOF) at the rate of a large FP64 product; the two kernels
// move 3.2 GB.  FP64 arithmetic bounds it: at n = 8 1764 vector instructions per wave,
// 65% of the cycles at three waves per SIMD (about 100 of them per face point for
// the two conormals, 1 / det, |N| and the exchange); the address unit is busy 59%.
// In FP32 (1647 instructions) the VALU is saturated.
// Others, apply before -> now: 73^3 Q3 919 -> 612 us, 58^3 Q4 899 -> 568, 42^3 Q6
// 873 -> 537, 146^3 Q1 2076 -> 1412; FP32 37^3 Q7 339 -> 229, 48^3 Q7 713 -> 515.
// Part of the translation unit dg_trilinear.hip.
#pragma once

#include "dg_internal.hpp"
#include "dg_kernels.hpp"
#include "dg_lines.hpp"
#include "dg_geom.hpp"
#include "dg_tables.hpp"

#include <algorithm>
#include <type_traits>

namespace dg {

// One wave per axis works on the same kFaces<n> elements: 3 waves per block.
constexpr int kFaceBlock = 192;
__host__ __device__ constexpr int faces_per_wave(int n) { return 64 / (2 * n); }

// LDS place of entry (r, c) of side q: q SS + r RS + c, from a search over the
// bank conflicts of the row, column and tile accesses (16 lanes at a time for
// 8-byte words, 32 for 4-byte words); none at n = 2, 4, 8.
template <int N, typename TC>
struct FaceLay {
  static constexpr bool f64 = sizeof(TC) == 8;
  static constexpr int RS = N == 2 ? 3 : N == 4 ? 5 : N == 7 ? 10 : N == 8 ? 9 : N == 5 ? (f64 ? 6 : 5) : 6;
  static constexpr int SS = N == 2 ? 6 : N == 3 ? (f64 ? 25 : 41) : N == 4 ? 20 : N == 5 ? (f64 ? 39 : 25) :
                            N == 6 ? (f64 ? 39 : 53) : N == 7 ? (f64 ? 75 : 83) : 72;
  static_assert(SS >= (N - 1) * RS + N && RS >= N, "rows and sides apart");
};

// ordering point between LDS accesses of the lanes of one wave (they execute
// together and their LDS operations complete in order)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// value of the lane QP selects inside each four: 0xB1 the other side of the
// face, 0xA0 the T^- side for both
template <int QP>
__device__ __forceinline__ float quad(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), QP, 0xf, 0xf, true));
}
template <int QP>
__device__ __forceinline__ double quad(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, QP, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), QP, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// u and g of one line v, to a side's entry (node r along B, c along A at r RS + c)
template <int N, typename TC, typename TT>
__device__ __forceinline__ void put_trace(const TT& T, const TC (&v)[N], bool end, int at, TC* sU, TC* sG) {
  TC a = TC(0), b = TC(0);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    a += T.d0[i] * v[i];
    b += T.d1[i] * v[i];
  }
  sU[at] = end ? v[N - 1] : v[0];
  sG[at] = end ? b : a;
}

// Traces u and raw normal derivatives g of the sides of a wave's faces normal
// to axis D; elem[q] is the element of side q, or -1 - (an element to read
// instead) where the side is absent (its row is replaced by zeros later).
template <int N, int D, typename TC, typename TIN, typename TT>
__device__ __forceinline__ void load_traces(const TT& T, const TIN* __restrict__ x, const int* elem, bool lower,
                                            TC* sU, TC* sG) {
  constexpr int NN = N * N, N3 = NN * N, SIDES = 2 * faces_per_wave(N);
  constexpr int RS = FaceLay<N, TC>::RS, SS = FaceLay<N, TC>::SS;
  constexpr int st = D == 0 ? 1 : (D == 1 ? N : NN);  // along D
  const int lane = threadIdx.x & 63;
  if constexpr (N % 2 == 0 && D > 0) {
    // two lines, neighbours along x, per lane: twice as wide loads, which cost
    // the address unit as much as single ones
    typedef TIN pair_t __attribute__((ext_vector_type(2), aligned(sizeof(TIN))));
    constexpr int HP = NN / 2;
#pragma unroll 1
    for (int q = lane; q < SIDES * HP; q += 64) {
      const int sd = q / HP, t = 2 * (q - sd * HP), tb = t % N, ta = t / N;
      const int ee = elem[sd], e = ee < 0 ? -1 - ee : ee;
      const TIN* p = x + (int64_t)e * N3 + (D == 1 ? tb + ta * NN : t);
      TC v[N], w[N];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const pair_t r = *(const pair_t*)(p + i * st);
        const TIN r0 = r.x, r1 = r.y;
        v[i] = load_as<TC, TIN>(&r0);
        w[i] = load_as<TC, TIN>(&r1);
      }
      const int at = sd * SS + tb * RS + ta;
      put_trace<N>(T, v, (sd & 1) == 0 && !lower, at, sU, sG);
      put_trace<N>(T, w, (sd & 1) == 0 && !lower, at + RS, sU, sG);
    }
    return;
  }
#pragma unroll 2
  for (int q = lane; q < SIDES * NN; q += 64) {
    const int sd = q / NN, t = q - sd * NN, tb = t % N, ta = t / N;
    const int ee = elem[sd], e = ee < 0 ? -1 - ee : ee;
    const TIN* p = x + (int64_t)e * N3 + (D == 0 ? tb * N + ta * NN : (D == 1 ? tb + ta * NN : tb + ta * N));
    TC v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = load_as<TC, TIN>(p + i * st);
    put_trace<N>(T, v, (sd & 1) == 0 && !lower, sd * SS + tb * RS + ta, sU, sG);
  }
}
// The same for x-lines from n = 5 on: a lane's line is 40 bytes or more, so
// the wave reads whole elements (PS of them at a time) and turns them through
// LDS; read by lines, every 16 bytes of a lane were an access of their own.
template <int N, typename TC>
struct TileX {
  static constexpr bool use = N >= 5;
  static constexpr int PS = use ? 64 / (N * N) : 1, TS = N | 1, TILE = use ? N * N * TS : 1;
};
template <int N, typename TC, typename TIN, typename TT>
__device__ __forceinline__ void load_traces_x(const TT& T, const TIN* __restrict__ x, const int* elem, bool lower,
                                              TC* sU, TC* sG, TC* tile) {
  constexpr int NN = N * N, N3 = NN * N, SIDES = 2 * faces_per_wave(N);
  constexpr int RS = FaceLay<N, TC>::RS, SS = FaceLay<N, TC>::SS;
  constexpr int PS = TileX<N, TC>::PS, TS = TileX<N, TC>::TS, TILE = TileX<N, TC>::TILE;
  static_assert(SIDES % PS == 0, "whole passes");
  const int lane = threadIdx.x & 63;
  // in pairs where an element has an even number of values
  constexpr int W = N % 2 == 0 ? 2 : 1, KW = (N3 / W + 63) / 64;
  typedef TIN wide_t __attribute__((ext_vector_type(W), aligned(sizeof(TIN))));
  wide_t r[PS][KW];
  auto load = [&](int s0) {
#pragma unroll
    for (int s = 0; s < PS; ++s) {
      const int ee = __builtin_amdgcn_readfirstlane(elem[s0 + s]), e = ee < 0 ? -1 - ee : ee;
      const TIN* p = x + (int64_t)e * N3;
#pragma unroll
      for (int k = 0; k < KW; ++k) r[s][k] = *(const wide_t*)(p + min(W * (k * 64 + lane), N3 - W));
    }
  };
  load(0);
  const int ls = lane / NN, t = lane - ls * NN, tb = t % N, ta = t / N;
#pragma unroll 1
  for (int s0 = 0; s0 < SIDES; s0 += PS) {
#pragma unroll
    for (int s = 0; s < PS; ++s)
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        const int at = W * (k * 64 + lane);
        if (at < N3) {
#pragma unroll
          for (int w = 0; w < W; ++w) {
            const TIN one = r[s][k][w];
            tile[s * TILE + at + w + at / N * (TS - N)] = load_as<TC, TIN>(&one);
          }
        }
      }
    if (s0 + PS < SIDES) load(s0 + PS);
    wave_sync();
    if (ls < PS) {
      const int sd = s0 + ls;
      TC v[N];
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] = tile[ls * TILE + t * TS + i];
      put_trace<N>(T, v, (sd & 1) == 0 && !lower, sd * SS + tb * RS + ta, sU, sG);
    }
    wave_sync();
  }
}

// The faces of one wave: the upper faces normal to axis D of F elements, or (lower)
// F faces of the boundary layer below, which have their upper element only.
struct FaceSet {
  int D, nD, stD;
  bool lower;
  int64_t f0, nf;  // first face, faces of this kind
  template <int N, typename TC>
  __device__ __forceinline__ FaceSet(const MeshArgs<TC>& m, int64_t nreg, std::integral_constant<int, N>) {
    D = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    nD = D == 0 ? m.nx : (D == 1 ? m.ny : m.nz);
    stD = D == 0 ? 1 : (D == 1 ? m.nx : m.nx * m.ny);
    lower = (int64_t)blockIdx.x >= nreg;
    f0 = (lower ? (int64_t)blockIdx.x - nreg : xcd_remap(blockIdx.x, nreg)) * faces_per_wave(N);
    nf = lower ? m.E / nD : m.E;
  }
  // element and first vertex of each side (both below 2^31), by lanes below 2 F;
  // an absent side: -1 - (the element below)
  template <int N, typename TC>
  __device__ __forceinline__ void sides(const MeshArgs<TC>& m, std::integral_constant<int, N>, int* el, int* vx) const {
    const int lane = threadIdx.x & 63;
    if (lane < 2 * faces_per_wave(N)) {
      const unsigned nx = m.nx, ny = m.ny, q = (unsigned)min(f0 + (lane >> 1), nf - 1);
      unsigned ex, ey, ez;
      if (!lower) {
        const unsigned r = q / nx;
        ex = q - r * nx;
        ez = r / ny;
        ey = r - ez * ny;
      } else {  // element q of the boundary layer
        const unsigned n1 = D == 0 ? ny : nx, b = q / n1, a = q - b * n1;
        ex = D == 0 ? 0 : a;
        ey = D == 0 ? a : (D == 1 ? 0 : b);
        ez = D == 2 ? 0 : b;
      }
      const int e = (int)(ex + nx * (ey + ny * ez)), c = (int)(D == 0 ? ex : (D == 1 ? ey : ez));
      const int sv = D == 0 ? 1 : (D == 1 ? (int)nx + 1 : (int)((nx + 1) * (ny + 1)));
      int id = e, v = (int)(ex + (nx + 1) * (ey + (ny + 1) * ez));
      if (lane & 1) {  // the element across the upper face
        const int d = c < nD - 1 ? 1 : 1 - nD;
        if (lower || (c == nD - 1 && !m.periodic)) {
          id = -1 - e;
        } else {
          id = e + d * stD;
          v += d * sv;
        }
      }
      el[lane] = id;
      vx[lane] = v;
    }
    wave_sync();
  }
};

// The corners of the sides, 3 corner + axis at stride 25: loaded early, stored later
template <int N, typename TC>
struct Corners {
  static constexpr int SIDES = 2 * faces_per_wave(N), NC = (SIDES * 8 + 63) / 64;
  TC cor[NC][3];
  __device__ __forceinline__ void load(const MeshArgs<TC>& m, const int* vx) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int r = 0; r < NC; ++r) {
      const int q = lane + 64 * r, cc = q & 7;
      const int v = vx[SIDES % 8 == 0 ? q >> 3 : min(q >> 3, SIDES - 1)] + (cc & 1) +
                    (m.nx + 1) * (((cc >> 1) & 1) + (m.ny + 1) * (cc >> 2));
      const TC* X = m.vert + (int64_t)3 * v;
#pragma unroll
      for (int a = 0; a < 3; ++a) cor[r][a] = X[a];
    }
  }
  __device__ __forceinline__ void store(TC* sC) const {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int r = 0; r < NC; ++r) {
      const int q = lane + 64 * r;
      if (SIDES % 8 == 0 || q < SIDES * 8)
#pragma unroll
        for (int a = 0; a < 3; ++a) sC[(q >> 3) * 25 + 3 * (q & 7) + a] = cor[r][a];
    }
  }
};

// waves per SIMD asked of the register allocator: FP64 fits 128 registers up to
// n = 5 (at n = 3 LDS leaves room for three) and 168 above; the sensitivity, which
// reads a second vector, 128 up to n = 4 and, but for n = 5 and 8, two waves above.
// FP32 takes 104 registers at n = 8 where it may, 89 with five waves (48^3 Q7 531 ->
// 519 us; six spill, 543).
__host__ __device__ constexpr int face_min_waves(int n, int bytes, bool dA) {
  if (bytes == 4) return n == 8 ? 5 : 4;
  return n <= (dA ? 4 : 5) && n != 3 ? 4 : (dA && (n == 6 || n == 7) ? 2 : 3);
}

// DA: the sensitivity instead of the apply: with the coefficient G = 1/2 (1 on a
// Dirichlet face) the rows of both sides are projected to the nodes and summed
// against the traces of z, one value per face, into parts[7 e + 1 + 2 D + side]
// (dg_trilinear.hip).
template <int N, typename TIN, typename TC, bool DA>
__global__ __launch_bounds__(kFaceBlock) __attribute__((amdgpu_waves_per_eu(face_min_waves(N, sizeof(TC), DA)))) void k_tri_faces(
    MeshArgs<TC> m, const TIN* __restrict__ x, int64_t nreg, const int* skip, const TIN* __restrict__ z,
    double* __restrict__ parts) {
  constexpr int NN = N * N, F = faces_per_wave(N), SIDES = 2 * F;
  constexpr int RS = FaceLay<N, TC>::RS, SS = FaceLay<N, TC>::SS;
  constexpr bool FULL = SIDES * N == 64;
  __shared__ TC sBuf[3][2][SIDES * SS], sCor[3][SIDES * 25];
  __shared__ TC sTile[TileX<N, TC>::PS * TileX<N, TC>::TILE];
  __shared__ int sEl[3][SIDES], sVx[3][SIDES];
  if (skip != nullptr && *skip) return;
  constexpr bool CTAB = sizeof(TC) == 4;
  [[maybe_unused]] constexpr KTables<TC> ktab = CTAB ? ctab::make<N, TC>() : KTables<TC>{};
  auto tabs = [&]() -> decltype(auto) {
    if constexpr (CTAB) {
      return (ktab);
    } else {  // each stage loads the tables it uses (see k_apply_ppd)
      uint64_t a = (uint64_t)m.tab;
      asm volatile("" : "+s"(a));
      typedef const __attribute__((address_space(4))) Tables<TC>* ConstTab;
      return *(const Tables<TC>*)(ConstTab)a;
    }
  };
  const FaceSet fset(m, nreg, std::integral_constant<int, N>{});
  const int D = fset.D, lane = threadIdx.x & 63;
  const bool lower = fset.lower;
  if (fset.f0 >= fset.nf) return;
  TC* sU = sBuf[D][0];
  TC* sG = sBuf[D][1];
  TC* sC = sCor[D];
  int* el = sEl[D];
  fset.sides(m, std::integral_constant<int, N>{}, el, sVx[D]);
  Corners<N, TC> cor;
  cor.load(m, sVx[D]);
  auto traces = [&](const TIN* __restrict__ vec) {
    const auto& T = tabs();
    if (D == 0) {
      if constexpr (TileX<N, TC>::use) load_traces_x<N, TC, TIN>(T, vec, el, lower, sU, sG, sTile);
      else load_traces<N, 0, TC, TIN>(T, vec, el, lower, sU, sG);
    } else if (D == 1) {
      load_traces<N, 1, TC, TIN>(T, vec, el, lower, sU, sG);
    } else {
      load_traces<N, 2, TC, TIN>(T, vec, el, lower, sU, sG);
    }
  };
  traces(x);
  cor.store(sC);
  wave_sync();
  // ---- the lane's side and line
  const int side = lane & 1;
  const bool on = FULL || lane < SIDES * N;
  const int fj = on ? lane >> 1 : 0, f = fj / N, j = fj - f * N, sd = 2 * f + side;
  const int row = sd * SS + j * RS, col = sd * SS + j;
  TC u[N], g[N], v[N], gb[N], ga[N], gd[N];
  {  // along axis A at t_B = j: bu = B u, du = Dg bu, bg = B g, turned
    const auto& T = tabs();
#pragma unroll
    for (int i = 0; i < N; ++i) u[i] = sU[row + i];
#pragma unroll
    for (int i = 0; i < N; ++i) g[i] = sG[row + i];
    if (el[sd] < 0) {
#pragma unroll
      for (int i = 0; i < N; ++i) u[i] = g[i] = TC(0);
    }
    contract_eo<N, TC, 1>(T.eB, u, v);
    contract_eo<N, TC, -1>(T.eDg, v, ga);
    contract_eo<N, TC, 1>(T.eB, g, gd);
    wave_sync();
    if (on) {
#pragma unroll
      for (int i = 0; i < N; ++i) sU[row + i] = v[i];
#pragma unroll
      for (int i = 0; i < N; ++i) sG[row + i] = ga[i];
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < N; ++i) u[i] = sU[col + i * RS];
#pragma unroll
    for (int i = 0; i < N; ++i) g[i] = sG[col + i * RS];
    wave_sync();
    if (on) {
#pragma unroll
      for (int i = 0; i < N; ++i) sU[row + i] = gd[i];
    }
    wave_sync();
  }
  {  // along axis B at Gauss point j of A: v = B bu, gb = Dg v, ga = B du, gd = B bg
    const auto& T = tabs();
    contract_eo<N, TC, 1>(T.eB, u, v);
    contract_eo<N, TC, -1>(T.eDg, v, gb);
    contract_eo<N, TC, 1>(T.eB, g, ga);
#pragma unroll
    for (int i = 0; i < N; ++i) u[i] = sU[col + i * RS];
    contract_eo<N, TC, 1>(T.eB, u, gd);
  }
  {  // ---- points (xi_A, xi_B) = (x_j, x_i), own side; J's column along B is constant, A and D affine in xi_B
    const auto& T = *m.tab;
    const FaceLine<TC> L(sC + sd * 25, D, side == 0 && !lower ? 1 : 0, T.gx[j]);
    const TC odd = D == 1 ? TC(1) : TC(-1);
    const bool has = el[2 * f + 1] >= 0;
    const TC G = DA ? (has ? TC(0.5) : TC(1)) : m.G[(int64_t)6 * el[2 * f] + 2 * D + (lower ? 0 : 1)];
    TC pen = (D == 0 ? m.sg[0] : (D == 1 ? m.sg[1] : m.sg[2])) * G * (has ? TC(2) : TC(1));
    const TC gs = side != 0 || lower ? -G : G;  // sign of J on this side, outward N on a lower boundary
    const TC wj = T.gw[j];
    [[maybe_unused]] TC sN = TC(1);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const TC tb = T.gx[i], w = wj * T.gw[i];
      const V3<TC> ja = lin(L.ap, tb, L.aq), jd = lin(L.dp, tb, L.dq);
      const V3<TC> nd = cross(ja, L.jb);
      const V3<TC> Nv = {quad<0xA0>(nd.x), quad<0xA0>(nd.y), quad<0xA0>(nd.z)};
      // c = adj N / det; in FP32 N is divided first: nothing of h^4 but |N|^2 is formed,
      TC idet = recip_det(dot(jd, nd)), NN2 = dot(Nv, Nv);
      V3<TC> Nc = Nv;
      if constexpr (sizeof(TC) == 4) {
        Nc = {Nv.x * idet, Nv.y * idet, Nv.z * idet};
        idet = TC(1);
        // which is subnormal at edges near 1e-10, where |N| is not: where it is below 2^-62
        // at the line's first point, 2^64 |N|^2 and 2^-32 of the penalty instead (N is affine
        // in xi_B and the Gauss points are off the ends, so on a valid face |N|^2 differs by
        // less than 2^12 along the line)
        if (i == 0) {
          const bool tiny = NN2 < 0x1p-62f;
          sN = tiny ? 0x1p64f : 1.0f;
          pen *= tiny ? 0x1p-32f : 1.0f;
        }
        NN2 *= sN;
      }
      const TC cd = dot(nd, Nc), ca = dot(cross(L.jb, jd), Nc), cb = dot(cross(jd, ja), Nc);
      TC fl = (cd * gd[i] + ca * ga[i] + odd * (cb * gb[i])) * idet;
      fl += quad<0xB1>(fl);
      const TC Jm = v[i] - quad<0xB1>(v[i]);
      const TC area = root(NN2);
      const TC co = -w * gs * Jm * idet;
      v[i] = w * (pen * area * Jm - gs * fl);
      gd[i] = co * cd;
      ga[i] = co * ca;
      gb[i] = co * cb;
      // points in groups: no spills at 168 (n = 8) and 128 (n = 5) registers (back to back
      // the faces of 48^3 Q7 took 497 us one by one, 450 by four)
      if (sizeof(TC) == 8 && ((N == 8 && i == 3) || (N == 5 && (i & 1)))) __builtin_amdgcn_sched_barrier(0);
    }
  }
  {  // along axis B: x = P + Dg^T Rb; from D = 1 on B^T x, B^T Ra, B^T Rd
    const auto& T = tabs();
    contract_eo<N, TC, -1>(T.eDgt, gb, u);
    const TC odd = D == 1 ? TC(1) : TC(-1);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += odd * u[i];
    if (DA || D >= 1) {
      contract_eo<N, TC, 1>(T.eBt, v, u);
      contract_eo<N, TC, 1>(T.eBt, ga, g);
      contract_eo<N, TC, 1>(T.eBt, gd, gb);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        v[i] = u[i];
        ga[i] = g[i];
        gd[i] = gb[i];
      }
    }
    wave_sync();
    if (on) {
#pragma unroll
      for (int i = 0; i < N; ++i) sU[col + i * RS] = v[i];
#pragma unroll
      for (int i = 0; i < N; ++i) sG[col + i * RS] = ga[i];
    }
    wave_sync();
  }
  // ---- lanes side by side from here: the lines of a side are stored by neighbouring lanes
  int lane2 = on ? lane : 0;
  asm volatile("" : "+v"(lane2));  // not formed (and kept) earlier
  const int sd2 = lane2 / N, j2 = lane2 - sd2 * N, row2 = sd2 * SS + j2 * RS;
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = sU[row2 + i];
#pragma unroll
  for (int i = 0; i < N; ++i) ga[i] = sG[row2 + i];
  wave_sync();
  if (on) {
#pragma unroll
    for (int i = 0; i < N; ++i) sU[col + i * RS] = gd[i];
  }
  wave_sync();
#pragma unroll
  for (int i = 0; i < N; ++i) gd[i] = sU[row2 + i];
  {  // along axis A: x + Dg^T Ra, for D = 2 B^T; to the face buffer
    const auto& T = tabs();
    contract_eo<N, TC, -1>(T.eDgt, ga, u);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += u[i];
    if (DA || D == 2) {
      contract_eo<N, TC, 1>(T.eBt, v, u);
      contract_eo<N, TC, 1>(T.eBt, gd, g);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        v[i] = u[i];
        gd[i] = g[i];
      }
    }
    const int e = el[sd2];
    const bool own = on && e >= 0 && fset.f0 + (sd2 >> 1) < fset.nf;
    if constexpr (DA) {
      // the rows against the traces of z, summed per face in lane order
      wave_sync();
      traces(z);
      wave_sync();
      TC p = TC(0);
#pragma unroll
      for (int i = 0; i < N; ++i) p += v[i] * sU[row2 + i] + gd[i] * sG[row2 + i];
      wave_sync();
      if (on) sU[lane] = own ? p : TC(0);
      wave_sync();
      if (lane < F && fset.f0 + lane < fset.nf) {
        TC t = TC(0);
        for (int i = 0; i < 2 * N; ++i) t += sU[lane * 2 * N + i];
        parts[(int64_t)7 * el[2 * lane] + 1 + 2 * D + (lower ? 0 : 1)] = t;
      }
    } else if (own) {
      TC* fb = ((sd2 & 1) != 0 || lower ? m.fb : m.fbu) + ((int64_t)e * 3 + D) * (2 * NN) + j2;
#pragma unroll
      for (int i = 0; i < N; ++i) fb[i * N] = v[i];
#pragma unroll
      for (int i = 0; i < N; ++i) fb[NN + i * N] = gd[i];
    }
  }
}

// blocks: F elements' upper faces each, then the boundary layers (the axis with
// most of them sets their number)
template <int N>
static unsigned face_blocks(const MeshArgs<double>& m, int64_t& nreg) {
  const int64_t F = faces_per_wave(N), most = m.periodic ? 0 : m.E / std::min(m.nx, std::min(m.ny, m.nz));
  nreg = (m.E + F - 1) / F;
  return (unsigned)(nreg + (most + F - 1) / F);
}
template <int N>
static hipError_t run_tri_faces(int prec, const MeshArgs<double>& m64, const MeshArgs<float>& m32, const void* x,
                                const int* skip, hipStream_t s) {
  int64_t nreg;
  const dim3 grid(face_blocks<N>(m64, nreg)), block(kFaceBlock);
  switch (prec) {
    case 0:
      hipLaunchKernelGGL((k_tri_faces<N, double, double, false>), grid, block, 0, s, m64, (const double*)x, nreg, skip,
                         (const double*)nullptr, (double*)nullptr);
      break;
    case 1: hipLaunchKernelGGL((k_tri_faces<N, float, float, false>), grid, block, 0, s, m32, (const float*)x, nreg, skip,
                         (const float*)nullptr, (double*)nullptr); break;
    case 2:
      hipLaunchKernelGGL((k_tri_faces<N, uint16_t, float, false>), grid, block, 0, s, m32, (const uint16_t*)x, nreg, skip,
                         (const uint16_t*)nullptr, (double*)nullptr);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
template <int N>
static hipError_t run_tri_faces_dA(const MeshArgs<double>& m, const double* u, const double* v, double* parts,
                                   hipStream_t s) {
  int64_t nreg;
  const dim3 grid(face_blocks<N>(m, nreg)), block(kFaceBlock);
  hipLaunchKernelGGL((k_tri_faces<N, double, double, true>), grid, block, 0, s, m, v, nreg, (const int*)nullptr, u,
                     parts);
  return hipGetLastError();
}
static hipError_t launch_tri_faces(int n, int prec, const MeshArgs<double>& m64, const MeshArgs<float>& m32,
                                   const void* x, const int* skip, hipStream_t s) {
  switch (n) {
    case 2: return run_tri_faces<2>(prec, m64, m32, x, skip, s);
    case 3: return run_tri_faces<3>(prec, m64, m32, x, skip, s);
    case 4: return run_tri_faces<4>(prec, m64, m32, x, skip, s);
    case 5: return run_tri_faces<5>(prec, m64, m32, x, skip, s);
    case 6: return run_tri_faces<6>(prec, m64, m32, x, skip, s);
    case 7: return run_tri_faces<7>(prec, m64, m32, x, skip, s);
    case 8: return run_tri_faces<8>(prec, m64, m32, x, skip, s);
  }
  return hipErrorInvalidValue;
}
static hipError_t launch_tri_faces_dA(int n, const MeshArgs<double>& m, const double* u, const double* v,
                                      double* parts, hipStream_t s) {
  switch (n) {
    case 2: return run_tri_faces_dA<2>(m, u, v, parts, s);
    case 3: return run_tri_faces_dA<3>(m, u, v, parts, s);
    case 4: return run_tri_faces_dA<4>(m, u, v, parts, s);
    case 5: return run_tri_faces_dA<5>(m, u, v, parts, s);
    case 6: return run_tri_faces_dA<6>(m, u, v, parts, s);
    case 7: return run_tri_faces_dA<7>(m, u, v, parts, s);
    case 8: return run_tri_faces_dA<8>(m, u, v, parts, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace dg
