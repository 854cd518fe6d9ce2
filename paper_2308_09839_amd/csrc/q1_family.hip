// Element families beyond the trilinear hexahedron, named in the paper's
// conclusions (Section 7) as the next cases for its matrix-free algorithm:
// linear tetrahedra (simplicial elements) and triquadratic and tricubic
// hexahedra (higher-order elements).  The operators are the same scalar Laplace and
// isotropic elasticity with cell-wise coefficients (Section 2), applied
// without a matrix by the gather / local product / scatter-add of Section 3.
//
// Linear tetrahedra: one thread per element.  With E_c = X_c - X_0 (c = 1, 2,
// 3) the cross products c_1 = E_2 x E_3, c_2 = E_3 x E_1, c_3 = E_1 x E_2 and
// c_0 = -(c_1 + c_2 + c_3) are det J times the (constant) physical gradients
// of the four basis functions, det J = E_1 . c_1 and the volume det J / 6, so
//   Laplace      v_a = k (c_a . g) / (6 det J),  g = sum_b c_b u_b,
//   elasticity   v_a = S c_a / (6 det J),  S = lambda tr(H) I + mu (H + H^T),
//                H = sum_b u_b (x) c_b (= det J grad u).
// Hexahedra of order P = 2 (27 nodes) and 3 (64 nodes): (P+1)^2 lanes per
// element, each with a line of P+1 nodes, then of quadrature points of the (P+1)^3
// Gauss rule.  At a point: the Jacobian J, its adjugate A (rows the cross products
// of the columns, so J^-1 = A / det J), the reference gradients g of the input and
// the reference flux f, with v_a = sum_q grad_hat phi_a(q) . f(q):
//   Laplace      f = k w A (sum_c g_c A_c) / det J,
//   elasticity   f_i = w S_i A^T / det J,  H = G A (det J grad u, rows of G
//                the reference gradients of the components), S as above;
// The diagonal keeps one thread per node and point.  Both element kinds scatter with
// global atomics (the paper's one-thread-per-element strategy), after
// y = x on Dirichlet nodes and 0 elsewhere.
#include <hip/hip_runtime.h>

#include "q1_elem.hpp"
#include "q1_internal.hpp"

namespace q1 {
namespace {

constexpr int kFB = 256;  // threads per block

__device__ __forceinline__ void gadd(double *p, double v) { unsafeAtomicAdd(p, v); }
__device__ __forceinline__ void gadd(float *p, float v) { unsafeAtomicAdd(p, v); }

// y = x on Dirichlet nodes, 0 elsewhere (before the atomic scatter); the same
// with 1 for the diagonal
template <typename T, int DPN>
__global__ void k_fam_init(int64_t nn, const uint8_t *__restrict__ mask,
                           const T *__restrict__ x, T *__restrict__ y,
                           const int *__restrict__ stop) {
  if (stop && *stop) return;
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= nn * DPN) return;
  const bool fx = mask && mask[i / DPN];
  y[i] = fx ? (x ? x[i] : T(1)) : T(0);
}

// ---- linear tetrahedra -----------------------------------------------------

template <typename T>
struct TetGeom {
  T c[4][3];  // det J times the physical gradients
  T s;        // 1 / (6 det J)
};

template <typename T>
__device__ __forceinline__ TetGeom<T> tet_geom(const T X[3][4]) {
  TetGeom<T> G;
  const T E1[3] = {X[0][1] - X[0][0], X[1][1] - X[1][0], X[2][1] - X[2][0]};
  const T E2[3] = {X[0][2] - X[0][0], X[1][2] - X[1][0], X[2][2] - X[2][0]};
  const T E3[3] = {X[0][3] - X[0][0], X[1][3] - X[1][0], X[2][3] - X[2][0]};
  cross(E2, E3, G.c[1]);
  cross(E3, E1, G.c[2]);
  cross(E1, E2, G.c[3]);
#pragma unroll
  for (int r = 0; r < 3; ++r) G.c[0][r] = -(G.c[1][r] + G.c[2][r] + G.c[3][r]);
  G.s = rcp(T(6) * dot3(E1, G.c[1]));
  return G;
}

template <typename T, int PH, bool MASKED>
__global__ __launch_bounds__(kFB) void k_tet_apply(int64_t ne, int64_t nn,
                                                   const T *__restrict__ xyz,
                                                   const int32_t *__restrict__ conn,
                                                   const T *__restrict__ coef,
                                                   const uint8_t *__restrict__ mask,
                                                   const T *__restrict__ x, T *__restrict__ y,
                                                   const int *__restrict__ stop) {
  constexpr int DPN = phys_dpn(PH);
  if (stop && *stop) return;
  const int64_t e = int64_t(blockIdx.x) * kFB + threadIdx.x;
  if (e >= ne) return;
  int32_t nid[4];
  bool fixed[4];
  T X[3][4], u[DPN][4];
#pragma unroll
  for (int a = 0; a < 4; ++a) nid[a] = conn[a * ne + e];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    fixed[a] = MASKED && mask[nid[a]] != 0;
#pragma unroll
    for (int r = 0; r < 3; ++r) X[r][a] = xyz[r * nn + nid[a]];
#pragma unroll
    for (int j = 0; j < DPN; ++j) u[j][a] = fixed[a] ? T(0) : x[int64_t(nid[a]) * DPN + j];
  }
  T v[DPN][4];
  tet_element<T, PH>(X, u, coef[e], PH == 3 ? coef[ne + e] : T(0), v);
#pragma unroll
  for (int a = 0; a < 4; ++a)
    if (!fixed[a])
#pragma unroll
      for (int j = 0; j < DPN; ++j) gadd(&y[int64_t(nid[a]) * DPN + j], v[j][a]);
}

// diag: Laplace k |c_a|^2 / (6 det J); elasticity ((lambda + mu) c_ai^2 + mu |c_a|^2) / (6 det J)
template <typename T, int PH, bool MASKED>
__global__ __launch_bounds__(kFB) void k_tet_diag(int64_t ne, int64_t nn,
                                                  const T *__restrict__ xyz,
                                                  const int32_t *__restrict__ conn,
                                                  const T *__restrict__ coef,
                                                  const uint8_t *__restrict__ mask,
                                                  T *__restrict__ d) {
  constexpr int DPN = phys_dpn(PH);
  const int64_t e = int64_t(blockIdx.x) * kFB + threadIdx.x;
  if (e >= ne) return;
  int32_t nid[4];
  T X[3][4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    nid[a] = conn[a * ne + e];
#pragma unroll
    for (int r = 0; r < 3; ++r) X[r][a] = xyz[r * nn + nid[a]];
  }
  const TetGeom<T> G = tet_geom(X);
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    if (MASKED && mask[nid[a]]) continue;
    const T cc = dot3(G.c[a], G.c[a]);
    if constexpr (PH == 1) {
      gadd(&d[nid[a]], coef[e] * G.s * cc);
    } else {
      const T lam = coef[e], mu = coef[ne + e];
#pragma unroll
      for (int i = 0; i < 3; ++i)
        gadd(&d[int64_t(nid[a]) * 3 + i], G.s * ((lam + mu) * G.c[a][i] * G.c[a][i] + mu * cc));
    }
  }
}

// ---- triquadratic and tricubic hexahedra ------------------------------------
//
// Order P = 2 (27 nodes) or 3 (64 nodes): nodes at t_m = -1 + 2m/P per
// direction, local node a = i + (P+1) j + (P+1)^2 k, P+1 Gauss points per
// direction.  In the diagonal's kernel a block holds 256 / (P+1)^3 elements, thread r
// of an element staging node r and then evaluating quadrature point r.

template <int P>
struct QP {
  static constexpr int N = P + 1;          // nodes (and Gauss points) per direction
  static constexpr int NPTS = N * N * N;   // nodes (and points) per element
  static constexpr int E = 256 / NPTS;     // elements per block
};

// The apply's lanes and LDS areas: N^2 lanes per element, EW elements per wavefront,
// LS lanes between neighbouring elements; entry (x, y, z) of element le at
// x + A y + B z + S le, in an array of pairs and one of single values.  The strides are the best of a search under the bank
// rules that the conflict counters fit: 16-byte accesses take lanes {0-3, 12-15, 20-23,
// 24-27}, {4-11, 16-19, 28-31} and the same of the upper half, four passes over 256 B;
// 8-byte ones 16 lanes at a time over 128 B.  Dense arrays (A = N, B = N^2, S = 3 N^3, no
// pairs) kept the LDS busy 2.7 times as long as without conflicts.
template <int P>
struct QL;
template <>
struct QL<2> {
  static constexpr int EW = 7, LS = 1, A = 6, B = 19, S = 55;
  static __device__ __forceinline__ int elem(int lane) { return lane % 7; }
  static __device__ __forceinline__ int line(int lane) { return min(lane / 7, 8); }  // 63: as 56
};
template <>
struct QL<3> {
  static constexpr int EW = 4, LS = 1, A = 5, B = 20, S = 92;
  static __device__ __forceinline__ int elem(int lane) { return lane & 3; }
  static __device__ __forceinline__ int line(int lane) { return lane >> 2; }
};
template <typename T>
struct alignas(2 * sizeof(T)) Two {
  T a, b;
};

// 1-D Lagrange basis of order P on [-1, 1] and its derivative (quadratic: the
// closed forms; cubic: the product formula over the other nodes)
template <typename T, int P>
__device__ __forceinline__ T lag(int i, T t) {
  if constexpr (P == 2) {
    return i == 0 ? T(0.5) * t * (t - T(1)) : i == 1 ? T(1) - t * t : T(0.5) * t * (t + T(1));
  } else {
    T v = T(1);
#pragma unroll
    for (int m = 0; m <= P; ++m)
      if (m != i) v *= (t - (T(-1) + T(2 * m) / T(P))) / (T(2 * (i - m)) / T(P));
    return v;
  }
}
template <typename T, int P>
__device__ __forceinline__ T dlag(int i, T t) {
  if constexpr (P == 2) {
    return i == 0 ? t - T(0.5) : i == 1 ? T(-2) * t : t + T(0.5);
  } else {
    T d = T(0);
#pragma unroll
    for (int l = 0; l <= P; ++l) {
      if (l == i) continue;
      T v = T(1) / (T(2 * (i - l)) / T(P));
#pragma unroll
      for (int m = 0; m <= P; ++m)
        if (m != i && m != l) v *= (t - (T(-1) + T(2 * m) / T(P))) / (T(2 * (i - m)) / T(P));
      d += v;
    }
    return d;
  }
}
// Gauss-Legendre points and weights with P + 1 points
template <typename T, int P>
__device__ __forceinline__ T gpt(int q) {
  if constexpr (P == 2) {
    return q == 0 ? -T(0.77459666924148337703585307995648)
                  : q == 1 ? T(0) : T(0.77459666924148337703585307995648);
  } else {  // +-sqrt(3/7 +- (2/7) sqrt(6/5))
    const T a = T(0.33998104358485626480266575910324), b = T(0.86113631159405257522394648889281);
    return q == 0 ? -b : q == 1 ? -a : q == 2 ? a : b;
  }
}
template <typename T, int P>
__device__ __forceinline__ T gwt(int q) {
  if constexpr (P == 2) {
    return q == 1 ? T(8) / T(9) : T(5) / T(9);
  } else {  // (18 +- sqrt(30)) / 36
    const T wa = T(0.65214515486254614262693605077800), wb = T(0.34785484513745385737306394922200);
    return q == 0 || q == 3 ? wb : wa;
  }
}

// The per-thread 1-D tables: basis and derivative of the functions at one
// point (phase 2), or of one function at the points (phase 3).
template <typename T, int P>
struct Tab1 {
  T b[P + 1], d[P + 1];
};
template <typename T, int P>
__device__ __forceinline__ Tab1<T, P> at_point(int q) {
  Tab1<T, P> t;
  const T p = gpt<T, P>(q);
#pragma unroll
  for (int i = 0; i <= P; ++i) {
    t.b[i] = lag<T, P>(i, p);
    t.d[i] = dlag<T, P>(i, p);
  }
  return t;
}
template <typename T, int P>
__device__ __forceinline__ Tab1<T, P> of_function(int i) {
  Tab1<T, P> t;
#pragma unroll
  for (int q = 0; q <= P; ++q) {
    t.b[q] = lag<T, P>(i, gpt<T, P>(q));
    t.d[q] = dlag<T, P>(i, gpt<T, P>(q));
  }
  return t;
}

// Phase 2 at quadrature point r of a staged element: the Jacobian's
// adjugate rows A (A[0] = j1 x j2, A[1] = j2 x j0, A[2] = j0 x j1), det J, and
// the reference gradients G of NF staged fields.
template <typename T, int P, int NF>
__device__ __forceinline__ T qp_point(int r, const T (*sX)[QP<P>::NPTS],
                                      const T (*sU)[QP<P>::NPTS], T A[3][3], T G[NF][3]) {
  constexpr int N = QP<P>::N, NPTS = QP<P>::NPTS;
  const Tab1<T, P> tx = at_point<T, P>(r % N), ty = at_point<T, P>((r / N) % N),
                   tz = at_point<T, P>(r / (N * N));
  T J[3][3];
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int d = 0; d < 3; ++d) J[c][d] = T(0);
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int d = 0; d < 3; ++d) G[f][d] = T(0);
#pragma unroll
  for (int a = 0; a < NPTS; ++a) {
    const int i = a % N, j = (a / N) % N, k = a / (N * N);
    const T d0 = tx.d[i] * ty.b[j] * tz.b[k];
    const T d1 = tx.b[i] * ty.d[j] * tz.b[k];
    const T d2 = tx.b[i] * ty.b[j] * tz.d[k];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const T xc = sX[c][a];
      J[c][0] += xc * d0;
      J[c][1] += xc * d1;
      J[c][2] += xc * d2;
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const T uf = sU[f][a];
      G[f][0] += uf * d0;
      G[f][1] += uf * d1;
      G[f][2] += uf * d2;
    }
  }
  const T j0[3] = {J[0][0], J[1][0], J[2][0]};
  const T j1[3] = {J[0][1], J[1][1], J[2][1]};
  const T j2[3] = {J[0][2], J[1][2], J[2][2]};
  cross(j1, j2, A[0]);
  cross(j2, j0, A[1]);
  cross(j0, j1, A[2]);
  return dot3(j0, A[0]);
}

// Sum-factorised apply of order P, N = P + 1: N^2 lanes per element, each holding a
// line of N values in registers, floor(64 / N^2) elements per wavefront (7 or 4).
// Per field (coordinate or input component), with B[q][i] = L_i(p_q), D[q][i] = L_i'(p_q):
//   A  lane (j, k), line in i:   S0 = B f, S1 = D f                    at (qx, j, k)
//   B  lane (qx, k), line in j:  S0 = B S0, S1 = B S1, S2 = D S0       at (qx, qy, k)
//   C  lane (qx, qy), line in k: g_xi = B S1, g_eta = B S2, g_zeta = D S0, kept in registers;
// then the flux at the lane's N points (as in the comment at the top of this file) and,
// per component, the transpose of C, B and A on it.  The lines turn through LDS, each
// value written and read once per pass, one field at a time in 3 N^3 values per element;
// an element's lanes lie in one wavefront, whose LDS instructions execute in order, so no
// workgroup barrier is needed.  Lines are evaluated by even and odd parts (the points and
// nodes are symmetric): 10 operations for B f and D f at the three points of order 2, not
// 18.  The last node of a line is added to the next element's first when the two lanes
// hold the same node id, which saves a third (order 2) or a quarter of the atomics.
// Coordinates are taken from the element's middle node (order 3: a node next to the middle),
// since the Jacobian is of differences only and pass A's values would round at the size of the
// coordinates: error of an FP64 apply against 80 bits, absolute coordinates -> here, order 2 on
// 9 x 8 x 7 elements 9.3e-16 -> 1.6e-16, order 3 on 4 x 5 x 4 2.5e-15 -> 2.2e-15 (6.6e-16 and
// 2.8e-15 with direct sums per point); FP32, order 2 on 33 x 29 x 41, 2.3e-6 -> 1.7e-7 (1.6e-6).
// Its cost is 1 to 3%.
//
// What bounds it: the LDS turns (busy 71% of the time at order 2 in FP64), then the
// gathers' cache accesses and FP64 issue.  FP64 Laplace, order 2 on 64^3 74 us, order 3 on
// 42^3 65 us; with an atomic per lane and node in place of the rows (2.4 sums to a request;
// the requests leave L2 for memory) 111 and 119 us; one thread per node and point, which
// read each line N times and met at workgroup barriers, 285 and 349 us.  Measured and
// dropped: box tiles on lattices with sums kept in LDS over a march in z (114 us at order
// 2: their barriers and accumulator traffic cost what the gathers and atomics saved).

// Values and derivatives of the interpolant of f at the N points.
template <typename T, int P>
struct Line {
  static constexpr int N = P + 1, H = N / 2;  // H pairs of nodes (and points); order 2: a centre
  // coefficient of the even (s = +1) or odd part of node pair n at the positive point q
  static __device__ __forceinline__ T b(int q, int n, int s) {
    return T(0.5) * (lag<T, P>(N - 1 - n, gpt<T, P>(N - 1 - q)) +
                     T(s) * lag<T, P>(n, gpt<T, P>(N - 1 - q)));
  }
  static __device__ __forceinline__ T d(int q, int n, int s) {
    return T(0.5) * (dlag<T, P>(N - 1 - n, gpt<T, P>(N - 1 - q)) +
                     T(s) * dlag<T, P>(n, gpt<T, P>(N - 1 - q)));
  }
  template <bool VB, bool VD>
  static __device__ __forceinline__ void eval(const T (&f)[N], T (&B)[N], T (&D)[N]) {
    T e[H], o[H];
#pragma unroll
    for (int n = 0; n < H; ++n) {
      e[n] = f[n] + f[N - 1 - n];
      o[n] = f[N - 1 - n] - f[n];
    }
#pragma unroll
    for (int q = 0; q < H; ++q) {
      if constexpr (VB) {
        T E = b(q, 0, 1) * e[0], O = b(q, 0, -1) * o[0];
#pragma unroll
        for (int n = 1; n < H; ++n) {
          E += b(q, n, 1) * e[n];
          O += b(q, n, -1) * o[n];
        }
        if constexpr (N % 2) E += lag<T, P>(H, gpt<T, P>(N - 1 - q)) * f[H];
        B[q] = E - O;
        B[N - 1 - q] = E + O;
      }
      if constexpr (VD) {  // the derivative's even part comes from the odd node sums
        T E = d(q, 0, -1) * o[0], O = d(q, 0, 1) * e[0];
#pragma unroll
        for (int n = 1; n < H; ++n) {
          E += d(q, n, -1) * o[n];
          O += d(q, n, 1) * e[n];
        }
        if constexpr (N % 2) O += dlag<T, P>(H, gpt<T, P>(N - 1 - q)) * f[H];
        D[q] = E - O;
        D[N - 1 - q] = E + O;
      }
    }
    if constexpr (N % 2) {  // the centre point is the centre node
      if constexpr (VB) B[H] = f[H];
      if constexpr (VD) D[H] = dlag<T, P>(N - 1, T(0)) * o[0];
    }
  }
  // v (+)= B^T a or D^T a
  template <bool DERIV, bool ADD>
  static __device__ __forceinline__ void transp(const T (&a)[N], T (&v)[N]) {
    T e[H], o[H];
#pragma unroll
    for (int q = 0; q < H; ++q) {
      e[q] = a[q] + a[N - 1 - q];
      o[q] = a[N - 1 - q] - a[q];
    }
#pragma unroll
    for (int n = 0; n < H; ++n) {
      T E, O;  // node N-1-n gets E + O, node n gets E - O (values), O + E, O - E (derivatives)
      if constexpr (!DERIV) {
        E = b(0, n, 1) * e[0];
        O = b(0, n, -1) * o[0];
      } else {
        E = d(0, n, 1) * o[0];
        O = d(0, n, -1) * e[0];
      }
#pragma unroll
      for (int q = 1; q < H; ++q) {
        E += (DERIV ? d(q, n, 1) * o[q] : b(q, n, 1) * e[q]);
        O += (DERIV ? d(q, n, -1) * e[q] : b(q, n, -1) * o[q]);
      }
      if constexpr (N % 2 && DERIV) O += dlag<T, P>(N - 1, T(0)) * a[H];
      if constexpr (ADD) {
        v[n] += E - O;
        v[N - 1 - n] += E + O;
      } else {
        v[n] = E - O;
        v[N - 1 - n] = E + O;
      }
    }
    if constexpr (N % 2) {
      T c = DERIV ? dlag<T, P>(H, gpt<T, P>(N - 1)) * o[0]
                  : lag<T, P>(H, gpt<T, P>(N - 1)) * e[0] + a[H];
      if constexpr (ADD) c += v[H];
      v[H] = c;
    }
  }
};

// order of this wavefront's LDS instructions, for the compiler (no instruction)
__device__ __forceinline__ void lds_turn() { asm volatile("" ::: "memory"); }

template <typename T, int PH, bool MASKED, int P>
__global__ __launch_bounds__(kFB) void k_qp_apply(int64_t ne, int64_t nn,
                                                  const T *__restrict__ xyz,
                                                  const int32_t *__restrict__ conn,
                                                  const T *__restrict__ coef,
                                                  const uint8_t *__restrict__ mask,
                                                  const T *__restrict__ x, T *__restrict__ y,
                                                  const int *__restrict__ stop) {
  constexpr int DPN = phys_dpn(PH), N = P + 1, L = N * N;
  using Q = QL<P>;
  using Ln = Line<T, P>;
  if (stop && *stop) return;
  // Fields at a time.  Small meshes leave a SIMD one wave, whose time is its chain of LDS
  // turns; two fields share each turn's latency: order 3, FP64 elasticity, 4 x 5 x 6 elements
  // 11.6 -> 10.8 us (11.1 with one thread per node and point; the two launches take 10.3), 13 x
  // 15 x 17 14.1 -> 13.8, 21 x 20 x 19 20.9 -> 21.1.  Registers allow two waves per SIMD there,
  // and two areas of LDS as well; order 2 would lose the third.
  constexpr int F = P == 3 && DPN == 3 ? 2 : 1;
  constexpr int NP = Q::EW * Q::S, FS = NP + (NP + 1) / 2;
  __shared__ Two<T> area[kFB / 64][F * FS];  // per field: pairs, then single values
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  Two<T> *pairs = area[w];
  T *singles = reinterpret_cast<T *>(pairs + NP);
  // lanes past the last whole element repeat another's work (the same values to the same places)
  const int le = Q::elem(lane), r = Q::line(lane);
  // each XCD takes a contiguous range of the elements: the nodes that neighbours share
  // are gathered and added to through one L2
  const unsigned blk = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int64_t ew = (int64_t(blk) * (kFB / 64) + w) * Q::EW + le;
  const bool active = lane < Q::EW * L && ew < ne;
  const int64_t e = ew < ne ? ew : ne - 1;
  const int ra = r % N, rb = r / N;
  // the lane's lines: in x at (ra, rb) = (y, z), in y at (x, z), in z at (x, y)
  Two<T> *px = pairs + Q::S * le + Q::A * ra + Q::B * rb;
  Two<T> *py = pairs + Q::S * le + ra + Q::B * rb, *pz = pairs + Q::S * le + ra + Q::A * rb;
  T *sy = singles + (py - pairs), *sz = singles + (pz - pairs);
  int32_t nid[N];
  bool fixed[N];
  T f[3 + DPN][N];
#pragma unroll
  for (int i = 0; i < N; ++i) nid[i] = conn[(i + int64_t(N) * r) * ne + e];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    fixed[i] = MASKED && mask[nid[i]] != 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) f[c][i] = xyz[c * nn + nid[i]];
#pragma unroll
    for (int j = 0; j < DPN; ++j) f[3 + j][i] = x[int64_t(nid[i]) * DPN + j];
    if (MASKED && fixed[i])
#pragma unroll
      for (int j = 0; j < DPN; ++j) f[3 + j][i] = T(0);
  }
  const T c0 = coef[e], c1 = PH == 3 ? coef[ne + e] : T(0);

  T G[3 + DPN][3][N];  // reference gradients at the lane's points (ra, rb, 0..N-1)
#pragma unroll
  for (int m = 0; m < 3 + DPN; m += F) {
    T B[F][N], D[F][N], U[N], a[F][N], b[F][N], c[F][N];
#pragma unroll
    for (int h = 0; h < F; ++h) {
      if (m + h < 3) {  // from the element's middle node, which line (1, 1) holds
        const T o = __shfl(f[m + h][1], (N + 1) * Q::EW + le);
#pragma unroll
        for (int i = 0; i < N; ++i) f[m + h][i] -= o;
      }
      Ln::template eval<true, true>(f[m + h], B[h], D[h]);
#pragma unroll
      for (int q = 0; q < N; ++q) px[h * FS + q] = {B[h][q], D[h][q]};
    }
    lds_turn();
#pragma unroll
    for (int h = 0; h < F; ++h)
#pragma unroll
      for (int q = 0; q < N; ++q) {
        const Two<T> t = py[h * FS + Q::A * q];
        a[h][q] = t.a;
        b[h][q] = t.b;
      }
    lds_turn();
#pragma unroll
    for (int h = 0; h < F; ++h) {
      Ln::template eval<true, true>(a[h], B[h], D[h]);
      Ln::template eval<true, false>(b[h], U, U);
#pragma unroll
      for (int q = 0; q < N; ++q) {
        py[h * FS + Q::A * q] = {U[q], D[h][q]};
        sy[2 * h * FS + Q::A * q] = B[h][q];
      }
    }
    lds_turn();
#pragma unroll
    for (int h = 0; h < F; ++h)
#pragma unroll
      for (int q = 0; q < N; ++q) {
        const Two<T> t = pz[h * FS + Q::B * q];
        a[h][q] = t.a;
        b[h][q] = t.b;
        c[h][q] = sz[2 * h * FS + Q::B * q];
      }
    lds_turn();
#pragma unroll
    for (int h = 0; h < F; ++h) {
      Ln::template eval<true, false>(a[h], G[m + h][0], G[m + h][0]);
      Ln::template eval<true, false>(b[h], G[m + h][1], G[m + h][1]);
      Ln::template eval<false, true>(c[h], G[m + h][2], G[m + h][2]);
    }
  }
  // the flux of component c and direction d, in place of the input's gradients
  const T wxy = gwt<T, P>(ra) * gwt<T, P>(rb);
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const T j0[3] = {G[0][0][q], G[1][0][q], G[2][0][q]};
    const T j1[3] = {G[0][1][q], G[1][1][q], G[2][1][q]};
    const T j2[3] = {G[0][2][q], G[1][2][q], G[2][2][q]};
    T A[3][3];
    cross(j1, j2, A[0]);
    cross(j2, j0, A[1]);
    cross(j0, j1, A[2]);
    const T s = wxy * gwt<T, P>(q) * rcp(dot3(j0, A[0]));
    if constexpr (PH == 1) {
      T p[3];  // det J times the physical gradient
#pragma unroll
      for (int m = 0; m < 3; ++m)
        p[m] = G[3][0][q] * A[0][m] + G[3][1][q] * A[1][m] + G[3][2][q] * A[2][m];
      const T ks = c0 * s;
#pragma unroll
      for (int d = 0; d < 3; ++d) G[3][d][q] = ks * dot3(A[d], p);
    } else {
      T H[3][3];  // det J times the displacement gradient
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
          H[i][j] = G[3 + i][0][q] * A[0][j] + G[3 + i][1][q] * A[1][j] + G[3 + i][2][q] * A[2][j];
      const T ltr = c0 * (H[0][0] + H[1][1] + H[2][2]);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        T Si[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) Si[j] = c1 * (H[i][j] + H[j][i]) + (i == j ? ltr : T(0));
#pragma unroll
        for (int d = 0; d < 3; ++d) G[3 + i][d][q] = s * dot3(Si, A[d]);
      }
    }
  }
  T v[DPN][N];
#pragma unroll
  for (int m = 0; m < DPN; m += F) {
    T a[F][N], b[F][N], c[F][N], u0[N], u1[N];
#pragma unroll
    for (int h = 0; h < F && m + h < DPN; ++h) {
      Ln::template transp<false, false>(G[3 + m + h][0], a[h]);
      Ln::template transp<false, false>(G[3 + m + h][1], b[h]);
      Ln::template transp<true, false>(G[3 + m + h][2], c[h]);
#pragma unroll
      for (int q = 0; q < N; ++q) {
        pz[h * FS + Q::B * q] = {a[h][q], b[h][q]};
        sz[2 * h * FS + Q::B * q] = c[h][q];
      }
    }
    lds_turn();
#pragma unroll
    for (int h = 0; h < F && m + h < DPN; ++h)
#pragma unroll
      for (int q = 0; q < N; ++q) {
        const Two<T> t = py[h * FS + Q::A * q];
        a[h][q] = t.a;
        b[h][q] = t.b;
        c[h][q] = sy[2 * h * FS + Q::A * q];
      }
    lds_turn();
#pragma unroll
    for (int h = 0; h < F && m + h < DPN; ++h) {
      Ln::template transp<false, false>(a[h], u0);
      Ln::template transp<true, false>(b[h], u1);
      Ln::template transp<false, true>(c[h], u1);
#pragma unroll
      for (int q = 0; q < N; ++q) py[h * FS + Q::A * q] = {u0[q], u1[q]};
    }
    lds_turn();
#pragma unroll
    for (int h = 0; h < F && m + h < DPN; ++h)
#pragma unroll
      for (int q = 0; q < N; ++q) {
        const Two<T> t = px[h * FS + q];
        a[h][q] = t.a;
        b[h][q] = t.b;
      }
    lds_turn();
#pragma unroll
    for (int h = 0; h < F && m + h < DPN; ++h) {
      Ln::template transp<true, false>(a[h], v[m + h]);
      Ln::template transp<false, true>(b[h], v[m + h]);
    }
  }
  // the line's last node goes to the next element's lane when that starts with it
  const int32_t next = __shfl(nid[0], (lane + Q::LS) & 63);
  const bool give = active && le + 1 < Q::EW && ew + 1 < ne && next == nid[P];
  const bool take = __shfl(int(give), (lane - Q::LS) & 63) && active && le > 0;
#pragma unroll
  for (int m = 0; m < DPN; ++m) {
    const T in = __shfl(v[m][P], (lane - Q::LS) & 63);
    if (take) v[m][0] += in;
  }
  // The sums go out in the order of the rows (line, element, node), through LDS: where ids
  // run along x, consecutive lanes add to consecutive addresses, and a 64-byte atomic
  // request carries several of them instead of two or three.
  constexpr int ENT = Q::EW * L * N;  // entries of the wavefront
  static_assert(sizeof(area[0]) >= ENT * (DPN * sizeof(T) + sizeof(int32_t)), "sums and ids fit");
  T *out = reinterpret_cast<T *>(pairs);
  int32_t *ids = reinterpret_cast<int32_t *>(out + ENT * DPN);
  const int at = (r * Q::EW + le) * N;
  lds_turn();
  if (lane < Q::EW * L)
#pragma unroll
    for (int i = 0; i < N; ++i) {
#pragma unroll
      for (int m = 0; m < DPN; ++m) out[(at + i) * DPN + m] = v[m][i];
      ids[at + i] = active && !fixed[i] && !(i == P && give) ? nid[i] : -1;
    }
  lds_turn();
  // (all LDS reads before the first addition: under its branch each waited for the one before)
  constexpr int K = (ENT * DPN + 63) / 64;
  int32_t n[K];
  T sum[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int j = min(k * 64 + lane, ENT * DPN - 1);
    n[k] = ids[j / DPN];
    sum[k] = out[j];
  }
  lds_turn();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int j = k * 64 + lane;
    if (j < ENT * DPN && n[k] >= 0) gadd(&y[int64_t(n[k]) * DPN + j % DPN], sum[k]);
  }
}

// diag: Laplace sum_q k w |t|^2 / det J, elasticity
// sum_q w ((lambda + mu) t_i^2 + mu |t|^2) / det J, with t = sum_c dphi_c A[c]
// (det J times the physical gradient of the node's basis function)
template <typename T, int PH, bool MASKED, int P>
__global__ __launch_bounds__(kFB) void k_qp_diag(int64_t ne, int64_t nn,
                                                 const T *__restrict__ xyz,
                                                 const int32_t *__restrict__ conn,
                                                 const T *__restrict__ coef,
                                                 const uint8_t *__restrict__ mask,
                                                 T *__restrict__ dg) {
  constexpr int DPN = phys_dpn(PH);
  constexpr int N = QP<P>::N, NPTS = QP<P>::NPTS, E = QP<P>::E;
  __shared__ T sX[E][3][NPTS];
  __shared__ T sA[E][10][NPTS];  // adjugate rows and w / det J per point
  const int le = int(threadIdx.x) / NPTS, r = int(threadIdx.x) - NPTS * le;
  const int64_t e = int64_t(blockIdx.x) * E + le;
  const bool active = le < E && e < ne;
  int64_t g = 0;
  bool fixed = true;
  if (active) {
    g = conn[int64_t(r) * ne + e];
    fixed = MASKED && mask[g] != 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) sX[le][c][r] = xyz[c * nn + g];
  }
  __syncthreads();
  if (active) {
    T A[3][3], G[1][3];  // (the coordinate field stands in for the unused input)
    const T det = qp_point<T, P, 1>(r, sX[le], sX[le], A, G);
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int m = 0; m < 3; ++m) sA[le][3 * c + m][r] = A[c][m];
    sA[le][9][r] = gwt<T, P>(r % N) * gwt<T, P>((r / N) % N) * gwt<T, P>(r / (N * N)) * rcp(det);
  }
  __syncthreads();
  if (active && !fixed) {
    const Tab1<T, P> fx = of_function<T, P>(r % N), fy = of_function<T, P>((r / N) % N),
                     fz = of_function<T, P>(r / (N * N));
    T acc[DPN];
#pragma unroll
    for (int j = 0; j < DPN; ++j) acc[j] = T(0);
    const T c0 = coef[e], c1 = PH == 3 ? coef[ne + e] : T(0);
#pragma unroll
    for (int q = 0; q < NPTS; ++q) {
      const int qx = q % N, qy = (q / N) % N, qz = q / (N * N);
      const T d0 = fx.d[qx] * fy.b[qy] * fz.b[qz];
      const T d1 = fx.b[qx] * fy.d[qy] * fz.b[qz];
      const T d2 = fx.b[qx] * fy.b[qy] * fz.d[qz];
      T t[3];
#pragma unroll
      for (int m = 0; m < 3; ++m)
        t[m] = d0 * sA[le][m][q] + d1 * sA[le][3 + m][q] + d2 * sA[le][6 + m][q];
      const T tt = dot3(t, t), s = sA[le][9][q];
      if constexpr (PH == 1) {
        acc[0] += c0 * s * tt;
      } else {
#pragma unroll
        for (int i = 0; i < 3; ++i) acc[i] += s * ((c0 + c1) * t[i] * t[i] + c1 * tt);
      }
    }
#pragma unroll
    for (int j = 0; j < DPN; ++j) gadd(&dg[g * DPN + j], acc[j]);
  }
}

template <typename T, int PH>
int family_apply_t(Op &op, const void *xv, void *yv, hipStream_t s, const int *stop) {
  constexpr int DPN = phys_dpn(PH);
  const T *x = static_cast<const T *>(xv);
  T *y = static_cast<T *>(yv);
  const int64_t ndof = op.n_nodes * DPN;
  hipLaunchKernelGGL((k_fam_init<T, DPN>), dim3(unsigned((ndof + kFB - 1) / kFB)), dim3(kFB), 0,
                     s, op.n_nodes, op.mask, x, y, stop);
  if (op.n_elems > 0) {
    const T *xyz = static_cast<const T *>(op.xyz), *coef = static_cast<const T *>(op.coef);
    const bool m = op.mask != nullptr;
    if (op.elem == Q1_TET4) {
      const dim3 grid(unsigned((op.n_elems + kFB - 1) / kFB));
      hipLaunchKernelGGL((m ? k_tet_apply<T, PH, true> : k_tet_apply<T, PH, false>), grid,
                         dim3(kFB), 0, s, op.n_elems, op.n_nodes, xyz, op.conn, coef, op.mask,
                         x, y, stop);
    } else {
      auto run = [&](auto pc) {
        constexpr int P = decltype(pc)::value, EB = kFB / 64 * QL<P>::EW;
        const dim3 grid(unsigned(((op.n_elems + EB - 1) / EB + 7) / 8 * 8));
        hipLaunchKernelGGL((m ? k_qp_apply<T, PH, true, P> : k_qp_apply<T, PH, false, P>), grid,
                           dim3(kFB), 0, s, op.n_elems, op.n_nodes, xyz, op.conn, coef, op.mask,
                           x, y, stop);
      };
      if (op.elem == Q1_HEX27)
        run(std::integral_constant<int, 2>{});
      else
        run(std::integral_constant<int, 3>{});
    }
  }
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

template <typename T, int PH>
int family_diag_t(Op &op, void *dv, hipStream_t s) {
  constexpr int DPN = phys_dpn(PH);
  T *d = static_cast<T *>(dv);
  const int64_t ndof = op.n_nodes * DPN;
  hipLaunchKernelGGL((k_fam_init<T, DPN>), dim3(unsigned((ndof + kFB - 1) / kFB)), dim3(kFB), 0,
                     s, op.n_nodes, op.mask, static_cast<const T *>(nullptr), d,
                     static_cast<const int *>(nullptr));
  if (op.n_elems > 0) {
    const T *xyz = static_cast<const T *>(op.xyz), *coef = static_cast<const T *>(op.coef);
    const bool m = op.mask != nullptr;
    if (op.elem == Q1_TET4) {
      const dim3 grid(unsigned((op.n_elems + kFB - 1) / kFB));
      hipLaunchKernelGGL((m ? k_tet_diag<T, PH, true> : k_tet_diag<T, PH, false>), grid,
                         dim3(kFB), 0, s, op.n_elems, op.n_nodes, xyz, op.conn, coef, op.mask, d);
    } else if (op.elem == Q1_HEX27) {
      const dim3 grid(unsigned((op.n_elems + QP<2>::E - 1) / QP<2>::E));
      hipLaunchKernelGGL((m ? k_qp_diag<T, PH, true, 2> : k_qp_diag<T, PH, false, 2>), grid,
                         dim3(kFB), 0, s, op.n_elems, op.n_nodes, xyz, op.conn, coef, op.mask, d);
    } else {
      const dim3 grid(unsigned((op.n_elems + QP<3>::E - 1) / QP<3>::E));
      hipLaunchKernelGGL((m ? k_qp_diag<T, PH, true, 3> : k_qp_diag<T, PH, false, 3>), grid,
                         dim3(kFB), 0, s, op.n_elems, op.n_nodes, xyz, op.conn, coef, op.mask, d);
    }
  }
  Q1_HIP(hipGetLastError());
  return Q1_OK;
}

}  // namespace

int launch_apply_family(Op &op, const void *x, void *y, hipStream_t s, const int *stop) {
  if (op.variant == Q1_V_BLOCK) return launch_apply_tile(op, x, y, s, stop);  // tetrahedra
  const bool f64 = op.dtype == Q1_F64;
  if (op.physics == Q1_LAPLACE)
    return f64 ? family_apply_t<double, 1>(op, x, y, s, stop)
               : family_apply_t<float, 1>(op, x, y, s, stop);
  if (op.physics == Q1_ELASTICITY)
    return f64 ? family_apply_t<double, 3>(op, x, y, s, stop)
               : family_apply_t<float, 3>(op, x, y, s, stop);
  return fail(Q1_EUNSUPPORTED, "element family %d: physics %d", op.elem, op.physics);
}

int launch_diag_family(Op &op, void *d, hipStream_t s) {
  const bool f64 = op.dtype == Q1_F64;
  if (op.physics == Q1_LAPLACE)
    return f64 ? family_diag_t<double, 1>(op, d, s) : family_diag_t<float, 1>(op, d, s);
  if (op.physics == Q1_ELASTICITY)
    return f64 ? family_diag_t<double, 3>(op, d, s) : family_diag_t<float, 3>(op, d, s);
  return fail(Q1_EUNSUPPORTED, "element family %d: physics %d", op.elem, op.physics);
}

}  // namespace q1
