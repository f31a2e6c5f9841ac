// Fused element kernels of the matrix-free Neo-Hookean operator for gfx950.
//
// One workgroup processes one tile of ET consecutive elements with one thread per
// quadrature point (Q^3 per element).  Inside a kernel the element vector and the
// quadrature vector never leave the chip (Fig. libceedapi caption: E, B and D fused):
//
//   gather (E)  ->  sum-factorised interpolation, three 1D contractions staged in LDS
//   ->  collocated derivative B_xi B_I^+ (three more contractions, Section II-B)
//   ->  pointwise constitutive map in registers (Section II-A)
//   ->  transposed derivative and interpolation in LDS  ->  element records, summed per
//       node in a fixed order by a node-centric assembly pass (E^T, no atomics).
//
// Quadrature-point data are read/written as [tile][field][field_stride(Q)] so each field of a
// tile is one contiguous, coalesced sweep.  Dirichlet flags ride in the top bits of the
// element-to-node map, so masking costs no extra memory traffic.
#include <cmath>
#include <cstdlib>
#include <string>
#include <type_traits>

#include "common.h"

namespace hpmg {
namespace {

template <int Q>
struct QT {
  static constexpr int Q3 = Q * Q * Q;
  static constexpr int ET = elems_per_tile(Q);
  static constexpr int NQ = field_stride(Q);
  static constexpr int NT = tile_threads(Q);
};

// One 1D contraction along direction DIR of an array with dims (N1, N2, N3), N1
// fastest, for NC components stored back to back.  Output dims replace N_DIR by NO.
// TR = false: out_o = sum_i M[o][i] in_i (M is [NO][NI]);
// TR = true:  out_o = sum_i M[i][o] in_i (M is [NI][NO], the transpose is applied).
template <typename T, int N1, int N2, int N3, int DIR, int NO, bool TR, int NC>
__device__ __forceinline__ void stage(const T *__restrict__ in, T *__restrict__ out,
                                      const T *__restrict__ M, int q, bool live) {
  constexpr int NI = DIR == 0 ? N1 : DIR == 1 ? N2 : N3;
  constexpr int O1 = DIR == 0 ? NO : N1, O2 = DIR == 1 ? NO : N2, O3 = DIR == 2 ? NO : N3;
  constexpr int NIN = N1 * N2 * N3, NOUT = O1 * O2 * O3;
  constexpr int STR = DIR == 0 ? 1 : DIR == 1 ? N1 : N1 * N2;
  if (live && q < NOUT) {
    const int o1 = q % O1, o2 = (q / O1) % O2, o3 = q / (O1 * O2);
    const int o = DIR == 0 ? o1 : DIR == 1 ? o2 : o3;
    const int base = (DIR == 0 ? 0 : o1) + N1 * ((DIR == 1 ? 0 : o2) + N2 * (DIR == 2 ? 0 : o3));
    T m[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) m[i] = TR ? M[i * NO + o] : M[o * NI + i];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      T acc = 0;
#pragma unroll
      for (int i = 0; i < NI; ++i) acc += m[i] * in[c * NIN + base + i * STR];
      out[c * NOUT + q] = acc;
    }
  }
}

// Nodes [NC][P^3] in `a` -> quadrature values [NC][Q^3] in `b` (a is overwritten).
template <typename T, int P, int Q, int NC>
__device__ __forceinline__ void interp(T *a, T *b, const T *sB, int q, bool live) {
  stage<T, P, P, P, 0, Q, false, NC>(a, b, sB, q, live);
  __syncthreads();
  stage<T, Q, P, P, 1, Q, false, NC>(b, a, sB, q, live);
  __syncthreads();
  stage<T, Q, Q, P, 2, Q, false, NC>(a, b, sB, q, live);
  __syncthreads();
}

// Quadrature values [NC][Q^3] in `b` -> nodes [NC][P^3] in `a` (transpose of interp).
template <typename T, int P, int Q, int NC>
__device__ __forceinline__ void interp_t(T *b, T *a, const T *sB, int q, bool live) {
  stage<T, Q, Q, Q, 2, P, true, NC>(b, a, sB, q, live);
  __syncthreads();
  stage<T, Q, Q, P, 1, P, true, NC>(a, b, sB, q, live);
  __syncthreads();
  stage<T, Q, P, P, 0, P, true, NC>(b, a, sB, q, live);
  __syncthreads();
}

// Reference gradient at quadrature point q from quadrature values (collocated
// derivative): G[c][k] = d(component c)/d xi_k.
//
// The empty asm statements pin each component's sums before the next component's LDS
// reads are issued.  Without them the scheduler hoists all 3 x 15 reads ahead of the
// first FMA, which costs ~50 extra VGPRs in FP64 and one wave per SIMD of occupancy.
template <typename T, int Q, int NC>
__device__ __forceinline__ void grad_q(const T *in, const T *sD, int q, T (&G)[NC][3]) {
  constexpr int Q3 = Q * Q * Q;
  const int q1 = q % Q, q2 = (q / Q) % Q, q3 = q / (Q * Q);
  T d1[Q], d2[Q], d3[Q];
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    d1[j] = sD[q1 * Q + j];
    d2[j] = sD[q2 * Q + j];
    d3[j] = sD[q3 * Q + j];
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    T g0 = 0, g1 = 0, g2 = 0;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      g0 += d1[j] * in[c * Q3 + j + Q * (q2 + Q * q3)];
      g1 += d2[j] * in[c * Q3 + q1 + Q * (j + Q * q3)];
      g2 += d3[j] * in[c * Q3 + q1 + Q * (q2 + Q * j)];
    }
    asm volatile("" : "+v"(g0), "+v"(g1), "+v"(g2)::"memory");
    G[c][0] = g0;
    G[c][1] = g1;
    G[c][2] = g2;
  }
}

template <typename T>
__device__ __forceinline__ T det3(const T (&m)[3][3]) {
  return m[0][0] * (m[1][1] * m[2][2] - m[1][2] * m[2][1]) -
         m[0][1] * (m[1][0] * m[2][2] - m[1][2] * m[2][0]) +
         m[0][2] * (m[1][0] * m[2][1] - m[1][1] * m[2][0]);
}

// adj(m) / det  (inverse), given det.
template <typename T>
__device__ __forceinline__ void inv3(const T (&m)[3][3], T det, T (&r)[3][3]) {
  const T id = T(1) / det;
  r[0][0] = (m[1][1] * m[2][2] - m[1][2] * m[2][1]) * id;
  r[0][1] = (m[0][2] * m[2][1] - m[0][1] * m[2][2]) * id;
  r[0][2] = (m[0][1] * m[1][2] - m[0][2] * m[1][1]) * id;
  r[1][0] = (m[1][2] * m[2][0] - m[1][0] * m[2][2]) * id;
  r[1][1] = (m[0][0] * m[2][2] - m[0][2] * m[2][0]) * id;
  r[1][2] = (m[0][2] * m[1][0] - m[0][0] * m[1][2]) * id;
  r[2][0] = (m[1][0] * m[2][1] - m[1][1] * m[2][0]) * id;
  r[2][1] = (m[0][1] * m[2][0] - m[0][0] * m[2][1]) * id;
  r[2][2] = (m[0][0] * m[1][1] - m[0][1] * m[1][0]) * id;
}

// Symmetric tau stored as (xx, yy, zz, yz, xz, xy).
__device__ __forceinline__ constexpr int sym_index(int i, int j) {
  return i == j ? i : (i + j == 1 ? 5 : (i + j == 2 ? 4 : 3));
}

// Kinematics and Kirchhoff stress from the reference gradient G = du/dxi and the
// inverse geometric Jacobian D = dxi/dX (Section II-A):
//   H = G D, J - 1 = tr H + ((tr H)^2 - tr H^2)/2 + det H (no cancellation),
//   log J = log1p(J - 1), tau = mu (H + H^T + H H^T) + lambda log J I,
//   A = dxi/dx = D F^{-1}.
// J - 1 and log J are always evaluated in double.
template <typename T>
struct Kin {
  T A[3][3];
  T tau[6];
  T c;       // lambda log J
  double logJ;
  double Jm1;
  T H[3][3];
};

template <typename T>
__device__ __forceinline__ void kinematics(const T (&G)[3][3], const T (&D)[3][3], T mu, T lam,
                                           Kin<T> &k) {
  for (int i = 0; i < 3; ++i)
    for (int J = 0; J < 3; ++J) k.H[i][J] = G[i][0] * D[0][J] + G[i][1] * D[1][J] + G[i][2] * D[2][J];
  double Hd[3][3];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) Hd[i][j] = (double)k.H[i][j];
  const double tr = Hd[0][0] + Hd[1][1] + Hd[2][2];
  double tr2 = 0.0;
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) tr2 += Hd[i][j] * Hd[j][i];
  k.Jm1 = tr + 0.5 * (tr * tr - tr2) + det3(Hd);
  k.logJ = log1p(k.Jm1);
  k.c = lam * (T)k.logJ;
  for (int i = 0; i < 3; ++i)
    for (int j = i; j < 3; ++j) {
      T b = k.H[i][0] * k.H[j][0] + k.H[i][1] * k.H[j][1] + k.H[i][2] * k.H[j][2];
      T t = mu * (k.H[i][j] + k.H[j][i] + b);
      if (i == j) t += k.c;
      k.tau[sym_index(i, j)] = t;
    }
  T F[3][3], Fi[3][3];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) F[i][j] = (i == j ? T(1) : T(0)) + k.H[i][j];
  inv3(F, (T)(1.0 + k.Jm1), Fi);
  for (int a = 0; a < 3; ++a)
    for (int j = 0; j < 3; ++j) k.A[a][j] = D[a][0] * Fi[0][j] + D[a][1] * Fi[1][j] + D[a][2] * Fi[2][j];
}

// Residual pointwise map: f[i][k] = W sum_j tau_ij A_kj  (W tau (dxi/dx)^T).
template <typename T>
__device__ __forceinline__ void residual_qf(const Kin<T> &k, T W, T (&f)[3][3]) {
  for (int i = 0; i < 3; ++i)
    for (int a = 0; a < 3; ++a) {
      T s = 0;
      for (int j = 0; j < 3; ++j) s += k.tau[sym_index(i, j)] * k.A[a][j];
      f[i][a] = W * s;
    }
}

__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// a + b where b may be a product: rounded before the sum.
template <typename T>
__device__ __forceinline__ T add_rounded(T a, T b) {
#pragma clang fp contract(off)
  return a + b;
}

// a0 b0 + a1 b1 + a2 b2 and c + a b, in FP64 with their roundings fixed: left to the
// compiler, which product becomes the plain one differs between instances of a kernel, and
// with it the last bit of an operator that the coarse solves amplify.
__device__ __forceinline__ double dot3(double a0, double b0, double a1, double b1, double a2, double b2) {
  return __builtin_fma(a2, b2, __builtin_fma(a0, b0, a1 * b1));
}
__device__ __forceinline__ float dot3(float a0, float b0, float a1, float b1, float a2, float b2) {
  return a0 * b0 + a1 * b1 + a2 * b2;
}
__device__ __forceinline__ double add_product(double c, double a, double b) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float add_product(float c, float a, float b) { return c + a * b; }

// Jacobian pointwise map (eqs. Jacobian, dtau, depsilon in current configuration):
//   g = G A = grad_x du;  s = g tau + lambda tr(g) I + (mu - lambda log J)(g + g^T);
//   f = W s A^T.
template <typename T>
__device__ __forceinline__ void jacobian_qf(const T (&G)[3][3], const T (&A)[3][3], const T (&tau)[6],
                                            T c, T W, T mu, T lam, T (&f)[3][3]) {
  T g[3][3];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) g[i][j] = dot3(G[i][0], A[0][j], G[i][1], A[1][j], G[i][2], A[2][j]);
  const T trg = g[0][0] + g[1][1] + g[2][2];
  const T m2 = mu - c;
  T s[3][3];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      T v = dot3(g[i][0], tau[sym_index(0, j)], g[i][1], tau[sym_index(1, j)], g[i][2], tau[sym_index(2, j)]);
      v = add_product(v, m2, g[i][j] + g[j][i]);
      if (i == j) v = add_product(v, lam, trg);
      s[i][j] = v;
    }
  for (int i = 0; i < 3; ++i)
    for (int a = 0; a < 3; ++a) f[i][a] = W * dot3(s[i][0], A[a][0], s[i][1], A[a][1], s[i][2], A[a][2]);
}

// Adjoint pointwise map, written as the transpose of jacobian_qf: for a cotangent
// C = dw/dxi, s*(M) = M tau^T + lambda tr(M) I + (mu - c)(M + M^T) with M = C A, and
// f = W s*(M) A^T.
template <typename T>
__device__ __forceinline__ void adjoint_qf(const T (&C)[3][3], const T (&A)[3][3], const T (&tau)[6],
                                           T c, T W, T mu, T lam, T (&f)[3][3], T (&M)[3][3]) {
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) M[i][j] = C[i][0] * A[0][j] + C[i][1] * A[1][j] + C[i][2] * A[2][j];
  const T trM = M[0][0] + M[1][1] + M[2][2];
  const T m2 = mu - c;
  T s[3][3];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      // (M tau^T)_ij = sum_m M_im tau_jm
      T v = M[i][0] * tau[sym_index(j, 0)] + M[i][1] * tau[sym_index(j, 1)] + M[i][2] * tau[sym_index(j, 2)];
      v += m2 * (M[i][j] + M[j][i]);
      if (i == j) v += lam * trM;
      s[i][j] = v;
    }
  for (int i = 0; i < 3; ++i)
    for (int a = 0; a < 3; ++a) f[i][a] = W * (s[i][0] * A[a][0] + s[i][1] * A[a][1] + s[i][2] * A[a][2]);
}

// Jacobian pointwise map in the initial configuration (the S(E) form of the same
// model, Section V / Table different-storage): with dF = G D = grad_X du,
//   S  = mu I + (c - mu) C^-1                     (c = lambda log J),
//   dC = dF^T F + F^T dF,
//   dS = (mu - c) C^-1 dC C^-1 + (lambda / 2) tr(C^-1 dC) C^-1,
//   dP = dF S + F dS,   f = W dP D^T.
// hv holds grad_X u (9, row-major) and, when TUNED, C^-1 (6, symmetric) and c; the
// "native" form recomputes C^-1 and c from grad_X u (J - 1 without cancellation).
template <bool TUNED>
__device__ __forceinline__ void jacobian_qf_initial(const double (&G)[3][3], const double (&gv)[NGEO],
                                                    const double *hv, double mu, double lam,
                                                    double (&f)[3][3]) {
  double D[3][3], H[3][3], dF[3][3], F[3][3], Ci[3][3];
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int J = 0; J < 3; ++J) {
      D[k][J] = gv[1 + k * 3 + J];
      H[k][J] = hv[k * 3 + J];
    }
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int J = 0; J < 3; ++J) {
      dF[i][J] = G[i][0] * D[0][J] + G[i][1] * D[1][J] + G[i][2] * D[2][J];
      F[i][J] = (i == J ? 1.0 : 0.0) + H[i][J];
    }
  double c;
  if (TUNED) {
#pragma unroll
    for (int I = 0; I < 3; ++I)
#pragma unroll
      for (int J = 0; J < 3; ++J) Ci[I][J] = hv[9 + sym_index(I, J)];
    c = hv[15];
  } else {
    const double tr = H[0][0] + H[1][1] + H[2][2];
    double tr2 = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) tr2 += H[i][j] * H[j][i];
    const double Jm1 = tr + 0.5 * (tr * tr - tr2) + det3(H);
    c = lam * log1p(Jm1);
    double Fi[3][3];
    inv3(F, 1.0 + Jm1, Fi);
#pragma unroll
    for (int I = 0; I < 3; ++I)
#pragma unroll
      for (int J = 0; J < 3; ++J) Ci[I][J] = Fi[I][0] * Fi[J][0] + Fi[I][1] * Fi[J][1] + Fi[I][2] * Fi[J][2];
  }
  double dC[3][3];
#pragma unroll
  for (int I = 0; I < 3; ++I)
#pragma unroll
    for (int J = 0; J < 3; ++J) {
      double v = 0.0;
#pragma unroll
      for (int a = 0; a < 3; ++a) v += dF[a][I] * F[a][J] + F[a][I] * dF[a][J];
      dC[I][J] = v;
    }
  double M[3][3], tr = 0.0;
#pragma unroll
  for (int I = 0; I < 3; ++I)
#pragma unroll
    for (int J = 0; J < 3; ++J) {
      M[I][J] = Ci[I][0] * dC[0][J] + Ci[I][1] * dC[1][J] + Ci[I][2] * dC[2][J];
      if (I == J) tr += M[I][J];
    }
  double dS[3][3], Sm[3][3];
#pragma unroll
  for (int I = 0; I < 3; ++I)
#pragma unroll
    for (int J = 0; J < 3; ++J) {
      const double e1 = M[I][0] * Ci[0][J] + M[I][1] * Ci[1][J] + M[I][2] * Ci[2][J];
      dS[I][J] = (mu - c) * e1 + 0.5 * lam * tr * Ci[I][J];
      Sm[I][J] = (I == J ? mu : 0.0) + (c - mu) * Ci[I][J];
    }
  double dP[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int J = 0; J < 3; ++J) {
      double v = 0.0;
#pragma unroll
      for (int K = 0; K < 3; ++K) v += dF[i][K] * Sm[K][J] + F[i][K] * dS[K][J];
      dP[i][J] = v;
    }
  const double W = gv[0];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int k = 0; k < 3; ++k) f[i][k] = W * (dP[i][0] * D[k][0] + dP[i][1] * D[k][1] + dP[i][2] * D[k][2]);
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2.  Give
// every XCD a contiguous range of tiles so neighbouring elements (which share nodes,
// hence gathered values) run under the same L2.
__device__ __forceinline__ int64_t xcd_tile() {
  constexpr unsigned NX = 8;
  const unsigned b = blockIdx.x, G = gridDim.x;
  const unsigned m = G / NX, r = G % NX, x = b % NX, j = b / NX;
  return (int64_t)x * m + (x < r ? x : r) + j;
}

// Record traffic of FP64 operators of order 4 and 2 (P = 5, 3) goes through contiguous
// sweeps: the Jacobian kernel writes each tile's records from LDS as one run, and the
// assembly writes its output from LDS in whole-line nontemporal sweeps.  Records of up
// to 160 MiB (keep_records) are stored with plain stores, so that they stay in the
// 256 MB last-level cache for the assembly that follows; larger ones stream out with
// nontemporal stores.  Measured, us an apply, plain / nontemporal record stores:
//                                     one operator repeated   four operators in turn
//   Q2 on 43^3 elements (52 MB)              77 / 85                 86 / 88
//   Q4 on 34^3 (118 MB)                     170 / 181               204 / 195
//   Q2 on 60^3 (140 MB)                     196 / 216               234 / 230
//   Q4 on 37^3 (152 MB)                     248 / 237               260 / 256
//   Q4 on 40^3 (192 MB)                     320 / 301               326 / 316
//   Q2 on 72^3 (242 MB)                     413 / 394               411 / 400
// The line is drawn for one operator, as in a Krylov solve, where it lies between 140 and 152
// MB; for operators in turn it lies between 52 and 118 MB.  An earlier form of the kernels with
// per-node stores: Q4 34^3 217 us against 188, Q2 43^3 88.4 against 87.2, Q2 86^3 785 against
// 724.  In FP32 the per-node stores were as fast or faster.
template <typename T>
__host__ __device__ constexpr bool sweep_records(int P) {
  return std::is_same<T, double>::value && (P == 5 || P == 3);
}
template <typename T>
bool keep_records(int64_t E, int P) {
  return (double)E * P * P * P * 3 * sizeof(T) <= 160.0 * (1 << 20);
}

// A residual's state of more than 240 MiB, which all but fills the 256 MiB last-level cache,
// streams out past it (MODE 8 of k_jacobian_lines); a smaller one goes there with plain
// stores, where the next pass finds it.  Plain stores of a state beyond the cache are bound
// by its write-back: residual alone 308 us on 34^3 Q4 elements (614 MiB) against 234
// streaming.  Measured, us, residual and a Jacobian action behind it, plain / streaming:
//                                one operator repeated   three in turn
//   Q4 on 20^3 (125 MiB)                91 / 97             102 / 97
//   22^3 (166 MiB)                     114 / 121            130 / 122
//   23^3 (190 MiB)                     134 / 138            151 / 140
//   24^3 (216 MiB)                     154 / 154            171 / 162
//   25^3 (244 MiB)                     173 / 172            191 / 184
//   Q2 on 40^3 (222 MiB)               148 / 152            165 / 153
//   41^3 (240 MiB)                     159 / 163            178 / 165
//   42^3 (257 MiB)                     173 / 173            193 / 179
//   43^3 (276 MiB)                     182 / 183            202 / 193
// (the residual alone at 25^3 115 / 99, at Q2 43^3 123 / 106).  The line is drawn for one
// operator: the two meet near 216 MiB at Q4 and 257 at Q2, and 240 is in between; with operators
// in turn streaming wins at every size measured.
inline bool stream_state(int64_t tiles, int Q) {
  return (double)tiles * NSTATE * field_stride(Q) * sizeof(double) > 240.0 * (1 << 20);
}

// Inside a V-cycle or an eigenvalue estimate (Finish sm or pq), a linearisation of 60 to 130
// MiB is loaded with plain loads: it stays in the 256 MiB last-level cache beside the records
// and vectors, and the next action (a smoothing step, an iteration, the level below) reads it
// there.  Measured, us, Q4 -> Q2 -> Q1, plain / nontemporal loads, a V-cycle with four coarse
// iterations and a setup:
//                 state       V-cycle       setup
//   FP64 15^3     53 MiB    408 / 403   1035 / 1025
//        16^3     64        440 / 447   1114 / 1129
//        18^3     91        512 / 526   1341 / 1369
//        20^3    125        631 / 649   1646 / 1696
//        21^3    145        737 / 732   1846 / 1867
//        22^3    166        812 / 801   2110 / 2083
//   FP32 18^3     46        382 / 375    986 / 984
//        20^3     63        437 / 443   1146 / 1159
//        22^3     83        507 / 518   1359 / 1378
//        25^3    122        673 / 666   1774 / 1813
//        26^3    137        737 / 727   1968 / 1966
// A single action keeps the nontemporal loads: with the states of five operators in turn, 20^3
// FP64 takes 42.1 us with them and 47.3 with plain ones.
template <typename T>
bool keep_state(int64_t tiles, int Q) {
  const double b = (double)tiles * NSTATE * field_stride(Q) * sizeof(T);
  return b >= 60.0 * (1 << 20) && b <= 130.0 * (1 << 20);
}

__device__ __forceinline__ double mat_mu(double mu0, const double *mu_e, int64_t e) {
  return mu_e ? mu_e[e] : mu0;
}

template <typename T>
__device__ __forceinline__ void load_tables(T *dst, const T *__restrict__ src, int off, int n, int t, int nt) {
  for (int i = t; i < n; i += nt) dst[i] = src[off + i];
}

// Loads the three components of a node (all issued before any is used) and writes them
// to LDS as [c][P^3]; constrained components become zero when `masked`.
template <typename S, typename T>
__device__ __forceinline__ void gather_node(const S *__restrict__ v, uint32_t w, bool masked, T *a, int q,
                                            int P3) {
  const S *p = v + (int64_t)(w & EMAP_ID_MASK) * 3;
  const S x0 = p[0], x1 = p[1], x2 = p[2];
  a[q] = (masked && ((w >> EMAP_BC_SHIFT) & 1u)) ? T(0) : (T)x0;
  a[P3 + q] = (masked && ((w >> (EMAP_BC_SHIFT + 1)) & 1u)) ? T(0) : (T)x1;
  a[2 * P3 + q] = (masked && ((w >> (EMAP_BC_SHIFT + 2)) & 1u)) ? T(0) : (T)x2;
}

// ------------------------------------------------------------------------------------
// a1: geometric factors.
// ------------------------------------------------------------------------------------
template <int P, int Q>
__global__ __launch_bounds__(QT<Q>::NT) void k_qdata(const uint32_t *__restrict__ emap,
                                                     const double *__restrict__ X,
                                                     const double *__restrict__ tab,
                                                     double *__restrict__ geo,
                                                     unsigned *__restrict__ flags, int64_t E) {
  using T = double;
  constexpr int Q3 = QT<Q>::Q3, ET = QT<Q>::ET, NQ = QT<Q>::NQ, NT = QT<Q>::NT, P3 = P * P * P;
  constexpr int S0 = 3 * Q3, S1 = 3 * Q3;
  __shared__ T sB[Q * P], sD[Q * Q], sW[Q];
  __shared__ T lds[ET * (S0 + S1)];
  const int tq = threadIdx.x, el = tq / Q3, q = tq % Q3;
  const int64_t tile = xcd_tile();
  const int64_t e = tile * ET + el;
  const bool live = tq < ET * Q3 && e < E;
  load_tables(sB, tab, TAB_B, Q * P, tq, NT);
  load_tables(sD, tab, TAB_D, Q * Q, tq, NT);
  load_tables(sW, tab, TAB_W, Q, tq, NT);
  T *a = lds + (live ? el : 0) * S0, *b = lds + ET * S0 + (live ? el : 0) * S1;
  if (live && q < P3) {
    const uint32_t node = emap[e * P3 + q] & EMAP_ID_MASK;
#pragma unroll
    for (int c = 0; c < 3; ++c) a[c * P3 + q] = X[(int64_t)node * 3 + c];
  }
  __syncthreads();
  interp<T, P, Q, 3>(a, b, sB, q, live);
  T G[3][3];
  if (live) grad_q<T, Q, 3>(b, sD, q, G);
  if (!live) return;
  const T det = det3(G);
  if (!(det > 0.0)) atomicOr(flags, det == det ? HPMG_FLAG_NONPOSITIVE_J : HPMG_FLAG_NONFINITE);
  T Di[3][3];
  inv3(G, det, Di);  // Di[k][J] = dxi_k / dX_J
  const int q1 = q % Q, q2 = (q / Q) % Q, q3 = q / (Q * Q);
  double *g = geo + tile * NGEO * NQ + tq;
  g[0] = sW[q1] * sW[q2] * sW[q3] * det;
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int J = 0; J < 3; ++J) g[(1 + k * 3 + J) * NQ] = Di[k][J];
}

// ------------------------------------------------------------------------------------
// a4-a7: residual (FP64, MODE 4 below) and a5: Jacobian action from the stored
// linearisation (FP64 or FP32), with register-blocked 1D contractions.
//
// With one thread per point, each 1D contraction would cost a thread one LDS read per
// input of every output.  Here every contraction stage is run by "line tasks": a task
// owns one line of points along the contraction direction (for one component), reads
// the line once, forms all of its outputs in registers from the 1D table (the same for
// every lane, so it is read through the scalar cache, not LDS) and writes them back in
// place.  That is one LDS read and one write per point and stage.
// Nodal (P^3) and quadrature (Q^3) arrays share one Q^3 frame per component, indexed
// i1 + Q i2 + Q^2 i3, so the interpolation stages can work in place.  The pointwise
// work (state loads, quadrature function, gather, records) keeps the one-thread-per-
// point mapping and the tile layout of the other kernels.
// Bound by memory: at Q4, 34^3 elements, FP64, the 858 MB of an apply's element kernel pass
// in 137-144 us (6.1 TB/s) where one operator is used again and in 152 where four take turns;
// the assembly's 213 MB then take 53 us instead of 33, its records and lists no longer being in
// the last-level cache.
// ------------------------------------------------------------------------------------

// First frame offset and stride of line r of a stage along DIR whose lines run over
// the other two directions with extents L1 (the faster one) and L2.
template <int Q, int DIR, int L1>
__device__ __forceinline__ int line_base(int r) {
  const int r1 = r % L1, r2 = r / L1;
  return DIR == 0 ? Q * (r1 + Q * r2) : DIR == 1 ? r1 + Q * Q * r2 : r1 + Q * r2;
}
template <int Q, int DIR>
__device__ __forceinline__ constexpr int line_step() {
  return DIR == 0 ? 1 : DIR == 1 ? Q : Q * Q;
}

// y = M x with M [NO][NI] row-major (TR = false) or y = M^T x with M [NI][NO] (TR = true).
template <typename T, int NI, int NO, bool TR>
__device__ __forceinline__ void line_apply(const T *__restrict__ M, const T (&x)[NI], T (&y)[NO]) {
#pragma unroll
  for (int o = 0; o < NO; ++o) {
    T acc = 0;
#pragma unroll
    for (int i = 0; i < NI; ++i) acc += M[TR ? i * NO + o : o * NI + i] * x[i];
    y[o] = acc;
  }
}

// One in-place contraction stage along DIR (NI inputs -> NO outputs per line) of the
// three component frames of each of the tile's elements (element el at buf + el * ELS,
// component c at + c * Q^3).  Lines run over extents L1 x L2 of the other directions.
template <typename T, int Q, int DIR, int NI, int NO, bool TR, int L1, int L2, int ET, int ELS>
__device__ __forceinline__ void line_stage(T *buf, const T *__restrict__ M, int tid, int nt, int nel) {
  constexpr int NL = L1 * L2, TASKS = 3 * NL, Q3 = Q * Q * Q, ST = line_step<Q, DIR>();
  for (int t = tid; t < ET * TASKS; t += nt) {
    const int el = t / TASKS, r = t % TASKS, c = r / NL;
    if (el >= nel) break;
    T *p = buf + el * ELS + c * Q3 + line_base<Q, DIR, L1>(r % NL);
    T x[NI], y[NO];
#pragma unroll
    for (int i = 0; i < NI; ++i) x[i] = p[i * ST];
    line_apply<T, NI, NO, TR>(M, x, y);
#pragma unroll
    for (int i = 0; i < NO; ++i) p[i * ST] = y[i];
  }
}

template <typename T, int NI, int NO, bool TR, int ST>
__device__ __forceinline__ void line_task(T *p, const T *__restrict__ M) {
  T x[NI], y[NO];
#pragma unroll
  for (int i = 0; i < NI; ++i) x[i] = p[i * ST];
  line_apply<T, NI, NO, TR>(M, x, y);
#pragma unroll
  for (int i = 0; i < NO; ++i) p[i * ST] = y[i];
}

// Element records [e][a][c] out of the tile's LDS frames (component c of element te at
// f + te * els + c * Q^3, nodes at their frame index).  SWEEP 1 / 2: contiguous sweeps over
// the tile's run of records (each store instruction covers whole cache lines) with plain
// (1) or nontemporal (2) stores; 0: three strided stores per node.  The two sweep kinds are
// separate instances: a run-time choice lets the compiler merge both stores into a plain
// one.
template <typename T, int P, int Q, int SWEEP>
__device__ __forceinline__ void store_tile_records(T *__restrict__ ev, int64_t tile, int nel, const T *f, int els) {
  constexpr int Q2 = Q * Q, Q3 = Q2 * Q, P3 = P * P * P, ET = QT<Q>::ET, NT = QT<Q>::NT;
  const int tq = threadIdx.x;
  if constexpr (SWEEP > 0) {
    T *o = ev + tile * (int64_t)(ET * P3 * 3);
    const int nd = nel * P3 * 3;
    for (int d = tq; d < nd; d += NT) {
      const int r = d / 3, c = d - 3 * r, te = r / P3, a = r - te * P3;
      const int an = (a % P) + Q * ((a / P) % P) + Q2 * (a / (P * P));
      if constexpr (SWEEP == 1)
        o[d] = f[te * els + c * Q3 + an];
      else
        __builtin_nontemporal_store(f[te * els + c * Q3 + an], o + d);
    }
  } else {
    const int el = tq / Q3, q = tq % Q3;
    if (el < nel && q < P3) {
      const T *v = f + el * els + (q % P) + Q * ((q / P) % P) + Q2 * (q / (P * P));
      const T y0 = v[0], y1 = v[Q3], y2 = v[2 * Q3];
      T *o = ev + ((tile * ET + el) * P3 + q) * 3;
      o[0] = y0;
      o[1] = y1;
      o[2] = y2;
    }
  }
}

// MODE 0: the 16-scalar current-configuration state (sqrt(W) dxi/dx, tau, lambda log J;
// T = double or float).
// MODE 1 / 2: the initial-configuration forms, 19 / 26 scalars (geometry W, grad_X xi
// + grad_X u [+ C^-1, lambda log J]); T = double.
// MODE 3: the 20-scalar current-configuration form (dxi/dx, J, grad_X u, W): tau and
// lambda log J are rebuilt from grad_X u and J; T = double.
// MODE 4: the residual (du is u, unmasked; T = double): kinematics and the Kirchhoff
// flux from the geometry (W, dxi/dX), the 16-scalar state written to state_out when it
// is given, non-positive or non-finite J raised in flags.
// MODE 8: the residual of MODE 4 with a state too large for the last-level cache: whole
// lines of it leave with nontemporal stores (stream_state).
// MODE 9: MODE 0 with plain loads of a state that stays in the last-level cache from one
// action to the next (keep_state).
// MODE 5: the Jacobian with the linearisation recomputed at u (T = double or float; u
// is converted to T): u and du go through the forward stages side by side (half the
// barriers of one after the other, and nothing of u to keep in registers meanwhile); the
// kinematics of u from the geometry at every point, then the action on du as in MODE 0.
// MODE 6 / 7: the adjoint (vector-Jacobian product; du is the cotangent w of the masked
// residual) from the 16-scalar state / recomputed at u (T = double or float).  With mub or
// lamb given, the parameter gradients of every element: the point values are two more
// frames, summed line by line along x, z and y in the transposed stages by the threads
// counted from the last, most of which have no line of their own there.  With a thread per
// point, all contractions out of LDS (two workgroups per compute unit) and one thread an
// element summing the parameters, the FP64 product took 165 us on 20^3 Q4 elements and 53.5
// on 23^3 Q3 ones, assembly included; this form 46-50 and 38-41 (recomputed 180 -> 61 and
// 56 -> 49; MODE 7 is held to 128 registers for four waves per SIMD, 63 and 51 without).
// SWEEP: how the records are stored (store_tile_records).
template <typename T, int P, int Q, int MODE, int SWEEP>
__global__ __launch_bounds__(QT<Q>::NT, MODE == 7 ? 4 : 1) void k_jacobian_lines(
    const uint32_t *__restrict__ emap, const T *__restrict__ du, const T *__restrict__ state,
    const double *__restrict__ geo, const double *__restrict__ sinit,
    const T *__restrict__ tab, double mu0, double lam0, const double *__restrict__ mu_e,
    const double *__restrict__ lam_e, T *__restrict__ ev, int64_t E, const double *__restrict__ stop,
    double *__restrict__ state_out, unsigned *__restrict__ flags, const double *__restrict__ u,
    double *__restrict__ mub, double *__restrict__ lamb) {
  constexpr bool KEEP = MODE == 9, APPLY = MODE == 0 || KEEP, RES = MODE == 4 || MODE == 8;
  constexpr bool VJP = MODE == 6 || MODE == 7, TWO = MODE == 5 || MODE == 7, STATE = APPLY || MODE == 6;
  constexpr int NH = MODE == 2 ? 16 : MODE == 3 ? 19 : 9;
  static_assert(!RES || std::is_same<T, double>::value, "the residual form is FP64");
  if (stop && *stop != 0.0) return;  // a stopped PCG (uniform over the grid)
  constexpr int Q2 = Q * Q, Q3 = Q2 * Q, P3 = P * P * P, ET = QT<Q>::ET, NQ = QT<Q>::NQ, NT = QT<Q>::NT;
  // Per element: v [3][Q^3] (du, then its values at the points, then the z-derivative
  // G[c][2] and the z-flux in place, then the nodal result) and G [3][2][Q^3] (the x- and
  // y-derivatives, then the x- and y-flux): 9 Q^3 scalars, so that more tiles fit in LDS.
  // MODES 5 and 7 carry two fields, u and then du, each in frames of its own; MODES 6 and 7
  // end with the two parameter frames.
  constexpr int NF = TWO ? 2 : 1, FS = 9 * Q3, PS = NF * FS, ELS = PS + (VJP ? 2 * Q3 : 0);
  __shared__ T lds[ET * ELS];
  const int tq = threadIdx.x, el = tq / Q3, q = tq % Q3;
  const int64_t tile = xcd_tile();
  const int64_t e = tile * ET + el;
  const int nel = (int)((E - tile * ET) < ET ? (E - tile * ET) : ET);
  const bool live = tq < ET * Q3 && e < E;
  const T *tB = tab + TAB_B, *tD = tab + TAB_D;
  T *v = lds + (live ? el : 0) * ELS + (NF - 1) * FS, *G = v + 3 * Q3;
  // Frame index of node q (q < P^3).
  const int qn = (q % P) + Q * ((q / P) % P) + Q2 * (q / (P * P));
  T sv[STATE ? NSTATE : 1];
  double gv[STATE || MODE == 3 ? 1 : NGEO], hv[STATE ? 1 : NH];
  const bool par = VJP && (mub || lamb);
  // Stages over 3 Q^2 lines per element give a thread the same (element, component, line)
  // every time, only the line's direction changes: its offsets are formed once (all orders
  // but Q = 2, whose tile has more lines than threads).
  constexpr int LT = ET * 3 * Q2, NL = (LT + NT - 1) / NT;
  constexpr bool FI = NL == 1;
  const int e3 = tq / (3 * Q2), r3 = tq % (3 * Q2), c3 = r3 / Q2, ln3 = r3 % Q2;
  const bool a3 = tq < LT && e3 < nel;
  T *const p3 = lds + (a3 ? e3 * ELS + c3 * Q3 : 0);
  const int lb0 = line_base<Q, 0, Q>(ln3), lb1 = line_base<Q, 1, Q>(ln3), lb2 = line_base<Q, 2, Q>(ln3);
  // f(i, v frame of the line's component, its frame in G, first offset of its x, y and z
  // line) for the i-th of this thread's lines, for fields f0 .. NF - 1.
  auto lines = [&](int f0, auto &&f) {
    if constexpr (FI) {
      if (a3)
#pragma unroll
        for (int k = f0; k < NF; ++k) f(k, p3 + k * FS, p3 + k * FS + (3 + c3) * Q3, lb0, lb1, lb2);
    } else {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int t = tq + i * NT, te = t / (3 * Q2), r = t % (3 * Q2), c = r / Q2, ln = r % Q2;
        T *p = lds + te * ELS + c * Q3;
        if (t < LT && te < nel)
#pragma unroll
          for (int k = f0; k < NF; ++k)
            f(i * NF + k, p + k * FS, p + k * FS + (3 + c) * Q3, line_base<Q, 0, Q>(ln), line_base<Q, 1, Q>(ln),
              line_base<Q, 2, Q>(ln));
      }
    }
  };
  if (live && q < P3) {
    const uint32_t w = emap[e * P3 + q];
    const T *src = du + (int64_t)(w & EMAP_ID_MASK) * 3;
    const T x0 = src[0], x1 = src[1], x2 = src[2];
    if constexpr (TWO) {
      const double *su = u + (int64_t)(w & EMAP_ID_MASK) * 3;
      T *vu = v - FS;
      const double u0 = su[0], u1 = su[1], u2 = su[2];
      vu[qn] = (T)u0;
      vu[Q3 + qn] = (T)u1;
      vu[2 * Q3 + qn] = (T)u2;
    }
    // u is taken whole (the residual); du has its constrained components zeroed
    const uint32_t bc = RES ? 0u : (w >> EMAP_BC_SHIFT);
    v[qn] = (bc & 1u) ? T(0) : x0;
    v[Q3 + qn] = ((bc >> 1) & 1u) ? T(0) : x1;
    v[2 * Q3 + qn] = ((bc >> 2) & 1u) ? T(0) : x2;
  }
  if (live) {
    if constexpr (STATE) {
      const T *s = state + tile * NSTATE * NQ + tq;
#pragma unroll
      for (int f = 0; f < NSTATE; ++f) sv[f] = KEEP ? s[f * NQ] : __builtin_nontemporal_load(s + f * NQ);
      if (par) gv[0] = __builtin_nontemporal_load(geo + tile * NGEO * NQ + tq);  // W
    } else if constexpr (MODE == 3) {
      gv[0] = __builtin_nontemporal_load(geo + tile * NGEO * NQ + tq);  // W only
      const double *h = sinit + tile * NINIT * NQ + tq;
#pragma unroll
      for (int f = 0; f < 9; ++f) hv[f] = __builtin_nontemporal_load(h + f * NQ);
#pragma unroll
      for (int f = 0; f < 10; ++f) hv[9 + f] = __builtin_nontemporal_load(h + (16 + f) * NQ);
    } else if constexpr (RES || TWO) {
      const double *g = geo + tile * NGEO * NQ + tq;
#pragma unroll
      for (int f = 0; f < NGEO; ++f) gv[f] = __builtin_nontemporal_load(g + f * NQ);
    } else {
      const double *g = geo + tile * NGEO * NQ + tq;
#pragma unroll
      for (int f = 0; f < NGEO; ++f) gv[f] = __builtin_nontemporal_load(g + f * NQ);
      const double *h = sinit + tile * NINIT * NQ + tq;
#pragma unroll
      for (int f = 0; f < NH; ++f) hv[f] = __builtin_nontemporal_load(h + f * NQ);
    }
  }
  __syncthreads();
  // Interpolation to the points, one direction at a time, in place.
  if constexpr (P == Q) {
    lines(0, [&](int, T *p, T *, int l0, int, int) { line_task<T, P, Q, false, 1>(p + l0, tB); });
    __syncthreads();
    lines(0, [&](int, T *p, T *, int, int l1, int) { line_task<T, P, Q, false, Q>(p + l1, tB); });
  } else {
#pragma unroll
    for (int k = 0; k < NF; ++k) line_stage<T, Q, 0, P, Q, false, P, P, ET, ELS>(lds + k * FS, tB, tq, NT, nel);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NF; ++k) line_stage<T, Q, 1, P, Q, false, Q, P, ET, ELS>(lds + k * FS, tB, tq, NT, nel);
  }
  __syncthreads();
  // The z lines end at the points; their collocated derivative stays in registers until
  // every x and y line has read the values.
  T dz[NL * NF][Q];
  lines(0, [&](int i, T *p, T *, int, int, int l2) {
    T x[P], y[Q];
#pragma unroll
    for (int j = 0; j < P; ++j) x[j] = p[l2 + j * Q2];
    line_apply<T, P, Q, false>(tB, x, y);
#pragma unroll
    for (int j = 0; j < Q; ++j) p[l2 + j * Q2] = y[j];
    line_apply<T, Q, Q, false>(tD, y, dz[i]);
  });
  __syncthreads();
  // G[c][k] = D_k v[c] for k = 0, 1: each thread an x and a y line, so that no wave holds
  // both directions at once (with the directions on neighbouring threads every wave ran
  // both: 17 % more vector instructions at Q4).
  lines(0, [&](int, T *p, T *g, int l0, int l1, int) {
    T x[Q], y[Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) x[j] = p[l0 + j];
    line_apply<T, Q, Q, false>(tD, x, y);
#pragma unroll
    for (int j = 0; j < Q; ++j) g[l0 + j] = y[j];
#pragma unroll
    for (int j = 0; j < Q; ++j) x[j] = p[l1 + j * Q];
    line_apply<T, Q, Q, false>(tD, x, y);
#pragma unroll
    for (int j = 0; j < Q; ++j) g[Q3 + l1 + j * Q] = y[j];
  });
  __syncthreads();
  // G[c][2] over v[c]
  lines(0, [&](int i, T *p, T *, int, int, int l2) {
#pragma unroll
    for (int j = 0; j < Q; ++j) p[l2 + j * Q2] = dz[i][j];
  });
  __syncthreads();
  // Quadrature function, one thread per point, flux written over the gradient
  // (components k = 0, 1 in G, k = 2 in v).
  double so[MODE == 8 ? NSTATE : 1] = {};
  if (live) {
    T Gq[3][3], f[3][3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      Gq[c][0] = G[(c * 2) * Q3 + q];
      Gq[c][1] = G[(c * 2 + 1) * Q3 + q];
      Gq[c][2] = v[c * Q3 + q];
    }
    if constexpr (APPLY) {
      T A[3][3], tau[6];
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int j = 0; j < 3; ++j) A[k][j] = sv[k * 3 + j];
#pragma unroll
      for (int m = 0; m < 6; ++m) tau[m] = sv[9 + m];
      const T c = sv[15], W = T(1);  // the weight is in the scaled dxi/dx
      const T mu = (T)mat_mu(mu0, mu_e, e), lam = (T)mat_mu(lam0, lam_e, e);
      jacobian_qf(Gq, A, tau, c, W, mu, lam, f);
    } else if constexpr (MODE == 3) {
      const double mu = mat_mu(mu0, mu_e, e), lam = mat_mu(lam0, lam_e, e);
      double A[3][3], tau[6];
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int j = 0; j < 3; ++j) A[k][j] = hv[9 + k * 3 + j];
      const double c = lam * log1p(hv[18]);
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = i; j < 3; ++j) {
          const double hh = hv[i * 3] * hv[j * 3] + hv[i * 3 + 1] * hv[j * 3 + 1] + hv[i * 3 + 2] * hv[j * 3 + 2];
          tau[sym_index(i, j)] = mu * (hv[i * 3 + j] + hv[j * 3 + i] + hh) + (i == j ? c : 0.0);
        }
      jacobian_qf(Gq, A, tau, c, gv[0], mu, lam, f);
    } else if constexpr (MODE == 6) {
      // the weight rides in the scaled dxi/dx: M below is sqrt(W) w's gradient
      T A[3][3], tau[6], M[3][3];
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int j = 0; j < 3; ++j) A[k][j] = sv[k * 3 + j];
#pragma unroll
      for (int m = 0; m < 6; ++m) tau[m] = sv[9 + m];
      const T c = sv[15], mu = (T)mat_mu(mu0, mu_e, e), lam = (T)mat_mu(lam0, lam_e, e);
      adjoint_qf(Gq, A, tau, c, T(1), mu, lam, f, M);
      if (par) {
        // tau = 2 mu e + c I and c = lambda log J
        const T sw = (T)sqrt(gv[0]);
        T d = 0;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int j = 0; j < 3; ++j) d += M[i][j] * (tau[sym_index(i, j)] - (i == j ? c : T(0)));
        lds[el * ELS + PS + q] = sw * (d / mu);
        lds[el * ELS + PS + Q3 + q] = sw * (T)((double)c / (double)lam) * (M[0][0] + M[1][1] + M[2][2]);
      }
    } else if constexpr (TWO) {
      const T *vu = v - FS, *Gf = G - FS;  // u's frames
      T Gu[3][3], D[3][3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        Gu[c][0] = Gf[(c * 2) * Q3 + q];
        Gu[c][1] = Gf[(c * 2 + 1) * Q3 + q];
        Gu[c][2] = vu[c * Q3 + q];
      }
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int J = 0; J < 3; ++J) D[k][J] = (T)gv[1 + k * 3 + J];
      const T mu = (T)mat_mu(mu0, mu_e, e), lam = (T)mat_mu(lam0, lam_e, e);
      Kin<T> k;
      kinematics(Gu, D, mu, lam, k);
      if constexpr (MODE == 5) {
        jacobian_qf(Gq, k.A, k.tau, k.c, (T)gv[0], mu, lam, f);
      } else {
        T M[3][3];
        const T W = (T)gv[0];
        adjoint_qf(Gq, k.A, k.tau, k.c, W, mu, lam, f, M);
        if (par) {
          T d = 0;
#pragma unroll
          for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j)
              d += M[i][j] * (k.H[i][j] + k.H[j][i] + k.H[i][0] * k.H[j][0] + k.H[i][1] * k.H[j][1] +
                              k.H[i][2] * k.H[j][2]);
          lds[el * ELS + PS + q] = W * d;
          lds[el * ELS + PS + Q3 + q] = W * (T)k.logJ * (M[0][0] + M[1][1] + M[2][2]);
        }
      }
    } else if constexpr (RES) {
      double D[3][3];
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int J = 0; J < 3; ++J) D[k][J] = gv[1 + k * 3 + J];
      Kin<double> k;
      kinematics(Gq, D, mat_mu(mu0, mu_e, e), mat_mu(lam0, lam_e, e), k);
      if (!(k.Jm1 > -1.0)) atomicOr(flags, k.Jm1 == k.Jm1 ? HPMG_FLAG_NONPOSITIVE_J : HPMG_FLAG_NONFINITE);
      residual_qf(k, gv[0], f);
      if (MODE == 8 || state_out) {
        // sqrt(W) dxi/dx, tau, lambda log J (the weight rides in the scaled dxi/dx)
        const double sw = sqrt(gv[0]);
        double *o = state_out + tile * NSTATE * NQ + tq;
        auto put = [&](int i, double x) {
          if constexpr (MODE == 8)
            so[i] = x;
          else
            o[i * NQ] = x;
        };
#pragma unroll
        for (int kk = 0; kk < 3; ++kk)
#pragma unroll
          for (int j = 0; j < 3; ++j) put(kk * 3 + j, sw * k.A[kk][j]);
#pragma unroll
        for (int m = 0; m < 6; ++m) put(9 + m, k.tau[m]);
        put(15, k.c);
      }
    } else {
      jacobian_qf_initial<MODE == 2>(Gq, gv, hv, mat_mu(mu0, mu_e, e), mat_mu(lam0, lam_e, e), f);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      G[(i * 2) * Q3 + q] = f[i][0];
      G[(i * 2 + 1) * Q3 + q] = f[i][1];
      v[i * Q3 + q] = f[i][2];
    }
  }
  if constexpr (MODE == 8) {
    // the padding too (zeros), so that every line goes out whole
    if (tq < NQ) {
      double *o = state_out + tile * NSTATE * NQ + tq;
#pragma unroll
      for (int i = 0; i < NSTATE; ++i) __builtin_nontemporal_store(so[i], o + i * NQ);
    }
  }
  __syncthreads();
  // Sums of the parameter frames along one direction: f(frame of the parameter, element,
  // parameter, line) for `lines` lines of each.
  auto param_lines = [&](int lines, auto &&f) {
    if (par)
      for (int t = NT - 1 - tq; t < 2 * nel * lines; t += NT) {
        const int te = t / (2 * lines), r = t % (2 * lines), k = r / lines;
        f(lds + te * ELS + PS + k * Q3, te, k, r % lines);
      }
  };
  auto line_sum = [&](const T *p, int step) {
    T t = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) t += p[i * step];
    return t;
  };
  // Transposed derivative, x and y directions in place on the flux arrays.
  lines(NF - 1, [&](int, T *, T *g, int l0, int l1, int) {
    line_task<T, Q, Q, true, 1>(g + l0, tD);
    line_task<T, Q, Q, true, Q>(g + Q3 + l1, tD);
  });
  if constexpr (VJP) param_lines(Q2, [&](T *p, int, int, int ln) { p[ln * Q] = line_sum(p + ln * Q, 1); });
  __syncthreads();
  // z direction: h = D_z^T f_z + (x and y parts), then the first transposed
  // interpolation stage (B_z^T, Q -> P) in registers; the result goes to v, over the
  // z-flux line it was formed from.
  lines(NF - 1, [&](int, T *p, T *g, int, int, int l2) {
    const T *fxy = g + l2;
    T *o = p + l2;
    T x[Q], y[Q], z[P];
#pragma unroll
    for (int i = 0; i < Q; ++i) x[i] = o[i * Q2];
    line_apply<T, Q, Q, true>(tD, x, y);
#pragma unroll
    for (int i = 0; i < Q; ++i) y[i] += fxy[i * Q2] + fxy[Q3 + i * Q2];
    line_apply<T, Q, P, true>(tB, y, z);
#pragma unroll
    for (int i = 0; i < P; ++i) o[i * Q2] = z[i];
  });
  if constexpr (VJP) param_lines(Q, [&](T *p, int, int, int ln) { p[ln * Q] = line_sum(p + ln * Q, Q2); });
  __syncthreads();
  if constexpr (VJP)
    param_lines(1, [&](T *p, int te, int k, int) {
      double *o = k ? lamb : mub;
      if (o) o[tile * ET + te] = (double)line_sum(p, Q);
    });
  if constexpr (P == Q) {
    lines(NF - 1, [&](int, T *p, T *, int, int l1, int) { line_task<T, Q, P, true, Q>(p + l1, tB); });
    __syncthreads();
    lines(NF - 1, [&](int, T *p, T *, int l0, int, int) { line_task<T, Q, P, true, 1>(p + l0, tB); });
  } else {
    line_stage<T, Q, 1, Q, P, true, Q, P, ET, ELS>(lds + (NF - 1) * FS, tB, tq, NT, nel);
    __syncthreads();
    line_stage<T, Q, 0, Q, P, true, P, P, ET, ELS>(lds + (NF - 1) * FS, tB, tq, NT, nel);
  }
  __syncthreads();
  store_tile_records<T, P, Q, SWEEP>(ev, tile, nel, lds + (NF - 1) * FS, ELS);
}

// Launches k_jacobian_lines with the record-store form for its order, precision and size.
template <typename T, int P, int Q, int MODE, typename... A>
void lines_launch(unsigned tiles, hipStream_t s, bool keep, A... a) {
  if constexpr (sweep_records<T>(P)) {
    if (keep)
      k_jacobian_lines<T, P, Q, MODE, 1><<<tiles, QT<Q>::NT, 0, s>>>(a...);
    else
      k_jacobian_lines<T, P, Q, MODE, 2><<<tiles, QT<Q>::NT, 0, s>>>(a...);
  } else {
    k_jacobian_lines<T, P, Q, MODE, 0><<<tiles, QT<Q>::NT, 0, s>>>(a...);
  }
}

// ------------------------------------------------------------------------------------
// Alternative linearisations at u, per point, [tile][26][field_stride]: grad_X u (9),
// C^-1 (6), lambda log J (1), dxi/dx (9), J - 1 (1).  With the constant W and
// grad_X xi, fields 0-8 are the 19-scalar initial-configuration "native" form, 0-15 the
// 26-scalar "tuned" form; fields 0-8 and 16-25 with W are the 20-scalar current-
// configuration form (dxi/dx, J, grad_X u, W).
// ------------------------------------------------------------------------------------
template <int P, int Q>
__global__ __launch_bounds__(QT<Q>::NT) void k_state_initial(
    const uint32_t *__restrict__ emap, const double *__restrict__ u, const double *__restrict__ geo,
    const double *__restrict__ tab, double mu0, double lam0, const double *__restrict__ mu_e,
    const double *__restrict__ lam_e, double *__restrict__ sinit, unsigned *__restrict__ flags, int64_t E) {
  using T = double;
  constexpr int Q3 = QT<Q>::Q3, ET = QT<Q>::ET, NQ = QT<Q>::NQ, NT = QT<Q>::NT, P3 = P * P * P;
  constexpr int S0 = 3 * Q3;
  __shared__ T sB[Q * P], sD[Q * Q];
  __shared__ T lds[2 * ET * S0];
  const int tq = threadIdx.x, el = tq / Q3, q = tq % Q3;
  const int64_t tile = xcd_tile();
  const int64_t e = tile * ET + el;
  const bool live = tq < ET * Q3 && e < E;
  load_tables(sB, tab, TAB_B, Q * P, tq, NT);
  load_tables(sD, tab, TAB_D, Q * Q, tq, NT);
  T *a = lds + (live ? el : 0) * S0, *b = lds + ET * S0 + (live ? el : 0) * S0;
  if (live && q < P3) gather_node(u, emap[e * P3 + q], false, a, q, P3);
  __syncthreads();
  interp<T, P, Q, 3>(a, b, sB, q, live);
  if (!live) return;
  T G[3][3], D[3][3];
  grad_q<T, Q, 3>(b, sD, q, G);
  const double *g = geo + tile * NGEO * NQ + tq;
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int J = 0; J < 3; ++J) D[k][J] = g[(1 + k * 3 + J) * NQ];
  Kin<T> k;
  kinematics(G, D, mat_mu(mu0, mu_e, e), mat_mu(lam0, lam_e, e), k);
  if (!(k.Jm1 > -1.0)) atomicOr(flags, k.Jm1 == k.Jm1 ? HPMG_FLAG_NONPOSITIVE_J : HPMG_FLAG_NONFINITE);
  T F[3][3], Fi[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) F[i][j] = (i == j ? 1.0 : 0.0) + k.H[i][j];
  inv3(F, 1.0 + k.Jm1, Fi);
  double *o = sinit + tile * NINIT * NQ + tq;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int J = 0; J < 3; ++J) o[(i * 3 + J) * NQ] = k.H[i][J];
#pragma unroll
  for (int I = 0; I < 3; ++I)
#pragma unroll
    for (int J = I; J < 3; ++J)
      o[(9 + sym_index(I, J)) * NQ] = Fi[I][0] * Fi[J][0] + Fi[I][1] * Fi[J][1] + Fi[I][2] * Fi[J][2];
  o[15 * NQ] = k.c;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int j = 0; j < 3; ++j) o[(16 + a * 3 + j) * NQ] = k.A[a][j];
  o[25 * NQ] = k.Jm1;
}

// ------------------------------------------------------------------------------------
// External dead loads (eq. variational-form, right-hand side).
// Body force: per element int phi_a dV = sum_q B3[q][a] W_q, a transposed
// interpolation of the point weights, times rho0 g; element records.
// ------------------------------------------------------------------------------------
template <int P, int Q>
__global__ __launch_bounds__(QT<Q>::NT) void k_body_load(const double *__restrict__ geo,
                                                         const double *__restrict__ tab, double g0, double g1,
                                                         double g2, double *__restrict__ ev, int64_t E) {
  using T = double;
  constexpr int Q3 = QT<Q>::Q3, ET = QT<Q>::ET, NQ = QT<Q>::NQ, NT = QT<Q>::NT, P3 = P * P * P;
  __shared__ T sB[Q * P];
  __shared__ T lds[2 * ET * Q3];
  const int tq = threadIdx.x, el = tq / Q3, q = tq % Q3;
  const int64_t tile = xcd_tile();
  const int64_t e = tile * ET + el;
  const bool live = tq < ET * Q3 && e < E;
  load_tables(sB, tab, TAB_B, Q * P, tq, NT);
  T *a = lds + (live ? el : 0) * Q3, *b = lds + ET * Q3 + (live ? el : 0) * Q3;
  if (live) b[q] = geo[tile * NGEO * NQ + tq];  // W
  __syncthreads();
  interp_t<T, P, Q, 1>(b, a, sB, q, live);
  if (live && q < P3) {
    double *o = ev + ((int64_t)e * P3 + q) * 3;
    const T v = a[q];
    o[0] = v * g0;
    o[1] = v * g1;
    o[2] = v * g2;
  }
}

// Traction on element faces, one thread per face: the face's P^2 nodes (local face
// 0..5 = xi_1 = -1, +1, xi_2 = -1, +1, xi_3 = -1, +1), area element |X_,s x X_,r| from
// the in-face derivatives at the Q^2 Gauss points, records [face][P^2][3] = int phi t dA
// and the node of each record.
template <int P, int Q>
__global__ void k_traction_load(const double *__restrict__ X, const int32_t *__restrict__ elem_nodes,
                                const int32_t *__restrict__ face_elem, const int32_t *__restrict__ face_id,
                                const double *__restrict__ tab, double t0, double t1, double t2, int64_t nf,
                                int64_t E, double *__restrict__ rec, int32_t *__restrict__ rec_node,
                                unsigned *__restrict__ flags) {
  const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= nf) return;
  const int32_t e = face_elem[f], id = face_id[f];
  double *out = rec + f * P * P * 3;
  int32_t *nodes = rec_node + f * P * P;
  if (e < 0 || e >= E || id < 0 || id > 5) {  // reported to the host, nothing written
    atomicOr(flags, 4u);
    for (int k = 0; k < P * P; ++k) {
      nodes[k] = -1;
      out[3 * k] = out[3 * k + 1] = out[3 * k + 2] = 0.0;
    }
    return;
  }
  const int d = id / 2, ad = (id % 2) ? P - 1 : 0;
  const int sd = d == 0 ? 1 : 0, rd = d == 2 ? 1 : 2;  // in-face directions, s < r
  const int str[3] = {1, P, P * P};
  double x[P * P][3];
  for (int c = 0; c < P; ++c)
    for (int b = 0; b < P; ++b) {
      const int a = ad * str[d] + b * str[sd] + c * str[rd];
      const int32_t n = elem_nodes[(int64_t)e * P * P * P + a];
      nodes[b + P * c] = n;
      for (int k = 0; k < 3; ++k) x[b + P * c][k] = X[(int64_t)n * 3 + k];
    }
  double acc[P * P];
  for (int k = 0; k < P * P; ++k) acc[k] = 0.0;
  const double *B = tab + TAB_B, *G = tab + TAB_G, *w = tab + TAB_W;
  for (int j = 0; j < Q; ++j)
    for (int i = 0; i < Q; ++i) {
      double ts[3] = {0, 0, 0}, tr[3] = {0, 0, 0};
      for (int c = 0; c < P; ++c)
        for (int b = 0; b < P; ++b) {
          const double gs = G[i * P + b] * B[j * P + c], gr = B[i * P + b] * G[j * P + c];
          for (int k = 0; k < 3; ++k) {
            ts[k] += gs * x[b + P * c][k];
            tr[k] += gr * x[b + P * c][k];
          }
        }
      const double n0 = ts[1] * tr[2] - ts[2] * tr[1], n1 = ts[2] * tr[0] - ts[0] * tr[2],
                   n2 = ts[0] * tr[1] - ts[1] * tr[0];
      const double dA = sqrt(n0 * n0 + n1 * n1 + n2 * n2) * w[i] * w[j];
      for (int c = 0; c < P; ++c)
        for (int b = 0; b < P; ++b) acc[b + P * c] += B[i * P + b] * B[j * P + c] * dA;
    }
  for (int k = 0; k < P * P; ++k) {
    out[3 * k] = acc[k] * t0;
    out[3 * k + 1] = acc[k] * t1;
    out[3 * k + 2] = acc[k] * t2;
  }
}

// ------------------------------------------------------------------------------------
// a8: diagonal.  Per quadrature point and component i, the 3x3 block
//   K^(i)_kl = W [ (A tau A^T)_kl + (mu - c)(A A^T)_kl + (lambda + mu - c) A_ki A_li ]
// (from the stored sqrt(W) A the weight comes out of the products itself)
// (the Jacobian map with G = e_i grad(phi)^T); the node value is
//   sum_q sum_kl K^(i)_kl dphi/dxi_k dphi/dxi_l,
// a tensor product of the 1D elementwise tables B*B, B*G, G*G, contracted in three
// transposed 1D stages for each of the six (k, l) pairs and summed in pair order.  Line
// tasks as in k_jacobian_lines, a task taking all pairs of its line so that the tables stay
// in scalar registers, three barriers after the point stage.  One thread per point and
// pair, with every contraction's operands read from LDS and 24 barriers, took 130-147 us for
// 25^3 Q4 elements in FP64; this form 70-83, of which the 250 MB of state take 44 (summing
// the pairs that share an x table before the x stage saves another 8 us, but rounds
// otherwise than before, which the coarse solves of a V-cycle amplify to 1e-9 and more).
// ------------------------------------------------------------------------------------
template <typename T, int P, int Q, int SWEEP>
__global__ __launch_bounds__(QT<Q>::NT) void k_diagonal(
    const T *__restrict__ state, const T *__restrict__ tab, double mu0, double lam0,
    const double *__restrict__ mu_e, const double *__restrict__ lam_e, T *__restrict__ ev, int64_t E) {
  constexpr int Q2 = Q * Q, Q3 = Q2 * Q, ET = QT<Q>::ET, NQ = QT<Q>::NQ, NT = QT<Q>::NT, P3 = P * P * P;
  constexpr int ELS = 18 * Q3;  // per element: frame 3 p + i of pair p, component i
  __shared__ T lds[ET * ELS];
  const int tq = threadIdx.x, el = tq / Q3, q = tq % Q3;
  const int64_t tile = xcd_tile();
  const int64_t e = tile * ET + el;
  const int nel = (int)((E - tile * ET) < ET ? (E - tile * ET) : ET);
  const bool live = tq < ET * Q3 && e < E;
  const T *tBB = tab + TAB_BB, *tBG = tab + TAB_BG, *tGG = tab + TAB_GG;
  if (live) {
    T A[3][3], tau[6];
    const T *s = state + tile * NSTATE * NQ + tq;
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int j = 0; j < 3; ++j) A[k][j] = __builtin_nontemporal_load(s + (k * 3 + j) * NQ);
#pragma unroll
    for (int m = 0; m < 6; ++m) tau[m] = __builtin_nontemporal_load(s + (9 + m) * NQ);
    const T c = __builtin_nontemporal_load(s + 15 * NQ);  // the weight is in the scaled dxi/dx
    const T mu = (T)mat_mu(mu0, mu_e, e), lam = (T)mat_mu(lam0, lam_e, e);
    T AT[3][3];  // A tau
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int j = 0; j < 3; ++j)
        AT[k][j] = A[k][0] * tau[sym_index(0, j)] + A[k][1] * tau[sym_index(1, j)] + A[k][2] * tau[sym_index(2, j)];
    constexpr int pk[6] = {0, 1, 2, 1, 0, 0}, pl[6] = {0, 1, 2, 2, 2, 1};
    T *K = lds + el * ELS + q;
#pragma unroll
    for (int p = 0; p < 6; ++p) {
      const int k = pk[p], l = pl[p];
      const T m1 = AT[k][0] * A[l][0] + AT[k][1] * A[l][1] + AT[k][2] * A[l][2];
      const T m2 = A[k][0] * A[l][0] + A[k][1] * A[l][1] + A[k][2] * A[l][2];
      const T sc = (k == l) ? T(1) : T(2);
#pragma unroll
      for (int i = 0; i < 3; ++i)
        K[(3 * p + i) * Q3] = sc * (m1 + (mu - c) * m2 + (lam + mu - c) * A[k][i] * A[l][i]);
    }
  }
  __syncthreads();
  // z lines, in place (pair order 00, 11, 22, 12, 02, 01)
  for (int t = tq; t < ET * 3 * Q2; t += NT) {
    const int te = t / (3 * Q2), r = t % (3 * Q2), i = r / Q2;
    if (te >= nel) break;
    T *f = lds + te * ELS + i * Q3 + line_base<Q, 2, Q>(r % Q2);
#pragma unroll
    for (int p = 0; p < 6; ++p)
      line_task<T, Q, P, true, Q2>(f + 3 * p * Q3, p == 2 ? tGG : p == 3 || p == 4 ? tBG : tBB);
  }
  __syncthreads();
  // y lines, in place
  for (int t = tq; t < ET * 3 * Q * P; t += NT) {
    const int te = t / (3 * Q * P), r = t % (3 * Q * P), i = r / (Q * P);
    if (te >= nel) break;
    T *f = lds + te * ELS + i * Q3 + line_base<Q, 1, Q>(r % (Q * P));
#pragma unroll
    for (int p = 0; p < 6; ++p)
      line_task<T, Q, P, true, Q>(f + 3 * p * Q3, p == 1 ? tGG : p == 3 || p == 5 ? tBG : tBB);
  }
  __syncthreads();
  // x lines, summed over the pairs in order
  for (int t = tq; t < ET * 3 * P * P; t += NT) {
    const int te = t / (3 * P * P), r = t % (3 * P * P), i = r / (P * P);
    if (te >= nel) break;
    T *f = lds + te * ELS + i * Q3 + line_base<Q, 0, P>(r % (P * P));
    T acc[P];
#pragma unroll
    for (int p = 0; p < 6; ++p) {
      T x[Q], y[P];
#pragma unroll
      for (int j = 0; j < Q; ++j) x[j] = f[3 * p * Q3 + j];
      line_apply<T, Q, P, true>(p == 0 ? tGG : p >= 4 ? tBG : tBB, x, y);
#pragma unroll
      for (int o = 0; o < P; ++o) acc[o] = p ? acc[o] + y[o] : y[o];
    }
#pragma unroll
    for (int o = 0; o < P; ++o) f[o] = acc[o];
  }
  __syncthreads();
  store_tile_records<T, P, Q, SWEEP>(ev, tile, nel, lds, ELS);
}


// ------------------------------------------------------------------------------------
// Element matrices of an order-1 coarse operator on the fine quadrature (24 x 24 per
// element): column j = (node b, component k) is the element response to the unit
// nodal vector e_j, i.e. the Jacobian pointwise map applied to the rank-one gradient
// e_k (grad_xi phi_b)^T and integrated against every test function.  Exactly the
// matrix-free coarse operator, stored densely (3.7x fewer bytes per apply than the
// fine-quadrature linearisation at Q = 5).
// ------------------------------------------------------------------------------------
constexpr int ELB = 8;  // elements per workgroup (8 x 24 = 192 threads)
constexpr int ELMAT_PACKED = 300;  // 24 x 25 / 2 entries of the symmetric element matrix
__device__ __forceinline__ constexpr int elmat_index(int r, int j) { return r * (47 - r) / 2 + j; }

// T: precision of the state, tables, arithmetic and result (FP32 for the mixed-precision
// preconditioner, FP64 otherwise).
template <typename T, int Q>
__global__ __launch_bounds__(ELB * 24) void k_elmat_build(const T *__restrict__ state,
                                                          const T *__restrict__ tab, double mu0,
                                                          double lam0, const double *__restrict__ mu_e,
                                                          const double *__restrict__ lam_e,
                                                          T *__restrict__ K, int64_t E) {
  constexpr int Q3 = Q * Q * Q, ET = QT<Q>::ET, NQ = QT<Q>::NQ;
  __shared__ T sB[Q * 2], sG[Q * 2];
  const int t = threadIdx.x, el = t / 24, j = t % 24;
  const int64_t e = (int64_t)blockIdx.x * ELB + el;
  if (t < 2 * Q) {
    sB[t] = tab[TAB_B + t];
    sG[t] = tab[TAB_G + t];
  }
  __syncthreads();
  if (e >= E) return;
  const int b = j / 3, k = j % 3, b1 = b & 1, b2 = (b >> 1) & 1, b3 = b >> 2;
  const T mu = (T)mat_mu(mu0, mu_e, e), lam = (T)mat_mu(lam0, lam_e, e);
  const T *s = state + ((e / ET) * NSTATE) * NQ + (e % ET) * Q3;
  T acc[24];
#pragma unroll
  for (int r = 0; r < 24; ++r) acc[r] = T(0);
  for (int q = 0; q < Q3; ++q) {
    const int q1 = q % Q, q2 = (q / Q) % Q, q3 = q / (Q * Q);
    T A[3][3], tau[6];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int jj = 0; jj < 3; ++jj) A[a][jj] = s[(a * 3 + jj) * NQ + q];
#pragma unroll
    for (int m = 0; m < 6; ++m) tau[m] = s[(9 + m) * NQ + q];
    const T c = s[15 * NQ + q], W = T(1);  // the weight is in the scaled dxi/dx
    // reference gradient of basis b at q
    const T Bx = sB[q1 * 2 + b1], By = sB[q2 * 2 + b2], Bz = sB[q3 * 2 + b3];
    const T Gx = sG[q1 * 2 + b1], Gy = sG[q2 * 2 + b2], Gz = sG[q3 * 2 + b3];
    const T dp[3] = {Gx * By * Bz, Bx * Gy * Bz, Bx * By * Gz};
    T v[3], w[3];
#pragma unroll
    for (int jj = 0; jj < 3; ++jj) v[jj] = dp[0] * A[0][jj] + dp[1] * A[1][jj] + dp[2] * A[2][jj];
#pragma unroll
    for (int jj = 0; jj < 3; ++jj)
      w[jj] = v[0] * tau[sym_index(0, jj)] + v[1] * tau[sym_index(1, jj)] + v[2] * tau[sym_index(2, jj)];
    // s = g tau + lambda tr(g) I + (mu - c)(g + g^T), g = e_k v^T
    T sm[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int jj = 0; jj < 3; ++jj) {
        T val = (i == k ? w[jj] + (mu - c) * v[jj] : T(0)) + (jj == k ? (mu - c) * v[i] : T(0));
        if (i == jj) val += lam * v[k];
        sm[i][jj] = val;
      }
    T f[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int d = 0; d < 3; ++d) f[i][d] = W * (sm[i][0] * A[d][0] + sm[i][1] * A[d][1] + sm[i][2] * A[d][2]);
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      const int a1 = a & 1, a2 = (a >> 1) & 1, a3 = a >> 2;
      const T ax = sB[q1 * 2 + a1], ay = sB[q2 * 2 + a2], az = sB[q3 * 2 + a3];
      const T gx = sG[q1 * 2 + a1], gy = sG[q2 * 2 + a2], gz = sG[q3 * 2 + a3];
      const T d0 = gx * ay * az, d1 = ax * gy * az, d2 = ax * ay * gz;
#pragma unroll
      for (int i = 0; i < 3; ++i) acc[a * 3 + i] += d0 * f[i][0] + d1 * f[i][1] + d2 * f[i][2];
    }
  }
  // The matrix is symmetric: store its upper triangle, row-major (entry (r, j), r <= j,
  // at r (47 - r) / 2 + j); column j supplies rows r <= j.
  T *out = K + (int64_t)e * ELMAT_PACKED;
#pragma unroll
  for (int r = 0; r < 24; ++r)
    if (r <= j) out[elmat_index(r, j)] = acc[r];
}

// y_e = K_e x_e for order-1 elements (records for the node-centric assembly).  The
// workgroup's packed matrices (8 x 300 contiguous values) are staged through LDS with
// coalesced loads; thread r then forms row r from the triangle.
template <typename T>
__global__ __launch_bounds__(ELB * 24) void k_elmat_apply(const uint32_t *__restrict__ emap,
                                                          const T *__restrict__ K, const T *__restrict__ x,
                                                          T *__restrict__ ev, int64_t E,
                                                          const double *__restrict__ stop) {
  if (stop && *stop != 0.0) return;  // a stopped PCG (uniform over the grid)
  __shared__ T sx[ELB * 24];
  __shared__ T sK[ELB * ELMAT_PACKED];
  const int t = threadIdx.x, el = t / 24, r = t % 24;
  const int64_t e0 = (int64_t)blockIdx.x * ELB, e = e0 + el;
  const bool live = e < E;
  const int64_t nel = (E - e0) < ELB ? (E - e0) : ELB;
  const T *Kb = K + e0 * ELMAT_PACKED;
  for (int i = t; i < nel * ELMAT_PACKED; i += ELB * 24) sK[i] = Kb[i];
  if (live) {
    const uint32_t w = emap[e * 8 + r / 3];
    const int c = r % 3;
    sx[t] = ((w >> (EMAP_BC_SHIFT + c)) & 1u) ? T(0) : x[(int64_t)(w & EMAP_ID_MASK) * 3 + c];
  }
  __syncthreads();
  if (!live) return;
  const T *Ke = sK + el * ELMAT_PACKED;
  const T *xe = sx + el * 24;
  T acc = 0;
#pragma unroll
  for (int jj = 0; jj < 24; ++jj) acc += Ke[jj < r ? elmat_index(jj, r) : elmat_index(r, jj)] * xe[jj];
  ev[e * 24 + r] = acc;
}

// The order-1 operator assembled into 3 x 3 node blocks, sliced ELL by slot (column
// node cols[j][n], -1 - n past the row's end: a zero block; entry (i, k) at
// vals[j][3 i + k][n] when node_major (each entry of a slot's blocks contiguous over the
// nodes, for a thread per node), else at vals[j][n][3 i + k] (a node's three rows
// contiguous, for a thread per row)).  One
// thread per (slot, row node) sums the block over the elements that hold both nodes,
// in the row node's incidence order (so the result is reproducible), in double, and
// masks it like the matrix-free apply: constrained columns are zero, constrained rows
// identity rows.
template <typename T>
__global__ __launch_bounds__(256) void k_ell_build(bool node_major, int64_t nn, int W, const int32_t *__restrict__ cols,
                                                   const int32_t *__restrict__ off, const int32_t *__restrict__ inc,
                                                   const uint32_t *__restrict__ emap, const T *__restrict__ K,
                                                   T *__restrict__ vals) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)W * nn) return;
  const int j = (int)(t / nn);
  const int64_t n = t - (int64_t)j * nn;
  const int32_t c = cols[t];
  // entry m of this block at blk[m * ms]
  T *blk = node_major ? vals + (int64_t)j * 9 * nn + n : vals + t * 9;
  const int64_t ms = node_major ? nn : 1;
  if (c < 0) {  // padding: a zero block
#pragma unroll
    for (int m = 0; m < 9; ++m) blk[m * ms] = T(0);
    return;
  }
  double a[9];
#pragma unroll
  for (int m = 0; m < 9; ++m) a[m] = 0.0;
  uint32_t rbc = 0, cbc = 0;
  for (int32_t k = off[n]; k < off[n + 1]; ++k) {
    const int32_t rec = inc[k];
    const int64_t e = rec / 8;
    const int la = rec % 8;
    rbc = (emap[rec] >> EMAP_BC_SHIFT) & 7u;
    const T *Ke = K + e * ELMAT_PACKED;
    for (int lb = 0; lb < 8; ++lb) {
      const uint32_t wb = emap[e * 8 + lb];
      if ((int32_t)(wb & EMAP_ID_MASK) != c) continue;
      cbc = (wb >> EMAP_BC_SHIFT) & 7u;
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int kk = 0; kk < 3; ++kk) {
          const int r = la * 3 + i, q = lb * 3 + kk;
          a[i * 3 + kk] += (double)Ke[r <= q ? elmat_index(r, q) : elmat_index(q, r)];
        }
    }
  }
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int kk = 0; kk < 3; ++kk) {
      double v = ((cbc >> kk) & 1u) ? 0.0 : a[i * 3 + kk];
      if ((rbc >> i) & 1u) v = (c == n && i == kk) ? 1.0 : 0.0;
      blk[(i * 3 + kk) * ms] = (T)v;
    }
}

// ------------------------------------------------------------------------------------
// a11: p-transfer on the same elements (eq. mg_prolong).
// Both directions by line tasks (as in k_jacobian_lines) over frames of P_f^3 values per
// component.  With one thread per fine node and stage, index arithmetic and LDS reads bound
// them: 39 us (prolongation) and 27 us (restriction) for Q2 <-> Q4 on 34^3 elements in
// FP32, against 31 and 23 by lines; two tiles a workgroup (their dependent loads in flight
// together) take the pair with its assembly from 80 to 70.5 us, four to 67 there but Q2 <-> Q1
// on 43^3 elements from 31 back to 33.
// ------------------------------------------------------------------------------------
// Elements of a transfer workgroup, and the fine nodes of a thread.
constexpr int TR_TILES = 2;
template <int PF>
struct TR {
  static constexpr int ET = TR_TILES * QT<PF>::ET, NT = QT<PF>::NT, IT = (ET * PF * PF * PF + NT - 1) / NT;
};

template <typename T, int PF, int PC>
__global__ __launch_bounds__(TR<PF>::NT) void k_prolong_add(
    const uint32_t *__restrict__ emap_c, const uint32_t *__restrict__ emap_f, const T *__restrict__ xc,
    const T *__restrict__ tab_c, T *__restrict__ yf, int64_t E) {
  constexpr int F3 = PF * PF * PF, C3 = PC * PC * PC, ET = TR<PF>::ET, NT = TR<PF>::NT, IT = TR<PF>::IT, ELS = 3 * F3;
  __shared__ T lds[ET * ELS];
  const int tq = threadIdx.x;
  const int64_t e0 = xcd_tile() * ET;
  const int nel = (int)((E - e0) < ET ? (E - e0) : ET);
  const T *M = tab_c + tab_ctof(PF);
  // Every element sharing a fine node interpolates the same value there (the coarse
  // field is continuous); the node's owner element adds it.  No atomics, and the
  // result does not depend on the order in which workgroups run.
  uint32_t wf[IT];
#pragma unroll
  for (int k = 0; k < IT; ++k) wf[k] = tq + k * NT < nel * F3 ? emap_f[e0 * F3 + tq + k * NT] : 0u;
  for (int t = tq; t < nel * C3; t += NT) {
    const int te = t / C3, a = t % C3;
    gather_node(xc, emap_c[e0 * C3 + t], true, lds + te * ELS,
                (a % PC) + PF * ((a / PC) % PC) + PF * PF * (a / (PC * PC)), F3);
  }
  T y[IT][3];
#pragma unroll
  for (int k = 0; k < IT; ++k) {
    const T *p = yf + (int64_t)(wf[k] & EMAP_ID_MASK) * 3;
#pragma unroll
    for (int c = 0; c < 3; ++c) y[k][c] = (wf[k] & EMAP_OWNER) ? p[c] : T(0);
  }
  __syncthreads();
  line_stage<T, PF, 0, PC, PF, false, PC, PC, ET, ELS>(lds, M, tq, NT, nel);
  __syncthreads();
  line_stage<T, PF, 1, PC, PF, false, PF, PC, ET, ELS>(lds, M, tq, NT, nel);
  __syncthreads();
  line_stage<T, PF, 2, PC, PF, false, PF, PF, ET, ELS>(lds, M, tq, NT, nel);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < IT; ++k)
    if (wf[k] & EMAP_OWNER) {
      const int t = tq + k * NT;
      const T *v = lds + t / F3 * ELS + t % F3;
      T *p = yf + (int64_t)(wf[k] & EMAP_ID_MASK) * 3;
#pragma unroll
      for (int c = 0; c < 3; ++c)
        if (!((wf[k] >> (EMAP_BC_SHIFT + c)) & 1u)) p[c] = y[k][c] + v[c * F3];
    }
}

template <typename T, int PF, int PC>
__global__ __launch_bounds__(TR<PF>::NT) void k_restrict(
    const uint32_t *__restrict__ emap_f, const T *__restrict__ rf, const T *__restrict__ tab_c,
    T *__restrict__ ev_c, int64_t E) {
  constexpr int F3 = PF * PF * PF, C3 = PC * PC * PC, ET = TR<PF>::ET, NT = TR<PF>::NT, IT = TR<PF>::IT, ELS = 3 * F3;
  __shared__ T lds[ET * ELS];
  const int tq = threadIdx.x;
  const int64_t e0 = xcd_tile() * ET;
  const int nel = (int)((E - e0) < ET ? (E - e0) : ET);
  const T *M = tab_c + tab_ctof(PF);
  // Transpose of the owner-written prolongation: each fine node's value enters
  // through its owner element only.
  uint32_t w[IT];
  T x[IT][3];
#pragma unroll
  for (int k = 0; k < IT; ++k) w[k] = tq + k * NT < nel * F3 ? emap_f[e0 * F3 + tq + k * NT] : 0u;
#pragma unroll
  for (int k = 0; k < IT; ++k) {
    const T *p = rf + (int64_t)(w[k] & EMAP_ID_MASK) * 3;
#pragma unroll
    for (int c = 0; c < 3; ++c)
      x[k][c] = (w[k] & EMAP_OWNER) && !((w[k] >> (EMAP_BC_SHIFT + c)) & 1u) ? p[c] : T(0);
  }
#pragma unroll
  for (int k = 0; k < IT; ++k) {
    const int t = tq + k * NT;
    if (t < nel * F3)
#pragma unroll
      for (int c = 0; c < 3; ++c) lds[t / F3 * ELS + c * F3 + t % F3] = x[k][c];
  }
  __syncthreads();
  line_stage<T, PF, 2, PF, PC, true, PF, PF, ET, ELS>(lds, M, tq, NT, nel);
  __syncthreads();
  line_stage<T, PF, 1, PF, PC, true, PF, PC, ET, ELS>(lds, M, tq, NT, nel);
  __syncthreads();
  line_stage<T, PF, 0, PF, PC, true, PC, PC, ET, ELS>(lds, M, tq, NT, nel);
  __syncthreads();
  // records [e][a][c] of the workgroup's elements: one contiguous run
  for (int d = tq; d < nel * C3 * 3; d += NT) {
    const int r = d / 3, c = d - 3 * r, te = r / C3, a = r - te * C3;
    ev_c[e0 * (C3 * 3) + d] = lds[te * ELS + c * F3 + (a % PC) + PF * ((a / PC) % PC) + PF * PF * (a / (PC * PC))];
  }
}

// ------------------------------------------------------------------------------------
// Strain energy per element (deterministic serial sum over the element's points).
// ------------------------------------------------------------------------------------
template <int P, int Q>
__global__ __launch_bounds__(QT<Q>::NT) void k_energy(const uint32_t *__restrict__ emap,
                                                      const double *__restrict__ u,
                                                      const double *__restrict__ geo,
                                                      const double *__restrict__ tab, double mu0,
                                                      double lam0, const double *__restrict__ mu_e,
                                                      const double *__restrict__ lam_e,
                                                      double *__restrict__ out, int64_t E) {
  using T = double;
  constexpr int Q3 = QT<Q>::Q3, ET = QT<Q>::ET, NQ = QT<Q>::NQ, NT = QT<Q>::NT, P3 = P * P * P;
  constexpr int S0 = 3 * Q3, S1 = 3 * Q3;
  __shared__ T sB[Q * P], sD[Q * Q];
  __shared__ T lds[ET * (S0 + S1)];
  const int tq = threadIdx.x, el = tq / Q3, q = tq % Q3;
  const int64_t tile = xcd_tile();
  const int64_t e = tile * ET + el;
  const bool live = tq < ET * Q3 && e < E;
  load_tables(sB, tab, TAB_B, Q * P, tq, NT);
  load_tables(sD, tab, TAB_D, Q * Q, tq, NT);
  T *a = lds + (live ? el : 0) * S0, *b = lds + ET * S0 + (live ? el : 0) * S1;
  if (live && q < P3) {
    const uint32_t node = emap[e * P3 + q] & EMAP_ID_MASK;
#pragma unroll
    for (int c = 0; c < 3; ++c) a[c * P3 + q] = u[(int64_t)node * 3 + c];
  }
  __syncthreads();
  interp<T, P, Q, 3>(a, b, sB, q, live);
  T psi = 0;
  if (live) {
    T G[3][3], D[3][3];
    grad_q<T, Q, 3>(b, sD, q, G);
    const double *g = geo + tile * NGEO * NQ + tq;
    const T W = g[0];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int J = 0; J < 3; ++J) D[k][J] = g[(1 + k * 3 + J) * NQ];
    const T mu = mat_mu(mu0, mu_e, e), lam = mat_mu(lam0, lam_e, e);
    Kin<T> k;
    kinematics(G, D, mu, lam, k);
    T tre = 0;
    for (int i = 0; i < 3; ++i) {
      tre += k.H[i][i];
      for (int j = 0; j < 3; ++j) tre += 0.5 * k.H[i][j] * k.H[i][j];
    }
    psi = W * (0.5 * lam * k.logJ * k.logJ - mu * k.logJ + mu * tre);
  }
  __syncthreads();
  if (live) a[q] = psi;
  __syncthreads();
  if (live && q == 0) {
    T s = 0;
    for (int i = 0; i < Q3; ++i) s += a[i];
    out[e] = s;
  }
}

// Geometric factors out of the tiled layout into [E][10][Q^3].
template <int Q>
__global__ void k_export_geo(const double *__restrict__ geo, double *__restrict__ out, int64_t E) {
  constexpr int Q3 = QT<Q>::Q3, ET = QT<Q>::ET, NQ = QT<Q>::NQ;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = E * NGEO * Q3;
  if (i >= total) return;
  const int64_t e = i / (NGEO * Q3);
  const int f = (int)((i / Q3) % NGEO), q = (int)(i % Q3);
  const int64_t tile = e / ET;
  const int el = (int)(e % ET);
  out[i] = geo[(tile * NGEO + f) * NQ + el * Q3 + q];
}

// Internal element map with Dirichlet bits.
__global__ void k_build_emap(const int32_t *__restrict__ en, const uint8_t *__restrict__ mask,
                             uint32_t *__restrict__ emap, int64_t n, int64_t N,
                             unsigned *__restrict__ flags) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int32_t node = en[i];
  if (node < 0 || node >= N) {
    atomicOr(flags, 4u);
    emap[i] = 0;
    return;
  }
  uint32_t w = (uint32_t)node;
  if (mask) {
    for (int c = 0; c < 3; ++c)
      if (mask[(int64_t)node * 3 + c]) w |= 1u << (EMAP_BC_SHIFT + c);
  }
  emap[i] = w;
}

// Sum of node n's element records in the fixed order of its incidence list, the loads of
// four records in flight together: one at a time, Q2 applies on 43^3 elements took 84.6 us
// in FP64 and 49.2 in FP32 against 81.2 and 45.7, Q4 on 34^3 208 and 118.5 against 203 and 117
// (operators in turn).
template <typename T>
__device__ __forceinline__ void node_sum(const int32_t *__restrict__ off, const int32_t *__restrict__ inc,
                                         const T *__restrict__ ev, int64_t n, T (&a)[3]) {
  const int32_t k0 = off[n], k1 = off[n + 1];
  a[0] = a[1] = a[2] = T(0);
  for (int32_t k = k0; k < k1; k += 4) {
    T v[4][3];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const T *p = ev + (int64_t)inc[k + j < k1 ? k + j : k] * 3;
#pragma unroll
      for (int c = 0; c < 3; ++c) v[j][c] = p[c];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (k + j < k1)
#pragma unroll
        for (int c = 0; c < 3; ++c) a[c] += v[j][c];
  }
}

// Node-centric assembly: y[n] = sum of the node's element records, in the fixed order
// of its incidence list; constrained components take `src` (or zero).
template <typename T>
__global__ __launch_bounds__(256) void k_assemble(int64_t N, const int32_t *__restrict__ off,
                                                  const int32_t *__restrict__ inc, const T *__restrict__ ev,
                                                  const uint8_t *__restrict__ mask, const T *__restrict__ src,
                                                  T fill, T *__restrict__ y) {
  // One node per thread; consecutive node ranges stay on one XCD (see xcd_tile), so
  // the records of neighbouring nodes, which share elements, meet in the same L2.
  const int64_t n = xcd_tile() * blockDim.x + threadIdx.x;
  if (n < N) {
    T a[3];
    node_sum(off, inc, ev, n, a);
    T *o = y + n * 3;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (mask && mask[n * 3 + c]) a[c] = src ? src[n * 3 + c] : fill;
      o[c] = a[c];
    }
  }
}

// The same node sums with the output staged in LDS and written by the workgroup in
// contiguous nontemporal sweeps (256 consecutive nodes = 768 consecutive values), so
// every store instruction covers whole cache lines.
template <typename T>
__global__ __launch_bounds__(256) void k_assemble_staged(int64_t N, const int32_t *__restrict__ off,
                                                         const int32_t *__restrict__ inc, const T *__restrict__ ev,
                                                         const uint8_t *__restrict__ mask, const T *__restrict__ src,
                                                         T fill, T *__restrict__ y) {
  __shared__ T buf[3 * 256];
  // consecutive node ranges stay on one XCD (see xcd_tile): neighbouring nodes share
  // elements, so their records meet in the same L2
  const int64_t n0 = xcd_tile() * 256, n = n0 + threadIdx.x;
  if (n < N) {
    T a[3];
    node_sum(off, inc, ev, n, a);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (mask && mask[n * 3 + c]) a[c] = src ? src[n * 3 + c] : fill;
      buf[3 * threadIdx.x + c] = a[c];
    }
  }
  __syncthreads();
  const int nv = 3 * (int)((N - n0) < 256 ? (N - n0) : 256);
  T *o = y + n0 * 3;
  for (int d = threadIdx.x; d < nv; d += 256) __builtin_nontemporal_store(buf[d], o + d);
}

// The same node sums (A in, in itself on constrained components) finished as a step of the
// Chebyshev smoother instead of being stored, so that A in is neither written nor read
// again and a launch falls away (a V-cycle on 20^3 Q4 elements, one right-hand side, 1085 ->
// 979 us in FP64 and 820 -> 750 in FP32, node_sum's four-wide loads included):
//   SMOOTH_STEP:  in = d: r -= D^-1 A d; d = c1 d + c2 r; x += d
//   SMOOTH_FIRST: in = x: r = D^-1 (b - A x); d = c1 r; x += d
//   SMOOTH_RESIDUAL: in = x: r = b - A x
//   SMOOTH_START: the sums are a restricted residual, 0 on constrained components:
//     b = sums, r = D^-1 b; d = c1 r; x = d (the first step from x = 0)
// The vectors are read and written in contiguous sweeps of 768 values; their loads go out
// before the sums.
template <typename T, int KIND>
__global__ __launch_bounds__(256) void k_assemble_smooth(int64_t N, const int32_t *__restrict__ off,
                                                         const int32_t *__restrict__ inc, const T *__restrict__ ev,
                                                         const uint8_t *__restrict__ mask, Smooth sm) {
  __shared__ T buf[3 * 256];
  const int64_t n0 = xcd_tile() * 256, n = n0 + threadIdx.x;
  const int nv = 3 * (int)((N - n0) < 256 ? (N - n0) : 256);
  T *r = (T *)sm.r + n0 * 3, *d = (T *)sm.d + n0 * 3, *x = (T *)sm.x + n0 * 3;
  T *b = (T *)sm.b + n0 * 3;
  const T *dinv = (const T *)sm.dinv + n0 * 3;
  const T c1 = (T)sm.c1, c2 = (T)sm.c2;
  constexpr bool STEP = KIND == SMOOTH_STEP, START = KIND == SMOOTH_START;
  T vd[3], vx[3], vr[3], vi[3];
  bool fixed[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int i = threadIdx.x + 256 * j;
    const bool in = i < nv;
    fixed[j] = in && mask && mask[n0 * 3 + i];
    vd[j] = in && STEP ? d[i] : T(0);
    vx[j] = in && !START ? x[i] : T(0);
    vr[j] = in && !START ? (STEP ? r[i] : b[i]) : T(0);
    vi[j] = in && KIND != SMOOTH_RESIDUAL ? dinv[i] : T(0);
  }
  if (n < N) {
    T a[3];
    node_sum(off, inc, ev, n, a);
#pragma unroll
    for (int c = 0; c < 3; ++c) buf[3 * threadIdx.x + c] = a[c];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int i = threadIdx.x + 256 * j;
    if (i >= nv) continue;
    const T A = fixed[j] ? (STEP ? vd[j] : vx[j]) : buf[i];  // START: 0 where constrained
    if constexpr (START) {
      const T ri = vi[j] * A, di = ri * c1;
      b[i] = A;
      r[i] = ri;
      d[i] = di;
      x[i] = di;
    } else if constexpr (KIND == SMOOTH_RESIDUAL) {
      r[i] = vr[j] - A;
    } else {
      const T ri = STEP ? fma_t(-vi[j], A, vr[j]) : vi[j] * (vr[j] - A);
      const T di = STEP ? fma_t(c1, vd[j], c2 * ri) : ri * c1;
      r[i] = ri;
      d[i] = di;
      x[i] = add_rounded(vx[j], di);
    }
  }
}

// The same assembly fused with the partial dot product p . y of the assembled result
// and the direction p (= src), one partial per workgroup (fixed tree): the Jacobi-PCG
// step needs p^T A p right after A p.
template <typename T>
__global__ __launch_bounds__(256) void k_assemble_dot(int64_t N, const int32_t *__restrict__ off,
                                                      const int32_t *__restrict__ inc, const T *__restrict__ ev,
                                                      const uint8_t *__restrict__ mask, const T *__restrict__ src,
                                                      T *__restrict__ y, double *__restrict__ partial,
                                                      const double *__restrict__ stop) {
  if (stop && *stop != 0.0) return;  // a stopped PCG (uniform over the grid)
  __shared__ double red[256];
  const int64_t tile = xcd_tile();
  const int64_t n = tile * blockDim.x + threadIdx.x;
  double pq = 0.0;
  if (n < N) {
    T a[3];
    node_sum(off, inc, ev, n, a);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (mask && mask[n * 3 + c]) a[c] = src[n * 3 + c];
      y[n * 3 + c] = a[c];
      pq += (double)src[n * 3 + c] * (double)a[c];
    }
  }
  red[threadIdx.x] = pq;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < (unsigned)w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[tile] = red[0];
}

inline unsigned grid1d(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// y = assembled element records of `op`; constrained components take src (or `fill`)
// unless they are to be kept (masked = false).
template <typename T>
hipError_t assemble(const hpmg_op_s &op, const T *src, T *y, hipStream_t s, T fill = T(0), bool masked = true) {
  const uint8_t *mask = masked ? op.mask : nullptr;
  int64_t g = (op.N + 255) / 256;
  if (g < 1) g = 1;
  if (sweep_records<T>(op.P))
    k_assemble_staged<T><<<(unsigned)g, 256, 0, s>>>(op.N, op.csr_off, op.csr_inc, (const T *)op.evec, mask, src,
                                                      fill, y);
  else
    k_assemble<T><<<(unsigned)g, 256, 0, s>>>(op.N, op.csr_off, op.csr_inc, (const T *)op.evec, mask, src, fill,
                                               y);
  return hipGetLastError();
}

// The first record of every node (incidence lists are in record order) owns it.
__global__ void k_mark_owners(int64_t N, const int32_t *__restrict__ off, const int32_t *__restrict__ inc,
                              uint32_t *__restrict__ emap) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n < N && off[n] < off[n + 1]) emap[inc[off[n]]] |= EMAP_OWNER;
}

// ------------------------------------------------------------------------------------
// (P, Q) dispatch.
// ------------------------------------------------------------------------------------
#define HPMG_PQ_LIST(X) \
  X(2, 2) X(2, 3) X(2, 4) X(2, 5) X(3, 3) X(3, 4) X(3, 5) X(4, 4) X(4, 5) X(5, 5) X(5, 6)

#define HPMG_PP_LIST(X) X(3, 2) X(4, 2) X(5, 2) X(4, 3) X(5, 3) X(5, 4)

}  // namespace

bool supported_pq(int P, int Q) {
#define X(p, q) if (P == p && Q == q) return true;
  HPMG_PQ_LIST(X)
#undef X
  return false;
}

static bool supported_pp(int Pf, int Pc) {
#define X(f, c) if (Pf == f && Pc == c) return true;
  HPMG_PP_LIST(X)
#undef X
  return false;
}

hipError_t launch_build_emap(const hpmg_op_s &op, hipStream_t s) {
  const int64_t n = op.E * op.P * op.P * op.P;
  k_build_emap<<<grid1d(n, 256), 256, 0, s>>>(op.elem_nodes, op.mask, op.emap, n, op.N, op.flags);
  return hipGetLastError();
}

hipError_t launch_mark_owners(const hpmg_op_s &op, hipStream_t s) {
  k_mark_owners<<<grid1d(op.N, 256), 256, 0, s>>>(op.N, op.csr_off, op.csr_inc, op.emap);
  return hipGetLastError();
}

hipError_t launch_qdata(const hpmg_op_s &op, const double *X, hipStream_t s) {
#define X(p, q)                                                                              \
  if (op.P == p && op.Q == q) {                                                              \
    k_qdata<p, q><<<(unsigned)op.tiles, QT<q>::NT, 0, s>>>(op.emap, X, op.tab64, op.geo, op.flags, op.E); \
    return hipGetLastError();                                                                \
  }
  HPMG_PQ_LIST(X)
#undef X
  return hipErrorInvalidValue;
}

// Residual: the element kernel writes element records, the node-centric assembly pass
// sums them (deterministic).
hipError_t launch_residual(const hpmg_op_s &op, const double *u, double *r, bool store, hipStream_t s) {
  const bool stream = store && stream_state(op.tiles, op.Q);
#define X(p, q)                                                                                  \
  if (op.P == p && op.Q == q) {                                                                  \
    const auto go = [&](auto mode) {                                                             \
      lines_launch<double, p, q, decltype(mode)::value>(                                         \
          (unsigned)op.tiles, s, keep_records<double>(op.E, p), op.emap, u, (const double *)nullptr, op.geo,      \
          (const double *)nullptr, op.tab64, op.mu, op.lam, op.mu_e, op.lam_e, (double *)op.evec, op.E,           \
          (const double *)nullptr, store ? op.state64 : nullptr, op.flags, (const double *)nullptr,               \
          (double *)nullptr, (double *)nullptr);                                                 \
    };                                                                                           \
    if (stream)                                                                                  \
      go(std::integral_constant<int, 8>());                                                      \
    else                                                                                         \
      go(std::integral_constant<int, 4>());                                                      \
    hipError_t e = hipGetLastError();                                                            \
    if (e != hipSuccess) return e;                                                               \
    return assemble<double>(op, nullptr, r, s);                                                  \
  }
  HPMG_PQ_LIST(X)
#undef X
  return hipErrorInvalidValue;
}

template <typename T, int P, int Q>
static hipError_t jacobian_pq(const hpmg_op_s &op, const hpmg_op_s &f, int mode, const double *u, const T *du,
                              T *ev, const double *stop, bool again, hipStream_t s) {
  const T *state = std::is_same<T, double>::value ? (const T *)f.state64 : (const T *)f.state32;
  const T *tab = std::is_same<T, double>::value ? (const T *)op.tab64 : (const T *)op.tab32;
  const bool keep = keep_records<T>(op.E, P);
  const unsigned g = (unsigned)op.tiles;
  if constexpr (std::is_same<T, double>::value) {
    if (mode == HPMG_INITIAL_NATIVE || mode == HPMG_INITIAL_TUNED || mode == HPMG_CURRENT_20) {
      if (mode == HPMG_INITIAL_NATIVE)
        lines_launch<T, P, Q, 1>(g, s, keep, op.emap, du, nullptr, op.geo, op.sinit, tab, op.mu, op.lam, op.mu_e,
                                 op.lam_e, ev, op.E, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
      else if (mode == HPMG_INITIAL_TUNED)
        lines_launch<T, P, Q, 2>(g, s, keep, op.emap, du, nullptr, op.geo, op.sinit, tab, op.mu, op.lam, op.mu_e,
                                 op.lam_e, ev, op.E, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
      else
        lines_launch<T, P, Q, 3>(g, s, keep, op.emap, du, nullptr, op.geo, op.sinit, tab, op.mu, op.lam, op.mu_e,
                                 op.lam_e, ev, op.E, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
      return hipGetLastError();
    }
  }
  if (mode == HPMG_STORED) {
    const auto go = [&](auto m) {
      lines_launch<T, P, Q, decltype(m)::value>(g, s, keep, op.emap, du, state, nullptr, nullptr, tab, f.mu, f.lam,
                                                f.mu_e, f.lam_e, ev, op.E, stop, nullptr, nullptr, nullptr, nullptr,
                                                nullptr);
    };
    if (again && keep_state<T>(op.tiles, Q))
      go(std::integral_constant<int, 9>());
    else
      go(std::integral_constant<int, 0>());
  } else {
    lines_launch<T, P, Q, 5>(g, s, keep, op.emap, du, (const T *)nullptr, op.geo, (const double *)nullptr, tab,
                             op.mu, op.lam, op.mu_e, op.lam_e, ev, op.E, (const double *)nullptr,
                             (double *)nullptr, (unsigned *)nullptr, u, (double *)nullptr, (double *)nullptr);
  }
  return hipGetLastError();
}

template <typename T>
static hipError_t assemble_smooth(const hpmg_op_s &op, const Smooth &sm, hipStream_t s) {
  const unsigned g = grid1d(op.N, 256);
  const T *ev = (const T *)op.evec;
  if (sm.kind == SMOOTH_STEP)
    k_assemble_smooth<T, SMOOTH_STEP><<<g, 256, 0, s>>>(op.N, op.csr_off, op.csr_inc, ev, op.mask, sm);
  else if (sm.kind == SMOOTH_FIRST)
    k_assemble_smooth<T, SMOOTH_FIRST><<<g, 256, 0, s>>>(op.N, op.csr_off, op.csr_inc, ev, op.mask, sm);
  else if (sm.kind == SMOOTH_RESIDUAL)
    k_assemble_smooth<T, SMOOTH_RESIDUAL><<<g, 256, 0, s>>>(op.N, op.csr_off, op.csr_inc, ev, op.mask, sm);
  else
    k_assemble_smooth<T, SMOOTH_START><<<g, 256, 0, s>>>(op.N, op.csr_off, op.csr_inc, ev, op.mask, sm);
  return hipGetLastError();
}

// What follows the element records of an apply: a smoother step (sm), or y with (pq) or
// without the per-workgroup partials of du . y.
template <typename T>
struct Finish {
  T *y = nullptr;
  double *pq = nullptr;
  const double *stop = nullptr;
  const Smooth *sm = nullptr;
};
template <typename T>
static hipError_t finish_apply(const hpmg_op_s &op, const T *du, const Finish<T> &f, hipStream_t s) {
  if (f.sm) return assemble_smooth<T>(op, *f.sm, s);
  if (!f.pq) return assemble<T>(op, du, f.y, s);
  k_assemble_dot<T><<<grid1d(op.N, 256), 256, 0, s>>>(op.N, op.csr_off, op.csr_inc, (const T *)op.evec, op.mask,
                                                      du, f.y, f.pq, f.stop);
  return hipGetLastError();
}

// pq set: the assembly also writes per-workgroup partials of du . y (ceil(N / 256)).
// stop set: the stored-mode kernels return at once while *stop != 0.
template <typename T>
static hipError_t jacobian_t(const hpmg_op_s &op, int mode, const double *u, const T *du, const Finish<T> &fin,
                             hipStream_t s) {
  const hpmg_op_s &f = op.fine ? *op.fine : op;
  T *ev = (T *)op.evec;
  const int tprec = std::is_same<T, double>::value ? HPMG_F64 : HPMG_F32;
  if (mode == HPMG_STORED && op.P == 2 && op.elmat && op.elmat_prec == tprec &&
      op.elmat_version == f.state_version) {
    k_elmat_apply<T><<<grid1d(op.E, ELB), ELB * 24, 0, s>>>(op.emap, (const T *)op.elmat, du, ev, op.E, fin.stop);
    hipError_t e2 = hipGetLastError();
    if (e2 != hipSuccess) return e2;
    return finish_apply<T>(op, du, fin, s);
  }
  hipError_t e = hipErrorInvalidValue;
#define X(p, q) \
  if (op.P == p && op.Q == q) e = jacobian_pq<T, p, q>(op, f, mode, u, du, ev, fin.stop, fin.sm || fin.pq, s);
  HPMG_PQ_LIST(X)
#undef X
  if (e != hipSuccess) return e;
  return finish_apply<T>(op, du, fin, s);
}

template <typename T>
static hipError_t jacobian_dot_t(const hpmg_op_s &op, const void *du, void *y, double *pq, const double *stop,
                                 hipStream_t s) {
  Finish<T> f;
  f.y = (T *)y;
  f.pq = pq;
  f.stop = stop;
  return jacobian_t<T>(op, HPMG_STORED, nullptr, (const T *)du, f, s);
}

hipError_t launch_jacobian_dot(const hpmg_op_s &op, int prec, const void *du, void *y, double *pq,
                               const double *stop, hipStream_t s) {
  return prec == HPMG_F64 ? jacobian_dot_t<double>(op, du, y, pq, stop, s)
                          : jacobian_dot_t<float>(op, du, y, pq, stop, s);
}

template <typename T>
static hipError_t jacobian_smooth_t(const hpmg_op_s &op, const Smooth &sm, hipStream_t s) {
  Finish<T> f;
  f.sm = &sm;
  return jacobian_t<T>(op, HPMG_STORED, nullptr, (const T *)(sm.kind == SMOOTH_STEP ? sm.d : sm.x), f, s);
}

hipError_t launch_jacobian_smooth(const hpmg_op_s &op, int prec, const Smooth &sm, hipStream_t s) {
  return prec == HPMG_F64 ? jacobian_smooth_t<double>(op, sm, s) : jacobian_smooth_t<float>(op, sm, s);
}

template <typename T>
static hipError_t jacobian_apply_t(const hpmg_op_s &op, int mode, const double *u, const void *du, void *y,
                                   hipStream_t s) {
  Finish<T> f;
  f.y = (T *)y;
  return jacobian_t<T>(op, mode, u, (const T *)du, f, s);
}

hipError_t launch_jacobian(const hpmg_op_s &op, int prec, int mode, const double *u, const void *du,
                           void *y, hipStream_t s) {
  return prec == HPMG_F64 ? jacobian_apply_t<double>(op, mode, u, du, y, s)
                          : jacobian_apply_t<float>(op, mode, u, du, y, s);
}

template <typename T, int P, int Q>
static void diagonal_launch(const hpmg_op_s &op, const hpmg_op_s &f, const T *state, const T *tab, hipStream_t s) {
  const unsigned g = (unsigned)op.tiles;
  T *ev = (T *)op.evec;
  if constexpr (sweep_records<T>(P)) {
    if (keep_records<T>(op.E, P))
      k_diagonal<T, P, Q, 1><<<g, QT<Q>::NT, 0, s>>>(state, tab, f.mu, f.lam, f.mu_e, f.lam_e, ev, op.E);
    else
      k_diagonal<T, P, Q, 2><<<g, QT<Q>::NT, 0, s>>>(state, tab, f.mu, f.lam, f.mu_e, f.lam_e, ev, op.E);
  } else {
    k_diagonal<T, P, Q, 0><<<g, QT<Q>::NT, 0, s>>>(state, tab, f.mu, f.lam, f.mu_e, f.lam_e, ev, op.E);
  }
}

hipError_t launch_diagonal(const hpmg_op_s &op, int prec, void *diag, hipStream_t s) {
  const hpmg_op_s &f = op.fine ? *op.fine : op;
#define X(p, q)                                                                 \
  if (op.P == p && op.Q == q) {                                                 \
    if (prec == HPMG_F64)                                                       \
      diagonal_launch<double, p, q>(op, f, f.state64, op.tab64, s);             \
    else                                                                        \
      diagonal_launch<float, p, q>(op, f, f.state32, op.tab32, s);              \
    hipError_t e = hipGetLastError();                                           \
    if (e != hipSuccess) return e;                                              \
    return prec == HPMG_F64 ? assemble<double>(op, nullptr, (double *)diag, s, 1.0) \
                            : assemble<float>(op, nullptr, (float *)diag, s, 1.0f); \
  }
  HPMG_PQ_LIST(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_prolong_add(const hpmg_op_s &c, const hpmg_op_s &f, int prec, const void *xc, void *yf,
                              hipStream_t s) {
  const unsigned grid = grid1d(f.E, TR_TILES * elems_per_tile(f.P));
#define X(pf, pc)                                                                                     \
  if (f.P == pf && c.P == pc) {                                                                       \
    if (prec == HPMG_F64)                                                                             \
      k_prolong_add<double, pf, pc><<<grid, TR<pf>::NT, 0, s>>>(c.emap, f.emap, (const double *)xc,    \
                                                                c.tab64, (double *)yf, f.E);          \
    else                                                                                              \
      k_prolong_add<float, pf, pc><<<grid, TR<pf>::NT, 0, s>>>(c.emap, f.emap, (const float *)xc,      \
                                                               c.tab32, (float *)yf, f.E);            \
    return hipGetLastError();                                                                         \
  }
  HPMG_PP_LIST(X)
#undef X
  (void)supported_pp;
  return hipErrorInvalidValue;
}

template <typename T, int PF, int PC>
static hipError_t restrict_t(const hpmg_op_s &f, const hpmg_op_s &c, const void *rf, const T *tab, void *rc,
                             const Smooth *start, hipStream_t s) {
  const unsigned grid = grid1d(f.E, TR<PF>::ET);
  k_restrict<T, PF, PC><<<grid, TR<PF>::NT, 0, s>>>(f.emap, (const T *)rf, tab, (T *)c.evec, f.E);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return start ? assemble_smooth<T>(c, *start, s) : assemble<T>(c, nullptr, (T *)rc, s);
}

hipError_t launch_restrict(const hpmg_op_s &f, const hpmg_op_s &c, int prec, const void *rf, void *rc,
                           hipStream_t s, const Smooth *start) {
#define X(pf, pc)                                                                                \
  if (f.P == pf && c.P == pc)                                                                    \
    return prec == HPMG_F64 ? restrict_t<double, pf, pc>(f, c, rf, c.tab64, rc, start, s)        \
                            : restrict_t<float, pf, pc>(f, c, rf, c.tab32, rc, start, s);
  HPMG_PP_LIST(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_energy(const hpmg_op_s &op, const double *u, double *psi, hipStream_t s) {
#define X(p, q)                                                                                  \
  if (op.P == p && op.Q == q) {                                                                  \
    k_energy<p, q><<<(unsigned)op.tiles, QT<q>::NT, 0, s>>>(op.emap, u, op.geo, op.tab64, op.mu, op.lam, \
                                                            op.mu_e, op.lam_e, op.scratch, op.E); \
    hipError_t e = hipGetLastError();                                                            \
    if (e != hipSuccess) return e;                                                               \
    return launch_sum(op.E, op.scratch, op.scratch + op.E, psi, s);                              \
  }
  HPMG_PQ_LIST(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_body_load(const hpmg_op_s &op, const double *g, double *f_ext, hipStream_t s) {
#define X(p, q)                                                                                      \
  if (op.P == p && op.Q == q) {                                                                      \
    k_body_load<p, q><<<(unsigned)op.tiles, QT<q>::NT, 0, s>>>(op.geo, op.tab64, g[0], g[1], g[2], op.evec, \
                                                               op.E);                                \
    hipError_t e = hipGetLastError();                                                                \
    return e != hipSuccess ? e : assemble<double>(op, nullptr, f_ext, s);                            \
  }
  HPMG_PQ_LIST(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_traction_load(const hpmg_op_s &op, const double *coords, int64_t nf, const int32_t *face_elem,
                                const int32_t *face_id, const double *t, double *rec, int32_t *rec_node,
                                hipStream_t s) {
#define X(p, q)                                                                                      \
  if (op.P == p && op.Q == q) {                                                                      \
    k_traction_load<p, q><<<grid1d(nf, 64), 64, 0, s>>>(coords, op.elem_nodes, face_elem, face_id,        \
                                                         op.tab64,                                    \
                                                         t[0], t[1], t[2], nf, op.E, rec, rec_node,   \
                                                         op.flags);                                  \
    return hipGetLastError();                                                                        \
  }
  HPMG_PQ_LIST(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_assemble_csr(int64_t N, const int32_t *off, const int32_t *inc, const double *rec,
                               const uint8_t *mask, double *y, hipStream_t s) {
  k_assemble<double><<<grid1d(N, 256), 256, 0, s>>>(N, off, inc, rec, mask, nullptr, 0.0, y);
  return hipGetLastError();
}

hipError_t launch_state_initial(const hpmg_op_s &op, const double *u, hipStream_t s) {
#define X(p, q)                                                                                      \
  if (op.P == p && op.Q == q) {                                                                      \
    k_state_initial<p, q><<<(unsigned)op.tiles, QT<q>::NT, 0, s>>>(op.emap, u, op.geo, op.tab64, op.mu, \
                                                                   op.lam, op.mu_e, op.lam_e, op.sinit, \
                                                                   op.flags, op.E);                  \
    return hipGetLastError();                                                                        \
  }
  HPMG_PQ_LIST(X)
#undef X
  return hipErrorInvalidValue;
}

template <typename T>
static hipError_t vjp_t(const hpmg_op_s &op, int mode, const double *u, const T *w, T *ub, double *mub,
                        double *lamb, hipStream_t s) {
  T *ev = (T *)op.evec;
  const T *state = std::is_same<T, double>::value ? (const T *)op.state64 : (const T *)op.state32;
  const T *tab = std::is_same<T, double>::value ? (const T *)op.tab64 : (const T *)op.tab32;
  const unsigned g = (unsigned)op.tiles;
#define X(p, q)                                                                                      \
  if (op.P == p && op.Q == q) {                                                                      \
    const bool keep = keep_records<T>(op.E, p);                                                      \
    if (mode == HPMG_STORED)                                                                         \
      lines_launch<T, p, q, 6>(g, s, keep, op.emap, w, state, op.geo, nullptr, tab, op.mu, op.lam,   \
                               op.mu_e, op.lam_e, ev, op.E, nullptr, nullptr, nullptr, u, mub, lamb); \
    else                                                                                             \
      lines_launch<T, p, q, 7>(g, s, keep, op.emap, w, nullptr, op.geo, nullptr, tab, op.mu, op.lam, \
                               op.mu_e, op.lam_e, ev, op.E, nullptr, nullptr, nullptr, u, mub, lamb); \
    hipError_t e = hipGetLastError();                                                                \
    if (e != hipSuccess) return e;                                                                   \
    /* unmasked assembly: constrained columns of u_bar are kept */                                   \
    return assemble<T>(op, nullptr, ub, s, T(0), false);                                             \
  }
  HPMG_PQ_LIST(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_vjp(const hpmg_op_s &op, int prec, int mode, const double *u, const void *w, void *ub,
                      double *mub, double *lamb, hipStream_t s) {
  if (prec == HPMG_F64) return vjp_t<double>(op, mode, u, (const double *)w, (double *)ub, mub, lamb, s);
  return vjp_t<float>(op, mode, u, (const float *)w, (float *)ub, mub, lamb, s);
}

hipError_t launch_elmat_build(const hpmg_op_s &op, int prec, hipStream_t s) {
  const hpmg_op_s &f = op.fine ? *op.fine : op;  // the operator holding the linearisation
  const unsigned g = grid1d(op.E, ELB);
#define X(q)                                                                                          \
  if (op.Q == q) {                                                                                    \
    if (prec == HPMG_F64)                                                                             \
      k_elmat_build<double, q><<<g, ELB * 24, 0, s>>>(f.state64, op.tab64, f.mu, f.lam, f.mu_e, f.lam_e, \
                                                      op.elmat, op.E);                               \
    else                                                                                              \
      k_elmat_build<float, q><<<g, ELB * 24, 0, s>>>(f.state32, op.tab32, f.mu, f.lam, f.mu_e, f.lam_e,  \
                                                     (float *)op.elmat, op.E);                        \
    return hipGetLastError();                                                                         \
  }
  X(2) X(3) X(4) X(5)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_ell_build(const hpmg_op_s &op, int prec, bool node_major, int64_t W, const int32_t *cols,
                            void *vals,
                            hipStream_t s) {
  if (op.P != 2 || !op.elmat || op.elmat_prec != prec) return hipErrorInvalidValue;
  const unsigned g = grid1d(W * op.N, 256);
  if (prec == HPMG_F64)
    k_ell_build<double><<<g, 256, 0, s>>>(node_major, op.N, (int)W, cols, op.csr_off, op.csr_inc, op.emap,
                                          (const double *)op.elmat, (double *)vals);
  else
    k_ell_build<float><<<g, 256, 0, s>>>(node_major, op.N, (int)W, cols, op.csr_off, op.csr_inc, op.emap,
                                         (const float *)op.elmat, (float *)vals);
  return hipGetLastError();
}

hipError_t launch_export_qdata(const hpmg_op_s &op, double *out, hipStream_t s) {
  const int64_t total = op.E * NGEO * op.Q * op.Q * op.Q;
  switch (op.Q) {
    case 2: k_export_geo<2><<<grid1d(total, 256), 256, 0, s>>>(op.geo, out, op.E); break;
    case 3: k_export_geo<3><<<grid1d(total, 256), 256, 0, s>>>(op.geo, out, op.E); break;
    case 4: k_export_geo<4><<<grid1d(total, 256), 256, 0, s>>>(op.geo, out, op.E); break;
    case 5: k_export_geo<5><<<grid1d(total, 256), 256, 0, s>>>(op.geo, out, op.E); break;
    case 6: k_export_geo<6><<<grid1d(total, 256), 256, 0, s>>>(op.geo, out, op.E); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace hpmg
