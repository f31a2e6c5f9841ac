// Vector kernels for the Krylov and multigrid drivers: boundary-condition fills,
// precision casts, fused axpy-type updates, and deterministic FP64 reductions.
//
// Reductions run on a fixed grid (RED_BLOCKS workgroups of 256 threads): each thread
// accumulates a grid-strided slice in double, a 64-lane wavefront reduces with
// cross-lane shuffles, the four wavefronts of a workgroup combine through LDS, and a
// single workgroup sums the RED_BLOCKS partials in a fixed tree.  The result does not
// depend on timing, so repeated runs are bitwise identical.
#include <algorithm>

#include "common.h"

namespace hpmg {
namespace {

constexpr int BS = 256;

inline unsigned grid_for(int64_t n) {
  int64_t g = (n + BS - 1) / BS;
  if (g < 1) g = 1;
  if (g > 65535 * 16) g = 65535 * 16;
  return (unsigned)g;
}

#define GRID_STRIDE(i, n) \
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n); i += (int64_t)gridDim.x * blockDim.x)

// The fixed reduction grids give a thread many strides of a long vector: f(k, i) loads the
// values of entry i into slot k, g(k, i) uses them, in the order of a plain strided loop,
// with STRIDES strides' loads in flight together (one at a time, a reduction over 3.1 M FP64
// entries moved 3.5 TB/s: 14.1 us against 9.6; the update of the eigenvalue estimate's PCG
// in FP32 17.3 against 16.0, its direction 12.0 against 9.7).
constexpr int STRIDES = 4;
template <typename F, typename G>
__device__ __forceinline__ void strided(int64_t n, F f, G g) {
  const int64_t st = (int64_t)gridDim.x * blockDim.x;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i + (STRIDES - 1) * st < n; i += STRIDES * st) {
#pragma unroll
    for (int k = 0; k < STRIDES; ++k) f(k, i + k * st);
#pragma unroll
    for (int k = 0; k < STRIDES; ++k) g(k, i + k * st);
  }
  for (; i < n; i += st) {
    f(0, i);
    g(0, i);
  }
}

template <typename T>
__global__ void k_init_bc(int64_t nn, const uint8_t *__restrict__ mask, const T *__restrict__ x,
                          T *__restrict__ y) {
  GRID_STRIDE(i, 3 * nn) { y[i] = (mask && x && mask[i]) ? x[i] : T(0); }
}

__global__ void k_cast_d2f(int64_t n, const double *__restrict__ a, float *__restrict__ b) {
  GRID_STRIDE(i, n) { b[i] = (float)a[i]; }
}

__global__ void k_cast_f2d(int64_t n, const float *__restrict__ a, double *__restrict__ b) {
  GRID_STRIDE(i, n) { b[i] = (double)a[i]; }
}

template <typename T>
__global__ void k_axpby(int64_t n, T a, const T *__restrict__ x, T b, T *__restrict__ y) {
  GRID_STRIDE(i, n) { y[i] = a * x[i] + b * y[i]; }
}

template <typename T>
__global__ void k_waxpby(int64_t n, T a, const T *__restrict__ x, T b, const T *__restrict__ y,
                         T *__restrict__ w) {
  GRID_STRIDE(i, n) { w[i] = a * x[i] + b * y[i]; }
}

template <typename T>
__global__ void k_recip(int64_t n, T *__restrict__ x) {
  GRID_STRIDE(i, n) { x[i] = T(1) / x[i]; }
}

// The smoother's first step from x = 0: r = Dinv b; d = r / theta; x = d.
template <typename T>
__global__ void k_cheb_first(int64_t n, const T *__restrict__ dinv, const T *__restrict__ b, T *__restrict__ r,
                             T *__restrict__ d, T *__restrict__ x, T inv_theta) {
  GRID_STRIDE(i, n) {
    const T ri = dinv[i] * b[i];
    const T di = ri * inv_theta;
    r[i] = ri;
    d[i] = di;
    x[i] = di;
  }
}

// ---- reductions -------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// Block sum of NV values per thread into out[v * gridDim.x + blockIdx.x].
template <int NV>
__device__ __forceinline__ void block_store(double (&v)[NV], double *__restrict__ partial) {
  __shared__ double s[NV][BS / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const double w = wave_sum(v[k]);
    if (lane == 0) s[k][wid] = w;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      double t = 0.0;
      for (int j = 0; j < BS / 64; ++j) t += s[k][j];
      partial[k * gridDim.x + blockIdx.x] = t;
    }
  }
}

template <typename T>
__global__ __launch_bounds__(BS) void k_dot_partial(int64_t n, const T *__restrict__ x,
                                                    const T *__restrict__ y, double *__restrict__ partial) {
  double v[1] = {0.0};
  T a[STRIDES], b[STRIDES];
  strided(n, [&](int k, int64_t i) { a[k] = x[i], b[k] = y[i]; },
          [&](int k, int64_t) { v[0] += (double)a[k] * (double)b[k]; });
  block_store<1>(v, partial);
}

template <typename T>
__global__ __launch_bounds__(BS) void k_dot_pair_partial(int64_t n, const T *__restrict__ z,
                                                         const T *__restrict__ a, const T *__restrict__ b,
                                                         double *__restrict__ partial) {
  double v[2] = {0.0, 0.0};
  T p[STRIDES], q[STRIDES], w[STRIDES];
  strided(n, [&](int k, int64_t i) { w[k] = z[i], p[k] = a[i], q[k] = b[i]; },
          [&](int k, int64_t) {
            const double zi = (double)w[k];
            v[0] += zi * (double)p[k];
            v[1] += zi * (double)q[k];
          });
  block_store<2>(v, partial);
}

__global__ __launch_bounds__(BS) void k_sum_partial(int64_t n, const double *__restrict__ x,
                                                    double *__restrict__ partial) {
  double v[1] = {0.0};
  double a[STRIDES];
  strided(n, [&](int k, int64_t i) { a[k] = x[i]; }, [&](int k, int64_t) { v[0] += a[k]; });
  block_store<1>(v, partial);
}

// PCG start from x = 0 (x null: the iterate is not formed): r = b, z = D^-1 r, p = z,
// partials of r.z and r.r.
template <typename T>
__global__ __launch_bounds__(BS) void k_pcg_start(int64_t n, const T *__restrict__ dinv, const T *__restrict__ b,
                                                  T *__restrict__ x, T *__restrict__ r, T *__restrict__ z,
                                                  T *__restrict__ p, double *__restrict__ partial) {
  double v[2] = {0.0, 0.0};
  T vb[STRIDES], vi[STRIDES];
  strided(n, [&](int k, int64_t i) { vb[k] = b[i], vi[k] = dinv[i]; },
          [&](int k, int64_t i) {
            const T ri = vb[k], zi = vi[k] * ri;
            if (x) x[i] = T(0);
            r[i] = ri;
            z[i] = zi;
            p[i] = zi;
            v[0] += (double)ri * (double)zi;
            v[1] += (double)ri * (double)ri;
          });
  block_store<2>(v, partial);
}

// Sum of RED_BLOCKS values by a workgroup of as many threads in a fixed tree (thread 0).
__device__ __forceinline__ double block_tree(double v) {
  __shared__ double s[RED_BLOCKS];
  s[threadIdx.x] = v;
  __syncthreads();
  for (int w = RED_BLOCKS / 2; w > 0; w >>= 1) {
    if (threadIdx.x < (unsigned)w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  const double t = s[0];
  __syncthreads();
  return t;
}

// One workgroup: out[k] = sum of partial[k * nb .. k * nb + nb) in a fixed tree.
__global__ __launch_bounds__(RED_BLOCKS) void k_final(const double *__restrict__ partial, int nb, int nv,
                                                      double *__restrict__ out) {
  for (int k = 0; k < nv; ++k) {
    const double t = block_tree(threadIdx.x < (unsigned)nb ? partial[k * nb + threadIdx.x] : 0.0);
    if (threadIdx.x == 0) out[k] = t;
  }
}

// NV sums of partial[v * stride + 0 .. nb) by the whole workgroup in a fixed order
// (strided per-thread sums, a wave butterfly, the waves in order); every thread gets
// the results.
template <int NV>
__device__ __forceinline__ void block_reduce_fixed_n(const double *__restrict__ partial, int nb, int stride,
                                                     double (&out)[NV]) {
  __shared__ double s[NV][BS / 64];
  double t[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) t[v] = 0.0;
  for (int i = threadIdx.x; i < nb; i += BS)
#pragma unroll
    for (int v = 0; v < NV; ++v) t[v] += partial[v * stride + i];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    t[v] = wave_sum(t[v]);
    if (lane == 0) s[v][wid] = t[v];
  }
  __syncthreads();
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    double r = 0.0;
#pragma unroll
    for (int w = 0; w < BS / 64; ++w) r += s[v][w];
    out[v] = r;
  }
  __syncthreads();
}

__device__ __forceinline__ double block_reduce_fixed(const double *__restrict__ partial, int nb) {
  double o[1];
  block_reduce_fixed_n<1>(partial, nb, 0, o);
  return o[0];
}

// Fused Jacobi-PCG iteration (four launches: the operator's element kernel, its
// assembly fused with the partials of p.q, update2 and dir2).  The curvature p.q arrives
// as workgroup partials of the fused assembly; rz alternates between scalar slots 8 and
// 9 so that no workgroup overwrites a value another one still reads.  The convergence
// test runs on the device: dir2 raises sc[SC_STOP], after which every kernel of later
// iterations returns at once, so the host can queue many iterations and read the
// scalars rarely.  k_pcg_begin: the scalars of the start from k_pcg_start's partials.
__global__ __launch_bounds__(RED_BLOCKS) void k_pcg_begin(const double *__restrict__ partial,
                                                          double *__restrict__ sc) {
  const double rz = block_tree(partial[threadIdx.x]), rr = block_tree(partial[RED_BLOCKS + threadIdx.x]);
  if (threadIdx.x == 0) {
    sc[2] = sc[8] = rz;
    sc[3] = sc[SC_RR0] = rr;
    sc[5] = 0.0;
    sc[SC_STOP] = 0.0;
    sc[SC_COUNT] = 0.0;
  }
}

// update2: alpha = rz / pq, x += alpha p (skipped when x is null: the eigenvalue estimate
// needs only the coefficients), r -= alpha q, z = D^-1 r, partials of r.z, r.r.
template <typename T>
__global__ __launch_bounds__(BS) void k_pcg_update2(int64_t n, double *__restrict__ sc, int parity, int nb_pq,
                                                    const double *__restrict__ pq_partial,
                                                    const T *__restrict__ p, const T *__restrict__ q,
                                                    T *__restrict__ x, T *__restrict__ r,
                                                    const T *__restrict__ dinv, T *__restrict__ z,
                                                    double *__restrict__ partial, double *__restrict__ alpha_rec) {
  if (sc[SC_STOP] != 0.0) return;
  const double pq = block_reduce_fixed(pq_partial, nb_pq);
  const double alpha = pq > 0.0 ? sc[8 + parity] / pq : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sc[1] = pq;
    if (!(pq > 0.0)) sc[5] = 1.0;
    if (alpha_rec) *alpha_rec = alpha;
  }
  const T a = (T)alpha;
  double v[2] = {0.0, 0.0};
  T vx[STRIDES], vp[STRIDES], vr[STRIDES], vq[STRIDES], vi[STRIDES];
  strided(
      n,
      [&](int k, int64_t i) {
        if (x) vx[k] = x[i], vp[k] = p[i];
        vr[k] = r[i], vq[k] = q[i], vi[k] = dinv[i];
      },
      [&](int k, int64_t i) {
        if (x) x[i] = vx[k] + a * vp[k];
        const T ri = vr[k] - a * vq[k];
        r[i] = ri;
        const T zi = vi[k] * ri;
        z[i] = zi;
        v[0] += (double)ri * (double)zi;
        v[1] += (double)ri * (double)ri;
      });
  block_store<2>(v, partial);
}

// dir2: rz_new and r.r from the partials, beta = rz_new / rz, p = z + beta p; counts the
// iteration and decides whether to stop.
template <typename T>
__global__ __launch_bounds__(BS) void k_pcg_dir2(int64_t n, double *__restrict__ sc, int parity,
                                                 const double *__restrict__ partial, const T *__restrict__ z,
                                                 T *__restrict__ p, double rtol2, double *__restrict__ beta_rec) {
  if (sc[SC_STOP] != 0.0) return;
  double red2[2];
  block_reduce_fixed_n<2>(partial, RED_BLOCKS, RED_BLOCKS, red2);
  const double rz_new = red2[0], rr = red2[1];
  const double rz = sc[8 + parity];
  const bool broke = sc[5] != 0.0;
  const double beta = rz != 0.0 ? rz_new / rz : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (broke) {
      sc[SC_STOP] = 1.0;
    } else {
      sc[8 + (parity ^ 1)] = rz_new;
      sc[2] = rz_new;
      sc[3] = rr;
      sc[SC_COUNT] += 1.0;
      if (beta_rec) *beta_rec = beta;
      if (rtol2 >= 0.0 && rr <= rtol2 * sc[SC_RR0]) sc[SC_STOP] = 1.0;
    }
  }
  if (broke) return;
  const T b = (T)beta;
  T vz[STRIDES], vp[STRIDES];
  strided(n, [&](int k, int64_t i) { vz[k] = z[i], vp[k] = p[i]; },
          [&](int k, int64_t i) { p[i] = vz[k] + b * vp[k]; });
}

__global__ __launch_bounds__(BS) void k_fcg_update(int64_t n, double *__restrict__ sc, int it,
                                                   const double *__restrict__ p, const double *__restrict__ q,
                                                   double *__restrict__ x, const double *__restrict__ r,
                                                   double *__restrict__ rn, double *__restrict__ partial) {
  const double pq = sc[FCG_PQ], rz = sc[FCG_RZ + (it & 1)];
  const bool brk = !(pq > 0.0) || !isfinite(rz);
  const double a = brk ? 0.0 : rz / pq;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sc[FCG_BRK] = brk ? 1.0 : 0.0;
    sc[FCG_ALPHA] = a;
  }
  double v[1] = {0.0};
  double vx[STRIDES], vp[STRIDES], vr[STRIDES], vq[STRIDES];
  strided(n, [&](int k, int64_t i) { vx[k] = x[i], vp[k] = p[i], vr[k] = r[i], vq[k] = q[i]; },
          [&](int k, int64_t i) {
            x[i] = vx[k] + a * vp[k];
            const double ri = vr[k] - a * vq[k];
            rn[i] = ri;
            v[0] += ri * ri;
          });
  block_store<1>(v, partial);
}

__global__ __launch_bounds__(BS) void k_fcg_dir(int64_t n, double *__restrict__ sc, int it,
                                                const double *__restrict__ z, double *__restrict__ p) {
  const double zrn = sc[FCG_ZRN], rz = sc[FCG_RZ + (it & 1)];
  const double beta = (zrn - sc[FCG_ZR]) / rz;
  if (blockIdx.x == 0 && threadIdx.x == 0) sc[FCG_RZ + ((it + 1) & 1)] = zrn;
  GRID_STRIDE(i, n) { p[i] = z[i] + beta * p[i]; }
}

__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// Jacobi-PCG iteration `it` on an assembled operator held as 3 x 3 blocks in sliced ELL
// (slot j of node n: column node cols[j][n], or -1 - n for padding past the row's end,
// whose block is zero), replacing the element kernel, the fused assembly and dir2 of the
// four-launch iteration.  Prologue (it > 0, every workgroup alike): r.z and r.r of
// iteration it - 1 from the update's partials, beta, the stopping test (as in dir2; the
// count is set, not incremented, so a repeated prologue changes nothing).  The body
// forms the new direction p = z + beta p_old on the fly for every column node read,
// with one fused multiply-add, so all threads that need a node's p agree bit for bit;
// the row's own value goes to p_new (p_old and p_new alternate between two buffers),
// q = A p to y, and the partial of p.q to pq_part[workgroup].  WC > 0 fixes the width
// at compile time, so the loads of several slots can be issued together.  nn = 0 runs
// the prologue alone.  Two bodies and block layouts (node_major; by default by size):
//  * rows: a thread per scalar row, the three rows of a node on neighbouring lanes (they
//    read the same column nodes); block entry (i, k) at vals[j][n][3 i + k].  Three
//    times the threads of the other form: the faster one while the coarse level is small
//    (per iteration at 21^3 nodes 23.4 against 34.5 us in FP64).
//  * nodes: a thread per node and its three rows; entry (i, k) at vals[j][3 i + k][n],
//    so each of a block's nine loads is one contiguous run over the workgroup's nodes.
//    The faster one once the block matrix streams from HBM (per iteration at 61^3 nodes
//    154.9 against 202.6 us in FP64, 68.5 against 105.6 us in FP32); equal at 41^3.

// The prologue; false: the iteration stops (every thread of the grid agrees).
__device__ __forceinline__ bool ell_prologue(double *__restrict__ sc, const double *__restrict__ partial, int it,
                                             double rtol2, double &beta) {
  beta = 0.0;
  if (it == 0) return true;
  double red2[2];
  block_reduce_fixed_n<2>(partial, RED_BLOCKS, RED_BLOCKS, red2);
  const double rz_new = red2[0], rr = red2[1];
  const double rz = sc[8 + ((it - 1) & 1)];
  const bool broke = sc[5] != 0.0;
  const bool conv = !broke && rtol2 >= 0.0 && rr <= rtol2 * sc[SC_RR0];
  beta = rz != 0.0 ? rz_new / rz : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (!broke) {
      sc[8 + (it & 1)] = rz_new;
      sc[2] = rz_new;
      sc[3] = rr;
      sc[SC_COUNT] = (double)it;
    }
    if (broke || conv) sc[SC_STOP] = 1.0;
  }
  return !(broke || conv);
}

template <typename T, int WC>
__global__ __launch_bounds__(BS) void k_ell_pcg_rows(int64_t nn, int W, const int32_t *__restrict__ cols,
                                                     const T *__restrict__ vals, const T *__restrict__ z,
                                                     const T *__restrict__ p_old, T *__restrict__ p_new,
                                                     T *__restrict__ y, double *__restrict__ sc,
                                                     const double *__restrict__ partial, int it, double rtol2,
                                                     double *__restrict__ pq_part) {
  if (sc[SC_STOP] != 0.0) return;
  double beta;
  if (!ell_prologue(sc, partial, it, rtol2, beta) || nn == 0) return;
  const bool first = it == 0;
  const T b = (T)beta;
  double v[1] = {0.0};
  const int64_t t = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (t < 3 * nn) {
    const int64_t n = t / 3;
    const int i = (int)(t - 3 * n);
    // direction value of node c, component k (the same expression wherever it is formed)
    auto pdir = [&](int64_t c, int k) { return first ? z[c * 3 + k] : fma_t(b, p_old[c * 3 + k], z[c * 3 + k]); };
    auto slot = [&](int j, int32_t c0) {
      const int64_t c = c0 < 0 ? -1 - (int64_t)c0 : (int64_t)c0;
      const T *A = vals + ((int64_t)j * nn + n) * 9 + 3 * i;
      return A[0] * pdir(c, 0) + A[1] * pdir(c, 1) + A[2] * pdir(c, 2);
    };
    T acc = 0;
    if constexpr (WC > 0) {
      // all column ids first (one wait), then the blocks in groups whose loads are
      // issued together (9 in FP32, 3 in FP64, as the registers allow)
      constexpr int UR = sizeof(T) == 4 ? 9 : 3;
      static_assert(WC % UR == 0, "width must be a multiple of the unroll");
      int32_t cj[WC];
#pragma unroll
      for (int j = 0; j < WC; ++j) cj[j] = cols[(int64_t)j * nn + n];
      for (int j0 = 0; j0 < WC; j0 += UR) {
        T part[UR];
#pragma unroll
        for (int u = 0; u < UR; ++u) part[u] = slot(j0 + u, cj[j0 + u]);
#pragma unroll
        for (int u = 0; u < UR; ++u) acc += part[u];
      }
    } else {
      for (int j = 0; j < W; ++j) acc += slot(j, cols[(int64_t)j * nn + n]);
    }
    const T pn = pdir(n, i);
    p_new[t] = pn;
    y[t] = acc;
    v[0] = (double)pn * (double)acc;
  }
  block_store<1>(v, pq_part);
}

template <typename T, int WC>
__global__ __launch_bounds__(BS) void k_ell_pcg_nodes(int64_t nn, int W, const int32_t *__restrict__ cols,
                                                      const T *__restrict__ vals, const T *__restrict__ z,
                                                      const T *__restrict__ p_old, T *__restrict__ p_new,
                                                      T *__restrict__ y, double *__restrict__ sc,
                                                      const double *__restrict__ partial, int it, double rtol2,
                                                      double *__restrict__ pq_part) {
  if (sc[SC_STOP] != 0.0) return;
  double beta;
  if (!ell_prologue(sc, partial, it, rtol2, beta) || nn == 0) return;
  const bool first = it == 0;
  const T b = (T)beta;
  double v[1] = {0.0};
  const int64_t n = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (n < nn) {
    auto pdir = [&](int64_t c, int k) { return first ? z[c * 3 + k] : fma_t(b, p_old[c * 3 + k], z[c * 3 + k]); };
    // the block of slot j (column node c0) times the direction at that node
    auto slot = [&](int j, int32_t c0, T (&part)[3]) {
      const int64_t c = c0 < 0 ? -1 - (int64_t)c0 : (int64_t)c0;
      T pd[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) pd[k] = pdir(c, k);
      const T *A = vals + (int64_t)j * 9 * nn + n;
#pragma unroll
      for (int i = 0; i < 3; ++i)
        part[i] = A[(3 * i) * nn] * pd[0] + A[(3 * i + 1) * nn] * pd[1] + A[(3 * i + 2) * nn] * pd[2];
    };
    T acc[3] = {0, 0, 0};
    if constexpr (WC > 0) {
      constexpr int UR = sizeof(T) == 4 ? 3 : 1;
      static_assert(WC % UR == 0, "width must be a multiple of the unroll");
      int32_t cj[WC];
#pragma unroll
      for (int j = 0; j < WC; ++j) cj[j] = cols[(int64_t)j * nn + n];
      for (int j0 = 0; j0 < WC; j0 += UR) {
        T part[UR][3];
#pragma unroll
        for (int u = 0; u < UR; ++u) slot(j0 + u, cj[j0 + u], part[u]);
#pragma unroll
        for (int u = 0; u < UR; ++u)
#pragma unroll
          for (int i = 0; i < 3; ++i) acc[i] += part[u][i];
      }
    } else {
      for (int j = 0; j < W; ++j) {
        T part[3];
        slot(j, cols[(int64_t)j * nn + n], part);
#pragma unroll
        for (int i = 0; i < 3; ++i) acc[i] += part[i];
      }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const T pn = pdir(n, i);
      p_new[n * 3 + i] = pn;
      y[n * 3 + i] = acc[i];
      v[0] += (double)pn * (double)acc[i];
    }
  }
  block_store<1>(v, pq_part);
}

// ---- the whole coarse solve in one launch -------------------------------------------
// Launched iteration by iteration, the assembled coarse level is bound by latency while its
// blocks stay on the chip: two launches, two passes over the partial sums and nine dependent
// rounds of loads, 21-24 us an iteration from 5^3 to 26^3 nodes, of which the blocks
// themselves (18 MB at 21^3 in FP64) would take 3.  The register files of the 256 compute
// units hold 128 MB, so here a thread keeps a scalar row (81 entries) for the whole solve;
// what remains of an iteration is two sums over the grid, each a store and a load through
// the memory side (about 1.5 us), the neighbours' z fetched while the first is under way,
// and 81 LDS reads a row.  Measured per iteration, launch to launch: 11^3 nodes 24 -> 4.4 us
// (FP64), 21^3 23.6 -> 5.8 us (FP64), 26^3 25 -> 6.8 us (FP32); a whole V-cycle Q4 -> Q2 -> Q1 to
// a coarse tolerance of 1e-3, by launches against one launch: 20^3 elements FP64 1042 -> 674 us
// with a right-hand side of 17 coarse iterations, 2852 -> 1114 with one of 97; FP32 806 -> 471 and
// 2426 -> 889; 25^3 FP32 1117 -> 710 (19) and 3151 -> 1199 (110).
// 512 rows a workgroup and not fewer, since the sums cost more with every workgroup that
// posts and reads them (21^3 nodes: 55 workgroups 191 us a solve, 127 221, 251 275).  The sums
// are taken over blocks of 256 rows, in the order of the launches' kernels, so that row-major
// blocks of at most 131,072 rows (the 512 x 256 threads of those kernels' grids) give the same
// bits either way; beyond that, or with node-major blocks, the launches group them otherwise.
constexpr int CP_NT = 512;
constexpr int CP_RING = 8;  // sets of slots in rotation
// What a slot or an exchanged value holds while it is empty: a NaN that no arithmetic
// produces (a NaN to be posted is replaced by the plain one).
template <typename T>
struct CpBits;
template <>
struct CpBits<double> {
  using U = unsigned long long;
  static constexpr U EMPTY = 0x7ff8c0a45e5e7c01ull;
  static __device__ __forceinline__ U of(double v) {
    return (U)__double_as_longlong(v == v ? v : __builtin_nan(""));
  }
  static __device__ __forceinline__ double value(U u) { return __longlong_as_double((long long)u); }
};
template <>
struct CpBits<float> {
  using U = unsigned int;
  static constexpr U EMPTY = 0x7fc5e7c1u;
  static __device__ __forceinline__ U of(float v) { return __float_as_uint(v == v ? v : __builtin_nanf("")); }
  static __device__ __forceinline__ float value(U u) { return __uint_as_float(u); }
};

template <typename U>
__device__ __forceinline__ U agent_load(const U *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename U>
__device__ __forceinline__ void agent_store(U *p, U v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Empties the slots and both exchange buffers.
template <typename T>
__global__ void k_coarse_begin(CoarsePcg a, int64_t n_slots) {
  using B = CpBits<T>;
  typename B::U *z0 = (typename B::U *)a.z[0], *z1 = (typename B::U *)a.z[1];
  unsigned long long *slots = reinterpret_cast<unsigned long long *>(a.slots);
  GRID_STRIDE(i, n_slots) { slots[i] = CpBits<double>::EMPTY; }
  GRID_STRIDE(i, 3 * a.nn) {
    z0[i] = B::EMPTY;
    z1[i] = B::EMPTY;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) a.sc[1] = a.sc[SC_COUNT] = a.sc[SC_LOST] = 0.0;
}

// Sum over the wave in the order of wave_sum (lanes 32 apart, then 16, 8, 4, 2 and 1), in
// every lane, by lane moves of the vector ALU instead of an LDS round trip a step.
__device__ __forceinline__ double lane_pair(double v, int lo, int hi) {
  return v + __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <int CTRL>
__device__ __forceinline__ double add_rotated(double v) {
  const long long b = __double_as_longlong(v);
  return lane_pair(v, __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, false),
                   __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ double wave_total(double v) {
  {
    const long long b = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane32_swap((int)b, (int)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((int)(b >> 32), (int)(b >> 32), false, false);
    v = lane_pair(__longlong_as_double(((long long)(int)hi[0] << 32) | (unsigned)lo[0]), (int)lo[1], (int)hi[1]);
  }
  {
    const long long b = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane16_swap((int)b, (int)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((int)(b >> 32), (int)(b >> 32), false, false);
    v = lane_pair(__longlong_as_double(((long long)(int)hi[0] << 32) | (unsigned)lo[0]), (int)lo[1], (int)hi[1]);
  }
  v = add_rotated<0x128>(v);  // row_ror:8, 4, 2, 1
  v = add_rotated<0x124>(v);
  v = add_rotated<0x122>(v);
  return add_rotated<0x121>(v);
}

template <int RPT>
struct CpShared {
  double part[2][RPT][CP_NT / 64], total[2][4];
  int lost;
};

// Sums NV values over all rows, in the same order in every workgroup and, for row-major blocks
// of at most 131,072 rows, in that of the launch-per-iteration form: a partial for every BS
// rows (four waves each), then these as block_reduce_fixed_n does, or as k_final does for the
// FIRST sums.  Each workgroup
// posts its partials in set `epoch` % 8 of the slots, and its first waves read everybody's
// while the others run `meanwhile(first thread, threads)`.  A slot is emptied four epochs
// before it is used again: all have read it then (when a workgroup posts epoch e, all have
// read epoch e - 2), and an ACK call (every other one) lies in between, which posts only
// after all that its workgroup stored before has been acknowledged.
// false: a wait took over a.wait (every thread of the workgroup agrees).
template <int NV, int RPT, bool ACK, bool FIRST, typename F>
__device__ __forceinline__ bool cp_sum(const CoarsePcg &a, int epoch, const double (&in)[RPT][NV], double (&out)[NV],
                                       CpShared<RPT> &sh, F meanwhile) {
  using B = CpBits<double>;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, G = a.groups, K = a.rows / BS;
  const int nb = (int)((3 * a.nn + BS - 1) / BS);
#pragma unroll
  for (int s = 0; s < RPT; ++s)
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const double w = wave_total(in[s][k]);
      if (lane == 0) sh.part[k][s][wid] = w;
    }
  if (ACK) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  const int pollers = FIRST ? 1 : nb < 256 ? (nb + 63) / 64 : 4;
  if (wid < pollers) {
    // partial k of this workgroup's block b: rows BS b .. BS (b + 1)
    auto partial = [&](int k, int b) {
      const double *w = &sh.part[k][b / (CP_NT / BS)][b % (CP_NT / BS) * (BS / 64)];
      double t = 0.0;
#pragma unroll
      for (int j = 0; j < BS / 64; ++j) t += w[j];
      return t;
    };
    unsigned long long *slots = reinterpret_cast<unsigned long long *>(a.slots);
    const size_t copy = (size_t)CP_RING * 2 * nb, set = (size_t)(epoch % CP_RING) * 2 * nb;
    if (G > 1 && wid == 0) {
      const int b = lane / COARSE_PCG_COPIES, gb = blockIdx.x * K + b;
      if (b < K && gb < nb) {
        unsigned long long *mine = slots + lane % COARSE_PCG_COPIES * copy + gb;
#pragma unroll
        for (int k = 0; k < NV; ++k) agent_store(mine + set + k * nb, B::of(partial(k, b)));
        const size_t later = (size_t)((epoch + CP_RING / 2) % CP_RING) * 2 * nb;
        agent_store(mine + later, B::EMPTY);
        agent_store(mine + later + nb, B::EMPTY);
      }
    }
    const unsigned long long *read = slots + (blockIdx.x % COARSE_PCG_COPIES) * copy + set;
    const unsigned t0 = (unsigned)wall_clock64();
    // the sums of block i < nb
    auto get = [&](int i, double (&x)[NV]) {
      if (G == 1) {
#pragma unroll
        for (int k = 0; k < NV; ++k) x[k] = partial(k, i);
        return;
      }
      for (;;) {
        unsigned long long q[NV];
        bool all = true;
#pragma unroll
        for (int k = 0; k < NV; ++k) q[k] = agent_load(read + k * nb + i);
#pragma unroll
        for (int k = 0; k < NV; ++k) {
          all = all && q[k] != B::EMPTY;
          x[k] = B::value(q[k]);
        }
        if (all) return;
        if ((int)((unsigned)wall_clock64() - t0) > (int)a.wait) {
          sh.lost = 1;
          return;
        }
      }
    };
    double x[NV];
    if constexpr (FIRST) {
      double y[4][NV];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int k = 0; k < NV; ++k) y[q][k] = 0.0;
        for (int i = lane + 64 * q; i < nb; i += BS) {
          get(i, x);
#pragma unroll
          for (int k = 0; k < NV; ++k) y[q][k] += x[k];
        }
      }
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        const double t = wave_total((y[0][k] + y[2][k]) + (y[1][k] + y[3][k]));
        if (lane < 4) sh.total[k][lane] = lane == 0 ? t : 0.0;
      }
    } else {
      double y[NV];
#pragma unroll
      for (int k = 0; k < NV; ++k) y[k] = 0.0;
      for (int i = tid; i < nb; i += BS) {
        get(i, x);
#pragma unroll
        for (int k = 0; k < NV; ++k) y[k] += x[k];
      }
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        const double t = wave_total(y[k]);
        if (lane == 0) sh.total[k][wid] = t;
      }
      if (wid == 0 && lane >= pollers && lane < 4)
#pragma unroll
        for (int k = 0; k < NV; ++k) sh.total[k][lane] = 0.0;
    }
  } else {
    meanwhile(64 * pollers, CP_NT - 64 * pollers);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    out[k] = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w) out[k] += sh.total[k][w];
  }
  return sh.lost == 0;
}

// The halo's z out of its exchange buffer into zh, by `count` threads from `first` on (a
// value that is still empty has not arrived).
template <typename T>
__device__ __forceinline__ void cp_fetch(const typename CpBits<T>::U *__restrict__ zx, const int32_t *ids, T *zh,
                                         int nh, int *lost, int wait, int first, int count) {
  using B = CpBits<T>;
  constexpr int NF = sizeof(T) == 4 ? 2 : 1;  // nodes whose loads are in flight together
  const unsigned t0 = (unsigned)wall_clock64();
  for (int u = (int)threadIdx.x - first; u < nh; u += NF * count) {
    typename B::U q[NF][3];
    int64_t from[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const int uf = u + f * count;
      from[f] = (int64_t)ids[uf < nh ? uf : u] * 3;
    }
    for (;;) {
      bool all = true;
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int k = 0; k < 3; ++k) q[f][k] = agent_load(zx + from[f] + k);
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int k = 0; k < 3; ++k) all = all && q[f][k] != B::EMPTY;
      if (all) break;
      if ((int)((unsigned)wall_clock64() - t0) > wait) {
        *lost = 1;
        break;
      }
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const int uf = u + f * count;
      if (uf < nh)
#pragma unroll
        for (int k = 0; k < 3; ++k) zh[3 * uf + k] = B::value(q[f][k]);
    }
  }
}

template <typename T, int RPT>
__global__ __launch_bounds__(CP_NT) void k_coarse_pcg(CoarsePcg a) {
  using B = CpBits<T>;
  using U = typename B::U;
  constexpr int W = COARSE_PCG_W;
  extern __shared__ __align__(16) char smem[];
  __shared__ CpShared<RPT> sh;
  const int tid = threadIdx.x, g = blockIdx.x;
  const int64_t n3 = 3 * a.nn, row0 = (int64_t)g * a.rows;
  const int rows = (int)(n3 - row0 < a.rows ? n3 - row0 : a.rows);
  const int h0 = a.halo_off[g], nh = a.halo_off[g + 1] - h0;
  T *p = reinterpret_cast<T *>(smem);                // directions: own rows, then the halo nodes'
  T *ph = p + a.rows, *zh = ph + 3 * a.max_halo;     // the halo's part, and its z
  int32_t *ids = reinterpret_cast<int32_t *>(zh + 3 * a.max_halo);
  if (tid == 0) sh.lost = 0;
  for (int u = tid; u < nh; u += CP_NT) ids[u] = a.halo_ids[h0 + u];
  // zero entries of rows past the end and of padding slots meet p[0], which nothing else
  // writes where the first row's node is shared with the workgroup before
  for (int u = tid; u < a.rows; u += CP_NT) p[u] = T(0);
  T A[RPT][3 * W], x[RPT], r[RPT], z[RPT], di[RPT], po[RPT];
  uint32_t off[RPT][(W + 1) / 2];  // first entry of each column's direction, two to a word
  bool whole[RPT];                 // the row's node is all in this workgroup
  double v[RPT][2];
  U *const z0 = (U *)a.z[0], *const z1 = (U *)a.z[1];
#pragma unroll
  for (int s = 0; s < RPT; ++s) {
    const int row = tid + s * CP_NT;
    const bool live = row < rows;
    const int64_t d = row0 + (live ? row : 0), n = d / 3;
    const int i = (int)(d - 3 * n);
    whole[s] = live && 3 * n >= row0 && 3 * n + 3 <= row0 + rows;
    const T *vals = (const T *)a.vals;
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const bool in = live && j < a.W;
      const uint32_t o = in ? a.cols[(int64_t)j * n3 + d] : 0u;
      off[s][j / 2] = j % 2 ? off[s][j / 2] | (o << 16) : o;
#pragma unroll
      for (int k = 0; k < 3; ++k)
        A[s][3 * j + k] = !in            ? T(0)
                          : a.node_major ? vals[((int64_t)j * 9 + 3 * i + k) * a.nn + n]
                                         : vals[((int64_t)j * a.nn + n) * 9 + 3 * i + k];
      if (j % 3 == 2) asm volatile("" ::: "memory");
    }
    x[s] = po[s] = T(0);
    r[s] = live ? ((const T *)a.b)[d] : T(0);
    di[s] = live ? ((const T *)a.dinv)[d] : T(0);
    z[s] = di[s] * r[s];
    if (live) agent_store(z0 + d, B::of(z[s]));
    v[s][0] = (double)r[s] * (double)z[s];
    v[s][1] = (double)r[s] * (double)r[s];
  }
  __syncthreads();  // ids
  int epoch = 0, it = 0;
  double sum[2], pq[1];
  bool ok = cp_sum<2, RPT, false, true>(
      a, epoch++, v, sum, sh, [z0, ids, zh, nh, lost = &sh.lost, wait = (int)a.wait](int t, int c) {
        cp_fetch<T>(z0, ids, zh, nh, lost, wait, t, c);
      });
  double rz = sum[0], beta = 0.0;
  const double rr0 = sum[1];
  while (ok && it < a.maxit) {
    // p = z + beta p: the own rows' z from registers, the halo's as their owners stored it
    const T bt = (T)beta;
#pragma unroll
    for (int s = 0; s < RPT; ++s) {
      po[s] = it ? fma_t(bt, po[s], z[s]) : z[s];
      if (whole[s]) p[tid + s * CP_NT] = po[s];
    }
    for (int e = tid; e < 3 * nh; e += CP_NT) ph[e] = it ? fma_t(bt, ph[e], zh[e]) : zh[e];
    __syncthreads();
    T q[RPT];
    double c[RPT][1];
#pragma unroll
    for (int s = 0; s < RPT; ++s) {
      // column by column as in the launch-per-iteration form
      T acc = 0;
#pragma unroll
      for (int j = 0; j < W; ++j) {
        const T *pc = p + ((off[s][j / 2] >> (j % 2 ? 16 : 0)) & 0xffffu);
        acc += A[s][3 * j] * pc[0] + A[s][3 * j + 1] * pc[1] + A[s][3 * j + 2] * pc[2];
        // a few columns' reads at a time: all at once would not fit the registers
        if (j % 3 == 2) asm volatile("" : "+v"(acc)::"memory");
      }
      q[s] = acc;
      c[s][0] = (double)po[s] * (double)q[s];
    }
    ok = cp_sum<1, RPT, true, false>(a, epoch++, c, pq, sh, [](int, int) {});
    if (!ok || !(pq[0] > 0.0)) {  // breakdown: x as it is; the host looks at p.q
      if (g == 0 && tid == 0) a.sc[1] = pq[0];
      break;
    }
    const T al = (T)(rz / pq[0]);
    U *const zw = it & 1 ? z0 : z1, *const zo = it & 1 ? z1 : z0;
#pragma unroll
    for (int s = 0; s < RPT; ++s) {
      const int row = tid + s * CP_NT;
      x[s] += al * po[s];
      r[s] = r[s] - al * q[s];
      z[s] = di[s] * r[s];
      if (row < rows) {
        agent_store(zw + row0 + row, B::of(z[s]));
        agent_store(zo + row0 + row, B::EMPTY);  // all have fetched it before they posted p.q
      }
      v[s][0] = (double)r[s] * (double)z[s];
      v[s][1] = (double)r[s] * (double)r[s];
    }
    ok = cp_sum<2, RPT, false, false>(
        a, epoch++, v, sum, sh, [zw, ids, zh, nh, lost = &sh.lost, wait = (int)a.wait](int t, int c) {
          cp_fetch<T>(zw, ids, zh, nh, lost, wait, t, c);
        });
    if (!ok) break;
    ++it;
    beta = rz != 0.0 ? sum[0] / rz : 0.0;
    rz = sum[0];
    if (sum[1] <= a.rtol2 * rr0) break;
  }
  if (!ok) {
    if (tid == 0) a.sc[SC_LOST] = 1.0;
    return;
  }
#pragma unroll
  for (int s = 0; s < RPT; ++s) {
    const int row = tid + s * CP_NT;
    if (row < rows) ((T *)a.x)[row0 + row] = x[s];
  }
  if (g == 0 && tid == 0) a.sc[SC_COUNT] = (double)it;
}

}  // namespace

// A row to a thread (162 registers of matrix in FP64), or two in FP32.
int coarse_pcg_max_rows(int prec) { return (prec == HPMG_F64 ? 1 : 2) * CP_NT; }

size_t coarse_pcg_lds(int prec, int rows, int max_halo) {
  return (size_t)(rows + 6 * max_halo) * prec_size(prec) + (size_t)max_halo * sizeof(int32_t);
}

// A set of slots for each of the ring and copy: two values per block of BS rows.
size_t coarse_pcg_slots(int64_t nn) {
  return (size_t)COARSE_PCG_COPIES * CP_RING * 2 * (size_t)((3 * nn + BS - 1) / BS);
}

hipError_t launch_coarse_pcg(int prec, const CoarsePcg &a, hipStream_t s) {
  const size_t lds = coarse_pcg_lds(prec, a.rows, a.max_halo);
  const int64_t n_slots = (int64_t)coarse_pcg_slots(a.nn);
  const unsigned clear = grid_for(std::max<int64_t>(3 * a.nn, n_slots)), g = (unsigned)a.groups;
  if (prec == HPMG_F64) {
    k_coarse_begin<double><<<clear, BS, 0, s>>>(a, n_slots);
    k_coarse_pcg<double, 1><<<g, CP_NT, lds, s>>>(a);
  } else {
    k_coarse_begin<float><<<clear, BS, 0, s>>>(a, n_slots);
    if (a.rows <= CP_NT)
      k_coarse_pcg<float, 1><<<g, CP_NT, lds, s>>>(a);
    else
      k_coarse_pcg<float, 2><<<g, CP_NT, lds, s>>>(a);
  }
  return hipGetLastError();
}

hipError_t launch_fcg_update(int64_t n, double *sc, int it, const double *p, const double *q, double *x,
                             const double *r, double *rn, double *partial, hipStream_t s) {
  k_fcg_update<<<RED_BLOCKS, BS, 0, s>>>(n, sc, it, p, q, x, r, rn, partial);
  k_final<<<1, RED_BLOCKS, 0, s>>>(partial, RED_BLOCKS, 1, sc + FCG_RR);
  return hipGetLastError();
}

hipError_t launch_fcg_dir(int64_t n, double *sc, int it, const double *z, double *p, hipStream_t s) {
  k_fcg_dir<<<grid_for(n), BS, 0, s>>>(n, sc, it, z, p);
  return hipGetLastError();
}

hipError_t launch_pcg_start(int prec, int64_t n, const void *dinv, const void *b, void *x, void *r, void *z, void *p,
                            double *partial, double *sc, hipStream_t s) {
  if (prec == HPMG_F64)
    k_pcg_start<double><<<RED_BLOCKS, BS, 0, s>>>(n, (const double *)dinv, (const double *)b, (double *)x,
                                                  (double *)r, (double *)z, (double *)p, partial);
  else
    k_pcg_start<float><<<RED_BLOCKS, BS, 0, s>>>(n, (const float *)dinv, (const float *)b, (float *)x, (float *)r,
                                                 (float *)z, (float *)p, partial);
  k_pcg_begin<<<1, RED_BLOCKS, 0, s>>>(partial, sc);
  return hipGetLastError();
}

int ell_pcg_blocks(int64_t nn, bool node_major) {
  return node_major ? (int)((nn + BS - 1) / BS) : (int)((3 * nn + BS - 1) / BS);
}

hipError_t launch_ell_pcg_apply(int prec, bool nodes, int64_t nn, int W, const int32_t *cols, const void *vals,
                                const void *z,
                                const void *p_old, void *p_new, void *y, double *sc, const double *partial, int it,
                                double rtol2, double *pq_part, hipStream_t s) {
  const unsigned g = nn > 0 ? (unsigned)ell_pcg_blocks(nn, nodes) : 1u;
#define ELL_LAUNCH(TT, WC)                                                                                    \
  do {                                                                                                        \
    if (nodes)                                                                                                \
      k_ell_pcg_nodes<TT, WC><<<g, BS, 0, s>>>(nn, W, cols, (const TT *)vals, (const TT *)z, (const TT *)p_old, \
                                               (TT *)p_new, (TT *)y, sc, partial, it, rtol2, pq_part);          \
    else                                                                                                      \
      k_ell_pcg_rows<TT, WC><<<g, BS, 0, s>>>(nn, W, cols, (const TT *)vals, (const TT *)z, (const TT *)p_old,  \
                                              (TT *)p_new, (TT *)y, sc, partial, it, rtol2, pq_part);           \
  } while (0)
  // 27: every node of a hexahedral mesh interior
  if (prec == HPMG_F64) {
    if (W == 27)
      ELL_LAUNCH(double, 27);
    else
      ELL_LAUNCH(double, 0);
  } else {
    if (W == 27)
      ELL_LAUNCH(float, 27);
    else
      ELL_LAUNCH(float, 0);
  }
#undef ELL_LAUNCH
  return hipGetLastError();
}

hipError_t launch_pcg_update2(int prec, int64_t n, double *sc, int parity, int nb_pq, const double *pq_partial,
                              const void *p, const void *q, void *x, void *r, const void *dinv, void *z,
                              double *partial, double *alpha_rec, hipStream_t s) {
  if (prec == HPMG_F64)
    k_pcg_update2<double><<<RED_BLOCKS, BS, 0, s>>>(n, sc, parity, nb_pq, pq_partial, (const double *)p,
                                                    (const double *)q, (double *)x, (double *)r,
                                                    (const double *)dinv, (double *)z, partial, alpha_rec);
  else
    k_pcg_update2<float><<<RED_BLOCKS, BS, 0, s>>>(n, sc, parity, nb_pq, pq_partial, (const float *)p,
                                                   (const float *)q, (float *)x, (float *)r, (const float *)dinv,
                                                   (float *)z, partial, alpha_rec);
  return hipGetLastError();
}

hipError_t launch_pcg_dir2(int prec, int64_t n, double *sc, int parity, const double *partial, const void *z,
                           void *p, double rtol2, double *beta_rec, hipStream_t s) {
  // every workgroup sums the partials again, so not more of them than fill the device
  const unsigned g = (unsigned)std::min<int64_t>((n + BS * STRIDES - 1) / (BS * STRIDES), 2048);
  if (prec == HPMG_F64)
    k_pcg_dir2<double><<<g, BS, 0, s>>>(n, sc, parity, partial, (const double *)z, (double *)p, rtol2,
                                                 beta_rec);
  else
    k_pcg_dir2<float><<<g, BS, 0, s>>>(n, sc, parity, partial, (const float *)z, (float *)p, rtol2,
                                                beta_rec);
  return hipGetLastError();
}


size_t prec_size(int prec) { return prec == HPMG_F64 ? sizeof(double) : sizeof(float); }

#define DISPATCH(prec, CALL_D, CALL_F) \
  do {                                 \
    if ((prec) == HPMG_F64) {          \
      CALL_D;                          \
    } else {                           \
      CALL_F;                          \
    }                                  \
    return hipGetLastError();          \
  } while (0)

hipError_t launch_init_bc(int prec, int64_t nn, const uint8_t *mask, const void *x, void *y, hipStream_t s) {
  DISPATCH(prec, (k_init_bc<double><<<grid_for(3 * nn), BS, 0, s>>>(nn, mask, (const double *)x, (double *)y)),
           (k_init_bc<float><<<grid_for(3 * nn), BS, 0, s>>>(nn, mask, (const float *)x, (float *)y)));
}

__global__ void k_inject(int64_t nc, const int32_t *__restrict__ map, const double *__restrict__ uf,
                         double *__restrict__ uc) {
  GRID_STRIDE(i, 3 * nc) { uc[i] = uf[(int64_t)map[i / 3] * 3 + i % 3]; }
}

hipError_t launch_inject(int64_t nc, const int32_t *map, const double *uf, double *uc, hipStream_t s) {
  k_inject<<<grid_for(3 * nc), BS, 0, s>>>(nc, map, uf, uc);
  return hipGetLastError();
}

hipError_t launch_cast_state(int64_t n, const double *a, float *b, hipStream_t s) {
  k_cast_d2f<<<grid_for(n), BS, 0, s>>>(n, a, b);
  return hipGetLastError();
}

hipError_t launch_cast(int64_t n, int to_prec, const void *x, void *y, hipStream_t s) {
  if (to_prec == HPMG_F32)
    k_cast_d2f<<<grid_for(n), BS, 0, s>>>(n, (const double *)x, (float *)y);
  else
    k_cast_f2d<<<grid_for(n), BS, 0, s>>>(n, (const float *)x, (double *)y);
  return hipGetLastError();
}

hipError_t launch_axpby(int prec, int64_t n, double a, const void *x, double b, void *y, hipStream_t s) {
  DISPATCH(prec, (k_axpby<double><<<grid_for(n), BS, 0, s>>>(n, a, (const double *)x, b, (double *)y)),
           (k_axpby<float><<<grid_for(n), BS, 0, s>>>(n, (float)a, (const float *)x, (float)b, (float *)y)));
}

hipError_t launch_waxpby(int prec, int64_t n, double a, const void *x, double b, const void *y, void *w,
                         hipStream_t s) {
  DISPATCH(prec,
           (k_waxpby<double><<<grid_for(n), BS, 0, s>>>(n, a, (const double *)x, b, (const double *)y, (double *)w)),
           (k_waxpby<float><<<grid_for(n), BS, 0, s>>>(n, (float)a, (const float *)x, (float)b, (const float *)y,
                                                       (float *)w)));
}

hipError_t launch_recip(int prec, int64_t n, void *x, hipStream_t s) {
  DISPATCH(prec, (k_recip<double><<<grid_for(n), BS, 0, s>>>(n, (double *)x)),
           (k_recip<float><<<grid_for(n), BS, 0, s>>>(n, (float *)x)));
}

hipError_t launch_cheb_first(int prec, int64_t n, const void *dinv, const void *b, void *r, void *d, void *x,
                             double inv_theta, hipStream_t s) {
  DISPATCH(prec,
           (k_cheb_first<double><<<grid_for(n), BS, 0, s>>>(n, (const double *)dinv, (const double *)b, (double *)r,
                                                            (double *)d, (double *)x, inv_theta)),
           (k_cheb_first<float><<<grid_for(n), BS, 0, s>>>(n, (const float *)dinv, (const float *)b, (float *)r,
                                                           (float *)d, (float *)x, (float)inv_theta)));
}

hipError_t launch_dot(int prec, int64_t n, const void *x, const void *y, double *partial, double *out,
                      hipStream_t s) {
  if (prec == HPMG_F64)
    k_dot_partial<double><<<RED_BLOCKS, BS, 0, s>>>(n, (const double *)x, (const double *)y, partial);
  else
    k_dot_partial<float><<<RED_BLOCKS, BS, 0, s>>>(n, (const float *)x, (const float *)y, partial);
  k_final<<<1, RED_BLOCKS, 0, s>>>(partial, RED_BLOCKS, 1, out);
  return hipGetLastError();
}

hipError_t launch_dot_pair(int prec, int64_t n, const void *z, const void *a, const void *b, double *partial,
                           double *out, hipStream_t s) {
  if (prec == HPMG_F64)
    k_dot_pair_partial<double><<<RED_BLOCKS, BS, 0, s>>>(n, (const double *)z, (const double *)a,
                                                         (const double *)b, partial);
  else
    k_dot_pair_partial<float><<<RED_BLOCKS, BS, 0, s>>>(n, (const float *)z, (const float *)a, (const float *)b,
                                                        partial);
  k_final<<<1, RED_BLOCKS, 0, s>>>(partial, RED_BLOCKS, 2, out);
  return hipGetLastError();
}

hipError_t launch_sum(int64_t n, const double *x, double *partial, double *out, hipStream_t s) {
  k_sum_partial<<<RED_BLOCKS, BS, 0, s>>>(n, x, partial);
  k_final<<<1, RED_BLOCKS, 0, s>>>(partial, RED_BLOCKS, 1, out);
  return hipGetLastError();
}

}  // namespace hpmg
