// Internal declarations shared by the host library and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>

#include "../../include/hpmg.h"

namespace hpmg {

// ---------------------------------------------------------------------------------
// Quadrature tiling.  Quadrature-point arrays (geometric factors, stored
// linearisation) are laid out [tile][field][field_stride(Q)], the first ET * Q^3 of a field
// its points: the ET consecutive elements of a tile are processed by one workgroup with one
// thread per quadrature point, so each field is read by one contiguous, fully coalesced
// sweep of the workgroup.
// ---------------------------------------------------------------------------------
// Workgroups of 256 threads (Q = 5: of 250 points); at Q = 4 an element's 64 points are one
// wave, whose workgroup needs no barriers: against four elements a workgroup, Q3 applies on
// 30^3 elements in FP32 38.8 -> 37.4 us and the FP32 adjoint on 23^3 30.6 -> 29.3, FP64 alike
// (71.4).  Measured and not better: one or three elements at Q = 5 (Q4 34^3 FP64 205.1 and
// 215.5 against 204.3 us), half-sized workgroups at Q = 2 and 3 (within 3 % either way).
constexpr int elems_per_tile(int Q) {
  return Q == 2 ? 32 : Q == 3 ? 9 : Q == 4 ? 1 : Q == 5 ? 2 : 1;
}
constexpr int tile_threads(int Q) {
  return ((elems_per_tile(Q) * Q * Q * Q + 63) / 64) * 64;
}

// Distance between the fields of a tile: its points rounded up to whole 128-byte lines in
// either precision, so that a wave's load of a field covers the fewest lines (Q = 5: 256
// for 250 points).  Unpadded, FP64 and FP32 Q4 applies on 34^3 elements took 216 and 124 us
// against 208 and 118, Q2 on 43^3 in FP32 50.5 against 49.4; the padding is 2.4 % (Q = 5),
// 5 % (Q = 3) and 4 % (Q = 6) of the arrays.
constexpr int field_stride(int Q) { return (elems_per_tile(Q) * Q * Q * Q + 31) / 32 * 32; }

constexpr int NGEO = 10;    // W, dxi_k/dX_J (row-major)
// Stored linearisation per point: sqrt(W) dxi_k/dx_j (9), tau (xx yy zz yz xz xy),
// lambda log J.  Every use is W times a form bilinear in dxi/dx, so the weight rides in
// the scaled dxi/dx and is not stored (16 scalars instead of 17).
constexpr int NSTATE = 16;
constexpr int NINIT = 26;   // grad_X u (9), C^-1 (6), lambda log J (1), dxi/dx (9), J - 1 (1)

// Reference tables, in the operator's precision, at fixed offsets (max 8 x 8 each).
constexpr int TAB_B = 0;      // [Q][P] interpolation
constexpr int TAB_G = 64;     // [Q][P] reference derivative
constexpr int TAB_D = 128;    // [Q][Q] collocated derivative
constexpr int TAB_W = 192;    // [Q]    1D Gauss weights
constexpr int TAB_BB = 200;   // [Q][P] B*B   (elementwise, diagonal assembly)
constexpr int TAB_BG = 264;   // [Q][P] B*G
constexpr int TAB_GG = 328;   // [Q][P] G*G
constexpr int TAB_CTOF = 392; // [Pf][P] interpolation from this order to order Pf - 1,
                              // slot (Pf - 2) of 64 values, Pf = P+1 .. 6
constexpr int TAB_SIZE = 392 + 5 * 64;
__host__ __device__ constexpr int tab_ctof(int Pf) { return TAB_CTOF + (Pf - 2) * 64; }

// Element-to-node map used by the kernels: node id in the low 28 bits, the Dirichlet
// flags of the node's three components in bits 28..30.
constexpr uint32_t EMAP_ID_MASK = (1u << 28) - 1u;
constexpr int EMAP_BC_SHIFT = 28;
// Set on exactly one record of every node (its first record in element order): the
// element that writes the node in the p-transfers.
constexpr uint32_t EMAP_OWNER = 1u << 31;
constexpr int64_t MAX_NODES = int64_t(1) << 28;

constexpr int RED_BLOCKS = 512;  // fixed grid of the deterministic reductions

// Device scalar slots of a multigrid handle used by the fused Jacobi-PCG: r.z (2), r.r
// (3), breakdown flag (5), r.z of the current iteration, alternating (8, 9), stop flag
// (10), completed iterations (11), r.r of the start (12); per-iteration alpha and beta
// when recorded for the eigenvalue estimate (SC_ALPHA + k, SC_BETA + k, k < PCG_RECORD).
constexpr int SC_STOP = 10, SC_COUNT = 11, SC_RR0 = 12;
// Flexible CG (FP64, device scalars): p.q, r.r of the new residual, breakdown flag,
// alpha, z.r_new and z.r_old of the Polak-Ribiere beta, r.z alternating (FCG_RZ + 0, 1).
constexpr int FCG_PQ = 13, FCG_RR = 14, FCG_BRK = 15, FCG_ALPHA = 16, FCG_ZRN = 17, FCG_ZR = 18, FCG_RZ = 19;
// Set when a workgroup of the one-launch coarse solve gave up waiting for the others.
constexpr int SC_LOST = 21;
constexpr int PCG_RECORD = 64;
constexpr int SC_ALPHA = 32, SC_BETA = SC_ALPHA + PCG_RECORD, SC_N = SC_BETA + PCG_RECORD;

}  // namespace hpmg

struct hpmg_op_s {
  int P = 0, Q = 0;
  int64_t E = 0, N = 0;
  const int32_t *elem_nodes = nullptr;
  const uint8_t *mask = nullptr;
  hpmg_op_s *fine = nullptr;  // non-null for coarse operators
  double mu = 0.0, lam = 0.0;
  const double *mu_e = nullptr, *lam_e = nullptr;
  int ET = 0, NQ = 0, NT = 0;
  int64_t tiles = 0;
  // workspace carve-up
  char *ws = nullptr;
  size_t ws_bytes = 0;
  double *tab64 = nullptr;
  float *tab32 = nullptr;
  uint32_t *emap = nullptr;
  double *geo = nullptr;       // fine only
  double *state64 = nullptr;   // fine only
  double *sinit = nullptr;     // fine only, caller-provided: [tile][26][field_stride] (hpmg_state_initial)
  bool sinit_ready = false;
  float *state32 = nullptr;    // fine only
  double *scratch = nullptr;   // reductions
  int32_t *csr_off = nullptr;  // node -> incidences (element-local records), [N + 1]
  int32_t *csr_inc = nullptr;  // record index e * P^3 + a, sorted per node, [E * P^3]
  double *evec = nullptr;      // element output records [E][P^3][3] (FP64 or FP32)
  double *elmat = nullptr;     // P = 2 only: element matrices [E][300], upper triangle row-major (FP64 or FP32)
  int elmat_prec = -1;         // precision of the built element matrices (-1: none)
  uint64_t elmat_version = 0;  // state version they were built from
  uint64_t state_version = 0;  // fine operators: bumped at every stored linearisation
  unsigned *flags = nullptr;
  bool geo_ready = false, state_ready = false, state32_ready = false;
  void *host_extra = nullptr;  // host-side tables and scalars owned by the handle
};

namespace hpmg {

// Error reporting (thread-local message).
int fail(int status, const std::string &msg);
int hip_fail(hipError_t e, const char *what);
#define HPMG_HIP(call)                                     \
  do {                                                     \
    hipError_t _e = (call);                                \
    if (_e != hipSuccess) return ::hpmg::hip_fail(_e, #call); \
  } while (0)

// Host tabulation (basis.cpp).
int tabulate(int P, int Q, double *B, double *G, double *D, double *xq, double *wq, double *gll);
int ctof_table(int Pf, int Pc, double *M);

// Launchers (op_kernels.hip / vec_kernels.hip).  All return hipError_t of the launch.
bool supported_pq(int P, int Q);
hipError_t launch_build_emap(const hpmg_op_s &op, hipStream_t s);
hipError_t launch_mark_owners(const hpmg_op_s &op, hipStream_t s);
// Stored-mode apply whose assembly also writes per-workgroup partials of du . y
// (ceil(N / 256) of them, in pq).  With `stop` set, every kernel of the apply returns at once while *stop != 0.
hipError_t launch_jacobian_dot(const hpmg_op_s &op, int prec, const void *du, void *y, double *pq,
                               const double *stop, hipStream_t s);
// Stored-mode apply to a smoother's vector, its assembly finished as a Chebyshev step, the
// first step from a nonzero x, or the residual (k_assemble_smooth); c1, c2: the step's
// factors, c1 = 1 / theta for the first.  SMOOTH_START belongs to launch_restrict.
enum { SMOOTH_STEP, SMOOTH_FIRST, SMOOTH_RESIDUAL, SMOOTH_START };
struct Smooth {
  int kind;
  const void *dinv;
  void *b, *r, *d, *x;
  double c1, c2;
};
hipError_t launch_jacobian_smooth(const hpmg_op_s &op, int prec, const Smooth &sm, hipStream_t s);
// Fused Jacobi-PCG iteration on the slots above; all kernels return at once while
// sc[SC_STOP] != 0.  update2 records alpha in *alpha_rec, dir2 beta in *beta_rec (when
// not null), counts the iteration in sc[SC_COUNT] and sets the stop flag on breakdown
// or when r.r <= rtol2 * sc[SC_RR0] (rtol2 < 0: never).
// The start from x = 0 (x null: not formed): r = b, z = D^-1 r, p = z and the scalars.
hipError_t launch_pcg_start(int prec, int64_t n, const void *dinv, const void *b, void *x, void *r, void *z, void *p,
                            double *partial, double *sc, hipStream_t s);
// FCG steps on the slots above (FP64): update: alpha = r.z / p.q from the device
// scalars (0 on a breakdown, p.q <= 0 or r.z not finite, which sets sc[FCG_BRK]),
// x += alpha p, rn = r - alpha q, sc[FCG_RR] = rn.rn.  dir: beta = (z.rn - z.r) / r.z,
// r.z <- z.rn, p = z + beta p.  r.z of iteration `it` is read from FCG_RZ + (it & 1).
hipError_t launch_fcg_update(int64_t n, double *sc, int it, const double *p, const double *q, double *x,
                             const double *r, double *rn, double *partial, hipStream_t s);
hipError_t launch_fcg_dir(int64_t n, double *sc, int it, const double *z, double *p, hipStream_t s);
// The iteration on an order-1 operator assembled into 3 x 3 blocks (sliced ELL, width W,
// nn nodes): one launch replaces the element kernel, the fused assembly and dir2;
// ell_pcg_blocks(nn, node_major) workgroups write pq_part.  nn = 0 runs only the
// stopping test of the iteration before `it` (to close a batch).  node_major: blocks
// held entry-major over the nodes and a thread per node (else a node's rows contiguous
// and a thread per row), the same choice as the block build's (launch_ell_build).
// By default coarse levels of at least this many nodes are node-major.
constexpr int64_t ELL_NODE_MAJOR_MIN = 65536;
int ell_pcg_blocks(int64_t nn, bool node_major);
hipError_t launch_ell_pcg_apply(int prec, bool node_major, int64_t nn, int W, const int32_t *cols,
                                const void *vals, const void *z, const void *p_old, void *p_new, void *y, double *sc,
                                const double *partial, int it, double rtol2, double *pq_part, hipStream_t s);
// The whole Jacobi-PCG of the same operator in one launch (k_coarse_pcg): `groups`
// workgroups own `rows` consecutive scalar rows each (a multiple of 256, at most
// coarse_pcg_max_rows) and hold them in registers.  cols: uint16 [W][3 nn], where the
// direction of the column's node starts in the row's workgroup: entry 3 n - row0 for a
// node all of whose rows the workgroup owns, else rows + 3 k for node halo_ids[k] of its
// list halo_ids[halo_off[g] .. halo_off[g + 1]).  slots: coarse_pcg_slots(nn) doubles.
// Stops as dir2 does, or after maxit iterations; sets sc[SC_COUNT], and sc[SC_LOST] if a
// workgroup waited longer than `wait` for another (x is then not to be used).  A breakdown
// (p.q in sc[1], else 0 there) leaves x as it is, without update2's step of length zero.
struct CoarsePcg {
  int64_t nn;
  int rows, groups, W, max_halo, maxit;
  long long wait;  // in ticks of the device's 100 MHz clock (COARSE_PCG_TICKS a second), below 2^31
  bool node_major;
  double rtol2;
  const void *vals;
  const uint16_t *cols;
  const int32_t *halo_off, *halo_ids;
  const void *b, *dinv;
  void *x;
  void *z[2];  // exchange buffers, 3 nn values each
  double *slots, *sc;
};
constexpr int COARSE_PCG_W = 27;  // most columns of a row
constexpr double COARSE_PCG_TICKS = 1e8;
// Every workgroup posts its sums in this many places, so that few read the same lines.
constexpr int COARSE_PCG_COPIES = 8;
int coarse_pcg_max_rows(int prec);
size_t coarse_pcg_slots(int64_t nn);
size_t coarse_pcg_lds(int prec, int rows, int max_halo);
hipError_t launch_coarse_pcg(int prec, const CoarsePcg &a, hipStream_t s);
// Assembles the order-1 element matrices of `op` (built in precision prec) into the
// sliced-ELL blocks; constrained rows become identity rows, constrained columns zero.
hipError_t launch_ell_build(const hpmg_op_s &op, int prec, bool node_major, int64_t W, const int32_t *cols,
                            void *vals, hipStream_t s);
hipError_t launch_pcg_update2(int prec, int64_t n, double *sc, int parity, int nb_pq, const double *pq_partial,
                              const void *p, const void *q, void *x, void *r, const void *dinv, void *z,
                              double *partial, double *alpha_rec, hipStream_t s);
hipError_t launch_pcg_dir2(int prec, int64_t n, double *sc, int parity, const double *partial, const void *z,
                           void *p, double rtol2, double *beta_rec, hipStream_t s);
hipError_t launch_inject(int64_t nc, const int32_t *map, const double *uf, double *uc, hipStream_t s);
hipError_t launch_state_initial(const hpmg_op_s &op, const double *u, hipStream_t s);
hipError_t launch_body_load(const hpmg_op_s &op, const double *g, double *f_ext, hipStream_t s);
hipError_t launch_traction_load(const hpmg_op_s &op, const double *X, int64_t nf, const int32_t *face_elem,
                                const int32_t *face_id, const double *t, double *rec, int32_t *rec_node,
                                hipStream_t s);
hipError_t launch_assemble_csr(int64_t N, const int32_t *off, const int32_t *inc, const double *rec,
                               const uint8_t *mask, double *y, hipStream_t s);
hipError_t launch_qdata(const hpmg_op_s &op, const double *coords, hipStream_t s);
hipError_t launch_residual(const hpmg_op_s &op, const double *u, double *r, bool store, hipStream_t s);
hipError_t launch_jacobian(const hpmg_op_s &op, int prec, int mode, const double *u, const void *du,
                           void *y, hipStream_t s);
hipError_t launch_diagonal(const hpmg_op_s &op, int prec, void *diag, hipStream_t s);
hipError_t launch_prolong_add(const hpmg_op_s &coarse, const hpmg_op_s &fine, int prec,
                              const void *xc, void *yf, hipStream_t s);
// start: the coarse residual goes to start->b and the smoother's first step from x = 0 is
// made at once (rc unused).
hipError_t launch_restrict(const hpmg_op_s &fine, const hpmg_op_s &coarse, int prec, const void *rf,
                           void *rc, hipStream_t s, const Smooth *start = nullptr);
hipError_t launch_energy(const hpmg_op_s &op, const double *u, double *psi, hipStream_t s);
hipError_t launch_vjp(const hpmg_op_s &op, int prec, int mode, const double *u, const void *w, void *ub,
                      double *mub, double *lamb, hipStream_t s);
hipError_t launch_export_qdata(const hpmg_op_s &op, double *out, hipStream_t s);
hipError_t launch_elmat_build(const hpmg_op_s &op, int prec, hipStream_t s);

// Vector kernels.
hipError_t launch_init_bc(int prec, int64_t n_nodes, const uint8_t *mask, const void *x, void *y,
                          hipStream_t s);  // y = mask ? x : 0
hipError_t launch_cast_state(int64_t n, const double *a, float *b, hipStream_t s);
hipError_t launch_dot(int prec, int64_t n, const void *x, const void *y, double *partial,
                      double *out, hipStream_t s);
hipError_t launch_sum(int64_t n, const double *x, double *partial, double *out, hipStream_t s);
hipError_t launch_axpby(int prec, int64_t n, double a, const void *x, double b, void *y, hipStream_t s);
hipError_t launch_waxpby(int prec, int64_t n, double a, const void *x, double b, const void *y,
                         void *w, hipStream_t s);  // w = a x + b y
hipError_t launch_dot_pair(int prec, int64_t n, const void *z, const void *a, const void *b,
                           double *partial, double *out, hipStream_t s);  // out = {z.a, z.b}
hipError_t launch_cast(int64_t n, int to_prec, const void *x, void *y, hipStream_t s);
hipError_t launch_recip(int prec, int64_t n, void *x, hipStream_t s);
hipError_t launch_cheb_first(int prec, int64_t n, const void *dinv, const void *b, void *r, void *d, void *x,
                             double inv_theta, hipStream_t s);  // from x = 0


size_t prec_size(int prec);

}  // namespace hpmg
