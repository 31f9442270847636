// Device-side state and kernel launchers of the KFBI library (HIP, gfx950).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "host_tables.h"

namespace kfbi {

struct HipError {
  hipError_t code;
  std::string where;
};

#define KFBI_HIP(call)                                                        \
  do {                                                                        \
    hipError_t e_ = (call);                                                   \
    if (e_ != hipSuccess) throw ::kfbi::HipError{e_, #call};                  \
  } while (0)

// Grid fields inside the library use a padded layout: [comp][z][y][x] with row pitch
// P = N + 1 (a power of two), so that every row starts on a 2 KB (FP64) boundary.
// Caller-visible fields use the unpadded layout (pitch N).

template <typename T>
struct PrecTables {          // per-precision device copies of the DST tables, and the fields
  T *tw = nullptr, *sp = nullptr;        // DST twiddles exp(-2 pi i m/M) (complex) and sin(pi n/M)
  T *rhs = nullptr, *work = nullptr;     // matvec right-hand side (zero off irregular nodes), work field
  T *gbuf = nullptr;                     // coupled 3D FP64: x-y transform of kappa V1 (one component),
                                         // kept from a step's volume solve for its final solve
};

// Per-kernel-class launch timer: HIP events recorded around each launch on the launch
// stream, without synchronising; durations are harvested when queried or when the pool fills.
struct Timer {
  static constexpr int kPairs = 2048;
  std::vector<hipEvent_t> ev;
  int used = 0;
  double total_ms = 0;
  int64_t n = 0;
  void create() {
    ev.resize(2 * kPairs);
    for (auto &e : ev) KFBI_HIP(hipEventCreate(&e));
  }
  void destroy() {
    for (auto &e : ev) (void)hipEventDestroy(e);
    ev.clear();
    used = 0;
  }
  void harvest() {
    for (int i = 0; i < used; ++i) {
      KFBI_HIP(hipEventSynchronize(ev[2 * i + 1]));
      float ms = 0;
      KFBI_HIP(hipEventElapsedTime(&ms, ev[2 * i], ev[2 * i + 1]));
      total_ms += ms;
      ++n;
    }
    used = 0;
  }
  void tic(bool on, hipStream_t st) {
    if (!on) return;
    if (used == kPairs) harvest();
    KFBI_HIP(hipEventRecord(ev[2 * used], st));
  }
  void toc(bool on, hipStream_t st) {
    if (!on) return;
    KFBI_HIP(hipEventRecord(ev[2 * used + 1], st));
    ++used;
  }
  void reset() {
    harvest();
    total_ms = 0;
    n = 0;
  }
};

// A set of z planes as bits (plane z = bit z % 64 of word z / 64; up to 1024 planes), passed to
// kernels by value so that testing a plane needs no memory access.
struct PlaneBits {
  uint64_t w[16] = {};
};

// Device tables of the interface kernels (kfbi_kernels.hip), FP64 weights in every precision.
struct InterfaceTables {
  int64_t n_slots = 0;                               // arms of the irregular nodes, padded to 64s
  int32_t *arm_idx = nullptr, *arm_head = nullptr;   // density points [K][slot]; (position, arms of the node) [slot]
  double *arm_w = nullptr;                           // [comp][K][slot]
  // for the row pass that forms the correction itself: the listed row of each slot, the first slot of each listed
  // row of one component (and the end)
  int32_t *arm_row = nullptr, *row_slot = nullptr;
  int32_t *st_pos = nullptr, *q_idx = nullptr;       // grid and density points of the nodes [M][S], [M][Kn]
  double *st_nw = nullptr, *q_w = nullptr;           // their weights [comp][M][S], [comp][M][Kn]
};

// Rows of padded fields: the indices of some rows (null: every row) and their bits, 16 words per field
// (2D) or plane (3D); cols (optional): the nodes of each listed row that matter, cells / 64 words.
struct RowSet {
  const int32_t *list = nullptr;
  int64_t n = 0;
  const uint64_t *bits = nullptr, *cols = nullptr;
};

// Whether the passes of a 2D product take row sets, by the bytes of its fields (a batch: of all its
// problems).  Below, a pass fits on the GPU at once and the list's load only lengthens it; above, about 30% of
// the rows of the closed curves here are left out.  One product, every row / row sets (us): FP64 128 21.5 /
// 22.9, 256 22.9 / 23.9, 512 (2.1 MB) 27.0 / 27.4, coupled 512 (4.2 MB) 31.6 / 31.0, 1024 35.3 / 33.8, coupled
// 1024 53.4 / 49.5; FP32 coupled 512 (2.1 MB) 29.2 / 29.5, 1024 (4.2 MB) 31.3 / 30.8.
// A batch of 64 (64..1024 cells): x pass 38 -> 30 us and last axis 45 -> 37 in FP32, 72 -> 61 and 60 -> 54 in FP64.
inline bool row_sets_pay(int64_t bytes) { return bytes >= 4000000; }

// Whether box solves take the last axis as tridiagonal columns (column_direct), by type.
struct ColumnRule {
  bool f64 = false, f32 = false;
  template <typename T>
  bool of() const {
    return sizeof(T) == 8 ? f64 : f32;
  }
  bool operator==(const ColumnRule &o) const { return f64 == o.f64 && f32 == o.f32; }
  bool operator<(const ColumnRule &o) const { return f64 != o.f64 ? f64 < o.f64 : f32 < o.f32; }
};

struct DevProblem {
  HostTables ht;
  bool on_device = false;
  int dev = 0;
  int dim = 0, ncomp = 1, Mfft = 0;
  int64_t N = 0, M = 0, P = 0;
  int64_t comp_stride = 0;     // padded elements per component
  int S = 0;                   // extrapolation stencil size
  double h = 0, kappa = 0, D[2][3] = {{1, 1, 1}, {1, 1, 1}};   // diagonal conductivity per component
  double lam_scale = 1;        // (2/M)^d normalisation of the inverse transforms

  InterfaceTables itab;
  int8_t *inside_pad = nullptr;  // padded-layout tissue mask
  // sparse matvec box solve: rows of the flattened [comp][z][y] row list that carry irregular
  // nodes (in) / extrapolation-stencil nodes (out), and their [z][y] bits
  bool sparse = true;
  ColumnRule columns;          // whether the last axis is solved as tridiagonal systems instead of by DSTs
  int32_t *rows_in = nullptr, *rows_out = nullptr;
  int64_t n_rows_in = 0, n_rows_out = 0;
  // columns of each listed row, in 3D from 256 cells on: there about half of a row pass's traffic goes.  Smaller
  // passes wait longer for the words than they save (64^3 4.15 -> 4.7 us, coupled 2D 512 6.05 -> 7.1).
  uint64_t *cols_in = nullptr, *cols_out = nullptr;
  uint64_t *mask_in = nullptr, *mask_out = nullptr;     // [z][16] bit rows: y rows with rhs / stencil nodes
  int32_t *zlist_in = nullptr, *zlist_out = nullptr;     // planes that hold any rhs / stencil row
  int n_planes_in = 0, n_planes_out = 0;
  PlaneBits planes_in_bits, planes_out_bits;             // the same sets as bits
  RowSet set_in() const { return {rows_in, n_rows_in, mask_in, cols_in}; }
  RowSet set_out() const { return {rows_out, n_rows_out, mask_out, cols_out}; }
  double *lam = nullptr;       // (4/h^2) sin^2(k pi / 2M), k = 1..N

  PrecTables<double> f64;
  PrecTables<float> f32;

  // reductions / scratch
  double *red = nullptr;       // small device scratch for dot products
  double *host_red = nullptr;  // pinned host mirror

  // kept for kfbi_get_tiles / kfbi_set_tiles: every pass has one tile shape
  int tile_w[2][3] = {{1, 1, 1}, {1, 1, 1}};

  bool profile = false;
  Timer t_dst_x, t_dst_y, t_dst_last, t_correct, t_gather, t_dst_x_correct, t_dst_x_rows, t_dst_y_sparse, t_dst_last_sparse,
      t_dst_last_out, t_dst_x_fhn, t_dst_x_fe1, t_dst_y1, t_dst_last_anti, t_dst_last_diff, t_dst_x_be1,
      t_dst_last_comb;
  hipStream_t stream = nullptr;

  template <typename T>
  PrecTables<T> &tab();
};

template <>
inline PrecTables<double> &DevProblem::tab<double>() { return f64; }
template <>
inline PrecTables<float> &DevProblem::tab<float>() { return f32; }

// Mode solve parameters of one problem: eigenvalues (4/h^2) sin^2(k pi / 2M), k = 1..N,
// diagonal conductivities of the (one or two) components per axis, kappa, and the (2/M)^d
// factor; the mode sum of component c is sum_a D_{c,a} lambda_{k_a}.
struct ModeParams {
  const double *lam;
  double D0[3], D1[3], kappa, norm;   // conductivity per axis of component 0 and 1
  double h2;                          // h^2 (the direct last-axis solve)
};

// One two-dimensional, one-component problem of a batch as the batched interface kernels see
// it: its tables, its fields inside the size-group buffers, and its offset in the
// concatenated interface vectors.
template <typename T>
struct BatchItem {
  InterfaceTables tab;
  T *rhs, *fpad, *work;        // padded fields inside the group buffers
  int64_t M, ioff;
};

// The blocks of one batched launch: (problem, block within the problem), on the device.
struct BatchBlocks {
  const int2 *ref = nullptr;
  int n = 0;
};

// ---- launchers (defined in dst.hip / kfbi_kernels.hip)
// Box solve: dst = S(src). Layout flags: true = caller (unpadded) layout, false = padded.
template <typename T>
void box_solve(DevProblem &p, const T *src, bool src_plain, T *dst, bool dst_plain, hipStream_t st);

// Box solve of the matrix-vector product: rhs (padded, sparse) -> work (padded); only the
// extrapolation-stencil values of work are meaningful afterwards.
template <typename T, typename TP>
void box_solve_matvec(DevProblem &p, const TP *psi, hipStream_t st);

// Box solve of src (padded) into work when only the extrapolation-stencil values of the result
// are read afterwards (identical there to box_solve).
template <typename T>
void box_solve_stencils(DevProblem &p, const T *src, hipStream_t st);

// 1/x from the hardware reciprocal estimate refined by Newton steps (two in FP64, one in FP32):
// within an ulp or two of the IEEE quotient at a fraction of the cost of a full division.
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  r = fma(r, fma(-x, r, 1.0), r);
  return r;
}
__device__ __forceinline__ float recip(float x) {
  float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.0f), r);
}

// Waits until the step counter *seq_host (pinned host memory, stored by a one-thread kernel with
// a system-scope release after the work it follows) reaches expect: polls it for up to 20 ms,
// then synchronises the stream, which also reports any error.  Returns the counter's value.
int poll_step_counter(const int *seq_host, int expect, hipStream_t st);

// FitzHugh-Nagumo reaction (Sec. 7) and its two half steps in the Strang splitting (Sec. 3):
// forward Euler, and backward Euler with q eliminated and Newton on V.  inv_cm = 1 / C_m and
// inv_den = 1 / (1 + dth zeta) for the half step dth, so that no node divides by constants.
struct FhnCoef {
  double Cm, H, theta, alpha, zeta, tol;
  int maxit;
  double inv_cm, inv_den;
};

// Forward Euler over dth: (v, g) <- (v - dth I_ion(v, g) / C_m, g + dth (alpha v - zeta g)).
__device__ __forceinline__ void fhn_fe(double &v, double &g, double dth, const FhnCoef &m) {
  const double I = m.H * (g - v * (v - m.theta) * (1.0 - v));
  const double v1 = v + dth * (-I * m.inv_cm);
  const double q1 = g + dth * (m.alpha * v - m.zeta * g);
  v = v1;
  g = q1;
}

// Backward Euler over dth from (vb, g): q' = (g + dth alpha V') / (1 + dth zeta) is eliminated
// and Newton solves for V'; it stops once |F| <= tol and takes one more step.
__device__ __forceinline__ void fhn_be(double vb, double g, double dth, const FhnCoef &m, double &V, double &q) {
  const double a = dth * m.alpha * m.inv_den;
  const double qb = g * m.inv_den;
  const double c = dth * m.H * m.inv_cm;
  double x = vb;
  for (int it = 0; it < m.maxit; ++it) {
    const double cub = x * (x - m.theta) * (1.0 - x);
    const double F = x - vb + c * (qb + a * x - cub);
    const double dcub = -3.0 * x * x + 2.0 * (1.0 + m.theta) * x - m.theta;
    const double dF = 1.0 + c * (a - dcub);
    const bool ok = fabs(F) <= m.tol;
    x = x - F * recip(dF);
    if (ok) break;
  }
  V = x;
  q = qb + a * x;
}

// Pointwise state of a coupled bidomain step (caller layout, pitch N) handed to the box
// solves that carry the reaction half steps in their x passes.
struct FhnArgs {
  double *V, *q;
  const double *stim;         // I_stim or null
  double dth, kappa, beta;
  FhnCoef m;
};

// Box solves of a coupled (two-component, FP64) bidomain step whose x passes pair row r of
// component 0 with row r of component 1, so that both potentials of a node share one complex
// value and the pointwise work of the splitting rides in those passes:
//   bidomain_volume_solve: S f for f = (kappa V1, -kappa V1 + beta I), (V1, q1) the forward
//     Euler half step of (V, q), into work (extrapolation-stencil values, as
//     box_solve_stencils); V and q are left unchanged.  Without I (3D, M >= 64) the source is
//     antisymmetric and the forward x and y passes run over the one field kappa V1;
//   bidomain_final_solve: S(f + C psi) with C psi taken from rhs (launch_correct), into work;
//     with fuse_be the inverse x pass instead finishes the step: V <- 2 (u_i - u_e) - V1 and the
//     backward Euler half step from q1 into V and q, and work is left holding the y-inverse
//     output (3D, M >= 64: of u_i - u_e alone, in component 0, the only field the update
//     needs).  Each pass recomputes (V1, q1) from the unchanged (V, q).
void bidomain_volume_solve(DevProblem &p, const FhnArgs &a, hipStream_t st);
void bidomain_final_solve(DevProblem &p, const FhnArgs &a, bool fuse_be, hipStream_t st);

// The correction C psi into the product's right-hand side (overwritten at the irregular nodes), or
// added to a padded field; T the grid side's precision, TP the density's.
template <typename T, typename TP>
void launch_correct(DevProblem &p, const TP *psi, hipStream_t st);
void launch_add_correction(DevProblem &p, const double *psi, double *field_padded, hipStream_t st);
// n.D grad u+ at the nodes from the T grid values u and the jumps of psi (null: none).
template <typename T, typename TP>
void launch_gather(DevProblem &p, const T *u, const TP *psi, TP *out, hipStream_t st);

// Batched 2D launches over all problems: the correction into rhs (overwrite) or fpad (accumulate),
// and the gather from work; psi and out concatenated.
int correct_blocks(const DevProblem &p);   // blocks of one problem in those launches
int gather_blocks(const DevProblem &p);
template <typename T, typename TP>
void launch_batch_correct(const BatchItem<T> *items, const BatchBlocks &b, const TP *psi, bool into_fpad,
                          hipStream_t st);
template <typename T, typename TP>
void launch_batch_gather(const BatchItem<T> *items, const BatchBlocks &b, const TP *psi, TP *out, hipStream_t st);
// Grouped 2D box solve of G equal-size problems (padded layout, stride cs, msv on the device), one
// launch per pass; direct: the last axis solved directly.  Where it is, `in` and `out` may name the rows
// outside which the source is zero and the rows the result is read on (row sets of the whole group).
// Merged: several such groups (each with its own size) in one launch per pass, so the tiles of small grids
// run beside those of large ones instead of in launches of their own that cannot fill the GPU.
// Sizes 64..1024, all direct or none; the groups are those of one precision.  Same results.
struct MultiGroupDesc {
  int Mfft = 0, G = 0;
  bool direct = true;
  int64_t cs = 0;
  const void *src = nullptr;
  void *dst = nullptr;
  const ModeParams *msv = nullptr;
  const void *tw = nullptr, *sp = nullptr;
  RowSet in, out;
};
constexpr int kMaxMultiGroups = 8;
template <typename T>
void box_solve_group(const MultiGroupDesc &d, hipStream_t st);
template <typename T>
void box_solve_multi(const MultiGroupDesc *groups, int ngroups, hipStream_t st);

// The last axis of a box solve as tridiagonal systems along its columns (lastaxis.hip): in -> out
// (may alias), padded layout.  Forms as in the DST pass: 0-2 by the plane sets given (none; both;
// zout alone), 3-5 those of a bidomain step.
template <typename T>
struct LastAxis {
  const T *in = nullptr;
  T *out = nullptr;
  int dim = 3, ncomp = 1, M = 0;
  int64_t cs = 0;                       // component stride
  ModeParams ms{};
  const ModeParams *msv = nullptr;      // 2D: per-problem parameters of nprob fields at stride pstride
  int nprob = 1;
  int64_t pstride = 0;
  const uint64_t *bin = nullptr, *bout = nullptr;   // 2D: row bits per problem (null: every row)
  const PlaneBits *zin = nullptr, *zout = nullptr;
  int form = 0;
  const T *in2 = nullptr;
};
// Whether the columns are solved directly: where the slowest mode decays across the box, s M^2 >= 2 (the isotropic boxes
// have 9.9 in 2D and 19.7 in 3D, more with a reaction term), and from 6 on in FP64 up to 32 cells.  Below that the
// starting values come out of a difference of nearly equal sums, whose error the transforms' exceeds on larger grids
// and in FP32 only.  Root mean square over seeded smooth sources, columns / transforms: FP64 at s M^2 2.1, 3 and 5,
// 16^2 2.45, 1.20 and 1.11, 32^2 1.24, 1.20 and 0.98, 32^3 1.18, 1.14 and 1.02; 64^2 0.96, 0.91 and 0.87, 64^3 0.92, 0.88
// and 0.90, 256^2 0.81, 0.73 and 0.73; FP32 0.55 to 0.82 at any size and s M^2.  So boxes whose last axis conducts more
// than five (2D) or ten (3D) times the others keep the transforms (FP64 up to 32 cells 1.6 and 3.3 times), as do
// reaction terms so large (s >= 1e12) that mu drops out of the recursions.
ColumnRule column_direct(int dim, int ncomp, int M, double h, const double D[2][3], double kappa);
template <typename T>
void last_axis_direct(const LastAxis<T> &l, hipStream_t st);
template <typename T>
void last_axis_direct_multi(const MultiGroupDesc *groups, int ngroups, hipStream_t st);
void upload_tables(DevProblem &p);
void free_tables(DevProblem &p);

}  // namespace kfbi
