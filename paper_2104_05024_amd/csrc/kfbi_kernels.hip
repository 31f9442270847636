// Interface-side kernels of the KFBI matrix-vector product and the table upload.
//
//  k_correct : density -> right-hand-side correction at irregular grid nodes (Sec. 5.3, eq.
//              correct): rhs_p = sum_arms s_p D_{c,a}/h^2 ([u_a] d + [u_aa] d^2 / 2).  The jumps at
//              the arm's grid-line intersection (single-layer interface problem, Sec. 5.1 eq.
//              single; jump relations from [u] = 0 and [n.D grad u] = psi for diagonal D_c) are
//              weighted sums of the density values of the crossing's transfer stencil, so an arm's
//              whole term is one weighted sum, its weights formed at setup.
//  k_gather  : n.D grad u+ at every interface node from its 6/10-node quadratic fit with the
//              Taylor-expanded jump added to values on the "-" side (Sec. 5.4, eqs. taylor-i-po,
//              taylor-i-co, ji).  The jumps at the node are linear in the density values of its
//              transfer stencil, so the fit is a weighted sum of grid values plus one of density
//              values, the second's weights formed at setup.
//
// Folding the jumps into these weights takes the product of the 256^3 shell from 760 bytes of
// tables per crossing and 1,500 per node to 400 per crossing (200 per arm) and 400 per node, and
// from three launches with two intermediate arrays to two without.
//
// Precision: the density, the weights and the sums are FP64 in every product.  Only the grid side
// follows the product's precision T: the correction is rounded to the T right-hand side that the T
// box solve transforms, and the gather reads the T grid values into its FP64 fit.  The density and
// the result are TP at the boundary (FP32 callers pass theirs, widened and rounded here).
#include <cmath>
#include <type_traits>
#include <stdexcept>

#include "device.h"

namespace kfbi {
namespace {

constexpr int kBlock = 256;

inline unsigned nblk(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// One arm per thread: all of its loads are independent of each other's results but for the
// density values behind their indices.  The arms of a node are consecutive slots within 64 (setup
// pads), and the first of them (count > 0) adds up the others' terms, at most 2D in all.
// One thread per node instead would walk its arms one after the other.
template <typename T, typename TP, int D, int K, int NC>
__device__ __forceinline__ void correct_slot(const InterfaceTables &t, int64_t s, const TP *__restrict__ psi,
                                             int64_t M, T *__restrict__ field, int64_t comp_stride, int accumulate) {
  const int64_t ns = t.n_slots;
  int32_t j[K];
#pragma unroll
  for (int k = 0; k < K; ++k) j[k] = t.arm_idx[k * ns + s];
  const int2 head = reinterpret_cast<const int2 *>(t.arm_head)[s];   // padded position, arms of the node
  double v[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const double *w = t.arm_w + (int64_t)c * K * ns;
    v[c] = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) v[c] += w[k * ns + s] * (double)psi[c * M + j[k]];
  }
  double sum[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) sum[c] = v[c];
#pragma unroll
  for (int i = 1; i < 2 * D; ++i)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const double o = __shfl_down(v[c], i, 64);
      sum[c] += i < head.y ? o : 0.0;
    }
  if (head.y > 0) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      T *o = field + c * comp_stride + head.x;
      *o = accumulate ? (T)(*o + (T)sum[c]) : (T)sum[c];
    }
  }
}

// Sum over the G lanes of a group (G = 8 or 16, aligned); every lane receives the total.
// A butterfly of DPP moves within a row of 16 lanes: swap neighbours, swap pairs (quad
// permutes 1,0,3,2 and 2,3,0,1), then mirror within half rows and within the row, each step
// pairing every lane with one of the other half of its current block.  VALU moves only, so the
// LDS pipe, which a lane shuffle would use, stays free.  Additions are commutative, so every
// lane holds bitwise the same total.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const int2 w = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_update_dpp(0, w.x, CTRL, 0xF, 0xF, false),
                                              __builtin_amdgcn_update_dpp(0, w.y, CTRL, 0xF, 0xF, false)));
}
template <int G>
__device__ __forceinline__ double group_sum(double v) {
  static_assert(G == 8 || G == 16, "group of 8 or 16 lanes");
  v += dpp_f64<0xB1>(v);                           // quad_perm 1,0,3,2
  v += dpp_f64<0x4E>(v);                           // quad_perm 2,3,0,1
  v += dpp_f64<0x141>(v);                          // row_half_mirror
  if constexpr (G >= 16) v += dpp_f64<0x140>(v);   // row_mirror
  return v;
}

constexpr int gather_group(int S) { return S <= 8 ? 8 : 16; }

// n.D_c grad u+ at node q by a group of consecutive lanes: lane k takes stencil point k and
// density point k.  One thread per node leaves the GPU short of parallelism (40,960 nodes are 640
// wavefronts for 1024 SIMDs, each a chain of index, value and sum).  Tables are [node][point], so
// that a group's loads are contiguous.  psi null: the jumps are zero (volume solve).
template <typename TU, typename TP, int S, int KN, int NC>
__device__ __forceinline__ void gather_node(const InterfaceTables &t, int64_t q, int k, const TU *__restrict__ u,
                                            int64_t comp_stride, const TP *__restrict__ psi, int64_t M,
                                            TP *__restrict__ out) {
  const bool us = k < S, ps = psi && k < KN;
  const int32_t pos = us ? t.st_pos[q * S + k] : 0, j = ps ? t.q_idx[q * KN + k] : 0;
  double v[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const double nw = us ? t.st_nw[(c * M + q) * S + k] : 0.0, qw = ps ? t.q_w[(c * M + q) * KN + k] : 0.0;
    v[c] = us ? nw * (double)u[c * comp_stride + pos] : 0.0;
    if (ps) v[c] += qw * (double)psi[c * M + j];
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const double sum = group_sum<gather_group(S)>(v[c]);
    if (k == c) out[c * M + q] = (TP)sum;
  }
}

template <typename T, typename TP, int D, int K, int NC>
__global__ __launch_bounds__(kBlock) void k_correct(InterfaceTables t, const TP *__restrict__ psi, int64_t M,
                                                    T *__restrict__ field, int64_t comp_stride, int accumulate) {
  const int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (s < t.n_slots) correct_slot<T, TP, D, K, NC>(t, s, psi, M, field, comp_stride, accumulate);
}

template <typename TU, typename TP, int S, int KN, int NC>
__global__ __launch_bounds__(kBlock) void k_gather(InterfaceTables t, const TU *__restrict__ u, int64_t comp_stride,
                                                   const TP *__restrict__ psi, int64_t M, TP *__restrict__ out) {
  constexpr int G = gather_group(S);
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x, q = i / G;
  if (q < M) gather_node<TU, TP, S, KN, NC>(t, q, (int)(i % G), u, comp_stride, psi, M, out);
}

// Batched 2D forms: block b of the launch is block blocks[b].y of problem blocks[b].x (a table, read
// with one scalar load, where a search over prefix sums was a chain of loads per thread).
template <typename T, typename TP>
__global__ __launch_bounds__(kBlock) void k_batch_correct(const BatchItem<T> *__restrict__ items,
                                                          const int2 *__restrict__ blocks,
                                                          const TP *__restrict__ psi, int into_fpad) {
  const int2 b = blocks[blockIdx.x];
  const BatchItem<T> &it = items[b.x];
  const int64_t s = (int64_t)b.y * kBlock + threadIdx.x;
  if (s < it.tab.n_slots)
    correct_slot<T, TP, 2, 4, 1>(it.tab, s, psi + it.ioff, it.M, into_fpad ? it.fpad : it.rhs, 0, into_fpad);
}

template <typename T, typename TP>
__global__ __launch_bounds__(kBlock) void k_batch_gather(const BatchItem<T> *__restrict__ items,
                                                         const int2 *__restrict__ blocks,
                                                         const TP *__restrict__ psi, TP *__restrict__ out) {
  const int2 b = blocks[blockIdx.x];
  const BatchItem<T> &it = items[b.x];
  constexpr int G = gather_group(6);
  const int64_t i = (int64_t)b.y * kBlock + threadIdx.x, q = i / G;
  if (q < it.M)
    gather_node<T, TP, 6, 5, 1>(it.tab, q, (int)(i % G), it.work, 0, psi ? psi + it.ioff : nullptr, it.M,
                                out + it.ioff);
}

template <typename T>
T *dalloc(size_t n) {
  T *p = nullptr;
  if (n == 0) n = 1;
  KFBI_HIP(hipMalloc(&p, n * sizeof(T)));
  return p;
}
template <typename T>
T *dupload(const std::vector<T> &v) {
  T *p = dalloc<T>(v.size());
  if (!v.empty()) KFBI_HIP(hipMemcpy(p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
  return p;
}
template <typename T>
std::vector<T> cast_vec(const std::vector<double> &v) {
  return std::vector<T>(v.begin(), v.end());
}

// DST tables in FP64 as built on the host; every precision keeps its copy, its fields and its rhs.
struct NumTables {
  std::vector<double> tw, sp;
};

template <typename T>
void upload_prec(DevProblem &p, PrecTables<T> &tb, const NumTables &h) {
  tb.tw = dupload(cast_vec<T>(h.tw));
  tb.sp = dupload(cast_vec<T>(h.sp));
  const size_t field = (size_t)p.ncomp * p.comp_stride;
  tb.rhs = dalloc<T>(field);
  tb.work = dalloc<T>(field);
  KFBI_HIP(hipMemset(tb.rhs, 0, field * sizeof(T)));
  KFBI_HIP(hipMemset(tb.work, 0, field * sizeof(T)));
  if (p.dim == 3) {
    if (sizeof(T) == sizeof(double) && p.ncomp == 2) {
      tb.gbuf = dalloc<T>((size_t)p.comp_stride);
      KFBI_HIP(hipMemset(tb.gbuf, 0, (size_t)p.comp_stride * sizeof(T)));
    }
  }
}

template <typename T>
void free_prec(PrecTables<T> &tb) {
  T **all[] = {&tb.tw, &tb.sp, &tb.rhs, &tb.work, &tb.gbuf};
  for (T **q : all) {
    if (*q) (void)hipFree(*q);
    *q = nullptr;
  }
}

}  // namespace

template <typename T, typename TP>
static void correct_into(DevProblem &p, const TP *psi, T *field, int accumulate, hipStream_t st) {
  const InterfaceTables &t = p.itab;
  if (t.n_slots == 0) return;
  const unsigned g = nblk(t.n_slots);
  const int64_t cs = p.comp_stride;
  if (p.dim == 2) {
    if (p.ncomp == 2) k_correct<T, TP, 2, 4, 2><<<g, kBlock, 0, st>>>(t, psi, p.M, field, cs, accumulate);
    else k_correct<T, TP, 2, 4, 1><<<g, kBlock, 0, st>>>(t, psi, p.M, field, cs, accumulate);
  } else {
    if (p.ncomp == 2) k_correct<T, TP, 3, kLsqNodes, 2><<<g, kBlock, 0, st>>>(t, psi, p.M, field, cs, accumulate);
    else k_correct<T, TP, 3, kLsqNodes, 1><<<g, kBlock, 0, st>>>(t, psi, p.M, field, cs, accumulate);
  }
  KFBI_HIP(hipGetLastError());
}

template <typename T, typename TP>
void launch_correct(DevProblem &p, const TP *psi, hipStream_t st) {
  correct_into<T, TP>(p, psi, p.tab<T>().rhs, 0, st);
}
template void launch_correct<double, double>(DevProblem &, const double *, hipStream_t);
template void launch_correct<float, double>(DevProblem &, const double *, hipStream_t);
template void launch_correct<float, float>(DevProblem &, const float *, hipStream_t);

void launch_add_correction(DevProblem &p, const double *psi, double *field_padded, hipStream_t st) {
  correct_into<double, double>(p, psi, field_padded, 1, st);
}

template <typename T, typename TP>
void launch_gather(DevProblem &p, const T *u, const TP *psi, TP *out, hipStream_t st) {
  const unsigned g = nblk(p.M * gather_group(p.S));
  const InterfaceTables &t = p.itab;
  const int64_t cs = p.comp_stride;
  if (p.dim == 2) {
    if (p.ncomp == 2) k_gather<T, TP, 6, 5, 2><<<g, kBlock, 0, st>>>(t, u, cs, psi, p.M, out);
    else k_gather<T, TP, 6, 5, 1><<<g, kBlock, 0, st>>>(t, u, cs, psi, p.M, out);
  } else {
    if (p.ncomp == 2) k_gather<T, TP, 10, kLsqNodes, 2><<<g, kBlock, 0, st>>>(t, u, cs, psi, p.M, out);
    else k_gather<T, TP, 10, kLsqNodes, 1><<<g, kBlock, 0, st>>>(t, u, cs, psi, p.M, out);
  }
  KFBI_HIP(hipGetLastError());
}
template void launch_gather<double, double>(DevProblem &, const double *, const double *, double *, hipStream_t);
template void launch_gather<float, double>(DevProblem &, const float *, const double *, double *, hipStream_t);
template void launch_gather<float, float>(DevProblem &, const float *, const float *, float *, hipStream_t);

int correct_blocks(const DevProblem &p) { return (int)nblk(p.itab.n_slots); }
int gather_blocks(const DevProblem &p) { return (int)nblk(p.M * gather_group(p.S)); }

template <typename T, typename TP>
void launch_batch_correct(const BatchItem<T> *items, const BatchBlocks &b, const TP *psi, bool into_fpad,
                          hipStream_t st) {
  if (b.n == 0) return;
  k_batch_correct<T, TP><<<(unsigned)b.n, kBlock, 0, st>>>(items, b.ref, psi, into_fpad ? 1 : 0);
  KFBI_HIP(hipGetLastError());
}
template <typename T, typename TP>
void launch_batch_gather(const BatchItem<T> *items, const BatchBlocks &b, const TP *psi, TP *out, hipStream_t st) {
  if (b.n == 0) return;
  k_batch_gather<T, TP><<<(unsigned)b.n, kBlock, 0, st>>>(items, b.ref, psi, out);
  KFBI_HIP(hipGetLastError());
}
#define KFBI_BATCH_LAUNCH(T, TP)                                                                                 \
  template void launch_batch_correct<T, TP>(const BatchItem<T> *, const BatchBlocks &, const TP *, bool, hipStream_t); \
  template void launch_batch_gather<T, TP>(const BatchItem<T> *, const BatchBlocks &, const TP *, TP *, hipStream_t);
KFBI_BATCH_LAUNCH(double, double)
KFBI_BATCH_LAUNCH(float, double)
KFBI_BATCH_LAUNCH(float, float)
#undef KFBI_BATCH_LAUNCH

// Jump-relation coefficients of one component at a point with normal n and shape operator W
// (diagonal conductivity Dv): with a = psi / (n.D n),
//   [grad u] = a n,
//   [Hess u] = a W + n b^T + b n^T + c n n^T,  b = (g - 2 a W D n) / (n.D n),
//   c = (-a tr(D W) - 2 b.D n) / (n.D n),
// written as [Hess u]_ab = psi alpha_ab + sum_f g_f beta_ab,f (g = surface gradient of psi).
struct JumpCoef {
  int d;
  double nDn, n[3], Dn[3], WDn[3], W[9], trDW, WDnDn;
  JumpCoef(int d_, const double *nrm, const double *Wm, const double *Dv) : d(d_) {
    nDn = 0;
    for (int a = 0; a < d; ++a) {
      n[a] = nrm[a];
      Dn[a] = Dv[a] * nrm[a];
      nDn += n[a] * Dn[a];
    }
    trDW = 0;
    WDnDn = 0;
    for (int a = 0; a < d; ++a) {
      WDn[a] = 0;
      for (int b = 0; b < d; ++b) {
        W[a * d + b] = Wm[a * d + b];
        WDn[a] += Wm[a * d + b] * Dn[b];
      }
      trDW += Dv[a] * Wm[a * d + a];
    }
    for (int a = 0; a < d; ++a) WDnDn += WDn[a] * Dn[a];
  }
  double grad(int a) const { return n[a] / nDn; }
  double alpha(int a, int b) const {
    return (W[a * d + b] - 2.0 * (n[a] * WDn[b] + WDn[a] * n[b]) / nDn - trDW * n[a] * n[b] / nDn +
            4.0 * WDnDn * n[a] * n[b] / (nDn * nDn)) / nDn;
  }
  double beta(int a, int b, int f) const {
    return ((a == f ? n[b] : 0.0) + (b == f ? n[a] : 0.0)) / nDn - 2.0 * Dn[f] * n[a] * n[b] / (nDn * nDn);
  }
};

void upload_tables(DevProblem &p) {
  const HostTables &t = p.ht;
  const int d = t.dim, nc_ = t.ncomp;
  p.dim = d;
  p.ncomp = nc_;
  p.N = t.N;
  p.M = t.M;
  p.Mfft = t.cells;
  p.P = t.cells;
  p.comp_stride = p.P * (d == 3 ? p.N * p.N : p.N);
  p.S = t.S;
  p.h = t.h;
  p.kappa = t.kappa;
  for (int c = 0; c < 2; ++c)
    for (int a = 0; a < 3; ++a) p.D[c][a] = t.D[c < nc_ ? c : 0][a < d ? a : 0];
  p.lam_scale = 1.0;
  for (int a = 0; a < d; ++a) p.lam_scale *= 2.0 / (double)t.cells;
  p.columns = column_direct(d, nc_, t.cells, t.h, p.D, t.kappa);
  const int64_t N = p.N, M = p.M, nc = t.nc, P = p.P, K = t.K, Kn = t.Kn, S = t.S;
  auto padpos = [&](int64_t lin) { return (lin % N) + P * (lin / N); };
  if (padpos(N * (d == 3 ? N * N : N) - 1) >= (int64_t)1 << 31) throw std::invalid_argument("grid too large");
  NumTables h;

  // Correction records.  The arm of a crossing at node p (tissue side: s = +1) adds
  //   s D_{c,a} / h^2 ([u_a] d + [u_aa] d^2 / 2),  [u_a] = sum_k w0_k grad_a psi_k,
  //   [u_aa] = sum_k (w0_k alpha_aa + sum_f wg_kf beta_aa,f) psi_k,
  // a = the crossing's axis, so it is one weight per density point of the crossing's stencil.
  // Arms of a node take consecutive slots that do not straddle a multiple of 64.
  std::vector<std::vector<int64_t>> arms_of(t.irregular.size());
  auto rank = [&](int64_t lin) {
    return (int64_t)(std::lower_bound(t.irregular.begin(), t.irregular.end(), lin) - t.irregular.begin());
  };
  for (int64_t c = 0; c < nc; ++c) {
    arms_of[rank(t.c_pin[c])].push_back(2 * c);       // tissue-side node, s = +1
    arms_of[rank(t.c_pout[c])].push_back(2 * c + 1);  // "-"-side node, s = -1
  }
  const double ih2 = 1.0 / (t.h * t.h);
  auto coord = [&](int64_t lin, int a) {
    int64_t r = lin;
    for (int b = 0; b < a; ++b) r /= N;
    return t.lo + t.h * (double)(r % N + 1);
  };
  std::vector<int64_t> slot_of(t.irregular.size());
  int64_t ns = 0;
  for (size_t r = 0; r < t.irregular.size(); ++r) {
    const int64_t n = (int64_t)arms_of[r].size();
    if (n > 2 * d) throw std::logic_error("a grid node with more arms than directions");
    if (ns % 64 + n > 64) ns = (ns + 63) / 64 * 64;
    slot_of[r] = ns;
    ns += n;
  }
  ns = (ns + 63) / 64 * 64;
  std::vector<int32_t> arm_idx((size_t)K * ns, 0), arm_head((size_t)2 * ns, 0);
  std::vector<double> arm_w((size_t)nc_ * K * ns, 0.0);
  for (size_t r = 0; r < t.irregular.size(); ++r) {
    arm_head[2 * slot_of[r]] = (int32_t)padpos(t.irregular[r]);
    arm_head[2 * slot_of[r] + 1] = (int32_t)arms_of[r].size();
    for (size_t i = 0; i < arms_of[r].size(); ++i) {
      const int64_t c = arms_of[r][i] / 2, s = slot_of[r] + (int64_t)i;
      const bool plus = (arms_of[r][i] % 2) == 0;
      const int a = (int)t.c_axis[c];
      const double dist = coord(plus ? t.c_pout[c] : t.c_pin[c], a) - t.c_z[c * d + a];
      for (int k = 0; k < K; ++k) arm_idx[k * ns + s] = (int32_t)t.z_idx[c * K + k];
      for (int comp = 0; comp < nc_; ++comp) {
        const JumpCoef jc(d, &t.c_n[c * d], &t.c_W[c * d * d], t.D[comp]);
        const double al = jc.alpha(a, a), sc = (plus ? ih2 : -ih2) * t.D[comp][a];
        for (int k = 0; k < K; ++k) {
          const double w0 = t.z_w0[c * K + k];
          double bk = w0 * al;
          for (int f = 0; f < d; ++f) bk += t.z_wg[(c * K + k) * d + f] * jc.beta(a, a, f);
          arm_w[((size_t)comp * K + k) * ns + s] = sc * (w0 * jc.grad(a) * dist + 0.5 * bk * dist * dist);
        }
      }
    }
  }
  // Gather tables [node][point]: st_nw[comp] = n . D_comp (gradient weights of the stencil node), and
  // the jumps the fit adds on its "-" side points r_j,  sum_j nw_j (r.[grad u] + r.[Hess u] r / 2),
  // as one weight q_w per density point of the node's stencil.
  std::vector<int32_t> st_pos(M * S), q_idx(M * Kn);
  std::vector<double> st_nw((size_t)nc_ * M * S), q_w((size_t)nc_ * M * Kn);
  for (int64_t q = 0; q < M; ++q) {
    int self = -1;
    for (int k = 0; k < Kn; ++k) {
      q_idx[q * Kn + k] = (int32_t)t.q_idx[q * Kn + k];
      if (t.q_idx[q * Kn + k] == q && self < 0) self = k;
    }
    if (self < 0) throw std::logic_error("a node's transfer stencil without the node");
    for (int j = 0; j < S; ++j) st_pos[q * S + j] = (int32_t)padpos(t.st_lin[q * S + j]);
    for (int comp = 0; comp < nc_; ++comp) {
      const JumpCoef jc(d, &t.nrm[q * d], &t.W[q * d * d], t.D[comp]);
      double rg[3] = {0, 0, 0}, rh[3][3] = {};
      for (int j = 0; j < S; ++j) {
        double nw = 0;
        for (int a = 0; a < d; ++a) nw += t.nrm[q * d + a] * t.D[comp][a] * t.st_wgrad[(q * S + j) * d + a];
        st_nw[((size_t)comp * M + q) * S + j] = nw;
        if (!t.st_chi[q * S + j]) continue;
        const double *r = &t.st_r[(q * S + j) * d];
        for (int a = 0; a < d; ++a) {
          rg[a] += nw * r[a];
          for (int b = 0; b < d; ++b) rh[a][b] += 0.5 * nw * r[a] * r[b];
        }
      }
      double cq = 0, cg[3] = {0, 0, 0};
      for (int a = 0; a < d; ++a) {
        cq += rg[a] * jc.grad(a);
        for (int b = 0; b < d; ++b) {
          cq += rh[a][b] * jc.alpha(a, b);
          for (int f = 0; f < d; ++f) cg[f] += rh[a][b] * jc.beta(a, b, f);
        }
      }
      for (int k = 0; k < Kn; ++k) {
        double w = k == self ? cq : 0.0;
        for (int f = 0; f < d; ++f) w += cg[f] * t.q_wg[(q * Kn + k) * d + f];
        q_w[((size_t)comp * M + q) * Kn + k] = w;
      }
    }
  }
  // DST tables
  const int Mf = p.Mfft;
  h.tw.resize(2 * Mf);
  h.sp.resize(Mf / 2 + 1);
  std::vector<double> lam(N);
  for (int m = 0; m < Mf; ++m) {
    const double ang = -2.0 * M_PI * (double)m / (double)Mf;
    h.tw[2 * m] = std::cos(ang);
    h.tw[2 * m + 1] = std::sin(ang);
  }
  for (int n = 0; n <= Mf / 2; ++n) h.sp[n] = std::sin(M_PI * (double)n / (double)Mf);
  for (int64_t k = 1; k <= N; ++k) {
    const double sn = std::sin((double)k * M_PI / (2.0 * Mf));
    lam[k - 1] = 4.0 / (t.h * t.h) * sn * sn;
  }
  // tissue mask in the padded layout
  std::vector<int8_t> ins_pad((size_t)p.comp_stride, 0);
  for (int64_t lin = 0; lin < (int64_t)t.inside.size(); ++lin) ins_pad[padpos(lin)] = t.inside[lin];

  // sparse matvec rows: irregular-node rows (right-hand side) and stencil rows (output)
  {
    const int64_t planes = d == 3 ? N : 1, rows = planes * N;   // one plane in 2D
    std::vector<uint8_t> min_(rows, 0), mout(rows, 0);
    for (int64_t lin : t.irregular) min_[lin / N] = 1;
    for (int64_t lin : t.st_lin) mout[lin / N] = 1;
    std::vector<int32_t> rin, rout;
    for (int c = 0; c < t.ncomp; ++c)
      for (int64_t r = 0; r < rows; ++r) {
        if (min_[r]) rin.push_back((int32_t)(c * rows + r));
        if (mout[r]) rout.push_back((int32_t)(c * rows + r));
      }
    p.n_rows_in = (int64_t)rin.size();
    p.n_rows_out = (int64_t)rout.size();
    p.rows_in = dupload(rin);
    p.rows_out = dupload(rout);
    auto columns = [&](const std::vector<int32_t> &list, const std::vector<int64_t> &nodes) -> uint64_t * {
      if (d != 3 || p.Mfft < 256) return nullptr;
      const size_t KS = (size_t)p.Mfft / 64;
      std::vector<int64_t> at((size_t)rows, -1);   // place of each row of one component in the list
      const size_t per = list.size() / (size_t)t.ncomp;
      for (size_t i = 0; i < per; ++i) at[(size_t)list[i]] = (int64_t)i;
      std::vector<uint64_t> bits(list.size() * KS, 0);
      for (int64_t lin : nodes) {
        const int64_t x = lin % N, i = at[(size_t)(lin / N)];
        for (int c = 0; c < t.ncomp; ++c)
          bits[((size_t)c * per + (size_t)i) * KS + (size_t)(x >> 6)] |= uint64_t(1) << (x & 63);
      }
      return dupload(bits);
    };
    // listed row of each arm slot, first slot of each listed row (of one component: the same in the other)
    const size_t per = rin.size() / (size_t)t.ncomp;
    std::vector<int32_t> place((size_t)rows, 0), arm_row((size_t)ns, 0), row_slot(per + 1, (int32_t)ns);
    for (size_t i = 0; i < per; ++i) place[(size_t)rin[i]] = (int32_t)i;
    for (size_t r = t.irregular.size(); r-- > 0;) {
      const int32_t i = place[(size_t)(t.irregular[r] / N)];
      for (size_t a = 0; a < arms_of[r].size(); ++a) arm_row[(size_t)slot_of[r] + a] = i;
      row_slot[(size_t)i] = (int32_t)slot_of[r];
    }
    p.itab.arm_row = dupload(arm_row);
    p.itab.row_slot = dupload(row_slot);
    p.cols_in = columns(rin, t.irregular);
    p.cols_out = columns(rout, t.st_lin);
    std::vector<uint64_t> bin((size_t)planes * 16, 0), bout((size_t)planes * 16, 0);
    for (int64_t r = 0; r < rows; ++r) {
      const int64_t z = r / N, y = r % N;
      if (min_[r]) bin[(size_t)z * 16 + (y >> 6)] |= uint64_t(1) << (y & 63);
      if (mout[r]) bout[(size_t)z * 16 + (y >> 6)] |= uint64_t(1) << (y & 63);
    }
    p.mask_in = dupload(bin);
    p.mask_out = dupload(bout);
    std::vector<uint8_t> pin(planes, 0), pout(planes, 0);
    for (int64_t r = 0; r < rows; ++r) {
      if (min_[r]) pin[r / N] = 1;
      if (mout[r]) pout[r / N] = 1;
    }
    auto listed = [&](const std::vector<uint8_t> &f, int &n) {
      std::vector<int32_t> zs;
      for (int64_t z = 0; z < planes; ++z)
        if (f[z]) zs.push_back((int32_t)z);
      n = (int)zs.size();
      return dupload(zs);
    };
    p.zlist_in = listed(pin, p.n_planes_in);
    p.zlist_out = listed(pout, p.n_planes_out);
    p.planes_in_bits = PlaneBits{};
    p.planes_out_bits = PlaneBits{};
    for (int64_t z = 0; z < planes; ++z) {
      if (pin[z]) p.planes_in_bits.w[z >> 6] |= uint64_t(1) << (z & 63);
      if (pout[z]) p.planes_out_bits.w[z >> 6] |= uint64_t(1) << (z & 63);
    }
  }
  p.itab.n_slots = ns;
  p.itab.arm_idx = dupload(arm_idx);
  p.itab.arm_head = dupload(arm_head);
  p.itab.arm_w = dupload(arm_w);
  p.itab.st_pos = dupload(st_pos);
  p.itab.st_nw = dupload(st_nw);
  p.itab.q_idx = dupload(q_idx);
  p.itab.q_w = dupload(q_w);
  p.inside_pad = dupload(ins_pad);
  p.lam = dupload(lam);
  upload_prec<double>(p, p.f64, h);
  upload_prec<float>(p, p.f32, h);
  p.red = dalloc<double>(4096);
  KFBI_HIP(hipHostMalloc(&p.host_red, 4096 * sizeof(double), hipHostMallocDefault));
  Timer *ts[] = {&p.t_dst_x, &p.t_dst_y, &p.t_dst_last, &p.t_correct, &p.t_gather, &p.t_dst_x_correct, &p.t_dst_x_rows,
                 &p.t_dst_y_sparse, &p.t_dst_last_sparse, &p.t_dst_last_out, &p.t_dst_x_fhn, &p.t_dst_x_fe1,
                 &p.t_dst_y1, &p.t_dst_last_anti, &p.t_dst_last_diff, &p.t_dst_x_be1, &p.t_dst_last_comb};
  for (Timer *tm : ts) tm->create();
}

void free_tables(DevProblem &p) {
  int32_t **ip[] = {&p.itab.arm_idx, &p.itab.arm_head, &p.itab.st_pos, &p.itab.q_idx,
                    &p.itab.arm_row, &p.itab.row_slot,
                    &p.rows_in,      &p.rows_out,      &p.zlist_in,    &p.zlist_out};
  double **wp[] = {&p.itab.arm_w, &p.itab.st_nw, &p.itab.q_w};
  for (double **q : wp) {
    if (*q) (void)hipFree(*q);
    *q = nullptr;
  }
  p.itab.n_slots = 0;
  uint64_t **bp[] = {&p.mask_in, &p.mask_out, &p.cols_in, &p.cols_out};
  for (uint64_t **q : bp) {
    if (*q) (void)hipFree(*q);
    *q = nullptr;
  }
  for (int32_t **q : ip) {
    if (*q) (void)hipFree(*q);
    *q = nullptr;
  }
  if (p.inside_pad) (void)hipFree(p.inside_pad);
  if (p.lam) (void)hipFree(p.lam);
  if (p.red) (void)hipFree(p.red);
  if (p.host_red) (void)hipHostFree(p.host_red);
  p.inside_pad = nullptr;
  p.lam = nullptr;
  p.red = nullptr;
  p.host_red = nullptr;
  free_prec(p.f64);
  free_prec(p.f32);
  Timer *ts[] = {&p.t_dst_x, &p.t_dst_y, &p.t_dst_last, &p.t_correct, &p.t_gather, &p.t_dst_x_correct, &p.t_dst_x_rows,
                 &p.t_dst_y_sparse, &p.t_dst_last_sparse, &p.t_dst_last_out, &p.t_dst_x_fhn, &p.t_dst_x_fe1,
                 &p.t_dst_y1, &p.t_dst_last_anti, &p.t_dst_last_diff, &p.t_dst_x_be1, &p.t_dst_last_comb};
  for (Timer *tm : ts) tm->destroy();
}

}  // namespace kfbi
