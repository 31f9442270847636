// Batched two-dimensional Neumann problems (many interfaces of uneven grid sizes at once).
//
// Every problem keeps its own setup tables; the batch adds
//   * groups: problems with the same grid size and kind of last axis (columns or the fused
//     transform pass) share padded field buffers (stride N * M), so each pass of a group is one
//     launch (blockIdx.y = problem on the last axis, with per-problem mode parameters), or one
//     launch over all groups of a kind from 64 cells on;
//   * work lists: the correction and gather kernels of all problems run as one launch
//     each, a table naming the problem of every block;
//   * GMRES(m) for all problems in lockstep on concatenated vectors [problem][M_p]: per-problem
//     dot products, Gram-Schmidt (two passes), norms and basis updates are segment kernels;
//     the Givens least-squares updates run on the host, one synchronisation per iteration.
//     One Arnoldi step (the batched product, both Gram-Schmidt passes, the norm, v_{j+1}, the
//     new Hessenberg column to pinned host memory and j <- j + 1)
//     reads j from device memory, so a single hipGraph serves every iteration; it is
//     captured on first use and replayed.
//   * mixed precision as for one problem: FP64 residuals and refinement, FP32-operator inner
//     GMRES with per-problem tolerances.
#include <algorithm>
#include <cmath>
#include <memory>
#include <stdexcept>
#include <vector>

#include "arnoldi.h"
#include "batch.h"

namespace kfbi {
namespace {

constexpr int kB = 256;
constexpr int kPackRows = 16;
inline unsigned nb(int64_t n) { return (unsigned)((n + kB - 1) / kB); }

template <typename T>
T *balloc(size_t n) {
  T *p = nullptr;
  KFBI_HIP(hipMalloc(&p, std::max<size_t>(n, 1) * sizeof(T)));
  KFBI_HIP(hipMemset(p, 0, std::max<size_t>(n, 1) * sizeof(T)));
  return p;
}

// out[y * np + p] = <A_y, w> over segment p, for y <= *jlim (all y if jlim is null)
__global__ __launch_bounds__(kB) void k_seg_dot(const double *__restrict__ A, int64_t lda,
                                                const int *__restrict__ jlim, const double *__restrict__ w,
                                                const int64_t *__restrict__ off, int np, double *__restrict__ out) {
  const int p = blockIdx.x, y = blockIdx.y;
  if (jlim && y > *jlim) return;
  __shared__ double sh[kB];
  const int64_t b = off[p], e = off[p + 1];
  const double *a = A + (int64_t)y * lda;
  double s = 0;
  for (int64_t i = b + threadIdx.x; i < e; i += kB) s += a[i] * w[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int o = kB / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[(int64_t)y * np + p] = sh[0];
}

// The orthogonalisation of one Arnoldi step for every problem at once, one workgroup per problem (segments of
// at most 1024 E entries): the coefficients into hcols ([pass][ld][np], then np squared norms), V_{j+1} also into
// vin.  Two launches (with k_end_step), 11.5 and 5.1 us for 64 problems of 128..2048 entries, instead of nine of 3-5 us.
template <int E>
__global__ __launch_bounds__(kSmallThreads) void k_seg_orthogonalise(double *V, int64_t L, const double *w,
                                                                     const int64_t *__restrict__ off,
                                                                     const int *__restrict__ jdev, int ld, int np,
                                                                     double *__restrict__ hcols, double *vin) {
  __shared__ double hcol[2][kSmallColumn];
  const int p = blockIdx.x, K = *jdev + 1;
  const int64_t b = off[p];
  const double nrm2 = orthogonalise_block<E>(V + b, L, w + b, off[p + 1] - b, K, vin + b, hcol);
  for (int k = threadIdx.x; k < K; k += kSmallThreads) {
    hcols[(int64_t)k * np + p] = hcol[0][k];
    hcols[(int64_t)(ld + k) * np + p] = hcol[1][k];
  }
  if (threadIdx.x == 0) hcols[(int64_t)2 * ld * np + p] = nrm2;
}

// w -= sum_{i <= j} h[i][pid] V_i
__global__ __launch_bounds__(kB) void k_seg_combine(double *__restrict__ w, const double *__restrict__ V,
                                                    int64_t L, const int *__restrict__ jdev,
                                                    const double *__restrict__ h, const int16_t *__restrict__ pid,
                                                    int np) {
  const int64_t e = (int64_t)blockIdx.x * kB + threadIdx.x;
  if (e >= L) return;
  const int j = *jdev, p = pid[e];
  double acc = w[e];
  for (int i = 0; i <= j; ++i) acc -= h[(int64_t)i * np + p] * V[(int64_t)i * L + e];
  w[e] = acc;
}

// V_{j+1} = w / sqrt(nn[pid]) (zero where the norm vanishes), also into vin
__global__ __launch_bounds__(kB) void k_seg_next(const double *__restrict__ w, const double *__restrict__ nn,
                                                 const int16_t *__restrict__ pid, double *__restrict__ V, int64_t L,
                                                 const int *__restrict__ jdev, double *__restrict__ vin) {
  const int64_t e = (int64_t)blockIdx.x * kB + threadIdx.x;
  if (e >= L) return;
  const double n2 = nn[pid[e]], v = n2 > 0 ? w[e] / sqrt(n2) : 0.0;
  V[(int64_t)(*jdev + 1) * L + e] = v;
  vin[e] = v;
}

// the step counter: seq <- seq + 1, also stored to the host's copy
__global__ void k_count(int *seq, int *seq_host) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    const int s = *seq + 1;
    *seq = s;
    __threadfence_system();
    __hip_atomic_store(seq_host, s, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// V_0 = r * s[pid] (s = 1/beta, or 0 for problems that are done), also into vin; j <- 0
__global__ __launch_bounds__(kB) void k_seg_scale(const double *__restrict__ r, const double *__restrict__ s,
                                                  const int16_t *__restrict__ pid, double *__restrict__ out,
                                                  double *__restrict__ vin, int *__restrict__ jdev, int64_t L) {
  const int64_t e = (int64_t)blockIdx.x * kB + threadIdx.x;
  if (e == 0) *jdev = 0;
  if (e >= L) return;
  const double v = r[e] * s[pid[e]];
  out[e] = v;
  vin[e] = v;
}

// x += sum_{i < jmax} y[i][pid] V_i
__global__ __launch_bounds__(kB) void k_seg_update(double *__restrict__ x, const double *__restrict__ V, int64_t L,
                                                   const double *__restrict__ y, const int16_t *__restrict__ pid,
                                                   int np, int jmax) {
  const int64_t e = (int64_t)blockIdx.x * kB + threadIdx.x;
  if (e >= L) return;
  const int p = pid[e];
  double acc = x[e];
  for (int i = 0; i < jmax; ++i) acc += y[(int64_t)i * np + p] * V[(int64_t)i * L + e];
  x[e] = acc;
}

__global__ __launch_bounds__(kB) void k_axpby(double *__restrict__ z, double a, const double *__restrict__ x,
                                              double b, const double *__restrict__ y, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
  if (i < n) z[i] = a * x[i] + (y ? b * y[i] : 0.0);
}

// zero the segments of problems whose mask entry is 0
__global__ __launch_bounds__(kB) void k_seg_mask(double *__restrict__ v, const int16_t *__restrict__ pid,
                                                 const double *__restrict__ keep, int64_t L) {
  const int64_t e = (int64_t)blockIdx.x * kB + threadIdx.x;
  if (e < L && keep[pid[e]] == 0.0) v[e] = 0.0;
}

// caller layout (concatenated [problem][N_p^2]) <-> padded group buffers
// block b takes kPackRows grid rows of problem blocks[b].x from row blocks[b].y * kPackRows on, a
// wavefront per row at a time
__global__ __launch_bounds__(kB) void k_pack(double *__restrict__ plain, const int64_t *__restrict__ goff,
                                             const PackItem *__restrict__ it, const int2 *__restrict__ blocks,
                                             int which, int to_padded) {
  const int2 b = blocks[blockIdx.x];
  const PackItem &q = it[b.x];
  double *pad = which == 0 ? q.fpad : q.work;
  double *pl = plain + goff[b.x];
  const int64_t N = q.N;
  for (int r = threadIdx.x / 64; r < kPackRows; r += kB / 64) {
    const int64_t y = (int64_t)b.y * kPackRows + r;
    if (y >= N) break;
    for (int64_t x = threadIdx.x % 64; x < N; x += 64) {
      if (to_padded) pad[y * q.P + x] = pl[y * N + x];
      else pl[y * N + x] = pad[y * q.P + x];
    }
  }
}

}  // namespace

void Batch::init(int n, const kfbi_interface *ifaces, const kfbi_grid *grids, const kfbi_coeffs *coeffs) {
  if (n < 1 || n > 32767) throw std::invalid_argument("batch size");
  np = n;
  probs.resize(n);
  for (int i = 0; i < n; ++i) {
    if (ifaces[i].dim != 2 || grids[i].dim != 2 || coeffs[i].ncomp != 1)
      throw std::invalid_argument("batched problems are two-dimensional with one component");
    const int c = grids[i].cells;
    if (c < 16 || c > 1024 || (c & (c - 1)) != 0) throw std::invalid_argument("cells must be 2^k in [16, 1024]");
    probs[i] = std::make_unique<DevProblem>();
    build_host_tables(ifaces[i], grids[i], coeffs[i], probs[i]->ht);
  }
  for (int i = 0; i < n; ++i) {
    KFBI_HIP(hipGetDevice(&probs[i]->dev));
    upload_tables(*probs[i]);
    probs[i]->on_device = true;
  }
  // groups by size and by kind of last axis: a member whose last axis is not solved by columns leaves the others'
  // passes as they are
  std::vector<std::pair<int, ColumnRule>> kinds;
  for (auto &p : probs) kinds.emplace_back((int)p->Mfft, p->columns);
  std::sort(kinds.begin(), kinds.end());
  kinds.erase(std::unique(kinds.begin(), kinds.end()), kinds.end());
  group_of.assign(n, 0);
  slot_of.assign(n, 0);
  for (const auto &[s, columns] : kinds) {
    Group g;
    g.Mfft = s;
    g.columns = columns;
    g.N = s - 1;
    g.cs = (int64_t)g.N * s;
    for (int i = 0; i < n; ++i)
      if (probs[i]->Mfft == s && probs[i]->columns == columns) {
        group_of[i] = (int)groups.size();
        slot_of[i] = (int)g.members.size();
        g.members.push_back(i);
      }
    const size_t fs = (size_t)g.members.size() * g.cs;
    g.rhs64 = balloc<double>(fs);
    g.fpad64 = balloc<double>(fs);
    g.work64 = balloc<double>(fs);
    g.rhs32 = balloc<float>(fs);
    g.fpad32 = balloc<float>(fs);
    g.work32 = balloc<float>(fs);
    std::vector<ModeParams> ms;
    for (int i : g.members) {
      const DevProblem &p = *probs[i];
      ModeParams m{};
      m.lam = p.lam;
      for (int a = 0; a < 3; ++a) m.D0[a] = m.D1[a] = p.D[0][a];
      m.kappa = p.kappa;
      m.norm = p.lam_scale;
      m.h2 = p.h * p.h;
      ms.push_back(m);
    }
    // rows of the members that matter to a product: the members' lists at their slots, their bits in slot order
    auto set_of = [&](bool out) {
      std::vector<int32_t> list;
      std::vector<uint64_t> bits;
      for (size_t k = 0; k < g.members.size(); ++k) {
        const DevProblem &p = *probs[g.members[k]];
        const RowSet rs = out ? p.set_out() : p.set_in();
        std::vector<int32_t> l((size_t)rs.n);
        std::vector<uint64_t> w(16);
        if (rs.n) KFBI_HIP(hipMemcpy(l.data(), rs.list, l.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
        KFBI_HIP(hipMemcpy(w.data(), rs.bits, 16 * sizeof(uint64_t), hipMemcpyDeviceToHost));
        for (int32_t r : l) list.push_back((int32_t)(k * (size_t)g.N) + r);
        bits.insert(bits.end(), w.begin(), w.end());
      }
      int32_t *dl = balloc<int32_t>(list.size());
      uint64_t *db = balloc<uint64_t>(bits.size());
      KFBI_HIP(hipMemcpy(dl, list.data(), list.size() * sizeof(int32_t), hipMemcpyHostToDevice));
      KFBI_HIP(hipMemcpy(db, bits.data(), bits.size() * sizeof(uint64_t), hipMemcpyHostToDevice));
      return RowSet{dl, (int64_t)list.size(), db};
    };
    g.rows_in = set_of(false);
    g.rows_out = set_of(true);
    g.msv = balloc<ModeParams>(ms.size());
    KFBI_HIP(hipMemcpy(g.msv, ms.data(), ms.size() * sizeof(ModeParams), hipMemcpyHostToDevice));
    groups.push_back(g);
  }
  // concatenated interface vectors and work lists
  off.assign(n + 1, 0);
  goff.assign(n + 1, 0);
  std::vector<int2> cb, gb, pb;   // blocks of the correction, gather and packing launches
  for (int i = 0; i < n; ++i) {
    const DevProblem &p = *probs[i];
    off[i + 1] = off[i] + p.M;
    goff[i + 1] = goff[i] + p.N * p.N;
    for (int k = 0; k < correct_blocks(p); ++k) cb.push_back(make_int2(i, k));
    for (int k = 0; k < gather_blocks(p); ++k) gb.push_back(make_int2(i, k));
    for (int k = 0; k < (int)((p.N + kPackRows - 1) / kPackRows); ++k) pb.push_back(make_int2(i, k));
  }
  L = off[n];
  longest = 1;
  for (int k = 0; k < n; ++k) longest = std::max(longest, off[k + 1] - off[k]);
  if (L == 0) throw std::invalid_argument("no interface nodes");
  std::vector<int16_t> pidh(L);
  for (int i = 0; i < n; ++i)
    for (int64_t e = off[i]; e < off[i + 1]; ++e) pidh[e] = (int16_t)i;
  pid = balloc<int16_t>(L);
  KFBI_HIP(hipMemcpy(pid, pidh.data(), L * sizeof(int16_t), hipMemcpyHostToDevice));
  off_dev = balloc<int64_t>(n + 1);
  KFBI_HIP(hipMemcpy(off_dev, off.data(), (n + 1) * sizeof(int64_t), hipMemcpyHostToDevice));
  goff_dev = balloc<int64_t>(n + 1);
  KFBI_HIP(hipMemcpy(goff_dev, goff.data(), (n + 1) * sizeof(int64_t), hipMemcpyHostToDevice));
  auto blocks_of = [&](const std::vector<int2> &v, BatchBlocks &bl) {
    int2 *q = balloc<int2>(v.size());
    KFBI_HIP(hipMemcpy(q, v.data(), v.size() * sizeof(int2), hipMemcpyHostToDevice));
    bl.ref = q;
    bl.n = (int)v.size();
  };
  blocks_of(cb, correct_bl);
  blocks_of(gb, gather_bl);
  blocks_of(pb, pack_bl);
  std::vector<BatchItem<double>> i64(n);
  std::vector<BatchItem<float>> i32(n);
  std::vector<PackItem> pk(n);
  auto fill = [&](auto &it, auto *rhs, auto *fpad, auto *work, const DevProblem &p, int i) {
    it.tab = p.itab;
    it.rhs = rhs;
    it.fpad = fpad;
    it.work = work;
    it.M = p.M;
    it.ioff = off[i];
  };
  for (int i = 0; i < n; ++i) {
    const DevProblem &p = *probs[i];
    const Group &g = groups[group_of[i]];
    const int64_t o = (int64_t)slot_of[i] * g.cs;
    fill(i64[i], g.rhs64 + o, g.fpad64 + o, g.work64 + o, p, i);
    fill(i32[i], g.rhs32 + o, g.fpad32 + o, g.work32 + o, p, i);
    pk[i] = PackItem{g.fpad64 + o, g.work64 + o, p.N, (int64_t)g.Mfft};
  }
  items64 = balloc<BatchItem<double>>(n);
  items32 = balloc<BatchItem<float>>(n);
  packs = balloc<PackItem>(n);
  KFBI_HIP(hipMemcpy(items64, i64.data(), n * sizeof(BatchItem<double>), hipMemcpyHostToDevice));
  KFBI_HIP(hipMemcpy(items32, i32.data(), n * sizeof(BatchItem<float>), hipMemcpyHostToDevice));
  KFBI_HIP(hipMemcpy(packs, pk.data(), n * sizeof(PackItem), hipMemcpyHostToDevice));
  // Krylov workspace
  V = balloc<double>((size_t)(kMaxRestart + 1) * L);
  vin = balloc<double>(L);
  w = balloc<double>(L);
  r = balloc<double>(L);
  d = balloc<double>(L);
  t = balloc<double>(L);
  gp = balloc<double>(L);
  x = balloc<double>(L);
  dx = balloc<double>(L);
  hcols = balloc<double>((size_t)3 * (kMaxRestart + 1) * n);
  KFBI_HIP(hipHostMalloc(&hhost, (size_t)3 * (kMaxRestart + 1) * n * sizeof(double), hipHostMallocDefault));
  KFBI_HIP(hipHostMalloc(&seqhost, sizeof(int), hipHostMallocDefault));
  *seqhost = 0;
  seq_next = 0;
  ydev = balloc<double>((size_t)kMaxRestart * n);
  sdev = balloc<double>(n);
  nrm = balloc<double>(n);
  jdev = balloc<int>(1);
  seqdev = balloc<int>(1);
  KFBI_HIP(hipMemset(seqdev, 0, sizeof(int)));
  KFBI_HIP(hipStreamCreateWithFlags(&cap, hipStreamNonBlocking));
}

void Batch::release() {
  drop_graphs();
  for (Group &g : groups) {
    void *ps[] = {g.rhs64, g.fpad64, g.work64, g.rhs32, g.fpad32, g.work32, g.msv,
                  const_cast<int32_t *>(g.rows_in.list),   const_cast<uint64_t *>(g.rows_in.bits),
                  const_cast<int32_t *>(g.rows_out.list),  const_cast<uint64_t *>(g.rows_out.bits)};
    for (void *q : ps)
      if (q) (void)hipFree(q);
  }
  groups.clear();
  void *ps[] = {pid, off_dev, goff_dev, const_cast<int2 *>(correct_bl.ref), const_cast<int2 *>(gather_bl.ref),
                const_cast<int2 *>(pack_bl.ref), items64, items32, packs, V, vin, w, r, d, t, gp, x, dx,
                hcols, ydev, sdev, nrm, jdev, seqdev};
  for (void *q : ps)
    if (q) (void)hipFree(q);
  if (cap) (void)hipStreamDestroy(cap);
  cap = nullptr;
  if (hhost) (void)hipHostFree(hhost);
  if (seqhost) (void)hipHostFree(seqhost);
  seqhost = nullptr;
  hhost = nullptr;
  for (auto &p : probs)
    if (p && p->on_device) free_tables(*p);
  probs.clear();
}

void Batch::drop_graphs() {
  for (auto &kind : graph)
    for (hipGraphExec_t &e : kind) {
      if (e) (void)hipGraphExecDestroy(e);
      e = nullptr;
    }
}

template <typename T>
void Batch::box_all(bool from_fpad, bool stencils, hipStream_t st) {
  int64_t bytes = 0;
  for (const Group &g : groups) bytes += (int64_t)g.members.size() * g.cs * (int64_t)sizeof(T);
  const bool sets = row_sets_pay(bytes);
  auto desc = [&](const Group &g) {
    const PrecTables<T> &tb = const_cast<DevProblem &>(*probs[g.members[0]]).tab<T>();
    const T *src;
    if constexpr (sizeof(T) == 8) src = from_fpad ? g.fpad64 : g.rhs64;
    else src = from_fpad ? g.fpad32 : g.rhs32;
    const bool direct = g.columns.of<T>(), listed = direct && sets;
    return MultiGroupDesc{g.Mfft, (int)g.members.size(), direct, g.cs, src, g.work<T>(), g.msv, tb.tw, tb.sp,
                          !from_fpad && listed ? g.rows_in : RowSet{}, stencils && listed ? g.rows_out : RowSet{}};
  };
  for (bool direct : {true, false}) {
    MultiGroupDesc d[kMaxMultiGroups];
    int k = 0;
    for (const Group &g : groups) {
      if (g.columns.of<T>() != direct) continue;
      if (merged && g.Mfft >= 64) d[k++] = desc(g);   // at most the five sizes 64..1024 (one rule for both types)
      else box_solve_group<T>(desc(g), st);
    }
    if (k > 1) box_solve_multi<T>(d, k, st);
    else if (k == 1) box_solve_group<T>(d[0], st);
  }
}

template <typename T, typename TP>
void Batch::matvec(const TP *in, TP *out, hipStream_t st) {
  launch_batch_correct<T, TP>(items<T>(), correct_bl, in, false, st);
  box_all<T>(false, true, st);
  launch_batch_gather<T, TP>(items<T>(), gather_bl, in, out, st);
}
template void Batch::matvec<double, double>(const double *, double *, hipStream_t);
template void Batch::matvec<float, float>(const float *, float *, hipStream_t);

void Batch::apply_vec(int prec, const double *in, double *out, hipStream_t st) {
  if (prec == 0) matvec<double>(in, out, st);
  else matvec<float>(in, out, st);
}

// per-problem squared norms of v into nrm (device) and hhost[0..np) (host)
void Batch::seg_norms(const double *v, std::vector<double> &out, hipStream_t st) {
  k_seg_dot<<<dim3(np, 1), kB, 0, st>>>(v, 0, nullptr, v, off_dev, np, nrm);
  KFBI_HIP(hipGetLastError());
  KFBI_HIP(hipMemcpyAsync(hhost, nrm, np * sizeof(double), hipMemcpyDeviceToHost, st));
  host_wait(st);
  out.resize(np);
  for (int p = 0; p < np; ++p) out[p] = std::sqrt(std::max(0.0, hhost[p]));
}

void Batch::arnoldi_step(int prec, bool small, int m, hipStream_t st) {
  const int ld = kMaxRestart + 1;
  apply_vec(prec, vin, w, st);
  if (small) {
    switch ((longest + kSmallThreads - 1) / kSmallThreads) {
#define KFBI_SMALL(EE)                                                                                           \
  case EE:                                                                                                       \
    k_seg_orthogonalise<EE><<<np, kSmallThreads, 0, st>>>(V, L, w, off_dev, jdev, ld, np, hcols, vin);           \
    break;
      KFBI_SMALL(1) KFBI_SMALL(2) KFBI_SMALL(3) KFBI_SMALL(4) KFBI_SMALL(5)
#undef KFBI_SMALL
    }
  } else {
    for (int pass = 0; pass < 2; ++pass) {
      double *h = hcols + (size_t)pass * ld * np;
      k_seg_dot<<<dim3(np, m), kB, 0, st>>>(V, L, jdev, w, off_dev, np, h);
      k_seg_combine<<<nb(L), kB, 0, st>>>(w, V, L, jdev, h, pid, np);
    }
    double *hn = hcols + (size_t)2 * ld * np;
    k_seg_dot<<<dim3(np, 1), kB, 0, st>>>(w, 0, nullptr, w, off_dev, np, hn);
    k_seg_next<<<nb(L), kB, 0, st>>>(w, hn, pid, V, L, jdev, vin);
  }
  KFBI_HIP(hipGetLastError());
  k_end_step<<<1, 64, 0, st>>>(hcols, hhost, ld, np, jdev, seqdev, seqhost);
  KFBI_HIP(hipGetLastError());
}

void Batch::host_wait(hipStream_t st) {
  k_count<<<1, 1, 0, st>>>(seqdev, seqhost);
  KFBI_HIP(hipGetLastError());
  seq_next = poll_step_counter(seqhost, seq_next + 1, st);
}

void Batch::run_step(int prec, bool small, int m, hipStream_t st) {
  if (!use_graph) {
    arnoldi_step(prec, small, m, st);
    return;
  }
  hipGraphExec_t &exec = graph[prec][small];
  if (!exec || graph_m[prec][small] != m) {
    if (exec) (void)hipGraphExecDestroy(exec);
    exec = nullptr;
    // captured on the batch's own stream, replayed on the caller's
    hipGraph_t g = nullptr;
    KFBI_HIP(hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal));
    try {
      arnoldi_step(prec, small, m, cap);
    } catch (...) {
      (void)hipStreamEndCapture(cap, &g);
      if (g) (void)hipGraphDestroy(g);
      throw;
    }
    KFBI_HIP(hipStreamEndCapture(cap, &g));
    const hipError_t e = hipGraphInstantiate(&exec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    KFBI_HIP(e);
    graph_m[prec][small] = m;
  }
  KFBI_HIP(hipGraphLaunch(exec, st));
}

// GMRES(m) on A x = b for every problem at once; tol[p] absolute; x updated in place.
void Batch::gmres(int prec, const double *b, double *xv, bool x_zero, const std::vector<double> &tol, int restart,
                  int maxit, std::vector<int> &its, int &matvecs, std::vector<double> &res, hipStream_t st) {
  const int m = std::max(1, std::min(restart, kMaxRestart));
  const int ld = kMaxRestart + 1;
  its.assign(np, 0);
  if (x_zero) {
    KFBI_HIP(hipMemcpyAsync(r, b, L * sizeof(double), hipMemcpyDeviceToDevice, st));
  } else {
    apply_vec(prec, xv, t, st);
    ++matvecs;
    k_axpby<<<nb(L), kB, 0, st>>>(r, 1.0, b, -1.0, t, L);
  }
  std::vector<double> beta;
  seg_norms(r, beta, st);
  std::vector<char> active(np);
  for (int p = 0; p < np; ++p) active[p] = beta[p] > tol[p];
  std::vector<double> H((size_t)np * (m + 1) * m), cs((size_t)np * m), sn((size_t)np * m), g((size_t)np * (m + 1));
  std::vector<int> jend(np);
  std::vector<char> done(np), broke(np);   // broke: the last column gave nothing (breakdown)
  std::vector<double> s(np), yh((size_t)m * np);
  int total = 0;
  while (total < maxit && std::any_of(active.begin(), active.end(), [](char a) { return a; })) {
    for (int p = 0; p < np; ++p) {
      s[p] = active[p] ? 1.0 / beta[p] : 0.0;
      done[p] = !active[p];
      broke[p] = 0;
      jend[p] = 0;
      std::fill(&g[(size_t)p * (m + 1)], &g[(size_t)p * (m + 1)] + m + 1, 0.0);
      g[(size_t)p * (m + 1)] = active[p] ? beta[p] : 0.0;
    }
    KFBI_HIP(hipMemcpyAsync(sdev, s.data(), np * sizeof(double), hipMemcpyHostToDevice, st));
    k_seg_scale<<<nb(L), kB, 0, st>>>(r, sdev, pid, V, vin, jdev, L);
    KFBI_HIP(hipGetLastError());
    for (int j = 0; j < m && total < maxit; ++j) {
      run_step(prec, one_workgroup(longest, j + 1, true), m, st);
      ++matvecs;
      ++total;
      seq_next = poll_step_counter(seqhost, seq_next + 1, st);   // the step ends with the counter
      bool all = true;
      for (int p = 0; p < np; ++p) {
        if (done[p]) continue;
        double *Hp = &H[(size_t)p * (m + 1) * m];
        double *gp_ = &g[(size_t)p * (m + 1)];
        double *c_ = &cs[(size_t)p * m], *s_ = &sn[(size_t)p * m];
        for (int i = 0; i <= j; ++i)
          Hp[(size_t)i * m + j] = hhost[(size_t)i * np + p] + hhost[(size_t)ld * np + (size_t)i * np + p];
        Hp[(size_t)(j + 1) * m + j] = std::sqrt(std::max(0.0, hhost[(size_t)2 * ld * np + p]));
        for (int i = 0; i < j; ++i) {
          const double a = Hp[(size_t)i * m + j], c = Hp[(size_t)(i + 1) * m + j];
          Hp[(size_t)i * m + j] = c_[i] * a + s_[i] * c;
          Hp[(size_t)(i + 1) * m + j] = -s_[i] * a + c_[i] * c;
        }
        const double a = Hp[(size_t)j * m + j], c = Hp[(size_t)(j + 1) * m + j];
        const double den = std::hypot(a, c);
        c_[j] = den > 0 ? a / den : 1.0;
        s_[j] = den > 0 ? c / den : 0.0;
        Hp[(size_t)j * m + j] = den;
        Hp[(size_t)(j + 1) * m + j] = 0.0;
        gp_[j + 1] = -s_[j] * gp_[j];
        gp_[j] = c_[j] * gp_[j];
        jend[p] = j + 1;
        its[p] += 1;
        broke[p] = den == 0.0;
        if (std::fabs(gp_[j + 1]) <= tol[p] || broke[p]) done[p] = 1;
        else all = false;
      }
      if (all) break;
    }
    // least-squares coefficients, x += V y
    int jmax = 0;
    std::fill(yh.begin(), yh.end(), 0.0);
    for (int p = 0; p < np; ++p) {
      if (!active[p]) continue;
      const double *Hp = &H[(size_t)p * (m + 1) * m];
      const double *gp_ = &g[(size_t)p * (m + 1)];
      const int je = jend[p];
      jmax = std::max(jmax, je);
      std::vector<double> y(je);
      for (int i = je - 1; i >= 0; --i) {
        double acc = gp_[i];
        for (int k = i + 1; k < je; ++k) acc -= Hp[(size_t)i * m + k] * y[k];
        y[i] = Hp[(size_t)i * m + i] != 0.0 ? acc / Hp[(size_t)i * m + i] : 0.0;
      }
      for (int i = 0; i < je; ++i) yh[(size_t)i * np + p] = y[i];
    }
    if (jmax > 0) {
      KFBI_HIP(hipMemcpyAsync(ydev, yh.data(), (size_t)jmax * np * sizeof(double), hipMemcpyHostToDevice, st));
      k_seg_update<<<nb(L), kB, 0, st>>>(xv, V, L, ydev, pid, np, jmax);
      KFBI_HIP(hipGetLastError());
    }
    // An FP32 inner solve ends on its Arnoldi-relation residual, as the single solver's does: the refinement takes
    // the FP64 residual itself, and a check by an FP32 product, near its rounding for large coupled or fine
    // problems, restarts by luck (64 problems: 19 or 54 FP32 products, from one problem alone).  After a breakdown
    // the relation's residual is zero for a column that was left out, so those problems are checked.
    if (prec == 1) {
      for (int p = 0; p < np; ++p) {
        if (!active[p] || jend[p] == 0 || broke[p]) continue;
        beta[p] = std::fabs(g[(size_t)p * (m + 1) + jend[p]]);
        active[p] = beta[p] > tol[p];
      }
      if (std::none_of(active.begin(), active.end(), [](char a) { return a; })) break;
    }
    // true residual
    apply_vec(prec, xv, t, st);
    ++matvecs;
    k_axpby<<<nb(L), kB, 0, st>>>(r, 1.0, b, -1.0, t, L);
    seg_norms(r, beta, st);
    for (int p = 0; p < np; ++p) active[p] = active[p] && beta[p] > tol[p];
  }
  res = beta;
}

void Batch::pack(const double *plain, int which, bool to_padded, hipStream_t st) {
  // the caller's array is only read when packing into the padded buffers
  k_pack<<<(unsigned)pack_bl.n, kB, 0, st>>>(const_cast<double *>(plain), goff_dev, packs, pack_bl.ref, which,
                                             to_padded ? 1 : 0);
  KFBI_HIP(hipGetLastError());
}

int Batch::solve(const double *g, const double *f, double *u, double *psi, const kfbi_solve_opts &o,
                 kfbi_solve_info *info, hipStream_t st) {
  // volume part: u_V = S f, g' = g - n.D grad u_V+
  pack(f, 0, true, st);
  box_all<double>(true, true, st);
  launch_batch_gather<double, double>(items64, gather_bl, nullptr, t, st);
  if (g) k_axpby<<<nb(L), kB, 0, st>>>(gp, 1.0, g, -1.0, t, L);
  else k_axpby<<<nb(L), kB, 0, st>>>(gp, -1.0, t, 0.0, nullptr, L);
  KFBI_HIP(hipGetLastError());
  std::vector<double> gn;
  seg_norms(gp, gn, st);
  std::vector<double> tol_abs(np);
  for (int p = 0; p < np; ++p) tol_abs[p] = o.tol * gn[p];
  if (!o.x0) KFBI_HIP(hipMemsetAsync(psi, 0, L * sizeof(double), st));
  std::vector<int> its(np, 0), outer(np, 0), mv64(np, 0), mv32(np, 0);
  std::vector<double> res(np, 0), res0(np, 0);
  int mv = 0;
  if (o.precision == 0) {
    gmres(0, gp, psi, !o.x0, tol_abs, o.restart, o.max_iters, its, mv, res, st);
    for (int p = 0; p < np; ++p) mv64[p] = mv;
    res0 = gn;
  } else {
    bool have_x = o.x0 != 0;
    int total = 0;
    std::vector<int> inner;
    for (int k = 0;; ++k) {
      if (have_x) {
        apply_vec(0, psi, t, st);
        for (int p = 0; p < np; ++p) mv64[p] += 1;
        k_axpby<<<nb(L), kB, 0, st>>>(d, 1.0, gp, -1.0, t, L);
      } else {
        KFBI_HIP(hipMemcpyAsync(d, gp, L * sizeof(double), hipMemcpyDeviceToDevice, st));
      }
      seg_norms(d, res, st);
      if (k == 0) res0 = res;
      bool all = true;
      std::vector<double> keep(np), tin(np);
      for (int p = 0; p < np; ++p) {
        keep[p] = res[p] > tol_abs[p] ? 1.0 : 0.0;
        if (keep[p] != 0.0) all = false;
        tin[p] = std::max(o.inner_tol * res[p], 0.5 * tol_abs[p]);
      }
      if (all || k >= o.max_outer || total >= o.max_iters) break;
      // problems already converged take no part in this refinement step
      KFBI_HIP(hipMemcpyAsync(sdev, keep.data(), np * sizeof(double), hipMemcpyHostToDevice, st));
      k_seg_mask<<<nb(L), kB, 0, st>>>(d, pid, sdev, L);
      KFBI_HIP(hipMemsetAsync(dx, 0, L * sizeof(double), st));
      int mvi = 0;
      gmres(1, d, dx, true, tin, o.restart, o.max_iters - total, inner, mvi, res, st);
      int mx = 0;
      for (int p = 0; p < np; ++p) {
        its[p] += inner[p];
        mx = std::max(mx, inner[p]);
        if (keep[p] != 0.0) {
          mv32[p] += mvi;
          outer[p] += 1;
        }
      }
      total += mx;
      k_axpby<<<nb(L), kB, 0, st>>>(psi, 1.0, psi, 1.0, dx, L);
      have_x = true;
    }
  }
  // u = S(f + C psi)
  launch_batch_correct<double, double>(items64, correct_bl, psi, true, st);
  box_all<double>(true, false, st);
  pack(u, 1, false, st);
  KFBI_HIP(hipStreamSynchronize(st));
  bool ok = true;
  for (int p = 0; p < np; ++p) {
    const bool conv = res[p] <= tol_abs[p];
    ok = ok && conv;
    if (info) {
      kfbi_solve_info &in = info[p];
      in = kfbi_solve_info{};
      in.iters = its[p];
      in.outer = outer[p];
      in.matvecs_fp64 = mv64[p];
      in.matvecs_fp32 = mv32[p];
      in.rel_resid = gn[p] > 0 ? res[p] / gn[p] : 0.0;
      in.gp_norm = gn[p];
      in.start_resid = gn[p] > 0 ? res0[p] / gn[p] : 0.0;
      in.true_resid = -1.0;
    }
  }
  return ok ? KFBI_OK : KFBI_ENOCONV;
}

}  // namespace kfbi
