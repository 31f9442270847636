// The last axis of the box solve as constant-coefficient tridiagonal systems (gfx950).
//
// After the sine transforms of the other axes every column of the last axis (z in 3D, y in 2D)
// carries the system  D_c T u_c + (B u)_c = f_c  with T = tridiag(-1, 2, -1) / h^2 (u = 0 at both
// ends) and a matrix B that is constant along the column: b + kappa (one component), or
// [[b_i + kappa, -kappa], [-kappa, b_e + kappa]] (coupled pair), b_c the other axes' part of the
// mode sum.  Transforming the last axis too and dividing by the mode eigenvalues takes two DSTs
// per column; this takes a few multiply-adds per value instead, in one read and one write:
//
//  * the pair is split into two scalar systems by the rotation that diagonalises
//    D^{-1/2} B D^{-1/2} (constant along the column), each  (h^2 T + s) w = h^2 g;
//  * mu + 1/mu = 2 + s, 0 < mu < 1: on the infinite line the solution is a forward and a backward
//    first-order recursion,  p_j = g_j + mu p_{j-1},  w_j = p_j + mu w_{j+1}  (times h^2 mu);
//    both ends' u = 0 are met by the odd, 2M-periodic extension of g, whose sums give the
//    recursions' starting values in closed form;
//  * a column is cut into chunks of LC rows, one thread each: the chunk's two weighted sums go
//    through LDS, one thread per system and direction turns them into the values entering the
//    chunks, and every thread runs the two recursions over its rows in registers.
//
// What bounds it: memory, one read and one write.  256^3 pair in FP64: dense 531 MB in 84 us (6.3 TB/s; the fused
// transform pass took 142), masked 273 MB in 46 us (5.9 TB/s; 130, and 66 here before a product's passes worked in one
// field).  The masked form issues 685 vector instructions per wavefront in 14% of its cycles, and waits for memory in
// 35%.  The column's constants and the values entering its chunks are worked out once per column, not by every chunk's
// thread (15% slower).  16 rows per thread: the pair's rows take 64 registers, four waves fit a SIMD, and 16 columns by
// 16 chunks are a workgroup of 256 threads over whole 128-byte lines.  FP32, scalar 256^3, masked: 38.5 -> 19.4 us.
//
// The recursions use delta = 1 - mu (from s without cancellation; mu^n likewise through
// 1 - mu^{2n} = delta_n (2 - delta_n)): with mu itself, its rounding alone would cost M eps in the
// lowest modes.  All arithmetic is FP64 in both precisions: the kernel waits on memory, not on it.
#include <cmath>
#include <stdexcept>

#include "device.h"

namespace kfbi {
namespace {

constexpr int col_chunk(int M) { return M <= 64 ? 8 : (M >= 1024 ? 32 : 16); }   // rows per thread

// Columns per workgroup: whole 128-byte lines (16 FP64 / 32 FP32 columns; 64 bytes of FP32 from
// 512 rows on, where 32 columns would be 1024 threads) and about 256 threads.
template <typename T>
constexpr int col_width(int M) {
  const int line = M >= 512 ? 16 : 128 / (int)sizeof(T), ch = M / col_chunk(M);
  const int w = 256 / ch > line ? 256 / ch : line, cap = M > 32 ? M : 32;
  return w < cap ? w : cap;
}

// Row bits [r0, r0 + n) of a plane set, r0 a multiple of n (n = 8, 16 or 32).
template <int NW>
__device__ __forceinline__ uint32_t chunk_bits(const PlaneBits &b, int r0) {
  uint64_t w = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) w = (r0 >> 6) == i ? b.w[i] : w;
  return (uint32_t)(w >> (r0 & 63));
}

// The same from a table of 16 words per problem (null: every row).
__device__ __forceinline__ uint32_t chunk_bits(const uint64_t *__restrict__ bits, int problem, int r0) {
  return bits ? (uint32_t)(bits[(int64_t)problem * 16 + (r0 >> 6)] >> (r0 & 63)) : ~0u;
}

// Rows of one component of a column tile, row i of the thread's chunk at base + i * RS.  Rows that a
// thread does not have (masked planes, the row past the end, columns past the pad column) take an
// offset beyond the buffer's range: such loads return zero and such stores are dropped, so that a
// thread's loads are issued back to back without branches (with branches the FP32 loads waited
// for each other: 38 us at 256^3, scalar).  A component of 2 GiB or more (3D, 1024) branches.
template <typename T, bool BUFFER>
struct RowIO {
  T *p;
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ __forceinline__ RowIO(const T *p_, int64_t bytes) : p(const_cast<T *>(p_)) {
    if constexpr (BUFFER) rsrc = __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00020000);
  }
  static constexpr unsigned kOut = 0x80000000u;
  __device__ __forceinline__ T load(bool ok, int64_t base, int64_t row) const {
    if constexpr (!BUFFER) {
      return ok ? p[base + row] : T(0);
    } else {
      const unsigned vo = ok ? (unsigned)base * (unsigned)sizeof(T) : kOut, so = (unsigned)row * (unsigned)sizeof(T);
      if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rsrc, vo, so, 0));
      else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rsrc, vo, so, 0));
    }
  }
  __device__ __forceinline__ void store(bool ok, int64_t base, int64_t row, T v) const {
    if constexpr (!BUFFER) {
      if (ok) p[base + row] = v;
    } else {
      const unsigned vo = ok ? (unsigned)base * (unsigned)sizeof(T) : kOut, so = (unsigned)row * (unsigned)sizeof(T);
      if constexpr (sizeof(T) == 8) {
        typedef unsigned u2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), rsrc, vo, so, 0);
      } else {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rsrc, vo, so, 0);
      }
    }
  }
};

// One scalar system's constants.
struct Decay {
  double d, mu, inv_mu, inv_rho;   // 1 - mu, mu, 1 / mu, mu / (1 - mu^2)
  __device__ __forceinline__ explicit Decay(double s) {
    const double rho = sqrt(s * (4.0 + s)), t = 2.0 + s + rho, r = recip(t);
    d = (s + rho) * r;
    mu = 2.0 * r;
    inv_mu = 0.5 * t;
    inv_rho = recip(rho);
  }
};

// 1 - mu^n from 1 - mu, n a power of two.
template <int n>
__device__ __forceinline__ double decay_pow(double d) {
#pragma unroll
  for (int i = 1; i < n; i <<= 1) d = d * (2.0 - d);
  return d;
}

// p <- g + (1 - d) p
__device__ __forceinline__ double decay_add(double p, double d, double g) { return fma(-d, p, p + g); }

// What a column's threads share, in LDS: the sums of every chunk (then the values entering it), the
// constants of the column (computed by one thread for all chunks), and the two whole sums.
template <int NC, int CH, int XC>
struct ColumnShared {
  double fs[CH][XC][NC], bs[CH][XC][NC];
  double A[NC * NC][XC];            // into the decoupled variables (the pair's last in FP64: A11 - A10); its transpose leads back
  double d[NC][XC], mu[NC][XC], wk[NC][XC], inv_mu[NC][XC];   // mu: times the pair's weight; wk = 1 / (1 - mu^2)
  double tot[2 * NC][XC];
};

// What one launch reads and writes; ib / ob: the bits of the thread's chunk of rows in the sets (2D: forms 0 and 1):
//   0 every row of every component in and out;
//   1 rows in zin read (the others are zero), rows in zout written;
//   2 every row read, rows in zout written;
//   3 coupled pair, input (g, -g) with g in component 0, rows in zout written;
//   4 coupled pair, only component 0 - component 1 written, into component 0;
//   5 as 4 for the input (g, -g) plus the pair in ain2 on the rows in zin.
template <typename T, int M, int NC, int DIM, int FORM, int XC>
__device__ __forceinline__ void column_solve(const T *__restrict__ ain, T *__restrict__ a, int64_t P, int64_t cs,
                                             const ModeParams &ms, int y, uint32_t ib, uint32_t ob,
                                             const T *__restrict__ ain2, int x0,
                                             ColumnShared<NC, M / col_chunk(M), XC> &sh) {
  constexpr int N = M - 1, LC = col_chunk(M), CH = M / LC;
  const int xo = threadIdx.x % XC, c = threadIdx.x / XC, r0 = c * LC;
  const int x = x0 + xo;
  const bool in_row = M % XC == 0 || x < M;   // x = N is the pad column: zero in, zero out
  const int64_t RS = DIM == 3 ? (int64_t)N * P : P;
  const int64_t base = (int64_t)r0 * RS + x;
  constexpr bool BUF = DIM == 2 || M <= 512;
  // The small eigenvalue's row as A10 (f0 + f1) + (A11 - A10) f1 (see below); FP32 values carry 2^29 times the rounding
  // that this is there for
  constexpr bool SUM = sizeof(T) == 8;
  const int64_t bytes = (int64_t)N * RS * (int64_t)sizeof(T);
  auto wants = [&](int i) { return FORM < 1 || FORM > 3 || ((ob >> i) & 1); };
  auto inside = [&](int i) { return in_row && (i < LC - 1 || c < CH - 1); };
  // all loads of the thread, in flight while the column's constants are computed
  double g[NC][LC];
  T f[FORM == 3 || FORM == 5 ? 1 : NC][LC], f2[FORM == 5 ? 2 : 1][FORM == 5 ? LC : 1];
  {
    const RowIO<T, BUF> i0(ain, bytes), i1(NC == 2 && FORM != 3 && FORM != 5 ? ain + cs : ain, bytes),
        j0(FORM == 5 ? ain2 : ain, bytes), j1(FORM == 5 ? ain2 + cs : ain, bytes);
#pragma unroll
    for (int i = 0; i < LC; ++i) {
      const bool rd = inside(i) && (FORM != 1 || ((ib >> i) & 1));
      f[0][i] = i0.load(rd, base, i * RS);
      if constexpr (NC == 2 && FORM != 3 && FORM != 5) f[1][i] = i1.load(rd, base, i * RS);
      if constexpr (FORM == 5) {
        const bool r2 = inside(i) && ((ib >> i) & 1);
        f2[0][i] = j0.load(r2, base, i * RS);
        f2[1][i] = j1.load(r2, base, i * RS);
      }
    }
  }
  if (c == 0) {
    const double h2 = ms.h2;
    const double lx = ms.lam[x < N ? x : N - 1], ly = DIM == 3 ? ms.lam[y] : 0.0;
    double s[NC], wt[2] = {1.0, 1.0};
    if constexpr (NC == 2) {
      const double b0 = ms.D0[0] * lx + ms.D0[1] * ly, b1 = ms.D1[0] * lx + ms.D1[1] * ly, kap = ms.kappa;
      const double dz0 = ms.D0[DIM - 1], dz1 = ms.D1[DIM - 1], i0 = recip(dz0), i1 = recip(dz1);
      const double p = (b0 + kap) * i0, q = (b1 + kap) * i1;
      // X = dz1 b0 - dz0 b1, exactly 0 where the conductivities are proportional
      auto cross = [&](int ax) {
        const double t = dz0 * ms.D1[ax];
        return fma(dz1, ms.D0[ax], -t) + fma(-dz0, ms.D1[ax], t);
      };
      const double X = lx * cross(0) + (DIM == 3 ? ly * cross(1) : 0.0);
      // (p - q) / 2 and half the eigenvalues' difference, of [[p, -c], [-c, q]] with c^2 = kappa^2 / (dz0 dz1)
      const double hd = 0.5 * (X + kap * (dz1 - dz0)) * (i0 * i1), rr = sqrt(hd * hd + kap * i0 * (kap * i1));
      const double l1 = 0.5 * (p + q) + rr;
      // the eigenvalues' product without cancellation: det = b0 b1 + kappa (b0 + b1)
      const double l2 = (b0 * b1 + kap * (b0 + b1)) * i0 * i1 * recip(l1);
      // Rows (1, r) or (r, 1) into the decoupled variables, the larger entry 1, and weights w on the way back (squares
      // of the normalised rows' larger entries: no square roots, whose rounding would be one and the same everywhere).
      // rho: the smaller entry of the small eigenvalue's row.  That row is applied as A10 (f0 + f1) + (A11 - A10) f1:
      // sources near (g, -g), a step's among them, cancel in it, and 1 / l2 magnifies what is left (by l1 / l2, about
      // kappa over the mode sums), so the difference is taken without cancellation from
      //   rho = 1 - 2 X / (S + X + R) where hd >= 0, 1 + 2 X / (S - X + R) where hd < 0,
      // S = kappa (dz0 + dz1), R = 2 dz0 dz1 rr (S +- X > 0 there).
      const bool first = hd >= 0.0;   // the large eigenvalue's row has its larger entry at component 0
      double big2 = 1.0, rho = 0.0, rel = first ? 1.0 : -1.0;
      if (rr > 0.0) {
        const double ir = recip(rr);
        big2 = 0.5 + 0.5 * (fabs(hd) * ir);
        rel = 2.0 * X * recip(kap * (dz0 + dz1) + (first ? X : -X) + 2.0 * dz0 * dz1 * rr);
        if (fabs(rel) < 0.5) {
          rho = first ? 1.0 - rel : 1.0 + rel;
        } else {
          rho = 0.5 * kap * (first ? i0 : i1) * (ir * recip(big2));
          rel = first ? 1.0 - rho : rho - 1.0;
        }
      }
      sh.A[0][xo] = first ? 1.0 : -rho * dz1 * i0;
      sh.A[1][xo] = first ? -rho * dz0 * i1 : 1.0;
      sh.A[2][xo] = first ? rho : 1.0;
      sh.A[3][xo] = SUM ? rel : sh.A[2][xo] + rel;
      wt[0] = big2 * (first ? i0 : i1);
      wt[1] = big2 * (first ? i1 : i0);
      s[0] = h2 * l1;
      s[1] = h2 * l2;
    } else {
      const double iz = recip(ms.D0[DIM - 1]);
      sh.A[0][xo] = iz;
      s[0] = h2 * ((DIM == 3 ? ms.D0[0] * lx + ms.D0[1] * ly : ms.D0[0] * lx) + ms.kappa) * iz;
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const Decay dk(s[k]);
      sh.d[k][xo] = dk.d;
      sh.mu[k][xo] = wt[k] * dk.mu;
      sh.wk[k][xo] = dk.inv_mu * dk.inv_rho;
      sh.inv_mu[k][xo] = dk.inv_mu;
    }
  }
  __syncthreads();
  double d[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) d[k] = sh.d[k][xo];
  if constexpr (NC == 2) {
    const double A00 = sh.A[0][xo], A01 = sh.A[1][xo], A10 = sh.A[2][xo], A11 = sh.A[3][xo];
#pragma unroll
    for (int i = 0; i < LC; ++i) {
      double f0 = (double)f[0][i], f1, both = f0;
      if constexpr (FORM == 3 || FORM == 5) f1 = -f0;
      else f1 = (double)f[1][i];
      if constexpr (FORM == 5) {
        both = (double)f2[0][i] + (double)f2[1][i];
        f0 += (double)f2[0][i];
        f1 += (double)f2[1][i];
      } else if constexpr (SUM) {
        both = f0 + f1;
      }
      g[0][i] = A00 * f0 + A01 * f1;
      g[1][i] = A10 * both + A11 * f1;
    }
  } else {
    const double A00 = sh.A[0][xo];
#pragma unroll
    for (int i = 0; i < LC; ++i) g[0][i] = A00 * (double)f[0][i];
  }
  // the chunk's sums, weighted towards its last row (forward) and its first row (backward)
  {
    double fs[NC], bs[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) fs[k] = bs[k] = 0.0;
#pragma unroll
    for (int i = 0; i < LC; ++i)
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        fs[k] = decay_add(fs[k], d[k], g[k][i]);
        bs[k] = decay_add(bs[k], d[k], g[k][LC - 1 - i]);
      }
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      sh.fs[c][xo][k] = fs[k];
      sh.bs[c][xo][k] = bs[k];
    }
  }
  __syncthreads();
  // the values entering the chunks, by 2 NC threads of the column (one per system and direction):
  // the whole sum, the image term from both directions' sums, then the recursion over the chunks
  for (int t = c; t < 2 * NC; t += CH) {
    const int k = t >> 1;
    const double dL = decay_pow<LC>(sh.d[k][xo]);
    double v = 0.0;
#pragma unroll
    for (int j = 0; j < CH; ++j)
      v = decay_add(v, dL, (t & 1) ? sh.bs[CH - 1 - j][xo][k] : sh.fs[j][xo][k]);
    if (t & 1) v = decay_add(v, sh.d[k][xo], 0.0);
    sh.tot[t][xo] = v;   // sums of mu^{M-j} g_j (forward) and mu^j g_j (backward)
  }
  __syncthreads();
  for (int t = c; t < 2 * NC; t += CH) {
    const int k = t >> 1;
    const double dL = decay_pow<LC>(sh.d[k][xo]), dM = decay_pow<CH>(dL);
    const double own = sh.tot[t][xo], other = sh.tot[t ^ 1][xo];
    double v = fma(-dM, own, own - other) * recip(dM * (2.0 - dM));   // over 1 - mu^{2M}
    if (t & 1) v *= sh.inv_mu[k][xo];
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      double &e = (t & 1) ? sh.bs[CH - 1 - j][xo][k] : sh.fs[j][xo][k];
      const double sum = e;
      e = v;
      v = decay_add(v, dL, sum);
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    double p = sh.fs[c][xo][k];
#pragma unroll
    for (int i = 0; i < LC; ++i) {
      p = decay_add(p, d[k], g[k][i]);
      g[k][i] = p;
    }
    double w = (fma(-d[k], p, p) + sh.bs[c][xo][k]) * sh.wk[k][xo];
#pragma unroll
    for (int i = LC - 1; i >= 0; --i) {
      w = decay_add(w, d[k], g[k][i]);
      g[k][i] = w;
    }
  }
  // back to the components; the pad column's zeros stay zeros
  const RowIO<T, BUF> o0(a, bytes), o1(NC == 2 && FORM < 4 ? a + cs : a, bytes);
  const double scale = x < N ? ms.h2 * ms.norm * (0.5 * M) : 0.0;
  const double s0 = scale * sh.mu[0][xo];
  if constexpr (NC == 2) {
    const double s1 = scale * sh.mu[1][xo];
    const double B00 = s0 * sh.A[0][xo], B01 = s0 * sh.A[1][xo], B10 = s1 * sh.A[2][xo],
                 B11 = (SUM ? B10 : 0.0) + s1 * sh.A[3][xo];
#pragma unroll
    for (int i = 0; i < LC; ++i) {
      const double u0 = B00 * g[0][i] + B10 * g[1][i], u1 = B01 * g[0][i] + B11 * g[1][i];
      const bool wr = inside(i) && wants(i);
      if constexpr (FORM >= 4) {
        o0.store(wr, base, i * RS, (T)(u0 - u1));
      } else {
        o0.store(wr, base, i * RS, (T)u0);
        o1.store(wr, base, i * RS, (T)u1);
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < LC; ++i) o0.store(inside(i) && wants(i), base, i * RS, (T)(s0 * g[0][i]));
  }
}

template <int M, int XC>
constexpr int col_threads() { return M / col_chunk(M) * XC; }

// Waves per SIMD that the register allocation has to leave: four for 3D FP32 pairs (masked 256^3 pair 36 us; with 130
// registers, so three waves, 49).
template <typename T, int M, int NC, int DIM>
constexpr int col_waves() { return sizeof(T) == 4 && NC == 2 && DIM == 3 && M <= 512 ? 4 : 1; }

template <typename T, int M, int NC, int DIM, int FORM>
__global__ __launch_bounds__((col_threads<M, col_width<T>(M)>()), (col_waves<T, M, NC, DIM>())) void k_column(
    const T *ain, T *a, int64_t P, int64_t cs, ModeParams ms0, const ModeParams *__restrict__ msv, int64_t pstride,
    PlaneBits zin, PlaneBits zout, const uint64_t *__restrict__ bin, const uint64_t *__restrict__ bout,
    const T *__restrict__ ain2) {
  constexpr int XC = col_width<T>(M);
  __shared__ ColumnShared<NC, M / col_chunk(M), XC> sh;
  const int by = blockIdx.y;
  const int64_t off = DIM == 3 ? (int64_t)by * P : (int64_t)by * pstride;
  const ModeParams ms = DIM == 2 && msv ? msv[by] : ms0;
  constexpr int NW = (M + 62) / 64;
  const int r0 = threadIdx.x / XC * col_chunk(M);
  uint32_t ib = ~0u, ob = ~0u;
  if constexpr (DIM == 3) {
    if constexpr (FORM == 1 || FORM == 5) ib = chunk_bits<NW>(zin, r0);
    if constexpr (FORM >= 1 && FORM <= 3) ob = chunk_bits<NW>(zout, r0);
  } else if constexpr (FORM == 1) {
    ib = chunk_bits(bin, by, r0);
    ob = chunk_bits(bout, by, r0);
  }
  column_solve<T, M, NC, DIM, FORM, XC>(ain + off, a + off, P, cs, ms, by, ib, ob, ain2 ? ain2 + off : nullptr,
                                        blockIdx.x * XC, sh);
}

template <typename T, int M, int NC, int DIM, int FORM>
void launch_form(const LastAxis<T> &l, hipStream_t st) {
  constexpr int XC = col_width<T>(M);
  const dim3 g((M + XC - 1) / XC, DIM == 3 ? M - 1 : l.nprob);
  k_column<T, M, NC, DIM, FORM><<<g, col_threads<M, XC>(), 0, st>>>(
      l.in, l.out, M, l.cs, l.ms, l.msv, l.pstride, l.zin ? *l.zin : PlaneBits{}, l.zout ? *l.zout : PlaneBits{},
      l.bin, l.bout, l.in2);
  KFBI_HIP(hipGetLastError());
}

template <typename T, int M>
void launch_column(const LastAxis<T> &l, hipStream_t st) {
  if (l.dim == 2) {
    const bool masked = l.bin || l.bout;
    if (l.ncomp == 2) {
      if (masked) launch_form<T, M, 2, 2, 1>(l, st);
      else launch_form<T, M, 2, 2, 0>(l, st);
    } else {
      if (masked) launch_form<T, M, 1, 2, 1>(l, st);
      else launch_form<T, M, 1, 2, 0>(l, st);
    }
    return;
  }
  if (l.form >= 3) {
    // the forms of a bidomain step (FP64, coupled)
    if constexpr (sizeof(T) == 8) {
      if (l.form == 3) launch_form<T, M, 2, 3, 3>(l, st);
      else if (l.form == 4) launch_form<T, M, 2, 3, 4>(l, st);
      else launch_form<T, M, 2, 3, 5>(l, st);
    }
  } else if (l.ncomp == 2) {
    if (l.zin) launch_form<T, M, 2, 3, 1>(l, st);
    else if (l.zout) launch_form<T, M, 2, 3, 2>(l, st);
    else launch_form<T, M, 2, 3, 0>(l, st);
  } else {
    if (l.zin) launch_form<T, M, 1, 3, 1>(l, st);
    else if (l.zout) launch_form<T, M, 1, 3, 2>(l, st);
    else launch_form<T, M, 1, 3, 0>(l, st);
  }
}

// ---------------------------------------------------------------- merged 2D groups

template <typename T>
struct MultiColumn {
  struct G {
    T *a;
    int64_t cs;
    const ModeParams *msv;
    const uint64_t *bin, *bout;
    int M, begin, gx;
  } g[kMaxMultiGroups];
  int ng;
};

// One workgroup size for every grid size of a merged launch.
constexpr int kMultiThreads = 512;
constexpr int multi_width(int M) { return kMultiThreads * col_chunk(M) / M; }
constexpr int kMultiShared = 2 * kMultiThreads + 7 * multi_width(64);   // doubles, the largest of any size
static_assert(sizeof(ColumnShared<1, 8, multi_width(64)>) <= kMultiShared * sizeof(double));
static_assert(multi_width(64) >= multi_width(128) && multi_width(64) >= multi_width(1024));

template <typename T>
__global__ __launch_bounds__(kMultiThreads) void k_column_multi(MultiColumn<T> mp) {
  __shared__ double lds[kMultiShared];
  int k = 0;
#pragma unroll
  for (int j = 1; j < kMaxMultiGroups; ++j)
    if (j < mp.ng && (int)blockIdx.x >= mp.g[j].begin) k = j;
  const auto &g = mp.g[k];
  const int b = (int)blockIdx.x - g.begin, pr = b / g.gx, bx = b - pr * g.gx;
  T *a = g.a + pr * g.cs;
  const ModeParams ms = g.msv[pr];
  auto bits = [&](const uint64_t *t, int M, int XC) { return chunk_bits(t, pr, (int)threadIdx.x / XC * col_chunk(M)); };
  switch (g.M) {
#define KFBI_COLUMN_CASE(MM)                                                                                       \
    case MM:                                                                                                       \
      column_solve<T, MM, 1, 2, 1, multi_width(MM)>(                                                               \
          a, a, MM, 0, ms, 0, bits(g.bin, MM, multi_width(MM)), bits(g.bout, MM, multi_width(MM)), nullptr,        \
          bx * multi_width(MM),                                                                                    \
          *reinterpret_cast<ColumnShared<1, MM / col_chunk(MM), multi_width(MM)> *>(lds));                         \
      break;
    KFBI_COLUMN_CASE(64) KFBI_COLUMN_CASE(128) KFBI_COLUMN_CASE(256) KFBI_COLUMN_CASE(512)
    KFBI_COLUMN_CASE(1024)
#undef KFBI_COLUMN_CASE
  }
}

}  // namespace

// Smallest s M^2 over the columns (the lowest modes of the other axes): how many times e the
// slowest solution decays across the box, squared.
ColumnRule column_direct(int dim, int ncomp, int M, double h, const double D[2][3], double kappa) {
  const double sn = std::sin(0.5 * M_PI / M), lam = 4.0 / (h * h) * sn * sn;
  double b[2], dz[2];
  for (int c = 0; c < 2; ++c) {
    const double *Dc = D[c < ncomp ? c : 0];
    b[c] = lam * (dim == 3 ? Dc[0] + Dc[1] : Dc[0]);
    dz[c] = Dc[dim - 1];
  }
  double l = (b[0] + kappa) / dz[0];
  if (ncomp == 2) {
    const double p = l, q = (b[1] + kappa) / dz[1], hd = 0.5 * (p - q);
    const double big = 0.5 * (p + q) + std::sqrt(hd * hd + kappa / dz[0] * (kappa / dz[1]));
    l = (b[0] * b[1] + kappa * (b[0] + b[1])) / (dz[0] * dz[1]) / big;
  }
  const double s = l * h * h;
  const bool f32 = s * M * M >= 2.0 && s < 1e12;
  return {f32 && (M > 32 || s * M * M >= 6.0), f32};
}

template <typename T>
void last_axis_direct(const LastAxis<T> &l, hipStream_t st) {
  if (l.form >= 3 && (l.dim != 3 || l.ncomp != 2 || sizeof(T) != 8))
    throw std::invalid_argument("the step's last-axis forms take the coupled 3D pair in FP64");
  if ((l.form == 3 && !l.zout) || (l.form == 5 && (!l.zin || !l.in2)) || (l.form < 3 && l.zin && !l.zout))
    throw std::invalid_argument("last axis: missing plane mask or input");
  switch (l.M) {
    case 16: launch_column<T, 16>(l, st); break;
    case 32: launch_column<T, 32>(l, st); break;
    case 64: launch_column<T, 64>(l, st); break;
    case 128: launch_column<T, 128>(l, st); break;
    case 256: launch_column<T, 256>(l, st); break;
    case 512: launch_column<T, 512>(l, st); break;
    case 1024: launch_column<T, 1024>(l, st); break;
    default: throw std::invalid_argument("unsupported grid size");
  }
}
template void last_axis_direct<double>(const LastAxis<double> &, hipStream_t);
template void last_axis_direct<float>(const LastAxis<float> &, hipStream_t);

template <typename T>
void last_axis_direct_multi(const MultiGroupDesc *gd, int ng, hipStream_t st) {
  if (ng < 1 || ng > kMaxMultiGroups) throw std::invalid_argument("merged passes take 1 to 8 groups");
  MultiColumn<T> mp{};
  int blocks = 0;
  for (int j = 0; j < ng; ++j) {
    const int M = gd[j].Mfft;
    if (M < 64 || M > 1024 || (M & (M - 1)) || gd[j].G < 1 || gd[j].cs != (int64_t)(M - 1) * M || !gd[j].msv)
      throw std::invalid_argument("merged passes: sizes 64..1024, padded groups");
    const int gx = (M + multi_width(M) - 1) / multi_width(M);
    mp.g[j] = {static_cast<T *>(gd[j].dst), gd[j].cs, gd[j].msv, gd[j].in.bits, gd[j].out.bits, M, blocks, gx};
    blocks += gx * gd[j].G;
  }
  mp.ng = ng;
  k_column_multi<T><<<blocks, kMultiThreads, 0, st>>>(mp);
  KFBI_HIP(hipGetLastError());
}
template void last_axis_direct_multi<double>(const MultiGroupDesc *, int, hipStream_t);
template void last_axis_direct_multi<float>(const MultiGroupDesc *, int, hipStream_t);

}  // namespace kfbi
