// Parts of an Arnoldi step that one problem's solver and the batch's share.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace kfbi {
namespace {

constexpr int kSmallThreads = 1024, kSmallMax = 5 * kSmallThreads;
constexpr int kSmallColumn = 66;   // room of a Hessenberg column

// Whether one workgroup orthogonalises a step against K basis vectors of n entries: it reads the basis four times by
// itself, so from K n = 24,576 on the many-block kernels are faster.  One iteration of a 128^2 problem, one workgroup /
// many blocks (us): 1,025 entries, 19 vectors 39.5 / 41.1, 30 48.2 / 42.2; 2,049, 7 36.2 / 38.9, 15 45.2 / 40.3; 4,097,
// 3 35.9 / 38.6, 11 52.8 / 39.1, 56 149 / 54; 513 entries never lose.  batch: one workgroup for each problem, against
// kernels whose work grows with the problems too: 36,864 entries of the longest (1 problem of 5,120 entries, 7 vectors
// 48.8 / 47.1; 16 of 2,049, 19 56.9 / 64.3, 30 72.9 / 64.9; 64 of 2,049, 15 68.6 / 68.3, 46 160 / 114).
constexpr bool one_workgroup(int64_t n, int K, bool batch) {
  return n <= kSmallMax && (n <= 512 || K * n <= (batch ? 36 : 24) * 1024);
}

// Both classical Gram-Schmidt passes of w_in against V_0..V_{K-1} (stride ldv), the norm and V_K = w / ||w|| (also
// into vnext) for n <= 1024 E entries, by one workgroup; the passes' coefficients in hcol.  Returns ||w||^2.
// Bound by latency, then by what one workgroup reads (the basis four times).
template <int E>
__device__ __forceinline__ double orthogonalise_block(double *V, int64_t ldv, const double *w_in, int64_t n, int K,
                                                      double *vnext, double (&hcol)[2][kSmallColumn]) {
  constexpr int NT = kSmallThreads, NW = NT / 64, HS = kSmallColumn;
  __shared__ double ws[E * NT];
  __shared__ double hp[HS + NW];   // partial dots: P parts of each of the K vectors
  __shared__ double red[NW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double w[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = tid + NT * e;
    w[e] = i < n ? w_in[i] : 0.0;
    ws[i] = w[e];
  }
  const int P = K < NW ? NW / K : 1;   // wavefronts sharing one vector
  for (int pass = 0; pass < 2; ++pass) {
    __syncthreads();
    for (int t = wave; t < K * P; t += NW) {
      const int k = t / P, part = t - k * P;
      const double *v = V + (int64_t)k * ldv;
      double acc = 0;
#pragma unroll 16
      for (int i = lane + 64 * part; i < n; i += 64 * P) acc += v[i] * ws[i];
      for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
      if (lane == 0) hp[t] = acc;
    }
    __syncthreads();
    if (tid < K) {
      double h = hp[tid * P];
      for (int part = 1; part < P; ++part) h += hp[tid * P + part];
      hcol[pass][tid] = h;
    }
    __syncthreads();
    double acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0;
#pragma unroll 4
    for (int k = 0; k < K; ++k) {
      const double h = hcol[pass][k];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int i = tid + NT * e;
        acc[e] += i < n ? h * V[(int64_t)k * ldv + i] : 0.0;
      }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      w[e] -= acc[e];
      if (pass == 0) ws[tid + NT * e] = w[e];
    }
  }
  double sq = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) sq += w[e] * w[e];
  for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off, 64);
  if (lane == 0) red[wave] = sq;
  __syncthreads();
  double nrm2 = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) nrm2 += red[k];
  const double sc = nrm2 > 0 ? 1.0 / sqrt(nrm2) : 0.0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int i = tid + NT * e;
    if (i < n) {
      V[(int64_t)K * ldv + i] = w[e] * sc;
      if (vnext) vnext[i] = w[e] * sc;
    }
  }
  return nrm2;
}

// End of an Arnoldi step whose coefficients are in device memory ([pass][ld][np], then np squared norms): those of
// the j + 1 vectors into pinned host memory, j <- j + 1, the step counter.  One wavefront, since a system fence by
// many writes the L2 back many times.  Its time grows with problems and vectors; against a copy of the whole array and a
// counter kernel an iteration of 1,024 problems takes 72 us, not 156 (6 vectors), 132, not 196 (61), of 2,048 225, not 418
// (61).
__global__ __launch_bounds__(64) void k_end_step(const double *__restrict__ h, double *__restrict__ host, int ld,
                                                 int np, int *j, int *seq, int *seq_host) {
  const int K = *j + 1, lane = threadIdx.x;
  auto copy = [&](int64_t from, int64_t n) {
#pragma unroll 8
    for (int64_t i = lane; i < n; i += 64) host[from + i] = h[from + i];
  };
  copy(0, (int64_t)K * np);
  copy((int64_t)ld * np, (int64_t)K * np);
  copy((int64_t)2 * ld * np, np);
  __threadfence_system();
  if (lane == 0) {
    *j = K;
    const int s = *seq + 1;
    *seq = s;
    __hip_atomic_store(seq_host, s, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

}  // namespace
}  // namespace kfbi
