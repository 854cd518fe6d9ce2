// Reductions shared by the solver kernels and the applies that take a step of the solver:
// per-block partial sums, re-reduced in a fixed order by every block of a later kernel.
#pragma once

#include <hip/hip_runtime.h>

#include "q1_internal.hpp"

namespace q1 {

constexpr int kRT = 256;      // threads per reduction block
constexpr int kMaxRB = 1024;  // partial sums per reduction (4 blocks per compute unit)

// Device status record, read by the host every few iterations.
struct Status {
  int done, status, iter, pad;
  double rr, bb, rho, aux;
  double rho2[2];  // rho_k at k & 1, as the kernels of the PCG pass it on
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Sum of N values over the block, returned to every thread (fixed order).
template <int N>
__device__ __forceinline__ void block_sum(double (&v)[N]) {
  __shared__ double sh[N][kRT / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = wave_sum(v[i]);
  __syncthreads();
  if (lane == 0)
#pragma unroll
    for (int i = 0; i < N; ++i) sh[i][w] = v[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    double s = sh[i][0];
#pragma unroll
    for (int k = 1; k < kRT / 64; ++k) s += sh[i][k];
    v[i] = s;
  }
}

// Re-reduce the partials written by an earlier kernel, R rows of cnt[r] >= 1
// partials each: thread t adds partials t, t + 256, ... of each row in order,
// then the fixed block sum (the same value in every block).  The loads of four
// rounds are issued together, at clamped indices, before any of them is added.
template <int R>
__device__ __forceinline__ void sum_partials_nc(const double *const (&rows)[R],
                                                const int (&cnt)[R], double (&out)[R]) {
  constexpr int U = 4;
  int m = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    out[r] = 0.0;
    m = cnt[r] > m ? cnt[r] : m;
  }
  for (int j0 = int(threadIdx.x); j0 < m; j0 += U * kRT) {
    double a[U][R];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < R; ++r) a[u][r] = rows[r][min(j0 + u * kRT, cnt[r] - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (j0 + u * kRT < cnt[r]) out[r] += a[u][r];
  }
  block_sum<R>(out);
}

// the same with one count for every row
template <int R>
__device__ __forceinline__ void sum_partials_n(const double *const (&rows)[R], int nb,
                                               double (&out)[R]) {
  int cnt[R];
#pragma unroll
  for (int r = 0; r < R; ++r) cnt[r] = nb;
  sum_partials_nc<R>(rows, cnt, out);
}

__device__ __forceinline__ double sum_partials(const double *__restrict__ part, int nb) {
  double out[1];
  sum_partials_n<1>({part}, nb, out);
  return out[0];
}

// The test after iteration `it` of the PCG and beta = rho_it / rho_{it-1}, the same in every
// block (of kRT threads); block 0 records the status and rho_it.  True: the solve stops.
// part_num, part_rr: nb partials of rho_it and of r.r.  done: this thread's reading of st->done,
// which block 0 of the same launch may raise between the readings of two waves.  So every
// thread takes part in the sums whatever it read: one that read the raised flag stops by it,
// one that did not by the test that raised it, and the waves of a block never part.
__device__ __forceinline__ bool direction_test(int done, const double *part_num,
                                               const double *part_rr, int nb, double tol2, int it,
                                               int maxit, Status *st, double &beta) {
  const double den = st->rho2[(it + 1) & 1], bb = st->bb;  // neither is written in this kernel
  double t[2];
  sum_partials_n<2>({part_num, part_rr}, nb, t);
  const double num = t[0], rr = t[1];
  const bool conv = rr <= tol2 * bb, bad = !isfinite(rr);
  const bool stop = done || conv || bad || it >= maxit;
  beta = num / den;
  if (!done && blockIdx.x == 0 && threadIdx.x == 0) {
    st->iter = it;
    st->rr = rr;
    st->rho = num;
    st->rho2[it & 1] = num;
    if (stop) {
      st->done = 1;
      st->status = conv ? Q1_OK : (bad ? Q1_EBREAKDOWN : Q1_ENOCONV);
    }
  }
  return stop;
}

// p = z + beta p, rounded the same way wherever it is compiled (z = w r is rounded first)
template <typename TP, typename T>
__device__ __forceinline__ TP direction_value(T z, TP p, double beta) {
  return TP(__builtin_fma(beta, double(p), double(z)));
}

}  // namespace q1
