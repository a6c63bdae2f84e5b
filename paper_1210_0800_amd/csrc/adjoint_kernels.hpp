// Adjoint of the least-squares solution x = argmin ||b - A x|| for a loss
// L(x) with gradient g = dL/dRe(x) + i dL/dIm(x):
//   w  = R^{-H} g      (forward substitution)
//   z  = R^{-1} w      (back substitution of Section 6, Figure 3)
//   gb = Q w           (= A z, the gradient with respect to b)
//   r  = b - A x
//   gA = r z^H - gb x^H
// with z = (A^H A)^{-1} g for A = Q R of full column rank.
#pragma once
#include "mgs_kernels.hpp"

namespace mgsq {

// gb = Q w and r = b - A x, split over column chunks of ADJ_CH columns so
// that the grid covers the device (rows x chunks x 2 products): each thread
// sums one row of one chunk in the fused accumulator (the chunk holding
// column 0 of r starts from b); adj_finish_kernel merges the chunk partials
// of a row in chunk order, so results are reproducible.
constexpr int ADJ_CH = 8;
constexpr int ADJ_T = 64;
template <class P>
__global__ __launch_bounds__(ADJ_T) void adj_partial_kernel(int m, int n, const double *Q, int ldq, size_t planeQ,
                                                             const double *A, int lda, size_t planeA,
                                                             const double *b, const double *x, const double *w,
                                                             typename Partial<P>::T *partial) {
  using Acc = typename P::Acc;
  const int i = blockIdx.x * ADJ_T + threadIdx.x;
  const int cb = blockIdx.y, which = blockIdx.z;  // 0: Q w, 1: b - A x
  if (i >= m) return;
  const int nchunk = (n + ADJ_CH - 1) / ADJ_CH;
  const int j0 = cb * ADJ_CH, j1 = j0 + ADJ_CH < n ? j0 + ADJ_CH : n;
  Acc acc;
  if (which == 0) {
    P::acc_zero(acc);
#pragma unroll 4
    for (int k = j0; k < j1; ++k)
      P::acc_cmul(acc, P::load(Q + (size_t)k * ldq + i, planeQ), P::load(w + k, (size_t)n));
  } else {
    if (cb == 0)
      P::acc_set(acc, P::load(b + i, (size_t)m));
    else
      P::acc_zero(acc);
#pragma unroll 4
    for (int j = j0; j < j1; ++j)
      P::acc_cmul(acc, P::load(A + (size_t)j * lda + i, planeA), P::cneg(P::load(x + j, (size_t)n)));
  }
  partial[((size_t)which * nchunk + cb) * m + i] = Partial<P>::pack(acc);
}

template <class P>
__global__ __launch_bounds__(WG) void adj_finish_kernel(int m, int n, const typename Partial<P>::T *partial,
                                                         double *gb, double *r) {
  using Acc = typename P::Acc;
  const int i = blockIdx.x * WG + threadIdx.x;
  const int which = blockIdx.y;
  if (i >= m) return;
  const int nchunk = (n + ADJ_CH - 1) / ADJ_CH;
  const typename Partial<P>::T *p = partial + (size_t)which * nchunk * m + i;
  Acc acc = Partial<P>::unpack(p[0]);
  for (int c = 1; c < nchunk; ++c) P::acc_merge(acc, Partial<P>::unpack(p[(size_t)c * m]));
  P::store((which == 0 ? gb : r) + i, (size_t)m, P::acc_value(acc));
}

// gA(i, j) = r_i conj(z_j) - gb_i conj(x_j): two fused updates from zero.
template <class P>
__global__ __launch_bounds__(WG) void adj_rank2_kernel(int m, int n, const double *r, const double *z,
                                                        const double *gb, const double *x, double *gA, int ldga,
                                                        size_t planeG) {
  using C = typename P::C;
  const int i = blockIdx.x * WG + threadIdx.x;
  const int j = blockIdx.y;
  if (i >= m || j >= n) return;
  C a = P::czero();
  P::upd(a, P::cneg(P::load(r + i, (size_t)m)), P::conj(P::load(z + j, (size_t)n)));
  P::upd(a, P::load(gb + i, (size_t)m), P::conj(P::load(x + j, (size_t)n)));
  P::store(gA + (size_t)j * ldga + i, planeG, a);
}

}  // namespace mgsq
