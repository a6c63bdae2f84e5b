// Precision form: FP64 blocked MGS factorisation with the trailing Gram and
// update products on FP64 MFMA, then iterative refinement with the residual
// and the solution accumulated in dd / qd.
//
// Factorisation of [A b] in FP64, panels of NB = 64 columns:
//   factor panel p by MGS (Figure 1 restricted to the panel, the step
//   kernel with plain complex doubles), then for the columns right of it,
//   W = Q_p^H A_t (written into R) and A_t -= Q_p W.  b rides along as the
//   last column, so its panel projections y_p = W(:, n) are those of the
//   factorisation (the augmented semantics of Equation (1)).
// Correction solve of A d = r: the same panel projections replayed on r
// (w_p = Q_p^H r, r -= Q_p w_p), then back substitution with R.
// Refinement: r = b - A x in dd / qd, d = FP64 solve of fl64(r),
// x += d in dd / qd, until ||d|| <= tol ||x||, stagnation, or max_iter.
#pragma once
#include "mgs_kernels.hpp"
#include "resident_kernels.hpp"

namespace mgsq {

typedef double v4d __attribute__((ext_vector_type(4)));

// v_mfma_f64_16x16x4f64 operand layout on gfx950 (checked on the device):
// A[i][k] in lane i + 16k, B[k][j] in lane j + 16k, D[i][j] in lane
// j + 16 (i % 4), register i / 4.
__device__ __forceinline__ v4d mfma16x16x4(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int NBP = 64;  // panel width of the blocked factorisation

// The reduction index of a 16x16x4 product may follow any order of the
// summed rows, as long as both operands use it.  The kernels below give
// lane i + 16 kk the rows (or panel columns) 4 kk + s of a block of 16 in
// product step s = 0..3: each lane then reads 4 consecutive entries of its
// column at once, and the 4 lanes that share a column cover 128
// contiguous bytes, one cache line per column instead of a quarter of one
// per load.

// Four consecutive doubles from p[0..3]; entries at or past `lim` (counted
// from p) read as zero.  Whole blocks take wide loads.
__device__ __forceinline__ void load4(const double *p, int lim, double (&v)[4]) {
  if (lim >= 4) {
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = p[s];
  } else {
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = s < lim ? p[s] : 0.0;
  }
}

// W (NBP x N) = Q_p^H (NBP x m) A_t (m x N), complex, planar FP64.
// Q_p: the panel's first column (plane stride plane), A_t: the first
// trailing column, W: output with leading dimension ldw (R's block row).
// One workgroup per 16 x 16 tile of W (grid: trailing column tiles x panel
// column tiles, 4 x 124 = 496 workgroups for the first 2048 panel, enough
// to occupy every compute unit); its QHA_SLICES waves each reduce over one
// slice of the m rows (a multiple of 16), and the slice partials are then
// summed in slice order through LDS, so the result does not depend on
// timing.
constexpr int QHA_SLICES = 8;
__global__ __launch_bounds__(64 * QHA_SLICES) void zgemm_qha_kernel(int m, int N, int nbp, const double *Qp, int ldq,
                                                                     const double *At, int lda, size_t plane,
                                                                     double *W, int ldw, size_t planeW) {
  __shared__ double red[QHA_SLICES - 1][64][8];
  const int lane = threadIdx.x & 63, ks = threadIdx.x >> 6;
  const int i0 = blockIdx.y * 16;  // panel column tile
  const int j0 = blockIdx.x * 16;  // trailing column tile
  const int li = lane & 15, lk = lane >> 4;
  const int qc = i0 + li;  // panel column read by this lane (A operand)
  const int tc = j0 + li;  // trailing column read by this lane (B operand)
  const bool qok = qc < nbp, tok = tc < N;
  const int mq = ((m + 16 * QHA_SLICES - 1) / (16 * QHA_SLICES)) * 16;  // rows per slice, multiple of 16
  const int k0 = ks * mq, k1 = min(m, k0 + mq);
  v4d cr = {0.0, 0.0, 0.0, 0.0}, ci = {0.0, 0.0, 0.0, 0.0};
  const double *qr = Qp + (size_t)(qok ? qc : 0) * ldq, *qi = qr + plane;
  const double *ar = At + (size_t)(tok ? tc : 0) * lda, *ai = ar + plane;
#pragma unroll 2
  for (int kb = k0; kb < k1; kb += 16) {
    const int row = kb + 4 * lk;  // rows row .. row + 3 of this lane
    const int lim = k1 - row;
    double a_r[4], a_i[4], b_r[4], b_i[4];
    load4(qr + row, qok ? lim : 0, a_r);
    load4(qi + row, qok ? lim : 0, a_i);
    load4(ar + row, tok ? lim : 0, b_r);
    load4(ai + row, tok ? lim : 0, b_i);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      // conj(q) a: re = qr ar + qi ai, im = qr ai - qi ar
      cr = mfma16x16x4(a_r[s], b_r[s], cr);
      cr = mfma16x16x4(a_i[s], b_i[s], cr);
      ci = mfma16x16x4(a_r[s], b_i[s], ci);
      ci = mfma16x16x4(-a_i[s], b_r[s], ci);
    }
  }
  if (ks > 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      red[ks - 1][lane][r] = cr[r];
      red[ks - 1][lane][4 + r] = ci[r];
    }
  }
  __syncthreads();
  if (ks != 0) return;
#pragma unroll
  for (int s = 0; s < QHA_SLICES - 1; ++s) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      cr[r] += red[s][lane][r];
      ci[r] += red[s][lane][4 + r];
    }
  }
  const int oc = j0 + li;
  if (oc < N) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int orow = i0 + lk + 4 * r;
      if (orow < nbp) {
        W[(size_t)oc * ldw + orow] = cr[r];
        W[(size_t)oc * ldw + orow + planeW] = ci[r];
      }
    }
  }
}

// A_t (m x N) -= Q_p (m x nbp) W (nbp x N).  One wave per 16 x 16 tile of
// A_t, K = nbp in blocks of 16 panel columns (the lane order above: W
// read 4 consecutive rows at a time, Q_p one column per product step,
// 16 consecutive rows across the lanes).
__global__ __launch_bounds__(256) void zgemm_update_kernel(int m, int N, int nbp, const double *Qp, int ldq,
                                                            double *At, int lda, size_t plane, const double *W,
                                                            int ldw, size_t planeW) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int tiles_m = (m + 15) / 16;
  const int tile = blockIdx.x * 4 + wave;
  const int ti = tile % tiles_m, tj = tile / tiles_m;
  if (tj * 16 >= N) return;
  const int i0 = ti * 16, j0 = tj * 16;
  const int li = lane & 15, lk = lane >> 4;
  // output tile values (D layout): row i0 + lk + 4r, column j0 + li
  const int oc = j0 + li;
  const bool cok = oc < N;
  v4d cr, ci;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int orow = i0 + lk + 4 * r;
    const bool ok = cok && orow < m;
    cr[r] = ok ? At[(size_t)oc * lda + orow] : 0.0;
    ci[r] = ok ? At[(size_t)oc * lda + orow + plane] : 0.0;
  }
  const int arow = i0 + li;  // A operand row (Q_p)
  const bool aok = arow < m;
  const double *wr = W + (size_t)(cok ? oc : 0) * ldw, *wi = wr + planeW;
  for (int kb = 0; kb < nbp; kb += 16) {
    const int k = kb + 4 * lk;  // panel columns k .. k + 3 of this lane
    const int lim = nbp - k;
    double w_r[4], w_i[4];
    load4(wr + k, cok ? lim : 0, w_r);
    load4(wi + k, cok ? lim : 0, w_i);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bool kok = aok && s < lim;
      const double q_r = kok ? Qp[(size_t)(k + s) * ldq + arow] : 0.0;
      const double q_i = kok ? Qp[(size_t)(k + s) * ldq + arow + plane] : 0.0;
      // a -= q w: re -= qr wr - qi wi, im -= qr wi + qi wr
      cr = mfma16x16x4(-q_r, w_r[s], cr);
      cr = mfma16x16x4(q_i, w_i[s], cr);
      ci = mfma16x16x4(-q_r, w_i[s], ci);
      ci = mfma16x16x4(-q_i, w_r[s], ci);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int orow = i0 + lk + 4 * r;
    if (cok && orow < m) {
      At[(size_t)oc * lda + orow] = cr[r];
      At[(size_t)oc * lda + orow + plane] = ci[r];
    }
  }
}

// ------------------------------------------------------- refinement ------
struct RefineCtl {
  int status;  // 0 running, 1 converged, 2 stagnated, 3 factorisation failed or a wait timed out
  int iters;
  double dprev;
  double err_est;
  unsigned int bar;    // arrivals at the grid barrier of proj_replay_kernel (zero at the start of a solve)
  unsigned int abort;  // set when one of its waits timed out
};

// Columns of Q64 (m x (n+1), ld m) from the leading limbs of A and b.
template <int L>
__global__ __launch_bounds__(256) void copy_hi_kernel(int m, int n, const double *A, int lda, const double *b,
                                                       double *Q64, RefineCtl *ctl, int *info) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int j = blockIdx.y;
  if (blockIdx.x == 0 && j == 0 && threadIdx.x == 0) {
    ctl->status = 0;
    ctl->iters = 0;
    ctl->dprev = INFINITY;
    ctl->err_est = INFINITY;
    ctl->bar = 0u;
    ctl->abort = 0u;
    *info = 0;
  }
  if (i >= m) return;
  const size_t plane64 = (size_t)m * (n + 1);
  if (j < n) {
    const size_t planeA = (size_t)lda * n;
    Q64[(size_t)j * m + i] = A[(size_t)j * lda + i];
    Q64[(size_t)j * m + i + plane64] = A[(size_t)j * lda + i + planeA];
  } else {
    Q64[(size_t)n * m + i] = b[i];
    Q64[(size_t)n * m + i + plane64] = b[i + m];
  }
}

// mgs_qr64: [A b] (FP64 complex planar, lda) into the working matrix
// Q64 (m x (n+1), column n = b or zero); clears info.
__global__ __launch_bounds__(256) void copy64_in_kernel(int m, int n, const double *A, int lda, const double *b,
                                                         double *Q64, int *info) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int j = blockIdx.y;
  if (blockIdx.x == 0 && j == 0 && threadIdx.x == 0) *info = 0;
  if (i >= m) return;
  const size_t plane64 = (size_t)m * (n + 1);
  if (j < n) {
    const size_t planeA = (size_t)lda * n;
    Q64[(size_t)j * m + i] = A[(size_t)j * lda + i];
    Q64[(size_t)j * m + i + plane64] = A[(size_t)j * lda + i + planeA];
  } else {
    Q64[(size_t)n * m + i] = b != nullptr ? b[i] : 0.0;
    Q64[(size_t)n * m + i + plane64] = b != nullptr ? b[i + m] : 0.0;
  }
}
// mgs_qr64: Q (m x n, ldq), R (n x n, ldr) and y (n) out of Q64 / R64.
// Block column j < n copies column j of Q and of R; j == n copies y.
__global__ __launch_bounds__(256) void copy64_out_kernel(int m, int n, const double *Q64, const double *R64,
                                                          double *Q, int ldq, double *R, int ldr, double *y) {
  const int j = blockIdx.y;
  const size_t plane64 = (size_t)m * (n + 1), planeR64 = (size_t)n * (n + 1);
  if (j < n) {
    const size_t planeQ = (size_t)ldq * n, planeR = (size_t)ldr * n;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < m; i += gridDim.x * 256) {
      Q[(size_t)j * ldq + i] = Q64[(size_t)j * m + i];
      Q[(size_t)j * ldq + i + planeQ] = Q64[(size_t)j * m + i + plane64];
    }
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
      R[(size_t)j * ldr + i] = R64[(size_t)j * n + i];
      R[(size_t)j * ldr + i + planeR] = R64[(size_t)j * n + i + planeR64];
    }
  } else if (y != nullptr) {
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
      y[i] = R64[(size_t)n * n + i];
      y[i + n] = R64[(size_t)n * n + i + planeR64];
    }
  }
}

__global__ __launch_bounds__(256) void fill_zero_kernel(double *p, size_t count) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256) p[i] = 0.0;
}

// r = b - A x accumulated in quad-double whatever the working precision
// (A, b, x stored with LP limbs are widened exactly), split over column
// chunks: block (rb, cb) sums the columns [cb*CH, cb*CH + CH) of rows
// rb*256 .. into partial[cb][row].  Only the FP64 rounding of r feeds the
// correction; twice the working precision for dd keeps the residual's own
// error below the dd solution's.
template <int LP>
__device__ __forceinline__ cqd load_qd_from(const double *p, size_t plane) {
  cqd v;
  v.re.x0 = p[0];
  v.im.x0 = p[plane];
  v.re.x1 = LP > 1 ? p[2 * plane] : 0.0;
  v.im.x1 = LP > 1 ? p[3 * plane] : 0.0;
  v.re.x2 = LP > 2 ? p[4 * plane] : 0.0;
  v.im.x2 = LP > 2 ? p[5 * plane] : 0.0;
  v.re.x3 = LP > 2 ? p[6 * plane] : 0.0;
  v.im.x3 = LP > 2 ? p[7 * plane] : 0.0;
  return v;
}
template <int LP>
__global__ __launch_bounds__(256) void residual_partial_kernel(int m, int n, int chunk, const double *A, int lda,
                                                                const double *b, const double *x,
                                                                Partial<PrecQD>::T *partial, const RefineCtl *ctl) {
  if (ctl->status != 0) return;
  using P = PrecQD;
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int cb = blockIdx.y;
  if (i >= m) return;
  const size_t planeA = (size_t)lda * n;
  P::Acc acc;
  if (cb == 0)
    P::acc_set(acc, load_qd_from<LP>(b + i, (size_t)m));
  else
    P::acc_zero(acc);
  const int j1 = min(n, (cb + 1) * chunk);
  for (int j = cb * chunk; j < j1; ++j)
    P::acc_cmul(acc, load_qd_from<LP>(A + (size_t)j * lda + i, planeA), P::cneg(load_qd_from<LP>(x + j, (size_t)n)));
  partial[(size_t)cb * m + i] = Partial<P>::pack(acc);
}

// Sum the chunk partials in chunk order; r64 = FP64 rounding of r.
template <class P>
__global__ __launch_bounds__(256) void residual_finish_kernel(int m, int nchunk,
                                                               const typename Partial<P>::T *partial, double *r64,
                                                               const RefineCtl *ctl) {
  if (ctl->status != 0) return;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= m) return;
  typename P::Acc acc = Partial<P>::unpack(partial[i]);
  for (int c = 1; c < nchunk; ++c) P::acc_merge(acc, Partial<P>::unpack(partial[(size_t)c * m + i]));
  typename P::C v = P::acc_value(acc);
  double tmp[2 * P::L];
  P::store(tmp, 1, v);  // tmp[0] = re hi, tmp[1] = im hi (planes 0 and 1)
  r64[i] = tmp[0];
  r64[i + m] = tmp[1];
}

// w = Q_p^H r: one block per panel column, rows summed in a fixed order.
__global__ __launch_bounds__(256) void proj_w_kernel(int m, const double *Qp, int ldq, size_t plane,
                                                      const double *r, double *w, size_t planew,
                                                      const RefineCtl *ctl) {
  if (ctl->status != 0) return;
  __shared__ double sr[4], si[4];
  const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double *qr = Qp + (size_t)c * ldq, *qi = qr + plane;
  double ar = 0.0, ai = 0.0;
  for (int i = tid; i < m; i += 256) {
    const double xr = r[i], xi = r[i + m];
    ar = __fma_rn(qr[i], xr, ar);
    ar = __fma_rn(qi[i], xi, ar);
    ai = __fma_rn(qr[i], xi, ai);
    ai = __fma_rn(-qi[i], xr, ai);
  }
#pragma unroll
  for (int mask = 32; mask >= 1; mask >>= 1) {
    ar += __shfl_xor(ar, mask);
    ai += __shfl_xor(ai, mask);
  }
  if (lane == 0) {
    sr[wave] = ar;
    si[wave] = ai;
  }
  __syncthreads();
  if (tid == 0) {
    w[c] = ((sr[0] + sr[1]) + sr[2]) + sr[3];
    w[c + planew] = ((si[0] + si[1]) + si[2]) + si[3];
  }
}

// r -= Q_p w, one row per thread.
__global__ __launch_bounds__(256) void proj_r_kernel(int m, int nbp, const double *Qp, int ldq, size_t plane,
                                                      const double *w, size_t planew, double *r,
                                                      const RefineCtl *ctl) {
  if (ctl->status != 0) return;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= m) return;
  double xr = r[i], xi = r[i + m];
  for (int c = 0; c < nbp; ++c) {
    const double qr = Qp[(size_t)c * ldq + i], qi = Qp[(size_t)c * ldq + i + plane];
    const double wr = w[c], wi = w[c + planew];
    xr = __fma_rn(-qr, wr, xr);
    xr = __fma_rn(qi, wi, xr);
    xi = __fma_rn(-qr, wi, xi);
    xi = __fma_rn(-qi, wr, xi);
  }
  r[i] = xr;
  r[i + m] = xi;
}

// The correction's projections of all panels in one cooperative launch (one
// per refinement step instead of two per panel): for each panel of NBP
// columns w_p = Q_p^H r, then r -= Q_p w_p.  Workgroup g holds rows 64 g ..
// 64 g + 63 of r in registers for the whole launch, a row per lane, and wave
// v its rows' entries of columns 16 v .. 16 v + 15 of the panel: both
// products use them from one (coalesced) read, issued a panel ahead.  The
// 16 columns' sums over the wave's rows halve the lanes and the values
// together, step by step (31 additions for 32 sums).  Between workgroups
// only the 128 partial sums per workgroup and panel pass, through `part`:
// every workgroup reads all of them and adds them in one fixed order, so
// that one exchange per panel is enough (bounded by it: 2048 x 2048, 781 ->
// 111 us per step; one exchange of w and one of r, by two grid barriers,
// before).
//
// `part` ([min(3, panels)][G][2 NBP]) holds the empty marker until a value is written
// (device-scope), so readers poll the data; a workgroup clears what it wrote
// for panel p-1 when it has read all of panel p (which nobody sends before
// having read panel p-1), and its stores are complete before it sends panel
// p+1, which precedes any look at panel p+2 in the same place.  Before the
// first panel every workgroup clears its places and the grid meets once
// (ctl->bar, which grows by G per step from `base`).  On a time-out the step
// ends with status 3 and MGS_INFO_SYNC_TIMEOUT in info.  m <= PR_MAX_ROWS.
constexpr int PR_MAX_ROWS = 4096;
constexpr int PR_ROWS = 64;  // rows per workgroup
// One step of a wave's sums: the lanes with (lane & BIT) == 0 go on with a,
// the others with b; CTRL brings the other lane's value.
template <int BIT, int CTRL>
__device__ __forceinline__ double pr_fold(double a, double b, int lane) {
  const bool up = (lane & BIT) != 0;
  return (up ? b : a) + dpp_shift<CTRL, 0xf>(up ? a : b);
}
__global__ __launch_bounds__(256) void proj_replay_kernel(int m, int n, const double *Q, size_t planeQ,
                                                           const double *r, double *w, size_t planew, double *part,
                                                           RefineCtl *ctl, int *info, unsigned int base,
                                                           long long spin_ticks, unsigned jitter) {
  if (ctl->status != 0) return;
  constexpr int WC = NBP / 4;  // panel columns per wave
  __shared__ double ws[2][2 * NBP];   // w in two halves of the workgroups
  __shared__ double xs[4][2][PR_ROWS];  // the waves' parts of Q_p w_p
  __shared__ int bad;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = gridDim.x, g = blockIdx.x;
  const int row = g * PR_ROWS + lane;
  const int np = (n + NBP - 1) / NBP;
  const size_t slot = (size_t)2 * NBP * G;  // doubles per panel of `part`
  // this lane's place among a workgroup's sums: real parts, then imaginary
  const int at = (lane >> 5) * NBP + wave * WC + ((lane >> 1) & (WC - 1));
  double *own = part + (size_t)g * 2 * NBP + at;
  const double e = __longlong_as_double(RES_EMPTY);
  if (tid == 0) bad = 0;
  if (tid < 2 * NBP) ws[1][tid] = 0.0;
  PollBound poll;
  auto give_up = [&]() __attribute__((always_inline)) {
    if (!poll.due()) return false;
    if (__hip_atomic_load(&ctl->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u && !poll.late(spin_ticks))
      return false;
    __hip_atomic_store(&ctl->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
  };
  auto fail = [&]() __attribute__((always_inline)) {
    if (tid == 0) {
      ctl->status = 3;
      __hip_atomic_store(info, MGS_INFO_SYNC_TIMEOUT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  double qr[WC], qi[WC];
  auto load_panel = [&](int p, double (&vr)[WC], double (&vi)[WC]) __attribute__((always_inline)) {
    const int c0 = p * NBP + wave * WC;
    const double *src = Q + (size_t)c0 * m + row;
#pragma unroll
    for (int c = 0; c < WC; ++c) {
      const bool in = c0 + c < n && row < m;
      vr[c] = in ? src[(size_t)c * m] : 0.0;
      vi[c] = in ? src[(size_t)c * m + planeQ] : 0.0;
    }
  };
  load_panel(0, qr, qi);
  double xr = row < m ? r[row] : 0.0, xi = row < m ? r[row + m] : 0.0;
  if (G > 1) {
    if ((lane & 1) == 0) {
      for (int k = 0; k < 3 && k < np; ++k) coh_store(own + k * slot, e);
    }
    wait_vmem();
    __syncthreads();
    if (tid == 0) {
      atomicAdd(&ctl->bar, 1u);
      while (__hip_atomic_load(&ctl->bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < base + (unsigned int)G) {
        if (give_up()) {
          bad = 1;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
  }
  __syncthreads();
  if (bad != 0) return fail();
  int buf = 0, prev = 2;  // panel p mod 3, p - 1 mod 3
  for (int p = 0; p < np; ++p) {
    res_jitter(jitter, (unsigned)p);
    // v[c], v[WC + c]: q_c^H r over this lane's row, then over the wave's
    double v[2 * WC];
#pragma unroll
    for (int c = 0; c < WC; ++c) {
      v[c] = __fma_rn(qi[c], xi, qr[c] * xr);
      v[WC + c] = __fma_rn(-qi[c], xr, qr[c] * xi);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      lane_swap32(v[i], v[i + 16]);
      v[i] += v[i + 16];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      lane_swap16(v[i], v[i + 8]);
      v[i] += v[i + 8];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = pr_fold<8, 0x128>(v[i], v[i + 4], lane);  // row_ror:8: lane ^ 8
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = pr_fold<4, 0x141>(v[i], v[i + 2], lane);  // row_half_mirror: lane ^ 7
    v[0] = pr_fold<2, 0x4E>(v[0], v[1], lane);                                   // quad_perm: lane ^ 2
    v[0] += dpp_shift<0xB1, 0xf>(v[0]);                                          // quad_perm: lane ^ 1
    double nr[WC], ni[WC];
    if (G == 1) {
      if ((lane & 1) == 0) ws[0][at] = v[0];
      load_panel(p + 1, nr, ni);
    } else {
      wait_vmem();  // the cleared places of panel p - 2
      if ((lane & 1) == 0) coh_store(own + buf * slot, v[0]);
      load_panel(p + 1, nr, ni);
      // sum tid mod 2 NBP of the workgroups of one parity
      const double *src = part + buf * slot + (tid & (2 * NBP - 1));
      const int h = tid / (2 * NBP);
      double sum = 0.0;
      constexpr int NF = 16;  // reads in flight
      for (int g0 = h; g0 < G; g0 += 2 * NF) {
        double t[NF];
        while (true) {
          bool miss = false;
#pragma unroll
          for (int i = 0; i < NF; ++i) {
            const int gi = g0 + 2 * i;
            t[i] = gi < G ? coh_load(src + (size_t)gi * 2 * NBP) : 0.0;
            miss = miss || __double_as_longlong(t[i]) == RES_EMPTY;
          }
          if (__ballot(miss) == 0) break;
          if (give_up()) {
            bad = 1;
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
#pragma unroll
        for (int i = 0; i < NF; ++i) sum += t[i];
      }
      ws[h][tid & (2 * NBP - 1)] = sum;
    }
    __syncthreads();
    if (bad != 0) return fail();
    if (G > 1 && p > 0 && (lane & 1) == 0) coh_store(own + prev * slot, e);
    if (g == 0 && tid < NBP && p * NBP + tid < n) {
      w[p * NBP + tid] = ws[0][tid] + ws[1][tid];
      w[p * NBP + tid + planew] = ws[0][NBP + tid] + ws[1][NBP + tid];
    }
    double ar = 0.0, ai = 0.0;
#pragma unroll
    for (int c = 0; c < WC; ++c) {
      const int k = wave * WC + c;
      const double wr = ws[0][k] + ws[1][k], wi = ws[0][NBP + k] + ws[1][NBP + k];
      ar = __fma_rn(qr[c], wr, ar);
      ar = __fma_rn(-qi[c], wi, ar);
      ai = __fma_rn(qr[c], wi, ai);
      ai = __fma_rn(qi[c], wr, ai);
    }
    xs[wave][0][lane] = ar;
    xs[wave][1][lane] = ai;
    __syncthreads();
    xr -= (xs[0][0][lane] + xs[1][0][lane]) + (xs[2][0][lane] + xs[3][0][lane]);
    xi -= (xs[0][1][lane] + xs[1][1][lane]) + (xs[2][1][lane] + xs[3][1][lane]);
#pragma unroll
    for (int c = 0; c < WC; ++c) {
      qr[c] = nr[c];
      qi[c] = ni[c];
    }
    prev = buf;
    buf = buf == 2 ? 0 : buf + 1;
  }
}

// The FP64 solution as the dd / qd starting x (first solve).
template <class P>
__global__ __launch_bounds__(256) void set_x_kernel(int n, const double *x64, double *x) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  for (int p = 0; p < 2 * P::L; ++p) x[i + (size_t)p * n] = (p < 2) ? x64[i + (size_t)p * n] : 0.0;
}

// x += d (d in FP64), with the stopping test on ||d|| and ||x||: stop when
// ||d|| <= tol ||x|| (converged) or ||d|| > ||d_prev|| / 2 (stalled), and
// nothing more once info is set (a triangular solve timed out).  One block.
template <class P>
__global__ __launch_bounds__(256) void refine_update_kernel(int n, const double *d64, double *x, double tol,
                                                             int iter, RefineCtl *ctl, const int *info) {
  if (ctl->status != 0) return;
  if (*info != 0) {
    if (threadIdx.x == 0) ctl->status = 3;
    return;
  }
  __shared__ double red[2][4];
  __shared__ int stag;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double dn = 0.0, xn = 0.0;
  for (int i = tid; i < n; i += 256) {
    const double dr = d64[i], di = d64[i + n];
    dn = __fma_rn(dr, dr, __fma_rn(di, di, dn));
    const double xr = x[i], xi = x[i + n];
    xn = __fma_rn(xr, xr, __fma_rn(xi, xi, xn));
  }
#pragma unroll
  for (int mask = 32; mask >= 1; mask >>= 1) {
    dn += __shfl_xor(dn, mask);
    xn += __shfl_xor(xn, mask);
  }
  if (lane == 0) {
    red[0][wave] = dn;
    red[1][wave] = xn;
  }
  __syncthreads();
  dn = sqrt(((red[0][0] + red[0][1]) + red[0][2]) + red[0][3]);
  xn = sqrt(((red[1][0] + red[1][1]) + red[1][2]) + red[1][3]);
  if (tid == 0) stag = (iter > 1 && dn > 0.5 * ctl->dprev) ? 1 : 0;
  __syncthreads();
  if (stag) {
    // The corrections stopped shrinking: converged to the attainable
    // accuracy when the last applied one was already below sqrt(tol) of x,
    // a failure otherwise.  The stalled correction is not applied.
    if (tid == 0) ctl->status = (ctl->err_est <= sqrt(tol)) ? 1 : 2;
    return;
  }
  for (int i = tid; i < n; i += 256) {
    typename P::C v = P::load(x + i, (size_t)n);
    P::add_cd(v, d64[i], d64[i + n]);
    P::store(x + i, (size_t)n, v);
  }
  if (tid == 0) {
    ctl->iters = iter;
    ctl->err_est = xn > 0.0 ? dn / xn : dn;
    ctl->dprev = dn;
    if (dn <= tol * xn) ctl->status = 1;
  }
}

// Skip the refinement when the factorisation reported a bad column.
__global__ void refine_check_kernel(const int *info, RefineCtl *ctl) {
  if (threadIdx.x == 0 && blockIdx.x == 0 && *info != 0) ctl->status = 3;
}

__global__ void refine_finish_kernel(const RefineCtl *ctl, int *iters, double *err_est, int *info) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  if (iters) *iters = ctl->iters;
  if (err_est) *err_est = ctl->err_est;
  if (*info == 0) *info = ctl->status == 1 ? 0 : (ctl->status == 2 ? -1 : -2);
}

}  // namespace mgsq
