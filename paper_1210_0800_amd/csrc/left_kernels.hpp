// Left-looking MGS in one persistent launch, for qd (whose columns are too
// wide to keep all of them in registers): the operations of Figure 1
// (Section 3) on the augmented matrix of Equation (1), one column at a time
// per workgroup.
//
// A workgroup takes the next column of [A b] that nobody has taken (a counter),
// loads it once, applies the projections k = 0, 1, ..., c-1 in order as they
// become available, writes it once, and takes another.  The columns handed on
// are the unnormalised ones: u_k is column k after its last projection, and
//   r_kj = (u_k^H a_j) / r_kk,   a_j -= ((u_k^H a_j) / ||u_k||^2) u_k,
// equal to q_k^H a_j and r_kj q_k in exact arithmetic, so neither the square
// root nor the normalisation is on the chain from column to column: a link
// is u_k's hand-off, one inner product beside ||u_k||^2 (formed once, by its
// owner), one product and one update.  1 / ||u_k||^2 and 1 / r_kk go to a
// record per column; left_finish_kernel then scales Q's columns and R's
// rows by 1 / r_kk.  The right-hand side, whose size has nothing to do with
// the columns', uses q_k = u_k / r_kk itself.
//
// What bounds it: up to one column per workgroup, the chain (5.5 us a link at
// 80 rows, 8.1 at 320, where one launch per column took 16 and 24); beyond,
// the issue of the qd operations (1024 x 1024: 1.08e10 wave instructions,
// 17.5 ms of 30.2; one launch per column 71.5) and waiting at the chain.
// Equal work per compute unit by dealing the second workgroup of each its
// columns in reverse was slower (42.7 ms against 32.6 a solve), as was a
// raised wave priority near the chain at 300 columns (5.2 against 4.7 ms).
//
// u_k passes through Q with device-scope stores.  Q and the records hold the
// empty marker until written, so readers poll the data itself; when Q is A
// (in place) they wait for a counter per wave instead, which moves once the
// wave's stores are complete (wave w of every workgroup holds the same rows,
// so no barrier is needed on either side either way).  Every wait is
// bounded by a wall-clock limit and ends through the abort flag that all
// waits observe.  Column c waits only for columns before it, and those were
// taken before it, by workgroups that run or have finished: so the launch
// needs no more than one workgroup on the card at a time to end, and is an
// ordinary one.  (Columns dealt by workgroup number wait for workgroups that
// may not have started, e.g. behind another stream's kernel, and need a
// cooperative launch; those do not run beside each other.)
#pragma once
#include "../../include/mgsqr.h"
#include "batched_kernels.hpp"

namespace mgsq {

// Words of LeftArgs::sync: the next column to take, the workgroups that have
// met, and what came of it (0 open, 1 all met, 2 not).
constexpr int LEFT_NEXT = 192, LEFT_MET = 208, LEFT_MODE = 224;

struct LeftArgs {
  int m, n, ncols;  // ncols = n + 1 when b is augmented
  const double *A;
  int lda;
  size_t planeA;
  const double *b;
  double *Q;
  int ldq;
  size_t planeQ;
  double *R;
  int ldr;
  size_t planeR;
  double *y;
  double *rho;
  int *info;
  double *rec;         // per column k: 1 / ||u_k||^2, then 1 / r_kk (L doubles each)
  unsigned int *sync;  // RES_SYNC_WORDS words: per-wave counters (up to 8), LEFT_NEXT, _MET, _MODE, the abort flag
  int meet;  // several workgroups share a compute unit: 50 us on the wall clock; else 0
  int marked;            // Q holds the empty marker at the start (Q is not A)
  long long spin_ticks;  // wall-clock limit of one wait
  unsigned jitter;       // race checks: seed of the timing jitter (0: none)
};

// Counters and abort flag cleared, info cleared, records marked empty, and
// (np planes) the columns of Q.  Grid: rows / 256, at least one workgroup
// per column.
__global__ __launch_bounds__(256) void left_init_kernel(unsigned int *sync, int *info, double *rec, int nrec, int m,
                                                        int n, double *Q, int ldq, size_t planeQ, int np) {
  const double e = __longlong_as_double(RES_EMPTY);
  const int i = blockIdx.x * 256 + threadIdx.x, j = blockIdx.y;
  if (i < m && j < n) {
    for (int p = 0; p < np; ++p) Q[(size_t)j * ldq + i + p * planeQ] = e;
  }
  if (blockIdx.x != 0) return;
  if (j == 0) {
    for (int t = threadIdx.x; t < RES_SYNC_WORDS; t += 256) sync[t] = 0u;
    if (threadIdx.x == 0) *info = 0;
  }
  for (int t = j * 256 + threadIdx.x; t < nrec; t += gridDim.y * 256) rec[t] = e;
}

// RPT rows per thread (m <= 64 NW RPT), NW waves, PC workgroups per compute
// unit (the register budget: two hide each other's loads and barriers).
template <class P, int RPT, int NW, int PC>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW * PC < 4 ? 1 : NW * PC / 4))) void
mgs_left_kernel(LeftArgs a) {
  using C = typename P::C;
  using Acc = typename P::Acc;
  using RAcc = typename P::RAcc;
  using Rl = typename P::R;
  using G = GridSum<P>;
  constexpr int H = G::H, L = P::L, RWG = 64 * NW;
  __shared__ double xch[2][2][H][NW];  // wave totals, [buffer][part][word][wave]
  __shared__ double lrec[2][L];        // 1 / ||u_k||^2 of the step
  __shared__ int emax;                 // a large column's exponent
  __shared__ int taken;                // the workgroup's column
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  int buf = 0, seen = 0;
  unsigned step = 0;
  C col[RPT], u[RPT];

  // This wave's total of t: the real part in the lower half of the lanes,
  // the imaginary part (the real one again for a real sum) in the upper.
  auto put = [&](RAcc re, RAcc im) __attribute__((always_inline)) {
    RAcc v = G::fold32(re, im);
    v = G::fold16(v, v);
    G::template rot<0x128>(v);  // row_ror:8
    G::template rot<0x124>(v);  // row_ror:4
    G::template rot<0x122>(v);  // row_ror:2
    G::template rot<0x121>(v);  // row_ror:1
    if ((lane & 31) == 0) {
      const double *p = reinterpret_cast<const double *>(&v);
#pragma unroll
      for (int i = 0; i < H; ++i) xch[buf][lane >> 5][i][wave] = p[i];
    }
  };
  // The block's total, by halves: a butterfly over the NW wave totals (the
  // merge is symmetric, so every wave ends with the same bits).  The buffers
  // alternate, so one barrier per sum is enough.
  auto total = [&]() __attribute__((always_inline)) {
    RAcc v;
    double *p = reinterpret_cast<double *>(&v);
#pragma unroll
    for (int i = 0; i < H; ++i) p[i] = xch[buf][lane >> 5][i][lane & (NW - 1)];
    if constexpr (NW >= 2) G::template rot<0xB1>(v);   // quad_perm: lane ^ 1
    if constexpr (NW >= 4) G::template rot<0x4E>(v);   // quad_perm: lane ^ 2
    if constexpr (NW >= 8) G::template rot<0x124>(v);  // row_ror:4: the totals repeat with period 8
    buf ^= 1;
    return P::racc_value(v);
  };
  // Part `which` of column k's record: one read, and the wait until it is
  // written (false on abort).
  auto read_record = [&](int k, int which, Rl &v) __attribute__((always_inline)) {
    const double *p = a.rec + ((size_t)k * 2 + which) * L;
    double *pv = reinterpret_cast<double *>(&v);
#pragma unroll
    for (int i = 0; i < L; ++i) pv[i] = coh_load(p + i);
  };
  auto wait_record = [&](int k, int which, Rl &v) __attribute__((always_inline)) {
    const double *pv = reinterpret_cast<const double *>(&v);
    PollBound poll;
    while (true) {
      bool miss = false;
#pragma unroll
      for (int i = 0; i < L; ++i) miss = miss || __double_as_longlong(pv[i]) == RES_EMPTY;
      if (__ballot(miss) == 0) return true;
      if (res_give_up(a, poll)) return false;
      __builtin_amdgcn_s_sleep(1);
      read_record(k, which, v);
    }
  };
  auto put_record = [&](int k, int which, const Rl &v) __attribute__((always_inline)) {
    double t[L];
    P::store_real(t, 1, v);
    if (tid == 0) {
#pragma unroll
      for (int i = 0; i < L; ++i) coh_store(a.rec + ((size_t)k * 2 + which) * L + i, t[i]);
    }
  };
  // The limbs of v (real part: lane 0, imaginary part: lane 32 of wave 0).
  auto store_parts = [&](double *p, size_t plane, const Rl &v) __attribute__((always_inline)) {
    if (wave == 0 && (lane & 31) == 0) P::store_real(p + (lane >> 5) * plane, 2 * plane, v);
  };

  // Columns that share a compute unit should be far apart, so where several
  // workgroups share one they meet first, and once all are on the card the
  // columns are dealt by workgroup number (workgroups i and i + 256 share a
  // unit: 1024 x 288 4.5 ms, by the counter alone 6.1).  If they have not met
  // after a.meet (50 us), one of them decides for the counter.
  bool dealt = false;
  if (a.meet > 0) {
    if (tid == 0) {
      unsigned int *mode = a.sync + LEFT_MODE, now;
      if (__hip_atomic_fetch_add(a.sync + LEFT_MET, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x)
        atomicCAS(mode, 0u, 1u);
      const long long t0 = wall_clock64();
      while ((now = __hip_atomic_load(mode, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0u) {
        if (wall_clock64() - t0 > a.meet) atomicCAS(mode, 0u, 2u);
        __builtin_amdgcn_s_sleep(2);
      }
      taken = (int)now;
    }
    __syncthreads();
    dealt = __builtin_amdgcn_readfirstlane(taken) == 1;
    __syncthreads();
  }
  for (int c = dealt ? (int)blockIdx.x - (int)gridDim.x : -1; c != a.ncols - 1;) {
    if (dealt) {
      c += gridDim.x;
    } else {
      // (every wave has read the last number before its sums' barriers)
      if (tid == 0)
        taken = (int)__hip_atomic_fetch_add(a.sync + LEFT_NEXT, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __syncthreads();
      c = __builtin_amdgcn_readfirstlane(taken);
    }
    if (c >= a.ncols) break;
    const bool isb = c == a.n;
    {
      const double *src = isb ? a.b : a.A + (size_t)c * a.lda;
      const size_t pl = isb ? (size_t)a.m : a.planeA;
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        const int i = r * RWG + tid;
        col[r] = i < a.m ? P::load(src + i, pl) : P::czero();
      }
    }
    // The power of two (`up`) of a column's largest entry when that is not
    // within 2^-64 .. 2^64.  u_c is divided by it when it is handed on, so that
    // 1 / ||u||^2 and u^H a are in range wherever those of q_c are; the column
    // itself stays as it is.  An infinity or a NaN stays one; the bound keeps
    // both powers normal numbers.
    double up = 1.0;
    if (!isb) {
      double t[2 * L], big = 0.0;
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        P::store(t, 1, col[r]);
        big = fmax(big, fmax(fabs(t[0]), fabs(t[1])));
      }
      if (__syncthreads_or(big >= 0x1p64 || (big > 0.0 && big <= 0x1p-64))) {
        if (tid == 0) emax = -2000;
        __syncthreads();
        if (big > 0.0) atomicMax(&emax, big < INFINITY ? ilogb(big) : 2000);
        __syncthreads();
        const int e = emax >= 2000 || (emax < 64 && emax >= -64) ? 0 : emax;
        up = ldexp(1.0, e > 1000 ? 1000 : e < -1000 ? -1000 : e);
      }
    }
    const int kend = c < a.n ? c : a.n;
#pragma unroll 1
    for (int k = 0; k < kend; ++k) {
      res_jitter(a.jitter, step++);
      if (!a.marked && !res_wait(a, k, wave, seen)) return;
      const double *src = a.Q + (size_t)k * a.ldq;
      PollBound poll;
      while (true) {
        bool miss = false;
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
          const int i = row_of(r, RWG);
          u[r] = i < a.m ? res_coh_load<P>(src + i, a.planeQ, miss) : P::czero();
        }
        if (!a.marked || __ballot(miss) == 0) break;
        if (res_give_up(a, poll)) return;
        __builtin_amdgcn_s_sleep(1);
      }
      Rl rec = P::rzero();
      if (isb || wave == 0) read_record(k, isb ? 1 : 0, rec);
      if (isb) {
        if (!wait_record(k, 1, rec)) return;
#pragma unroll
        for (int r = 0; r < RPT; ++r) u[r] = P::scale(u[r], rec);
      }
      Acc t;
      P::acc_zero(t);
#pragma unroll
      for (int r = 0; r < RPT; ++r) P::acc_cmulc(t, u[r], col[r]);
      put(G::parts(t)[0], G::parts(t)[1]);
      // 1 / ||u_k||^2 by way of the first wave (256 workgroups on one line,
      // not all their waves): before the sum's barrier when another
      // workgroup of the compute unit fills the wait, after it when the
      // wait is the chain's.
      if (PC > 1 && wave == 0 && !isb) {
        if (!wait_record(k, 0, rec)) return;
        if (lane == 0) P::store_real(&lrec[buf][0], 1, rec);
      }
      const int at = buf;
      lds_barrier();
      Rl v = total();
      if (isb) {
        store_parts(a.y + k, (size_t)a.n, v);
      } else {
        if (PC == 1 && wave == 0) {
          if (!wait_record(k, 0, rec)) return;
          if (lane == 0) P::store_real(&lrec[at][0], 1, rec);
        }
        if (PC == 1 && NW > 1) lds_barrier();
        if (NW > 1) {
          double *pw = reinterpret_cast<double *>(&rec);
#pragma unroll
          for (int i = 0; i < L; ++i) pw[i] = lrec[at][i];
        }
        store_parts(a.R + (size_t)c * a.ldr + k, a.planeR, v);
        v = P::rmul(v, rec);
      }
      const C rk = G::spread(v);
#pragma unroll
      for (int r = 0; r < RPT; ++r) P::upd(col[r], rk, u[r]);
    }
    if (up != 1.0) {
      double t[2 * L];
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        P::store(t, 1, col[r]);
#pragma unroll
        for (int i = 0; i < 2 * L; ++i) t[i] *= pow2_inverse(up);
        col[r] = P::load(t, 1);
      }
    }
    if (!isb) {
      // u_c out (column 0 is raw input: an entry with the marker's bits
      // leaves as a quiet NaN).
      double *dst = a.Q + (size_t)c * a.ldq;
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        const int i = row_of(r, RWG);
        if (i < a.m) res_coh_store<P>(dst + i, a.planeQ, col[r], c == 0);
      }
      if (!a.marked) {
        wait_vmem();
        if (lane == 0)
          __hip_atomic_fetch_max(a.sync + 16 * wave, (unsigned int)(c + 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    if (isb && a.rho == nullptr) continue;
    Acc t;
    P::acc_zero(t);
#pragma unroll
    for (int r = 0; r < RPT; ++r) P::acc_abs2(t, col[r]);
    put(G::parts(t)[0], G::parts(t)[0]);
    lds_barrier();
    const Rl s2 = total();
    if (wave != 0) continue;
    if (isb) {
      if (tid == 0) P::store_real(a.rho, 1, P::ok_norm(s2) ? P::sqrt_(s2) : P::rzero());
      continue;
    }
    put_record(c, 0, P::recip(s2));
    Rl rkk, inv;
    root_and_inverse<P>(s2, rkk, inv);
    put_record(c, 1, inv);
    if (tid == 0) {
      double t[L];
      P::store_real(t, 1, s2);
      const double n2 = t[0] * up * up;  // ||a_c||^2
      const bool ok = P::ok_norm(s2) && n2 < INFINITY && n2 > 0.0;
      if (!ok) info_first_bad(a.info, c + 1);
      // (a refused column's r_cc is not a pivot: later calls with R refuse it too)
      P::store_real(t, 1, rkk);
      if (!ok) t[0] = n2;
      double *d = a.R + (size_t)c * a.ldr + c;
#pragma unroll
      for (int i = 0; i < L; ++i) {
        d[(size_t)(2 * i) * a.planeR] = ok ? t[i] * up : t[i];
        d[(size_t)(2 * i + 1) * a.planeR] = 0.0;
      }
    }
  }
}

// Column j of Q times 1 / r_jj, R(k, j) times 1 / r_kk for k < j, zeros below
// R's diagonal.  One workgroup per column.
template <class P>
__global__ __launch_bounds__(256) void left_finish_kernel(int m, int n, double *Q, int ldq, size_t planeQ, double *R,
                                                          int ldr, size_t planeR, const double *rec) {
  using Rl = typename P::R;
  const int j = blockIdx.x;
  auto inverse = [&](int k) __attribute__((always_inline)) {
    Rl v;
    double *pv = reinterpret_cast<double *>(&v);
#pragma unroll
    for (int i = 0; i < P::L; ++i) pv[i] = rec[((size_t)k * 2 + 1) * P::L + i];
    return v;
  };
  const Rl inv = inverse(j);
  for (int i = threadIdx.x; i < m; i += 256) {
    double *p = Q + (size_t)j * ldq + i;
    P::store(p, planeQ, P::scale(P::load(p, planeQ), inv));
  }
  for (int k = threadIdx.x; k < n; k += 256) {
    double *p = R + (size_t)j * ldr + k;
    if (k < j)
      P::store(p, planeR, P::scale(P::load(p, planeR), inverse(k)));
    else if (k > j)
      P::store(p, planeR, P::czero());
  }
}

// Projections y = Q^H b: y_k = q_k^H b^(k-1), b^(k) = b^(k-1) - y_k q_k for
// k = 1..n, the operations of the augmented column of Equation (1).  One
// workgroup of 8 waves, b in registers (RPT rows per thread).  A chain of
// one inner product, one block sum (one barrier: two buffers alternate) and
// one update per column; q_k is loaded RING columns ahead, so the memory's
// latency is off the chain (700 x 500 double: 0.89 us a column with the
// loads on it and two barriers).
template <class P, int RPT, int RING>
__global__ __launch_bounds__(512) void project_kernel(int m, int n, const double *Q, int ldq, size_t planeQ,
                                                      const double *b, double *y) {
  using C = typename P::C;
  using Acc = typename P::Acc;
  using RAcc = typename P::RAcc;
  using Rl = typename P::R;
  using G = GridSum<P>;
  constexpr int NW = 8, H = G::H, RWG = 64 * NW;
  __shared__ double xch[2][2][H][NW];  // wave totals, [buffer][part][word][wave]
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // rows past m load the last row and hold a zero of b
  C bv[RPT];
  int row[RPT];
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const int i = r * RWG + tid;
    row[r] = i < m ? i : m - 1;
    bv[r] = i < m ? P::load(b + i, (size_t)m) : P::czero();
  }
  C q[RING][RPT];
  auto fetch = [&](int k, C (&v)[RPT]) __attribute__((always_inline)) {
    const double *qk = Q + (size_t)min(k, n - 1) * ldq;
#pragma unroll
    for (int r = 0; r < RPT; ++r) v[r] = P::load(qk + row[r], planeQ);
  };
  static_for<RING>([&](auto tI) __attribute__((always_inline)) {
    constexpr int t = decltype(tI)::value;
    fetch(t, q[t]);
  });
  int buf = 0;
#pragma unroll 1
  for (int k0 = 0; k0 < n; k0 += RING) {
    static_for<RING>([&](auto tI) __attribute__((always_inline)) {
      constexpr int t = decltype(tI)::value;
      const int k = k0 + t;
      Acc acc;
      P::acc_zero(acc);
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        if (r * RWG + tid >= m) q[t][r] = P::czero();
        P::acc_cmulc(acc, q[t][r], bv[r]);
      }
      RAcc v = G::fold32(G::parts(acc)[0], G::parts(acc)[1]);
      v = G::fold16(v, v);
      G::template rot<0x128>(v);
      G::template rot<0x124>(v);
      G::template rot<0x122>(v);
      G::template rot<0x121>(v);
      if ((lane & 31) == 0) {
        const double *p = reinterpret_cast<const double *>(&v);
#pragma unroll
        for (int i = 0; i < H; ++i) xch[buf][lane >> 5][i][wave] = p[i];
      }
      lds_barrier();
      {
        double *p = reinterpret_cast<double *>(&v);
#pragma unroll
        for (int i = 0; i < H; ++i) p[i] = xch[buf][lane >> 5][i][lane & (NW - 1)];
      }
      G::template rot<0xB1>(v);
      G::template rot<0x4E>(v);
      G::template rot<0x124>(v);
      buf ^= 1;
      const Rl yk = P::racc_value(v);
      if (wave == 0 && (lane & 31) == 0 && k < n) P::store_real(y + k + (size_t)(lane >> 5) * n, 2 * (size_t)n, yk);
      const C c = G::spread(yk);
#pragma unroll
      for (int r = 0; r < RPT; ++r) P::upd(bv[r], c, q[t][r]);
      fetch(k + RING, q[t]);
    });
  }
}

}  // namespace mgsq
