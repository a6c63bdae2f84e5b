// Small least-squares systems [A_s b_s], one workgroup each: batches of
// independent systems (the many paths of a homotopy, Section 2; the data
// stays on the card between them, Section 7) and single systems of at most
// 64 rows.
//
// Per system the operations are those of Figure 1 (Section 3) on the
// augmented matrix of Equation (1): column j receives the projections
// k = 1, ..., j-1 in order, then its norm r_jj and q_j = a_j / r_jj; then
// the back substitution of Section 6, Figure 3 on y = the projections of b.
//
// A wave is a grid of 16 row groups x 4 columns: lane 4 g + c holds rows
// g, g + 16, ... (RPL of them) of one column per slot, so that a wave works
// on 4 columns at a time with every lane busy (a column per wave left half
// the lanes idle at 32 rows) and an inner product is summed over only 16
// lanes.  The columns are dealt from the last one (b) on, 4 per wave and
// slot, so that the slots empty from the top as k grows; column 1, which
// never receives a projection, has no slot.  Sums: the two halves of the
// wave exchange so that one half carries on with the real and one with the
// imaginary part, the odd and even rows of 16 lanes likewise with two slots
// (permlane32_swap / permlane16_swap), then two rotations within a row: 5
// merges of real accumulators for two complex sums (6 + 6 each way in a scan
// of 64 lanes).  The tree of an inner product is the same whatever the wave
// count and the slot, so a system's results do not depend on the shape.
//
// One wave per system (NW = 1, large batches) needs no synchronisation at
// all.  With several waves (a short chain for few systems) q_k passes
// through a ring in LDS: the owner of column k+1 applies q_k to that column
// first, normalises and publishes it, and only then applies q_k to its other
// slots; the ring's entry is reused when every wave has read it.  Every
// wait is bounded by a wall-clock limit (MGS_INFO_SYNC_TIMEOUT in info).
#pragma once
#include "../../include/mgsqr.h"
#include "resident_kernels.hpp"

namespace mgsq {

constexpr int BAT_MAX_ROWS = 64;
constexpr int BAT_MAX_COLS = 64;          // columns of [A b]
constexpr size_t BAT_LDS_BYTES = 160 * 1024 - 1024;  // bound on 16 L m n, the size limit of the entry points
constexpr int BAT_CG = 4;                 // columns of a wave's lane grid
constexpr int BAT_RG = 64 / BAT_CG;       // row groups

struct BatArgs {
  int batch, m, n, ncols;  // ncols = n + 1 when b is given
  const double *A;         // [batch][L][2][n][lda]
  int lda;
  const double *b;  // [batch][L][2][m] or null
  double *Q;        // [batch][L][2][n][ldq]
  int ldq;
  double *R;  // [batch][L][2][n][ldr]
  int ldr;
  double *y;    // [batch][L][2][n] or null: the projections of b
  double *x;    // [batch][L][2][n] or null: R^{-1} y (b given)
  double *rho;  // [batch][L] or null
  int *info;    // [batch]
  long long spin_ticks;
  unsigned jitter;  // race checks: seed of the timing jitter (0: none)
};

// a's upper half of the wave against b's lower half: a = [a.lo, b.lo],
// b = [a.hi, b.hi].
__device__ __forceinline__ void lane_swap32(double &a, double &b) {
  const unsigned long long ua = __double_as_longlong(a), ub = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
  a = __longlong_as_double(((unsigned long long)hi[0] << 32) | lo[0]);
  b = __longlong_as_double(((unsigned long long)hi[1] << 32) | lo[1]);
}
// The same for a's odd rows of 16 lanes against b's even rows.
__device__ __forceinline__ void lane_swap16(double &a, double &b) {
  const unsigned long long ua = __double_as_longlong(a), ub = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
  a = __longlong_as_double(((unsigned long long)hi[0] << 32) | lo[0]);
  b = __longlong_as_double(((unsigned long long)hi[1] << 32) | lo[1]);
}

// Sums over the row groups of a wave's lane grid.
template <class P>
struct GridSum {
  using Acc = typename P::Acc;
  using RAcc = typename P::RAcc;
  using Rl = typename P::R;
  using C = typename P::C;
  static constexpr int H = sizeof(RAcc) / sizeof(double), L = P::L;

  // a and b folded over the halves (16: over the row pairs): a in the lower
  // half (even rows), b in the upper half (odd rows).
  __device__ static __forceinline__ RAcc fold32(RAcc a, RAcc b) {
    double *pa = reinterpret_cast<double *>(&a), *pb = reinterpret_cast<double *>(&b);
#pragma unroll
    for (int i = 0; i < H; ++i) lane_swap32(pa[i], pb[i]);
    P::racc_merge(a, b);
    return a;
  }
  __device__ static __forceinline__ RAcc fold16(RAcc a, RAcc b) {
    double *pa = reinterpret_cast<double *>(&a), *pb = reinterpret_cast<double *>(&b);
#pragma unroll
    for (int i = 0; i < H; ++i) lane_swap16(pa[i], pb[i]);
    P::racc_merge(a, b);
    return a;
  }
  // The rest of the sum, within rows of 16 lanes (4 row groups).
  __device__ static __forceinline__ Rl finish(RAcc v) {
    rot<0x128>(v);  // row_ror:8
    rot<0x124>(v);  // row_ror:4
    return P::racc_value(v);
  }
  template <int CTRL>
  __device__ static __forceinline__ void rot(RAcc &v) {
    RAcc o;
    double *po = reinterpret_cast<double *>(&o);
    const double *pv = reinterpret_cast<const double *>(&v);
#pragma unroll
    for (int i = 0; i < H; ++i) po[i] = dpp_shift<CTRL, 0xf>(pv[i]);
    P::racc_merge(v, o);
  }
  // v of the lower half in re, of the upper half in im, in every lane.
  __device__ static __forceinline__ C spread(const Rl &v) {
    C c;
    c.re = v;
    c.im = v;
    double *pr = reinterpret_cast<double *>(&c.re), *pi = reinterpret_cast<double *>(&c.im);
#pragma unroll
    for (int i = 0; i < L; ++i) lane_swap32(pr[i], pi[i]);
    return c;
  }
  __device__ static __forceinline__ const RAcc *parts(const Acc &t) { return reinterpret_cast<const RAcc *>(&t); }

  __device__ static __forceinline__ Rl real_sum(const Acc &t) {
    RAcc u = parts(t)[0];
    u = fold32(u, u);
    return finish(fold16(u, u));
  }
  __device__ static __forceinline__ C sum(const Acc &t) {
    const RAcc u = fold32(parts(t)[0], parts(t)[1]);
    return spread(finish(fold16(u, u)));
  }
  __device__ static __forceinline__ void sum2(const Acc &t0, const Acc &t1, C &c0, C &c1) {
    Rl v0 = finish(fold16(fold32(parts(t0)[0], parts(t0)[1]), fold32(parts(t1)[0], parts(t1)[1]))), v1 = v0;
    double *p0 = reinterpret_cast<double *>(&v0), *p1 = reinterpret_cast<double *>(&v1);
#pragma unroll
    for (int i = 0; i < L; ++i) lane_swap16(p0[i], p1[i]);
    c0 = spread(v0);
    c1 = spread(v1);
  }
};

// RPL rows per lane (m <= 16 RPL), SL slots (columns 2, 3, ... of [A b]: at
// most 4 NW SL), NW waves, at least WPE waves per SIMD (the register
// budget).
template <class P, int RPL, int SL, int NW, int WPE>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(WPE))) void mgs_batched_kernel(BatArgs a) {
  using C = typename P::C;
  using Acc = typename P::Acc;
  using Rl = typename P::R;
  using G = GridSum<P>;
  constexpr int NP = 2 * P::L;              // planes of a complex element
  constexpr int MP = BAT_RG * RPL;          // padded rows
  constexpr int STEP = BAT_CG * NW;         // columns per slot
  constexpr int RING = NW == 1 ? 2 : 8;     // q vectors kept
  __shared__ double qs[RING][NP][MP];       // q_c in entry c mod RING
  __shared__ double ys[NP][BAT_MAX_COLS];   // y
  __shared__ int pub;                       // q vectors published
  __shared__ int done[NW];                  // q vectors each wave has read
  __shared__ int status;                    // this system's info
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int cg = lane & (BAT_CG - 1), rg = lane / BAT_CG;
  const int sys = blockIdx.x;
  const int m = a.m, n = a.n, last = a.ncols - 1;
  const size_t planeA = (size_t)a.lda * n, planeQ = (size_t)a.ldq * n, planeR = (size_t)a.ldr * n;
  const double *A = a.A + (size_t)sys * NP * planeA;
  double *Q = a.Q + (size_t)sys * NP * planeQ;
  double *R = a.R + (size_t)sys * NP * planeR;
  double *x = a.x != nullptr ? a.x + (size_t)sys * NP * n : nullptr;
  double *y = a.y != nullptr ? a.y + (size_t)sys * NP * n : nullptr;
  if (tid == 0) {
    status = 0;
    pub = 0;
  }
  if (tid < NW) done[tid] = 0;
  const int first = last - (BAT_CG * w + cg);  // this lane's column in slot 0; slot s: first - STEP s
  auto load_col = [&](int j, C (&v)[RPL]) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      const int i = rg + BAT_RG * r;
      v[r] = P::czero();
      if (i < m && j >= 0) {
        if (j < n)
          v[r] = P::load(A + (size_t)j * a.lda + i, planeA);
        else
          v[r] = P::load(a.b + (size_t)sys * NP * m + i, (size_t)m);
      }
    }
  };
  C col[SL][RPL];
  static_for<SL>([&](auto sI) __attribute__((always_inline)) {
    constexpr int s = decltype(sI)::value;
    const int j = first - STEP * s;
    load_col(j >= 1 ? j : -1, col[s]);
  });
  C q[RPL];
  if (w == 0) load_col(0, q);
  __syncthreads();

  bool alive = true;
  // Bounded wait for `ready()`; false (and the status) on a time-out.
  auto wait_for = [&](auto ready) __attribute__((always_inline)) {
    PollBound poll;
    while (!ready()) {
      if (poll.due() && poll.late(a.spin_ticks)) {
        if (lane == 0) atomicExch(&status, MGS_INFO_SYNC_TIMEOUT);
        return false;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    return true;
  };
  // r_cc = ||v||, q_c = v / r_cc for column c in lane group gc of this wave
  // (every group computes, group gc stores): Q, the ring, R(c, c).
  auto normalise = [&](int c, int gc, C (&v)[RPL]) __attribute__((always_inline)) {
    Acc t;
    P::acc_zero(t);
#pragma unroll
    for (int r = 0; r < RPL; ++r) P::acc_abs2(t, v[r]);
    const Rl s2 = G::real_sum(t);
    Rl rkk, inv;
    root_and_inverse<P>(s2, rkk, inv);
#pragma unroll
    for (int r = 0; r < RPL; ++r) v[r] = P::scale(v[r], inv);
    if constexpr (NW > 1) {
      // the ring's entry is free once every wave has read q_{c - RING}
      if (alive && c >= RING)
        alive = wait_for([&]() __attribute__((always_inline)) {
          int lo = c;
#pragma unroll
          for (int i = 0; i < NW; ++i)
            lo = min(lo, __hip_atomic_load(&done[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
          return lo > c - RING;
        });
    }
    if (cg == gc) {
      double *dst = &qs[c & (RING - 1)][0][0];
#pragma unroll
      for (int r = 0; r < RPL; ++r) {
        const int i = rg + BAT_RG * r;
        P::store(dst + i, (size_t)MP, v[r]);
        if (i < m) P::store(Q + (size_t)c * a.ldq + i, planeQ, v[r]);
      }
      if (rg == 0) {
        if (!P::ok_norm(s2)) atomicCAS(&status, 0, c + 1);
        C d;
        d.re = rkk;
        d.im = P::rzero();
        P::store(R + (size_t)c * a.ldr + c, planeR, d);
      }
    }
    lds_wait();
    if (NW > 1 && lane == 0) __hip_atomic_store(&pub, c + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto dot = [&](const C (&v)[RPL]) __attribute__((always_inline)) {
    Acc t;
    P::acc_zero(t);
#pragma unroll
    for (int r = 0; r < RPL; ++r) P::acc_cmulc(t, q[r], v[r]);
    return t;
  };
  // r_kj of column j to R (to y for b), a_j -= r_kj q_k.
  auto update = [&](int k, int j, const C &rk, C (&v)[RPL]) __attribute__((always_inline)) {
    if (j > k) {
      if (rg == 0) {
        if (j < n)
          P::store(R + (size_t)j * a.ldr + k, planeR, rk);
        else {
          P::store(&ys[0][k], (size_t)BAT_MAX_COLS, rk);
          if (y != nullptr) P::store(y + k, (size_t)n, rk);
        }
      }
#pragma unroll
      for (int r = 0; r < RPL; ++r) P::upd(v[r], rk, q[r]);
    }
  };

  if (w == 0) normalise(0, 0, q);
  for (int k = 0; k < n; ++k) {
    // slots holding a column past k: the largest column of slot s is
    // last - 4 w - STEP s
    const int above = last - BAT_CG * w - k;
    if (above <= 0) break;
    const int nact = (above + STEP - 1) / STEP;
    res_jitter(a.jitter, (unsigned)k);
    if constexpr (NW > 1) {
      if (!wait_for([&]() __attribute__((always_inline)) {
            return __hip_atomic_load(&pub, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > k;
          })) {
        alive = false;
        break;
      }
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int r = 0; r < RPL; ++r) q[r] = P::load(&qs[k & (RING - 1)][0][rg + BAT_RG * r], (size_t)MP);
    if constexpr (NW > 1) {
      lds_wait();
      if (lane == 0) __hip_atomic_store(&done[w], k + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    // position of column k + 1 among the slots (its slot, wave and group)
    const int pos = last - (k + 1);
    const int s1 = pos / STEP, w1 = (pos - s1 * STEP) / BAT_CG, g1 = pos & (BAT_CG - 1);
    const bool own = k + 1 < n && w1 == w;
    if constexpr (NW == 1) {
      static_for<SL / 2>([&](auto pI) __attribute__((always_inline)) {
        constexpr int s = 2 * decltype(pI)::value;
        if (s + 1 < nact) {
          C r0, r1;
          G::sum2(dot(col[s]), dot(col[s + 1]), r0, r1);
          update(k, first - STEP * s, r0, col[s]);
          update(k, first - STEP * (s + 1), r1, col[s + 1]);
        } else if (s < nact) {
          update(k, first - STEP * s, G::sum(dot(col[s])), col[s]);
        }
      });
      if (own) {
        static_for<SL>([&](auto sI) __attribute__((always_inline)) {
          constexpr int s = decltype(sI)::value;
          if (s == s1) {
#pragma unroll
            for (int r = 0; r < RPL; ++r) q[r] = col[s][r];
          }
        });
        normalise(k + 1, g1, q);
      }
    } else {
      // the next column first: its projection, its norm, its publication
      C qk[RPL];
#pragma unroll
      for (int r = 0; r < RPL; ++r) qk[r] = q[r];
#pragma unroll 1
      for (int pass = own ? 0 : 1; pass < 2; ++pass) {
        static_for<SL>([&](auto sI) __attribute__((always_inline)) {
          constexpr int s = decltype(sI)::value;
          if (s < nact && (pass == 0 ? s == s1 : !(own && s == s1)))
            update(k, first - STEP * s, G::sum(dot(col[s])), col[s]);
        });
        if (pass == 0) {
          static_for<SL>([&](auto sI) __attribute__((always_inline)) {
            constexpr int s = decltype(sI)::value;
            if (s == s1) {
#pragma unroll
              for (int r = 0; r < RPL; ++r) q[r] = col[s][r];
            }
          });
          normalise(k + 1, g1, q);
          if (!alive) break;
#pragma unroll
          for (int r = 0; r < RPL; ++r) q[r] = qk[r];
        }
      }
      if (!alive) break;
    }
  }
  if constexpr (NW > 1) {
    if (lane == 0) __hip_atomic_store(&done[w], BAT_MAX_COLS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  // rho = ||b - Q y|| (Equation (1)): b is the first column of wave 0.
  if (a.rho != nullptr && a.ncols > n && w == 0) {
    Acc t;
    P::acc_zero(t);
#pragma unroll
    for (int r = 0; r < RPL; ++r) P::acc_abs2(t, col[0][r]);
    const Rl s2 = G::real_sum(t);
    if (lane == 0) P::store_real(a.rho + (size_t)sys * P::L, 1, P::ok_norm(s2) ? P::sqrt_(s2) : P::rzero());
  }
  // Zeros below the diagonal of R.
  for (int j = w; j < n; j += NW) {
    const int i = j + 1 + lane;
    if (i < n) P::store(R + (size_t)j * a.ldr + i, planeR, P::czero());
  }
  __syncthreads();
  const int bad = status;
  if (tid == 0) a.info[sys] = bad;
  if (a.ncols == n || x == nullptr || w != 0 || bad != 0) return;
  // Back substitution (Figure 3) by wave 0: lane j holds y_j and 1 / r_jj;
  // for k = n-1 .. 0, x_k = y_k / r_kk (times the reciprocal), then
  // y_j -= r_jk x_k for j < k (column k of R read coalesced, two ahead).
  const int jl = lane < n ? lane : n - 1;
  C yv = P::load(&ys[0][jl], (size_t)BAT_MAX_COLS);
  const Rl inv = P::recip(P::load(R + (size_t)jl * a.ldr + jl, planeR).re);
  auto rcol = [&](int k) __attribute__((always_inline)) {
    return P::load(R + (size_t)(k > 0 ? k : 0) * a.ldr + jl, planeR);
  };
  C rc = rcol(n - 1), rn = rcol(n - 2);
#pragma unroll 1
  for (int k = n - 1; k >= 0; --k) {
    const C r2 = rcol(k - 2);
    const C xk = wave_readlane(P::scale(yv, inv), k);
    if (lane == k) P::store(x + k, (size_t)n, xk);
    if (lane < k) P::upd(yv, rc, xk);
    rc = rn;
    rn = r2;
  }
}

}  // namespace mgsq
