// Small least-squares systems [A_s b_s], one workgroup each: batches of
// independent systems (the many paths of a homotopy, Section 2; the data
// stays on the card between them, Section 7) and single systems of at most
// 64 rows.
//
// Per system the operations are those of Figure 1 (Section 3) on the
// augmented matrix of Equation (1): column j receives the projections
// k = 1, ..., j-1 in order, then its norm r_jj; then the back substitution
// of Section 6, Figure 3 on y = the projections of b.  The projections are
// made with u_k, column k after its last one, before its normalisation:
//   r_kj = (u_k^H a_j) / r_kk,   a_j -= ((u_k^H a_j) / ||u_k||^2) u_k,
// equal to q_k^H a_j and r_kj q_k in exact arithmetic; the inner products
// and ||u_k||^2 come out of one sum, so the chain from column to column has
// one sum and one division and neither square root nor normalisation (one
// 32 x 32 system: double 41 -> 34 us, dd 80 -> 69 us).  qd, and dd past 32
// rows, use q_k itself (there the second reciprocal's registers and products
// cost more than the shorter chain gives: qd 453 against 502 us).  A u_k far
// from 1 is divided by a power of two, so that products with it have the
// range of products with q_k.
//
// A wave is a grid of 16 row groups x 4 columns (32 x 2 or 64 x 1 for few
// columns of many rows): lane 4 g + c holds rows g, g + 16, ... (RPL of them)
// of one column per slot, so that a wave works on 4 columns at a time with
// every lane busy (a column per wave left half the lanes idle at 32 rows) and
// an inner product is summed over only 16 lanes.  The columns are dealt from
// the last one (b) on, 4 per wave and slot, so that the slots empty from the
// top as k grows; column 1, which never receives a projection, has no slot.
// Sums: the two halves of the wave exchange so that one half carries on with
// the real and one with the imaginary part, the odd and even rows of 16 lanes
// likewise with two slots or with the norm (permlane32_swap /
// permlane16_swap), then two rotations within a row: 5 merges of real
// accumulators for two complex sums (6 + 6 each way in a scan of 64 lanes).
// The tree of a sum and every later operation is the same whatever the wave
// count and the slot, and the lane grid goes by the system's own size, so a
// system's results do not depend on the batch.
//
// One wave per system (NW = 1, large batches) needs no synchronisation at
// all.  With several waves (a short chain for few systems) u_k passes
// through a ring in LDS: the owner of column k+1 applies u_k to that slot
// first and publishes u_{k+1}, and only then goes on with its other slots;
// the ring's entry is reused when every wave has read it.  The first wave,
// whose columns are the last to be due, normalises: Q and R's diagonal.
// Every wait is bounded by a wall-clock limit (MGS_INFO_SYNC_TIMEOUT in
// info).
#pragma once
#include "../../include/mgsqr.h"
#include "resident_kernels.hpp"

namespace mgsq {

constexpr int BAT_MAX_ROWS = 64;
constexpr int BAT_MAX_COLS = 64;          // columns of [A b]
constexpr size_t BAT_LDS_BYTES = 160 * 1024 - 1024;  // bound on 16 L m n, the size limit of the entry points

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

// Whether the projections are made with the unnormalised u_k.  It takes the
// square root and the normalisation off the chain, for one multiplication of
// each sum and registers for both reciprocals.
template <class P, int RPL>
constexpr bool bat_unnormalised() {
  return P::L <= 2 && P::L * RPL <= 4;
}

// A lane grid of CG columns, RPL rows per lane (m <= 64 / CG RPL), SL slots
// (columns 2, 3, ... of [A b]: at most CG NW SL), NW waves, at least WPE waves
// per SIMD (the register budget).
template <class P, int RPL, int SL, int NW, int WPE, int CG>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(WPE))) void mgs_batched_kernel(BatArgs a) {
  using C = typename P::C;
  using Acc = typename P::Acc;
  using Rl = typename P::R;
  using G = GridSum<P>;
  constexpr int L = P::L, NP = 2 * L;       // limbs, planes of a complex element
  constexpr int RG = 64 / CG;               // row groups
  constexpr int MP = RG * RPL;              // padded rows
  constexpr int STEP = CG * NW;             // columns per slot
  constexpr int RING = NW == 1 ? 2 : 8;     // u vectors kept
  constexpr bool UF = bat_unnormalised<P, RPL>();  // u_k is column k unnormalised
  constexpr bool LATE = UF && NW > 1;       // R and y are divided by r_kk at the end
  __shared__ double us[RING][NP][MP];       // u_c in entry c mod RING
  __shared__ double ys[NP][BAT_MAX_COLS];   // y (NW > 1: over 1 / r_kk until the end)
  __shared__ double invs[L][LATE ? BAT_MAX_COLS : 1];  // 1 / r_kk
  __shared__ double ups[UF ? BAT_MAX_COLS : 1];  // what u_k (last: b) was divided by
  __shared__ int far;                       // one of them is not 1
  __shared__ int pub;                       // u vectors published
  __shared__ int done[NW];                  // u vectors each wave has read
  __shared__ int status;                    // this system's info
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cg = lane & (CG - 1), rg = lane / CG;
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
    pub = 1;
    if constexpr (UF) far = 0;
  }
  if (tid < NW) done[tid] = 0;
  const int first = last - (CG * w + cg);  // this lane's column in slot 0; slot s: first - STEP s
  auto load_col = [&](int j, C (&v)[RPL]) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      const int i = rg + RG * r;
      v[r] = P::czero();
      if (i < m && j >= 0) {
        if (j < n)
          v[r] = P::load(A + (size_t)j * a.lda + i, planeA);
        else
          v[r] = P::load(a.b + (size_t)sys * NP * m + i, (size_t)m);
      }
    }
  };
  bool wide = true;  // some ups is not 1
  auto put_u = [&](int c, const C (&v)[RPL]) __attribute__((always_inline)) {
    double *dst = &us[c & (RING - 1)][0][0];
#pragma unroll
    for (int r = 0; r < RPL; ++r) P::store(dst + rg + RG * r, (size_t)MP, v[r]);
    if constexpr (UF) {
      // (rare; in LDS, so that it costs the others no registers)
      if (wide && ups[c] != 1.0) {
        const double f = pow2_inverse(ups[c]);
#pragma unroll 1
        for (int i = 0; i < NP * RPL; ++i) dst[rg + RG * i] *= f;
      }
    }
  };
  // The power of two of column j (ups): that of its largest entry when that
  // is not within 2^-64 .. 2^64, else 1.  u_j is divided by it when it is
  // published, so that 1 / ||u||^2 and u^H a are in range wherever those of
  // q_j are; the columns themselves stay as they are.  b, which is never
  // published, is itself brought within 2^768, and out of the subnormal
  // range: exact but for entries 2^1700 below its largest.  An infinity or a
  // NaN stays one; the bound keeps both powers normal numbers.
  auto range = [&](int j, C (&v)[RPL]) __attribute__((always_inline)) {
    if constexpr (UF) {
      double t[NP], big = 0.0;
#pragma unroll
      for (int r = 0; r < RPL; ++r) {
        P::store(t, 1, v[r]);
        big = fmax(big, fmax(fabs(t[0]), fabs(t[1])));
      }
      const double hi = j == n ? 0x1p800 : 0x1p64, lo = j == n ? 0x1p-800 : 0x1p-64;
      auto out = [&](double v) __attribute__((always_inline)) { return v >= hi || (v > 0.0 && v <= lo); };
      double f = 1.0;
      if (__any(out(big))) {
#pragma unroll
        for (int k = CG; k < 64; k *= 2) big = fmax(big, __shfl_xor(big, k));
        int e = out(big) && big < INFINITY ? ilogb(big) : 0;
        if (j == n && e > 0) e -= 767;
        e = e > 1000 ? 1000 : (e < -1000 ? -1000 : e);
        f = ldexp(1.0, e);
        if (j == n && e != 0) {
#pragma unroll
          for (int r = 0; r < RPL; ++r) {
            P::store(t, 1, v[r]);
#pragma unroll
            for (int i = 0; i < NP; ++i) t[i] *= pow2_inverse(f);
            v[r] = P::load(t, 1);
          }
        }
        if (j >= 0 && j < n && e != 0) far = 1;
      }
      if (rg == 0 && j >= 0) ups[j] = f;
    }
  };
  C col[SL][RPL];
  static_for<SL>([&](auto sI) __attribute__((always_inline)) {
    constexpr int s = decltype(sI)::value;
    const int j = first - STEP * s;
    load_col(j >= 1 ? j : -1, col[s]);
  });
  static_for<SL>([&](auto sI) __attribute__((always_inline)) {
    constexpr int s = decltype(sI)::value;
    const int j = first - STEP * s;
    range(j >= 1 ? j : -1, col[s]);
  });
  C u[RPL];
  Rl s2, rkk, inv;  // ||u_k||^2, its root, 1 over that
  // Q's column c and R's diagonal from u (unnormalised) in lane group g1
  auto normalise = [&](int c, int g1, C (&v)[RPL]) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
      const int i = rg + RG * r;
      v[r] = P::scale(v[r], inv);
      if (cg == g1 && i < m) P::store(Q + (size_t)c * a.ldq + i, planeQ, v[r]);
    }
    if (rg == 0 && cg == g1) {
      double t[L];
      P::store_real(t, 1, s2);
      bool ok = P::ok_norm(s2);
      double n2 = 0.0;  // ||a_c||^2
      if constexpr (UF) {
        n2 = t[0] * ups[c] * ups[c];
        ok = ok && n2 < INFINITY && n2 > 0.0;
      }
      if (!ok) atomicCAS(&status, 0, c + 1);
      if constexpr (LATE) P::store_real(&invs[0][c], BAT_MAX_COLS, inv);
      // (a refused column's r_cc is not a pivot: later calls with R refuse it too)
      P::store_real(t, 1, rkk);
      if (UF && !ok) t[0] = n2;
#pragma unroll
      for (int i = 0; i < L; ++i) {
        double *p = R + (size_t)c * a.ldr + c + (size_t)(2 * i) * planeR;
        p[0] = UF && ok ? t[i] * ups[c] : t[i];
        p[planeR] = 0.0;
      }
    }
  };
  auto norm = [&](const C (&v)[RPL]) __attribute__((always_inline)) {
    Acc t;
    P::acc_zero(t);
#pragma unroll
    for (int r = 0; r < RPL; ++r) P::acc_abs2(t, v[r]);
    return t;
  };
  if (w == 0) {
    load_col(0, u);
    range(cg == 0 ? 0 : -1, u);
    if constexpr (UF) lds_wait();  // ups[0], of one lane, for all
    if constexpr (!UF) {
      s2 = G::template real_sum<CG>(norm(u));
      root_and_inverse<P>(s2, rkk, inv);
      normalise(0, 0, u);
    }
    if (cg == 0) put_u(0, u);
  }
  __syncthreads();
  if constexpr (UF) wide = __builtin_amdgcn_readfirstlane(far) != 0;

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
  auto dot = [&](const C (&v)[RPL]) __attribute__((always_inline)) {
    Acc t;
    P::acc_zero(t);
#pragma unroll
    for (int r = 0; r < RPL; ++r) P::acc_cmulc(t, u[r], v[r]);
    return t;
  };
  // r_kj of column j (this lane's part: the upper half's is the imaginary
  // one) to R, or to y for b; one lane per column and part stores.  With
  // several waves it is u_k^H a_j, to be divided by r_kk at the end: the
  // square root stays off the chain.
  auto store_r = [&](int k, int j, const Rl &v) __attribute__((always_inline)) {
    if ((lane & 15) < CG && j > k) {
      double t[L];
      P::store_real(t, 1, v);
      const int part = lane >> 5;
      if (j < n) {
        double *p = R + (size_t)j * a.ldr + k + part * planeR;
#pragma unroll
        for (int i = 0; i < L; ++i) p[(size_t)(2 * i) * planeR] = t[i];
      } else {
#pragma unroll
        for (int i = 0; i < L; ++i) {
          ys[2 * i + part][k] = t[i];
          if (!UF && y != nullptr) y[k + (size_t)(2 * i + part) * n] = t[i];
        }
      }
    }
  };
  auto update = [&](int k, int j, const Rl &t, C (&v)[RPL]) __attribute__((always_inline)) {
    const C c = G::spread(t);
    if (j > k) {
#pragma unroll
      for (int r = 0; r < RPL; ++r) P::upd(v[r], c, u[r]);
    }
  };
  // Column c, in slot s1 and lane group g1 of this wave, to the ring.
  auto publish = [&](int c, int s1, int g1) __attribute__((always_inline)) {
    C v[RPL];
    static_for<SL>([&](auto sI) __attribute__((always_inline)) {
      constexpr int s = decltype(sI)::value;
      if (s == s1) {
#pragma unroll
        for (int r = 0; r < RPL; ++r) v[r] = col[s][r];
      }
    });
    if constexpr (!UF) {
      s2 = G::template real_sum<CG>(norm(v));
      root_and_inverse<P>(s2, rkk, inv);
      normalise(c, g1, v);
    }
    if constexpr (NW > 1) {
      // the entry is free once every wave has read u_{c - RING}
      if (c >= RING)
        alive = wait_for([&]() __attribute__((always_inline)) {
          int lo = c;
#pragma unroll
          for (int i = 0; i < NW; ++i)
            lo = min(lo, __hip_atomic_load(&done[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
          return lo > c - RING;
        });
    }
    if (cg == g1) put_u(c, v);
    lds_wait();
    if (NW > 1 && lane == 0) __hip_atomic_store(&pub, c + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };

  // One instruction word, so that the loop's 8-byte instructions fall on other
  // fetch lines: 10,000 dd 32 x 32 systems 1062 -> 1047 us, one double 36.4 ->
  // 36.0.
  if constexpr (UF) asm volatile("s_nop 0");
  bool mine = false;  // u_k was published by this wave
  for (int k = 0; k < n; ++k) {
    // slots holding a column past k: the largest column of slot s is
    // last - 4 w - STEP s; the first wave goes on to normalise
    const int above = last - CG * w - k;
    if (above <= 0 && (!UF || w > 0)) break;
    const int nact = above > 0 ? (above + STEP - 1) / STEP : 0;
    res_jitter(a.jitter, (unsigned)k);
    if constexpr (NW > 1) {
      if (!mine && !wait_for([&]() __attribute__((always_inline)) {
            return __hip_atomic_load(&pub, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > k;
          })) {
        alive = false;
        break;
      }
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int r = 0; r < RPL; ++r) u[r] = P::load(&us[k & (RING - 1)][0][rg + RG * r], (size_t)MP);
    if constexpr (NW > 1) {
      lds_wait();
      if (lane == 0) __hip_atomic_store(&done[w], k + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    // position of column k + 1 among the slots (its slot, wave and group)
    const int pos = last - (k + 1);
    const int s1 = pos / STEP, g1 = pos & (CG - 1);
    const bool own = k + 1 < n && (pos - s1 * STEP) / CG == w;
    mine = own;
    if constexpr (NW == 1) {
      Rl iw;
      if constexpr (UF) {
        s2 = G::template real_sum<CG>(norm(u));
        iw = P::recip(s2);
        root_and_inverse<P>(s2, rkk, inv);
      }
      auto times = [&](const Rl &v, const Rl &f) __attribute__((always_inline)) { return UF ? P::rmul(v, f) : v; };
      static_for<SL / 2>([&](auto pI) __attribute__((always_inline)) {
        constexpr int s = 2 * decltype(pI)::value;
        const int j0 = first - STEP * s, j1 = first - STEP * (s + 1);
        if (s + 1 < nact) {
          const Rl v = G::template sum2<CG>(dot(col[s]), dot(col[s + 1]));
          store_r(k, (lane >> 4) & 1 ? j1 : j0, times(v, inv));
          Rl t0 = times(v, iw), t1;
          G::unpack16(t0, t1);
          update(k, j0, t0, col[s]);
          update(k, j1, t1, col[s + 1]);
        } else if (s < nact) {
          const Rl v = G::template sum<CG>(dot(col[s]));
          if (((lane >> 4) & 1) == 0) store_r(k, j0, times(v, inv));
          update(k, j0, times(v, iw), col[s]);
        }
      });
      if (own) publish(k + 1, s1, g1);
    } else {
      // the slot of the next column first, then its publication
      Rl iw;
      if (nact > 0) {
        const int sf = own ? s1 : 0;
        Rl vf;
        static_for<SL>([&](auto sI) __attribute__((always_inline)) {
          constexpr int s = decltype(sI)::value;
          if (s == sf) {
            if constexpr (UF) {
              vf = G::template sum_and_real<CG>(dot(col[s]), norm(u), s2);
              iw = P::recip(s2);
              update(k, first - STEP * s, P::rmul(vf, iw), col[s]);
            } else {
              vf = G::template sum<CG>(dot(col[s]));
              update(k, first - STEP * s, vf, col[s]);
            }
          }
        });
        if (own) publish(k + 1, s1, g1);
        if (((lane >> 4) & 1) == 0) store_r(k, first - STEP * sf, vf);
        static_for<SL>([&](auto sI) __attribute__((always_inline)) {
          constexpr int s = decltype(sI)::value;
          if (s < nact && s != sf) {
            const Rl v = G::template sum<CG>(dot(col[s]));
            update(k, first - STEP * s, UF ? P::rmul(v, iw) : v, col[s]);
            if (((lane >> 4) & 1) == 0) store_r(k, first - STEP * s, v);
          }
        });
      } else if constexpr (UF) {
        s2 = G::template real_sum<CG>(norm(u));
      }
      if constexpr (UF) {
        if (w == 0) root_and_inverse<P>(s2, rkk, inv);
      }
    }
    // u_k in every lane group: the first wave normalises column k
    if constexpr (UF) {
      if (w == 0) normalise(k, 0, u);
    }
    if (!alive) break;
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
    const Rl s2 = G::template real_sum<CG>(t);
    if (lane == 0) {
      double t2[L];
      P::store_real(t2, 1, P::ok_norm(s2) ? P::sqrt_(s2) : P::rzero());
#pragma unroll
      for (int i = 0; i < L; ++i) a.rho[(size_t)sys * L + i] = (UF ? t2[i] * ups[n] : t2[i]);
    }
  }
  // R below its diagonal: zeros.  Above it, and in y, what is still missing:
  // 1 / r_kk, and the power of two of b.
  auto late = [&](int k, const C &v) __attribute__((always_inline)) {
    Rl f;
    double *pf = reinterpret_cast<double *>(&f);
    if constexpr (LATE) {
#pragma unroll
      for (int i = 0; i < L; ++i) pf[i] = invs[i][k];
      return P::scale(v, f);
    }
    return v;
  };
  if constexpr (UF) __syncthreads();
  for (int j = w; j < n; j += NW) {
    if (lane >= n) continue;
    double *p = R + (size_t)j * a.ldr + lane;
    if (lane > j) P::store(p, planeR, P::czero());
    if constexpr (LATE) {
      if (lane < j) P::store(p, planeR, late(lane, P::load(p, planeR)));
    }
  }
  if constexpr (UF) {
    if (w == 0 && last == n && lane < n) {
      double t[NP];
      P::store(t, 1, late(lane, P::load(&ys[0][lane], (size_t)BAT_MAX_COLS)));
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        t[i] *= ups[n];
        ys[i][lane] = t[i];
        if (y != nullptr) y[lane + (size_t)i * n] = t[i];
      }
    }
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
  inv = P::recip(P::load(R + (size_t)jl * a.ldr + jl, planeR).re);
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
