// Newton's method for a polynomial system, all on the card (Section 7: the
// corrector of a path tracker solves thousands of linear systems; the
// system is transferred once, the evaluated Jacobian and system never leave
// the card).  Equation e of the system is
//   f_e(x) = sum_m c_em prod_t x_{v_emt}^{d_emt}
// (the workload of the paper's Table 6: 32 equations, 32 variables, 32
// monomials of 5 variables each).  One Newton step for a batch of points:
//   1. poly_eval_kernel: -f(x) and the Jacobian J(x) of every point, in the
//      layout of mgs_lstsq_batched (J column j = d f / d x_j; the same kernel
//      gives f itself to mgs_poly_eval);
//   2. the batched MGS on [J -f] and back substitution (batched_kernels.hpp):
//      the correction d, least-squares solution of J d = -f;
//   3. newton_update_kernel: x += d, and the FP64 norm of d.
#pragma once
#include "../../include/mgsqr.h"
#include "batched_kernels.hpp"

namespace mgsq {

constexpr int NT_MAX_MON = 64;   // monomials per equation (one lane each)
constexpr int NT_MAX_VARS = 63;  // variables (columns of [J -f] <= 64)
constexpr int NT_MAX_VPM = 8;    // variables per monomial
constexpr int NT_MAX_DEG = 16;   // exponent bound

// Powers x_j^d, d = 1..NT_TAB, kept per point; a higher one is a product of
// two or three of them.
constexpr int NT_TAB = 6;

template <class P>
__device__ __forceinline__ typename P::C nt_mul(const typename P::C &a, const typename P::C &b) {
  typename P::Acc acc;
  P::acc_zero(acc);
  P::acc_cmul(acc, a, b);
  return P::acc_value(acc);
}

// Dynamic LDS of poly_eval_kernel: the power table, then per wave the
// derivatives of its 64 lanes' monomials and a list of monomials per lane.
constexpr size_t nt_table_doubles(int L, int nvar) { return (size_t)2 * L * NT_TAB * nvar; }
constexpr size_t nt_wave_doubles(int L, int nvpm) { return (size_t)2 * L * 64 * nvpm + 64; }

// One workgroup evaluates neqb equations at one point; its waves take them
// HALF ? two at a time (nmon <= 32: a lane per monomial, an equation per half
// wave) : one at a time.  The powers of the point's variables are formed
// once per workgroup.  A lane forms its monomial c prod_t x_t^{d_t} and its
// derivatives c d_t x_t^{d_t - 1} prod_{u != t} x_u^{d_u} from suffix
// products (kept in the derivatives' places in LDS) and a running prefix
// product, so nothing but the current products is held in registers.  f_e is
// a sum over the lanes (fixed tree).  J(e, j) is summed by the lane of
// variable j in monomial order: every lane enters its monomial in the lists
// (bits in LDS) of its factors' variables, and all lanes walk their variable's
// lists at once.
// f_e (-f_e when negate) goes to b, J to A, both in the batched
// least-squares layout.
//
// Bound by the products: qd, 32 equations of 32 monomials of 5 variables at
// 1024 points took 3.1 ms with a power per factor, half the lanes idle and
// 1.7 KB of scratch per lane.  With a ballot per variable and factor in place
// of the lists in LDS (64 variables and 8 factors: 4000 instructions an
// equation) calls took 1.1 to 2.4 times as long (200 points, 63 variables, 64
// monomials of 8 factors: double 229 -> 97, dd 509 -> 264, qd 2285 -> 1841 us;
// 32 monomials of 5 factors: 33 -> 19, 45 -> 31, 256 -> 227).
template <class P, bool HALF>
__global__ __launch_bounds__(256) void poly_eval_kernel(int neq, int nvar, int nmon, int nvpm, const int *vars,
                                                        const int *exps, const double *coef, const double *x,
                                                        double *A, double *b, int neqb, bool negate) {
  using C = typename P::C;
  using Acc = typename P::Acc;
  using G = GridSum<P>;
  constexpr int NP = 2 * P::L, EQ = HALF ? 2 : 1, SEG = 64 / EQ;  // lanes per equation
  extern __shared__ double lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nwave = blockDim.x >> 6;
  const int s = blockIdx.y;
  const size_t tabp = (size_t)NT_TAB * nvar, dsp = (size_t)64 * nvpm;  // plane strides
  double *tab = lds;                                                      // [plane][d - 1][variable]
  double *ds = lds + nt_table_doubles(P::L, nvar) + wave * nt_wave_doubles(P::L, nvpm);  // [plane][lane * nvpm + t]
  unsigned long long *lists = reinterpret_cast<unsigned long long *>(ds + (size_t)2 * P::L * 64 * nvpm);  // [lane]
  const double *xp = x + (size_t)s * NP * nvar;
  if (tid < nvar) {
    const C v = P::load(xp + tid, (size_t)nvar);
    C p = v;
    P::store(tab + tid, tabp, p);
#pragma unroll 1
    for (int d = 2; d <= NT_TAB; ++d) {
      p = nt_mul<P>(p, v);
      P::store(tab + (size_t)(d - 1) * nvar + tid, tabp, p);
    }
  }
  __syncthreads();
  // x_v^d
  auto power = [&](int v, int d) __attribute__((always_inline)) {
    const int k = d < 1 ? 1 : (d > NT_TAB ? NT_TAB : d);
    C p = P::load(tab + (size_t)(k - 1) * nvar + v, tabp);
    if (d < 1) {
      p = P::czero();
      p.re = P::rone();
    }
#pragma unroll 1
    for (int i = d - NT_TAB; i > 0; i -= NT_TAB)
      p = nt_mul<P>(p, P::load(tab + (size_t)((i < NT_TAB ? i : NT_TAB) - 1) * nvar + v, tabp));
    return p;
  };
  const int seg = HALF ? lane >> 5 : 0, ml = lane & (SEG - 1);  // the lane's equation and monomial
  const int e1 = min(neq, (blockIdx.x + 1) * neqb);
#pragma unroll 1
  for (int e0 = blockIdx.x * neqb + wave * EQ; e0 < e1; e0 += nwave * EQ) {
    const int e = e0 + seg;
    const bool live = e < e1 && ml < nmon;
    const size_t base = live ? ((size_t)e * nmon + ml) * nvpm : 0;
    // the monomial's factors: indices and exponents outside their bounds are
    // clamped into them
    int vt[NT_MAX_VPM], dt[NT_MAX_VPM];
#pragma unroll
    for (int t = 0; t < NT_MAX_VPM; ++t) {
      vt[t] = -1;
      dt[t] = 0;
      if (t < nvpm) {
        const int v0 = vars[base + t], d0 = exps[base + t];
        vt[t] = v0 < 0 ? 0 : (v0 >= nvar ? nvar - 1 : v0);
        dt[t] = d0 < 0 ? 0 : (d0 > NT_MAX_DEG ? NT_MAX_DEG : d0);
      }
    }
    C pre = P::load(coef + (live ? (size_t)e * nmon + ml : 0), (size_t)neq * nmon);
    C suf = P::czero();
    suf.re = P::rone();
#pragma unroll
    for (int t = NT_MAX_VPM - 1; t >= 0; --t) {
      if (t < nvpm) {
        P::store(ds + lane * nvpm + t, dsp, suf);
        if (t > 0) {
          const C p = power(vt[t], dt[t]);
          suf = t == nvpm - 1 ? p : nt_mul<P>(p, suf);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < NT_MAX_VPM; ++t) {
      if (t < nvpm) {
        // (the exponent to the coefficient's side: d_t x_t^(d_t - 1) can overflow
        // where c d_t x_t^(d_t - 1) does not)
        C dv = nt_mul<P>(P::scale(pre, P::rfrom((double)dt[t])), power(vt[t], dt[t] - 1));
        if (t < nvpm - 1) dv = nt_mul<P>(dv, P::load(ds + lane * nvpm + t, dsp));
        if (dt[t] == 0) dv = P::czero();
        P::store(ds + lane * nvpm + t, dsp, dv);
        pre = nt_mul<P>(pre, power(vt[t], dt[t]));
      }
    }
    // f_e: the monomials of an equation, summed over its lanes; a lane without
    // one adds nothing, whatever the factors that it evaluated came to
    if (!live) pre = P::czero();
    Acc acc;
    P::acc_set(acc, pre);
    typename P::RAcc re = G::parts(acc)[0], im = G::parts(acc)[1];
    auto tree = [&](typename P::RAcc &v) __attribute__((always_inline)) {
      if constexpr (!HALF) v = G::fold32(v, v);
      v = G::fold16(v, v);
      G::template rot<0x128>(v);
      G::template rot<0x124>(v);
      G::template rot<0x122>(v);
      G::template rot<0x121>(v);
    };
    tree(re);
    tree(im);
    if (ml == 0 && e < e1) {
      C fe;
      fe.re = P::racc_value(re);
      fe.im = P::racc_value(im);
      P::store(b + (size_t)s * NP * neq + e, (size_t)neq, negate ? P::cneg(fe) : fe);
    }
    lds_wait();  // the derivatives of the other lanes
    // J(e, j): the lanes of an equation take SEG variables at a time
    const int slot = seg * SEG;
#pragma unroll 1
    for (int j0 = 0; j0 < nvar; j0 += SEG) {
      unsigned long long has[NT_MAX_VPM];  // monomials whose factor t is this lane's variable
      // (one list serves all factors: a wave's LDS operations run in order)
#pragma unroll
      for (int t = 0; t < NT_MAX_VPM; ++t) {
        has[t] = 0;
        if (t < nvpm) {
          const int j = vt[t] - j0;
          lists[lane] = 0;
          asm volatile("" ::: "memory");
          if (live && j >= 0 && j < SEG)
            __hip_atomic_fetch_or(&lists[slot + j], 1ull << ml, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          asm volatile("" ::: "memory");
          has[t] = lists[lane];
          asm volatile("" ::: "memory");
        }
      }
      Acc aj;
      P::acc_zero(aj);
#pragma unroll 1
      while (true) {
        unsigned long long any = 0;
#pragma unroll
        for (int t = 0; t < NT_MAX_VPM; ++t) any |= has[t];
        if (__ballot(any != 0) == 0) break;
        if (any != 0) {
          const int m = __ffsll((long long)any) - 1;
          int ts = 0;
          bool found = false;
#pragma unroll
          for (int t = 0; t < NT_MAX_VPM; ++t) {
            const bool hit = !found && ((has[t] >> m) & 1);
            ts = hit ? t : ts;
            has[t] &= ~(hit ? 1ull << m : 0ull);
            found = found || hit;
          }
          Acc d1;
          P::acc_set(d1, P::load(ds + (slot + m) * nvpm + ts, dsp));
          P::acc_merge(aj, d1);
        }
      }
      const int j = j0 + ml;
      if (e < e1 && j < nvar)
        P::store(A + (size_t)s * NP * neq * nvar + (size_t)j * neq + e, (size_t)neq * nvar, P::acc_value(aj));
    }
    lds_wait();  // read before the next equations overwrite them
  }
}

// x += d for every point (one wave per point, lane j = variable j), and the
// FP64 2-norm of d (leading limbs) into dnorm[s] when dnorm is given.  A
// point whose factorisation failed (info[s] != 0) keeps its x and gets a
// NaN norm.
template <class P>
__global__ __launch_bounds__(64) void newton_update_kernel(int nvar, double *x, const double *d, const int *info,
                                                           double *dnorm) {
  using C = typename P::C;
  constexpr int NP = 2 * P::L;
  const int lane = threadIdx.x, s = blockIdx.x;
  if (info[s] != 0) {
    if (dnorm != nullptr && lane == 0) dnorm[s] = __builtin_nan("");
    return;
  }
  double *xp = x + (size_t)s * NP * nvar;
  const double *dp = d + (size_t)s * NP * nvar;
  double sq = 0.0;
  if (lane < nvar) {
    C xv = P::load(xp + lane, (size_t)nvar);
    const C dv = P::load(dp + lane, (size_t)nvar);
    C m1 = P::czero();
    m1.re = P::rfrom(-1.0);
    P::upd(xv, m1, dv);  // x - (-1) d
    P::store(xp + lane, (size_t)nvar, xv);
    sq = dp[lane] * dp[lane] + dp[lane + nvar] * dp[lane + nvar];
  }
#pragma unroll
  for (int mask = 32; mask >= 1; mask >>= 1) sq += __shfl_xor(sq, mask);
  if (dnorm != nullptr && lane == 0) dnorm[s] = sqrt(sq);
}

}  // namespace mgsq
