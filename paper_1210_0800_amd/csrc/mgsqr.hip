// C ABI of the MGS least-squares library (declared in include/mgsqr.h):
// argument checks, launch-shape selection and kernel launches.  No
// allocation, no host<->device copies, no synchronisation.
#include "../../include/mgsqr.h"

#include <hip/hip_runtime.h>

#include <cstdint>
#include <atomic>
#include <mutex>

#include "adjoint_kernels.hpp"
#include "backsolve_kernels.hpp"
#include "batched_kernels.hpp"
#include "left_kernels.hpp"
#include "mgs_kernels.hpp"
#include "newton_kernels.hpp"
#include "precision_kernels.hpp"
#include "resident_kernels.hpp"

using namespace mgsq;

// Workspace of mgs_qr_noalloc: a fixed device array, one copy per GPU the
// code object is loaded on, held until the process ends.  Host code never
// uses this name as an address (it denotes a host-side stand-in): the
// device address comes from hipGetSymbolAddress (scratch_address below).
static_assert(MGS_NOALLOC_SCRATCH_BYTES % 256 == 0, "scratch size");
static __device__ __align__(256) unsigned char scratch[MGS_NOALLOC_SCRATCH_BYTES];

namespace {

bool aligned8(const void *p) { return p != nullptr && (reinterpret_cast<uintptr_t>(p) & 7u) == 0; }
size_t round256(size_t b) { return (b + 255) & ~size_t(255); }
int max_rows(int prec) { return prec == 4 ? MGS_MAX_ROWS_QD : MGS_MAX_ROWS_DD; }
bool prec_ok(int prec) { return prec == 1 || prec == 2 || prec == 4; }
int pow2_at_least(int v) {
  int p = 1;
  while (p < v) p <<= 1;
  return p;
}
int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Launch shape of one factorisation (rows padded to the shape, zeros beyond m):
//   trailing role: a team of TW waves per column, RPT rows per lane
//     (RPT a power of two, at most 16 for dd and 8 for qd, so that the
//     column stays in registers);
//   panel role: RP = RPT*TW/4 rows per thread (at least 1) over the block's
//     256 threads, panel width BWM = elements-per-thread budget / RP.
struct Shape {
  int tw, rpt, rp;
};
Shape choose_shape(int m, int prec, int ncols = 0) {
  const int rpt_max = prec == 1 ? 32 : (prec == 2 ? 16 : 8);
  Shape s;
  s.tw = pow2_at_least(ceil_div(m, 64 * rpt_max));
  // qd with few columns: up to 4 waves per trailing column, so that the
  // trailing columns of a launch give about 1024 waves (4 per compute unit)
  // and each wave's share of a projection stays short.
  if (prec == 4)
    while (s.tw < 4 && ncols * s.tw < 1024) s.tw *= 2;
  s.rpt = pow2_at_least(ceil_div(m, 64 * s.tw));
  s.rp = s.rpt * s.tw / NWAVE > 1 ? s.rpt * s.tw / NWAVE : 1;
  return s;
}
constexpr int bw_for(int L, int RP) {
  // complex elements per thread held by the panel role: FP64 16, dd 8;
  // the panel width is capped (FP64 / dd 4) so that its loops unroll fully
  // and every register array keeps static indices.  qd: one column per
  // panel (the panel role's qd arithmetic is the serial part of each
  // launch, and its look-ahead work grows with the square of the width).
  return L == 1 ? (16 / RP >= 4 ? 4 : (16 / RP >= 1 ? 16 / RP : 1))
                : L == 2 ? (8 / RP >= 4 ? 4 : (8 / RP >= 1 ? 8 / RP : 1))
                         : 1;
}

// LDS budget for staged q vectors (gfx950: 160 KiB per CU).
constexpr size_t QSTAGE_BYTES = 128 * 1024;

template <class P, int RPT, int TW>
int launch_steps(StepArgs a, hipStream_t st) {
  constexpr int RP = RPT * TW / NWAVE > 1 ? RPT * TW / NWAVE : 1;
  constexpr int BWM = bw_for(P::L, RP);
  constexpr int TEAMS = NWAVE / TW;
  a.bw = BWM;
  a.npanel = ceil_div(a.n, a.bw);
  a.mpad = RPT * 64 * TW > RP * WG ? RPT * 64 * TW : RP * WG;
  const size_t qbytes = sizeof(double) * 2 * P::L * (size_t)a.mpad;
  a.qstage = (int)(QSTAGE_BYTES / qbytes);
  if (a.qstage > a.bw) a.qstage = a.bw;
  if (a.qstage < 1) return MGS_ERR_DIMS;
  const size_t shmem = qbytes * a.qstage;
  auto kern = mgs_step_kernel<P, RPT, TW, RP, BWM>;
  if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)shmem) != hipSuccess)
    return MGS_ERR_LAUNCH;
  const int last = a.ncols > a.n ? a.npanel : a.npanel - 1;
  for (int t = 0; t <= last; ++t) {
    a.t = t;
    const int jstart = (t + 1) * a.bw < a.n ? (t + 1) * a.bw : a.n;
    const int ntrail = t >= 1 ? a.ncols - jstart : 0;
    const int tblocks = ntrail > 0 ? ceil_div(ntrail, TEAMS) : 0;
    const int grid = (t < a.npanel ? 1 : 0) + tblocks;
    if (grid == 0) continue;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(WG), shmem, st, a);
    if (hipGetLastError() != hipSuccess) return MGS_ERR_LAUNCH;
  }
  return MGS_OK;
}

template <class P>
int dispatch_shape(const StepArgs &a, const Shape &sh, hipStream_t st) {
  if constexpr (P::L == 1) {
    if (sh.tw == 1) {
      switch (sh.rpt) {
        case 1: return launch_steps<P, 1, 1>(a, st);
        case 2: return launch_steps<P, 2, 1>(a, st);
        case 4: return launch_steps<P, 4, 1>(a, st);
        case 8: return launch_steps<P, 8, 1>(a, st);
        case 16: return launch_steps<P, 16, 1>(a, st);
        case 32: return launch_steps<P, 32, 1>(a, st);
      }
    } else if (sh.rpt == 32 && sh.tw == 2) {
      return launch_steps<P, 32, 2>(a, st);
    }
  } else if constexpr (P::L == 2) {
    if (sh.tw == 1) {
      switch (sh.rpt) {
        case 1: return launch_steps<P, 1, 1>(a, st);
        case 2: return launch_steps<P, 2, 1>(a, st);
        case 4: return launch_steps<P, 4, 1>(a, st);
        case 8: return launch_steps<P, 8, 1>(a, st);
        case 16: return launch_steps<P, 16, 1>(a, st);
      }
    } else if (sh.rpt == 16 && sh.tw == 2) {
      return launch_steps<P, 16, 2>(a, st);
    } else if (sh.rpt == 16 && sh.tw == 4) {
      return launch_steps<P, 16, 4>(a, st);
    }
  } else {
    if (sh.tw == 1) {
      switch (sh.rpt) {
        case 1: return launch_steps<P, 1, 1>(a, st);
        case 2: return launch_steps<P, 2, 1>(a, st);
        case 4: return launch_steps<P, 4, 1>(a, st);
        case 8: return launch_steps<P, 8, 1>(a, st);
      }
    } else if (sh.rpt == 8 && sh.tw == 2) {
      return launch_steps<P, 8, 2>(a, st);
    } else if (sh.tw == 4) {
      switch (sh.rpt) {
        case 1: return launch_steps<P, 1, 4>(a, st);
        case 2: return launch_steps<P, 2, 4>(a, st);
        case 4: return launch_steps<P, 4, 4>(a, st);
        case 8: return launch_steps<P, 8, 4>(a, st);
      }
    }
  }
  return MGS_ERR_DIMS;
}

struct DevInfo {
  int cus;  // compute units when cooperative launches are supported, else 0
  long long wclk_khz;
};
bool dev_info(DevInfo &d);

// Race checks: the timing-jitter seed handed to the kernels that
// synchronise across waves or workgroups (mgs_set_jitter; 0: none).
std::atomic<unsigned> g_jitter{0};

// What a launch with bounded waits is given: their wall-clock limit (2 s) and
// the jitter's seed.  Tests of the time-out paths (mgs_set_wait_limit) give
// the calling thread's `t_limit_in`-th launch from here another limit and,
// where it is a triangular solve, long pauses.
thread_local int t_limit_in = 0;
thread_local long long t_limit_ticks = 0;
struct WaitArgs {
  long long ticks;
  unsigned jitter;
};
WaitArgs wait_args(long long wclk_khz) {
  if (t_limit_in > 0 && --t_limit_in == 0) return {t_limit_ticks, TS_STALL};
  return {wclk_khz * 2000, g_jitter.load(std::memory_order_relaxed)};
}

// R x = y, or R^H x = y with FWD.  Up to 128 rows one workgroup; beyond, one
// per 128 rows in a cooperative launch, or, where that is refused, one
// workgroup that takes the blocks in turn.  keep_info: info holds the status
// of what came before and is not cleared.
template <class P, bool FWD = false>
int trsv_launch(int n, const double *R, int ldr, const double *y, double *x, int *info, hipStream_t st,
                bool keep_info = false, size_t planeR = 0, const int *skip = nullptr, size_t planeY = 0) {
  if (planeR == 0) planeR = (size_t)ldr * n;
  if (planeY == 0) planeY = (size_t)n;
  const int waves = ceil_div(n, TS_ROWS) < TS_WAVES ? ceil_div(n, TS_ROWS) : TS_WAVES;
  const int G = ceil_div(n, TS_ROWS * waves);
  DevInfo d;
  const bool have = dev_info(d);
  WaitArgs wait = wait_args(have ? d.wclk_khz : 100000);
  int marked = G > 1 ? 1 : 0, keep = keep_info ? 1 : 0;
  auto kern = trsv_kernel<P, FWD>;
  if (marked) {
    hipLaunchKernelGGL((bs_mark_kernel<P::L>), dim3(ceil_div(n, 256)), dim3(256), 0, st, n, x, info, keep,
                       skip);
    if (hipGetLastError() != hipSuccess) return MGS_ERR_LAUNCH;
    if (have && d.cus >= G) {
      void *args[] = {&n, &R, &ldr, &planeR, &y, &planeY, &x, &info, &keep, &skip, &marked, &wait.ticks, &wait.jitter};
      if (hipLaunchCooperativeKernel(reinterpret_cast<const void *>(kern), dim3(G), dim3(64 * waves), args, 0, st) ==
          hipSuccess)
        return MGS_OK;
      (void)hipGetLastError();
    }
  }
  hipLaunchKernelGGL(kern, dim3(1), dim3(64 * waves), 0, st, n, R, ldr, planeR, y, planeY, x, info, keep, skip, marked,
                     wait.ticks, wait.jitter);
  return hipGetLastError() == hipSuccess ? MGS_OK : MGS_ERR_LAUNCH;
}

// Columns in flight: as the registers allow (256 a lane).
template <class P>
int project_launch(int m, int n, const double *Q, int ldq, const double *b, double *y, hipStream_t st) {
  const size_t planeQ = (size_t)ldq * n;
#define MGS_PROJ_CASE(RPTV, RINGV)                                                                                \
  case RPTV:                                                                                                      \
    hipLaunchKernelGGL((project_kernel<P, RPTV, RINGV>), dim3(1), dim3(512), 0, st, m, n, Q, ldq, planeQ, b, y); \
    break;
  switch (pow2_at_least(ceil_div(m, 512))) {
    MGS_PROJ_CASE(1, (P::L == 4 ? 3 : 4))
    MGS_PROJ_CASE(2, (P::L == 4 ? 2 : 4))
    MGS_PROJ_CASE(4, (P::L == 4 ? 1 : P::L == 2 ? 2 : 4))
    default:
      if constexpr (P::L == 4) {
        return MGS_ERR_DIMS;  // past the qd row limit
      } else {
        switch (8) { MGS_PROJ_CASE(8, (P::L == 2 ? 1 : 2)) }
      }
  }
#undef MGS_PROJ_CASE
  return hipGetLastError() == hipSuccess ? MGS_OK : MGS_ERR_LAUNCH;
}

// QR: working copy of b (2Lm doubles), then the synchronisation words of
// the single-launch schedule, then (the shapes that can take it: dd with
// m <= 1024, FP64 with m <= 2048 and at most 32 MiB) its hand-off copy of
// the n columns (2Lmn doubles).
size_t qr_w_bytes(int m, int prec) { return round256(sizeof(double) * 2 * (size_t)prec * m); }
bool res_rows_ok(int m, int prec) { return (prec == 2 && m <= 1024) || (prec == 1 && m <= 2048); }
size_t qr_u_bytes(int m, int n, int prec) {
  const size_t u = round256(sizeof(double) * 2 * (size_t)prec * m * n);
  return (res_rows_ok(m, prec) && u <= ((size_t)32 << 20)) ? u : 0;
}
size_t qr_work_bytes(int m, int n, int prec) {
  return qr_w_bytes(m, prec) + sizeof(unsigned int) * RES_SYNC_WORDS + qr_u_bytes(m, n, prec);
}
size_t solve_work_bytes(int n, int prec) { return round256(sizeof(double) * 2 * (size_t)prec * n); }
// adjoint: w (n), z (n), r (m), then the chunk partials of Q w and b - A x
// (2 x chunks x m accumulators).
size_t adj_acc_bytes(int prec) { return prec == 2 ? sizeof(Partial<PrecDD>::T) : sizeof(Partial<PrecQD>::T); }
size_t adjoint_work_bytes(int m, int n, int prec) {
  const size_t nchunk = (size_t)((n + ADJ_CH - 1) / ADJ_CH);
  return 2 * round256(sizeof(double) * 2 * (size_t)prec * n) + round256(sizeof(double) * 2 * (size_t)prec * m) +
         round256(adj_acc_bytes(prec) * 2 * nchunk * m);
}

template <class P>
int adjoint_launch(int m, int n, const double *A, int lda, const double *b, const double *Q, int ldq,
                   const double *R, int ldr, const double *x, const double *gx, double *gA, int ldga, double *gb,
                   void *work, int *info, hipStream_t st) {
  double *w = static_cast<double *>(work);
  double *z = w + round256(sizeof(double) * 2 * P::L * (size_t)n) / sizeof(double);
  double *r = z + round256(sizeof(double) * 2 * P::L * (size_t)n) / sizeof(double);
  auto *part =
      reinterpret_cast<typename Partial<P>::T *>(r + round256(sizeof(double) * 2 * P::L * (size_t)m) / sizeof(double));
  int rc = trsv_launch<P, true>(n, R, ldr, gx, w, info, st);
  if (rc != MGS_OK) return rc;
  // (info keeps what the first solve had to report)
  rc = trsv_launch<P>(n, R, ldr, w, z, info, st, true);
  if (rc != MGS_OK) return rc;
  hipLaunchKernelGGL((adj_partial_kernel<P>), dim3(ceil_div(m, ADJ_T), ceil_div(n, ADJ_CH), 2), dim3(ADJ_T), 0, st,
                     m, n, Q, ldq, (size_t)ldq * n, A, lda, (size_t)lda * n, b, x, w, part);
  if (hipGetLastError() != hipSuccess) return MGS_ERR_LAUNCH;
  hipLaunchKernelGGL((adj_finish_kernel<P>), dim3(ceil_div(m, WG), 2), dim3(WG), 0, st, m, n, part, gb, r);
  if (hipGetLastError() != hipSuccess) return MGS_ERR_LAUNCH;
  hipLaunchKernelGGL((adj_rank2_kernel<P>), dim3(ceil_div(m, WG), n), dim3(WG), 0, st, m, n, r, z, gb, x, gA, ldga,
                     (size_t)ldga * n);
  return hipGetLastError() == hipSuccess ? MGS_OK : MGS_ERR_LAUNCH;
}

// ------------------------------------------------------ precision form --
struct RefineWork {
  double *Q64, *R64, *y64, *d64, *r64;
  void *partial;
  RefineCtl *ctl;
  void *res;  // the FP64 panels' single launch: synchronisation words, then U (nullptr: none)
  size_t bytes;
};
// Synchronisation words and hand-off copy U of one FP64 panel (m x NBP)
// for the single-launch panel factorisation (m <= 2048), else nothing.
size_t panel_res_bytes(int m, int n) {
  if (m > 2048) return 0;
  const int nb = n < NBP ? n : NBP;
  return round256(sizeof(unsigned int) * RES_SYNC_WORDS) + round256(sizeof(double) * 2 * (size_t)m * nb);
}
RefineWork refine_layout(int m, int n, int prec, void *base) {
  const int nchunk = ceil_div(n, NBP);
  const size_t acc_bytes = sizeof(Partial<PrecQD>::T);  // the residual accumulates in qd
  (void)prec;
  size_t off = 0;
  auto take = [&](size_t b) {
    size_t o = off;
    off += round256(b);
    return static_cast<char *>(base) + o;
  };
  RefineWork w;
  w.Q64 = reinterpret_cast<double *>(take(sizeof(double) * 2 * (size_t)m * (n + 1)));
  w.R64 = reinterpret_cast<double *>(take(sizeof(double) * 2 * (size_t)n * (n + 1)));
  w.y64 = reinterpret_cast<double *>(take(sizeof(double) * 2 * (size_t)n));
  w.d64 = reinterpret_cast<double *>(take(sizeof(double) * 2 * (size_t)n));
  w.r64 = reinterpret_cast<double *>(take(sizeof(double) * 2 * (size_t)m));
  w.partial = take(acc_bytes * (size_t)nchunk * m);
  w.ctl = reinterpret_cast<RefineCtl *>(take(sizeof(RefineCtl)));
  w.res = panel_res_bytes(m, n) > 0 ? take(panel_res_bytes(m, n)) : nullptr;
  w.bytes = off;
  return w;
}

// mgs_qr64: Q64 (m x (n+1)) and R64 (n x (n+1)), FP64 complex, then the
// panel factorisation's single-launch area.
size_t qr64_work_bytes(int m, int n) {
  return round256(sizeof(double) * 2 * (size_t)m * (n + 1)) + round256(sizeof(double) * 2 * (size_t)n * (n + 1)) +
         panel_res_bytes(m, n);
}

template <class P>
int res_launch(const StepArgs &s, void *sync, double *u, hipStream_t st);

// FP64 blocked MGS of [A64 b64] held in Q64 (m x (n+1)); R64 (n x (n+1))
// receives R and, in its last column, y.
int factor64(int m, int n, const RefineWork &w, int *info, hipStream_t st) {
  const size_t planeQ = (size_t)m * (n + 1), planeR = (size_t)n * (n + 1);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(256), dim3(256), 0, st, w.R64, 2 * planeR);
  const Shape sh = choose_shape(m, 1);
  for (int k0 = 0; k0 < n; k0 += NBP) {
    const int nb = n - k0 < NBP ? n - k0 : NBP;
    StepArgs a;
    a.m = m;
    a.n = nb;
    a.ncols = nb;
    a.A = w.Q64 + (size_t)k0 * m;
    a.lda = m;
    a.planeA = planeQ;
    a.b = nullptr;
    a.Q = w.Q64 + (size_t)k0 * m;
    a.ldq = m;
    a.planeQ = planeQ;
    a.R = w.R64 + (size_t)k0 * n + k0;
    a.ldr = n;
    a.planeR = planeR;
    a.W = nullptr;
    a.y = nullptr;
    a.rho = nullptr;
    a.info = info;
    a.t = 0;
    a.kbase = k0;
    a.init_info = 0;
    // The panel in one cooperative launch when it fits, else one launch
    // per column pair.
    int rc = 1;
    if (w.res != nullptr) {
      double *u = reinterpret_cast<double *>(static_cast<char *>(w.res) +
                                             round256(sizeof(unsigned int) * RES_SYNC_WORDS));
      rc = res_launch<PrecD>(a, w.res, u, st);
    }
    if (rc == 1) rc = dispatch_shape<PrecD>(a, sh, st);
    if (rc != MGS_OK) return rc;
    const int N = n + 1 - (k0 + nb);  // trailing columns, b included
    if (N > 0) {
      const double *Qp = w.Q64 + (size_t)k0 * m;
      double *At = w.Q64 + (size_t)(k0 + nb) * m;
      double *Wb = w.R64 + (size_t)(k0 + nb) * n + k0;
      hipLaunchKernelGGL(zgemm_qha_kernel, dim3(ceil_div(N, 16), ceil_div(nb, 16)), dim3(64 * QHA_SLICES), 0, st, m, N,
                         nb, Qp, m, At, m, planeQ, Wb, n, planeR);
      const int tiles = ceil_div(m, 16) * ceil_div(N, 16);
      hipLaunchKernelGGL(zgemm_update_kernel, dim3(ceil_div(tiles, 4)), dim3(256), 0, st, m, N, nb, Qp, m, At, m,
                         planeQ, Wb, n, planeR);
    }
    if (hipGetLastError() != hipSuccess) return MGS_ERR_LAUNCH;
  }
  return MGS_OK;
}

template <class P>
int refine_solve(int m, int n, const double *A, int lda, const double *b, double *x, double tol, int max_iter,
                 int *iters, double *err_est, void *work, int *info, hipStream_t st) {
  RefineWork w = refine_layout(m, n, P::L, work);
  const size_t planeQ = (size_t)m * (n + 1), planeR = (size_t)n * (n + 1);
  hipLaunchKernelGGL((copy_hi_kernel<P::L>), dim3(ceil_div(m, 256), n + 1), dim3(256), 0, st, m, n, A, lda, b, w.Q64,
                     w.ctl, info);
  int rc = factor64(m, n, w, info, st);
  if (rc != MGS_OK) return rc;
  hipLaunchKernelGGL(refine_check_kernel, dim3(1), dim3(64), 0, st, info, w.ctl);
  const int *skip = &w.ctl->status;
  // x0: R x0 = y (the last column of R64)
  rc = trsv_launch<PrecD>(n, w.R64, n, w.R64 + (size_t)n * n, w.d64, info, st, true, planeR, skip, planeR);
  if (rc != MGS_OK) return rc;
  hipLaunchKernelGGL((set_x_kernel<P>), dim3(ceil_div(n, 256)), dim3(256), 0, st, n, w.d64, x);
  const int nchunk = ceil_div(n, NBP);
  // The correction's panel projections: one cooperative launch per step
  // (proj_replay_kernel) when it can run, else two launches per panel.  The
  // launches of a converged solve return at once, so the fixed max_iter
  // steps cost little past convergence.
  DevInfo d;
  // (the barrier count of all steps must fit the 32-bit counter; the partial
  // sums that pass between its workgroups lie where the residual's were, 64
  // bytes per row and panel against 16 to 32)
  const int pr_wgs = ceil_div(m, PR_ROWS);
  bool fused = m <= PR_MAX_ROWS && (long long)max_iter * pr_wgs < (1LL << 31) && dev_info(d) && d.cus >= pr_wgs &&
               (pr_wgs == 1 || sizeof(double) * 2 * NBP * (size_t)(nchunk < 3 ? nchunk : 3) * pr_wgs <=
                                   sizeof(Partial<PrecQD>::T) * (size_t)nchunk * m);
  for (int it = 1; it <= max_iter; ++it) {
    hipLaunchKernelGGL((residual_partial_kernel<P::L>), dim3(ceil_div(m, 256), nchunk), dim3(256), 0, st, m, n, NBP,
                       A, lda, b, x, static_cast<Partial<PrecQD>::T *>(w.partial), w.ctl);
    hipLaunchKernelGGL((residual_finish_kernel<PrecQD>), dim3(ceil_div(m, 256)), dim3(256), 0, st, m, nchunk,
                       static_cast<const Partial<PrecQD>::T *>(w.partial), w.r64, w.ctl);
    if (fused) {
      // arrivals at the grid barriers of the earlier steps (one each)
      unsigned int base = pr_wgs > 1 ? (unsigned int)(it - 1) * (unsigned int)pr_wgs : 0u;
      const double *Qa = w.Q64, *ra = w.r64;
      size_t pq = planeQ, pw = (size_t)n;
      double *wa = w.y64, *pa = static_cast<double *>(w.partial);
      RefineCtl *ctl = w.ctl;
      int mm = m, nn = n;
      WaitArgs wait = wait_args(d.wclk_khz);
      void *args[] = {&mm, &nn, &Qa, &pq, &ra, &wa, &pw, &pa, &ctl, &info, &base, &wait.ticks, &wait.jitter};
      if (hipLaunchCooperativeKernel(reinterpret_cast<const void *>(proj_replay_kernel), dim3(pr_wgs), dim3(256), args,
                                     0, st) != hipSuccess) {
        (void)hipGetLastError();
        fused = false;  // the barrier count is off from here: per-panel launches for the rest
      }
    }
    if (!fused) {
      for (int k0 = 0; k0 < n; k0 += NBP) {
        const int nb = n - k0 < NBP ? n - k0 : NBP;
        const double *Qp = w.Q64 + (size_t)k0 * m;
        hipLaunchKernelGGL(proj_w_kernel, dim3(nb), dim3(256), 0, st, m, Qp, m, planeQ, w.r64, w.y64 + k0, (size_t)n,
                           w.ctl);
        hipLaunchKernelGGL(proj_r_kernel, dim3(ceil_div(m, 256)), dim3(256), 0, st, m, nb, Qp, m, planeQ, w.y64 + k0,
                           (size_t)n, w.r64, w.ctl);
      }
    }
    rc = trsv_launch<PrecD>(n, w.R64, n, w.y64, w.d64, info, st, true, planeR, skip);
    if (rc != MGS_OK) return rc;
    hipLaunchKernelGGL((refine_update_kernel<P>), dim3(1), dim3(256), 0, st, n, w.d64, x, tol, it, w.ctl,
                       info);
    if (hipGetLastError() != hipSuccess) return MGS_ERR_LAUNCH;
  }
  hipLaunchKernelGGL(refine_finish_kernel, dim3(1), dim3(64), 0, st, w.ctl, iters, err_est, info);
  return hipGetLastError() == hipSuccess ? MGS_OK : MGS_ERR_LAUNCH;
}

// ------------------------------------------- single-launch schedule --------
bool dev_info(DevInfo &d) {
  static DevInfo cache[64];
  static bool have[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
  if (!have[dev]) {
    int cus = 0, wclk = 0, coop = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return false;
    if (hipDeviceGetAttribute(&wclk, hipDeviceAttributeWallClockRate, dev) != hipSuccess) return false;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess) return false;
    cache[dev].cus = coop ? cus : 0;
    cache[dev].wclk_khz = wclk > 0 ? wclk : 100000;
    have[dev] = true;
  }
  d = cache[dev];
  return true;
}

// Columns held by the workgroup holding the most, for panels of bw columns
// dealt in the reflected cyclic order of the resident kernel.
int res_max_cols(int ncols, int bw, int G) {
  const int np = ceil_div(ncols, bw);
  int best = 0;
  for (int g = 0; g < G; ++g) {
    int cnt = 0;
    for (int i = 0;; ++i) {
      const int qi = res_position(i, g, G);
      if (qi >= np) break;
      const int p = np - 1 - qi;
      cnt += (ncols - p * bw < bw) ? ncols - p * bw : bw;
    }
    if (cnt > best) best = cnt;
  }
  return best;
}

// Resident shapes (dd): workgroups of nw waves (up to 8, 2 per SIMD), RR
// rows per thread, CB column slots per workgroup (register budget 256 per
// lane).  Short columns take fewer waves (64 nw >= m), so that their block
// sums have fewer levels and their barriers fewer waves.
constexpr int RES_NW = 8;
// Column slots: 80 registers of columns per lane (dd: RR x CB <= 10 of 8
// registers; FP64: RR x CB <= 20 of 4), at most 8 slots.
constexpr int res_cb(int L, int rr) { return L == 2 ? (rr == 1 ? 8 : 5) : (rr <= 2 ? 8 : 5); }

struct ResPlan {
  int rr, nw, bw, np, G;
};
bool res_choose(int m, int ncols, int L, int cus, ResPlan &pl) {
  const int rr = pow2_at_least(ceil_div(m, 64 * RES_NW));
  if (rr > (L == 1 ? 4 : 2)) return false;
  int nw = RES_NW;
  if (rr == 1) {
    nw = pow2_at_least(ceil_div(m, 64));
    if (nw > RES_NW) nw = RES_NW;
  }
  const int cb = res_cb(L, rr);
  // Panels of one column: the look-ahead hand-off of the kernel assumes it.
  const int bws[1] = {1};
  for (int bw : bws) {
    const int np = ceil_div(ncols, bw);
    const int G = np < cus ? np : cus;
    if (res_max_cols(ncols, bw, G) <= cb) {
      pl.rr = rr;
      pl.nw = nw;
      pl.bw = bw;
      pl.np = np;
      pl.G = G;
      return true;
    }
  }
  return false;
}

#ifdef MGS_TRACE
// Diagnostic builds: device buffer of RES_TRACE_SLOTS stamps per column for
// the next single-launch factorisations (mgs_set_trace).
long long *g_trace = nullptr;
#endif

// Returns 1 when the single launch does not apply here (the caller then
// takes the per-panel schedule).
template <class P, int RR, int NW>
int res_launch_rr(ResArgs a, int cus, hipStream_t st) {
  constexpr int CB = res_cb(P::L, RR);
  auto kern = mgs_resident_kernel<P, RR, CB, NW>;
  // Only kernels that keep everything in registers and LDS take this
  // schedule: no private (scratch) memory in a cooperative launch.
  hipFuncAttributes fa;
  if (hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(kern)) != hipSuccess || fa.localSizeBytes != 0)
    return 1;
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(kern), 64 * NW, 0) !=
      hipSuccess)
    return 1;
  if ((long long)per_cu * cus < a.G) return 1;
  hipLaunchKernelGGL(resident_init_kernel, dim3(1), dim3(RES_SYNC_WORDS), 0, st, a.sync, a.info, a.init_info);
  if (hipGetLastError() != hipSuccess) return MGS_ERR_LAUNCH;
  void *args[] = {&a};
  if (hipLaunchCooperativeKernel(reinterpret_cast<const void *>(kern), dim3(a.G), dim3(64 * NW), args, 0, st) !=
      hipSuccess) {
    (void)hipGetLastError();
    return 1;
  }
  return MGS_OK;
}

// FP64 and dd only: the qd instantiations do not fit in registers.
template <class P>
int res_launch(const StepArgs &s, void *sync, double *u, hipStream_t st) {
  static_assert(P::L <= 2, "no qd instantiation of the single launch");
  DevInfo d;
  if (!dev_info(d) || d.cus <= 0) return 1;
  ResPlan pl;
  if (!res_choose(s.m, s.ncols, P::L, d.cus, pl)) return 1;
  ResArgs a;
  a.m = s.m;
  a.n = s.n;
  a.ncols = s.ncols;
  a.A = s.A;
  a.lda = s.lda;
  a.planeA = s.planeA;
  a.b = s.b;
  a.Q = s.Q;
  a.ldq = s.ldq;
  a.planeQ = s.planeQ;
  a.R = s.R;
  a.ldr = s.ldr;
  a.planeR = s.planeR;
  a.y = s.y;
  a.rho = s.rho;
  a.info = s.info;
  a.sync = static_cast<unsigned int *>(sync);
  a.U = u;
  a.ldu = s.m;
  a.planeU = (size_t)s.m * s.n;
  a.bw = pl.bw;
  a.np = pl.np;
  a.G = pl.G;
  a.xcd_group = pl.G % 8 == 0 ? pl.G / 8 : 0;
  a.defer = 12;
  const WaitArgs wait = wait_args(d.wclk_khz);
  a.spin_ticks = wait.ticks;
  a.jitter = wait.jitter;
  a.kbase = s.kbase;
  a.init_info = s.init_info;
#ifdef MGS_TRACE
  a.trace = g_trace;
#endif
  if constexpr (P::L == 1) {
    if (pl.rr == 4) return res_launch_rr<P, 4, 8>(a, d.cus, st);
  }
  if (pl.rr == 2) return res_launch_rr<P, 2, 8>(a, d.cus, st);
  switch (pl.nw) {
    case 1: return res_launch_rr<P, 1, 1>(a, d.cus, st);
    case 2: return res_launch_rr<P, 1, 2>(a, d.cus, st);
    case 4: return res_launch_rr<P, 1, 4>(a, d.cus, st);
    case 8: return res_launch_rr<P, 1, 8>(a, d.cus, st);
  }
  return 1;
}

// ------------------------------------------------ left-looking qd ------
// Workspace: the records (2 L n doubles, in the place of the working copy of
// b, 2 L m doubles) and the synchronisation words.  PC workgroups per compute
// unit, no more than columns.
template <class P, int RPT, int NW, int PC>
int left_launch_shape(LeftArgs a, int cus, int khz, hipStream_t st) {
  const int G = a.ncols < PC * cus ? a.ncols : PC * cus;
  a.meet = G > cus ? khz / 20 : 0;
  const int nrec = 2 * P::L * a.n;
  hipLaunchKernelGGL(left_init_kernel, dim3(a.marked ? ceil_div(a.m, 256) : 1, a.n), dim3(256), 0, st, a.sync, a.info,
                     a.rec, nrec, a.m, a.n, a.Q, a.ldq, a.planeQ, a.marked ? 2 * P::L : 0);
  if (hipGetLastError() != hipSuccess) return MGS_ERR_LAUNCH;
  hipLaunchKernelGGL((mgs_left_kernel<P, RPT, NW, PC>), dim3(G), dim3(64 * NW), 0, st, a);
  if (hipGetLastError() != hipSuccess) return MGS_ERR_LAUNCH;
  hipLaunchKernelGGL((left_finish_kernel<P>), dim3(a.n), dim3(256), 0, st, a.m, a.n, a.Q, a.ldq, a.planeQ, a.R, a.ldr,
                     a.planeR, a.rec);
  return hipGetLastError() == hipSuccess ? MGS_OK : MGS_ERR_LAUNCH;
}
// m <= 1024.
int left_launch_qd(const StepArgs &s, void *work, hipStream_t st) {
  using P = PrecQD;
  DevInfo d;
  const bool have = dev_info(d);
  const int cus = have && d.cus > 0 ? d.cus : 256;
  LeftArgs a;
  a.m = s.m;
  a.n = s.n;
  a.ncols = s.ncols;
  a.A = s.A;
  a.lda = s.lda;
  a.planeA = s.planeA;
  a.b = s.b;
  a.Q = s.Q;
  a.ldq = s.ldq;
  a.planeQ = s.planeQ;
  a.R = s.R;
  a.ldr = s.ldr;
  a.planeR = s.planeR;
  a.y = s.y;
  a.rho = s.rho;
  a.info = s.info;
  a.rec = static_cast<double *>(work);
  a.sync = reinterpret_cast<unsigned int *>(static_cast<char *>(work) + qr_w_bytes(s.m, P::L));
  a.marked = s.Q != s.A;
  const int khz = have ? (int)d.wclk_khz : 100000;
  const WaitArgs wait = wait_args(khz);
  a.spin_ticks = wait.ticks;
  a.jitter = wait.jitter;
  // One column per workgroup (up to an eighth more: a workgroup's first
  // column is soon done): one row per thread, the shortest link (80 x 80 5.5 us
  // a column, 320 x 256 8.1; with 2 rows per thread on half the waves 1.13
  // times that).  More columns than that: fewer, fuller waves, which halves
  // the sums' share, and several workgroups per compute unit to fill each
  // other's waits (500 x 500 5.2 ms, 1.11 times that with one; 1024 x 1024 30.2
  // ms, 1.11 times that with 8 waves of 2 rows, one workgroup).
  const bool single = s.ncols <= cus + cus / 8;
  if (s.m <= 64) return left_launch_shape<P, 1, 1, 1>(a, cus, khz, st);
  if (s.m <= 128) return left_launch_shape<P, 1, 2, 1>(a, cus, khz, st);
  if (s.m <= 256) return left_launch_shape<P, 1, 4, 1>(a, cus, khz, st);
  if (s.m <= 512)
    return single ? left_launch_shape<P, 1, 8, 1>(a, cus, khz, st) : left_launch_shape<P, 2, 4, 3>(a, cus, khz, st);
  return left_launch_shape<P, 4, 4, 2>(a, cus, khz, st);
}

// Small systems: one workgroup per system (returns MGS_ERR_DIMS when the
// columns do not fit the shape's slots).
template <class P, int RPL, int SL, int NW, int WPE, int CG = 4>
int batched_launch(const BatArgs &a, hipStream_t st) {
  if (a.m > 64 / CG * RPL || a.ncols - 1 > CG * NW * SL) return MGS_ERR_DIMS;
  if (a.batch == 0) return MGS_OK;
  hipLaunchKernelGGL((mgs_batched_kernel<P, RPL, SL, NW, WPE, CG>), dim3(a.batch), dim3(64 * NW), 0, st, a);
  return hipGetLastError() == hipSuccess ? MGS_OK : MGS_ERR_LAUNCH;
}
// The shape by batch size, all with the same results.  While the systems
// alone do not fill the card, several waves each shorten a system's chain;
// beyond, one wave per system does the least work (pairs of slots share a
// sum, nothing is synchronised).  Measured, us per call:
//   32 x 32, 8 waves of 1 slot / 1 wave of 8: double 34 / 48 at 1 system,
//   47 / 56 at 512, 80 / 63 at 1024; dd 69 / 128, 118 / 145, 215 / 149.
//   qd (one wave per SIMD), 4 waves of 2 slots / 2 of 4 / 1 of 8: 453 / 627 /
//   954 at 1, 480 / 657 / 1012 at 256, 928 / 681 / 1028 at 512, 1838 / 1288 /
//   1080 at 1024.
// More than 32 slotted columns, the slots per wave as the registers allow
// (waves x slots):
//   double 64 x 63, 16 x 1 / 4 x 4: 88 / 110 at 1, 105 / 127 at 256, 184 /
//   156 at 512, 1299 / 1110 at 4000 (42 x 42: 50 / 62 and 706 / 455);
//   dd 64 x 63, 8 x 2 / 4 x 4 / 2 x 8: 250 / 268 / 431 at 1, 281 / 304 / 471
//   at 256, 1062 / 1143 / 945 at 1024 (42 x 42: 121 / 128 / 186, 137 / 145 /
//   206, 516 / 366 / 417);
//   qd 48 x 40, 4 x 4 / 8 x 2: 841 / 1057 at 1, 3396 / 4567 at 1024.
// qd past 32 rows with at most 32 slotted columns (48 x 28), 4 waves of 2
// slots / 2 of 4: 517 / 698 at 1, 549 / 743 at 256, 2074 / 1509 at 1024.
template <class P, int RPL>
int batched_shape(const BatArgs &a, int cus, hipStream_t st) {
  const int slotted = a.ncols - 1;  // column 1 has no slot
  const bool one = a.batch <= cus, two = a.batch <= 2 * cus;  // systems per compute unit
  if constexpr (P::L == 4) {
    if constexpr (RPL >= 3) {
      if (slotted > 32) return batched_launch<P, RPL, 4, 4, 1>(a, st);
      return one ? batched_launch<P, RPL, 2, 4, 1>(a, st) : batched_launch<P, RPL, 4, 2, 1>(a, st);
    } else {
      if (one) return batched_launch<P, RPL, 2, 4, 1>(a, st);
      return two ? batched_launch<P, RPL, 4, 2, 1>(a, st) : batched_launch<P, RPL, 8, 1, 1>(a, st);
    }
  } else if constexpr (RPL >= 3) {
    if (slotted <= 32) return two ? batched_launch<P, RPL, 1, 8, 2>(a, st) : batched_launch<P, RPL, 8, 1, 1>(a, st);
    if constexpr (P::L == 1)
      return one ? batched_launch<P, RPL, 1, 16, 4>(a, st) : batched_launch<P, RPL, 4, 4, 2>(a, st);
    if (one) return batched_launch<P, RPL, 2, 8, 2>(a, st);
    return RPL == 3 ? batched_launch<P, RPL, 4, 4, 1>(a, st) : batched_launch<P, RPL, 8, 2, 1>(a, st);
  } else {
    return two ? batched_launch<P, RPL, 1, 8, 2>(a, st) : batched_launch<P, RPL, 8, 1, 2>(a, st);
  }
}
// Few slotted columns on many rows: a grid of fewer columns, so that a column's
// rows are spread over more lanes (RPL 1 or 2 in place of 2 to 4) and each wave
// of a small batch holds one or two columns.  The grid goes by the system's
// size alone (its bits do not depend on the batch).  us per call, 16 x 4 / now:
//   at most 8 columns, more than 32 rows, 64 x 1 (64 x 4): double 10.3 / 8.9 at 1,
//   26.7 / 16.9 at 4000; dd 14.0 / 9.1, 71 / 37; qd 85 / 38, 273 / 127 at 1500;
//   at most 8, 17 to 32 rows, 32 x 2 (20 x 8): double 11.2 / 10.3, 32.2 / 27.8; dd
//   19.2 / 16.0, 73 / 65; qd 104 / 73, 269 / 221 at 1500;
//   9 to 16, more than 32 rows, 32 x 2 (48 x 10): double 15.0 / 13.3, 51.9 / 44;
//   dd 26.1 / 24.6, 158 / 119; qd 154 / 134, 528 / 505 at 1500.
// 9 to 16 on 17 to 32 rows gain alone (28 x 16 double 19.7 -> 17.8) but lose in
// batches (34.5 -> 36.4 at 1500): 16 x 4.  9 to 16 on 64 x 1 likewise (48 x 10
// double 13.3 -> 11.9 with 16 waves, 15.9 -> 21.8 at 257).
template <class P>
int batched_few(const BatArgs &a, int cus, hipStream_t st) {
  const bool one = a.batch <= cus, two = a.batch <= 2 * cus;
  if (a.ncols - 1 <= 8) {
    if (a.m <= 32) return two ? batched_launch<P, 1, 1, 4, 1, 2>(a, st) : batched_launch<P, 1, 4, 1, 1, 2>(a, st);
    if constexpr (P::L == 4)
      return two ? batched_launch<P, 1, 2, 4, 1, 1>(a, st) : batched_launch<P, 1, 8, 1, 1, 1>(a, st);
    return two ? batched_launch<P, 1, 1, 8, 2, 1>(a, st) : batched_launch<P, 1, 8, 1, 2, 1>(a, st);
  }
  if constexpr (P::L == 4) {
    if (one) return batched_launch<P, 2, 2, 4, 1, 2>(a, st);
    return two ? batched_launch<P, 2, 4, 2, 1, 2>(a, st) : batched_launch<P, 2, 8, 1, 1, 2>(a, st);
  } else {
    if (one || (two && P::L == 1)) return batched_launch<P, 2, 1, 8, 2, 2>(a, st);
    return two ? batched_launch<P, 2, 2, 4, 2, 2>(a, st) : batched_launch<P, 2, 8, 1, 2, 2>(a, st);
  }
}
template <class P>
int batched_dispatch(const BatArgs &a, hipStream_t st) {
  DevInfo d;
  const int cus = dev_info(d) && d.cus > 0 ? d.cus : 256;
  if ((a.m > 16 && a.ncols - 1 <= 8) || (a.m > 32 && a.ncols - 1 <= 16)) return batched_few<P>(a, cus, st);
  if (a.m <= 16) return batched_shape<P, 1>(a, cus, st);
  if (a.m <= 32) return batched_shape<P, 2>(a, cus, st);
  if (a.m <= 48) return batched_shape<P, 3>(a, cus, st);
  return batched_shape<P, 4>(a, cus, st);
}
int batched_dispatch(int prec, const BatArgs &a, hipStream_t st) {
  if (prec == 1) return batched_dispatch<PrecD>(a, st);
  if (prec == 2) return batched_dispatch<PrecDD>(a, st);
  return batched_dispatch<PrecQD>(a, st);
}
bool batched_fits(int m, int n, int ncols, int prec) {
  return m <= BAT_MAX_ROWS && ncols <= BAT_MAX_COLS && sizeof(double) * 2 * prec * (size_t)n * m <= BAT_LDS_BYTES;
}

// ------------------------------------------------ allocation-free QR ----
// mgs_qr_noalloc keeps its workspace in `scratch` instead of a
// caller-supplied buffer; kernels get the device address from
// hipGetSymbolAddress, taken once per device with that device current.

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[MAX_DEVICES];

// The current device's address of `scratch` (nullptr on failure).
void *scratch_address() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

// Newton: J (batch systems of neq x nvar), b (batch x neq), R (batch x
// nvar x nvar), d (batch x nvar), each in the working precision; for one
// point in qd also y (nvar) and the workspace of mgs_qr.
struct NewtonWork {
  double *A, *b, *R, *d, *y;
  void *qrw;
  size_t qrw_bytes;
  size_t bytes;
};
NewtonWork newton_layout(int batch, int neq, int nvar, int prec, void *base) {
  size_t off = 0;
  auto take = [&](size_t nd) {
    const size_t o = off;
    off += round256(sizeof(double) * nd);
    return reinterpret_cast<double *>(static_cast<char *>(base) + o);
  };
  const size_t NP = 2 * (size_t)prec, B = (size_t)batch;
  NewtonWork w;
  w.A = take(B * NP * neq * nvar);
  w.b = take(B * NP * neq);
  w.R = take(B * NP * nvar * nvar);
  w.d = take(B * NP * nvar);
  w.y = nullptr;
  w.qrw = nullptr;
  w.qrw_bytes = 0;
  if (batch == 1 && prec == 4) {
    w.y = take(NP * nvar);
    w.qrw_bytes = qr_work_bytes(neq, nvar, prec);
    w.qrw = take((w.qrw_bytes + sizeof(double) - 1) / sizeof(double));
  }
  w.bytes = off;
  return w;
}
bool newton_dims_ok(int batch, int neq, int nvar, int nmon, int nvpm, int prec) {
  return batch >= 0 && batch <= 65535 && nvar >= 1 && nvar <= NT_MAX_VARS && neq >= nvar && nmon >= 1 && nmon <= NT_MAX_MON &&
         nvpm >= 1 && nvpm <= NT_MAX_VPM && batched_fits(neq, nvar, nvar + 1, prec);
}
// Evaluation of neq equations at batch points.  Few points: two equations per
// one-wave workgroup, spread over the card; from 8 workgroups per compute
// unit on, whole points, so that the powers are formed once (qd and dd: up
// to 4 waves, as many as LDS holds twice per compute unit).
template <class P, bool HALF>
int poly_launch_half(int batch, int neq, int nvar, int nmon, int nvpm, const int *vars, const int *exps,
                     const double *coef, const double *x, double *A, double *b, bool negate, hipStream_t st) {
  const int eq = HALF ? 2 : 1;
  const size_t table = nt_table_doubles(P::L, nvar) * sizeof(double);
  const size_t per_wave = nt_wave_doubles(P::L, nvpm) * sizeof(double);
  DevInfo d;
  const int cus = dev_info(d) && d.cus > 0 ? d.cus : 256;
  int waves = 1, neqb = eq;
  if ((long long)batch >= 2 * cus) {
    waves = ceil_div(neq, eq) < 4 ? ceil_div(neq, eq) : 4;
    while (waves > 1 && table + waves * per_wave > 80 * 1024) --waves;
    neqb = neq;
  } else {
    while (neqb < neq && (long long)batch * ceil_div(neq, neqb) > 8 * cus) neqb += eq;
  }
  const size_t shmem = table + waves * per_wave;
  auto kern = poly_eval_kernel<P, HALF>;
  if (shmem > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)shmem) != hipSuccess)
    return MGS_ERR_LAUNCH;
  hipLaunchKernelGGL(kern, dim3(ceil_div(neq, neqb), batch), dim3(64 * waves), shmem, st, neq, nvar, nmon, nvpm, vars,
                     exps, coef, x, A, b, neqb, negate);
  return hipGetLastError() == hipSuccess ? MGS_OK : MGS_ERR_LAUNCH;
}
template <class P>
int poly_launch(int batch, int neq, int nvar, int nmon, int nvpm, const int *vars, const int *exps, const double *coef,
                const double *x, double *A, double *b, bool negate, hipStream_t st) {
  return nmon <= 32 ? poly_launch_half<P, true>(batch, neq, nvar, nmon, nvpm, vars, exps, coef, x, A, b, negate, st)
                    : poly_launch_half<P, false>(batch, neq, nvar, nmon, nvpm, vars, exps, coef, x, A, b, negate, st);
}

template <class P>
int newton_launch(int batch, int neq, int nvar, int nmon, int nvpm, const int *vars, const int *exps,
                  const double *coef, double *x, int iters, double *dnorm, const NewtonWork &w, int *info,
                  long long wclk_khz, hipStream_t st) {
  for (int k = 0; k < iters; ++k) {
    const int pe = poly_launch<P>(batch, neq, nvar, nmon, nvpm, vars, exps, coef, x, w.A, w.b, true, st);
    if (pe != MGS_OK) return pe;
    if (w.qrw != nullptr) {
      // One point in qd: mgs_qr's left-looking launch, quicker than a batch of
      // one, then the back substitution, which adds a time-out to the
      // factorisation's status (a zero pivot is already there).
      int rc = mgs_qr_schedule(neq, nvar, P::L, w.A, neq, w.A, neq, w.R, nvar, w.b, w.y, nullptr, w.qrw, w.qrw_bytes,
                               info, MGS_SCHED_AUTO, reinterpret_cast<mgs_stream_t>(st));
      if (rc != MGS_OK) return rc;
      rc = trsv_launch<P>(nvar, w.R, nvar, w.y, w.d, info, st, true);
      if (rc != MGS_OK) return rc;
      hipLaunchKernelGGL((newton_update_kernel<P>), dim3(batch), dim3(64), 0, st, nvar, x, w.d, info,
                         dnorm != nullptr ? dnorm + (size_t)k * batch : nullptr);
      if (hipGetLastError() != hipSuccess) return MGS_ERR_LAUNCH;
      continue;
    }
    BatArgs a;
    a.batch = batch;
    a.m = neq;
    a.n = nvar;
    a.ncols = nvar + 1;
    a.A = w.A;
    a.lda = neq;
    a.b = w.b;
    a.Q = w.A;  // in place
    a.ldq = neq;
    a.R = w.R;
    a.ldr = nvar;
    a.y = nullptr;
    a.x = w.d;
    a.rho = nullptr;
    a.info = info;
    const WaitArgs wait = wait_args(wclk_khz);
    a.spin_ticks = wait.ticks;
    a.jitter = wait.jitter;
    const int rc = batched_dispatch(P::L, a, st);
    if (rc != MGS_OK) return rc;
    hipLaunchKernelGGL((newton_update_kernel<P>), dim3(batch), dim3(64), 0, st, nvar, x, w.d, info,
                       dnorm != nullptr ? dnorm + (size_t)k * batch : nullptr);
    if (hipGetLastError() != hipSuccess) return MGS_ERR_LAUNCH;
  }
  return MGS_OK;
}

}  // namespace

extern "C" {

void mgs_set_jitter(unsigned seed) { g_jitter.store(seed, std::memory_order_relaxed); }

void mgs_set_wait_limit(int launch, long long ticks) {
  t_limit_in = launch;
  t_limit_ticks = ticks;
}

#ifdef MGS_TRACE
// Diagnostic builds only (not declared in the public header).
void mgs_set_trace(long long *buf) { g_trace = buf; }
#endif

int mgs_abi_version(void) { return MGS_ABI_VERSION; }

const char *mgs_status_string(int status) {
  switch (status) {
    case MGS_OK: return "success";
    case MGS_ERR_DIMS: return "invalid dimensions (need 1 <= n <= m <= max rows, ld >= rows)";
    case MGS_ERR_POINTER: return "null, misaligned or illegally aliased pointer";
    case MGS_ERR_PREC: return "unsupported precision or block size";
    case MGS_ERR_WORKSPACE: return "workspace too small";
    case MGS_ERR_LAUNCH: return "kernel launch failed";
    case MGS_ERR_UNSUPPORTED: return "unsupported operation or schedule";
  }
  return "unknown status";
}

int mgs_workspace_size(int m, int n, int prec, int op, size_t *bytes) {
  if (op == MGS_OP_QR64 ? prec != 1
                        : (op == MGS_OP_QR || op == MGS_OP_SOLVE ? !prec_ok(prec) : (prec != 2 && prec != 4)))
    return MGS_ERR_PREC;
  if (n < 1 || m < n || m > (op == MGS_OP_QR64 ? MGS_MAX_ROWS_DD : max_rows(prec))) return MGS_ERR_DIMS;
  if (!bytes) return MGS_ERR_POINTER;
  switch (op) {
    case MGS_OP_QR: *bytes = qr_work_bytes(m, n, prec); return MGS_OK;
    case MGS_OP_SOLVE: *bytes = solve_work_bytes(n, prec); return MGS_OK;
    case MGS_OP_ADJOINT: *bytes = adjoint_work_bytes(m, n, prec); return MGS_OK;
    case MGS_OP_REFINE: *bytes = refine_layout(m, n, prec, nullptr).bytes; return MGS_OK;
    case MGS_OP_QR64: *bytes = qr64_work_bytes(m, n); return MGS_OK;
  }
  return MGS_ERR_UNSUPPORTED;
}

int mgs_qr_schedule(int m, int n, int prec, const double *A, int lda, double *Q, int ldq, double *R, int ldr,
                    const double *b, double *y, double *rho, void *work, size_t work_bytes, int *info,
                    int schedule, mgs_stream_t stream) {
  if (!prec_ok(prec)) return MGS_ERR_PREC;
  if (schedule < MGS_SCHED_AUTO || schedule > MGS_SCHED_SMALL) return MGS_ERR_UNSUPPORTED;
  if (n < 1 || m < n || m > max_rows(prec) || lda < m || ldq < m || ldr < n) return MGS_ERR_DIMS;
  if (!aligned8(A) || !aligned8(Q) || !aligned8(R) || !aligned8(info)) return MGS_ERR_POINTER;
  if (Q == A && ldq != lda) return MGS_ERR_POINTER;
  if (rho && !aligned8(rho)) return MGS_ERR_POINTER;
  if (!aligned8(work)) return MGS_ERR_POINTER;
  if (b && (!aligned8(b) || !aligned8(y))) return MGS_ERR_POINTER;
  if (work_bytes < qr_work_bytes(m, n, prec)) return MGS_ERR_WORKSPACE;
  Shape sh = choose_shape(m, prec, n + (b ? 1 : 0));
  StepArgs a;
  a.m = m;
  a.n = n;
  a.ncols = n + (b ? 1 : 0);
  a.A = A;
  a.lda = lda;
  a.planeA = (size_t)lda * n;
  a.b = b;
  a.Q = Q;
  a.ldq = ldq;
  a.planeQ = (size_t)ldq * n;
  a.R = R;
  a.ldr = ldr;
  a.planeR = (size_t)ldr * n;
  a.W = b ? static_cast<double *>(work) : nullptr;
  a.y = b ? y : nullptr;
  a.rho = b ? rho : nullptr;
  a.info = info;
  a.t = 0;
  a.kbase = 0;
  a.init_info = 1;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int mode = schedule;
  if (mode == MGS_SCHED_AUTO || mode == MGS_SCHED_SMALL) {
    int rc = 1;
    if (batched_fits(m, n, a.ncols, prec) && (prec <= 2 || mode == MGS_SCHED_SMALL)) {
      // Double and dd (and qd when asked for): the batched kernel on a batch
      // of one.
      DevInfo d;
      if (dev_info(d)) {
        BatArgs ba;
        ba.batch = 1;
        ba.m = m;
        ba.n = n;
        ba.ncols = a.ncols;
        ba.A = A;
        ba.lda = lda;
        ba.b = b;
        ba.Q = Q;
        ba.ldq = ldq;
        ba.R = R;
        ba.ldr = ldr;
        ba.y = a.y;
        ba.x = nullptr;
        ba.rho = a.rho;
        ba.info = info;
        const WaitArgs wait = wait_args(d.wclk_khz);
        ba.spin_ticks = wait.ticks;
        ba.jitter = wait.jitter;
        rc = batched_dispatch(prec, ba, st);
      }
    }
    if (rc != 1) return rc;
    if (mode == MGS_SCHED_SMALL) return MGS_ERR_DIMS;
  }
  if (mode == MGS_SCHED_AUTO || mode == MGS_SCHED_RESIDENT) {
    void *sync = static_cast<char *>(work) + qr_w_bytes(m, prec);
    double *u = reinterpret_cast<double *>(static_cast<char *>(sync) + sizeof(unsigned int) * RES_SYNC_WORDS);
    int rc = 1;
    if (qr_u_bytes(m, n, prec) > 0) rc = prec == 2 ? res_launch<PrecDD>(a, sync, u, st) : res_launch<PrecD>(a, sync, u, st);
    if (rc != 1) return rc;
    if (mode == MGS_SCHED_RESIDENT) return MGS_ERR_DIMS;
  }
  if (mode == MGS_SCHED_AUTO && prec == 4 && m <= 1024) return left_launch_qd(a, work, st);
  if (prec == 1) return dispatch_shape<PrecD>(a, sh, st);
  if (prec == 2) return dispatch_shape<PrecDD>(a, sh, st);
  return dispatch_shape<PrecQD>(a, sh, st);
}

int mgs_qr(int m, int n, int prec, const double *A, int lda, double *Q, int ldq, double *R, int ldr,
           const double *b, double *y, double *rho, void *work, size_t work_bytes, int *info,
           mgs_stream_t stream) {
  return mgs_qr_schedule(m, n, prec, A, lda, Q, ldq, R, ldr, b, y, rho, work, work_bytes, info, MGS_SCHED_AUTO,
                         stream);
}

int mgs_qr_noalloc(int m, int n, int prec, const double *A, int lda, double *Q, int ldq, double *R, int ldr,
                   const double *b, double *y, double *rho, int *info, mgs_stream_t stream) {
  if (!prec_ok(prec)) return MGS_ERR_PREC;
  if (n < 1 || m < n || m > max_rows(prec) || lda < m || ldq < m || ldr < n) return MGS_ERR_DIMS;
  const size_t need = qr_work_bytes(m, n, prec);
  if (need > MGS_NOALLOC_SCRATCH_BYTES) return MGS_ERR_WORKSPACE;
  void *work = scratch_address();
  if (work == nullptr) return MGS_ERR_LAUNCH;
  return mgs_qr_schedule(m, n, prec, A, lda, Q, ldq, R, ldr, b, y, rho, work, MGS_NOALLOC_SCRATCH_BYTES, info,
                         MGS_SCHED_AUTO, stream);
}

int ls_backsolve(int n, int prec, const double *R, int ldr, const double *y, double *x, int *info,
                 mgs_stream_t stream) {
  if (!prec_ok(prec)) return MGS_ERR_PREC;
  if (n < 1 || n > max_rows(prec) || ldr < n) return MGS_ERR_DIMS;
  if (!aligned8(R) || !aligned8(y) || !aligned8(x) || !aligned8(info)) return MGS_ERR_POINTER;
  if (x == y) return MGS_ERR_POINTER;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (prec == 1) return trsv_launch<PrecD>(n, R, ldr, y, x, info, st);
  if (prec == 2) return trsv_launch<PrecDD>(n, R, ldr, y, x, info, st);
  return trsv_launch<PrecQD>(n, R, ldr, y, x, info, st);
}

int ls_solve(int m, int n, int prec, const double *Q, int ldq, const double *R, int ldr,
             const double *b, double *x, void *work, size_t work_bytes, int *info,
             mgs_stream_t stream) {
  if (!prec_ok(prec)) return MGS_ERR_PREC;
  if (n < 1 || m < n || m > max_rows(prec) || ldq < m || ldr < n) return MGS_ERR_DIMS;
  if (!aligned8(Q) || !aligned8(R) || !aligned8(b) || !aligned8(x) || !aligned8(info) || !aligned8(work))
    return MGS_ERR_POINTER;
  if (work_bytes < solve_work_bytes(n, prec)) return MGS_ERR_WORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  double *y = static_cast<double *>(work);
  int rc = prec == 1   ? project_launch<PrecD>(m, n, Q, ldq, b, y, st)
           : prec == 2 ? project_launch<PrecDD>(m, n, Q, ldq, b, y, st)
                       : project_launch<PrecQD>(m, n, Q, ldq, b, y, st);
  if (rc != MGS_OK) return rc;
  if (prec == 1) return trsv_launch<PrecD>(n, R, ldr, y, x, info, st);
  if (prec == 2) return trsv_launch<PrecDD>(n, R, ldr, y, x, info, st);
  return trsv_launch<PrecQD>(n, R, ldr, y, x, info, st);
}

int ls_adjoint(int m, int n, int prec, const double *A, int lda, const double *b, const double *Q, int ldq,
               const double *R, int ldr, const double *x, const double *gx, double *gA, int ldga, double *gb,
               void *work, size_t work_bytes, int *info, mgs_stream_t stream) {
  if (prec != 2 && prec != 4) return MGS_ERR_PREC;
  if (n < 1 || m < n || m > max_rows(prec) || lda < m || ldq < m || ldr < n || ldga < m) return MGS_ERR_DIMS;
  if (!aligned8(A) || !aligned8(b) || !aligned8(Q) || !aligned8(R) || !aligned8(x) || !aligned8(gx) ||
      !aligned8(gA) || !aligned8(gb) || !aligned8(work) || !aligned8(info))
    return MGS_ERR_POINTER;
  if (gA == A || gA == Q || gb == b) return MGS_ERR_POINTER;
  if (work_bytes < adjoint_work_bytes(m, n, prec)) return MGS_ERR_WORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (prec == 2) return adjoint_launch<PrecDD>(m, n, A, lda, b, Q, ldq, R, ldr, x, gx, gA, ldga, gb, work, info, st);
  return adjoint_launch<PrecQD>(m, n, A, lda, b, Q, ldq, R, ldr, x, gx, gA, ldga, gb, work, info, st);
}

int mgs_refine_solve(int m, int n, int prec, const double *A, int lda, const double *b, double *x, int block,
                     double tol, int max_iter, int *iters, double *err_est, void *work, size_t work_bytes, int *info,
                     mgs_stream_t stream) {
  if (prec != 2 && prec != 4) return MGS_ERR_PREC;
  if (n < 1 || m < n || m > max_rows(prec) || lda < m || max_iter < 0) return MGS_ERR_DIMS;
  if (block != NBP) return MGS_ERR_PREC;
  if (!aligned8(A) || !aligned8(b) || !aligned8(x) || !aligned8(work) || !aligned8(info)) return MGS_ERR_POINTER;
  if (x == b || x == A) return MGS_ERR_POINTER;
  if (work_bytes < refine_layout(m, n, prec, nullptr).bytes) return MGS_ERR_WORKSPACE;
  if (!(tol >= 0.0)) return MGS_ERR_DIMS;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (prec == 2) return refine_solve<PrecDD>(m, n, A, lda, b, x, tol, max_iter, iters, err_est, work, info, st);
  return refine_solve<PrecQD>(m, n, A, lda, b, x, tol, max_iter, iters, err_est, work, info, st);
}

int mgs_qr64(int m, int n, const double *A, int lda, const double *b, double *Q, int ldq, double *R, int ldr,
             double *y, int block, void *work, size_t work_bytes, int *info, mgs_stream_t stream) {
  if (block != NBP) return MGS_ERR_PREC;
  if (n < 1 || m < n || m > MGS_MAX_ROWS_DD || lda < m || ldq < m || ldr < n) return MGS_ERR_DIMS;
  if (!aligned8(A) || !aligned8(Q) || !aligned8(R) || !aligned8(info) || !aligned8(work)) return MGS_ERR_POINTER;
  if (b != nullptr && (!aligned8(b) || !aligned8(y))) return MGS_ERR_POINTER;
  if (work_bytes < qr64_work_bytes(m, n)) return MGS_ERR_WORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  RefineWork w;
  w.Q64 = static_cast<double *>(work);
  w.R64 = reinterpret_cast<double *>(static_cast<char *>(work) + round256(sizeof(double) * 2 * (size_t)m * (n + 1)));
  w.res = panel_res_bytes(m, n) > 0 ? static_cast<char *>(work) + round256(sizeof(double) * 2 * (size_t)m * (n + 1)) +
                                          round256(sizeof(double) * 2 * (size_t)n * (n + 1))
                                    : nullptr;
  hipLaunchKernelGGL(copy64_in_kernel, dim3(ceil_div(m, 256), n + 1), dim3(256), 0, st, m, n, A, lda, b, w.Q64, info);
  if (hipGetLastError() != hipSuccess) return MGS_ERR_LAUNCH;
  const int rc = factor64(m, n, w, info, st);
  if (rc != MGS_OK) return rc;
  const int gx = ceil_div(m, 256) < 4 ? ceil_div(m, 256) : 4;
  hipLaunchKernelGGL(copy64_out_kernel, dim3(gx, n + 1), dim3(256), 0, st, m, n, w.Q64, w.R64, Q, ldq, R, ldr,
                     b != nullptr ? y : nullptr);
  return hipGetLastError() == hipSuccess ? MGS_OK : MGS_ERR_LAUNCH;
}

int mgs_poly_eval(int batch, int neq, int nvar, int nmon, int nvpm, int prec, const int *vars, const int *exps,
                  const double *coef, const double *x, double *J, double *F, mgs_stream_t stream) {
  if (!prec_ok(prec)) return MGS_ERR_PREC;
  if (batch < 0 || neq < 1 || neq > 65535 || nvar < 1 || nvar > NT_MAX_VARS || nmon < 1 || nmon > NT_MAX_MON ||
      nvpm < 1 || nvpm > NT_MAX_VPM || batch > 65535)
    return MGS_ERR_DIMS;
  if (batch == 0) return MGS_OK;
  if (!aligned8(coef) || !aligned8(x) || !aligned8(J) || !aligned8(F)) return MGS_ERR_POINTER;
  if (vars == nullptr || exps == nullptr || (reinterpret_cast<uintptr_t>(vars) & 3u) ||
      (reinterpret_cast<uintptr_t>(exps) & 3u))
    return MGS_ERR_POINTER;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (prec == 1) return poly_launch<PrecD>(batch, neq, nvar, nmon, nvpm, vars, exps, coef, x, J, F, false, st);
  if (prec == 2) return poly_launch<PrecDD>(batch, neq, nvar, nmon, nvpm, vars, exps, coef, x, J, F, false, st);
  return poly_launch<PrecQD>(batch, neq, nvar, nmon, nvpm, vars, exps, coef, x, J, F, false, st);
}

int mgs_newton_workspace_size(int batch, int neq, int nvar, int prec, size_t *bytes) {
  if (!prec_ok(prec)) return MGS_ERR_PREC;
  if (!newton_dims_ok(batch, neq, nvar, 1, 1, prec)) return MGS_ERR_DIMS;
  if (bytes == nullptr) return MGS_ERR_POINTER;
  *bytes = newton_layout(batch, neq, nvar, prec, nullptr).bytes;
  return MGS_OK;
}

int mgs_newton_batched(int batch, int neq, int nvar, int nmon, int nvpm, int prec, const int *vars, const int *exps,
                       const double *coef, double *x, int iters, double *dnorm, void *work, size_t work_bytes,
                       int *info, mgs_stream_t stream) {
  if (!prec_ok(prec)) return MGS_ERR_PREC;
  if (!newton_dims_ok(batch, neq, nvar, nmon, nvpm, prec) || iters < 0) return MGS_ERR_DIMS;
  if (batch == 0 || iters == 0) return MGS_OK;
  if (!aligned8(coef) || !aligned8(x) || !aligned8(work) || !aligned8(info)) return MGS_ERR_POINTER;
  if (vars == nullptr || exps == nullptr || (reinterpret_cast<uintptr_t>(vars) & 3u) ||
      (reinterpret_cast<uintptr_t>(exps) & 3u))
    return MGS_ERR_POINTER;
  if (dnorm != nullptr && !aligned8(dnorm)) return MGS_ERR_POINTER;
  const NewtonWork w = newton_layout(batch, neq, nvar, prec, work);
  if (work_bytes < w.bytes) return MGS_ERR_WORKSPACE;
  DevInfo d;
  if (!dev_info(d)) return MGS_ERR_LAUNCH;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (prec == 1)
    return newton_launch<PrecD>(batch, neq, nvar, nmon, nvpm, vars, exps, coef, x, iters, dnorm, w, info, d.wclk_khz,
                              st);
  if (prec == 2)
    return newton_launch<PrecDD>(batch, neq, nvar, nmon, nvpm, vars, exps, coef, x, iters, dnorm, w, info, d.wclk_khz,
                               st);
  return newton_launch<PrecQD>(batch, neq, nvar, nmon, nvpm, vars, exps, coef, x, iters, dnorm, w, info, d.wclk_khz,
                             st);
}

int mgs_lstsq_batched(int batch, int m, int n, int prec, const double *A, int lda, const double *b, double *Q,
                      int ldq, double *R, int ldr, double *y, double *x, double *rho, int *info,
                      mgs_stream_t stream) {
  if (!prec_ok(prec)) return MGS_ERR_PREC;
  const int ncols = n + (b ? 1 : 0);
  if (batch < 0 || n < 1 || m < n || lda < m || ldq < m || ldr < n) return MGS_ERR_DIMS;
  if (!batched_fits(m, n, ncols, prec)) return MGS_ERR_DIMS;
  if (batch == 0) return MGS_OK;  // nothing is read or written (empty tensors may have null pointers)
  if (!aligned8(A) || !aligned8(Q) || !aligned8(R) || !aligned8(info)) return MGS_ERR_POINTER;
  if (Q == A && ldq != lda) return MGS_ERR_POINTER;
  if (b != nullptr) {
    if (!aligned8(b) || (y == nullptr && x == nullptr)) return MGS_ERR_POINTER;
    if ((y != nullptr && !aligned8(y)) || (x != nullptr && !aligned8(x)) || (x != nullptr && x == y))
      return MGS_ERR_POINTER;
    if (rho != nullptr && !aligned8(rho)) return MGS_ERR_POINTER;
  }
  DevInfo d;
  if (!dev_info(d)) return MGS_ERR_LAUNCH;
  BatArgs a;
  a.batch = batch;
  a.m = m;
  a.n = n;
  a.ncols = ncols;
  a.A = A;
  a.lda = lda;
  a.b = b;
  a.Q = Q;
  a.ldq = ldq;
  a.R = R;
  a.ldr = ldr;
  a.y = b ? y : nullptr;
  a.x = b ? x : nullptr;
  a.rho = b ? rho : nullptr;
  a.info = info;
  const WaitArgs wait = wait_args(d.wclk_khz);
  a.spin_ticks = wait.ticks;
  a.jitter = wait.jitter;
  return batched_dispatch(prec, a, reinterpret_cast<hipStream_t>(stream));
}

}  // extern "C"
