// Triangular solves: the back substitution of Section 6, Figure 3 (for
// k = n..1, x_k = y_k / r_kk, then y_j -= r_jk x_k for j < k) and its mirror
// image, the forward substitution R^H w = g of the adjoint.
//
// A lane holds one part (real or imaginary) of one row of y, so a wave
// holds 32 rows and a step costs it half the operations of a complex row
// per lane; a workgroup is a block of up to 4 waves (128 rows), one per SIMD:
// a wave that absorbs columns must keep up with the one that solves, and two
// on a SIMD do not (dd n = 1024: 481 us with 8 waves, 320 with 4).  Each wave
// applies r_ic x_c to its rows for every column c solved before its own, in
// solve order, as x_c appears, then solves its own 32 columns: the lanes of
// row c form x_c (times the reciprocal of r_cc, formed up front), all lanes
// get it by readlane, and the rows it reaches receive r_ic x_c.  So every
// y_i receives its products in the order of the column-oriented loop.
//
// What bounds it is that chain: one multiply, one broadcast and one update
// per column.  x_c goes to the waves of the same workgroup through LDS and
// to the other workgroups through x itself (device-scope stores), both
// filled with the empty marker (a signalling NaN, which no arithmetic
// produces) beforehand, so that readers poll the data.  The entries of R are
// loaded RING columns ahead.  Every wait is bounded by a wall-clock limit
// (MGS_INFO_SYNC_TIMEOUT in info).  A launch of several workgroups is
// cooperative (all resident); one workgroup can also take all blocks in
// turn.
#pragma once
#include "../../include/mgsqr.h"
#include "resident_kernels.hpp"

namespace mgsq {

constexpr int TS_ROWS = 32;   // rows of a wave
constexpr int TS_WAVES = 4;   // waves of a workgroup, at most: one per SIMD
constexpr int TS_BLOCK = TS_ROWS * TS_WAVES;

// Race checks; with TS_STALL (tests of the time-out paths) about 100 us a step,
// so that the waits on a wave last longer than 16 turns.
constexpr unsigned TS_STALL = 0x57A11ED0u;
__device__ __forceinline__ void trsv_pause(unsigned seed, unsigned step) {
  if (seed == 0) return;
  res_jitter(seed, step);
  if (seed == TS_STALL)
    for (int i = 0; i < 32; ++i) __builtin_amdgcn_s_sleep(127);
}

// x := empty marker (all planes), info := 0 unless keep; nothing when
// *skip != 0.
template <int L>
__global__ __launch_bounds__(256) void bs_mark_kernel(int n, double *x, int *info, int keep, const int *skip) {
  if (skip != nullptr && *skip != 0) return;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i == 0 && info != nullptr && !keep) *info = 0;
  if (i < n) {
#pragma unroll
    for (int p = 0; p < 2 * L; ++p) x[i + (size_t)p * n] = __longlong_as_double(RES_EMPTY);
  }
}

// FWD = false: R x = y (columns descending, rows above the pivot updated).
// FWD = true: R^H x = y (columns ascending, entry (i, c) of R^H is
// conj(r_ci), rows below the pivot updated).  Workgroup g takes the blocks
// g, g + G, ... of blockDim / 2 rows in solve order; marked: x holds the
// empty marker (needed for more than one block), else the one block clears
// info itself.  keep: info stays as it is unless this solve has something to
// report (a time-out, or a bad diagonal entry where it was 0 or a later one).
template <class P, bool FWD>
__global__ __launch_bounds__(64 * TS_WAVES) void trsv_kernel(int n, const double *R, int ldr, size_t planeR,
                                                             const double *y, size_t planeY, double *x, int *info,
                                                             int keep, const int *skip, int marked,
                                                             long long spin_ticks, unsigned jitter) {
  if (skip != nullptr && *skip != 0) return;
  using Rl = typename P::R;
  constexpr int L = P::L, DIR = FWD ? 1 : -1;
  constexpr int RING = L == 4 ? 4 : 8;  // columns of R loaded ahead
  __shared__ double xs[2 * L][TS_BLOCK];  // the block's x, [plane][row], empty until solved
  // the wave's number as a scalar, so that all addresses of a step but the
  // lane's row are scalar arithmetic
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, part = lane & 1;
  const int nwave = blockDim.x >> 6, rows = nwave * TS_ROWS;
  const int nblk = (n + rows - 1) / rows;
  if (!marked && tid == 0 && info != nullptr && !keep) *info = 0;
  for (int b = blockIdx.x; b < nblk; b += gridDim.x) {
    const int r0 = (FWD ? b : nblk - 1 - b) * rows, r1 = min(r0 + rows, n);  // the block
    __syncthreads();
    for (int i = tid; i < 2 * L * TS_BLOCK; i += blockDim.x) (&xs[0][0])[i] = __longlong_as_double(RES_EMPTY);
    __syncthreads();
    const int w0 = r0 + wave * TS_ROWS, w1 = min(w0 + TS_ROWS, n);  // the wave's rows
    if (w0 >= n) continue;
    const int i = w0 + (lane >> 1);
    const bool mine = i < w1;
    const int ic = mine ? i : n - 1;  // clamped row for loads
    // Column c's entry of row i as this lane's factors of Re x_c and Im x_c:
    // (re, -im) for the real part, (im, re) for the imaginary one, of the
    // conjugate when FWD.  Rows that a column does not reach
    // (already solved) take the update too: their y is no longer used.
    struct Entry {
      Rl a, b;
    };
    const double *pa = R + (size_t)part * planeR + (FWD ? (size_t)ic * ldr : (size_t)ic);
    const double *pb = R + (size_t)(1 - part) * planeR + (FWD ? (size_t)ic * ldr : (size_t)ic);
    const unsigned long long neg = 1ull << 63;
    const unsigned long long na = FWD && part == 1 ? neg : 0, nb = !FWD && part == 0 ? neg : 0;
    auto rload = [&](int c) __attribute__((always_inline)) {
      const int cl = FWD ? min(c, n - 1) : max(c, 0);  // loads run past the last column
      const size_t at = FWD ? (size_t)cl : (size_t)cl * ldr;
      Entry e;
      double *ea = reinterpret_cast<double *>(&e.a), *eb = reinterpret_cast<double *>(&e.b);
#pragma unroll
      for (int l = 0; l < L; ++l) {
        ea[l] = pa[at + (size_t)(2 * l) * planeR];
        eb[l] = pb[at + (size_t)(2 * l) * planeR];
      }
      return e;
    };
    auto flip = [&](const Rl &v, unsigned long long bits) __attribute__((always_inline)) {
      Rl r;
      double *pr = reinterpret_cast<double *>(&r);
      const double *pv = reinterpret_cast<const double *>(&v);
#pragma unroll
      for (int l = 0; l < L; ++l) pr[l] = __longlong_as_double(__double_as_longlong(pv[l]) ^ bits);
      return r;
    };
    auto update = [&](Rl &v, const Entry &e, const Rl &xr, const Rl &xi) __attribute__((always_inline)) {
      P::upd_part(v, FWD ? flip(e.a, na) : e.a, xr, FWD ? e.b : flip(e.b, nb), xi);
    };
    Rl yv, xown;  // y_i and, once solved, x_i (the empty marker before)
    {
      double *pv = reinterpret_cast<double *>(&yv), *px = reinterpret_cast<double *>(&xown);
#pragma unroll
      for (int l = 0; l < L; ++l) {
        pv[l] = y[ic + (size_t)(2 * l + part) * planeY];
        px[l] = __longlong_as_double(RES_EMPTY);
      }
    }
    const Rl dg = P::load(R + (size_t)ic * ldr + ic, planeR).re;
    Rl inv = P::recip(dg);
    if (!mine) {
      yv = P::rzero();
      inv = P::rzero();
    }
    if (mine && part == 0 && !P::ok_norm(dg) && info != nullptr) info_first_bad(info, i + 1);
    const int own = FWD ? w0 : w1 - 1;  // first own column
    Entry rd[RING];
#pragma unroll
    for (int t = 0; t < RING; ++t) rd[t] = rload(own + DIR * t);

    // Columns c1, c1 + DIR, ... (count of them), x from `at(column)`, the
    // address of its first limb with planes `plane` apart; in chunks of 32:
    // lane 2 j + p holds part p of the chunk's column j, once it is there.
    auto absorb = [&](int c1, int count, auto at, size_t plane) __attribute__((always_inline)) {
      if (count <= 0) return true;
      Entry ra[RING];
#pragma unroll
      for (int t = 0; t < RING; ++t) ra[t] = rload(c1 + DIR * t);
#pragma unroll 1
      for (int s0 = 0; s0 < count; s0 += TS_ROWS) {
        trsv_pause(jitter, (unsigned)s0);
        const int s = min(s0 + (lane >> 1), count - 1);
        const double *src = at(c1 + DIR * s);
        Rl v = P::rzero();
        int avail = 0;  // columns of the chunk that are there
        PollBound poll;
        auto wait_col = [&](int j) __attribute__((always_inline)) {
          while (avail <= j) {
            double *pv = reinterpret_cast<double *>(&v);
            bool miss = false;
#pragma unroll
            for (int l = 0; l < L; ++l) {
              pv[l] = coh_load(src + (size_t)(2 * l + part) * plane);
              miss = miss || __double_as_longlong(pv[l]) == RES_EMPTY;
            }
            const unsigned long long gone = __ballot(miss);
            avail = gone == 0 ? TS_ROWS : (__ffsll((long long)gone) - 1) >> 1;
            if (avail > j) return true;
            if (poll.due() && poll.late(spin_ticks)) {
              if (lane == 0 && info != nullptr)
                __hip_atomic_store(info, MGS_INFO_SYNC_TIMEOUT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              return false;
            }
            __builtin_amdgcn_s_sleep(1);
          }
          return true;
        };
#pragma unroll 1
        for (int j0 = 0; j0 < TS_ROWS && s0 + j0 < count; j0 += RING) {
#pragma unroll
          for (int t = 0; t < RING; ++t) {
            const int j = j0 + t;
            if (s0 + j < count) {
              if (!wait_col(j)) return false;
              update(yv, ra[t], wave_readlane(v, 2 * j), wave_readlane(v, 2 * j + 1));
            }
            ra[t] = rload(c1 + DIR * (s0 + j + RING));
          }
        }
      }
      return true;
    };
    // 1. Columns solved by other blocks, then by the block's other waves.
    if (!absorb(FWD ? 0 : n - 1, FWD ? r0 : n - r1,
                [&](int c) __attribute__((always_inline)) { return (const double *)(x + c); }, (size_t)n))
      return;
    if (!absorb(FWD ? r0 : r1 - 1, FWD ? w0 - r0 : r1 - w1,
                [&](int c) __attribute__((always_inline)) { return (const double *)(&xs[0][c - r0]); },
                (size_t)TS_BLOCK))
      return;
    // 2. The wave's own columns, ahead of the waves that share its SIMD.
    // Every lane writes its x, solved or not, every 4 columns (LDS) and every
    // RING (x): no branch, so the loads in flight stay counted.
    __builtin_amdgcn_s_setprio(3);
    const int ncol = w1 - w0;
    const double *px = reinterpret_cast<const double *>(&xown);
#pragma unroll 1
    for (int s0 = 0; s0 < ncol; s0 += RING) {
      trsv_pause(jitter, 0x10000u + (unsigned)s0);
#pragma unroll
      for (int t = 0; t < RING; ++t) {
        const int c = own + DIR * (s0 + t), k = c - w0;  // k outside [0, ncol) past the block
        const Rl xl = P::rmul(yv, inv);
        const Rl xr = wave_readlane(xl, (2 * k) & 63), xi = wave_readlane(xl, (2 * k + 1) & 63);
        update(yv, rd[t], xr, xi);
        xown = lane_pick((lane >> 1) == k, xl, xown);
        if (t % 4 == 3) {
#pragma unroll
          for (int l = 0; l < L; ++l)
            __hip_atomic_store(&xs[2 * l + part][wave * TS_ROWS + (lane >> 1)], px[l], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        rd[t] = rload(c + DIR * RING);
      }
      if (mine) {
#pragma unroll
        for (int l = 0; l < L; ++l) coh_store(x + i + (size_t)(2 * l + part) * n, px[l]);
      }
    }
    __builtin_amdgcn_s_setprio(0);
  }
}

}  // namespace mgsq
