// Device arithmetic for the MGS kernels: double-double (dd, 2 FP64 limbs)
// and quad-double (qd, 4 FP64 limbs) complex numbers (paper, Section 1:
// extended precision as unevaluated sums of hardware doubles, after Dekker
// 1971 and Priest 1992; Section 4 for the complex cost).
//
// Everything is built from three error-free transformations: TwoSum
// (Knuth), FastTwoSum (Dekker) and TwoProd through the hardware FMA.  All
// code must be compiled with -ffp-contract=off so that each + - * is
// rounded on its own.
//
// The hot operations are fused rather than composed from scalar dd ops:
//  * inner-product accumulation keeps, per real component, the exact running
//    sum S of the leading limb products (TwoProd + TwoSum) and one FP64 word
//    C that gathers every lower-order term: the TwoProd and TwoSum errors and
//    the hi*lo cross products.  (S, C) is renormalised once, after the
//    reduction.  Error per component below about (2k+6) u^2 sum|q_i||a_i|
//    for k terms, u = 2^-53: the classical inner-product bound in twice the
//    working precision.
//  * the column update a - r q forms the two leading products exactly,
//    sums them into a_hi with TwoSum and collects the rest in one word;
//    error below about 8 u^2 (|a| + |r||q|), the classical axpy bound.
// qd numbers use level-structured sums: terms of magnitude ~u^k |x| are
// added at level k with TwoSum, the carries moved to level k+1, level 3 is
// summed in plain FP64.  Sums of products (inner products, the column
// update) stay in such level words until the end, with a fifth one for the
// rounding of level 3: no renormalisation between terms, one two-pass TwoSum
// distillation when the value is needed.
// Error below a small multiple of 2^-209 relative to the operands.
#pragma once
#include <hip/hip_runtime.h>

namespace mgsq {

// ------------------------------------------------------------------ EFTs --
__device__ __forceinline__ void two_sum(double a, double b, double &s, double &e) {
  s = a + b;
  double v = s - a;
  e = (a - (s - v)) + (b - v);
}
// Exact when exponent(a) >= exponent(b).
__device__ __forceinline__ void fast_two_sum(double a, double b, double &s, double &e) {
  s = a + b;
  e = b - (s - a);
}
__device__ __forceinline__ void two_prod(double a, double b, double &p, double &e) {
  p = a * b;
  e = __fma_rn(a, b, -p);
}

// --------------------------------------------------------------------- dd --
struct dd {
  double h, l;
};
struct cdd {
  dd re, im;
};

// Accurate dd + dd: both limb pairs summed exactly, carries folded in twice.
__device__ __forceinline__ dd dd_add(dd a, dd b) {
  double s, e, t, f;
  two_sum(a.h, b.h, s, e);
  two_sum(a.l, b.l, t, f);
  e += t;
  fast_two_sum(s, e, s, e);
  e += f;
  fast_two_sum(s, e, s, e);
  return {s, e};
}
// dd * dd: exact leading product, both cross terms through FMA.
__device__ __forceinline__ dd dd_mul(dd a, dd b) {
  double p, e;
  two_prod(a.h, b.h, p, e);
  e = __fma_rn(a.h, b.l, e);
  e = __fma_rn(a.l, b.h, e);
  fast_two_sum(p, e, p, e);
  return {p, e};
}
// 1/b by one Newton step from the FP64 reciprocal: x + x (1 - b x).
__device__ __forceinline__ dd dd_recip(dd b) {
  double x = 1.0 / b.h;
  // residual 1 - b x formed with FMA: exact for the hi limb
  double r = __fma_rn(-b.h, x, 1.0);
  r = __fma_rn(-b.l, x, r);
  double s, e;
  fast_two_sum(x, x * r, s, e);
  return {s, e};
}
// sqrt(s) for s > 0 by one Newton step of the FP64 square root:
// x + (s - x^2) / (2x), the residual from the exact square of x.
__device__ __forceinline__ dd dd_sqrt(dd s) {
  double x = sqrt(s.h);
  double p, e;
  two_prod(x, x, p, e);
  double d = ((s.h - p) - e) + s.l;  // s.h - p is exact (Sterbenz)
  double hs, hl;
  fast_two_sum(x, d * (0.5 / x), hs, hl);
  return {hs, hl};
}

// sqrt(s) and 1/sqrt(s) together from one FP64 square root and one FP64
// division: the root as in dd_sqrt (0.5/x is exactly half of 1/x), the
// inverse by one Newton step on the dd root started from 1/x, so the two
// results share their slow operations instead of chaining them.
__device__ __forceinline__ void dd_sqrt_recip(dd s, dd &root, dd &inv) {
  const double x = sqrt(s.h);
  const double y = 1.0 / x;
  double p, e;
  two_prod(x, x, p, e);
  const double d = ((s.h - p) - e) + s.l;
  fast_two_sum(x, d * (0.5 * y), root.h, root.l);
  double r = __fma_rn(-root.h, y, 1.0);
  r = __fma_rn(-root.l, y, r);
  fast_two_sum(y, y * r, inv.h, inv.l);
}

// ------------------------------------------------------------------- qd --
struct qd {
  double x0, x1, x2, x3;
};
struct cqd {
  qd re, im;
};

// Error-free two-pass distillation of four terms of decreasing magnitude
// into four limbs: the bottom-up TwoSum chain yields the leading double and
// three exact remainders, which are distilled again the same way.
__device__ __forceinline__ qd qd_renorm(double a0, double a1, double a2, double a3) {
  double s, e1, e2, e3, y0;
  two_sum(a2, a3, s, e3);
  two_sum(a1, s, s, e2);
  two_sum(a0, s, y0, e1);
  double f1, f2, y1;
  two_sum(e2, e3, s, f2);
  two_sum(e1, s, y1, f1);
  double y2, y3;
  two_sum(f1, f2, y2, y3);
  return {y0, y1, y2, y3};
}

// Five level words into four limbs: a third pass folds the fifth word in
// below the third limb instead of rounding it into the fourth word.
__device__ __forceinline__ qd qd_renorm5(double a0, double a1, double a2, double a3, double a4) {
  double s, y0, y1, y2, e1, e2, e3, e4, f1, f2, f3, g1, g2;
  two_sum(a3, a4, s, e4);
  two_sum(a2, s, s, e3);
  two_sum(a1, s, s, e2);
  two_sum(a0, s, y0, e1);
  two_sum(e3, e4, s, f3);
  two_sum(e2, s, s, f2);
  two_sum(e1, s, y1, f1);
  two_sum(f2, f3, s, g2);
  two_sum(f1, s, y2, g1);
  return {y0, y1, y2, g1 + g2};
}

__device__ __forceinline__ qd qd_add(qd a, qd b) {
  double s0, e0, s1, e1, s2, e2, s3, e3;
  two_sum(a.x0, b.x0, s0, e0);
  two_sum(a.x1, b.x1, s1, e1);
  two_sum(a.x2, b.x2, s2, e2);
  two_sum(a.x3, b.x3, s3, e3);
  // level 1: s1 + e0
  double t1, c1;
  two_sum(s1, e0, t1, c1);
  // level 2: s2 + e1 + c1
  double t2, c2, c3;
  two_sum(s2, e1, t2, c2);
  two_sum(t2, c1, t2, c3);
  // level 3 in FP64
  double t3 = ((s3 + e2) + (c2 + c3)) + e3;
  return qd_renorm(s0, t1, t2, t3);
}
__device__ __forceinline__ qd qd_neg(qd a) { return {-a.x0, -a.x1, -a.x2, -a.x3}; }

// The sum of the level-3 terms of a b and of its level-4 products in plain
// FP64, the smallest first.
__device__ __forceinline__ double qd_low_products(const qd &a, const qd &b) {
  double t = a.x1 * b.x3;
  t = __fma_rn(a.x2, b.x2, t);
  t = __fma_rn(a.x3, b.x1, t);
  t = __fma_rn(a.x0, b.x3, t);
  t = __fma_rn(a.x1, b.x2, t);
  t = __fma_rn(a.x2, b.x1, t);
  return __fma_rn(a.x3, b.x0, t);
}

// The level words of a product or of a b + c d, not renormalised.  Level 3
// in up to three words (the products of two factors, the carries out of
// level 2), each rounded at its own size, for sums that take them exactly.
struct qdprod {
  double x0, x1, x2, x3, y3, z3;
};
__device__ __forceinline__ qdprod qd_mul_levels(const qd &a, const qd &b) {
  // level 0 / 1 / 2 products split exactly
  double p00, q00, p01, q01, p10, q10, p02, q02, p11, q11, p20, q20;
  two_prod(a.x0, b.x0, p00, q00);
  two_prod(a.x0, b.x1, p01, q01);
  two_prod(a.x1, b.x0, p10, q10);
  two_prod(a.x0, b.x2, p02, q02);
  two_prod(a.x1, b.x1, p11, q11);
  two_prod(a.x2, b.x0, p20, q20);
  // level 1
  double s1, r1, r2;
  two_sum(p01, p10, s1, r1);
  two_sum(s1, q00, s1, r2);
  // level 2
  double s2, u1, u2, u3, u4, u5, u6;
  two_sum(p02, p11, s2, u1);
  two_sum(s2, p20, s2, u2);
  two_sum(s2, q01, s2, u3);
  two_sum(s2, q10, s2, u4);
  two_sum(s2, r1, s2, u5);
  two_sum(s2, r2, s2, u6);
  // level 3
  double s3 = qd_low_products(a, b);
  s3 += (q02 + q11) + (q20 + u1);
  return {p00, s1, s2, s3, (u2 + u3) + (u4 + (u5 + u6)), 0.0};
}
__device__ __forceinline__ qd qd_mul(const qd &a, const qd &b) {
  const qdprod m = qd_mul_levels(a, b);
  return qd_renorm(m.x0, m.x1, m.x2, m.x3 + m.y3);
}

// a b + c d, one part of a complex product: 190 operations.
__device__ __forceinline__ qdprod qd_dot2(const qd &a, const qd &b, const qd &c, const qd &d) {
  const qdprod m = qd_mul_levels(a, b);
  double p00, q00, p01, q01, p10, q10, p02, q02, p11, q11, p20, q20, s0, s1, s2, c0, d1, d2, d3, d4;
  two_prod(c.x0, d.x0, p00, q00);
  two_prod(c.x0, d.x1, p01, q01);
  two_prod(c.x1, d.x0, p10, q10);
  two_prod(c.x0, d.x2, p02, q02);
  two_prod(c.x1, d.x1, p11, q11);
  two_prod(c.x2, d.x0, p20, q20);
  two_sum(m.x0, p00, s0, c0);
  // level 1
  two_sum(m.x1, p01, s1, d1);
  two_sum(s1, p10, s1, d2);
  two_sum(s1, q00, s1, d3);
  two_sum(s1, c0, s1, d4);
  // level 2
  double e1, e2, e3, e4, e5, e6, e7, e8, e9;
  two_sum(m.x2, p02, s2, e1);
  two_sum(s2, p11, s2, e2);
  two_sum(s2, p20, s2, e3);
  two_sum(s2, q01, s2, e4);
  two_sum(s2, q10, s2, e5);
  two_sum(s2, d1, s2, e6);
  two_sum(s2, d2, s2, e7);
  two_sum(s2, d3, s2, e8);
  two_sum(s2, d4, s2, e9);
  // level 3
  double t = qd_low_products(c, d);
  t += (q02 + q11) + q20;
  return {s0, s1, s2, m.x3 + m.y3, t, (e1 + ((e2 + e3) + (e4 + e5))) + ((e6 + e7) + (e8 + e9))};
}
// The level words of a^2 (the symmetric products formed once from 2 a_i).
__device__ __forceinline__ qd qd_sqr_levels(const qd &a) {
  const double t0 = 2.0 * a.x0, t1 = 2.0 * a.x1;
  double p00, q00, p01, q01, p02, q02, p11, q11, s1, r1, s2, u1, u2, u3;
  two_prod(a.x0, a.x0, p00, q00);
  two_prod(t0, a.x1, p01, q01);
  two_prod(t0, a.x2, p02, q02);
  two_prod(a.x1, a.x1, p11, q11);
  two_sum(p01, q00, s1, r1);
  two_sum(p02, p11, s2, u1);
  two_sum(s2, q01, s2, u2);
  two_sum(s2, r1, s2, u3);
  double t = a.x2 * a.x2;
  t = __fma_rn(t1, a.x3, t);
  t = __fma_rn(t0, a.x3, t);
  t = __fma_rn(t1, a.x2, t);
  t += (q02 + q11) + (u1 + (u2 + u3));
  return {p00, s1, s2, t};
}

// A sum of qd terms given by level words: one word per level, the carries
// out of levels 0 to 3 exact, level 4 in plain FP64, never renormalised on
// the way.  The next term only waits for one addition per level (a
// renormalised sum is a chain of about 60).
struct qdsum {
  double x0, x1, x2, x3, x4;
};
__device__ __forceinline__ void qd_acc(qdsum &a, const qd &b) {
  double c, d1, d2, e1, e2, e3, f, g;
  two_sum(a.x0, b.x0, a.x0, c);
  two_sum(a.x1, b.x1, a.x1, d1);
  two_sum(a.x1, c, a.x1, d2);
  two_sum(a.x2, b.x2, a.x2, e1);
  two_sum(a.x2, d1, a.x2, e2);
  two_sum(a.x2, d2, a.x2, e3);
  two_sum(a.x3, b.x3, a.x3, f);
  two_sum(a.x3, e1 + (e2 + e3), a.x3, g);
  a.x4 += f + g;
}
__device__ __forceinline__ void qd_acc(qdsum &a, const qdprod &b) {
  double f, g;
  two_sum(a.x3, b.y3, a.x3, f);
  two_sum(a.x3, b.z3, a.x3, g);
  a.x4 += f + g;
  qd_acc(a, qd{b.x0, b.x1, b.x2, b.x3});
}
// a += b, level by level (symmetric in a and b: the same bits either way).
__device__ __forceinline__ void qd_merge(qdsum &a, const qdsum &b) {
  const double l = a.x4 + b.x4;
  a.x4 = 0.0;
  qd_acc(a, qd{b.x0, b.x1, b.x2, b.x3});
  a.x4 += l;
}
__device__ __forceinline__ qdsum qd_sum_from(const qd &v) { return {v.x0, v.x1, v.x2, v.x3, 0.0}; }
// The sum's value in four limbs.  When whole levels cancelled against each
// other the distillation leaves words of similar size; such a value (rare:
// a cancellation of more than about 50 bits) is swept from the top, one
// level per sweep, until its leading limb is the rounded value.
__device__ __forceinline__ qd qd_value(const qdsum &s) {
  qd y = qd_renorm5(s.x0, s.x1, s.x2, s.x3, s.x4);
  if (fabs(y.x1) > 0x1p-53 * fabs(y.x0)) {
#pragma unroll 1
    for (int i = 0; i < 4; ++i) {
      two_sum(y.x0, y.x1, y.x0, y.x1);
      two_sum(y.x1, y.x2, y.x1, y.x2);
      two_sum(y.x2, y.x3, y.x2, y.x3);
    }
  }
  return y;
}
__device__ __forceinline__ qd qd_from(double a) { return {a, 0.0, 0.0, 0.0}; }

// c - a b for a product within a relative 2^-50 of c, as three words: the
// levels cancel exactly in the sum, what is left is good to about
// 2^-214 |c|.
struct td {
  double h, l, ll;
};
__device__ __forceinline__ td qd_residual(const qd &c, const qd &a, const qd &b) {
  qdsum r = qd_sum_from(c);
  qd_acc(r, qd_mul_levels(qd_neg(a), b));
  const qd v = qd_renorm5(r.x0, r.x1, r.x2, r.x3, r.x4);
  // after the cancellation its leading words may overlap
  td d;
  double t;
  two_sum(v.x0, v.x1, d.h, t);
  two_sum(t, v.x2, d.l, t);
  d.ll = t + v.x3;
  return d;
}

// v + v c for a correction c of at most about 2^-100.
__device__ __forceinline__ qd qd_correct(const qd &v, const td &c) {
  double p, q, p1, q1, p2, q2;
  two_prod(v.x0, c.h, p, q);
  two_prod(v.x0, c.l, p1, q1);
  two_prod(v.x1, c.h, p2, q2);
  qdsum r = qd_sum_from(v);
  qd_acc(r, qdprod{0.0, 0.0, p, q, p1, p2});
  r.x4 += __fma_rn(v.x0, c.ll, __fma_rn(v.x1, c.l, __fma_rn(v.x2, c.h, q1 + q2)));
  return qd_renorm5(r.x0, r.x1, r.x2, r.x3, r.x4);
}
// 1/b from the dd reciprocal y (about 2^-104): with e = 1 - b y, formed
// once, 1/b = y / (1 - e) = y (1 + e + e^2 + O(e^3)).
__device__ __forceinline__ qd qd_recip(const qd &b) {
  const dd r = dd_recip({b.x0, b.x1});
  const qd y = {r.h, r.l, 0.0, 0.0};
  const td e = qd_residual(qd_from(1.0), b, y);
  return qd_correct(y, {e.h, e.l, __fma_rn(e.h, e.h, e.ll)});
}
// Inverse square root of s > 0 to about 2^-103, as a dd: one Newton step
// y + y (1 - s y^2) / 2 from the FP64 one, whose relative error (about
// 2^-52) it squares.  The step only needs dd precision: s enters through
// its two leading limbs, y^2 exactly (TwoProd), 1 - s y^2 is about 2^-52
// (its leading difference exact by Sterbenz), so one FP64 product of it
// with y is accurate to about 2^-105 relative to y.
__device__ __forceinline__ dd qd_rsqrt_dd(const qd &s) {
  const double y = 1.0 / sqrt(s.x0);
  double t, te;
  two_prod(y, y, t, te);
  const dd u = dd_mul({s.x0, s.x1}, {t, te});
  const double r = (1.0 - u.h) - u.l;
  dd out;
  fast_two_sum(y, 0.5 * (y * r), out.h, out.l);
  return out;
}
// sqrt(s) and 1/sqrt(s) together, s > 0, from the dd inverse square root y
// and x = s y: with e = 1 - x y (about 2^-102, formed once) both are their
// first values times (1 - e)^(-1/2) = 1 + e/2 + 3 e^2 / 8 + O(e^3), so one
// residual serves the two and the chain is one product, one residual and
// one correction long.
__device__ __forceinline__ void qd_sqrt_recip(const qd &s, qd &root, qd &inv) {
  const dd y1 = qd_rsqrt_dd(s);
  const qd y = {y1.h, y1.l, 0.0, 0.0};
  const qd x = qd_mul(s, y);
  const td e = qd_residual(qd_from(1.0), x, y);
  const td c = {0.5 * e.h, 0.5 * e.l, __fma_rn(0.375 * e.h, e.h, 0.5 * e.ll)};
  root = qd_correct(x, c);
  inv = qd_correct(y, c);
}
__device__ __forceinline__ qd qd_sqrt(const qd &s) {
  qd root, inv;
  qd_sqrt_recip(s, root, inv);
  return root;
}

// --------------------------------------------------------- precisions ----
// A precision policy gathers what the kernels need: planar load / store,
// accumulators for inner products and norms with their wave shuffles, the
// fused column update, scaling by a real, and sqrt / reciprocal.
// Planar layout: limb l of the real / imaginary part lives in plane 2l / 2l+1.

struct PrecDD {
  static constexpr int L = 2;
  using R = dd;
  using C = cdd;
  struct Acc {
    double sr, cr, si, ci;  // exact leading sum and low-order word, re / im
  };
  // One part of an Acc (the real part is its first half).
  struct RAcc {
    double s, c;
  };
  __device__ static __forceinline__ void racc_merge(RAcc &a, const RAcc &b) {
    double t;
    two_sum(a.s, b.s, a.s, t);
    a.c = (a.c + b.c) + t;
  }
  __device__ static __forceinline__ R racc_value(const RAcc &a) {
    R v;
    two_sum(a.s, a.c, v.h, v.l);
    return v;
  }

  __device__ static __forceinline__ C load(const double *p, size_t plane) {
    C v;
    v.re.h = p[0];
    v.im.h = p[plane];
    v.re.l = p[2 * plane];
    v.im.l = p[3 * plane];
    return v;
  }
  __device__ static __forceinline__ void store(double *p, size_t plane, const C &v) {
    p[0] = v.re.h;
    p[plane] = v.im.h;
    p[2 * plane] = v.re.l;
    p[3 * plane] = v.im.l;
  }
  __device__ static __forceinline__ C czero() { return {{0.0, 0.0}, {0.0, 0.0}}; }
  __device__ static __forceinline__ R rzero() { return {0.0, 0.0}; }
  __device__ static __forceinline__ R rfrom(double v) { return {v, 0.0}; }
  __device__ static __forceinline__ R rone() { return {1.0, 0.0}; }
  __device__ static __forceinline__ void acc_zero(Acc &a) { a.sr = a.cr = a.si = a.ci = 0.0; }

  // acc += conj(q) * a
  __device__ static __forceinline__ void acc_cmulc(Acc &acc, const C &q, const C &a) {
    double p1, e1, p2, e2, t1, t2;
    // real: qr ar + qi ai
    two_prod(q.re.h, a.re.h, p1, e1);
    two_prod(q.im.h, a.im.h, p2, e2);
    two_sum(acc.sr, p1, acc.sr, t1);
    two_sum(acc.sr, p2, acc.sr, t2);
    double c = acc.cr;
    c = __fma_rn(q.re.h, a.re.l, c);
    c = __fma_rn(q.re.l, a.re.h, c);
    c = __fma_rn(q.im.h, a.im.l, c);
    c = __fma_rn(q.im.l, a.im.h, c);
    acc.cr = c + ((e1 + e2) + (t1 + t2));
    // imag: qr ai - qi ar
    two_prod(q.re.h, a.im.h, p1, e1);
    two_prod(-q.im.h, a.re.h, p2, e2);
    two_sum(acc.si, p1, acc.si, t1);
    two_sum(acc.si, p2, acc.si, t2);
    c = acc.ci;
    c = __fma_rn(q.re.h, a.im.l, c);
    c = __fma_rn(q.re.l, a.im.h, c);
    c = __fma_rn(-q.im.h, a.re.l, c);
    c = __fma_rn(-q.im.l, a.re.h, c);
    acc.ci = c + ((e1 + e2) + (t1 + t2));
  }
  // acc += a * b (no conjugation): re a.re b.re - a.im b.im, im a.re b.im + a.im b.re
  __device__ static __forceinline__ void acc_cmul(Acc &acc, const C &a, const C &b) {
    double p1, e1, p2, e2, t1, t2;
    two_prod(a.re.h, b.re.h, p1, e1);
    two_prod(-a.im.h, b.im.h, p2, e2);
    two_sum(acc.sr, p1, acc.sr, t1);
    two_sum(acc.sr, p2, acc.sr, t2);
    double c = acc.cr;
    c = __fma_rn(a.re.h, b.re.l, c);
    c = __fma_rn(a.re.l, b.re.h, c);
    c = __fma_rn(-a.im.h, b.im.l, c);
    c = __fma_rn(-a.im.l, b.im.h, c);
    acc.cr = c + ((e1 + e2) + (t1 + t2));
    two_prod(a.re.h, b.im.h, p1, e1);
    two_prod(a.im.h, b.re.h, p2, e2);
    two_sum(acc.si, p1, acc.si, t1);
    two_sum(acc.si, p2, acc.si, t2);
    c = acc.ci;
    c = __fma_rn(a.re.h, b.im.l, c);
    c = __fma_rn(a.re.l, b.im.h, c);
    c = __fma_rn(a.im.h, b.re.l, c);
    c = __fma_rn(a.im.l, b.re.h, c);
    acc.ci = c + ((e1 + e2) + (t1 + t2));
  }
  __device__ static __forceinline__ void acc_set(Acc &acc, const C &v) {
    acc.sr = v.re.h;
    acc.cr = v.re.l;
    acc.si = v.im.h;
    acc.ci = v.im.l;
  }
  __device__ static __forceinline__ C conj(const C &v) { return {v.re, {-v.im.h, -v.im.l}}; }
  // v += (dr + i di) for FP64 dr, di
  __device__ static __forceinline__ void add_cd(C &v, double dr, double di) {
    v.re = dd_add(v.re, {dr, 0.0});
    v.im = dd_add(v.im, {di, 0.0});
  }
  __device__ static __forceinline__ C cneg(const C &v) { return {{-v.re.h, -v.re.l}, {-v.im.h, -v.im.l}}; }
  // acc.re += |a|^2
  __device__ static __forceinline__ void acc_abs2(Acc &acc, const C &a) {
    double p1, e1, p2, e2, t1, t2;
    two_prod(a.re.h, a.re.h, p1, e1);
    two_prod(a.im.h, a.im.h, p2, e2);
    two_sum(acc.sr, p1, acc.sr, t1);
    two_sum(acc.sr, p2, acc.sr, t2);
    double c = acc.cr;
    c = __fma_rn(2.0 * a.re.h, a.re.l, c);
    c = __fma_rn(2.0 * a.im.h, a.im.l, c);
    acc.cr = c + ((e1 + e2) + (t1 + t2));
  }
  __device__ static __forceinline__ void acc_merge(Acc &a, const Acc &b) {
    double t;
    two_sum(a.sr, b.sr, a.sr, t);
    a.cr = (a.cr + b.cr) + t;
    two_sum(a.si, b.si, a.si, t);
    a.ci = (a.ci + b.ci) + t;
  }
  __device__ static __forceinline__ void acc_merge_re(Acc &a, const Acc &b) {
    double t;
    two_sum(a.sr, b.sr, a.sr, t);
    a.cr = (a.cr + b.cr) + t;
  }
  __device__ static __forceinline__ Acc acc_shfl_xor(const Acc &a, int mask) {
    Acc b;
    b.sr = __shfl_xor(a.sr, mask);
    b.cr = __shfl_xor(a.cr, mask);
    b.si = __shfl_xor(a.si, mask);
    b.ci = __shfl_xor(a.ci, mask);
    return b;
  }
  __device__ static __forceinline__ Acc acc_shfl_xor_re(const Acc &a, int mask) {
    Acc b;
    b.sr = __shfl_xor(a.sr, mask);
    b.cr = __shfl_xor(a.cr, mask);
    b.si = b.ci = 0.0;
    return b;
  }
  __device__ static __forceinline__ C acc_value(const Acc &a) {
    C v;
    two_sum(a.sr, a.cr, v.re.h, v.re.l);
    two_sum(a.si, a.ci, v.im.h, v.im.l);
    return v;
  }
  __device__ static __forceinline__ R acc_value_re(const Acc &a) {
    R v;
    two_sum(a.sr, a.cr, v.h, v.l);
    return v;
  }

  // a -= r * q (complex r, q).
  //   re: a.re - r.re q.re + r.im q.im
  //   im: a.im - r.re q.im - r.im q.re
  __device__ static __forceinline__ void upd(C &a, const C &r, const C &q) {
    double p1, e1, p2, e2, s, t1, t2, c;
    two_prod(-r.re.h, q.re.h, p1, e1);
    two_prod(r.im.h, q.im.h, p2, e2);
    two_sum(a.re.h, p1, s, t1);
    two_sum(s, p2, s, t2);
    c = a.re.l;
    c = __fma_rn(-r.re.h, q.re.l, c);
    c = __fma_rn(-r.re.l, q.re.h, c);
    c = __fma_rn(r.im.h, q.im.l, c);
    c = __fma_rn(r.im.l, q.im.h, c);
    c += (e1 + e2) + (t1 + t2);
    fast_two_sum(s, c, a.re.h, a.re.l);
    two_prod(-r.re.h, q.im.h, p1, e1);
    two_prod(-r.im.h, q.re.h, p2, e2);
    two_sum(a.im.h, p1, s, t1);
    two_sum(s, p2, s, t2);
    c = a.im.l;
    c = __fma_rn(-r.re.h, q.im.l, c);
    c = __fma_rn(-r.re.l, q.im.h, c);
    c = __fma_rn(-r.im.h, q.re.l, c);
    c = __fma_rn(-r.im.l, q.re.h, c);
    c += (e1 + e2) + (t1 + t2);
    fast_two_sum(s, c, a.im.h, a.im.l);
  }
  // a * s for real s.
  __device__ static __forceinline__ C scale(const C &a, const R &s) {
    return {dd_mul(a.re, s), dd_mul(a.im, s)};
  }
  __device__ static __forceinline__ R rmul(const R &a, const R &b) { return dd_mul(a, b); }
  __device__ static __forceinline__ R rneg(const R &a) { return {-a.h, -a.l}; }
  // a -= r x + s z, one part of upd with the same operations.
  __device__ static __forceinline__ void upd_part(R &a, const R &r, const R &x, const R &s, const R &z) {
    double p1, e1, p2, e2, t, t1, t2, c;
    two_prod(-r.h, x.h, p1, e1);
    two_prod(-s.h, z.h, p2, e2);
    two_sum(a.h, p1, t, t1);
    two_sum(t, p2, t, t2);
    c = a.l;
    c = __fma_rn(-r.h, x.l, c);
    c = __fma_rn(-r.l, x.h, c);
    c = __fma_rn(-s.h, z.l, c);
    c = __fma_rn(-s.l, z.h, c);
    c += (e1 + e2) + (t1 + t2);
    fast_two_sum(t, c, a.h, a.l);
  }
  __device__ static __forceinline__ R sqrt_(const R &s) { return dd_sqrt(s); }
  __device__ static __forceinline__ R recip(const R &s) { return dd_recip(s); }
  __device__ static __forceinline__ void sqrt_recip(const R &s, R &root, R &inv) { dd_sqrt_recip(s, root, inv); }
  __device__ static __forceinline__ bool ok_norm(const R &s) {
    return s.h > 0.0 && s.h < INFINITY && s.l == s.l && fabs(s.l) < INFINITY;
  }
  __device__ static __forceinline__ void store_real(double *p, size_t stride, const R &v) {
    p[0] = v.h;
    p[stride] = v.l;
  }
};

struct PrecQD {
  static constexpr int L = 4;
  using R = qd;
  using C = cqd;
  struct Acc {
    qdsum re, im;
  };
  using RAcc = qdsum;
  __device__ static __forceinline__ void racc_merge(RAcc &a, const RAcc &b) { qd_merge(a, b); }
  __device__ static __forceinline__ R racc_value(const RAcc &a) { return qd_value(a); }

  __device__ static __forceinline__ C load(const double *p, size_t plane) {
    C v;
    v.re.x0 = p[0];
    v.im.x0 = p[plane];
    v.re.x1 = p[2 * plane];
    v.im.x1 = p[3 * plane];
    v.re.x2 = p[4 * plane];
    v.im.x2 = p[5 * plane];
    v.re.x3 = p[6 * plane];
    v.im.x3 = p[7 * plane];
    return v;
  }
  __device__ static __forceinline__ void store(double *p, size_t plane, const C &v) {
    p[0] = v.re.x0;
    p[plane] = v.im.x0;
    p[2 * plane] = v.re.x1;
    p[3 * plane] = v.im.x1;
    p[4 * plane] = v.re.x2;
    p[5 * plane] = v.im.x2;
    p[6 * plane] = v.re.x3;
    p[7 * plane] = v.im.x3;
  }
  __device__ static __forceinline__ R rzero() { return {0.0, 0.0, 0.0, 0.0}; }
  __device__ static __forceinline__ R rfrom(double v) { return {v, 0.0, 0.0, 0.0}; }
  __device__ static __forceinline__ R rone() { return {1.0, 0.0, 0.0, 0.0}; }
  __device__ static __forceinline__ C czero() { return {rzero(), rzero()}; }
  __device__ static __forceinline__ void acc_zero(Acc &a) { a = {{0.0, 0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0, 0.0}}; }
  __device__ static __forceinline__ void acc_cmulc(Acc &acc, const C &q, const C &a) {
    qd_acc(acc.re, qd_dot2(q.re, a.re, q.im, a.im));
    qd_acc(acc.im, qd_dot2(q.re, a.im, qd_neg(q.im), a.re));
  }
  __device__ static __forceinline__ void acc_abs2(Acc &acc, const C &a) {
    qd_acc(acc.re, qd_sqr_levels(a.re));
    qd_acc(acc.re, qd_sqr_levels(a.im));
  }
  __device__ static __forceinline__ void acc_cmul(Acc &acc, const C &a, const C &b) {
    qd_acc(acc.re, qd_dot2(a.re, b.re, qd_neg(a.im), b.im));
    qd_acc(acc.im, qd_dot2(a.re, b.im, a.im, b.re));
  }
  __device__ static __forceinline__ void acc_set(Acc &acc, const C &v) { acc = {qd_sum_from(v.re), qd_sum_from(v.im)}; }
  __device__ static __forceinline__ C conj(const C &v) { return {v.re, qd_neg(v.im)}; }
  __device__ static __forceinline__ void add_cd(C &v, double dr, double di) {
    v.re = qd_add(v.re, qd_from(dr));
    v.im = qd_add(v.im, qd_from(di));
  }
  __device__ static __forceinline__ C cneg(const C &v) { return {qd_neg(v.re), qd_neg(v.im)}; }
  __device__ static __forceinline__ void acc_merge(Acc &a, const Acc &b) {
    qd_merge(a.re, b.re);
    qd_merge(a.im, b.im);
  }
  __device__ static __forceinline__ void acc_merge_re(Acc &a, const Acc &b) { qd_merge(a.re, b.re); }
  __device__ static __forceinline__ qdsum shfl_sum(const qdsum &a, int mask) {
    return {__shfl_xor(a.x0, mask), __shfl_xor(a.x1, mask), __shfl_xor(a.x2, mask), __shfl_xor(a.x3, mask),
            __shfl_xor(a.x4, mask)};
  }
  __device__ static __forceinline__ Acc acc_shfl_xor(const Acc &a, int mask) {
    return {shfl_sum(a.re, mask), shfl_sum(a.im, mask)};
  }
  __device__ static __forceinline__ Acc acc_shfl_xor_re(const Acc &a, int mask) {
    return {shfl_sum(a.re, mask), {0.0, 0.0, 0.0, 0.0, 0.0}};
  }
  __device__ static __forceinline__ C acc_value(const Acc &a) { return {qd_value(a.re), qd_value(a.im)}; }
  __device__ static __forceinline__ R acc_value_re(const Acc &a) { return qd_value(a.re); }
  __device__ static __forceinline__ void upd(C &a, const C &r, const C &q) {
    const qd nr = qd_neg(r.re), ni = qd_neg(r.im);
    qdsum sr = qd_sum_from(a.re), si = qd_sum_from(a.im);
    qd_acc(sr, qd_dot2(nr, q.re, r.im, q.im));
    qd_acc(si, qd_dot2(nr, q.im, ni, q.re));
    a.re = qd_value(sr);
    a.im = qd_value(si);
  }
  __device__ static __forceinline__ C scale(const C &a, const R &s) { return {qd_mul(a.re, s), qd_mul(a.im, s)}; }
  __device__ static __forceinline__ R rmul(const R &a, const R &b) { return qd_mul(a, b); }
  __device__ static __forceinline__ R rneg(const R &a) { return qd_neg(a); }
  // a -= r x + s z, one part of upd with the same operations.
  __device__ static __forceinline__ void upd_part(R &a, const R &r, const R &x, const R &s, const R &z) {
    qdsum t = qd_sum_from(a);
    qd_acc(t, qd_dot2(qd_neg(r), x, qd_neg(s), z));
    a = qd_value(t);
  }
  __device__ static __forceinline__ R sqrt_(const R &s) { return qd_sqrt(s); }
  __device__ static __forceinline__ R recip(const R &s) { return qd_recip(s); }
  __device__ static __forceinline__ void sqrt_recip(const R &s, R &root, R &inv) { qd_sqrt_recip(s, root, inv); }
  __device__ static __forceinline__ bool ok_norm(const R &s) {
    return s.x0 > 0.0 && s.x0 < INFINITY && fabs(s.x1) < INFINITY && fabs(s.x2) < INFINITY &&
           fabs(s.x3) < INFINITY;
  }
  __device__ static __forceinline__ void store_real(double *p, size_t stride, const R &v) {
    p[0] = v.x0;
    p[stride] = v.x1;
    p[2 * stride] = v.x2;
    p[3 * stride] = v.x3;
  }
};

// Plain complex double (FP64), for the blocked factorisation of the
// precision form: ordinary rounding, FMA where the product is fused.
struct cd {
  double re, im;
};
struct PrecD {
  static constexpr int L = 1;
  using R = double;
  using C = cd;
  struct Acc {
    double re, im;
  };
  using RAcc = double;
  __device__ static __forceinline__ void racc_merge(RAcc &a, const RAcc &b) { a += b; }
  __device__ static __forceinline__ R racc_value(const RAcc &a) { return a; }
  __device__ static __forceinline__ C load(const double *p, size_t plane) { return {p[0], p[plane]}; }
  __device__ static __forceinline__ void store(double *p, size_t plane, const C &v) {
    p[0] = v.re;
    p[plane] = v.im;
  }
  __device__ static __forceinline__ C czero() { return {0.0, 0.0}; }
  __device__ static __forceinline__ R rzero() { return 0.0; }
  __device__ static __forceinline__ R rfrom(double v) { return v; }
  __device__ static __forceinline__ R rone() { return 1.0; }
  __device__ static __forceinline__ void acc_zero(Acc &a) { a.re = a.im = 0.0; }
  __device__ static __forceinline__ void acc_cmulc(Acc &acc, const C &q, const C &a) {
    acc.re = __fma_rn(q.re, a.re, acc.re);
    acc.re = __fma_rn(q.im, a.im, acc.re);
    acc.im = __fma_rn(q.re, a.im, acc.im);
    acc.im = __fma_rn(-q.im, a.re, acc.im);
  }
  __device__ static __forceinline__ void acc_cmul(Acc &acc, const C &a, const C &b) {
    acc.re = __fma_rn(a.re, b.re, acc.re);
    acc.re = __fma_rn(-a.im, b.im, acc.re);
    acc.im = __fma_rn(a.re, b.im, acc.im);
    acc.im = __fma_rn(a.im, b.re, acc.im);
  }
  __device__ static __forceinline__ void acc_abs2(Acc &acc, const C &a) {
    acc.re = __fma_rn(a.re, a.re, acc.re);
    acc.re = __fma_rn(a.im, a.im, acc.re);
  }
  __device__ static __forceinline__ void acc_set(Acc &acc, const C &v) {
    acc.re = v.re;
    acc.im = v.im;
  }
  __device__ static __forceinline__ void acc_merge(Acc &a, const Acc &b) {
    a.re += b.re;
    a.im += b.im;
  }
  __device__ static __forceinline__ void acc_merge_re(Acc &a, const Acc &b) { a.re += b.re; }
  __device__ static __forceinline__ Acc acc_shfl_xor(const Acc &a, int mask) {
    return {__shfl_xor(a.re, mask), __shfl_xor(a.im, mask)};
  }
  __device__ static __forceinline__ Acc acc_shfl_xor_re(const Acc &a, int mask) { return {__shfl_xor(a.re, mask), 0.0}; }
  __device__ static __forceinline__ C acc_value(const Acc &a) { return {a.re, a.im}; }
  __device__ static __forceinline__ R acc_value_re(const Acc &a) { return a.re; }
  __device__ static __forceinline__ C conj(const C &v) { return {v.re, -v.im}; }
  __device__ static __forceinline__ C cneg(const C &v) { return {-v.re, -v.im}; }
  // a -= r q
  __device__ static __forceinline__ void upd(C &a, const C &r, const C &q) {
    a.re = __fma_rn(-r.re, q.re, a.re);
    a.re = __fma_rn(r.im, q.im, a.re);
    a.im = __fma_rn(-r.re, q.im, a.im);
    a.im = __fma_rn(-r.im, q.re, a.im);
  }
  __device__ static __forceinline__ C scale(const C &a, const R &s) { return {a.re * s, a.im * s}; }
  __device__ static __forceinline__ R rmul(const R &a, const R &b) { return a * b; }
  __device__ static __forceinline__ R rneg(const R &a) { return -a; }
  // a -= r x + s z, one part of upd with the same operations.
  __device__ static __forceinline__ void upd_part(R &a, const R &r, const R &x, const R &s, const R &z) {
    a = __fma_rn(-r, x, a);
    a = __fma_rn(-s, z, a);
  }
  __device__ static __forceinline__ R sqrt_(const R &s) { return sqrt(s); }
  __device__ static __forceinline__ R recip(const R &s) { return 1.0 / s; }
  __device__ static __forceinline__ bool ok_norm(const R &s) { return s > 0.0 && s < INFINITY; }
  __device__ static __forceinline__ void store_real(double *p, size_t stride, const R &v) { p[0] = v; }
};

// A sum as the kernels leave it in memory for the next launch: the
// accumulator, in qd its value (four limbs a part, 64 bytes in place of 80).
template <class P>
struct Partial {
  using T = typename P::Acc;
  __device__ static __forceinline__ T pack(const typename P::Acc &a) { return a; }
  __device__ static __forceinline__ typename P::Acc unpack(const T &t) { return t; }
};
template <>
struct Partial<PrecQD> {
  using T = cqd;
  __device__ static __forceinline__ T pack(const PrecQD::Acc &a) { return PrecQD::acc_value(a); }
  __device__ static __forceinline__ PrecQD::Acc unpack(const T &t) { return {qd_sum_from(t.re), qd_sum_from(t.im)}; }
};

// r = sqrt(s) and 1 / r (dd and qd: the fused forms that share their
// slow steps; FP64: the square root, then the division).
template <class P>
__device__ __forceinline__ void root_and_inverse(const typename P::R &s, typename P::R &root, typename P::R &inv) {
  if constexpr (P::L >= 2) {
    P::sqrt_recip(s, root, inv);
  } else {
    root = P::sqrt_(s);
    inv = P::recip(root);
  }
}

}  // namespace mgsq
