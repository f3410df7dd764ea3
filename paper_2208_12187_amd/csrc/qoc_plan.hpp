// Choice of the scaling exponent s and the Taylor degrees (q for exp, qb for
// its Frechet block) of one slice, shared by the plan kernel and the host.
//
// theta = dt (|H0|_1 + sum_j |u[j][k]| |Hc[j]|_1) bounds |A_k|_1 by the
// triangle inequality (A_k = -i dt H_k), and |A^n| <= |A|^n in the 1-norm.
// With r = theta / 2^s:
//  * exp: the Taylor remainder after degree q is at most
//    r^(q+1)/(q+1)! * 1/(1 - r/(q+2)) (geometric bound on the tail ratios);
//    q is the least degree for which this is at most the unit roundoff ur.
//  * Frechet block exp([[X, E], [0, X]]): its top-right block is linear in E
//    and the degree-n term of the series contributes n X^(n-1)-type products,
//    so the remainder after degree qb is at most
//    |E| r^qb/qb! * 1/(1 - r/(qb+1)); qb (>= 2) is the least degree for which
//    the factor of |E| is at most ur.
//  * commutator series sum_n ad_X^n / n! and sum_n ad_X^n / (n + 1)! (Hermitian
//    path, but FP64 at d > 64): |ad_X| <= 2 r, so the exponential's rule at 2 r
//    bounds both remainders; m is that degree.
// Among s in [s0, s0 + 6], s0 = least s >= 0 with r <= 1, the value that
// minimises the number of complex d x d products of the path is taken:
//    exp:       (q - 1) + s    (Horner; expm_products(q) + s where the expm
//                                 runs Paterson-Stockmeyer: D = 128;
//                                 taylor_products(q) + s on segments at D <= 64)
//    gradient:  + frechet_products(qb) + 3 s   (block polynomial, squarings),
//               or plan_cost's count for the commutator series
#pragma once

#include <math.h>

namespace qoc {

struct SlicePlan {
  int s, q, qb;
  int m;  // commutator series: degree
};

#if defined(__HIPCC__)
#define QOC_HD __host__ __device__
#else
#define QOC_HD
#endif

// 1 / n as a literal of the unrolled loops below (no divisions: three of these
// searches per candidate s and slice).
QOC_HD constexpr double plan_inv(int n) { return 1.0 / n; }

QOC_HD inline int taylor_degree(double r, double ur) {
  int q = 1;
  double t = r * r * 0.5;  // r^(q+1)/(q+1)!
#pragma unroll
  for (int n = 1; n < 30; ++n) {
    if (!(t > ur * (1.0 - r * plan_inv(n + 2)))) break;
    q = n + 1;
    t *= r * plan_inv(n + 2);
  }
  return q;
}

QOC_HD inline int frechet_degree(double r, double ur) {
  int qb = 2;
  double t = r * r * 0.5;  // r^qb/qb!
#pragma unroll
  for (int n = 2; n < 31; ++n) {
    if (!(t > ur * (1.0 - r * plan_inv(n + 1)))) break;
    qb = n + 1;
    t *= r * plan_inv(n + 1);
  }
  return qb;
}

QOC_HD inline double inv_factorial(int n) {
  double f = 1.0;
  for (int i = 2; i <= n; ++i) f /= i;
  return f;
}

// Complex d x d products of the degree-q Taylor polynomial in delta form by
// Paterson-Stockmeyer with X^2 as the step: one for X^2, one per digit that
// holds a matrix below the top one (floor((q - 3) / 2) of them) and one for
// the last step (q >= 3); X + X^2 / 2 at q = 2.
QOC_HD inline int expm_products(int q) { return q < 2 ? 0 : (q == 2 ? 1 : 2 + (q - 3) / 2); }

// Complex d x d products of a Taylor polynomial of degree at least q in
// k_seg_fwd's evaluation: Horner, the degree-4 and degree-8 forms,
// Paterson-Stockmeyer with X^3 as the step.
QOC_HD inline int taylor_products(int q) { return q <= 3 ? q - 1 : (q == 4 ? 2 : (q <= 8 ? 3 : 2 + (q - 1) / 3)); }

// Complex d x d products of the degree-qb Taylor polynomial of the block
// [[X, E], [0, X]] by Paterson-Stockmeyer with the block's square as the
// step: three for the square, three per Horner step in the square that has a
// matrix digit (floor((qb - 3) / 2) of them), two for the last step's top
// right block (the top left one is counted with the squarings).
QOC_HD inline int frechet_products(int qb) { return 5 + 3 * (qb > 3 ? (qb - 3) / 2 : 0); }

// comm: the gradient's m products of the commutator series and, for s > 0,
// the exponential again (at D <= 64 it is kept: its count stands for the traffic,
// and for the slower kernel of squared slices), s doublings and the step of Y.
QOC_HD inline int plan_cost(int s, int q, int qb, int m, bool grad, bool ps_expm, bool comm) {
  const int expm = ps_expm ? expm_products(q) : comm ? taylor_products(q) : q - 1;
  int cost = expm + s;
  if (grad && comm) cost += m + (s > 0 ? expm + 2 + 3 * s : 0);
  else if (grad) cost += frechet_products(qb) + 3 * s;
  return cost;
}

// Least degree n >= 1 at which the remainder of sum_n x^n / (n + 1)! after degree
// n - 1, x^n / (n + 1)! * 1/(1 - x/(n + 2)), is at most ur.
QOC_HD inline int phi_degree(double x, double ur) {
  int q = 1;
  double t = x * 0.5;  // x^n/(n+1)!
#pragma unroll
  for (int n = 1; n < 30; ++n) {
    if (!(t > ur * (1.0 - x * plan_inv(n + 2)))) break;
    q = n + 1;
    t *= x * plan_inv(n + 2);
  }
  return q;
}

// What the plan is for: a gradient; Paterson-Stockmeyer exponentials; the
// commutator series; that summed by Horner's rule.
enum PlanFlags : int { PLAN_GRAD = 1, PLAN_PS = 2, PLAN_COMM = 4, PLAN_HORNER = 8 };

QOC_HD inline SlicePlan choose_plan(double theta, double ur, int flags) {
  const bool grad = (flags & PLAN_GRAD) != 0, ps_expm = (flags & PLAN_PS) != 0, comm = (flags & PLAN_COMM) != 0;
  // Infinite or NaN: nothing to compute, and no squarings (the state path takes 2^s steps).
  // By comparison: theta - theta of a product th * dt is contracted to its rounding error.
  if (!(theta <= 1.7976931348623157e308)) return SlicePlan{0, 1, 2, 1};
  int s0 = 0;
  while (ldexp(theta, -s0) > 1.0 && s0 < 60) ++s0;
  SlicePlan best = {s0, 1, 2, 1};
  int best_cost = 1 << 30;
  for (int s = s0; s <= s0 + 6; ++s) {
    double r = ldexp(theta, -s);
    int q = taylor_degree(r, ur);
    int qb = frechet_degree(r, ur);
    int m = comm ? taylor_degree(2 * r, ur) : 0;
    if (flags & PLAN_HORNER) {
      const int mz = phi_degree(2 * r, ur);
      m = m > mz ? m : mz;
    }
    int c = plan_cost(s, q, qb, m, grad, ps_expm, comm);
    // the degrees fall ever more slowly with s while each s adds the same:
    // past the minimum the count only grows
    if (c > best_cost) break;
    if (c < best_cost) {
      best_cost = c;
      best.s = s;
      best.q = q;
      best.qb = qb;
      best.m = m;
    }
  }
  return best;
}

// s, q, qb in a byte each (bits 24 and 25 are the kernels' flags), m on top.
QOC_HD inline int pack_plan(SlicePlan p) {
  return (int)((unsigned)p.s | ((unsigned)p.q << 8) | ((unsigned)p.qb << 16) | ((unsigned)p.m << 26));
}
QOC_HD inline int plan_order(int sq) { return (int)((unsigned)sq >> 26); }

}  // namespace qoc
