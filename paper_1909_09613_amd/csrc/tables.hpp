// Per-axis interpolation tables: the B-spline W_l and the WT factor T_l as
// polynomials in the in-cell coordinate.
//
// A particle at x~ (cell units) is split as x~ = base + sigma + g with
// base = floor(x~ - sigma) and g in [0, 1).  sigma is chosen per kernel so
// that all its nodes' weights are polynomials in g on [0, 1): for W_l no knot
// falls inside, for T_l exactly one (at kappa).  Node k (k = 0..K-1) is the
// lattice index base + first + k and carries
//     w_k(g) = sum_r c[k][r] g^r + alpha[k] * max(g - kappa, 0)^l.
// The tables are built on the host from the truncated-power form of each
// kernel (tables.cpp); the same evaluator runs on the host (table tests) and
// in the kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace wtpic {

constexpr int kMaxNodes = 6;   // l + 2 for l = 4
constexpr int kMaxCoef = 5;    // degree l + 1 coefficients for l = 4

template <class Real>
struct Tab {
  Real sigma;                   // lattice shift of the split
  Real one_minus_sigma;         // 1 - sigma, so that g = f + (1 - sigma) rounds once
  Real kappa;                   // interior knot in g (>= 1 when there is none)
  int first;                    // node offset from base
  int K;                        // node count
  Real c[kMaxNodes][kMaxCoef];  // polynomial coefficients, c[k][r] of g^r
  Real alpha[kMaxNodes];        // coefficient of the knot term
};

// T_l for c dt <= dx / 2 and l <= 3, where its l + 1 nodes' weights follow from
// its moments.  T_l reproduces polynomials of degree l - 1 (its transform,
// sinc^l(k dx/2) sinc(k c dt), has zeros of order l at the lattice's wave
// numbers), so that with the particle v past the middle of its nodes, v in
// [a - 1, a], and nodes at y_k from that middle,
//     sum w_k = 1, sum w_k y_k = v, sum w_k y_k^2 = v^2 + l/12 + a^2/3 (l = 3).
// These l equations leave one unknown: the outer weight on the side away from
// the particle is the single power p = beta max(a - |v|, 0)^l.
template <class Real>
struct TFac {
  Real sigma;   // the split: base is the cell before the particle's where f < sigma
  Real a;       // c dt / dx
  Real beta;    // 1 / (2 a l!)
  Real c;       // a^2 / 12
  int first;    // first node from base
};

// Split a position given as (cell, in-cell offset f in [0,1)) for a table.
template <class Real>
__host__ __device__ inline void tab_split(const Tab<Real>& t, int cell, Real f, int& base, Real& g) {
  if (t.sigma == Real(0)) {  // no split (folds away for constant tables)
    base = cell;
    g = f;
  } else {
    // selects rather than a branch: both sides are one instruction
    const bool below = f < t.sigma;
    base = cell - (below ? 1 : 0);
    g = below ? f + t.one_minus_sigma : f - t.sigma;
  }
}

template <class Real>
__host__ __device__ inline Real ipow(Real x, int l) {
  Real r = x;
  for (int i = 1; i < l; ++i) r *= x;
  return r;
}

// Weights w[0..K-1] at in-frame coordinate g (L = order, K = node count).
// top, if given, holds the leading coefficients c[k][L] (a copy the caller
// keeps elsewhere, e.g. in registers).
template <int L, int K, bool KNOT, class Real>
__host__ __device__ inline void tab_eval(const Tab<Real>& t, Real g, Real* w, const Real* top = nullptr) {
  Real tk = 0;
  if (KNOT) {
    Real d = g - t.kappa;
    d = d > Real(0) ? d : Real(0);
    tk = ipow(d, L);
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    Real acc = top ? top[k] : t.c[k][L];
#pragma unroll
    for (int r = L - 1; r >= 0; --r) acc = acc * g + t.c[k][r];
    if (KNOT) acc += t.alpha[k] * tk;
    w[k] = acc;
  }
}

// The split of an in-cell offset f for T_l's moments: base from the particle's
// cell, and v past the middle of the nodes, one rounding of f.
template <int L, class Real>
__host__ __device__ inline void tfac_split(const TFac<Real>& t, Real f, int& base, Real& v) {
  constexpr Real mid = L == 2 ? Real(1) : Real(1.5);
  const bool below = f < t.sigma;
  base = below ? -1 : 0;
  v = f - (below ? mid - Real(1) : mid);
}

// Weights w[0..L], L <= 3, of T_l from its moments, in coordinates about the
// middle of the nodes: the unknown p is at most a^2/12 (l = 3), so its rounding
// hardly counts, and the rest are short sums of v.  Root mean square error of a
// particle's weights against the exact factor, in 2^-24 (FP32; FP64 alike in 2^-53),
// here / from the table, a = 0.1, 0.3, 0.45, 0.5: linear 0.11 / 2.05, 0.34 / 1.00,
// 0.49 / 0.80, 0.26 / 0.23; quadratic 0.34 / 0.51, 0.38 / 0.75, 0.40 / 0.76, 0.40 / 0.43;
// cubic 0.46 / 0.72, 0.44 / 0.58, 0.44 / 0.58, 0.43 / 0.54.  (The quartic's lose
// more to the cancellation of its cubic terms, 0.63 / 0.47 at a = 0.5: tables.)
// About as many instructions as the cubic's table (19 against 20), and three
// constants besides the split where it has 20 per axis, which the particle loop
// keeps in scalar registers where it had to load the tables again for every
// particle.
template <int L, class Real>
__host__ __device__ inline void tfac_eval(const TFac<Real>& t, Real v, Real* w) {
  static_assert(L <= 3, "the quartic factor comes from its table");
  if constexpr (L == 1) {
    w[1] = fmax(fma(v, t.beta, Real(0.5)), Real(0));
    w[0] = Real(1) - w[1];
  } else {
    const Real m = fabs(v);
    const Real d = fmax(t.a - m, Real(0));
    if constexpr (L == 2) {
      const Real p = d * (d * t.beta);
      w[0] = p + fmax(-v, Real(0));
      w[1] = fma(Real(-2), p, Real(1) - m);
      w[2] = p + fmax(v, Real(0));
    } else {
      // h: half the outer weights' sum, x: half their difference, signed
      const Real p = (d * d) * (d * t.beta);
      const Real h = fma(Real(0.25) * v, v, t.c);
      const Real x = copysign(h - p, v);
      const Real s = Real(0.5) - h, y = fma(Real(-3), x, v);
      w[0] = h - x;
      w[1] = s - y;
      w[2] = s + y;
      w[3] = h + x;
    }
  }
}

// Weight differences w_k(e) - w_k(g) = (e - g) * sum_{r>=1} c[k][r] h_r(g, e),
// h_r = sum_{i+j=r-1} g^i e^j, written as d * (divided difference) so that a
// short step d = e - g keeps full relative precision.  Knot-free tables only.
// CONST: the table is a compile-time constant, whose zero coefficients are
// left out (a product with a zero the compiler must otherwise keep).
template <int L, bool CONST = false, class Real>
__host__ __device__ inline void tab_diff(const Tab<Real>& t, Real g, Real e, Real d, Real* dw) {
  Real h[kMaxCoef];
  h[1] = Real(1);
  Real gp = g;  // g^(r-1)
#pragma unroll
  for (int r = 2; r <= L; ++r) {
    h[r] = h[r - 1] * e + gp;
    gp *= g;
  }
#pragma unroll
  for (int k = 0; k <= L; ++k) {
    Real acc = t.c[k][L] * h[L];
#pragma unroll
    for (int r = L - 1; r >= 1; --r)
      if (!CONST || t.c[k][r] != Real(0)) acc += t.c[k][r] * h[r];
    dw[k] = d * acc;
  }
}

// Weights of a B-spline table's NW nodes at g, up to the cubic one in the
// closed form of its polynomials (checked in the particle kernel).  The
// cubic in its symmetric form, 11 instructions against 12 for the four Horner
// polynomials: with t = 1 - g, w0 = t^3/6, w1 = 2/3 - g^2 + g^3/2, w2 the same
// at t, w3 = g^3/6.  The closed forms need at most two constants that are no
// immediate operands, where FP64 read both tables from scalar memory for
// every particle.
template <int L, int NW, class Real>
__host__ __device__ inline void wtab_eval(const Tab<Real>& T, Real g, Real* w) {
  if constexpr (L == 3 && NW == 4) {
    const Real t = Real(1) - g;
    const Real g2 = g * g, t2 = t * t;
    w[0] = t2 * (t * Real(1.0 / 6.0));
    w[1] = fma(g2, fma(g, Real(0.5), Real(-1)), Real(2.0 / 3.0));
    w[2] = fma(t2, fma(t, Real(0.5), Real(-1)), Real(2.0 / 3.0));
    w[3] = g2 * (g * Real(1.0 / 6.0));
  } else if constexpr (L == 2 && NW == 3) {
    const Real t = Real(1) - g;
    w[0] = t * (t * Real(0.5));
    w[1] = fma(g, t, Real(0.5));
    w[2] = g * (g * Real(0.5));
  } else if constexpr (L == 1 && NW == 2) {
    w[0] = Real(1) - g;
    w[1] = g;
  } else {
    tab_eval<L, NW, false>(T, g, w);
  }
}

// Weight differences w_k(e) - w_k(g) = d * (divided difference), d = e - g,
// for a table's L + 1 nodes.  For the cubic B-spline with h2 = g + e and
// h3 = g^2 + g e + e^2: the differences of the four closed forms above are
// d (h3/6), d ((h2 - 1)/2 - h3/6), d (h3/2 - h2) and d (1 + h2 - h3)/2 for nodes
// 3, 0, 1 and 2.  In FP32 node 2 takes minus the others' sum (the weights sum to
// one), 12 instructions against the table's 16; in FP64 each node has its own,
// 13 instructions.  The quadratic one's d h2/2, d (h2/2 - 1) and d (1 - h2), each
// rounded once after h2.  Root mean square error of the three or four against the
// exact differences, over d, in 2^-53, here / from the table: quadratic 0.77 / 0.81,
// cubic 0.81 / 0.91 (with node 2 as in FP32 1.27).
template <int L, bool CONSTTAB, class Real>
__host__ __device__ inline void wtab_diff(const Tab<Real>& T, Real g, Real e, Real d, Real* dw) {
  if constexpr (L == 3) {
    const Real h2 = g + e;
    const Real h3 = fma(h2, e, g * g);
    const Real q = h3 * (d * Real(1.0 / 6.0));
    dw[3] = q;
    dw[0] = fma(h2 - Real(1), d * Real(0.5), -q);
    if constexpr (sizeof(Real) == 4) {
      dw[1] = fma(Real(3), q, -(d * h2));
      dw[2] = -(dw[0] + dw[1]) - q;
    } else {
      dw[1] = d * fma(Real(0.5), h3, -h2);
      dw[2] = (d * Real(0.5)) * ((Real(1) - h3) + h2);
    }
  } else if constexpr (L == 2) {
    const Real h2 = g + e, hd = d * Real(0.5);
    dw[0] = fma(h2, hd, -d);
    dw[1] = fma(-h2, d, d);
    dw[2] = h2 * hd;
  } else if constexpr (L == 1) {
    dw[0] = -d;
    dw[1] = d;
  } else {
    tab_diff<L, CONSTTAB>(T, g, e, d, dw);
  }
}

// The B-spline tables (kinds 0 and 1 below) depend only on l and the
// lattice, so they are built at compile time: the same truncated-power
// expansion as build_table, in double (every quantity is a small rational).
// The particle kernel uses them as literal constants.
constexpr double cx_binom(int n, int k) {
  double r = 1.0;
  for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
  return r;
}
constexpr double cx_frac(double x) {
  long long i = (long long)x;
  double f = x - (double)i;
  return f < 0.0 ? f + 1.0 : f;
}
template <class Real>
constexpr Tab<Real> make_wtab(int l, int kind) {
  Tab<Real> out{};
  double fact = 1.0;
  for (int i = 2; i <= l; ++i) fact *= i;
  const double lam = (kind == 0) ? 0.5 : 0.0;
  const double sigma = cx_frac(lam - 0.5 * (l + 1));
  const double first_f = sigma - lam - 0.5 * (l - 1);
  const int first = (int)(first_f < 0.0 ? first_f - 0.5 : first_f + 0.5);
  const int K = l + 1;
  const double D = sigma - first - lam;
  double c[kMaxNodes][kMaxCoef] = {};
  for (int k = 0; k < K; ++k)
    for (int j = 0; j <= l + 1; ++j) {
      const double beta = ((j & 1) ? -1.0 : 1.0) * cx_binom(l + 1, j) / fact;
      const double kp = (j - 0.5 * (l + 1)) + k - D;  // knot in g
      if (kp <= 1e-12) {
        for (int r = 0; r <= l; ++r) {
          double p = 1.0;
          for (int q = 0; q < l - r; ++q) p *= -kp;
          c[k][r] += beta * cx_binom(l, r) * p;
        }
      }
    }
  out.sigma = Real(sigma);
  out.one_minus_sigma = Real(1.0 - sigma);
  out.kappa = Real(2.0);
  out.first = first;
  out.K = K;
  for (int k = 0; k < kMaxNodes; ++k) {
    for (int r = 0; r < kMaxCoef; ++r) out.c[k][r] = Real(c[k][r]);
    out.alpha[k] = Real(0);
  }
  return out;
}

// Host: build the table of one kernel kind for order l.
//   kind 0: W_l on the half-integer lattice (nodes at m + 1/2)
//   kind 1: W_l on the integer lattice
//   kind 2: T_l(.; a) on the integer lattice, 0 < a < 1
// Returns false (and a message) on invalid input or an internal inconsistency.
bool build_table(int l, int kind, double a, Tab<double>& out, const char** err);

// Host: the constants of tfac_split and tfac_eval from a kind-2 table of 0 < a <= 1/2.
TFac<double> make_tfac(int l, double a, const Tab<double>& t);

template <class Real>
inline void convert_table(const Tab<double>& in, Tab<Real>& out) {
  out.sigma = Real(in.sigma);
  out.one_minus_sigma = Real(in.one_minus_sigma);
  out.kappa = Real(in.kappa);
  out.first = in.first;
  out.K = in.K;
  for (int k = 0; k < kMaxNodes; ++k) {
    for (int r = 0; r < kMaxCoef; ++r) out.c[k][r] = Real(in.c[k][r]);
    out.alpha[k] = Real(in.alpha[k]);
  }
}

}  // namespace wtpic
