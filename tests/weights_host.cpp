// Host side of test_weights_error.py: errors of T_l's weights and of the
// B-spline's weight differences, as the particle kernel evaluates them, against
// the functions themselves in long double.
#include <math.h>

#include <algorithm>
#include <random>

#include "tables.hpp"

using namespace wtpic;

namespace {

// T_l(y; a) as the sum of truncated powers that defines it.
long double factor(int l, long double a, long double y) {
  long double s = 0.0L, b = 1.0L, fact = 1.0L;
  for (int i = 2; i <= l; ++i) fact *= i;
  for (int j = 0; j <= l; ++j) {
    const long double p = std::max(y + a + 0.5L * l - j, 0.0L), q = std::max(y - a + 0.5L * l - j, 0.0L);
    s += b * (powl(p, l) - powl(q, l));
    b = -b * (l - j) / (j + 1);
  }
  return s / (2.0L * a * fact);
}

template <class Real, int L>
void compare(double a, int n, double out[4]) {
  Tab<double> td;
  const char* err = nullptr;
  if (!build_table(L, 2, a, td, &err) || td.K != L + 1) return;
  Tab<Real> t;
  convert_table(td, t);
  const TFac<double> fd = make_tfac(L, a, td);
  const TFac<Real> tf = {Real(fd.sigma), Real(fd.a), Real(fd.beta), Real(fd.c), fd.first};
  const long double unit = sizeof(Real) == 4 ? 0x1p-24L : 0x1p-53L;
  std::mt19937_64 rng(17);
  double sum[2] = {0, 0}, most[2] = {0, 0};
  for (int i = 0; i < n; ++i) {
    const Real f = std::min(Real((rng() >> 11) * 0x1p-53), Real(1) - Real(unit));
    Real w[2][L + 1];
    int base[2];
    // the table, split as for tables known at run time: g = fract(f - sigma)
    const Real d = f - t.sigma;
    base[0] = d < Real(0) ? -1 : 0;
    const Real g = std::min(Real(d - floor(d)), Real(1) - Real(unit));
    tab_eval<L, L + 1, true>(t, g, w[0]);
    base[0] += t.first;
    Real v;
    tfac_split<L>(tf, f, base[1], v);
    tfac_eval<L>(tf, v, w[1]);
    base[1] += tf.first;
    for (int k = 0; k < 2; ++k)
      for (int j = 0; j <= L; ++j) {
        const double e = (double)((w[k][j] - factor(L, a, (long double)f - (base[k] + j))) / unit);
        sum[k] += e * e;
        most[k] = std::max(most[k], fabs(e));
      }
  }
  for (int k = 0; k < 2; ++k) {
    out[k] = sqrt(sum[k] / n);
    out[2 + k] = most[k];
  }
}

// W_l(y), likewise.
long double bspline(int l, long double y) {
  long double s = 0.0L, b = 1.0L, fact = 1.0L;
  for (int i = 2; i <= l; ++i) fact *= i;
  for (int j = 0; j <= l + 1; ++j) {
    const long double p = y + 0.5L * (l + 1) - j;
    if (p > 0.0L) s += b * powl(p, l);
    b = -b * (l + 1 - j) / (j + 1);
  }
  return s / fact;
}

template <class Real, int L>
void compare_differences(int n, double out[4]) {
  constexpr Tab<Real> t = make_wtab<Real>(L, 1);
  const long double unit = sizeof(Real) == 4 ? 0x1p-24L : 0x1p-53L;
  std::mt19937_64 rng(19);
  double sum[2] = {0, 0}, most[2] = {0, 0};
  for (int i = 0; i < n; ++i) {
    const Real g = std::min(Real((rng() >> 11) * 0x1p-53), Real(1) - Real(unit));
    // a step of up to 1/16 cell (longer ones take S1 - S0) that ends in the cell
    const Real e = std::min(std::max(g + Real(((rng() >> 11) * 0x1p-53 - 0.5) / 8), Real(0)), Real(1));
    const Real d = e - g;
    if (d == Real(0) || (long double)d != (long double)e - (long double)g) continue;
    Real dw[2][L + 1];
    tab_diff<L, true>(t, g, e, d, dw[0]);
    wtab_diff<L, true>(t, g, e, d, dw[1]);
    for (int j = 0; j <= L; ++j) {
      // the particle's distance from node j
      const long double o = (long double)t.sigma - (t.first + j);
      // the mean of dW_l/dy = W_{l-1}(y + 1/2) - W_{l-1}(y - 1/2), at most a
      // parabola here, by Simpson's rule
      auto slope = [&](long double y) { return bspline(L - 1, o + y + 0.5L) - bspline(L - 1, o + y - 0.5L); };
      const long double m = 0.5L * ((long double)g + e);
      const long double x = L == 1 ? slope(m) : (slope(g) + 4.0L * slope(m) + slope(e)) / 6.0L;
      for (int k = 0; k < 2; ++k) {
        const double r = (double)((dw[k][j] / (long double)d - x) / unit);
        sum[k] += r * r;
        most[k] = std::max(most[k], fabs(r));
      }
    }
  }
  for (int k = 0; k < 2; ++k) {
    out[k] = sqrt(sum[k] / n);
    out[2 + k] = most[k];
  }
}

}  // namespace

// out: root mean square error of a place's weights (table, moments), largest
// error of one weight (table, moments), in units of 2^-24 (FP32) or 2^-53.
extern "C" void weight_errors(int l, int fp32, double a, int n, double out[4]) {
  for (int k = 0; k < 4; ++k) out[k] = -1.0;
  if (l == 1) fp32 ? compare<float, 1>(a, n, out) : compare<double, 1>(a, n, out);
  if (l == 2) fp32 ? compare<float, 2>(a, n, out) : compare<double, 2>(a, n, out);
  if (l == 3) fp32 ? compare<float, 3>(a, n, out) : compare<double, 3>(a, n, out);
}

// The same of the weight differences over the step (table, closed form).
extern "C" void difference_errors(int l, int fp32, int n, double out[4]) {
  for (int k = 0; k < 4; ++k) out[k] = -1.0;
  if (l == 1) fp32 ? compare_differences<float, 1>(n, out) : compare_differences<double, 1>(n, out);
  if (l == 2) fp32 ? compare_differences<float, 2>(n, out) : compare_differences<double, 2>(n, out);
  if (l == 3) fp32 ? compare_differences<float, 3>(n, out) : compare_differences<double, 3>(n, out);
}
