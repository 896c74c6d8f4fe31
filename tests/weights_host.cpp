// Host side of test_weights_error.py: errors of T_l's weights, as the particle
// kernel evaluates them, against the factor itself in long double.
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

}  // namespace

// out: root mean square error of a place's weights (table, moments), largest
// error of one weight (table, moments), in units of 2^-24 (FP32) or 2^-53.
extern "C" void weight_errors(int l, int fp32, double a, int n, double out[4]) {
  for (int k = 0; k < 4; ++k) out[k] = -1.0;
  if (l == 1) fp32 ? compare<float, 1>(a, n, out) : compare<double, 1>(a, n, out);
  if (l == 2) fp32 ? compare<float, 2>(a, n, out) : compare<double, 2>(a, n, out);
  if (l == 3) fp32 ? compare<float, 3>(a, n, out) : compare<double, 3>(a, n, out);
}
