#include "host_eig.h"

#include <algorithm>
#include <cfloat>
#include <cmath>

namespace hub {

namespace {

// Eigenvalues of T below x: the negative pivots of the factorisation of
// T - x from the top (Sturm's count).
int count_below(int m, const double* a, const double* b, double x, double tiny) {
  int n = 0;
  double d = a[0] - x;
  for (int i = 0;; ++i) {
    if (std::fabs(d) < tiny) d = -tiny;
    n += d < 0.0;
    if (i + 1 >= m) return n;
    d = a[i + 1] - x - b[i] * b[i] / d;
  }
}

// Vector z with (T - x) z = g e_r, z_r = 1, from the factorisations of T - x
// from the top and from the bottom, meeting at the row r where |g| is least
// (small components keep their relative accuracy).  Returns the Rayleigh
// correction g / |z|^2 and normalises z.
double twisted_vector(int m, const double* a, const double* b, double x, double tiny, std::vector<double>& z) {
  std::vector<double> dp(m), dm(m);
  auto safe = [&](double d) { return std::fabs(d) < tiny ? (d < 0.0 ? -tiny : tiny) : d; };
  dp[0] = a[0] - x;
  for (int i = 0; i + 1 < m; ++i) dp[i + 1] = a[i + 1] - x - b[i] * b[i] / safe(dp[i]);
  dm[m - 1] = a[m - 1] - x;
  for (int i = m - 2; i >= 0; --i) dm[i] = a[i] - x - b[i] * b[i] / safe(dm[i + 1]);
  int r = 0;
  double g = INFINITY;
  for (int i = 0; i < m; ++i) {
    const double gi = dp[i] + dm[i] - (a[i] - x);
    if (std::fabs(gi) < std::fabs(g)) {
      g = gi;
      r = i;
    }
  }
  z.assign(m, 0.0);
  z[r] = 1.0;
  for (int i = r - 1; i >= 0; --i) z[i] = -b[i] / safe(dp[i]) * z[i + 1];
  for (int i = r + 1; i < m; ++i) z[i] = -b[i - 1] / safe(dm[i]) * z[i - 1];
  double n2 = 0.0;
  for (double v : z) n2 += v * v;
  const double inv = 1.0 / std::sqrt(n2);
  for (double& v : z) v *= inv;
  return g / n2;
}

}  // namespace

double tridiag_lowest(int m, const double* a, const double* b, std::vector<double>& s) {
  double lo = INFINITY, hi = INFINITY, norm = 0.0;
  for (int i = 0; i < m; ++i) {  // Gershgorin; the lowest eigenvalue is at most the least diagonal element
    const double r = (i > 0 ? std::fabs(b[i - 1]) : 0.0) + (i + 1 < m ? std::fabs(b[i]) : 0.0);
    lo = std::min(lo, a[i] - r);
    hi = std::min(hi, a[i]);
    norm = std::max(norm, std::fabs(a[i]) + r);
  }
  const double eps = DBL_EPSILON * std::max(norm, DBL_MIN), tiny = eps * DBL_EPSILON;
  auto bisect = [&](int steps) {
    for (int k = 0; k < steps && hi - lo > 0.5 * eps; ++k) {
      const double mid = 0.5 * (lo + hi);
      if (count_below(m, a, b, mid, tiny) == 0) lo = mid;
      else hi = mid;
    }
    return 0.5 * (lo + hi);
  };
  // a bracket of 1e-6 of the spectrum, then Rayleigh quotient steps (cubic);
  // where they leave for another eigenvalue, bisection to the end
  double x = bisect(20);
  for (int k = 0; k < 4; ++k) {
    const double d = twisted_vector(m, a, b, x, tiny, s);
    x += d;
    if (!(std::fabs(d) > eps)) break;
  }
  if (count_below(m, a, b, x - 8 * eps, tiny) != 0 || count_below(m, a, b, x + 8 * eps, tiny) == 0) x = bisect(80);
  x += twisted_vector(m, a, b, x, tiny, s);
  return x;
}

}  // namespace hub
