// Worst and root-mean-square errors of GELU and its derivative against 64
// bits over [lo, hi]: gelu_both's, then those with erff and expf.
// Arguments: lo hi n.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "gelu.h"

struct HostOps {
  static float rcp(float x) { return 1.0f / x; }
  static float exp2(float x) { return ::exp2f(x); }
};

struct Err {
  double worst = 0.0, sq = 0.0;
  void add(double e) {
    worst = std::fmax(worst, std::fabs(e));
    sq += e * e;
  }
};

int main(int argc, char** argv) {
  if (argc != 4) return 1;
  const double lo = std::atof(argv[1]), hi = std::atof(argv[2]);
  const int n = std::atoi(argv[3]);
  Err h, d, he, de;
  for (int k = 0; k < n; ++k) {
    const float z = static_cast<float>(lo + (hi - lo) * k / (n - 1));
    const double Z = z, Phi = 0.5 * std::erfc(-Z / std::sqrt(2.0));
    const double H = Z * Phi, D = Phi + Z * std::exp(-0.5 * Z * Z) / std::sqrt(2.0 * M_PI);
    const hub::Gelu g = hub::gelu_both<HostOps>(z);
    h.add(g.h - H);
    d.add(g.d - D);
    const float pe = 1.0f + erff(z * 0.70710678118654752f);
    he.add(0.5f * z * pe - H);
    de.add(fmaf(z * 0.39894228040143268f, expf(-0.5f * z * z), 0.5f * pe) - D);
  }
  for (const Err& x : {h, d, he, de}) std::printf("%.17g %.17g\n", x.worst, std::sqrt(x.sq / n));
  const hub::Gelu big = hub::gelu_both<HostOps>(INFINITY), low = hub::gelu_both<HostOps>(-INFINITY);
  const hub::Gelu nan = hub::gelu_both<HostOps>(NAN), zero = hub::gelu_both<HostOps>(0.0f);
  std::printf("%d %d %d %d\n", std::isinf(big.h) && big.h > 0, std::isnan(low.h), std::isnan(nan.h) && std::isnan(nan.d),
              zero.h == 0.0f && zero.d == 0.5f);
  return 0;
}
