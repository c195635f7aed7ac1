// Reads "m a[0..m-1] b[0..m-2]" from stdin, writes the lowest eigenvalue and
// its eigenvector as tridiag_lowest finds them.
#include <cstdio>
#include <vector>

#include "host_eig.h"

int main() {
  int m = 0;
  if (std::scanf("%d", &m) != 1 || m < 1) return 1;
  std::vector<double> a(m), b(m), s;
  for (double& x : a)
    if (std::scanf("%lf", &x) != 1) return 1;
  for (int i = 0; i + 1 < m; ++i)
    if (std::scanf("%lf", &b[i]) != 1) return 1;
  std::printf("%.17g\n", hub::tridiag_lowest(m, a.data(), b.data(), s));
  for (double x : s) std::printf("%.17g\n", x);
  return 0;
}
