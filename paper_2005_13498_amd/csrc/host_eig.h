// Lowest eigenpair of a small symmetric tridiagonal matrix (host, FP64).
#pragma once

#include <vector>

namespace hub {

// T has the diagonal a[0..m-1] and the off-diagonal b[0..m-2], all b nonzero
// (an unreduced Lanczos matrix, whose eigenvalues are simple).  Returns the
// lowest eigenvalue and its normalised eigenvector in s[0..m-1].
double tridiag_lowest(int m, const double* a, const double* b, std::vector<double>& s);

}  // namespace hub
