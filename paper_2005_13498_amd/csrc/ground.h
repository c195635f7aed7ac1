// Kernels of the ground-state Lanczos (ground.hip): complex double, one
// vector, full reorthogonalisation.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace hub {

// The vectors an iteration is orthogonalised against: `deflate` (may be null)
// first, then the Lanczos vectors V[0], V[1], .. stored one after another.
struct GsBasis {
  const double2* deflate;
  const double2* V;
  int64_t dim;
  int nb;  // vectors, deflate included
};

constexpr int kGsDotRows = 32;    // most partial rows of the inner products
constexpr int kGsNormRows = 1024;  // most partial rows of the norms

// dotp[rows][2 nb] = partial <b_k, w>; returns the rows in *rows.
hipError_t launch_gs_dot(const GsBasis& B, const double2* w, double* dotp, int* rows, hipStream_t s);
// w -= sum_k b_k <b_k, w> with the inner products summed from dotp; |w|^2
// partials (nrows of them) to normp; the last vector's Re <b, w> is stored in
// *alpha (add: added to it).
hipError_t launch_gs_subtract(const GsBasis& B, double2* w, const double* dotp, int rows, double* normp, int* nrows,
                              double* alpha, bool add, hipStream_t s);
// out = sum_k c[k] V[k], k < m (device c); |out|^2 partials to normp.
hipError_t launch_gs_combine(const double2* V, int64_t dim, int m, const double* c, double2* out, double* normp,
                             int* nrows, hipStream_t s);
// dst = x / |x| with |x|^2 summed from normp (zero stays zero), also to dst2
// if given; |x| to *norm if given.
hipError_t launch_gs_scale(int64_t dim, const double2* x, const double* normp, int nrows, double2* dst, double2* dst2,
                           double* norm, hipStream_t s);
// x = seeded complex standard normal numbers, |x|^2 partials to normp.
hipError_t launch_gs_start(int64_t dim, uint64_t seed, double2* x, double* normp, int* nrows, hipStream_t s);
// x <- e^{i phi} x such that the first component whose modulus is within
// 1e-12 of the largest is real and positive.  partials: kGsNormRows doubles,
// first: kGsNormRows integers.
hipError_t launch_gs_phase(int64_t dim, double2* x, double* partials, int64_t* first, hipStream_t s);

}  // namespace hub
