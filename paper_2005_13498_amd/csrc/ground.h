// Kernels of the ground-state Lanczos (ground.hip): complex double, one
// vector.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace hub {

// Iteration q of a run: T's elements, the norm of what an orthogonalisation
// against every vector took out besides them, and 1 / beta (zero for zero),
// which normalises the stored vector q + 1.
struct GsIter {
  double alpha, beta, loss, inv;
};

// The vectors a product is orthogonalised against: `deflate` (may be null)
// first, then the Lanczos vectors first, first + 1, .. of V.  Vector k of V is
// it[k - 1].inv times what is stored; vector 0 and `deflate` are normalised.
struct GsBasis {
  const double2* deflate;
  const double2* V;
  const GsIter* it;
  int64_t dim;
  int first;
  int nb;  // vectors, deflate included
};

constexpr int kGsDotRows = 32;    // most partial rows of the inner products
constexpr int kGsNormRows = 1024;  // most partial rows of the norms

// dotp[rows][2 nb] = partial <b_k, w> with b_k as stored; returns the rows in
// *rows.  prev (may be null): the iteration before, whose beta is summed from
// normp and stored with its inverse.
hipError_t launch_gs_dot(const GsBasis& B, const double2* w, double* dotp, int* rows, const double* normp, int nrows,
                         GsIter* prev, hipStream_t s);
// w <- f w - sum_k b_k <b_k, f w> with the inner products summed from dotp;
// |w|^2 partials (nrows of them) to normp.  all = false, the pass over the
// vectors H v_q overlaps with: f normalises the last vector b, and w is H b as
// stored; it->alpha = Re <b, f w>.  all = true, over every vector: f = 1,
// it->alpha grows by that and it->loss is stored.
hipError_t launch_gs_subtract(const GsBasis& B, double2* w, const double* dotp, int rows, double* normp, int* nrows,
                              GsIter* it, bool all, hipStream_t s);
// beta and its inverse of one iteration from the norm partials.
hipError_t launch_gs_beta(const double* normp, int nrows, GsIter* it, hipStream_t s);
// out = sum_k c[k] V[k], k < m (device c); |out|^2 partials to normp.
hipError_t launch_gs_combine(const double2* V, int64_t dim, int m, const double* c, double2* out, double* normp,
                             int* nrows, hipStream_t s);
// dst = x / |x| with |x|^2 summed from normp (zero stays zero), also to dst2
// if given.
hipError_t launch_gs_scale(int64_t dim, const double2* x, const double* normp, int nrows, double2* dst, double2* dst2,
                           hipStream_t s);
// x = seeded complex standard normal numbers, |x|^2 partials to normp.
hipError_t launch_gs_start(int64_t dim, uint64_t seed, double2* x, double* normp, int* nrows, hipStream_t s);
// x <- e^{i phi} x such that the first component whose modulus is within
// 1e-12 of the largest is real and positive.  partials: kGsNormRows doubles,
// first: kGsNormRows integers.
hipError_t launch_gs_phase(int64_t dim, double2* x, double* partials, int64_t* first, hipStream_t s);

}  // namespace hub
