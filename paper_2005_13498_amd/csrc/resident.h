// Resident stepper of small sectors (resident.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.h"

namespace hub {

// Threads of a resident workgroup, and the most tile elements one thread
// owns per precision (c128, c64): the largest sector the stepper takes has
// kResidentThreads * kResidentEpt[prec] states.
constexpr int kResidentThreads = 1024;
constexpr int kResidentEpt[2] = {8, 16};

// One launch propagates nvec vectors of one sector for all their steps (Eq.
// (time-stepping), or the fourth-order scheme's two exponentials, each split
// into equal substeps), one workgroup per vector.  Device pointers unless
// noted.
struct ResidentArgs {
  int dim_up, dim_dn, gs_up, gs_dn, nc;
  uint8_t up_gclass[8], dn_gclass[8];  // class of each group of four slots
  const uint32_t* up_bits;
  const uint32_t* dn_bits;
  const double* eps_up;  // null without on-site energies
  const double* eps_dn;
  const uint16_t* up_tab;  // grouped tables [dim_up][gs_up], [dim_dn][gs_dn]
  const uint16_t* dn_tab;
  double U, norm_inf, tol, tau;  // tau: the length of one Krylov solve, dt / (n_exp substeps)
  int m_max, n_steps, nvec;
  int n_exp;     // exponentials per step (1: midpoint rule, 2: the fourth-order commutator-free scheme)
  int substeps;  // equal Krylov solves per exponential
  const double* coef_mid;  // [nvec][n_steps][n_exp][2 nc]: class coefficients of each exponential of each step
  const double* coef_obs;  // [nvec][n_steps + 1][2 nc] at the sample times, or null (no observables)
  void* v;                 // [nvec][dim] states, advanced in place
  void* slots;             // [nvec][m_max][dim] Krylov vectors u_1 .. u_{m_max - 1}
  CombineLog* log;         // [n_steps][nvec]
  double* obs;             // [n_steps + 1][nvec][kObsQ]: <D>, docc, |x|^2, Re <x|K(t)|x>
  int32_t* done;           // [nvec] steps whose results are in (a vector stops at m_max or non-finite)
};

// LDS bytes of a resident workgroup: the tables, strings and on-site energies
// (16-byte aligned pieces in the kernel's order), then the tile with a zero
// column and a zero row, (dim_up + 1) (dim_dn + 1) elements.  wide: hop table
// entries of 32 bits instead of 16.
inline size_t resident_lds_bytes(int dim_up, int dim_dn, int gs_up, int gs_dn, bool eps, int prec, bool wide = false) {
  auto a16 = [](size_t b) { return (b + 15) & ~size_t(15); };
  const size_t gb = wide ? 16 : 8;  // bytes of a group of four entries
  size_t t = a16(size_t(dim_dn) * (gs_dn / 4) * gb) + a16(size_t(dim_up) * (gs_up / 4) * gb) +
             a16(size_t(dim_up) * 4) + a16(size_t(dim_dn) * 4);
  if (eps) t += a16(size_t(dim_up) * 8) + a16(size_t(dim_dn) * 8);
  return t + size_t(dim_up + 1) * (dim_dn + 1) * (prec == 0 ? 16 : 8);
}

// Vectors from which the resident stepper is the faster one for its larger
// instantiations (1: at any number).  With 12 or 16 complex64 elements per
// thread it spills, and the launch path has four groups of eight vectors in
// flight, of fewer where the tile is long.  us for three steps, resident /
// launches, at 8, 12, 24, 32 and 48 vectors: 9,075 states (55 x 165) 501 / 456,
// 510 / 561, 519 / 619, 529 / 662, 590 / -; 10,584 (84 x 126) 665 / 507, 674 /
// 601, 690 / 693, 711 / 710, 808 / -; 15,876 (126 x 126) 1,057 / 507, 1,064 /
// 593, 1,151 / 697, 1,195 / 726, 1,219 / 1,264; 12 x 924 692 / 689, 697 / 1,145,
// 710 / 1,835, 726 / 2,387; 924 x 12 701 / 660, 707 / 775, 718 / 857, 737 / 929;
// 14 x 1,001 784 / 669, 788 / 1,161, 814 / 1,822; 1,001 x 14 866 / 623, 871 /
// 771, 891 / 857, 969 / 933, 1,006 / 1,613; at 4 and 8 13 x 715 481 / 466, 488 /
// 565.
inline int resident_min_vectors(int prec, int dim_up, int dim_dn) {
  const int64_t dim = static_cast<int64_t>(dim_up) * dim_dn;
  if (prec == 0 || dim <= 8 * kResidentThreads) return 1;
  constexpr int kLong = 768;
  const bool longer = dim_dn >= kLong || (dim_up >= kLong && dim <= 12 * kResidentThreads);
  if (dim <= 9600) return dim_dn >= 512 ? 5 : 9;
  return longer ? 9 : 33;
}

// Dynamic LDS the resident kernel of `prec` may use on this device (0 if none).
int resident_lds_limit(int prec);

// Launches nvec workgroups; returns hipErrorInvalidValue when the sector does
// not fit (dimension or LDS).
hipError_t launch_resident(int prec, const ResidentArgs& a, size_t lds, hipStream_t s);

}  // namespace hub
