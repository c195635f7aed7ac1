// Instantiation of the batched plain products for double complex vectors.
#include "batch_impl.h"

namespace hub {

hipError_t launch_batch_c128(const ApplyLaunch& L, int nvec, int cw) {
  return cw == 0 ? dev::batch_one<double>(L, nvec) : dev::batch_two<double>(L, nvec, cw);
}

}  // namespace hub
