// Instantiation of the batched plain products for float complex vectors.
#include "batch_impl.h"

namespace hub {

hipError_t launch_batch_c64(const ApplyLaunch& L, int nvec, int cw) {
  return cw == 0 ? dev::batch_one<float>(L, nvec) : dev::batch_two<float>(L, nvec, cw);
}

}  // namespace hub
