// Small kernels of several sizes in one launch.
#include "squant_kernels.h"

#include "squant_ks.h"

namespace squant {

kernel_t ks_mixed_kernel(int mode) {
  static const kernel_t k[4] = {squant_channel_ks_mixed<SQUANT_MODE_E>, squant_channel_ks_mixed<SQUANT_MODE_EK>,
                                squant_channel_ks_mixed<SQUANT_MODE_EKC>, squant_channel_ks_mixed<SQUANT_MODE_EC>};
  return k[mode];
}

}  // namespace squant
