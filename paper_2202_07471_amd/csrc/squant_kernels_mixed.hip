// One launch for a set of layers of different shapes; binary32 weights, the common shapes.
#include "squant_kernels.h"

#include "squant_mixed.h"

namespace squant {

kernel_t mixed_kernel_plain(int mode) {
  static const kernel_t k[4] = {squant_channel_mixed<SQUANT_MODE_E, false, false>, squant_channel_mixed<SQUANT_MODE_EK, false, false>,
                                squant_channel_mixed<SQUANT_MODE_EKC, false, false>, squant_channel_mixed<SQUANT_MODE_EC, false, false>};
  return k[mode];
}

}  // namespace squant
