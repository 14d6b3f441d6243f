// One launch for a set of layers of different shapes; binary32 weights, any shape.
#include "squant_kernels.h"

#include "squant_mixed.h"

namespace squant {

kernel_t mixed_kernel_any(int mode) {
  static const kernel_t k[4] = {squant_channel_mixed<SQUANT_MODE_E, false, true>, squant_channel_mixed<SQUANT_MODE_EK, false, true>,
                                squant_channel_mixed<SQUANT_MODE_EKC, false, true>, squant_channel_mixed<SQUANT_MODE_EC, false, true>};
  return k[mode];
}

}  // namespace squant
