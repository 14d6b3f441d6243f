// One launch for a set of layers of different shapes; 16-bit weights, any shape.
#include "squant_kernels.h"

#include "squant_mixed.h"

namespace squant {

kernel_t mixed_kernel_any_half(int mode) {
  static const kernel_t k[4] = {squant_channel_mixed<SQUANT_MODE_E, true, true>, squant_channel_mixed<SQUANT_MODE_EK, true, true>,
                                squant_channel_mixed<SQUANT_MODE_EKC, true, true>, squant_channel_mixed<SQUANT_MODE_EC, true, true>};
  return k[mode];
}

}  // namespace squant
