// One launch for a set of layers of different shapes; 16-bit weights, the common shapes.
#include "squant_kernels.h"

#include "squant_mixed.h"

namespace squant {

kernel_t mixed_kernel_plain_half(int mode) {
  static const kernel_t k[4] = {squant_channel_mixed<SQUANT_MODE_E, true, false>, squant_channel_mixed<SQUANT_MODE_EK, true, false>,
                                squant_channel_mixed<SQUANT_MODE_EKC, true, false>, squant_channel_mixed<SQUANT_MODE_EC, true, false>};
  return k[mode];
}

}  // namespace squant
