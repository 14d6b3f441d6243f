// One launch for a set of layers of different shapes; binary32 weights.
#include "squant_kernels.h"

#include "squant_mixed.h"

namespace squant {

kernel_t mixed_kernel_half(int mode);

kernel_t mixed_kernel(int mode, int wtype) {
  static const kernel_t k[4] = {squant_channel_mixed<SQUANT_MODE_E, false>, squant_channel_mixed<SQUANT_MODE_EK, false>,
                                squant_channel_mixed<SQUANT_MODE_EKC, false>, squant_channel_mixed<SQUANT_MODE_EC, false>};
  return wtype == SQUANT_W_F32 ? k[mode] : mixed_kernel_half(mode);
}

}  // namespace squant
