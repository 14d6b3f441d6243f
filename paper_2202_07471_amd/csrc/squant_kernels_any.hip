// The kernels that take any shape.
#include "squant_kernels.h"

#include "squant_generic.h"
#include "squant_stream.h"

namespace squant {

__global__ void __launch_bounds__(1024) squant_channel_generic(LaunchArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ GenericShared gs;
  int m;
  const TensorDesc d = locate(a, blockIdx.x, m);
  generic_channel(a, d, m, smem, gs);
}

kernel_t stream_kernel(int mode) {
  static const kernel_t k[4] = {squant_channel_stream<SQUANT_MODE_E>, squant_channel_stream<SQUANT_MODE_EK>,
                                squant_channel_stream<SQUANT_MODE_EKC>, squant_channel_stream<SQUANT_MODE_EC>};
  return k[mode];
}

kernel_t generic_kernel() { return squant_channel_generic; }

}  // namespace squant
