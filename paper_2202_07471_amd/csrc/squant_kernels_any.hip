// The kernels that take any shape.
#include "squant_kernels.h"

#include "squant_act.h"
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

__global__ void __launch_bounds__(256) squant_activation_range_kernel(BnArgs a) {
  __shared__ float red_lo[16], red_hi[16];
  const BnDesc d = a.layer[blockIdx.x];
  activation_range(d.gamma, d.beta, d.channels, d.relu != 0, a.n_sigma, a.levels_minus_1, a.out + d.out_index, red_lo,
                   red_hi);
}

void (*activation_range_kernel())(BnArgs) { return squant_activation_range_kernel; }

kernel_t generic_kernel() { return squant_channel_generic; }

}  // namespace squant
