// 1x1 / FC kernels, a workgroup per channel.  For one-element kernels E&K equals E and E&C
// equals E&K&C.
#include "squant_kernels.h"

#include "squant_k1.h"
#include "squant_k1_stream.h"

namespace squant {
namespace {

template <int NV>
kernel_t k1_of(bool channel_stage, bool half, bool tail) {
  static const kernel_t k[2][2][2] = {
      {{squant_channel_k1<SQUANT_MODE_E, NV, false, false>, squant_channel_k1<SQUANT_MODE_E, NV, false, true>},
       {squant_channel_k1<SQUANT_MODE_E, NV, true, false>, squant_channel_k1<SQUANT_MODE_E, NV, true, true>}},
      {{squant_channel_k1<SQUANT_MODE_EKC, NV, false, false>, squant_channel_k1<SQUANT_MODE_EKC, NV, false, true>},
       {squant_channel_k1<SQUANT_MODE_EKC, NV, true, false>, squant_channel_k1<SQUANT_MODE_EKC, NV, true, true>}}};
  return k[channel_stage][half][tail];
}

}  // namespace

kernel_t k1_kernel(int nv, int mode, int wtype, bool tail) {
  const bool stage = mode == SQUANT_MODE_EKC || mode == SQUANT_MODE_EC, half = wtype != SQUANT_W_F32;
  switch (nv) {
    case 1: return k1_of<1>(stage, half, tail);
    case 2: return k1_of<2>(stage, half, tail);
    case 3: return k1_of<3>(stage, half, tail);
    case 4: return k1_of<4>(stage, half, tail);
    case 5: return k1_of<5>(stage, half, tail);
    case 6: return k1_of<6>(stage, half, tail);
    case 7: return k1_of<7>(stage, half, tail);
    case 8: return k1_of<8>(stage, half, tail);
    case 10: return k1_of<10>(stage, half, tail);
    case 12: return k1_of<12>(stage, half, tail);
    case 14: return k1_of<14>(stage, half, tail);
    case 16: return k1_of<16>(stage, half, tail);
    default: return nullptr;
  }
}

kernel_t k1_stream_kernel(int mode) {
  return mode == SQUANT_MODE_EKC || mode == SQUANT_MODE_EC ? squant_channel_k1_stream<SQUANT_MODE_EKC>
                                                           : squant_channel_k1_stream<SQUANT_MODE_E>;
}

}  // namespace squant
