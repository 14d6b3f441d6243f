// 1x1 / FC kernels, a workgroup per channel.  For one-element kernels E&K equals E and E&C
// equals E&K&C.
#include "squant_kernels.h"

#include "squant_k1.h"
#include "squant_k1_stream.h"
#include "squant_plan.h"

namespace squant {
namespace {

template <int NV, int MODE>
kernel_t k1_of(bool half, bool tail) {
  static const kernel_t k[2][2] = {{squant_channel_k1<MODE, NV, false, false>, squant_channel_k1<MODE, NV, false, true>},
                                   {squant_channel_k1<MODE, NV, true, false>, squant_channel_k1<MODE, NV, true, true>}};
  return k[half][tail];
}
template <int NV>
kernel_t k1_of_nv(bool stage, bool half, bool tail) {
  if constexpr (k1_built(NV, true))
    if (stage) return k1_of<NV, SQUANT_MODE_EKC>(half, tail);
  if constexpr (k1_built(NV, false))
    if (!stage) return k1_of<NV, SQUANT_MODE_E>(half, tail);
  return nullptr;
}

}  // namespace

kernel_t k1_kernel(int nv, int mode, int wtype, bool tail) {
  const bool stage = mode == SQUANT_MODE_EKC || mode == SQUANT_MODE_EC, half = wtype != SQUANT_W_F32;
  switch (nv) {
    case 4: return k1_of_nv<4>(stage, half, tail);
    case 5: return k1_of_nv<5>(stage, half, tail);
    case 6: return k1_of_nv<6>(stage, half, tail);
    case 7: return k1_of_nv<7>(stage, half, tail);
    case 8: return k1_of_nv<8>(stage, half, tail);
    case 10: return k1_of_nv<10>(stage, half, tail);
    case 12: return k1_of_nv<12>(stage, half, tail);
    case 14: return k1_of_nv<14>(stage, half, tail);
    case 16: return k1_of_nv<16>(stage, half, tail);
    default: return nullptr;
  }
}

kernel_t k1_stream_kernel(int mode) {
  return mode == SQUANT_MODE_EKC || mode == SQUANT_MODE_EC ? squant_channel_k1_stream<SQUANT_MODE_EKC>
                                                           : squant_channel_k1_stream<SQUANT_MODE_E>;
}

}  // namespace squant
