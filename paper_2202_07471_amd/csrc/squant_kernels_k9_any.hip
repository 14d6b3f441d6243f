// 3x3 kernels for any channel count and alignment, and several narrow channels per wave.
#include "squant_kernels.h"

#include "squant_k9.h"
#include "squant_k9_team.h"

namespace squant {

kernel_t k9_any_kernel(int kpt, int threads, int mode) {
#define SQ_K9_ROW(T, KPT)                                                                                            \
  {squant_channel_k9<T, SQUANT_MODE_E, KPT, -1, 0, true>, squant_channel_k9<T, SQUANT_MODE_EK, KPT, -1, 0, true>,    \
   squant_channel_k9<T, SQUANT_MODE_EKC, KPT, -1, 0, true>, squant_channel_k9<T, SQUANT_MODE_EC, KPT, -1, 0, true>}
  static const kernel_t x1[4] = SQ_K9_ROW(256, 1), x2[4] = SQ_K9_ROW(256, 2), x4[4] = SQ_K9_ROW(256, 4);
  static const kernel_t x4_large[4] = SQ_K9_ROW(1024, 4);
#undef SQ_K9_ROW
  return kpt == 1 ? x1[mode] : kpt == 2 ? x2[mode] : threads <= 256 ? x4[mode] : x4_large[mode];
}

kernel_t k9_team_kernel(int mode) {
  static const kernel_t k[4] = {squant_channel_k9_team<SQUANT_MODE_E>, squant_channel_k9_team<SQUANT_MODE_EK>,
                                squant_channel_k9_team<SQUANT_MODE_EKC>, squant_channel_k9_team<SQUANT_MODE_EC>};
  return k[mode];
}

}  // namespace squant
