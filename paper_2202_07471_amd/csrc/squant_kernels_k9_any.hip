// 3x3 kernels for any channel count and alignment, and several narrow channels per wave.
#include "squant_kernels.h"

#include "squant_k9.h"
#include "squant_k9_team.h"

namespace squant {

kernel_t k9_any_kernel(int kpt, int threads, int mode, int wtype) {
  const bool half = wtype != SQUANT_W_F32;
#define SQ_K9_ROW(T, KPT, WT)                                                                                        \
  {squant_channel_k9<T, SQUANT_MODE_E, KPT, WT, 0, true>, squant_channel_k9<T, SQUANT_MODE_EK, KPT, WT, 0, true>,    \
   squant_channel_k9<T, SQUANT_MODE_EKC, KPT, WT, 0, true>, squant_channel_k9<T, SQUANT_MODE_EC, KPT, WT, 0, true>}
#define SQ_K9_WIDTHS(T, KPT) {SQ_K9_ROW(T, KPT, SQUANT_W_F32), SQ_K9_ROW(T, KPT, kWHalf)}
  static const kernel_t x1[2][4] = SQ_K9_WIDTHS(256, 1), x2[2][4] = SQ_K9_WIDTHS(256, 2), x4[2][4] = SQ_K9_WIDTHS(256, 4);
  static const kernel_t x4_large[2][4] = SQ_K9_WIDTHS(1024, 4);
#undef SQ_K9_WIDTHS
#undef SQ_K9_ROW
  return kpt == 1 ? x1[half][mode] : kpt == 2 ? x2[half][mode] : threads <= 256 ? x4[half][mode] : x4_large[half][mode];
}

kernel_t k9_team_kernel(int mode) {
  static const kernel_t k[4] = {squant_channel_k9_team<SQUANT_MODE_E>, squant_channel_k9_team<SQUANT_MODE_EK>,
                                squant_channel_k9_team<SQUANT_MODE_EKC>, squant_channel_k9_team<SQUANT_MODE_EC>};
  return k[mode];
}

}  // namespace squant
