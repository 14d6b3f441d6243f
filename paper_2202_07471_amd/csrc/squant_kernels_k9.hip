// 3x3 kernels, depthwise ones and stems.
#include "squant_kernels.h"

#include "squant_dw.h"
#include "squant_k9.h"
#include "squant_stem.h"

namespace squant {

kernel_t k9_kernel(int kpt, int threads, int mode, int wtype, bool any) {
  if (any) return k9_any_kernel(kpt, threads, mode, wtype);
  const bool half = wtype != SQUANT_W_F32;
#define SQ_K9_ROW(T, KPT, WT, NWC)                                                                                  \
  {squant_channel_k9<T, SQUANT_MODE_E, KPT, WT, NWC>, squant_channel_k9<T, SQUANT_MODE_EK, KPT, WT, NWC>,           \
   squant_channel_k9<T, SQUANT_MODE_EKC, KPT, WT, NWC>, squant_channel_k9<T, SQUANT_MODE_EC, KPT, WT, NWC>}
#define SQ_K9_WIDTHS(T, KPT, NWC) {SQ_K9_ROW(T, KPT, SQUANT_W_F32, NWC), SQ_K9_ROW(T, KPT, kWHalf, NWC)}
  static const kernel_t k9x1[2][4] = SQ_K9_WIDTHS(256, 1, 0);
  static const kernel_t k9x2[2][4] = SQ_K9_WIDTHS(256, 2, 0);
  static const kernel_t k9x4[2][4] = SQ_K9_WIDTHS(256, 4, 0);
  static const kernel_t k9x4_large[2][4] = SQ_K9_WIDTHS(1024, 4, 0);
  // four kernels per thread in workgroups of exactly two waves (aligned rows of 388 to 512 kernels) or one
  // (152 to 256): wave count compiled in, with two waves the 16-bit type as well
  static const kernel_t k9x4_two_waves[3][4] = {SQ_K9_ROW(256, 4, SQUANT_W_F32, 2), SQ_K9_ROW(256, 4, SQUANT_W_F16, 2),
                                                SQ_K9_ROW(256, 4, SQUANT_W_BF16, 2)};
  static const kernel_t k9x4_one_wave[2][4] = SQ_K9_WIDTHS(256, 4, 1);
#undef SQ_K9_WIDTHS
#undef SQ_K9_ROW
  if (kpt == 1) return k9x1[half][mode];
  if (kpt == 2) return k9x2[half][mode];
  if (threads == 2 * kWave) return k9x4_two_waves[wtype][mode];
  if (threads == kWave) return k9x4_one_wave[half][mode];
  return threads <= 256 ? k9x4[half][mode] : k9x4_large[half][mode];
}

kernel_t dw9_kernel(int mode) {
  static const kernel_t dw9[4] = {squant_channel_dw9<SQUANT_MODE_E>, squant_channel_dw9<SQUANT_MODE_EK>,
                                  squant_channel_dw9<SQUANT_MODE_EKC>, squant_channel_dw9<SQUANT_MODE_EC>};
  return dw9[mode];
}

kernel_t stem_kernel(int mode) {
  static const kernel_t k[4] = {squant_channel_stem<SQUANT_MODE_E>, squant_channel_stem<SQUANT_MODE_EK>,
                                squant_channel_stem<SQUANT_MODE_EKC>, squant_channel_stem<SQUANT_MODE_EC>};
  return k[mode];
}

kernel_t dw_team_kernel(int mode) {
  static const kernel_t k[4] = {squant_channel_dw_team<SQUANT_MODE_E>, squant_channel_dw_team<SQUANT_MODE_EK>,
                                squant_channel_dw_team<SQUANT_MODE_EKC>, squant_channel_dw_team<SQUANT_MODE_EC>};
  return k[mode];
}

}  // namespace squant
