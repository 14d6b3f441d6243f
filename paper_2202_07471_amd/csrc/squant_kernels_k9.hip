// 3x3 kernels, depthwise ones and stems.
#include "squant_kernels.h"

#include "squant_dw.h"
#include "squant_k9.h"
#include "squant_stem.h"

namespace squant {

kernel_t k9_kernel(int kpt, int threads, int mode, int wtype, bool any) {
  if (any) return k9_any_kernel(kpt, threads, mode);
#define SQ_K9_ROW(T, KPT)                                                                     \
  {squant_channel_k9<T, SQUANT_MODE_E, KPT>, squant_channel_k9<T, SQUANT_MODE_EK, KPT>,       \
   squant_channel_k9<T, SQUANT_MODE_EKC, KPT>, squant_channel_k9<T, SQUANT_MODE_EC, KPT>}
  static const kernel_t k9x1[4] = SQ_K9_ROW(256, 1);
  static const kernel_t k9x2[4] = SQ_K9_ROW(256, 2);
  static const kernel_t k9x4[4] = SQ_K9_ROW(256, 4);
  static const kernel_t k9x4_large[4] = SQ_K9_ROW(1024, 4);
#undef SQ_K9_ROW
  // four kernels per thread in workgroups of exactly two waves (cin 260 .. 512) or one
  // (cin 152 .. 256): weight type and wave count compiled in
#define SQ_K9_ROW_X(WT, NWC)                                                                  \
  {squant_channel_k9<256, SQUANT_MODE_E, 4, WT, NWC>, squant_channel_k9<256, SQUANT_MODE_EK, 4, WT, NWC>, \
   squant_channel_k9<256, SQUANT_MODE_EKC, 4, WT, NWC>, squant_channel_k9<256, SQUANT_MODE_EC, 4, WT, NWC>}
  static const kernel_t k9x4_two_waves[3][4] = {SQ_K9_ROW_X(SQUANT_W_F32, 2), SQ_K9_ROW_X(SQUANT_W_F16, 2),
                                                SQ_K9_ROW_X(SQUANT_W_BF16, 2)};
  static const kernel_t k9x4_one_wave[2][4] = {SQ_K9_ROW_X(SQUANT_W_F32, 1), SQ_K9_ROW_X(kWHalf, 1)};
#undef SQ_K9_ROW_X
  if (kpt == 1) return k9x1[mode];
  if (kpt == 2) return k9x2[mode];
  if (threads == 2 * kWave) return k9x4_two_waves[wtype][mode];
  if (threads == kWave) return k9x4_one_wave[wtype != SQUANT_W_F32][mode];
  return threads <= 256 ? k9x4[mode] : k9x4_large[mode];
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
