// 1x1 / FC kernels: a wave per channel, and several channels per wave.
#include "squant_kernels.h"

#include "squant_k1_rows.h"
#include "squant_k1_team.h"
#include "squant_k1_wave.h"

namespace squant {
namespace {

template <int NV>
kernel_t k1_wave_of(bool channel_stage, bool half, bool tail) {
  static const kernel_t k[2][2][2] = {
      {{squant_channel_k1_wave<SQUANT_MODE_E, NV, false, false>, squant_channel_k1_wave<SQUANT_MODE_E, NV, false, true>},
       {squant_channel_k1_wave<SQUANT_MODE_E, NV, true, false>, squant_channel_k1_wave<SQUANT_MODE_E, NV, true, true>}},
      {{squant_channel_k1_wave<SQUANT_MODE_EKC, NV, false, false>, squant_channel_k1_wave<SQUANT_MODE_EKC, NV, false, true>},
       {squant_channel_k1_wave<SQUANT_MODE_EKC, NV, true, false>, squant_channel_k1_wave<SQUANT_MODE_EKC, NV, true, true>}}};
  return k[channel_stage][half][tail];
}

template <int MODE, int TEAM, int NV, bool HALF>
kernel_t k1_rows_of(bool tail) {
  return tail ? squant_channel_k1_rows<MODE, TEAM, NV, HALF, true> : squant_channel_k1_rows<MODE, TEAM, NV, HALF, false>;
}
template <int TEAM>
kernel_t k1_rows_stage(int nv, bool tail) {
  switch (nv) {
    case 5: return k1_rows_of<SQUANT_MODE_EKC, TEAM, 5, false>(tail);
    case 6: return k1_rows_of<SQUANT_MODE_EKC, TEAM, 6, false>(tail);
    case 7: return k1_rows_of<SQUANT_MODE_EKC, TEAM, 7, false>(tail);
    default: return k1_rows_of<SQUANT_MODE_EKC, TEAM, 8, false>(tail);
  }
}
template <int MODE>
kernel_t k1_rows_half(int team, int nv, bool tail) {  // in vectors of eight
  if (team == 16) return nv <= 6 ? k1_rows_of<MODE, 16, 6, true>(tail) : k1_rows_of<MODE, 16, 8, true>(tail);
  return nv > 6 ? k1_rows_of<MODE, 32, 8, true>(tail) : nullptr;
}

}  // namespace

// Those that k1_rows_min leads to.
kernel_t k1_rows_kernel(int team, int nv, int mode, int wtype, bool tail) {
  const bool stage = mode == SQUANT_MODE_EKC || mode == SQUANT_MODE_EC;
  if (wtype != SQUANT_W_F32)
    return stage ? k1_rows_half<SQUANT_MODE_EKC>(team, nv, tail) : k1_rows_half<SQUANT_MODE_E>(team, nv, tail);
  if (stage) return team == 16 ? k1_rows_stage<16>(nv, tail) : k1_rows_stage<32>(nv, tail);
  if (team != 16 || nv > 6) return nullptr;
  return nv == 5 ? k1_rows_of<SQUANT_MODE_E, 16, 5, false>(tail) : k1_rows_of<SQUANT_MODE_E, 16, 6, false>(tail);
}

kernel_t k1_wave_kernel(int nv, int mode, int wtype, bool tail) {
  const bool stage = mode == SQUANT_MODE_EKC || mode == SQUANT_MODE_EC, half = wtype != SQUANT_W_F32;
  switch (nv) {
    case 2: return k1_wave_of<2>(stage, half, tail);
    case 3: return k1_wave_of<3>(stage, half, tail);
    case 4: return k1_wave_of<4>(stage, half, tail);
    case 5: return k1_wave_of<5>(stage, half, tail);
    case 6: return k1_wave_of<6>(stage, half, tail);
    case 7: return k1_wave_of<7>(stage, half, tail);
    case 8: return k1_wave_of<8>(stage, half, tail);
    default: return nullptr;
  }
}

kernel_t k1_team_kernel(int mode, bool any) {
  if (mode == SQUANT_MODE_EKC || mode == SQUANT_MODE_EC)
    return any ? squant_channel_k1_team<SQUANT_MODE_EKC, true> : squant_channel_k1_team<SQUANT_MODE_EKC, false>;
  return any ? squant_channel_k1_team<SQUANT_MODE_E, true> : squant_channel_k1_team<SQUANT_MODE_E, false>;
}

}  // namespace squant
