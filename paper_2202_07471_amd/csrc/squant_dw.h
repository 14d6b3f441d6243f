// SQuant kernel for depthwise convolutions with kernels other than 3x3 (cin per group = 1, up to 64
// elements: 5x5, 7x7 ...): an output channel is a single kernel, and a TEAM of 16, 32 or 64
// neighbouring lanes owns it, one element per lane, so a wave works on four, two or one channels
// and loads and stores are contiguous.  The generic kernel gave each such channel a workgroup:
// the 17 depthwise layers of a MobileNetV2-shaped set with 5x5 kernels (7136 channels of 25
// weights) took 10 of its 18 us.
//
// Every step is a butterfly over the team's lanes: absmax, the sum of the perturbations, and the
// k + 1 largest same-sign keys one after the other (k = round(|sum|) is rarely above three).
// SQuant-C on a one-kernel channel: after SQuant-K the channel's sum is the kernel's, at most 0.5,
// so nothing flips (E&K&C equals E&K); without SQuant-K (mode E&C) the kernel's one candidate, its
// largest same-sign element, flips when the sum rounds to 1 or more.
#pragma once

#include "squant_common.h"
#include "squant_io.h"
#include "squant_plan.h"

namespace squant {

// Largest value / sum over the TEAM lanes a lane belongs to, in every lane.
template <int TEAM>
__device__ __forceinline__ uint32_t dw_team_max(uint32_t v) {
  v = umax2(v, (uint32_t)dpp_i32<0xB1>((int)v));
  v = umax2(v, (uint32_t)dpp_i32<0x4E>((int)v));
  v = umax2(v, (uint32_t)dpp_i32<0x141>((int)v));
  v = umax2(v, (uint32_t)dpp_i32<0x140>((int)v));
  if (TEAM >= 32) v = umax2(v, (uint32_t)__shfl_xor((int)v, 16));
  if (TEAM >= 64) v = umax2(v, (uint32_t)__shfl_xor((int)v, 32));
  return v;
}
template <int TEAM>
__device__ __forceinline__ int32_t dw_team_sum(int32_t v) {  // 64 * 2^22 < 2^31
  v += dpp_i32<0xB1>(v);
  v += dpp_i32<0x4E>(v);
  v += dpp_i32<0x141>(v);
  v += dpp_i32<0x140>(v);
  if (TEAM >= 32) v += __shfl_xor(v, 16);
  if (TEAM >= 64) v += __shfl_xor(v, 32);
  return v;
}

// `item` is the workgroup's index within the tensor: it covers blockDim.x / TEAM channels.
template <int MODE, int TEAM>
__device__ __forceinline__ void dw_team_channels(const LaunchArgs& a, const TensorDesc& d, int item) {
  const int K = d.K, tid = threadIdx.x;
  const int i = tid & (TEAM - 1);
  const int channel = item * ((int)blockDim.x / TEAM) + tid / TEAM;
  const bool live = channel < d.M, in = i < K;
  const int c = live ? channel : d.M - 1;  // surplus teams shadow the last channel, store nothing
  const float qmaxf = (float)a.qmax;
  const float w = in ? load_weight(d.w, (size_t)c * K + i, a.wtype) : 0.0f;

  const float amax = __uint_as_float(dw_team_max<TEAM>(__float_as_uint(fabsf(w))));
  const float s = amax > 0.0f ? amax / qmaxf : 1.0f;
  if (live && i == 0) d.scales[channel] = s;
  int32_t P;
  int code = round_and_perturb(w, s, qmaxf, P);  // an element past the kernel: code 0, P 0

  if (MODE != SQUANT_MODE_E) {
    const int32_t E = dw_team_sum<TEAM>(P);
    const int32_t smask = E >> 31;
    const int32_t A = (E ^ smask) - smask;
    const int32_t k = (int32_t)((uint32_t)(A + kHalf - 1) >> 23);
    const int32_t flips = MODE == SQUANT_MODE_EC ? imin2(k, 1) : k;
    // unique keys, larger flips earlier, lower index first on ties; 0: not of the sum's sign
    const int32_t u = (P ^ smask) - smask;
    uint32_t key = in && u > 0 ? ((uint32_t)u << 6) | (uint32_t)(63 - i) : 0u;
    for (int32_t done = 0; __ballot(done < flips) != 0ull; ++done) {
      const uint32_t m = dw_team_max<TEAM>(key);
      if (done < flips && m != 0 && key == m) {
        code -= smask ? -1 : 1;
        key = 0;
      }
    }
  }

  // packed codes: the even lanes store their own nibble and their neighbour's (0 past the end)
  const uint32_t nibble = in ? (uint32_t)code & 0xFu : 0u;
  const uint32_t next = (uint32_t)dpp_i32<0xB1>((int)nibble);
  if (!live || !in) return;
  const size_t at = (size_t)channel * K + i;
  if (a.out_format == SQUANT_OUT_INT8) {
    static_cast<int8_t*>(d.out)[at] = (int8_t)code;
  } else if (a.out_format == SQUANT_OUT_INT4) {
    if ((i & 1) == 0) static_cast<uint8_t*>(d.out)[(size_t)channel * ((K + 1) / 2) + i / 2] = (uint8_t)(nibble | (next << 4));
  } else if (a.out_format == SQUANT_OUT_BF16) {
    static_cast<uint16_t*>(d.out)[at] = (uint16_t)bf16_bits((float)code * s);
  } else {  // SQUANT_OUT_F32
    static_cast<float*>(d.out)[at] = (float)code * s;
  }
}

template <int MODE>
__device__ __forceinline__ void dw_team_dispatch(const LaunchArgs& a, const TensorDesc& d, int item) {
  const int lanes = dw_team_lanes(d.K);
  if (lanes == 16) dw_team_channels<MODE, 16>(a, d, item);
  else if (lanes == 32) dw_team_channels<MODE, 32>(a, d, item);
  else dw_team_channels<MODE, 64>(a, d, item);
}

template <int MODE>
__global__ void __launch_bounds__(256) squant_channel_dw_team(LaunchArgs a) {
  int item;
  const TensorDesc d = locate(a, blockIdx.x, item);
  dw_team_dispatch<MODE>(a, d, item);
}

}  // namespace squant
