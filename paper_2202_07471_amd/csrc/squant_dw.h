// SQuant kernel for depthwise convolutions with kernels other than 3x3 (cin per group = 1, up to 64
// elements: 5x5, 7x7 ...): an output channel is a single kernel, and a TEAM of 4, 8 or 16
// neighbouring lanes owns it, four consecutive elements a lane, so a wave works on 16, 8 or 4 channels
// at once and a lane moves its four together.  Channels are short, and most of what a wave does is
// spent once for all its channels (reductions, one key after the other, addresses), so the fewer
// lanes a channel has the better.  us with one element a lane (teams of 16, 32 and 64 lanes) and now:
// 60 x [1065, 1, 7, 7] bfloat16 to 4 bit, SQuant-E alone, 16.4 and 8.4, 30 x [3000, 1, 5, 5] to binary32 13.2 and
// 7.9, MobileNetV2-shaped sets with 5x5 kernels to 4 bit 10.3 and 9.0, of 1.4 times the width with 7x7 ones 15.2 and 12.8.
//
// Every step is a butterfly over the team's lanes: absmax, the sum of the perturbations, and the
// k largest same-sign keys one after the other (k = round(|sum|) is rarely above three).
// SQuant-C on a one-kernel channel: after SQuant-K the channel's sum is the kernel's, at most 0.5,
// so nothing flips (E&K&C equals E&K); without SQuant-K (mode E&C) the kernel's one candidate, its
// largest same-sign element, flips when the sum rounds to 1 or more.
#pragma once

#include "squant_common.h"
#include "squant_io.h"
#include "squant_k1_team.h"  // reductions over a team
#include "squant_k9.h"       // rounding constants, pack_low_bytes
#include "squant_plan.h"

namespace squant {

// `item` is the workgroup's index within the tensor: it covers blockDim.x / TEAM channels.
template <int MODE, int TEAM>
__device__ __forceinline__ void dw_team_channels(const LaunchArgs& a, const TensorDesc& d, int item) {
  const int K = d.K, tid = threadIdx.x, i0 = 4 * (tid & (TEAM - 1));  // the lane's first element
  const int per_group = (int)blockDim.x / TEAM;
  const int first = item * per_group, rows = imin2(per_group, d.M - first);
  const int r = tid / TEAM;  // channel first + r
  const bool live = r < rows;
  const int own = live ? imin2(K - i0, 4) : 0;  // elements of the lane, none if <= 0
  const float qmaxf = (float)a.qmax;

  // the workgroup's channels as one range; what a lane reads of the next channel is dropped
  float w[4];
  {
    const uint32_t each = a.wtype == SQUANT_W_F32 ? 4u : 2u;
    const rsrc_t range = make_rsrc(static_cast<const uint8_t*>(d.w) + (size_t)first * K * each, each * (uint32_t)(rows * K));
    const uint32_t at = own > 0 ? each * (uint32_t)(r * K + i0) : 0x40000000u;
    if (a.wtype == SQUANT_W_F32) {
      const vu4 v = buffer_load_u4(range, at, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = __uint_as_float(v[e]);
    } else {  // one by one: of a longer piece the range would drop a last element that fills half a dword
      uint32_t v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = buffer_load_u16(range, at + 2u * e, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = a.wtype == SQUANT_W_BF16 ? widen_bf16(v[e]) : widen_f16(v[e]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = e < own ? w[e] : 0.0f;
  }

  const float amax = team_max_f32<TEAM>(fmaxf(fmaxf(fabsf(w[0]), fabsf(w[1])), fmaxf(fabsf(w[2]), fabsf(w[3]))));
  const float s = amax > 0.0f ? amax / qmaxf : 1.0f;
  if (live && i0 == 0) d.scales[first + r] = s;
  // the reciprocal only where every team of the wave is in its proven range
  const bool fast = __ballot(amax > 0.0f && !(amax >= 0x1p-60f && amax <= 0x1p60f)) == 0ull;
  float x[4];
  if (fast) {
    const float rs = reciprocal(s);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = div_by_reciprocal(w[e], s, rs);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = quotient(w[e], s);
  }
  uint32_t tb[4], pb[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {  // as in k9_round
    const float xc = __builtin_amdgcn_fmed3f(x[e], -qmaxf, qmaxf);
    const float t = xc + kRoundMagic;
    tb[e] = __float_as_uint(t);
    pb[e] = __float_as_uint(__builtin_fmaf((t - kRoundMagic) - xc, 8388608.0f, kQ23Magic));
  }
  uint32_t code = pack_low_bytes(tb[0], tb[1], tb[2], tb[3]);  // code + 128; elements past the kernel: 128

  if (MODE != SQUANT_MODE_E) {
    const int32_t E = team_sum_i32<TEAM>((int32_t)(pb[0] + pb[1] + pb[2] + pb[3] - 4u * kQ23Bias));  // 64 * 2^22 < 2^31
    const int32_t smask = E >> 31;
    const int32_t A = (E ^ smask) - smask;
    const int32_t k = (int32_t)((uint32_t)(A + kHalf - 1) >> 23);
    const int32_t flips = MODE == SQUANT_MODE_EC ? imin2(k, 1) : k;
    // unique keys, larger flips earlier, lower index first on ties; 0: not of the sum's sign
    uint32_t key[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int32_t P = (int32_t)(pb[e] - kQ23Bias), u = (P ^ smask) - smask;
      key[e] = u > 0 ? ((uint32_t)u << 6) | (uint32_t)(63 - (i0 + e)) : 0u;
    }
    if (__ballot(flips > 0) != 0ull) {
      // down to the key of rank `flips`; there are at least that many
      uint32_t least = team_max_u32<TEAM>(umax2(umax2(key[0], key[1]), umax2(key[2], key[3])));
      for (int32_t rank = 1; __ballot(rank < flips && least != 0u) != 0ull; ++rank) {
        const uint32_t next = team_max_u32<TEAM>(next_key_below(key, least));
        least = rank < flips ? next : least;
      }
      uint32_t hit = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) hit |= key[e] >= least && key[e] != 0u ? 1u << (8 * e) : 0u;
      hit = flips > 0 ? hit : 0u;
      code -= (hit ^ (uint32_t)smask) - (uint32_t)smask;  // no carry leaves a biased byte
    }
  }

  // whole fours together, at any alignment; what is left of a kernel by the lane that holds it
  if (own <= 0) return;
  if (a.out_format == SQUANT_OUT_INT8) {
    const rsrc_t out = make_rsrc(static_cast<uint8_t*>(d.out) + (size_t)first * K, (uint32_t)(rows * K));
    const uint32_t at = (uint32_t)(r * K + i0), c = code ^ 0x80808080u;
    if (own == 4) {
      buffer_store_u1_stream(c, out, at, 0);
    } else {
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (e < own) buffer_store_u8(c >> (8 * e), out, at + e);
    }
  } else if (a.out_format == SQUANT_OUT_INT4) {
    const int row = (K + 1) / 2;
    const rsrc_t out = make_rsrc(static_cast<uint8_t*>(d.out) + (size_t)first * row, (uint32_t)(rows * row));
    const uint32_t at = (uint32_t)(r * row + i0 / 2), c = pack_nibbles4(code);
    if (own > 2) buffer_store_u16_stream((uint16_t)c, out, at, 0);  // a missing element leaves 0
    else buffer_store_u8(c, out, at);
  } else {
    const vf4 v = dequant4(code, s);
    if (a.out_format == SQUANT_OUT_BF16) {
      const rsrc_t out = make_rsrc(static_cast<uint8_t*>(d.out) + (size_t)first * K * 2, 2u * (uint32_t)(rows * K));
      const uint32_t at = 2u * (uint32_t)(r * K + i0);
      const vu4 b = {bf16_bits(v.x), bf16_bits(v.y), bf16_bits(v.z), bf16_bits(v.w)};
      if (own == 4) {
        buffer_store_u2_stream(vu2{b.x | (b.y << 16), b.z | (b.w << 16)}, out, at, 0);
      } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
          if (e < own) buffer_store_u16_stream((uint16_t)b[e], out, at + 2u * e, 0);
      }
    } else {  // SQUANT_OUT_F32
      const rsrc_t out = make_rsrc(static_cast<uint8_t*>(d.out) + (size_t)first * K * 4, 4u * (uint32_t)(rows * K));
      const uint32_t at = 4u * (uint32_t)(r * K + i0);
      if (own == 4) {
        buffer_store_u4_stream(__builtin_bit_cast(vu4, v), out, at, 0);
      } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
          if (e < own) buffer_store_u1_stream(__float_as_uint(v[e]), out, at + 4u * e, 0);
      }
    }
  }
}

template <int MODE>
__device__ __forceinline__ void dw_team_dispatch(const LaunchArgs& a, const TensorDesc& d, int item) {
  const int lanes = dw_team_lanes(d.K) / kDwLaneElems;
  if (lanes == 4) dw_team_channels<MODE, 4>(a, d, item);
  else if (lanes == 8) dw_team_channels<MODE, 8>(a, d, item);
  else dw_team_channels<MODE, 16>(a, d, item);
}

template <int MODE>
__global__ void __launch_bounds__(256) squant_channel_dw_team(LaunchArgs a) {
  int item;
  const TensorDesc d = locate(a, blockIdx.x, item);
  dw_team_dispatch<MODE>(a, d, item);
}

}  // namespace squant
