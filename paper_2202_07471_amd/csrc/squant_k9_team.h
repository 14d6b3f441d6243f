// SQuant kernel for 3x3 channels of 2 to 32 kernels (first layers with three input channels, grouped
// convolutions, narrow networks): several output channels per wave.
//
// A channel of a few kernels does not fill a wave; with a workgroup per channel the launch is bound
// by the number of workgroups (15 x [3485, 3, 3, 3], 52 thousand channels of 27 weights: 29 us, and
// 0.7 us of memory traffic).  A TEAM of 4, 8, 16 or 32 neighbouring lanes owns a channel, one kernel
// per lane, through the register routines of squant_k9.h; every channel-wide step is a butterfly
// over the team's lanes, with no LDS and no barrier.  SQuant-C takes the candidates with the sign of
// the channel sum one after the other, the largest |v| first, lower kernel on ties: the keys
// (|v| << 5) | (31 - kernel) are unique, and need = round(|sum of at most 32 halves|) is small.
#pragma once

#include "squant_common.h"
#include "squant_io.h"
#include "squant_k9.h"
#include "squant_plan.h"

namespace squant {

template <int TEAM>
__device__ __forceinline__ uint32_t k9_team_max(uint32_t v) {
  v = umax2(v, (uint32_t)dpp_i32<0xB1>((int)v));
  v = umax2(v, (uint32_t)dpp_i32<0x4E>((int)v));
  if (TEAM >= 8) v = umax2(v, (uint32_t)dpp_i32<0x141>((int)v));
  if (TEAM >= 16) v = umax2(v, (uint32_t)dpp_i32<0x140>((int)v));
  if (TEAM >= 32) v = umax2(v, (uint32_t)__shfl_xor((int)v, 16));
  return v;
}
template <int TEAM>
__device__ __forceinline__ int32_t k9_team_sum(int32_t v) {  // 32 kernels of at most 4.5 * 2^23: < 2^31
  v += dpp_i32<0xB1>(v);
  v += dpp_i32<0x4E>(v);
  if (TEAM >= 8) v += dpp_i32<0x141>(v);
  if (TEAM >= 16) v += dpp_i32<0x140>(v);
  if (TEAM >= 32) v += __shfl_xor(v, 16);
  return v;
}

// `item` is the workgroup's index within the tensor: it covers blockDim.x / TEAM channels.
template <int MODE, int TEAM>
__device__ __forceinline__ void k9_team_channels(const LaunchArgs& a, const TensorDesc& d, int item) {
  constexpr bool kChannelStage = MODE == SQUANT_MODE_EKC || MODE == SQUANT_MODE_EC;
  const int N = d.N, tid = threadIdx.x, n = tid & (TEAM - 1);
  const int per_group = (int)blockDim.x / TEAM;
  const int first = item * per_group, rows = imin2(per_group, d.M - first);
  const int r = tid / TEAM;  // channel first + r
  const bool live = r < rows && n < N;
  const float qmaxf = (float)a.qmax;

  // the workgroup's channels as one range; a lane without a kernel reads zeros
  float w[9];
  {
    const uint32_t each = a.wtype == SQUANT_W_F32 ? 36u : 18u;
    const rsrc_t range = make_rsrc(static_cast<const uint8_t*>(d.w) + (size_t)first * N * each, each * (uint32_t)(rows * N));
    const uint32_t at = live ? each * (uint32_t)(r * N + n) : 0x40000000u;
    if (a.wtype == SQUANT_W_F32) {
      k9_load_kernel_row(w, 0, range, at, 0);
    } else {
      const K9Raw16 raw[1] = {k9_load_kernel16(range, at, 0)};
      if (a.wtype == SQUANT_W_BF16) k9_widen16<true>(raw, w);
      else k9_widen16<false>(raw, w);
    }
  }
  float amax = 0.0f;
#pragma unroll
  for (int i = 0; i < 9; ++i) amax = fmaxf(amax, fabsf(w[i]));
  amax = __uint_as_float(k9_team_max<TEAM>(__float_as_uint(amax)));
  const float s = amax > 0.0f ? amax / qmaxf : 1.0f;
  if (live && n == 0) d.scales[first + r] = s;

  K9Kernel kk;
  uint32_t pb[9];
  // the reciprocal only where every team of the wave is in its proven range
  const bool fast = __ballot(amax > 0.0f && !(amax >= 0x1p-60f && amax <= 0x1p60f)) == 0ull;
  if (fast) k9_round<true>(w, s, reciprocal(s), qmaxf, kk, pb);
  else k9_round<false>(w, s, 0.0f, qmaxf, kk, pb);
  if (MODE != SQUANT_MODE_E) {
    int32_t esum = 0;
    k9_flip<MODE, true>(pb, kk, esum, __ballot(live));
    if (kChannelStage) {
      const int32_t ec = k9_team_sum<TEAM>(esum);  // lanes without a kernel: 0
      const int32_t smask = ec >> 31;
      const int32_t mag = (ec ^ smask) - smask;
      uint32_t need = (uint32_t)flips_for(mag);
      // candidates of the wanted sign: bit 23 of the word set for a negative one, bit 24: none
      const bool wanted = live && (kk.cand >> 23) == (smask ? 1u : 0u);
      uint32_t key = wanted ? ((kk.cand & 0x7FFFFFu) << 5) | (uint32_t)(31 - n) : 0u;
      while (__ballot(need > 0) != 0ull) {
        const uint32_t m = k9_team_max<TEAM>(key);
        const bool take = need > 0 && m != 0;
        if (take && key == m) {
          kk.flips ^= kk.cand_bit;
          key = 0;
        }
        need = take ? need - 1 : 0u;  // out of candidates: this team is done
      }
    }
    k9_apply_flips(kk);
  }

  // Packed codes: an odd kernel starts in the middle of a byte, so a lane with an even one stores
  // its nine nibbles and the next lane's.
  const uint32_t p0 = pack_nibbles8(kk.d0, kk.d1), p1 = kk.d2 & 15u;
  const uint32_t q0 = (uint32_t)dpp_i32<0xB1>((int)p0), q1 = (uint32_t)dpp_i32<0xB1>((int)p1);
  if (!live) return;
  const size_t k = (size_t)(first + r) * N + n;
  if (a.out_format == SQUANT_OUT_INT8) {
    uint8_t* out = static_cast<uint8_t*>(d.out) + 9 * k;
    const uint64_t lo = ((uint64_t)kk.d0 | ((uint64_t)kk.d1 << 32)) ^ 0x8080808080808080ull;
    __builtin_memcpy(out, &lo, 8);
    out[8] = (uint8_t)(kk.d2 ^ 0x80u);
  } else if (a.out_format == SQUANT_OUT_INT4) {
    if ((n & 1) == 0) {
      const int row = (9 * N + 1) / 2;
      uint8_t* out = static_cast<uint8_t*>(d.out) + (size_t)(first + r) * row + (9 * n) / 2;
      const bool pair = n + 1 < N;
      __builtin_memcpy(out, &p0, 4);
      out[4] = (uint8_t)(p1 | (pair ? q0 << 4 : 0u));
      if (pair) {
        const uint32_t rest = (q0 >> 4) | (q1 << 28);
        __builtin_memcpy(out + 5, &rest, 4);
      }
    }
  } else {
    float v[9];
    const vf4 a0 = dequant4(kk.d0, s), a1 = dequant4(kk.d1, s);
    v[0] = a0.x; v[1] = a0.y; v[2] = a0.z; v[3] = a0.w;
    v[4] = a1.x; v[5] = a1.y; v[6] = a1.z; v[7] = a1.w;
    v[8] = ((float)(kk.d2 & 255u) - 128.0f) * s;
    if (a.out_format == SQUANT_OUT_BF16) {
      uint16_t* out = static_cast<uint16_t*>(d.out) + 9 * k;
#pragma unroll
      for (int i = 0; i < 9; ++i) out[i] = (uint16_t)bf16_bits(v[i]);
    } else {
      float* out = static_cast<float*>(d.out) + 9 * k;
#pragma unroll
      for (int i = 0; i < 9; ++i) out[i] = v[i];
    }
  }
}

template <int MODE>
__device__ __forceinline__ void k9_team_dispatch(const LaunchArgs& a, const TensorDesc& d, int item) {
  const int lanes = k9_team_lanes(d.N);
  if (lanes == 4) k9_team_channels<MODE, 4>(a, d, item);
  else if (lanes == 8) k9_team_channels<MODE, 8>(a, d, item);
  else if (lanes == 16) k9_team_channels<MODE, 16>(a, d, item);
  else k9_team_channels<MODE, 32>(a, d, item);
}

template <int MODE>
__global__ void __launch_bounds__(256) squant_channel_k9_team(LaunchArgs a) {
  int item;
  const TensorDesc d = locate(a, blockIdx.x, item);
  k9_team_dispatch<MODE>(a, d, item);
}

}  // namespace squant
