// SQuant kernel for channels of two to four kernels of 10 to 64 elements each: the 7x7 (5x5) stem of a network,
// whose input has three colours.  A wave owns a channel, one lane an element of every kernel, so loads are
// contiguous, every step is a reduction over the wave (DPP), and the kernels' chains run side by side; no LDS, no
// barrier.  What belongs to a kernel or to the channel is a scalar, SQuant-C on up to four candidates included.
//
// The generic routine gave such a channel a workgroup and went through LDS with a wave per kernel: 4096 channels of
// [3, 7, 7] took 17.7 us (8.2 here), and in a mixed launch of one-wave workgroups, where one wave does the three kernels
// one after the other, a ResNet-18 set of 0.39 times the width was waiting for them (14.9 us; 7.9 here).
#pragma once

#include "squant_common.h"
#include "squant_io.h"
#include "squant_plan.h"

namespace squant {

// Largest value over the wave (uniform).
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  return __float_as_uint(wave_max_dpp(__uint_as_float(v)));  // compares the bits as integers
}

// SQuant-E alone knows no kernels: the channel's elements side by side, at most four a lane.  A lane per element of a kernel
// left 48 of 64 idle with 4x4 kernels (200 K channels of [3, 4, 4]: 57.2 us, 50.0 through the generic routine).
__device__ __forceinline__ void stem_round_channel(const LaunchArgs& a, const TensorDesc& d, int m) {
  constexpr int kMost = kMaxStemCin;  // kernels of up to 64 elements
  const int lane = (int)(threadIdx.x & (kWave - 1)), L = d.N * d.K;
  const float qmaxf = (float)a.qmax;
  const size_t base = (size_t)m * L;
  float w[kMost], amax = 0.0f;
#pragma unroll
  for (int i = 0; i < kMost; ++i) {
    const int e = lane + i * kWave;
    w[i] = e < L ? load_weight(d.w, base + e, a.wtype) : 0.0f;
  }
#pragma unroll
  for (int i = 0; i < kMost; ++i) amax = fmaxf(amax, fabsf(w[i]));
  amax = wave_max_dpp(amax);
  const float s = amax > 0.0f ? amax / qmaxf : 1.0f;
  if (lane == 0) d.scales[m] = s;
#pragma unroll
  for (int i = 0; i < kMost; ++i) {
    if (i * kWave >= L) break;
    const int e = lane + i * kWave;
    int32_t P;
    const int code = round_and_perturb(w[i], s, qmaxf, P);  // past the channel: 0
    if (a.out_format == SQUANT_OUT_INT4) {
      // even elements store their own nibble and the next one's, which is the next lane's
      const uint32_t next = (uint32_t)dpp_i32<0xB1>(code);
      if (e < L && (e & 1) == 0)
        static_cast<uint8_t*>(d.out)[(size_t)m * ((L + 1) / 2) + e / 2] = (uint8_t)((code & 15) | ((next & 15u) << 4));
    } else if (e >= L) {
      continue;
    } else if (a.out_format == SQUANT_OUT_INT8) {
      static_cast<int8_t*>(d.out)[base + e] = (int8_t)code;
    } else if (a.out_format == SQUANT_OUT_BF16) {
      static_cast<uint16_t*>(d.out)[base + e] = (uint16_t)bf16_bits((float)code * s);
    } else {  // SQUANT_OUT_F32
      static_cast<float*>(d.out)[base + e] = (float)code * s;
    }
  }
}

// `item` is the workgroup's index within the tensor: one channel a wave.
template <int MODE>
__device__ __forceinline__ void stem_channels(const LaunchArgs& a, const TensorDesc& d, int item) {
  constexpr bool kChannelStage = MODE == SQUANT_MODE_EKC || MODE == SQUANT_MODE_EC;
  const int m = item * ((int)blockDim.x / kWave) + __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  if (m >= d.M) return;  // no step of the workgroup follows
  if constexpr (MODE == SQUANT_MODE_E) return stem_round_channel(a, d, m);
  const int lane = (int)(threadIdx.x & (kWave - 1)), K = d.K, N = d.N;
  const bool in = lane < K;
  const float qmaxf = (float)a.qmax;
  const size_t base = (size_t)m * N * K + lane;

  float w[kMaxStemCin];
#pragma unroll
  for (int n = 0; n < kMaxStemCin; ++n) w[n] = n < N && in ? load_weight(d.w, base + (size_t)n * K, a.wtype) : 0.0f;
  float amax = 0.0f;
#pragma unroll
  for (int n = 0; n < kMaxStemCin; ++n) amax = fmaxf(amax, fabsf(w[n]));
  amax = wave_max_dpp(amax);
  const float s = amax > 0.0f ? amax / qmaxf : 1.0f;
  if (lane == 0) d.scales[m] = s;

  int code[kMaxStemCin];
  int32_t P[kMaxStemCin];
#pragma unroll
  for (int n = 0; n < kMaxStemCin; ++n) code[n] = round_and_perturb(w[n], s, qmaxf, P[n]);  // past the kernel: 0, 0

  if (MODE != SQUANT_MODE_E) {
    uint32_t key[kMaxStemCin];  // unique, larger flips earlier, lower index first on ties; 0: not of the sum's sign
    int32_t sm[kMaxStemCin], k[kMaxStemCin], left[kMaxStemCin], want[kMaxStemCin], most = 0, ec = 0;
    uint32_t cand[kMaxStemCin];  // key of the candidate
#pragma unroll
    for (int n = 0; n < kMaxStemCin; ++n) {
      const int32_t E = wave_sum_dpp_small(P[n]);
      sm[n] = E >> 31;
      const int32_t A = (E ^ sm[n]) - sm[n];
      k[n] = MODE == SQUANT_MODE_EC ? 0 : (int32_t)((uint32_t)(A + kHalf - 1) >> 23);
      left[n] = A - (k[n] << 23);  // |sum| after k flips, < 0: over SQuant
      ec += (left[n] ^ sm[n]) - sm[n];
      want[n] = left[n] < 0 ? k[n] - 1 : k[n];  // the candidate's rank: last flipped, first un-flipped
      most = imax2(most, kChannelStage ? want[n] + 1 : k[n]);
      const int32_t u = E == 0 ? imax2(P[n], -P[n]) : (P[n] ^ sm[n]) - sm[n];  // sum 0: either sign may be picked
      key[n] = u > 0 ? ((uint32_t)u << 6) | (uint32_t)(63 - lane) : 0u;
      cand[n] = 0;
    }
    for (int32_t rank = 0; rank < most; ++rank) {
#pragma unroll
      for (int n = 0; n < kMaxStemCin; ++n) {
        const uint32_t top = wave_max_u32(key[n]);
        if (rank == want[n]) cand[n] = top;
        const bool mine = rank < k[n] && key[n] == top && top != 0;
        code[n] -= mine ? (sm[n] ? -1 : 1) : 0;
        key[n] = mine ? 0u : key[n];
      }
    }
    if (kChannelStage) {
      const int sgn = (ec > 0) - (ec < 0);
      const uint32_t kc = (uint32_t)flips_for(ec < 0 ? -ec : ec);
      uint32_t size[kMaxStemCin];  // |v| of the candidates of the channel's sign, 0: none
#pragma unroll
      for (int n = 0; n < kMaxStemCin; ++n) {
        const uint32_t mag = cand[n] >> 6;
        int32_t neg = sm[n];
        if (left[n] == 0 && k[n] == 0)  // a sum of 0: the candidate's own sign
          neg = __builtin_amdgcn_readlane(P[n], 63 - (int)(cand[n] & 63u)) >> 31;
        const bool over = left[n] < 0;
        if (over) neg = ~neg;
        size[n] = cand[n] != 0 && sgn == (neg ? -1 : 1) ? (over ? (uint32_t)kOne - mag : mag) : 0u;
      }
#pragma unroll
      for (int n = 0; n < kMaxStemCin; ++n) {
        uint32_t rank = 0;
#pragma unroll
        for (int i = 0; i < kMaxStemCin; ++i)
          if (i != n) rank += size[i] > size[n] || (size[i] == size[n] && i < n) ? 1u : 0u;
        if (size[n] != 0 && rank < kc && lane == 63 - (int)(cand[n] & 63u)) code[n] -= sgn;
      }
    }
  }

#pragma unroll
  for (int n = 0; n < kMaxStemCin; ++n) {
    if (n >= N) break;
    const size_t at = base + (size_t)n * K;
    if (a.out_format == SQUANT_OUT_INT4) {
      // the even elements of the row store their own nibble and the next one's, 0 past the end
      uint32_t next = (uint32_t)__shfl_down(code[n], 1);
      if (lane == K - 1) next = n + 1 < N ? (uint32_t)__builtin_amdgcn_readlane(code[n + 1 < kMaxStemCin ? n + 1 : n], 0) : 0u;
      const int e = n * K + lane;
      if (in && (e & 1) == 0)
        static_cast<uint8_t*>(d.out)[(size_t)m * ((N * K + 1) / 2) + e / 2] = (uint8_t)((code[n] & 15) | ((next & 15u) << 4));
    } else if (!in) {
      continue;
    } else if (a.out_format == SQUANT_OUT_INT8) {
      static_cast<int8_t*>(d.out)[at] = (int8_t)code[n];
    } else if (a.out_format == SQUANT_OUT_BF16) {
      static_cast<uint16_t*>(d.out)[at] = (uint16_t)bf16_bits((float)code[n] * s);
    } else {  // SQUANT_OUT_F32
      static_cast<float*>(d.out)[at] = (float)code[n] * s;
    }
  }
}

template <int MODE>
__global__ void __launch_bounds__(256) squant_channel_stem(LaunchArgs a) {
  int item;
  const TensorDesc d = locate(a, blockIdx.x, item);
  stem_channels<MODE>(a, d, item);
}

}  // namespace squant
