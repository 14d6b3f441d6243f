// SQuant kernel for short 1x1 / FC channels (cin <= 256, any length and alignment): several
// output channels per wave.
//
// A channel of a few hundred bytes does not fill a wave, let alone a workgroup: with one
// wave per channel the fixed work of the wave (reductions, search, barriers) outweighs the
// channel's own, and a batch of such layers ran at 5-30 % of the memory bandwidth.  Here a TEAM of 4, 8 or 16 neighbouring lanes owns a channel, so a wave works
// on 16, 8 or 4 channels at once; a lane holds NV 16-byte vectors of its channel (lane l of
// the team has vectors l, l + TEAM, ...).  Every channel-wide step is a butterfly over the
// team's lanes with DPP (quad permutes, then the 8- and 16-lane mirrors): no LDS, no barrier,
// loads and stores fully coalesced, and all lanes of the wave run the same instructions.
//
// SQuant-C on such a channel (every element its own candidate, Section 3.4): the `need`
// largest |P| with the sign of the channel sum flip, lowest index first on ties.  With at
// most 256 candidates per team this is done by repeated arg-max: keys are
// (u << 8) | (255 - index) with u = |P| for the eligible elements (unique, so the maximum
// names one element and prefers the lower index among equal |P|); each step takes the
// team-wide maximum, and the lane that holds it moves on to its next key.  The
// wave loops until every one of its teams has its `need` elements or runs out of
// candidates (typically 2-6 steps: need = round(|sum of cin perturbations|)).
//
// Bound by vector instructions.  The scale, its reciprocal, rounding, packing and keys are those of the 3x3 kernel (three-operation
// forms, a magic addition that leaves the code in a byte, biased perturbations); with divisions, a conversion per code and
// element-wise 16-bit stores before, 20 M weights took, us before and now: cin 128 bfloat16 to 4 bit 27.2 and 24.7, 200 to int8 32.9 and
// 29.9, 256 27.3 and 24.4, 181 binary32 25.3 and 22.9, 64 25.8 and 25.0; ResNet-50 set of 0.71 times the width 21.0 and 20.7.
#pragma once

#include "squant_common.h"
#include "squant_io.h"
#include "squant_k9.h"  // rounding constants, pack_low_bytes
#include "squant_plan.h"

namespace squant {

// Both rows' values of v in a pair of rows of 16 lanes: x from the even row, y from the odd one.
__device__ __forceinline__ vu2 row_pair(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return vu2{r[0], r[1]};
#else
  return vu2{v, v};
#endif
}

// Reductions over the TEAM (4, 8, 16 or 32) lanes a lane belongs to; every lane gets the result.
template <int TEAM>
__device__ __forceinline__ float team_max_f32(float v) {
  v = fmaxf(v, dpp_f32<0xB1>(v));                   // quad_perm [1,0,3,2]
  v = fmaxf(v, dpp_f32<0x4E>(v));                   // quad_perm [2,3,0,1]
  if (TEAM >= 8) v = fmaxf(v, dpp_f32<0x141>(v));   // row_half_mirror
  if (TEAM >= 16) v = fmaxf(v, dpp_f32<0x140>(v));  // row_mirror
  if (TEAM >= 32) {
    const vu2 r = row_pair(__float_as_uint(v));
    v = fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
  }
  return v;
}
template <int TEAM>
__device__ __forceinline__ uint32_t team_max_u32(uint32_t x) {
  int v = (int)x;
  v = (int)max((uint32_t)v, (uint32_t)dpp_i32<0xB1>(v));
  v = (int)max((uint32_t)v, (uint32_t)dpp_i32<0x4E>(v));
  if (TEAM >= 8) v = (int)max((uint32_t)v, (uint32_t)dpp_i32<0x141>(v));
  if (TEAM >= 16) v = (int)max((uint32_t)v, (uint32_t)dpp_i32<0x140>(v));
  if (TEAM >= 32) {
    const vu2 r = row_pair((uint32_t)v);
    v = (int)max(r.x, r.y);
  }
  return (uint32_t)v;
}
template <int TEAM>
__device__ __forceinline__ int32_t team_sum_i32(int32_t x) {  // modulo 2^32
  uint32_t v = (uint32_t)x;
  v += (uint32_t)dpp_i32<0xB1>((int)v);
  v += (uint32_t)dpp_i32<0x4E>((int)v);
  if (TEAM >= 8) v += (uint32_t)dpp_i32<0x141>((int)v);
  if (TEAM >= 16) v += (uint32_t)dpp_i32<0x140>((int)v);
  if (TEAM >= 32) {
    const vu2 r = row_pair(v);
    v = r.x + r.y;
  }
  return (int32_t)v;
}

typedef uint32_t u32_byte __attribute__((aligned(1)));
typedef uint32_t u32_half __attribute__((aligned(2)));
typedef uint16_t u16_byte __attribute__((aligned(1)));

// `item` is the workgroup's index within the tensor: it covers blockDim.x / TEAM channels.
//   TAIL  any cin and any alignment: rows are read through the descriptor of the workgroup's
//         channels, the elements behind a row's end (the next row's) are dropped, and the last,
//         partial vector of a row is stored element by element
template <int MODE, int TEAM, int NV, bool TAIL>
__device__ __forceinline__ void k1_team_channels(const LaunchArgs& a, const TensorDesc& d, int item) {
  constexpr bool kChannelStage = MODE == SQUANT_MODE_EKC || MODE == SQUANT_MODE_EC;
  constexpr int NE = 4 * NV;
  const int tid = threadIdx.x;
  const int per_group = (int)blockDim.x / TEAM;
  const int l = tid & (TEAM - 1);  // lane within the team
  const int channel = item * per_group + tid / TEAM;
  const bool live = channel < d.M;
  const int c = live ? channel : d.M - 1;  // surplus teams shadow the last channel, store nothing
  const int N = d.N;
  const float qmaxf = (float)a.qmax;

  const int nvec = TAIL ? (N + 3) >> 2 : N >> 2;
  float w[NE];
  if (TAIL) {
    const int first = item * per_group, rows = imin2(per_group, d.M - first);
    const uint32_t each = a.wtype == SQUANT_W_F32 ? 4u : 2u;
    const rsrc_t range = make_rsrc(static_cast<const uint8_t*>(d.w) + (size_t)first * N * each, (uint32_t)rows * N * each);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int n = 4 * (l + j * TEAM);  // first element of this vector
      const uint32_t at = each * (uint32_t)((c - first) * N + n);
      if (a.wtype == SQUANT_W_F32) {
        const vu4 v = buffer_load_u4(range, at, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) w[4 * j + e] = n + e < N ? __uint_as_float(v[e]) : 0.0f;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t h = buffer_load_u16(range, at + 2u * e, 0);
          const float v = a.wtype == SQUANT_W_BF16 ? widen_bf16(h) : widen_f16(h);
          w[4 * j + e] = n + e < N ? v : 0.0f;
        }
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int idx = l + j * TEAM;
      const bool in = idx < nvec;
      const size_t at = (size_t)c * N + 4 * (size_t)(in ? idx : 0);
      float v0, v1, v2, v3;
      if (a.wtype == SQUANT_W_F32) {
        const vf4 v = load_global_f4(static_cast<const float*>(d.w) + at);
        v0 = v.x; v1 = v.y; v2 = v.z; v3 = v.w;
      } else {
        const uint32_t* p = reinterpret_cast<const uint32_t*>(static_cast<const uint16_t*>(d.w) + at);
        const bool bf16 = a.wtype == SQUANT_W_BF16;
        widen_pair(load_global_u1(p), bf16, v0, v1);
        widen_pair(load_global_u1(p + 1), bf16, v2, v3);
      }
      w[4 * j] = in ? v0 : 0.0f; w[4 * j + 1] = in ? v1 : 0.0f;
      w[4 * j + 2] = in ? v2 : 0.0f; w[4 * j + 3] = in ? v3 : 0.0f;
    }
  }

  float amax = 0.0f;
#pragma unroll
  for (int e = 0; e < NE; e += 2) amax = fmaxf(fmaxf(amax, fabsf(w[e])), fabsf(w[e + 1]));
  amax = team_max_f32<TEAM>(amax);
  // the reciprocal path only where every team of the wave is in its range (same quotients
  // either way; the choice must be the same for the whole wave)
  const bool fast = __ballot(!scale_is_normal(amax)) == 0ull;
  const float s = channel_scale(amax, qmaxf, a.rcp_qmax, fast);
  if (live && l == 0) d.scales[channel] = s;
  if (fast) {
    const float rs = reciprocal(s);
#pragma unroll
    for (int e = 0; e < NE; ++e) w[e] = div_by_reciprocal(w[e], s, rs);  // the IEEE quotient either way
  } else {
#pragma unroll
    for (int e = 0; e < NE; ++e) w[e] = quotient(w[e], s);
  }

  // SQuant-E as in k9_round: codes + 128, four to a dword, and biased perturbations
  uint32_t code[NV], pb[NE], biased = 0;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    uint32_t tb[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float xc = __builtin_amdgcn_fmed3f(w[4 * j + e], -qmaxf, qmaxf);
      const float t = xc + kRoundMagic;
      tb[e] = __float_as_uint(t);
      if (kChannelStage) {
        pb[4 * j + e] = __float_as_uint(__builtin_fmaf((t - kRoundMagic) - xc, 8388608.0f, kQ23Magic));
        biased += pb[4 * j + e];
      }
    }
    code[j] = pack_low_bytes(tb[0], tb[1], tb[2], tb[3]);
  }

  if (kChannelStage) {
    const int32_t ec = team_sum_i32<TEAM>((int32_t)(biased - (uint32_t)NE * kQ23Bias));
    const int32_t mag = ec < 0 ? -ec : ec;
    const int32_t kc = (int32_t)flips_for(mag);
    uint32_t need = (uint32_t)(kc > N ? N : kc);  // the same in every lane of a team
    // unique keys: |P| above 255 - index for the elements with the sign of the sum, below 256 for the others
    const uint32_t sm = (uint32_t)(ec >> 31), zero = kQ23Bias ^ sm;  // pb ^ sm - zero: P for a positive sum, -P for a negative one
    uint32_t key[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const uint32_t n = 4 * (uint32_t)(l + (e >> 2) * TEAM) + (e & 3);
      key[e] = (__builtin_elementwise_sub_sat(pb[e] ^ sm, zero) << 8) | (255u - n);
    }
    // Every lane offers its largest key not yet taken; each step takes the largest
    // offer of the team, and its lane moves on to its next key: 1.5 instructions an element and step.
    // (Marking the element and clearing its key in every step took four; cin 180: 26.6 -> 22.5 us for
    // 64 x [1024, 180].)
    uint32_t offer = 0, taken = ~0u;  // taken: the lane's smallest key that flips
#pragma unroll
    for (int e = 0; e < NE; e += 2) offer = umax3(offer, key[e], key[e + 1]);
    while (__ballot(need > 0) != 0ull) {
      const uint32_t m = team_max_u32<TEAM>(offer);
      const bool take = need > 0 && m >= 256u;
      const uint32_t next = next_key_below(key, offer);
      const bool mine = take && offer == m;
      taken = mine ? m : taken;
      offer = mine ? next : offer;
      need = take ? need - 1 : 0u;  // out of candidates: this team is done
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      uint32_t hit = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) hit |= key[4 * j + e] >= taken ? 1u << (8 * e) : 0u;
      code[j] -= (hit ^ sm) - sm;  // one step against the sum; no carry leaves a biased byte
    }
  }

  if (!live) return;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int idx = l + j * TEAM;
    if (idx >= nvec) continue;
    const size_t at = (size_t)channel * N + 4 * (size_t)idx;  // first element of this vector
    const int left = TAIL ? N - 4 * idx : 4;                  // elements of it inside the row
    const bool whole = !TAIL || left >= 4;
    if (a.out_format == SQUANT_OUT_INT8) {
      uint32_t packed = code[j] ^ 0x80808080u;
      int8_t* out = static_cast<int8_t*>(d.out) + at;
      if (!TAIL) store_global_u1(out, packed);
      else if (whole) *reinterpret_cast<u32_byte*>(out) = packed;
      else
        for (int e = 0; e < left; ++e) out[e] = (int8_t)(packed >> (8 * e));
    } else if (a.out_format == SQUANT_OUT_INT4) {
      const uint32_t packed = pack_nibbles4(code[j]);
      uint8_t* out = static_cast<uint8_t*>(d.out) + (size_t)channel * ((N + 1) / 2) + 2 * (size_t)idx;
      if (!TAIL) store_global_u16(out, (uint16_t)packed);
      else if (left >= 3) *reinterpret_cast<u16_byte*>(out) = (uint16_t)packed;
      else out[0] = (uint8_t)packed;
    } else {
      const vf4 v = dequant4(code[j], s);
      if (a.out_format == SQUANT_OUT_BF16) {
        uint16_t* out = static_cast<uint16_t*>(d.out) + at;
        if (whole) {
          const uint32_t lo = bf16_bits(v.x) | (bf16_bits(v.y) << 16), hi = bf16_bits(v.z) | (bf16_bits(v.w) << 16);
          reinterpret_cast<u32_half*>(out)[0] = lo;
          reinterpret_cast<u32_half*>(out)[1] = hi;
        } else {
#pragma unroll
          for (int e = 0; e < 3; ++e)
            if (e < left) out[e] = (uint16_t)bf16_bits(v[e]);
        }
      } else {  // SQUANT_OUT_F32
        float* out = static_cast<float*>(d.out) + at;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (whole || e < left) out[e] = v[e];
      }
    }
  }
}

// Picks TEAM and NV from cin (<= kMaxTeamCin): the smallest team whose lanes hold the channel
// with one vector each, then 16 lanes with two or four vectors.
template <int MODE, bool TAIL>
__device__ __forceinline__ void k1_team_dispatch(const LaunchArgs& a, const TensorDesc& d, int item) {
  const int N = d.N;
  if (N <= 16) k1_team_channels<MODE, 4, 1, TAIL>(a, d, item);
  else if (N <= 32) k1_team_channels<MODE, 8, 1, TAIL>(a, d, item);
  else if (N <= 64) k1_team_channels<MODE, 16, 1, TAIL>(a, d, item);
  else if (N <= 128) k1_team_channels<MODE, 16, 2, TAIL>(a, d, item);
  else k1_team_channels<MODE, 16, 4, TAIL>(a, d, item);
}

// Compiled for eight waves per SIMD (64 VGPRs instead of 66: measured 1-4 % faster).
template <int MODE, bool TAIL>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(8))) squant_channel_k1_team(LaunchArgs a) {
  int m;
  const TensorDesc d = locate(a, blockIdx.x, m);
  k1_team_dispatch<MODE, TAIL>(a, d, m);
}

}  // namespace squant
