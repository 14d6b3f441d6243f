// SQuant kernel for 1x1 / FC channels that fit one wave: a wave owns a whole output channel.
//
// A channel of one or two thousand weights keeps a wave busy for about a microsecond, most of it
// waiting for its weights and then for the steps of the channel stage, which follow each other.
// With the wave as the unit (squant_k1.h with WAVE) every step runs without a workgroup barrier;
// a wave of a large launch walks up to kK1WaveSpan consecutive channels and asks for the next channel's
// weights as soon as the current ones are widened or consumed, so the loads travel while the wave
// works.  Every wave of the workgroup has an LDS area of its own; the waves never meet.
#pragma once

#include "squant_k1.h"
#include "squant_plan.h"

namespace squant {

// A wave's LDS area: the ranking list and the lanes' owner masks (at most 32 elements a lane).
struct alignas(16) K1WaveSel : K1List {
  uint32_t owner[kWave];
};

template <int MODE, int NV, int VE, bool HALF, bool TAIL, bool PREFETCH>
__device__ __forceinline__ void k1_wave_channels(const LaunchArgs& a, const TensorDesc& d, int c0, int c1,
                                                 K1WaveSel& sel) {
  constexpr int NE = 4 * NV;
  const int N = d.N;
  const size_t row = (size_t)N * (HALF ? 2 : 4);
  uint32_t raw[HALF ? NE / 2 : NE], tail;
  auto load = [&](int m) {
    k1_load<NE, VE, HALF, TAIL>(static_cast<const uint8_t*>(d.w) + (size_t)m * row, N, k1_tid<true>(), kWave, raw, tail);
  };
  if (PREFETCH && c0 < c1) load(c0);
#pragma unroll 1
  for (int m = c0; m < c1; ++m) {
    if (!PREFETCH) load(m);
    float w[NE];
    uint32_t code[NE / 4];
    k1_widen<NE, VE, HALF, TAIL>(raw, tail, a.wtype == SQUANT_W_BF16, N, k1_tid<true>(), kWave, w);
    if (PREFETCH && m + 1 < c1) load(m + 1);
    const float s = k1_solve<MODE, NE, VE, true, HALF>(w, N, (float)a.qmax, a.rcp_qmax, sel, sel.owner, code);
    k1_sync<true>();  // the channel's last LDS access
    // The next channel's weights are waited for here, before this one's stores: loads and stores
    // complete in one order, so a wait at the loop's head would also wait for the stores.
    if (PREFETCH) {
#pragma unroll
      for (auto& r : raw) asm volatile("" : "+v"(r));
      if (TAIL && HALF) asm volatile("" : "+v"(tail));
    }
    const int lane = k1_tid<true>();
    if (lane == 0) d.scales[m] = s;
    k1_emit_as<NE, VE, TAIL>(a.out_format, code, d.out, m, N, s, lane, kWave);
  }
}

// `item` is the workgroup's index within the tensor: each of its waves takes a.wave_span
// channels.  smem: one K1WaveSel per wave.
template <int MODE, int NV, int VE, bool HALF, bool TAIL, bool PREFETCH>
__device__ __forceinline__ void k1_wave_item(const LaunchArgs& a, const TensorDesc& d, int item,
                                             unsigned char* smem) {
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), waves = (int)blockDim.x / kWave;
  const int c0 = (item * waves + wave) * a.wave_span;
  const int c1 = c0 + a.wave_span < d.M ? c0 + a.wave_span : d.M;
  k1_wave_channels<MODE, NV, VE, HALF, TAIL, PREFETCH>(a, d, c0, c1, reinterpret_cast<K1WaveSel*>(smem)[wave]);
}

// For the mixed kernel: vectors per lane from the channel's length, 2 to 8; without the
// prefetch, whose registers that kernel does not have.
template <int MODE, bool HALF, bool TAIL>
__device__ __forceinline__ void k1_wave_dispatch(const LaunchArgs& a, const TensorDesc& d, int item,
                                                 unsigned char* smem) {
  switch (k1_wave_nv(d.N + 3)) {
    case 2: k1_wave_item<MODE, 2, 4, HALF, TAIL, false>(a, d, item, smem); break;
    case 3: k1_wave_item<MODE, 3, 4, HALF, TAIL, false>(a, d, item, smem); break;
    case 4: k1_wave_item<MODE, 4, 4, HALF, TAIL, false>(a, d, item, smem); break;
    case 5: k1_wave_item<MODE, 5, 4, HALF, TAIL, false>(a, d, item, smem); break;
    case 6: k1_wave_item<MODE, 6, 4, HALF, TAIL, false>(a, d, item, smem); break;
    case 7: k1_wave_item<MODE, 7, 4, HALF, TAIL, false>(a, d, item, smem); break;
    default: k1_wave_item<MODE, 8, 4, HALF, TAIL, false>(a, d, item, smem); break;
  }
}

// One kernel per vector count.  The next channel's weights share the registers with the
// current channel's perturbations and codes.  Five vectors are held to
// 80 VGPRs, 72 in 16 bits: the compiler left at five waves a SIMD takes 79 or 85, 71 or 79, as small changes elsewhere have it
// (to int8, us with 85 / 79 and so: 32 x [1224, 1224] binary32 45.4, 43.4; 32 x [1100, 1100] binary32 39.3, 37.9, bfloat16 33.9, 31.9).
template <int MODE, int NV, bool HALF, bool TAIL>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(NV <= 3 ? 8 : NV == 4 ? 6 : NV == 5 ? (HALF ? 7 : 6) : NV <= 6 ? 5 : 4)))
    squant_channel_k1_wave(LaunchArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];  // one K1WaveSel per wave
  int item;
  const TensorDesc d = locate(a, blockIdx.x, item);
  k1_wave_item<MODE, NV, k1_ve<NV, HALF>(), HALF, TAIL, true>(a, d, item, smem);
}

}  // namespace squant
