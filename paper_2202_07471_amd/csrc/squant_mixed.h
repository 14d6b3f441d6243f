// One launch for a set of layers of different shapes (the weight tensors of a network are
// independent problems, Section 4.2).  Every workgroup finds its tensor and output channel
// in the descriptor table, where the host has put the tensor's family, and runs that family's
// channel routine.  A workgroup that evaluates the rules of squant_plan.h itself starts its loads
// behind a chain of scalar steps, the longer the more rules there are (InceptionV3-style set of 1.4
// times the width 80.6 us, 74.5 with the family from the host; of twice the width 147 and 138;
// ResNet-50 set with odd channel counts 22.8 and 21.2; ResNet-18 set 16.3 and 16.05).  The workgroup
// size is the largest any member tensor needs (at most 256); the routines let surplus threads idle.
#pragma once

#include "squant_act.h"
#include "squant_dw.h"
#include "squant_generic.h"
#include "squant_k1_rows.h"
#include "squant_k1_team.h"
#include "squant_k1_wave.h"
#include "squant_k9.h"
#include "squant_ks.h"
#include "squant_plan.h"
#include "squant_stem.h"

namespace squant {

// Compiled for five waves per SIMD (at most 96 VGPRs, what the four-kernel 3x3 routine needs):
// these launches live on the number of resident workgroups.  Measured 2-4 % faster on the
// ResNet-50 and MobileNetV2 sets; eight waves spill in the 3x3 routine and cost ResNet-18 24 %.
// HALF: 16-bit weights.  ANY: carries the routines for other small kernels, for channel counts that
// are no multiple of four and for buffers off their alignment; a launch without such members takes
// the leaner kernel (ResNet-18 and MobileNetV2 sets 5 % faster in it).
// The code starts on 64 KB: these launches take a few microseconds, most of their instructions run for
// the first time on each compute unit, and the time followed the place the linker gave the kernel, which
// any change to a kernel before it moves (the same code on the ResNet-18 set: 16.4 us at offset 0x5400 of
// its 64 KB, 16.7 at 0x2800, 17.05 at 0x4c00).  On 64 KB the kernels before it no longer matter; changes
// inside it still move that time by 2 to 3 % (ResNet-18 sets of 1.1 to 1.35 times the width likewise).
template <int MODE, bool HALF, bool ANY>
__global__ void __launch_bounds__(kMixedMaxThreads)
    __attribute__((amdgpu_waves_per_eu(5), aligned(65536))) squant_channel_mixed(LaunchArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  // one area for whichever routine the workgroup takes
  constexpr size_t kArea = sizeof(K9Shared) > sizeof(K1Shared) ? sizeof(K9Shared) : sizeof(K1Shared);
  __shared__ __align__(16) unsigned char shared[kArea > sizeof(GenericShared) ? kArea : sizeof(GenericShared)];
  // The lists of rows of several channels a wave lie here too, with only the perturbations in dynamic LDS.  LDS is
  // handed out in pieces of 1280 bytes: with the lists there as well, 18 one-wave workgroups fitted a compute unit
  // instead of the 20 that its registers hold (MobileNetV2 set of twice the width 22.7 us, 22.1 now).
  static_assert(sizeof(shared) >= (size_t)kMixedMaxThreads / kWave * kK1RowsListLds, "lists of every wave");
  static_assert((sizeof(shared) + kK1RowsLds + 1279) / 1280 * 1280 * 20 <= 160 * 1024, "20 one-wave workgroups");
  K9Shared& sh = *reinterpret_cast<K9Shared*>(shared);
  GenericShared& gs = *reinterpret_cast<GenericShared*>(shared);
  // one-element kernels: E&K is E and E&C is E&K&C (SQuant-K has nothing to do, Section 3.4)
  constexpr int M1 = (MODE == SQUANT_MODE_EK) ? SQUANT_MODE_E
                     : (MODE == SQUANT_MODE_EC) ? SQUANT_MODE_EKC : MODE;
  constexpr int kWeights = HALF ? kWHalf : SQUANT_W_F32;
  int m;
  TensorDesc d = locate(a, blockIdx.x, m);
  const int family = d.K >> kFamilyShift;
  d.K &= (1 << kFamilyShift) - 1;
  // Per-thread work is chosen from the launch's workgroup size T, not from the variant the
  // tensor would get in a launch of its own: as few kernels / vectors per thread as T allows.
  // The host only admits tensors with cin <= 4T (3x3) or cin <= 16T (1x1).
  const int T = blockDim.x;
  if (family == 9) {
    // Workgroups of two waves, the common ones, have their wide channels compiled for that, and a wave that a narrow
    // channel leaves without a kernel ends at once: the hardware's barrier waits for the waves that are left
    // (ResNet-18 set 16.5 to 16.9 us without the two, 16.1 to 16.3 with).
    if (d.N <= kWave) {
      if (__builtin_amdgcn_readfirstlane((int)threadIdx.x) >= kWave) return;
      k9_channel<MODE, 1, kWeights, 1, ANY>(a, d, m, smem, sh);
    } else if (d.N <= T) {
      k9_channel<MODE, 1, kWeights, 0, ANY>(a, d, m, smem, sh);
    } else if (d.N <= 2 * T) {
      k9_channel<MODE, 2, kWeights, 0, ANY>(a, d, m, smem, sh);
    } else if (T == 2 * kWave) {
      // Keeps the two routines of four kernels a thread apart: the compiler otherwise joins their 16-bit loads ahead of the
      // branch, which took 82 registers for 62 with SQuant-E alone, 96 and 24 bytes of scratch memory for 78 with E&K and 56 bytes
      // with E&K&C (binary16, us so joined and now: ResNet-18 set with E 9.6 and 9.2, with E&K 11.4 and 10.6, of twice the width with
      // E&K&C 52.8 and 43.8, ResNet-50 set of twice the width 90.8 and 83.3; ResNet-18 set with E&K&C 13.6 and 13.7).
      if (HALF) asm volatile("");
      k9_channel<MODE, 4, kWeights, 2, ANY>(a, d, m, smem, sh);
    } else {
      k9_channel<MODE, 4, kWeights, 0, ANY>(a, d, m, smem, sh);
    }
  } else if (family == 1) {
    K1Shared& sh1 = *reinterpret_cast<K1Shared*>(shared);
    const int nvec = (d.N + 3) >> 2;
    if (nvec <= T) k1_channel<M1, 1, 4, HALF, ANY>(a, d, m, smem, sh1);
    else if (nvec <= 2 * T) k1_channel<M1, 2, 4, HALF, ANY>(a, d, m, smem, sh1);
    else if (nvec <= 3 * T) k1_channel<M1, 3, 4, HALF, ANY>(a, d, m, smem, sh1);
    else k1_channel<M1, 4, 4, HALF, ANY>(a, d, m, smem, sh1);
  } else if (family == 3) {
    dw9_channels<MODE>(a, d, m);
  } else if (family == 4) {
    k1_team_dispatch<M1, ANY>(a, d, m);
  } else if (ANY && family == 5) {
    ks_dispatch<MODE, HALF>(a, d, m, smem, sh);
  } else if (family == kFamilyRows) {
    // 16-bit rows come in vectors of eight: a multiple of four may end in half of one
    K1RowsList* lists = reinterpret_cast<K1RowsList*>(shared);
    if (k1_rows_team(d.N) == 16) k1_rows_dispatch<M1, 16, HALF, ANY || HALF>(a, d, m, smem, lists);
    else k1_rows_dispatch<M1, 32, HALF, ANY || HALF>(a, d, m, smem, lists);
  } else if (family == 6) {
    k1_wave_dispatch<M1, HALF, ANY>(a, d, m, smem);
  } else if (family == kFamilyStem) {
    stem_channels<MODE>(a, d, m);
  } else if (family == 7) {
    dw_team_dispatch<MODE>(a, d, m);
  } else if (family == kFamilyBn) {  // (see TensorDesc)
    activation_range(static_cast<const float*>(d.w), d.scales, d.M, d.N != 0, a.n_sigma, a.act_levels_minus_1,
                     static_cast<squant_act_range_t*>(d.out), sh.red_f, reinterpret_cast<float*>(sh.red_i));
  } else {
    generic_channel(a, d, m, smem, gs);
  }
}

}  // namespace squant
