// Small kernels other than 3x3.
#include "squant_kernels.h"

#include "squant_ks.h"

namespace squant {
namespace {

// The instantiation for (K, kernels per thread), workgroup size and mode.
template <int K, int KPT, bool HALF>
kernel_t ks_kernel_of(int threads, int mode, bool largest) {
#define SQ_KS_ROW(T)                                                                                      \
  {squant_channel_ks<T, SQUANT_MODE_E, K, KPT, HALF>, squant_channel_ks<T, SQUANT_MODE_EK, K, KPT, HALF>, \
   squant_channel_ks<T, SQUANT_MODE_EKC, K, KPT, HALF>, squant_channel_ks<T, SQUANT_MODE_EC, K, KPT, HALF>}
  static const kernel_t small[4] = SQ_KS_ROW(256);
  if (threads <= 256 || !largest) return small[mode];
  if constexpr (KPT == (1 << ks_max_kpt_log2(K))) {
    static const kernel_t large[4] = SQ_KS_ROW(1024);
    return large[mode];
  }
#undef SQ_KS_ROW
  return small[mode];
}
template <int K, bool HALF>
kernel_t ks_kernel_width(int kpt, int threads, int mode) {
  const bool largest = kpt == (1 << ks_max_kpt_log2(K));
  constexpr int top = 1 << ks_max_kpt_log2(K);
  if (kpt == 1) return ks_kernel_of<K, 1, HALF>(threads, mode, largest);
  if constexpr (top >= 2) if (kpt == 2) return ks_kernel_of<K, 2, HALF>(threads, mode, largest);
  if constexpr (top >= 4) if (kpt == 4) return ks_kernel_of<K, 4, HALF>(threads, mode, largest);
  if constexpr (top >= 8) if (kpt == 8) return ks_kernel_of<K, 8, HALF>(threads, mode, largest);
  return nullptr;
}
template <int K>
kernel_t ks_kernel_k(int kpt, int threads, int mode, int wtype) {
  return wtype == SQUANT_W_F32 ? ks_kernel_width<K, false>(kpt, threads, mode) : ks_kernel_width<K, true>(kpt, threads, mode);
}

}  // namespace

kernel_t ks_kernel(int K, int kpt, int threads, int mode, int wtype) {
  switch (K) {
    case 2: return ks_kernel_k<2>(kpt, threads, mode, wtype);
    case 3: return ks_kernel_k<3>(kpt, threads, mode, wtype);
    case 4: return ks_kernel_k<4>(kpt, threads, mode, wtype);
    case 5: return ks_kernel_k<5>(kpt, threads, mode, wtype);
    case 7: return ks_kernel_k<7>(kpt, threads, mode, wtype);
    case 16: return ks_kernel_k<16>(kpt, threads, mode, wtype);
    case 25: return ks_kernel_k<25>(kpt, threads, mode, wtype);
    case 49: return ks_kernel_k<49>(kpt, threads, mode, wtype);
    default: return nullptr;
  }
}

}  // namespace squant
