// The kernels as the host side sees them: one getter per family, each defined in the
// translation unit that instantiates the family (squant_kernels_*.hip, compiled in parallel).
#pragma once

#include <hip/hip_runtime.h>

#include "squant_act.h"
#include "squant_common.h"

namespace squant {

typedef void (*kernel_t)(LaunchArgs);

// mode: squant_mode_t, wtype: squant_wtype_t, threads: of the workgroup, tail: some channel is
// no whole number of 16-byte vectors, any: some channel count is no multiple of four or some
// buffer off its alignment.
kernel_t k9_kernel(int kpt, int threads, int mode, int wtype, bool any);
kernel_t k9_any_kernel(int kpt, int threads, int mode, int wtype);
kernel_t k9_team_kernel(int mode);
kernel_t dw9_kernel(int mode);
kernel_t dw_team_kernel(int mode);
kernel_t ks_kernel(int K, int kpt, int threads, int mode, int wtype);
kernel_t k1_kernel(int nv, int mode, int wtype, bool tail);
kernel_t k1_wave_kernel(int nv, int mode, int wtype, bool tail);
kernel_t k1_rows_kernel(int team, int nv, int mode, int wtype, bool tail);
kernel_t k1_stream_kernel(int mode);
kernel_t k1_team_kernel(int mode, bool any);
kernel_t mixed_kernel_plain(int mode);
kernel_t mixed_kernel_plain_half(int mode);
kernel_t mixed_kernel_any(int mode);
kernel_t mixed_kernel_any_half(int mode);
inline kernel_t mixed_kernel(int mode, int wtype, bool any) {
  if (wtype == SQUANT_W_F32) return any ? mixed_kernel_any(mode) : mixed_kernel_plain(mode);
  return any ? mixed_kernel_any_half(mode) : mixed_kernel_plain_half(mode);
}
kernel_t stem_kernel(int mode);
kernel_t stream_kernel(int mode);
kernel_t generic_kernel();
void (*activation_range_kernel())(BnArgs);

}  // namespace squant
