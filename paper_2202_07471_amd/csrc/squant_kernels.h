// The kernels as the host side sees them: one getter per family, each defined in the
// translation unit that instantiates the family (squant_kernels_*.hip, compiled in parallel).
#pragma once

#include <hip/hip_runtime.h>

#include "squant_common.h"

namespace squant {

typedef void (*kernel_t)(LaunchArgs);

// mode: squant_mode_t, wtype: squant_wtype_t, threads: of the workgroup, tail: some channel is
// no whole number of 16-byte vectors, any: some channel count is no multiple of four or some
// buffer off its alignment.
kernel_t k9_kernel(int kpt, int threads, int mode, int wtype, bool any);
kernel_t k9_any_kernel(int kpt, int threads, int mode);
kernel_t dw9_kernel(int mode);
kernel_t ks_kernel(int K, int kpt, int threads, int mode);
kernel_t ks_mixed_kernel(int mode);
kernel_t k1_kernel(int nv, int mode, int wtype, bool tail);
kernel_t k1_wave_kernel(int nv, int mode, int wtype, bool tail);
kernel_t k1_stream_kernel(int mode);
kernel_t k1_team_kernel(int mode);
kernel_t mixed_kernel(int mode, int wtype);
kernel_t stream_kernel(int mode);
kernel_t generic_kernel();

}  // namespace squant
