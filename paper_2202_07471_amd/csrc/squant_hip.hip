// SQuant weight-quantization solver, gfx950 (MI355X) kernels and C ABI.
//
// One workgroup owns one output channel from the first byte read to the last
// byte written: the channel's weights are read from HBM once (into registers
// for 3x3 and 1x1 kernels, into LDS otherwise), the absmax scale, rounding
// (SQuant-E), kernel-wise flip (SQuant-K), candidate update (Algorithm 3) and
// channel-wise flip (SQuant-C) all run on chip, and only the codes and one
// float scale go back to HBM.  Perturbations are Q23 integers, so every sum is
// order independent.  This file is the host side: argument checks, the choice
// of kernel variant per tensor, the grouping of a batch into launches.
//
// Section / algorithm numbers refer to "SQuant: On-the-Fly Data-Free
// Quantization via Diagonal Hessian Approximation" (ICLR 2022).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "squant.h"

#include "squant_act.h"
#include "squant_common.h"
#include "squant_generic.h"
#include "squant_k1_wave.h"
#include "squant_kernels.h"
#include "squant_k9.h"
#include "squant_plan.h"
#include "squant_stream.h"

namespace {

using namespace squant;

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

struct DeviceLimits { int lds_bytes; bool ok; };

DeviceLimits device_limits() {
  int dev = 0, lds = 0;
  if (hipGetDevice(&dev) != hipSuccess) return {0, false};
  if (hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
    return {0, false};
  return {lds, true};
}

constexpr int kStaticLds = 16 * 4 + 16 * 8 + 256 * 4 + 16 + 64;  // static __shared__ of the kernels, padded

size_t generic_lds_bytes(int64_t N, int64_t K) {
  const int64_t L = N * K;
  return (size_t)(4 * L + (K == 1 ? 0 : 8 * N) + ((L + 3) & ~(int64_t)3) + 16);
}

int generic_threads(int64_t N, int64_t K) {
  const int64_t L = N * K;
  int64_t want = (K == 1) ? (L + 7) / 8 : (K >= kWaveKernelMinK) ? N * kWave : N;
  want = (want + kWave - 1) / kWave * kWave;
  return (int)std::min<int64_t>(512, std::max<int64_t>(kWave, want));
}

int check_common(int32_t bits, int mode) {
  if (bits < 2 || bits > 8) return SQUANT_ERR_BITS;
  if (mode < SQUANT_MODE_E || mode > SQUANT_MODE_EC) return SQUANT_ERR_MODE;
  return SQUANT_OK;
}

// Weight type and output format; `out` may be null when only the enums are checked.
int check_format(int wtype, int output, int32_t bits, const void* w, const void* out) {
  if (wtype < SQUANT_W_F32 || wtype > SQUANT_W_BF16) return SQUANT_ERR_FORMAT;
  if (output < SQUANT_OUT_INT8 || output > SQUANT_OUT_BF16) return SQUANT_ERR_FORMAT;
  if (output == SQUANT_OUT_INT4 && bits > 4) return SQUANT_ERR_BITS;
  const uintptr_t wmask = wtype == SQUANT_W_F32 ? 3u : 1u;
  if (reinterpret_cast<uintptr_t>(w) & wmask) return SQUANT_ERR_FORMAT;
  if (output == SQUANT_OUT_F32 && (reinterpret_cast<uintptr_t>(out) & 3u)) return SQUANT_ERR_FORMAT;
  if (output == SQUANT_OUT_BF16 && (reinterpret_cast<uintptr_t>(out) & 1u)) return SQUANT_ERR_FORMAT;
  return SQUANT_OK;
}

int check_shape(int32_t cout, int32_t cin, int32_t kh, int32_t kw) {
  if (cout <= 0 || cin <= 0 || kh <= 0 || kw <= 0) return SQUANT_ERR_SHAPE;
  const int64_t K = (int64_t)kh * kw;
  const int64_t L = K * cin;
  if (K > (1 << 20) || L > (int64_t)1 << 30) return SQUANT_ERR_SHAPE;
  return SQUANT_OK;
}

constexpr int kMixed = 100;      // Group::variant of a launch of squant_channel_mixed
constexpr int kMixedWave = 101;  // the same for the tensors whose channels take one wave each
constexpr int kK1RowsThreads = 2 * kWave;  // workgroup of the kernel for several 1x1 / FC channels per wave
constexpr size_t kMixedMaxLds = 16 * 1024;  // a member that wants more LDS than this stays out of it

// Threads a register-kernel tensor of N kernels, up to `top` per thread, takes as a member of a
// mixed launch: its own workgroup (`own` threads) up to two waves, else two waves where more
// kernels per thread make it fit (a member of three waves would send every one-wave member to a
// launch of its own: InceptionV3-style and pruned ResNet-50 sets).
int mixed_threads(int own, int64_t N, int top) {
  return own <= 2 * kWave || (N + top - 1) / top > 2 * kWave ? own : 2 * kWave;
}

// A tensor with its family (squant_plan.h).
struct Member : TensorDesc {
  int family;
  bool any;  // see mixed_needs_any
};

struct Group {
  int variant;
  int threads;
  size_t lds;
  std::vector<Member> t;
  bool fixed_threads = false;  // mixed launch: a non-generic member has set the workgroup size
  float n_sigma = 0.0f;        // of the batch norms among the members
  int32_t act_levels_minus_1 = 0;
  bool wave_members = false;   // holds wave-per-channel 1x1 tensors: LDS for a selection area per wave
  bool rows_members = false;   // mixed launch: those of up to kMaxRowsCin elements go several to a wave
};

// threads / lds: of a launch of the tensor's own variant.  mix_threads: what the tensor needs as
// a member of a mixed launch (0: it cannot join one), where the per-thread work follows the
// launch's workgroup size.
struct Plan { int variant; int threads; size_t lds; int mix_threads; int family = 0; bool any = false; };

inline size_t round_up(size_t v, size_t to) { return (v + to - 1) / to * to; }

// The fallback that takes any channel: nothing is kept on chip.
Plan stream_plan(int64_t N) {
  const int th = (int)std::min<int64_t>(kStreamThreads, std::max<int64_t>(2 * kWave, round_up64(N)));
  return Plan{kStream, th, 16, 0};  // no dynamic LDS; 16 stands for "fits"
}

// The launch shape of a kernel variant for one tensor (every tensor fits one).
Plan plan_variant(int variant, int64_t N, int64_t K, int lds_limit) {
  // LDS: a selection area per wave of the launch's workgroup, added when the launch goes out
  if (is_k1_wave(variant)) return Plan{variant, kK1WaveThreads, 16, kWave};
  if (is_k1_wide(variant)) {  // LDS: the owners' masks, two words per thread
    const int th = (int)round_up64(((N + 3) / 4 + k1_variant_nv(variant) - 1) / k1_variant_nv(variant));
    return Plan{variant, th, (size_t)8 * th, 0};
  }
  switch (variant) {
    case kK9x1: case kK9x2: case kK9x4: {
      const int kpt = variant == kK9x4 ? 4 : variant == kK9x2 ? 2 : 1;
      // LDS: the channel's int8 codes, one more, whole chunks of 32
      const int th = (int)round_up64((N + kpt - 1) / kpt);
      return Plan{variant, th, round_up((size_t)9 * N + 1, 32), mixed_threads(th, N, 4)};
    }
    case kK1x1: case kK1x2: case kK1x3: case kK1x4: case kK1x5: case kK1x6: case kK1x7: case kK1x8:
    case kK1x16: {
      const int nv = k1_variant_nv(variant);
      const int64_t nvec = (N + 3) / 4;
      const int th = (int)k1_threads(nvec, nv);
      // the mixed kernel carries the routines of up to four vectors per thread
      const int mix = nv <= 4 ? th : nvec <= 4 * kMixedMaxThreads ? (int)round_up64((nvec + 3) / 4) : 0;
      // LDS: the owners' masks, a word per thread (of the launch's workgroup, which a mixed
      // launch may make larger), two with sixteen vectors
      const size_t lds = nv > 8 ? (size_t)8 * th : (size_t)4 * std::max(th, kMixedMaxThreads);
      return Plan{variant, th, lds, mix};
    }
    case kDw9: return Plan{kDw9, kWave, 16, kWave};     // no LDS; 16 stands for "fits"
    case kDwTeam: return Plan{kDwTeam, kWave, 16, kWave};
    case kK1Team: return Plan{kK1Team, kWave, 16, kWave};
    case kStem: return Plan{kStem, kWave, 16, kWave};
    case kK1Stream: {
      const size_t lds = round_up((size_t)N, 16);  // the channel's int8 codes
      if (lds + sizeof(K9Shared) + 64 > (size_t)lds_limit) return stream_plan(N);
      return Plan{kK1Stream, 1024, lds, 0};
    }
    default: break;
  }
  if (is_ks(variant)) {  // LDS: as for 3x3, or a dword per kernel for SQuant-C's ranking list before
    const int64_t kpt = ks_variant_kpt(variant);
    const int th = (int)round_up64((N + kpt - 1) / kpt);
    const int mix = ks_mixes(N, K) ? mixed_threads(th, N, 1 << ks_max_kpt_log2(K)) : 0;
    return Plan{variant, th, ks_lds_bytes(N, K), mix};
  }
  const size_t lds = generic_lds_bytes(N, K);
  if (lds + kStaticLds > (size_t)lds_limit) return stream_plan(N);
  const int th = generic_threads(N, K);
  return Plan{kGeneric, th, lds, th};
}

// Picks the family, kernel variant and launch shape for one tensor.
Plan plan_tensor(const void* w, const void* out, int64_t M, int64_t N, int64_t K, int lds_limit) {
  const bool aligned = pointers_aligned(w, out);
  const int family = tensor_family(M, N, K, aligned);
  Plan p = plan_variant(variant_of_family(family, N, K, aligned), N, K, lds_limit);
  p.family = family;
  p.any = mixed_needs_any(family, N, K, aligned);
  return p;
}

bool has_channel_stage(int mode) { return mode == SQUANT_MODE_EKC || mode == SQUANT_MODE_EC; }
int output_bits(int output) {
  return output == SQUANT_OUT_F32 ? 32 : output == SQUANT_OUT_BF16 ? 16 : output == SQUANT_OUT_INT4 ? 4 : 8;
}

// Whether a tensor may join a launch of the mixed kernel: the mixed kernel carries a routine
// for it that fits its workgroup size and LDS.
bool mixable(const Plan& p, size_t lds_cap) {
  return p.mix_threads > 0 && p.mix_threads <= kMixedMaxThreads && p.lds <= std::min(kMixedMaxLds, lds_cap);
}

// The kernel a tensor of plan p takes in a launch of its own variant: narrow 3x3 channels by teams.
Plan own_launch(Plan p, int64_t N, int64_t K) {
  if (K == 9 && N > 1 && N <= kMaxK9TeamCin) { p.variant = kK9Team; p.threads = 4 * kWave; p.lds = 16; }
  return p;
}

// Launches tensors [begin, end) of a group (at most kInlineDescs of them) as one kernel; rows: with the kernel for
// several 1x1 / FC channels per wave, wave_span of them.
int launch_part(const Group& g, bool rows, size_t begin, size_t end, int qmax, int mode, int output, int wtype,
                int wave_span, hipStream_t st) {
  LaunchArgs a;  // 11 KB: only the entries in use are filled in
  const int threads = rows ? kK1RowsThreads : g.threads;
  const bool mixed = g.variant == kMixed || g.variant == kMixedWave;
  a.n_sigma = g.n_sigma;
  a.act_levels_minus_1 = g.act_levels_minus_1;
  int64_t total = 0;
  bool uniform = true;
  bool tail = false;  // 1x1 / FC rows: any that is no whole number of 16-byte vectors
  bool any = false;   // any off the common channel counts and alignments (mixed: or another small kernel)
  auto items_of = [&](const Member& t) {
    if (t.K == 0) return (int64_t)1;  // a batch norm
    if (g.variant == kK9Team) { const int per = g.threads / k9_team_lanes(t.N); return (int64_t)(t.M + per - 1) / per; }
    const int64_t items = mixed ? mixed_work_items(t.M, t.N, t.K, threads, t.family)
                                : route_work_items(t.M, t.N, t.K, threads, t.family, wave_span);
    return ceil_div(items, items_per_workgroup(t.family));
  };
  const int64_t items0 = items_of(g.t[begin]);
  for (size_t i = begin; i < end; ++i) {
    const Member& t = g.t[i];
    const int64_t items = items_of(t);
    a.table[i - begin] = t;
    if (mixed) a.table[i - begin].K |= t.family << kFamilyShift;
    tail |= t.N % (wtype == SQUANT_W_F32 ? 4 : 8) != 0;
    any |= t.any;
    a.table[i - begin].first = a.first[i - begin] = (int32_t)total;  // first workgroup within this launch
    total += items;
    uniform &= items == items0;
    if (total > 0x7fffffff) return SQUANT_ERR_SHAPE;
  }
  if (total <= 0) return SQUANT_ERR_SHAPE;
  a.n_tensors = (int)(end - begin);
  a.total = (int32_t)total;
  a.uniform_m = uniform ? (int32_t)items0 : 0;
  a.uniform_shift = -1;
  if (uniform && (items0 & (items0 - 1)) == 0)
    for (int sh = 0; sh < 31; ++sh)
      if (((int64_t)1 << sh) == items0) a.uniform_shift = sh;
  a.qmax = qmax;
  a.rcp_qmax = 1.0f / (float)qmax;
  a.mode = mode;
  a.out_format = output;
  a.wtype = wtype;
  a.wave_span = wave_span;
  const int nv = k1_variant_nv(g.variant);
  const kernel_t kernel = is_ks(g.variant) ? ks_kernel(ks_variant_k(g.variant), ks_variant_kpt(g.variant), g.threads, mode, wtype)
                          : mixed ? mixed_kernel(mode, wtype, any)
                          : rows ? k1_rows_kernel(kWave / wave_span, k1_rows_nv(g.t[begin].N), mode, wtype, tail)
                          : is_k1_wave(g.variant) ? k1_wave_kernel(g.variant - kK1Wave, mode, wtype, tail)
                          : nv ? k1_kernel(nv, mode, wtype, tail)
                          : g.variant == kK1Stream ? k1_stream_kernel(mode)
                          : g.variant == kStream ? stream_kernel(mode)
                          : g.variant == kStem ? stem_kernel(mode)
                          : g.variant == kDw9 ? dw9_kernel(mode)
                          : g.variant == kK9Team ? k9_team_kernel(mode)
                          : g.variant == kDwTeam ? dw_team_kernel(mode)
                          : g.variant == kK1Team ? k1_team_kernel(mode, any)
                          : g.variant == kK9x1 ? k9_kernel(1, g.threads, mode, wtype, any)
                          : g.variant == kK9x2 ? k9_kernel(2, g.threads, mode, wtype, any)
                          : g.variant == kK9x4 ? k9_kernel(4, g.threads, mode, wtype, any)
                                               : generic_kernel();
  if (!kernel) return SQUANT_ERR_UNSUPPORTED;
  size_t lds = g.lds;
  if (rows) lds = (size_t)(threads / kWave) * (kK1RowsLds + kK1RowsListLds);
  else if (g.wave_members) lds = std::max(lds, (size_t)(threads / kWave) * (g.rows_members ? (size_t)kK1RowsLds : sizeof(K1WaveSel)));
  if (lds > 48 * 1024) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
      (void)hipGetLastError();
      return SQUANT_ERR_DEVICE;
    }
  }
  // by address: a call through the kernel's stub copies the arguments twice more
  void* args[] = {&a};
  if (hipLaunchKernel(reinterpret_cast<const void*>(kernel), dim3((unsigned)total), dim3(threads), args,
                      g.variant == kStream ? 0 : lds, st) != hipSuccess) {
    (void)hipGetLastError();
    return SQUANT_ERR_DEVICE;
  }
  return SQUANT_OK;
}

// The launch shape of a group of 1x1 / FC rows that take a workgroup each: one for all its tensors, by the longest row.
// Only with SQuant-C: SQuant-E alone is bound by memory in the shapes that k1_shape gives (4000 x 2000 binary32 7.4 us
// with 16 x 64, 8.4 with 4 x 256).
void shape_rows(Group& g, int wtype, int out_bits) {
  int64_t nvec = 0, rows = 0, weights = 0;
  for (const auto& t : g.t) {
    nvec = std::max<int64_t>(nvec, (t.N + 3) / 4);
    rows += t.M;
    weights += (int64_t)t.M * t.N;
  }
  const K1Shape sh = k1_launch_shape(nvec, rows, weights * ((wtype == SQUANT_W_F32 ? 32 : 16) + out_bits) / 8, out_bits == 32);
  g.variant = sh.nv <= 8 ? k1_variant_of(sh.nv) : kK1Wide + sh.nv;
  g.threads = sh.threads;
  g.lds = (size_t)(sh.nv > 8 ? 8 : 4) * sh.threads;  // the owners' masks
}

// A group goes out in launches of at most kInlineDescs tensors each.
int launch_group(Group& g, int qmax, int mode, int output, int wtype, hipStream_t st) {
  // Waves of the wave-per-channel 1x1 kernel walk several channels each where that still
  // leaves the chip (8192 resident waves) a few rounds of them, each asking for the next
  // channel's weights early; in a mixed launch one.  It pays while a wave holds little: rows of
  // up to 512 elements gain with four (131 K channels of 512: binary16 62.2 -> 58.1 us, binary32
  // 67.2 -> 65.3).  Longer 16-bit rows do best with two (131 K channels of 1024: 87.3 us with one,
  // 83.8 with two, 85.9 with four).  Longer binary32 rows have enough bytes in flight and lose by
  // the registers that wait (the same shape: 107.7, 117.3, 129.5 us), so they keep to one.
  int wave_span = 1;
  bool rows = false;
  if (k1_variant_nv(g.variant) != 0 && has_channel_stage(mode)) shape_rows(g, wtype, output_bits(output));
  if (is_k1_wave(g.variant)) {
    int64_t channels = 0, longest = 0;
    rows = true;
    for (const auto& t : g.t) {
      channels += t.M;
      longest = std::max<int64_t>(longest, t.N);
      rows &= k1_rows_nv(t.N) == k1_rows_nv(g.t[0].N) && k1_rows_team(t.N) == k1_rows_team(g.t[0].N);  // one kernel for all
    }
    for (const auto& t : g.t)
      rows = rows && channels >= k1_rows_min(t.N, wtype != SQUANT_W_F32, has_channel_stage(mode), output_bits(output));
    if (rows) {
      wave_span = kWave / k1_rows_team(longest);
    } else if (channels >= (int64_t)kK1WaveSpan * 2 * 8192) {
      wave_span = longest <= 512 ? kK1WaveSpan : wtype == SQUANT_W_F32 ? 1 : 2;
    }
  }
  for (size_t begin = 0; begin < g.t.size(); begin += kInlineDescs) {
    const size_t end = std::min(g.t.size(), begin + (size_t)kInlineDescs);
    if (int rc = launch_part(g, rows, begin, end, qmax, mode, output, wtype, wave_span, st)) return rc;
  }
  return SQUANT_OK;
}

// What squant_quantize_network adds to a batched call.
struct ActArgs {
  float n_sigma;
  int32_t bits;
  squant_act_range_t* ranges;
};

// The batched call.  bns: batch norms whose ranges join the mixed launch if there is one (a launch
// of their own takes 5 us, mostly its start and end); *bns is empty afterwards if they did.
int quantize_batched(const squant_tensor_t* h_tensors, int32_t n_tensors, squant_wtype_t wtype, int32_t bits,
                     squant_mode_t mode, squant_output_t output, void* d_workspace, size_t workspace_bytes,
                     std::vector<BnDesc>* bns, const ActArgs* act, hipStream_t st) {
  if (n_tensors < 0) return SQUANT_ERR_SHAPE;
  if (n_tensors == 0) return SQUANT_OK;
  if (!h_tensors) return SQUANT_ERR_NULL;
  if (int rc = check_common(bits, (int)mode)) return rc;
  for (int32_t i = 0; i < n_tensors; ++i) {
    const squant_tensor_t& t = h_tensors[i];
    if (!t.w || !t.codes || !t.scales) return SQUANT_ERR_NULL;
    if (int rc = check_shape(t.cout, t.cin, t.kh, t.kw)) return rc;
    if (int rc = check_format((int)wtype, (int)output, bits, t.w, t.codes)) return rc;
  }
  if (!d_workspace && workspace_bytes != 0) return SQUANT_ERR_WORKSPACE;
  const DeviceLimits lim = device_limits();
  if (!lim.ok) { (void)hipGetLastError(); return SQUANT_ERR_DEVICE; }

  // Group tensors by launch configuration.  Tensors whose variant runs in workgroups of at
  // most kMixedMaxThreads threads share ONE launch of the mixed kernel when they differ in
  // variant or launch shape (the layers of a network); a uniform set keeps its own kernel.
  std::vector<Plan> plans((size_t)n_tensors);
  const size_t lds_cap = (size_t)lim.lds_bytes - kStaticLds - sizeof(K9Shared) - sizeof(GenericShared);
  int small_kinds = 0;
  Plan small_first{};
  // Networks repeat their shapes: the plans of the last few are kept for the call.
  struct Seen { int64_t N = 0, K = 0; bool aligned = false, small = false; Plan p{}; } seen[16];
  for (int32_t i = 0; i < n_tensors; ++i) {
    const squant_tensor_t& t = h_tensors[i];
    const int64_t N = t.cin, K = (int64_t)t.kh * t.kw;
    const bool aligned = pointers_aligned(t.w, t.codes), small = t.cout * N * K < kSmallTensor;  // what a plan depends on
    Seen& last = seen[((uint32_t)N >> 2 ^ (uint32_t)N >> 6 ^ (uint32_t)K ^ (uint32_t)aligned) & 15u];
    if (last.N != N || last.K != K || last.aligned != aligned || last.small != small) {
      Plan p = plan_tensor(t.w, t.codes, t.cout, N, K, lim.lds_bytes);
      if (p.lds == 0) return SQUANT_ERR_UNSUPPORTED;
      // LDS size classes: next power of two >= 2 KB keeps the number of launches small
      size_t cls = 2048;
      while (cls < p.lds) cls <<= 1;
      p.lds = std::max(std::min(cls, lds_cap), p.lds);
      last.N = N; last.K = K; last.aligned = aligned; last.small = small; last.p = p;
    }
    const Plan& p = last.p;
    plans[(size_t)i] = p;
    if (mixable(p, lds_cap)) {
      if (small_kinds == 0) { small_first = p; small_kinds = 1; }
      else if (p.variant != small_first.variant || p.threads != small_first.threads ||
               p.lds != small_first.lds) small_kinds = 2;
    }
  }
  const bool use_mixed = small_kinds > 1;
  // One mixed launch while its workgroups stay at 128 threads (measured: ResNet-18 set 27 %,
  // MobileNetV2 set 12 % faster than two launches, ResNet-50 set the same).  When a member
  // needs 256 threads, the channels that take one wave get a launch of one-wave workgroups of
  // their own: four times as many of them fit a compute unit.
  int widest = 0;
  for (int32_t i = 0; i < n_tensors; ++i) {
    const Plan& p = plans[(size_t)i];
    if (use_mixed && mixable(p, lds_cap) && p.variant != kGeneric) widest = std::max(widest, p.mix_threads);
  }
  const bool two_classes = widest > 2 * kWave;
  std::vector<Group> groups;
  for (int32_t i = 0; i < n_tensors; ++i) {
    const squant_tensor_t& t = h_tensors[i];
    const bool in_mixed = use_mixed && mixable(plans[(size_t)i], lds_cap);
    const Plan p = in_mixed ? plans[(size_t)i] : own_launch(plans[(size_t)i], t.cin, (int64_t)t.kh * t.kw);
    const int need_threads = p.mix_threads;
    // a stem, the first member of its network, opens the launch of the wide members: they go first then
    // (a ResNet-50 set of 1.58 times the width with its activation ranges: 78.6 us, 92.5 the other way round)
    const int mixed_kind = two_classes && need_threads <= kWave && p.variant != kStem ? kMixedWave : kMixed;
    Group* g = nullptr;
    for (auto& c : groups) {
      if (in_mixed ? c.variant == mixed_kind
                   : (c.variant == p.variant && c.threads == p.threads && c.lds == p.lds)) { g = &c; break; }
    }
    if (!g) {
      groups.push_back(Group{in_mixed ? mixed_kind : p.variant, in_mixed ? need_threads : p.threads, p.lds, {}});
      g = &groups.back();
      g->t.reserve(std::min((size_t)(n_tensors - i) + (bns ? bns->size() : 0), (size_t)kInlineDescs));
    }
    if (in_mixed) {
      // the workgroup size follows the specialised routines (their kernels / vectors per thread
      // depend on it); the generic routine strides by whatever size it is given, so a generic
      // member only sets the size of a launch that has no other kind of member
      if (p.variant != kGeneric) {
        g->threads = g->fixed_threads ? std::max(g->threads, need_threads) : need_threads;
        g->fixed_threads = true;
      } else if (!g->fixed_threads) {
        g->threads = std::max(g->threads, need_threads);
      }
      g->lds = std::max(g->lds, p.lds);
    }
    g->t.push_back(Member{{t.w, t.codes, t.scales, t.cout, t.cin, (int32_t)((int64_t)t.kh * t.kw), 0}, p.family, p.any});
    g->wave_members |= is_k1_wave(p.variant);
  }
  for (auto& g : groups) {
    if (g.variant != kMixed && g.variant != kMixedWave) continue;
    int64_t channels = 0;
    for (const auto& t : g.t) channels += mixed_rows_member(t.family, t.N) ? t.M : 0;
    g.rows_members = mixed_rows_pay(channels, wtype != SQUANT_W_F32, has_channel_stage((int)mode), output_bits((int)output));
    if (!g.rows_members) continue;
    for (auto& t : g.t)
      if (mixed_rows_member(t.family, t.N)) t.family = kFamilyRows;
    // A launch ends with its last members, and waves with several channels take longest: where such members come last
    // (the classifier of a narrow network) they open the launch instead, if it is the only one (ResNet-50 sets of
    // 0.4, 0.45 and 0.5 times the width 10.4, 11.7 and 12.7 us without, 10.1, 11.4 and 12.2 with).
    if (g.variant == kMixed && !two_classes)
      std::rotate(g.t.begin(), std::find_if(g.t.rbegin(), g.t.rend(), [](const Member& t) { return t.family != kFamilyRows; }).base(),
                  g.t.end());
  }
  if (bns && !bns->empty()) {
    for (auto& g : groups) {
      if (g.variant != kMixed && g.variant != kMixedWave) continue;
      g.n_sigma = act->n_sigma;
      g.act_levels_minus_1 = (int32_t)((1 << act->bits) - 1);
      for (const BnDesc& b : *bns)
        g.t.push_back(Member{{b.gamma, act->ranges + b.out_index, const_cast<float*>(b.beta), b.channels, b.relu, 0, 0},
                             kFamilyBn, false});
      bns->clear();
      break;
    }
  }
  const int qmax = (1 << (bits - 1)) - 1;
  for (auto& g : groups)
    if (int rc = launch_group(g, qmax, (int)mode, (int)output, (int)wtype, st)) return rc;
  return SQUANT_OK;
}

}  // namespace

extern "C" {

int squant_quantize_ex(const void* d_w, squant_wtype_t wtype, int32_t cout, int32_t cin,
                       int32_t kh, int32_t kw, int32_t bits, squant_mode_t mode,
                       squant_output_t output, void* d_out, float* d_scales, void* stream) {
  if (!d_w || !d_out || !d_scales) return SQUANT_ERR_NULL;
  if (int rc = check_shape(cout, cin, kh, kw)) return rc;
  if (int rc = check_common(bits, (int)mode)) return rc;
  if (int rc = check_format((int)wtype, (int)output, bits, d_w, d_out)) return rc;
  const DeviceLimits lim = device_limits();
  if (!lim.ok) { (void)hipGetLastError(); return SQUANT_ERR_DEVICE; }
  const int64_t K = (int64_t)kh * kw;
  const Plan p = own_launch(plan_tensor(d_w, d_out, cout, cin, K, lim.lds_bytes), cin, K);
  if (p.lds == 0) return SQUANT_ERR_UNSUPPORTED;
  Group g{p.variant, p.threads, p.lds, {}};
  g.t.push_back(Member{{d_w, d_out, d_scales, cout, cin, (int32_t)K, 0}, p.family, p.any});
  g.wave_members = is_k1_wave(p.variant);
  return launch_group(g, (1 << (bits - 1)) - 1, (int)mode, (int)output, (int)wtype,
                      (hipStream_t)stream);
}

int squant_quantize(const float* d_w, int32_t cout, int32_t cin, int32_t kh, int32_t kw,
                    int32_t bits, squant_mode_t mode, int8_t* d_codes, float* d_scales,
                    void* stream) {
  return squant_quantize_ex(d_w, SQUANT_W_F32, cout, cin, kh, kw, bits, mode, SQUANT_OUT_INT8,
                            d_codes, d_scales, stream);
}

size_t squant_output_bytes(int32_t cout, int32_t cin, int32_t kh, int32_t kw, squant_output_t output) {
  if (check_shape(cout, cin, kh, kw) != SQUANT_OK) return 0;
  const size_t L = (size_t)cin * kh * kw;
  switch (output) {
    case SQUANT_OUT_INT8: return (size_t)cout * L;
    case SQUANT_OUT_INT4: return (size_t)cout * ((L + 1) / 2);
    case SQUANT_OUT_F32: return (size_t)cout * L * 4;
    case SQUANT_OUT_BF16: return (size_t)cout * L * 2;
  }
  return 0;
}

// The descriptors travel in the kernel arguments and no kernel needs memory beyond its inputs
// and outputs, so no call asks for a workspace.
size_t squant_batched_workspace_bytes(int32_t) { return 0; }

int squant_quantize_batched(const squant_tensor_t* h_tensors, int32_t n_tensors, int32_t bits,
                            squant_mode_t mode, void* d_workspace, size_t workspace_bytes,
                            void* stream) {
  return squant_quantize_batched_ex(h_tensors, n_tensors, SQUANT_W_F32, bits, mode,
                                    SQUANT_OUT_INT8, d_workspace, workspace_bytes, stream);
}

int squant_quantize_batched_ex(const squant_tensor_t* h_tensors, int32_t n_tensors,
                               squant_wtype_t wtype, int32_t bits, squant_mode_t mode,
                               squant_output_t output, void* d_workspace, size_t workspace_bytes,
                               void* stream) {
  return quantize_batched(h_tensors, n_tensors, wtype, bits, mode, output, d_workspace, workspace_bytes,
                          nullptr, nullptr, (hipStream_t)stream);
}

size_t squant_activation_workspace_bytes(int32_t) { return 0; }

namespace {
// Shared by squant_activation_ranges and squant_quantize_network; every descriptor names the
// entry of d_ranges it writes.  Launches of at most kInlineBn layers each.
int launch_activation_ranges(const std::vector<BnDesc>& layers, float n_sigma, int32_t bits,
                             squant_act_range_t* d_ranges, hipStream_t st) {
  for (size_t c0 = 0; c0 < layers.size(); c0 += kInlineBn) {
    BnArgs a{};
    const int cnt = (int)std::min<size_t>(kInlineBn, layers.size() - c0);
    for (int i = 0; i < cnt; ++i) a.layer[i] = layers[c0 + i];
    a.n_sigma = n_sigma;
    a.levels_minus_1 = (int32_t)((1 << bits) - 1);
    a.out = d_ranges;
    hipLaunchKernelGGL(activation_range_kernel(), dim3((unsigned)cnt), dim3(256), 0, st, a);
    if (hipGetLastError() != hipSuccess) return SQUANT_ERR_DEVICE;
  }
  return SQUANT_OK;
}

int check_activation_args(int32_t bits, float n_sigma) {
  if (bits < 2 || bits > 16) return SQUANT_ERR_BITS;
  if (!(n_sigma >= 0.0f) || !(n_sigma <= 3.0e38f)) return SQUANT_ERR_SHAPE;
  return SQUANT_OK;
}
}  // namespace

int squant_activation_ranges(const squant_bn_t* h_layers, int32_t n_layers, float n_sigma,
                             int32_t bits, squant_act_range_t* d_ranges, void* d_workspace,
                             size_t workspace_bytes, void* stream) {
  if (n_layers < 0) return SQUANT_ERR_SHAPE;
  if (n_layers == 0) return SQUANT_OK;
  if (!h_layers || !d_ranges) return SQUANT_ERR_NULL;
  if (int rc = check_activation_args(bits, n_sigma)) return rc;
  std::vector<BnDesc> layers;
  layers.reserve((size_t)n_layers);
  for (int32_t i = 0; i < n_layers; ++i) {
    const squant_bn_t& l = h_layers[i];
    if (!l.gamma || !l.beta) return SQUANT_ERR_NULL;
    if (l.channels <= 0) return SQUANT_ERR_SHAPE;
    layers.push_back(BnDesc{l.gamma, l.beta, l.channels, l.relu, i, 0});
  }
  if (!d_workspace && workspace_bytes != 0) return SQUANT_ERR_WORKSPACE;
  return launch_activation_ranges(layers, n_sigma, bits, d_ranges, (hipStream_t)stream);
}

size_t squant_network_workspace_bytes(int32_t) { return 0; }

int squant_quantize_network(const squant_layer_t* h_layers, int32_t n_layers, int32_t weight_bits,
                            squant_mode_t mode, int32_t act_bits, float n_sigma,
                            squant_act_range_t* d_ranges, void* d_workspace,
                            size_t workspace_bytes, void* stream) {
  if (n_layers < 0) return SQUANT_ERR_SHAPE;
  if (n_layers == 0) return SQUANT_OK;
  if (!h_layers) return SQUANT_ERR_NULL;
  if (int rc = check_activation_args(act_bits, n_sigma)) return rc;
  std::vector<squant_tensor_t> weights((size_t)n_layers);
  std::vector<BnDesc> bns;
  for (int32_t i = 0; i < n_layers; ++i) {
    weights[(size_t)i] = h_layers[i].weight;
    const squant_bn_t& l = h_layers[i].bn;
    if (!l.gamma) continue;
    if (!l.beta || !d_ranges) return SQUANT_ERR_NULL;
    if (l.channels <= 0) return SQUANT_ERR_SHAPE;
    bns.push_back(BnDesc{l.gamma, l.beta, l.channels, l.relu, i, 0});
  }
  if (!d_workspace && workspace_bytes != 0) return SQUANT_ERR_WORKSPACE;
  const ActArgs act{n_sigma, act_bits, d_ranges};
  if (int rc = quantize_batched(weights.data(), n_layers, SQUANT_W_F32, weight_bits, mode, SQUANT_OUT_INT8, nullptr, 0,
                                &bns, &act, (hipStream_t)stream))
    return rc;
  if (bns.empty()) return SQUANT_OK;
  return launch_activation_ranges(bns, n_sigma, act_bits, d_ranges, (hipStream_t)stream);
}

int64_t squant_max_channel_elems(int32_t kh, int32_t kw) {
  if (kh <= 0 || kw <= 0 || (int64_t)kh * kw > (1 << 20)) return 0;
  return (int64_t)1 << 30;  // the bound of the argument check: the streaming kernel takes any channel
}

const char* squant_status_string(int status) {
  switch (status) {
    case SQUANT_OK: return "ok";
    case SQUANT_ERR_NULL: return "null pointer";
    case SQUANT_ERR_SHAPE: return "bad shape";
    case SQUANT_ERR_BITS: return "bits must be in [2, 8]";
    case SQUANT_ERR_MODE: return "unknown mode";
    case SQUANT_ERR_WORKSPACE: return "workspace size given without a workspace";
    case SQUANT_ERR_DEVICE: return "HIP call failed";
    case SQUANT_ERR_UNSUPPORTED: return "unsupported (not returned by this version)";
    case SQUANT_ERR_FORMAT: return "unknown weight or output type, or misaligned buffer";
    default: return "unknown status";
  }
}

int squant_version(void) { return 200; }

}  // extern "C"
