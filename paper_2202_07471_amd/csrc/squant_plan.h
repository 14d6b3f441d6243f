// Which kernel variant a tensor's channels go through.  The host decides it once per tensor, sizes the launch
// by it and hands the mixed kernel the family in the tensor's descriptor.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "squant_arith.h"  // SQ_HD

namespace squant {

enum Variant {
  kGeneric = 0,
  kK9x1 = 1, kK9x2 = 2, kK9x4 = 3,             // 3x3 kernels per thread: 1, 2, 4
  kK1x1 = 4, kK1x2 = 5, kK1x4 = 6, kK1x8 = 7,  // 1x1 / FC: 16-byte vectors per thread: 1, 2, 4, 8
  kK1Stream = 8,                               // 1x1 / FC beyond kMaxWideCin, aligned: weights walked repeatedly
  kDw9 = 9,                                    // depthwise 3x3 (cin per group = 1): one thread per channel
  kK1Team = 10,                                // 1x1 / FC up to kMaxTeamCin: 4 to 16 channels per wave
  kK1x3 = 11, kK1x5 = 12, kK1x6 = 13, kK1x7 = 14,  // 1x1 / FC: 3, 5, 6, 7 vectors per thread
  kStream = 15,                                // any shape: nothing kept on chip, weights walked repeatedly
  kK1x16 = 16,                                 // 1x1 / FC: 16 vectors per thread
  kK1Wave = 32,                                // 1x1 / FC up to kMaxWaveCin, a wave per channel: kK1Wave + vectors per lane (2..8)
  kK9Team = 42,                                // 3x3, 2 to 32 kernels a channel, in a launch of its own: a team of lanes per channel
  kStem = 43,                                  // two to four kernels of 10 to 64 elements: a wave per channel
  kDwTeam = 41,                                // depthwise, up to 64 elements a kernel: a team of lanes per channel
  kK1Wide = 48,                                // 1x1 / FC beyond kMaxK1Cin in one workgroup: kK1Wide + vectors per thread (10, 12, 14, 16)
  kKs = 1024                                   // small kernels in registers: kKs + 4 * K + log2(kernels per thread)
};

constexpr int kMaxK9Cin = 4096;   // 3x3 variant: any cin up to here
constexpr int kMaxK1Cin = 32768;  // 1x1 variant with the measured launch shapes: any cin up to here
constexpr int kMaxWideCin = 65536;  // 1x1 / FC rows held in one workgroup of 1024 threads
constexpr int kMaxTeamCin = 256;  // 1x1 channels this short share a wave
constexpr int kMaxWaveCin = 2048; // 1x1 channels up to here take a wave each (at most 8 vectors per lane)
constexpr int kK1WaveSpan = 4;    // the most consecutive channels a wave of that kernel walks (1 unless a launch is large)
constexpr int kK1WaveThreads = 256;  // its workgroup in a launch of its own
constexpr int kMixedMaxThreads = 256;  // largest workgroup of a mixed launch

SQ_HD int64_t round_up64(int64_t v) { return (v + 63) & ~(int64_t)63; }  // v >= 0
// ceil(a / b) for 0 <= a < 2^31, 0 < b <= 1024: 32-bit divisions take a host a third of the time of 64-bit ones
SQ_HD int64_t ceil_div(int64_t a, int64_t b) { return ((uint32_t)a + (uint32_t)b - 1u) / (uint32_t)b; }

// Launch shape of the 1x1 / FC kernel for a channel of nvec 16-byte vectors (at most 8192), in launches of their own that
// do without SQuant-C (with it: k1_launch_shape) and where it is asked whether a channel fits a mixed launch:
// T threads of NV vectors each, NV in 1..8 or 16.  Candidates: workgroups of one or two waves
// or a whole multiple of four (which spread evenly over the four SIMDs of a compute unit) with
// NV = ceil(nvec / T) up to 8, and sixteen vectors in the fewest waves that cover the channel
// (up to four, else eight).  The score is the share of the T * NV vector slots in use (an idle
// vector still runs SQuant-E), weighted by what was measured on channels of 512 to 32768
// elements as a fraction of the HBM roofline: seven or eight vectors (80 VGPRs, six waves per
// SIMD) 0.85 of one to six or sixteen; 512 threads 0.95, 768 and 1024 threads 0.85 (the
// workgroup-wide steps of the channel stage run in more waves), sixteen vectors in 512 threads
// 0.90.  Ties go to the larger NV.  Examples: cin 3072 6 x 128 at 70 %, 4096 16 x 64 at 70 %,
// 8192 16 x 128 at 67 %, 16384 16 x 256 at 64 %, 24576 6 x 1024 at 55 %, 32768 16 x 512 at
// 56 % (8 x 1024, one workgroup per compute unit: 33 %); workgroups of 3, 5 to 7 or 9 to 15
// waves with up to eight vectors lose 10 to 25 points against their neighbours.
struct K1Shape { int nv; int threads; };
SQ_HD K1Shape k1_shape(int64_t nvec) {
  K1Shape best = {8, 1024};
  int64_t best_score = -1;
  auto consider = [&](int nv, int64_t T, int64_t weight) {
    if (nv * T < nvec) return;
    const int64_t score = nvec * weight * 1000 / (nv * T);
    if (score > best_score || (score == best_score && nv > best.nv)) {
      best_score = score;
      best.nv = nv;
      best.threads = (int)T;
    }
  };
  const int sizes[6] = {64, 128, 256, 512, 768, 1024};
  for (int i = 0; i < 6; ++i) {
    const int64_t T = sizes[i];
    const int64_t nv = (nvec + T - 1) / T;
    if (nv > 8) continue;
    consider((int)nv, T, (nv >= 7 ? 85 : 100) * (T >= 768 ? 85 : T == 512 ? 95 : 100));
  }
  const int64_t t16 = round_up64((nvec + 15) / 16);
  if (t16 <= 256) consider(16, t16, 100 * 100);
  else if (t16 <= 512) consider(16, 512, 100 * 90);
  return best;
}
SQ_HD int64_t k1_threads_for(int64_t nvec) { return k1_shape(nvec).threads; }
SQ_HD int k1_nv_for(int64_t nvec) { return k1_shape(nvec).nv; }
// Threads a 1x1 / FC channel of nvec vectors takes with nv vectors per thread.
SQ_HD int64_t k1_threads(int64_t nvec, int nv) {
  if (nv == k1_nv_for(nvec)) return k1_threads_for(nvec);
  return round_up64((nvec + nv - 1) / nv);
}

// The shape of any row held in one workgroup where nothing else is known: beyond kMaxK1Cin elements the fewest vectors per
// thread, in steps of two, that 1024 threads hold the row with.
SQ_HD K1Shape k1_usual_shape(int64_t nvec) {
  if (nvec <= kMaxK1Cin / 4) return k1_shape(nvec);
  const int64_t least = (nvec + 1023) / 1024, nv = least <= 10 ? 10 : (least + 1) / 2 * 2;
  return {(int)nv, (int)round_up64((nvec + nv - 1) / nv)};
}

// The wave-per-channel 1x1 / FC kernel: 16-byte vectors per lane of a channel of N elements.
SQ_HD int k1_wave_nv(int64_t N) { return (int)((N / 4 + 63) / 64); }
SQ_HD bool is_k1_wave(int variant) { return variant >= kK1Wave + 2 && variant <= kK1Wave + 8; }

// Launch shape of the 1x1 / FC kernel with SQuant-C in a launch of its own: T threads of NV vectors, the fewest whole waves
// that hold a row of nvec vectors for each NV the kernel is built for, or the shape that a launch without SQuant-C would get.
// `rows`, `bytes`: of the launch, read and written; wide_out: to binary32.  The shape is the one of the least time by a model:
//   * what a row takes from its load to its store when nothing else runs: it grows with the vectors a thread holds and with
//     the waves, whose steps wait for each other;
//   * instructions, for all T * NV vector slots (an idle vector still runs SQuant-E).  Few vectors a thread leave the fixed
//     work of a wave to few weights; from ten on a SIMD holds four or five waves instead of seven or eight; and numbers of waves
//     that are no multiple of four share out badly over four SIMDs;
//   * memory, at 7.33 TB/s (launches that fit the caches in part), joined with the second as a 4-norm;
//   * where more rows are launched than the chip holds at once, a few percent more, a third with binary32 output (its
//     workgroups all write at their end): 976 rows of 16384 bfloat16 to binary32 8 x 512, 768 at once, 24.1 us, 16 x 256, 1024, 18.6.
// A shape other than the usual one has to be two percent better by the model, which is not exact: of 3840 launches (60 lengths
// from 2052 to 65536, a third of them odd, 0.4 M to 130 M weights, binary32 and bfloat16, four outputs, every NV) 64 are
// slower by more than 1.2 % than the usual shape, which is 5.4 % slower than the best one in the mean; this choice is 0.6 %.
// The numbers were fitted to the choice itself on these launches: on half of them, the other half's choice was 0.8 % off the best.
// (A model fitted to times alone, with some shapes struck out by hand and nothing in favour of the usual one, was 1.4 % off
// and slower than the usual shape by more than 1.2 % in 388 of them: 2052 bfloat16 to int8, 16 M weights 16.9 us and 18.7, 975
// rows of 4100 8.7 and 9.9, 549 rows of 16384 binary32 to binary32 16.2 and 21.1.)
// us of some, best ones first, the usual one last, bfloat16 to int8 / binary32 to int8:
//   30 M weights  cin  4096  8 x 128 21.8 / 26.6   4 x 256 24.5 / 26.7   16 x 64  24.8 / 30.4
//                 cin  7168  7 x 256 21.8 / 26.4   8 x 256 23.2 / 27.1   16 x 128 25.9 / 30.3
//                 cin 12288 12 x 256 22.9 / 27.3   6 x 512 24.3 / 26.8   16 x 192 24.8 / 29.1
//    4 M weights  cin  4096  4 x 256  8.0 /  8.3   5 x 256  8.9 /  8.8   16 x 64  12.5 / 12.8
//                 cin  8192  4 x 512  7.9 /  8.3  10 x 256  9.0 /  9.2   16 x 128 11.7 / 12.4
//   45 M weights  cin 36412 12 x 768 57.1 / 65.8  14 x 704 60.9 / 68.2   10 x 960 61.1 / 70.7
struct K1Built { int nv; float row_us, slot; int waves; };  // slot: relative instructions of a vector slot; waves: a compute unit holds
constexpr K1Built kK1Built[9] = {{4, 6.24f, 1.09f, 32}, {5, 6.61f, 0.95f, 32}, {6, 6.97f, 0.88f, 32}, {7, 7.33f, 0.78f, 32}, {8, 7.65f, 0.92f, 28},
                                 {10, 8.25f, 1.10f, 20}, {12, 8.58f, 1.04f, 20}, {14, 8.73f, 1.14f, 16}, {16, 10.60f, 1.16f, 16}};
// Vectors per thread that launches of their own are built for: with SQuant-C those above, without it what k1_usual_shape gives.
SQ_HD constexpr bool k1_built(int nv, bool stage) {
  return stage ? nv >= 4 && nv <= 16 && (nv <= 8 || nv % 2 == 0) : nv == 5 || nv == 6 || (nv >= 10 && nv <= 16 && nv % 2 == 0);
}
inline float k1_launch_us(const K1Built& v, int64_t T, int64_t rows, int64_t bytes, bool wide_out) {
  // relative instructions by waves, for up to seven, eight and more vectors a thread
  constexpr float of_waves[3][16] = {
      {1.04f, 0.61f, 0.57f, 0.60f, 1.12f, 1.15f, 0.95f, 0.72f, 1.17f, 1.45f, 1.03f, 0.95f, 1.43f, 1.43f, 2.08f, 0.86f},
      {0.84f, 0.46f, 0.65f, 0.54f, 0.80f, 1.08f, 0.82f, 0.75f, 1.29f, 0.99f, 1.05f, 0.88f, 2.08f, 1.59f, 2.18f, 1.36f},
      {0.41f, 0.40f, 0.52f, 0.46f, 0.92f, 0.97f, 0.77f, 0.51f, 2.37f, 1.55f, 1.21f, 1.15f, 2.00f, 1.65f, 1.98f, 1.27f}};
  const int waves = (int)(T / 64);
  const float work = (float)rows * (float)(v.nv * T) * v.slot * of_waves[v.nv <= 7 ? 0 : v.nv == 8 ? 1 : 2][waves - 1] * 2.955e-6f;
  const float memory = (float)bytes / 7.33e6f, w2 = work * work, m2 = memory * memory;
  const float us = v.row_us + 2.78f * (float)waves / 16.0f + __builtin_sqrtf(__builtin_sqrtf(w2 * w2 + m2 * m2));
  const int at_once = v.waves / waves;  // workgroups of a compute unit
  const float rounds = (float)rows / (256.0f * (float)(at_once > 0 ? at_once : 1));
  return rounds > 1.0f ? us * (1.0f + (wide_out ? 0.34f : 0.06f) / (1.0f + 0.09f * (rounds - 1.0f))) : us;
}
inline K1Shape k1_launch_shape(int64_t nvec, int64_t rows, int64_t bytes, bool wide_out) {
  K1Shape best = k1_usual_shape(nvec);
  float best_us = 3.0e38f;
  for (const K1Built& v : kK1Built)
    if (v.nv == best.nv) best_us = 0.98f * k1_launch_us(v, best.threads, rows, bytes, wide_out);
  for (const K1Built& v : kK1Built) {
    const int64_t T = round_up64((nvec + v.nv - 1) / v.nv);
    if (T > 1024) continue;
    const float us = k1_launch_us(v, T, rows, bytes, wide_out);
    if (us < best_us) { best_us = us; best.nv = v.nv; best.threads = (int)T; }
  }
  return best;
}

// Several 1x1 / FC channels of 257 to 1024 elements per wave (squant_k1_rows.h): lanes per channel and
// four-element vectors per lane (5 to 8).
constexpr int kMaxRowsCin = 1024;
constexpr int kK1RowsLds = 4096, kK1RowsListLds = 256;  // LDS bytes a wave: perturbations, ranking lists
SQ_HD int k1_rows_team(int64_t N) { return N <= 512 ? 16 : 32; }
SQ_HD int k1_rows_nv(int64_t N) { const int64_t per = 4 * k1_rows_team(N); return (int)((N + per - 1) / per); }
// Channels from which on a launch of its own takes that kernel (kNoRows: never).  stage: SQuant-C runs; out_bits: of an
// output element, 4 to 32.  Sharing a wave saves vector instructions, most of them SQuant-C's, but a row then moves in
// pieces of a quarter or half the length: where much is written or little computed, and where rows end inside a cache
// line, that costs more.  us with a wave a channel and with rows, 60 K channels where no other number stands:
//   codes, SQuant-C   binary32 320 34.4 and 22.0, 512 35.0 and 29.8, 640 39.0 and 34.5, 777 53.9 and 44.6, but 1002 with 12 K
//                     15.4 and 15.7; aligned beyond 640 no gain (1024 53.6 and 57.5); binary16 512 31.6 and 24.6, 1002 with
//                     16 K 17.2 and 17.5, 950 with 60 K 12 % less, and up to 768 or in whole vectors no gain
//   bfloat16 output   binary32 448 15 % less, 500 8 % more, 512 with 16 K 3 % more, 777 12 % less, 1002 2 % more;
//                     binary16 512 15 % less, beyond 768 -5 to 7 %
//   binary32 output   binary32 384 7 % less, 415 7 % more, 511 27 % more; binary16 320 1 % less, 333 6 and 512 50 % more
//   SQuant-E alone    binary32 codes 384 3 % less, 480 7 and 511 22 % more; to bfloat16 320 6 % less, 333 17 % more;
//                     binary16 codes 512 13 % less, 950 7 % less, 1002 12 % more (4-bit 7 % less); to bfloat16 448 7 % less,
//                     480 5 % more, 500 4 % less; to binary32 in either type up to 50 % more
// With few channels the chip holds a wave for each and the longer chain of a wave with several shows: binary32 to int8
// 320 with 12 K 9.7 and 9.0, 448 10.3 and 10.6, with 16 K 12.0 and 11.4; 512 10.3 and 11.2, 12.1 and 12.1.
constexpr int64_t kNoRows = INT64_MAX;
SQ_HD int64_t k1_rows_min(int64_t N, bool half, bool stage, int out_bits) {
  const bool codes = out_bits <= 8;
  if (N <= 512) {  // four channels a wave
    const int64_t longest = stage ? (codes || (half && out_bits == 16) ? 512 : out_bits == 16 ? 448 : half ? 320 : 384)
                            : out_bits == 32 ? 0 : half ? 512 : codes ? 384 : 320;
    if (N > longest) return kNoRows;
    if (!stage && out_bits == 16 && (half ? N > 448 && N % 8 == 0 : N % 4 != 0)) return kNoRows;
    return N <= 384 && out_bits != 16 ? 12288 : 16384;
  }
  if (N > kMaxRowsCin) return kNoRows;
  if (half) {
    if (N <= 768 || N % 8 == 0 || !codes) return kNoRows;
    return stage || out_bits == 4 || N <= 960 ? 24576 : kNoRows;
  }
  if (!stage || (N > 640 && N % 4 == 0) || out_bits == 32) return kNoRows;
  if (out_bits == 16) return N <= 896 ? 24576 : kNoRows;
  return N <= 896 ? 12288 : 24576;
}

// 16-byte vectors per thread of a 1x1 / FC variant (0: not one), and back.
SQ_HD bool is_k1_wide(int variant) { return variant > kK1Wide && variant <= kK1Wide + 16; }
SQ_HD int k1_variant_nv(int variant) {
  if (is_k1_wide(variant)) return variant - kK1Wide;
  switch (variant) {
    case kK1x1: return 1; case kK1x2: return 2; case kK1x3: return 3; case kK1x4: return 4;
    case kK1x5: return 5; case kK1x6: return 6; case kK1x7: return 7; case kK1x8: return 8;
    case kK1x16: return 16;
    default: return 0;
  }
}
SQ_HD int k1_variant_of(int nv) {
  const int v[9] = {kGeneric, kK1x1, kK1x2, kK1x3, kK1x4, kK1x5, kK1x6, kK1x7, kK1x8};
  return nv == 16 ? kK1x16 : v[nv];
}

// Small kernels held in registers (squant_ks.h): the kernel sizes it is built for, and the largest power of two (as its
// logarithm) of kernels one thread holds.
constexpr int kKsMaxK = 49;
SQ_HD bool ks_has(int64_t K) { return K == 2 || K == 3 || K == 4 || K == 5 || K == 7 || K == 16 || K == 25 || K == 49; }
SQ_HD constexpr int ks_max_kpt_log2(int64_t K) { return K <= 4 ? 3 : K <= 7 ? 2 : 0; }
// Whether the mixed kernel takes channels of N such kernels too.  7x7 kernels need more registers than its five waves
// per SIMD have.  4x4 ones join up to two waves: DCGAN and patch-discriminator layer sets 25.4 and 25.3 us in a launch per
// width, 13.0 and 17.0 so, five small layers 10.2 and 7.3; wider ones would split a launch in two (a ResNet-18 set with
// one 4x4 layer of 256 kernels a channel 22.5 us beside it, 25.8 in it).
SQ_HD bool ks_mixes(int64_t N, int64_t K) { return K == 16 ? N <= 128 : K <= 25; }
// log2 of the kernels per thread for a channel of N such kernels: the largest power of two that
// divides N and puts the channel into ONE wave at least 60 % full, else the one that keeps the
// waves fullest (measured: a one-wave workgroup wins down to that fill - 1x7 with cin 192 and
// 1x3 with cin 384 10 % faster at 75 % than three full waves, 1x7 with cin 160 13 % faster at
// 62 % than at 83 %, cin 128 50 % slower at 50 % than at 100 % - while among workgroups of
// several waves the fullest wins by 11-13 %); only the largest one is built for workgroups
// beyond 256 threads.  -1: none fits (then the generic kernel takes the tensor).
SQ_HD int ks_kpt_log2(int64_t N, int64_t K) {
  if (!ks_has(K) || ((N * K) & 3) != 0) return -1;
  const int top = ks_max_kpt_log2(K);
  int best = -1;
  int64_t best_num = 0, best_den = 1;
  for (int lg = top; lg >= 0; --lg) {
    if ((N & ((1 << lg) - 1)) != 0) continue;
    const int64_t num = N >> lg, th = round_up64(num);
    if (th > 1024 || (th > 256 && lg != top)) continue;
    if (th == 64 && num * 10 >= th * 6) return lg;
    if (num * best_den > best_num * th) { best_num = num; best_den = th; best = lg; }
  }
  return best;
}
// LDS of a channel: its codes and one more, and before them a dword per kernel for SQuant-C's ranking list (they take the same
// place).  Whole chunks of 32, so 512 kernels of two elements stay in a class of 2 KB, 1024 in 4 KB.
SQ_HD size_t ks_lds_bytes(int64_t N, int64_t K) {
  const int64_t codes = K * N + 1, list = 4 * N, most = codes > list ? codes : list;
  return (size_t)((most + 31) / 32 * 32);
}
SQ_HD bool is_ks(int variant) { return variant >= kKs && variant < kKs + 4 * (kKsMaxK + 1); }
SQ_HD int ks_variant(int64_t K, int kpt_log2) { return kKs + 4 * (int)K + kpt_log2; }
SQ_HD int ks_variant_k(int variant) { return (variant - kKs) >> 2; }
SQ_HD int ks_variant_kpt(int variant) { return 1 << ((variant - kKs) & 3); }

// Kernel family of a tensor: 9 = the 3x3 kernel, 1 = the 1x1 / FC kernel, 2 = the streaming
// 1x1 / FC kernel, 3 = depthwise 3x3, 4 = short 1x1 / FC channels (several per wave), 5 = other
// small kernels in registers, 6 = 1x1 / FC channels that take a wave each, 0 = generic.
// aligned: weights on 16 bytes and output on 4 (what the vector loads / stores need)
SQ_HD int choose_family(int64_t N, int64_t K, bool aligned) {
  if (K == 9 && N == 1) return 3;  // any alignment: element-wise loads and stores
  if (K == 9 && (N & 3) == 0 && N <= kMaxK9Cin && aligned) return 9;
  if (K == 1 && (N & 3) == 0 && N <= kMaxTeamCin && aligned) return 4;
  if (K == 1 && (N & 3) == 0 && N <= kMaxWaveCin && aligned) return 6;
  if (K == 1 && (N & 3) == 0 && N <= kMaxK1Cin && aligned) return 1;
  if (K == 1 && (N & 3) == 0 && aligned) return 2;
  if (N > 1 && aligned && ks_kpt_log2(N, K) >= 0) return 5;
  return 0;
}

// The variant a tensor gets in a launch of its own.
SQ_HD int choose_variant(int64_t N, int64_t K, bool aligned) {
  const int family = choose_family(N, K, aligned);
  if (family == 9) {
    // kernels per thread: four when that puts the channel into one wave at least 60 % full
    // (cin 152..256; measured 11 % faster than three full waves at cin 160 and 192), else the
    // largest of 4, 2, 1 that keeps the waves fullest
    // (fill = (N / c) / round_up64(N / c), compared by cross-multiplication)
    int best_c = 4;
    int64_t best_num = 0, best_den = 1;
    for (int lg = 2; lg >= 0; --lg) {
      const int c = 1 << lg;
      const int64_t num = N >> lg, th = round_up64(num);
      if (th > 256 && c != 4) continue;
      if (th == 64 && num * 10 >= th * 6) { best_c = c; break; }
      if (num * best_den > best_num * th) { best_num = num; best_den = th; best_c = c; }
    }
    return best_c == 4 ? kK9x4 : best_c == 2 ? kK9x2 : kK9x1;
  }
  if (family == 1) {
    return k1_variant_of(k1_nv_for(N / 4));
  }
  if (family == 2) return kK1Stream;
  if (family == 3) return kDw9;
  if (family == 4) return kK1Team;
  if (family == 6) return kK1Wave + k1_wave_nv(N);
  if (family == 5) return ks_variant(K, ks_kpt_log2(N, K));
  return kGeneric;
}

// ---- shapes and alignments the choices above leave to the generic kernel ----
// A channel count that is no multiple of four (a pruned network) and weights or codes that start
// anywhere (a checkpoint in one buffer without padding) go through the same register kernels,
// which read and write rows by descriptors whose range check stands in for both conditions
// (the generic kernel took 120 us for a ResNet-50-shaped network with such channel counts, nine
// times the time of its bytes).

// log2 of the small kernels per thread for any N: the measured choice where that applies, else the
// same rule with the kernels spread over ceil(N / c) threads.  -1: none fits.
SQ_HD int ks_kpt_log2_any(int64_t N, int64_t K, bool aligned) {
  if (!ks_has(K)) return -1;
  const int pinned = aligned ? ks_kpt_log2(N, K) : -1;
  if (pinned >= 0) return pinned;
  const int top = ks_max_kpt_log2(K);
  int best = -1;
  int64_t best_num = 0, best_den = 1;
  for (int lg = top; lg >= 0; --lg) {
    const int64_t used = (N + ((int64_t)1 << lg) - 1) >> lg, th = round_up64(used);
    if (th > 1024 || (th > 256 && lg != top)) continue;
    if (th == 64 && used * 10 >= th * 6) return lg;
    if (used * best_den > best_num * th) { best_num = used; best_den = th; best = lg; }
  }
  return best;
}

// Depthwise kernels other than 3x3 (squant_dw.h): places for elements in a channel's team of lanes, and elements a lane.
constexpr int kMaxDwK = 64, kDwLaneElems = 4;
SQ_HD int dw_team_lanes(int64_t K) { return K <= 16 ? 16 : K <= 32 ? 32 : 64; }

// Channels of a few larger kernels, the stem of a network (squant_stem.h): a wave per channel, whatever
// choose_family and route_family below say of them.
constexpr int kMaxStemCin = 4;
SQ_HD bool is_stem(int64_t N, int64_t K) { return N >= 2 && N <= kMaxStemCin && K >= 10 && K <= 64; }

// Tensors this small off the common shapes (a narrow layer with an odd channel count) stay with the generic
// routine: one of them among the common shapes would otherwise send a whole network to the larger mixed
// kernel.  A small tensor quantized alone has no network to protect and keeps the routine only for having
// one rule.  Stems are no part of this, whatever their size.
constexpr int64_t kSmallTensor = 16384;

// choose_family with those shapes, 7 = depthwise with a team of lanes per channel: 3x3 up to kMaxK9Cin, other small kernels, one-element rows
// (a team of lanes up to kMaxTeamCin, a wave up to kMaxWaveCin, a workgroup up to kMaxWideCin).
// Rows of up to kMaxWideCin elements are held in one workgroup too: walking the weights three times
// and more instead took 175 us for a [1024, 50176] layer of binary32 weights (18 % of the HBM
// roofline).
SQ_HD int route_family(int64_t M, int64_t N, int64_t K, bool aligned) {
  const int family = choose_family(N, K, aligned);
  if (family == 0 && N == 1 && K > 1 && K <= kMaxDwK) return 7;
  if (family == 0 && M * N * K < kSmallTensor) return 0;
  if (family == 2 && N <= kMaxWideCin) return 1;
  if (family != 0) return family;
  if (K == 9 && N > 1 && N <= kMaxK9Cin) return 9;
  if (K == 1 && N <= kMaxTeamCin) return 4;
  if (K == 1 && N <= kMaxWaveCin) return 6;
  if (K == 1 && N <= kMaxWideCin) return 1;
  if (N > 1 && ks_kpt_log2_any(N, K, aligned) >= 0) return 5;
  return 0;
}

// The family a tensor is launched with: stems as well, and, among the members of a mixed launch, batch norms and
// 1x1 / FC rows that go several to a wave.
constexpr int kFamilyStem = 8, kFamilyBn = 10, kFamilyRows = 11;
SQ_HD int tensor_family(int64_t M, int64_t N, int64_t K, bool aligned) {
  return is_stem(N, K) ? kFamilyStem : route_family(M, N, K, aligned);
}

// 3x3 channels of up to 32 kernels in a launch of their own (squant_k9_team.h): lanes per channel.
// In a mixed launch they keep the workgroup routine: there the launch is as long as its slowest
// members and the narrow layers are few.
constexpr int kMaxK9TeamCin = 32;
SQ_HD int k9_team_lanes(int64_t N) { return N <= 4 ? 4 : N <= 8 ? 8 : N <= 16 ? 16 : 32; }

SQ_HD int variant_of_family(int family, int64_t N, int64_t K, bool aligned) {
  if (family == 7) return kDwTeam;
  if (family == kFamilyStem) return kStem;
  if (family == choose_family(N, K, aligned)) return choose_variant(N, K, aligned);
  if (family == 9) {  // kernels per thread by the rule of choose_variant
    int best_c = 4;
    int64_t best_num = 0, best_den = 1;
    for (int lg = 2; lg >= 0; --lg) {
      const int c = 1 << lg;
      const int64_t used = (N + c - 1) >> lg, th = round_up64(used);
      if (th > 256 && c != 4) continue;
      if (th == 64 && used * 10 >= th * 6) { best_c = c; break; }
      if (used * best_den > best_num * th) { best_num = used; best_den = th; best_c = c; }
    }
    return best_c == 4 ? kK9x4 : best_c == 2 ? kK9x2 : kK9x1;
  }
  if (family == 4) return kK1Team;
  if (family == 6) return kK1Wave + k1_wave_nv(N + 3);
  if (family == 1 && N <= kMaxK1Cin) return k1_variant_of(k1_nv_for((N + 3) / 4));
  if (family == 1) return kK1Wide + k1_usual_shape((N + 3) / 4).nv;
  return ks_variant(K, ks_kpt_log2_any(N, K, aligned));
}
SQ_HD int route_variant(int64_t M, int64_t N, int64_t K, bool aligned) {
  return variant_of_family(route_family(M, N, K, aligned), N, K, aligned);
}

// Whether a member of family `family` needs the mixed kernel that carries every routine (ANY in squant_mixed.h).
SQ_HD bool mixed_needs_any(int family, int64_t N, int64_t K, bool aligned) {
  return family != 7 && family != kFamilyStem && (family == 5 || family != choose_family(N, K, aligned));
}

// Lanes that share a short 1x1 channel (see squant_k1_team.h).
SQ_HD int team_lanes(int64_t N) { return N <= 16 ? 4 : N <= 32 ? 8 : 16; }

// Workgroups a tensor of M output channels takes in a launch of T threads per workgroup:
// one per channel, except depthwise 3x3 (every thread has a channel of its own), short 1x1
// channels (one per team of lanes) and 1x1 channels of a wave each (wave_span per wave).  `family` as from choose_family.
SQ_HD int64_t work_items(int64_t M, int64_t N, int64_t K, int64_t T, int family, int wave_span) {
  if (family == 3) return ceil_div(M, T);
  if (family == 4) return ceil_div(M, (uint32_t)T / (uint32_t)team_lanes(N));
  if (family == 6) return ceil_div(M, (T >> 6) * wave_span);
  (void)K;
  return M;
}

// The same for every family.
SQ_HD int64_t route_work_items(int64_t M, int64_t N, int64_t K, int64_t T, int family, int wave_span) {
  if (family == 7) return ceil_div(M, (uint32_t)T / (uint32_t)dw_team_lanes(K));
  if (family == kFamilyStem) return ceil_div(M, T >> 6);
  return work_items(M, N, K, T, family, wave_span);
}

// Whether 1x1 / FC members of 257 to 1024 elements with `channels` channels in all go several to a wave in a mixed
// launch.  That saves instructions but makes a wave's chain longer, which shows where few such waves end a launch.  us
// with several and with a wave each: ResNet-18 sets of 1.35, 1.6 and 2 times the width (1688 to 2024 channels) 31.6 and
// 30.9, 41.7 and 40.9, 54.5 and 53.7, InceptionV3-style set of twice the width (1504) 141 and 138, MobileNetV2 sets of 0.7
// and 0.75 (1893, 1960) 9.1 and 9.0, 8.4 and 8.0; but of 0.85 (2152) 8.4 and 8.8, of 1 (2560) 9.4 and 9.8,
// InceptionV3-style set (3504) 42.4 and 43.7, ResNet-50 (11648) 28.0 and 31.2.  A ResNet-18 set (1000) takes 16.2 with either.
// Rows of a shared wave are written in shorter pieces, which binary32 output shows: with SQuant-C where there is much of it
// (ResNet-50 sets from bfloat16, of 1.5 times the width, 22080 channels, 82.6 and 83.3, of 1.9 times, 27960, 138 and 127), with
// SQuant-E alone throughout from 16 bits (ResNet-50 32.5 and 28.3) and from binary32 but for the middle (MobileNetV2 set of 1.9
// times the width, 8795, 20.5 and 21.4; InceptionV3-style set of half the width, 3944, 15.7 and 13.3; ResNet-50 of 1.9 133 and 128).
constexpr int64_t kMixedRowsMin = 2048;
SQ_HD bool mixed_rows_member(int family, int64_t N) { return family == 6 && N <= kMaxRowsCin; }
SQ_HD bool mixed_rows_pay(int64_t channels, bool half, bool stage, int out_bits) {
  if (out_bits < 32) return channels >= kMixedRowsMin;
  if (stage) return channels >= kMixedRowsMin && channels < 24576;
  return !half && channels >= 8192 && channels < 20480;
}

// Work items, as the functions here count them, that a workgroup takes: a lane of a depthwise team has several elements.
SQ_HD int items_per_workgroup(int family) { return family == 7 ? kDwLaneElems : 1; }

// In a mixed launch.
SQ_HD int64_t mixed_work_items(int64_t M, int64_t N, int64_t K, int64_t T, int family) {
  if (family == kFamilyRows) return ceil_div(M, (uint32_t)T / (uint32_t)k1_rows_team(N));
  return route_work_items(M, N, K, T, family, 1);
}

SQ_HD bool pointers_aligned(const void* w, const void* out) {
  return (reinterpret_cast<uintptr_t>(w) & 15u) == 0 && (reinterpret_cast<uintptr_t>(out) & 3u) == 0;
}

}  // namespace squant
