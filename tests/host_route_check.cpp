// Host-side check of the routes added around choose_variant: shapes the measured choices cover keep
// them, every other shape a register kernel takes gets a launch that covers its channel within the
// kernel's limits, and the variant numbers of the families do not meet.
#include <cstdint>
#include <cstdio>
#include <initializer_list>

#include "squant_plan.h"

using namespace squant;

// How many families claim a variant number.
static int claims(int v) {
  int n = 0;
  n += is_k1_wave(v);
  n += is_ks(v);
  n += is_k1_wide(v);
  n += k1_variant_nv(v) != 0 && !is_k1_wide(v);
  for (int other : {(int)kGeneric, (int)kK9x1, (int)kK9x2, (int)kK9x4, (int)kK1Stream, (int)kDw9, (int)kK1Team, (int)kStream,
                    (int)kDwTeam, (int)kK9Team, (int)kStem})
    n += v == other;
  return n;
}

int main() {
  long bad = 0, kept = 0, rerouted = 0;
  for (int aligned = 0; aligned < 2; ++aligned)
    for (int64_t K : {1, 2, 3, 4, 5, 6, 7, 8, 9, 16, 25, 49, 64, 65})
      for (int64_t N = 1; N <= 70000; N += (N < 700 ? 1 : 97)) {
        const int64_t M = 1 << 20;  // no small tensor
        const int family = route_family(M, N, K, aligned != 0), measured = choose_family(N, K, aligned != 0);
        const int v = route_variant(M, N, K, aligned != 0);
        bad += claims(v) != 1;
        if (family == measured) {
          ++kept;
          bad += v != choose_variant(N, K, aligned != 0);
        } else {
          ++rerouted;
          bad += measured != 0 && !(measured == 2 && family == 1 && N <= kMaxWideCin);
          if (family == 1) {
            const int nv = k1_variant_nv(v);
            const int64_t nvec = (N + 3) / 4;
            const int64_t th = is_k1_wide(v) ? round_up64((nvec + nv - 1) / nv) : k1_threads(nvec, nv);
            bad += K != 1 || nv == 0 || nv * th < nvec || th > 1024 || N > kMaxWideCin || N <= kMaxWaveCin;
            bad += is_k1_wide(v) && nv != 10 && nv != 12 && nv != 14 && nv != 16;
          } else if (family == 6) {
            const int nv = v - kK1Wave;
            bad += K != 1 || nv < 2 || nv > 8 || 64 * 4 * nv < N || N <= kMaxTeamCin;
          } else if (family == 4) {
            bad += K != 1 || N > 4 * team_lanes(N) * (team_lanes(N) == 16 ? 4 : 1);
          } else if (family == 9) {
            const int c = v == kK9x4 ? 4 : v == kK9x2 ? 2 : v == kK9x1 ? 1 : 0;
            const int64_t th = c ? round_up64((N + c - 1) / c) : 0;
            bad += K != 9 || N < 2 || N > kMaxK9Cin || c == 0 || th * c < N || th > 1024 || (c != 4 && th > 256);
          } else if (family == 5) {
            const int c = ks_variant_kpt(v), top = 1 << ks_max_kpt_log2(K);
            const int64_t th = round_up64((N + c - 1) / c);
            bad += !ks_has(K) || ks_variant_k(v) != K || N < 2 || c > top || th * c < N || th > 1024 || (c != top && th > 256);
            const int64_t lds = (int64_t)ks_lds_bytes(N, K);   // the codes and one more, or the ranking list, and no more
            bad += lds < K * N + 1 || lds < 4 * N || lds >= (K * N + 1 > 4 * N ? K * N + 1 : 4 * N) + 32;
          } else if (family == 7) {
            bad += N != 1 || K > kMaxDwK || dw_team_lanes(K) < K;
            bad += route_work_items(130, N, K, 64, family, 1) != (130 + 64 / dw_team_lanes(K) - 1) / (64 / dw_team_lanes(K));
          } else {
            ++bad;
          }
        }
        if (K == 9 && N > 1 && N <= kMaxK9TeamCin) bad += k9_team_lanes(N) < N || 64 % k9_team_lanes(N) != 0;
        // small tensors off the common shapes stay generic, except depthwise ones
        if (measured == 0 && N * K < kSmallTensor && family != 7) bad += route_family(1, N, K, aligned != 0) != 0;
      }
  // the lengths that the GPU tests of the streaming 1x1 kernel and of the one that holds a row in one workgroup use
  for (int64_t N : {65540, 70000, 131072}) bad += route_variant(1, N, 1, true) != kK1Stream;
  for (int64_t N : {36000, 40000, 50000, 65536}) bad += !is_k1_wide(route_variant(1, N, 1, true));
  // what a tensor is launched with: stems ahead of the routes, everything else as routed; which members the lean mixed
  // kernel, without small kernels, remainders and odd alignments, may take; the families fit above the kernel size
  for (int aligned = 0; aligned < 2; ++aligned)
    for (int64_t K : {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 16, 25, 49, 63, 64, 65})
      for (int64_t N = 1; N <= 2100; ++N)
        for (int64_t M : {1, 61, 1 << 20}) {
          const int family = tensor_family(M, N, K, aligned != 0), v = variant_of_family(family, N, K, aligned != 0);
          const bool stem = N >= 2 && N <= 4 && K >= 10 && K <= 64;
          bad += (family == kFamilyStem) != stem || (v == kStem) != stem || claims(v) != 1;
          bad += !stem && (family != route_family(M, N, K, aligned != 0) || v != route_variant(M, N, K, aligned != 0));
          bad += family == kFamilyBn || family == kFamilyRows || family < 0 || family > 127;
          const bool needs = mixed_needs_any(family, N, K, aligned != 0);
          bad += family == 5 && !needs;
          bad += (family == 9 || family == 4 || family == 6 || family == 1) && needs != (N % 4 != 0 || !aligned);
          bad += (family == kFamilyStem || family == 7 || family == 3) && needs;
          bad += mixed_rows_member(family, N) != (K == 1 && N > kMaxTeamCin && N <= kMaxRowsCin && family == 6);
          for (int T : {64, 128, 256}) {
            const int64_t channels = stem ? T / 64 : family == 6 ? T / 64 : family == 7 ? T / dw_team_lanes(K)
                                     : family == 4 ? T / team_lanes(N) : family == 3 ? T : 1;
            bad += mixed_work_items(M, N, K, T, family) != (M + channels - 1) / channels;
          }
          if (ks_has(K)) bad += ks_mixes(N, K) != (K <= 7 || K == 25 || (K == 16 && N <= 128));
        }
  // several 1x1 / FC channels a wave: the lanes of a team hold the row and the last vector of each may be its end
  for (int64_t N = kMaxTeamCin + 1; N <= kMaxRowsCin; ++N) {
    const int64_t team = k1_rows_team(N), nv = k1_rows_nv(N), half = nv <= 6 ? 24 : 32;
    bad += team != 16 && team != 32;
    bad += nv < 5 || nv > 8 || team * (4 * nv - 4) >= N || N > team * 4 * nv;
    bad += team * (half - 8) >= N || N > team * half;
    for (int T : {64, 128, 256})
      for (int64_t M : {1, 7, 2051})
        bad += mixed_work_items(M, N, 1, T, kFamilyRows) != (M + T / team - 1) / (T / team);
  }
  // and in a launch of their own: only where a kernel is built for them
  long several = 0;
  for (int64_t N = 1; N <= 3000; ++N)
    for (int half = 0; half < 2; ++half)
      for (int stage = 0; stage < 2; ++stage)
        for (int out_bits : {4, 8, 16, 32}) {
          const int64_t least = k1_rows_min(N, half != 0, stage != 0, out_bits);
          if (N <= kMaxTeamCin) continue;  // these go by teams whatever it says
          if (least == kNoRows) continue;
          ++several;
          bad += N > kMaxRowsCin || least < 8192;
          const int64_t team = k1_rows_team(N), nv = k1_rows_nv(N);
          bad += half ? team == 32 && nv <= 6 : !stage && (team != 16 || nv > 6);
        }
  bad += several == 0;
  for (int half = 0; half < 2; ++half)
    for (int stage = 0; stage < 2; ++stage) {
      for (int out_bits : {4, 8, 16, 32}) bad += mixed_rows_pay(kMixedRowsMin - 1, half != 0, stage != 0, out_bits);
      for (int out_bits : {4, 8, 16})
        for (int64_t channels : {2048, 8192, 30000}) bad += !mixed_rows_pay(channels, half != 0, stage != 0, out_bits);
      bad += mixed_rows_pay(2048, half != 0, stage != 0, 32) != (stage != 0);
      bad += mixed_rows_pay(8192, half != 0, stage != 0, 32) != (stage != 0 || half == 0);
      bad += mixed_rows_pay(24576, half != 0, stage != 0, 32);
    }
  std::printf("route_mismatches=%ld kept=%ld rerouted=%ld\n", bad, kept, rerouted);
  return bad != 0 || rerouted == 0;
}
