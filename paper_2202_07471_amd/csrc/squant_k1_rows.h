// SQuant kernel for 1x1 / FC channels of 257 to 1024 elements: four or two output channels per wave.
//
// A wave with a channel of 512 elements spends half its vector instructions, and most of its scalar ones
// (a scalar instruction costs a SIMD about as much as a vector one: the unit serves four), on what it does
// once per channel: reductions, scale, thresholds, the ranking list, the store.  Here a TEAM of 16 or 32
// neighbouring lanes owns a channel and a lane holds up to 32 of its elements, so the wave does all that
// for four or two channels at once: whatever belongs to a channel is a value in its lanes, reductions are
// butterflies over the team (DPP, and a swap of neighbouring rows for 32 lanes), and the search for the
// elements that flip (squant_k1.h) runs in all teams side by side until the last has its bounds.
//
// The elements between the bounds, at most kRowsListCap a team, are ranked in registers: the wave puts its
// perturbations into LDS (in two halves, 4 KB a wave), every lane picks its candidates from there by index and
// writes their keys to the team's list, every lane takes one key back, and fifteen rotations of a row compare it
// with the others.
#pragma once

#include "squant_k1.h"
#include "squant_k1_team.h"
#include "squant_k1_wave.h"  // K1WaveSel
#include "squant_plan.h"

namespace squant {

constexpr int kRowsListCap = 16;  // one key a lane of a row

// A wave's LDS area for its perturbations, and the keys of one team.
template <int NE>
struct alignas(16) K1RowsLds {
  static constexpr int kHalf = (NE / 4 + 1) / 2 * 4;  // elements a lane keeps here at a time
  uint32_t b[kHalf * kWave];  // biased perturbations, vector by vector, lane by lane; later bit q of b[lane]: element q flips
};
typedef uint32_t K1RowsList[kRowsListCap];
static_assert(sizeof(K1WaveSel) <= kK1RowsLds, "members of a wave per channel fit beside");
static_assert(kWave / 16 * sizeof(K1RowsList) == kK1RowsListLds, "what the host sizes the launch by");

// Keeps the compiler from moving LDS accesses of a wave across (the LDS handles them in order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum of the lanes before a lane in its team, and its own.
template <int TEAM>
__device__ __forceinline__ uint32_t team_prefix_sum(uint32_t x) {
  int v = (int)x;
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
  if (TEAM == 32) v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row 0 into 1, 2 into 3
  return (uint32_t)v;
}
template <int TEAM>
__device__ __forceinline__ uint32_t team_min_u32(uint32_t x) { return ~team_max_u32<TEAM>(~x); }

// Sign (0 or ~0) and number of flips of a channel whose lanes' perturbation sums are `esum`.
template <int TEAM>
__device__ __forceinline__ uint32_t k1_rows_flips(int32_t esum, uint32_t& sm) {
  if (TEAM == 16) {
    // At most 512 elements of 2^22, so the sum wraps only where it is 2^31: every element is on an exact half on the
    // same side then (a subnormal scale puts the largest there too), and the lanes' sums tell which.
    const int32_t ec = team_sum_i32<TEAM>(esum);
    sm = (uint32_t)((ec == INT32_MIN ? esum : ec) >> 31);
    return (((uint32_t)ec ^ sm) - sm + (uint32_t)(kHalf - 1)) >> 23;
  }
  const int32_t low = team_sum_i32<TEAM>(esum & 0xFFFF);
  const int32_t high = team_sum_i32<TEAM>(esum >> 16) + (low >> 16);  // sum = high * 2^16 + (low & 0xFFFF)
  sm = (uint32_t)(high >> 31);
  const int64_t ec = (int64_t)high * 65536 + (low & 0xFFFF);
  return (uint32_t)((uint64_t)((ec < 0 ? -ec : ec) + (kHalf - 1)) >> 23);
}

// Bit q: element q of the lane has u >= thr; u = P (sm 0) or ~P (sm ~0), B[q] = kQ23Bias + P.  For a negative sum
// that is the opposite of P >= -thr, so one kind of compare serves the teams of both signs.
template <int NE>
__device__ __forceinline__ uint32_t k1_rows_at_least(const uint32_t (&B)[NE], uint32_t sm, int32_t thr) {
  const uint32_t t = kQ23Bias + (((uint32_t)thr ^ sm) - sm);
  uint32_t m = 0;
#pragma unroll
  for (int q = NE - 4; q >= 0; q -= 4) push_compares_lanes(m, t, &B[q]);
  return (m ^ sm) & (NE < 32 ? (1u << (NE & 31)) - 1u : ~0u);
}

// SQuant-C (see k1_channel_stage in squant_k1.h): bit q of the result: element q of the lane flips.  sm, need: of
// the lane's channel.
template <int TEAM, int NE, int VE>
__device__ __forceinline__ uint32_t k1_rows_select(const uint32_t (&B)[NE], uint32_t sm, uint32_t need, int N,
                                                   K1RowsLds<NE>& lds, K1RowsList* lists) {
  constexpr int kIndexBits = TEAM == 16 ? 9 : 10;  // a key is (u - lo) above the index from the end: at most 31 bits
  constexpr uint32_t kIndexMask = (1u << kIndexBits) - 1u;
  constexpr int32_t kWidest = 1 << (31 - kIndexBits);  // widest interval whose keys fit
  const int lane = k1_tid<true>(), l = lane & (TEAM - 1), team = lane / TEAM;
  const int32_t step = __builtin_amdgcn_readfirstlane((int32_t)(8388608.0f * __builtin_amdgcn_rcpf((float)N)));
  const int32_t least = 1 + (int32_t)sm, top = (1 << 22) + 1;

  // The first threshold aims between `need` and what the list holds.
  const uint32_t aim = need == 0 ? 0u : need + (need < 11 ? (uint32_t)(17 - need) >> 1 : 3u);
  int32_t thr = imax2((1 << 22) - (int32_t)aim * step, least);
  uint32_t m = k1_rows_at_least(B, sm, thr);
  uint32_t n = (uint32_t)team_sum_i32<TEAM>(__popc(m));
  int32_t lo = thr, hi = top;
  uint32_t m_lo = m, m_hi = 0, n_lo = n, n_hi = 0;
  bool tie = false;
  if (__ballot(!(n >= need && n <= (uint32_t)kRowsListCap && hi - lo <= kWidest)) != 0ull) {
    // Bounds as in squant_k1.h.  A team that has them goes on without changing them.
    bool found = n >= need;
    if (!found) {
      if (thr == least) { need = n; found = true; }  // fewer candidates of the wanted sign than flips: all flip
      else { hi = thr; m_hi = m; n_hi = n; lo = least; m_lo = 0; n_lo = 0; }
    }
    uint32_t gaps = 0;
    bool low_side = !found;  // the last threshold was too high
    for (int pass = 1;; ++pass) {
      const bool done = found && (n_lo == need || hi - lo == 1 ||
                                  (n_lo - n_hi <= (uint32_t)kRowsListCap && hi - lo <= kWidest));
      if (__ballot(!done) == 0ull) break;
      if (__ballot(gaps >= 2 && !done) != 0ull) {
        // weights of few levels pile up on few values: the bounds close in on elements (see squant_k1.h)
        const uint32_t base = (kQ23Bias ^ sm) - sm;  // B[q] ^ sm = base + u
        const uint32_t from = base + (uint32_t)lo, to = base + (uint32_t)(hi - 1);
        uint32_t above = ~0u, below = ~0u;
#pragma unroll
        for (int q = 0; q < NE; q += 2) {
          const uint32_t x0 = B[q] ^ sm, x1 = B[q + 1] ^ sm;
          above = umin3(above, x0 - from, x1 - from);
          below = umin3(below, to - x0, to - x1);
        }
        above = umin2(team_min_u32<TEAM>(above), (uint32_t)(hi - lo - 1));
        below = umin2(team_min_u32<TEAM>(below), (uint32_t)(hi - lo - 1) - above);
        if (found && !done) { lo += (int32_t)above; hi -= (int32_t)below; }
        gaps = 0;
      }
      if (found) {
        if ((pass & 3) == 0) {
          thr = lo + ((hi - lo) >> 1);
        } else {
          float want = n_lo - need > (uint32_t)(kRowsListCap - kRowsListCap / 4 - 2) ? (float)need + 0.25f * kRowsListCap
                                                                                  : (float)need - 0.25f * kRowsListCap;
          if (want <= (float)n_hi + 0.5f) want = 0.5f * (float)(n_hi + need);
          float part = (want - (float)n_hi) * __builtin_amdgcn_rcpf((float)(n_lo - n_hi));
          if (low_side) {
            const float base = __builtin_amdgcn_logf(fmaxf((float)n_hi, 0.5f));
            part = (__builtin_amdgcn_logf(want) - base) * __builtin_amdgcn_rcpf(__builtin_amdgcn_logf((float)n_lo) - base);
          }
          thr = hi - (int32_t)(part * (float)(hi - lo));
        }
        thr = imax2(thr, lo + 1);
      } else {
        thr = k1_lower_threshold(thr, n, need, 0.25f * kRowsListCap, N);
      }
      thr = imin2(imax2(thr, lo), hi - 1);
      m = k1_rows_at_least(B, sm, thr);
      n = (uint32_t)team_sum_i32<TEAM>(__popc(m));
      if (!done) {
        low_side = n < need;
        if (!low_side) {
          gaps += n == n_lo ? 2u : 0u;
          lo = thr; n_lo = n; m_lo = m; found = true;
        } else if (thr == least && !found) {
          need = n_lo = n_hi = n; m_lo = m_hi = m; found = true;  // all flip
        } else {
          hi = thr; n_hi = n; m_hi = m;
        }
      }
    }
    tie = n_lo != need && n_lo - n_hi > (uint32_t)kRowsListCap;  // that many equal elements
  }
  if (__ballot(n_lo != need) == 0ull) return m_lo;
  const uint32_t want = need - n_hi;
  uint32_t live = m_lo & ~m_hi, flip = m_hi;
  if (n_lo == need) { flip = m_lo; live = 0; }

  if (__ballot(tie) != 0ull) {
    // The lowest indices flip: the elements of a vector are consecutive and vectors ascend with the lane.
    uint32_t done = 0;
#pragma unroll 1
    for (int round = 0; round < NE / VE; ++round) {
      const uint32_t bits = (live >> (VE * round)) & ((1u << VE) - 1u);
      const uint32_t mine = (uint32_t)__popc(bits);
      uint32_t rank = done + team_prefix_sum<TEAM>(mine) - mine;
#pragma unroll
      for (int e = 0; e < VE; ++e)
        if (bits & (1u << e)) {
          if (tie && rank < want) flip |= 1u << (VE * round + e);
          ++rank;
        }
      done += (uint32_t)team_sum_i32<TEAM>((int32_t)mine);
    }
    if (tie) live = 0;
  }

  // ---- the list ----
  const uint32_t count = (uint32_t)__popc(live);
  const uint32_t incl = team_prefix_sum<TEAM>(count);
  const uint32_t total = (uint32_t)team_sum_i32<TEAM>((int32_t)count);
  constexpr int kHalf = K1RowsLds<NE>::kHalf;
  uint32_t* put = lists[team] + (incl - count);
  const uint32_t from = ((kQ23Bias ^ sm) - sm) + (uint32_t)lo;  // B[q] ^ sm = from + (u - lo)
#pragma unroll
  for (int begin = 0; begin < NE; begin += kHalf) {
    vu4* b = reinterpret_cast<vu4*>(lds.b) + lane;
#pragma unroll
    for (int q = begin; q < NE && q < begin + kHalf; q += 4) b[(q - begin) / 4 * kWave] = vu4{B[q], B[q + 1], B[q + 2], B[q + 3]};
    wave_lds_fence();
    uint32_t bits = begin == 0 ? live & ((1u << kHalf) - 1u) : live >> kHalf;
    while (bits != 0) {
      const uint32_t at = (uint32_t)__builtin_ctz(bits), q = at + begin;
      bits &= bits - 1;
      const uint32_t b = lds.b[(at >> 2) * (4 * kWave) + 4 * lane + (at & 3u)];
      const uint32_t index = (q / VE) * (TEAM * VE) + (uint32_t)l * VE + q % VE;
      *put++ = (((b ^ sm) - from) << kIndexBits) | (kIndexMask - index);
    }
    wave_lds_fence();
  }
  lds.b[lane] = 0;
  wave_lds_fence();
  const int at = lane & 15;  // with 32 lanes a team both rows rank the same list
  const uint32_t listed = lists[team][at];
  const uint32_t key = (uint32_t)at < total ? listed : 0u;
  uint32_t larger = 0;  // keys are below 2^31: the sign of a difference says which is larger
#define SQ_ROTATE(I) larger = __builtin_amdgcn_alignbit(larger, key - (uint32_t)dpp_i32<0x120 + I>((int)key), 31)
  SQ_ROTATE(1); SQ_ROTATE(2); SQ_ROTATE(3); SQ_ROTATE(4); SQ_ROTATE(5); SQ_ROTATE(6); SQ_ROTATE(7); SQ_ROTATE(8);
  SQ_ROTATE(9); SQ_ROTATE(10); SQ_ROTATE(11); SQ_ROTATE(12); SQ_ROTATE(13); SQ_ROTATE(14); SQ_ROTATE(15);
#undef SQ_ROTATE
  if ((uint32_t)at < total && (uint32_t)__popc(larger) < want) {
    const uint32_t index = kIndexMask - (key & kIndexMask), v = index / VE;
    atomicOr(&lds.b[team * TEAM + (v & (TEAM - 1))], 1u << ((v / TEAM) * VE + index % VE));
  }
  wave_lds_fence();
  return flip | lds.b[lane];
}

// The rows of the wave's channels in one format, as k1_emit: the lane's vectors at `at`, `step` bytes apart.
template <int NE, int VE, int FORMAT, int TEAM>
__device__ __forceinline__ void k1_rows_emit(const uint32_t (&code)[NE / 4], void* out_base, int c0, int rows, int row,
                                             int l, int N, float s) {
  constexpr int kUnit = FORMAT == SQUANT_OUT_INT8 ? VE : FORMAT == SQUANT_OUT_INT4 ? VE / 2
                        : FORMAT == SQUANT_OUT_BF16 ? 2 * VE : 4 * VE;  // bytes of a vector
  constexpr int NL = NE / VE;
  const uint32_t row_bytes = FORMAT == SQUANT_OUT_INT8 ? (uint32_t)N : FORMAT == SQUANT_OUT_INT4 ? (uint32_t)(N + 1) / 2
                             : FORMAT == SQUANT_OUT_BF16 ? 2u * (uint32_t)N : 4u * (uint32_t)N;
  uint8_t* out = static_cast<uint8_t*>(out_base) + (size_t)c0 * row_bytes;
  const rsrc_t range = make_rsrc(out, (uint32_t)rows * row_bytes);
  constexpr uint32_t kOutside = 0x40000000u;
  const uint32_t base = row < rows ? (uint32_t)row * row_bytes + (uint32_t)l * kUnit : kOutside;
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    // only the last vector of a lane may lie beyond the row's whole vectors
    const uint32_t at = j < NL - 1 || l + j * TEAM < N / VE ? base : kOutside;
    const uint32_t step = (uint32_t)(j * kUnit * TEAM);
    const uint32_t c0w = code[j * VE / 4], c1w = code[j * VE / 4 + VE / 4 - 1];
    if (FORMAT == SQUANT_OUT_INT8) {
      if (VE == 4) buffer_store_u1_stream(c0w ^ 0x80808080u, range, at, step);
      else buffer_store_u2_stream(vu2{c0w ^ 0x80808080u, c1w ^ 0x80808080u}, range, at, step);
    } else if (FORMAT == SQUANT_OUT_INT4) {
      if (VE == 4) buffer_store_u16_stream((uint16_t)pack_nibbles4(c0w), range, at, step);
      else buffer_store_u1_stream(pack_nibbles8(c0w, c1w), range, at, step);
    } else if (FORMAT == SQUANT_OUT_BF16) {
      const vf4 v = dequant4(c0w, s);
      const uint32_t o0 = bf16_bits(v.x) | (bf16_bits(v.y) << 16), o1 = bf16_bits(v.z) | (bf16_bits(v.w) << 16);
      if (VE == 4) {
        buffer_store_u2_stream(vu2{o0, o1}, range, at, step);
      } else {
        const vf4 u = dequant4(c1w, s);
        buffer_store_u4_stream(vu4{o0, o1, bf16_bits(u.x) | (bf16_bits(u.y) << 16),
                                   bf16_bits(u.z) | (bf16_bits(u.w) << 16)}, range, at, step);
      }
    } else if (VE == 4) {
      buffer_store_u4_stream(__builtin_bit_cast(vu4, dequant4(c0w, s)), range, at, step);
    } else {
      const vu2 c = team_interleave<TEAM>(c0w, c1w, (int)(threadIdx.x & (kWave - 1)));
      const int v = (l >> 1) + j * TEAM;  // the vector the first piece belongs to; the second: TEAM / 2 later
      const uint32_t piece = (uint32_t)row * row_bytes + (uint32_t)l * 16u;
      const bool in = row < rows;
      buffer_store_u4_stream(__builtin_bit_cast(vu4, dequant4(c.x, s)), range,
                             in && (j < NL - 1 || v < N / VE) ? piece : kOutside, step);
      buffer_store_u4_stream(__builtin_bit_cast(vu4, dequant4(c.y, s)), range,
                             in && (j < NL - 1 || v + TEAM / 2 < N / VE) ? piece + 16u * TEAM : kOutside, step);
    }
  }
}

// Vector instructions a channel of 512 binary16 weights, a wave per channel and here: 256 and 206; scalar ones 181 and 39.
// 131 K such channels to int8: 58.2 -> 45.3 us (3.5 -> 4.4 TB/s; SIMDs issue vector instructions 85 % of the time); the
// ResNet-50 set in its mixed launch 31.2 us with a wave a channel, 27.5 here, with odd channel counts 24.8 and 21.2.
// Where it is taken: k1_rows_min and mixed_rows_pay in squant_plan.h.
// `item`: the workgroup's index within the tensor; each of its waves takes 64 / TEAM channels of N elements,
// TEAM * (NE - VE) < N <= TEAM * NE.
// LDS: kK1RowsLds bytes at smem and a list per team at `lists`, for each wave.
template <int MODE, int TEAM, int NE, int VE, bool HALF, bool TAIL>
__device__ __forceinline__ void k1_rows_channels(const LaunchArgs& a, const TensorDesc& d, int item,
                                                 unsigned char* smem, K1RowsList* lists) {
  constexpr bool kChannelStage = MODE == SQUANT_MODE_EKC || MODE == SQUANT_MODE_EC;
  constexpr int NL = NE / VE, kRows = kWave / TEAM, kBytes = VE * (HALF ? 2 : 4);
  constexpr uint32_t kOutside = 0x40000000u;
  static_assert(sizeof(K1RowsLds<NE>) <= kK1RowsLds, "what the host sizes the launch by");
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), waves = (int)blockDim.x / kWave;
  const int lane = (int)(threadIdx.x & (kWave - 1)), l = lane & (TEAM - 1), row = lane / TEAM;
  const int c0 = (item * waves + wave) * kRows, N = d.N;
  const int rows = imin2(kRows, d.M - c0);
  if (rows <= 0) return;  // no step of the workgroup follows

  // ---- the rows: elements behind a row's end are 0 ----
  const uint32_t row_bytes = (HALF ? 2u : 4u) * (uint32_t)N;
  const uint8_t* src = static_cast<const uint8_t*>(d.w) + (size_t)c0 * row_bytes;
  const rsrc_t range = make_rsrc(src, (uint32_t)rows * row_bytes);
  const uint32_t base = row < rows ? (uint32_t)row * row_bytes + (uint32_t)l * kBytes : kOutside;
  const int first = VE * (l + (NL - 1) * TEAM);  // first element of the lane's last vector
  uint32_t raw[HALF ? NE / 2 : NE];
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const uint32_t at = j < NL - 1 || first < N ? base : kOutside;
    const uint32_t step = (uint32_t)(j * kBytes * TEAM);
    if (kBytes == 16) {
      const vu4 v = buffer_load_u4_stream(range, at, step);
      raw[4 * j] = v.x; raw[4 * j + 1] = v.y; raw[4 * j + 2] = v.z; raw[4 * j + 3] = v.w;
    } else {
      const vu2 v = buffer_load_u2_stream(range, at, step);
      raw[2 * j] = v.x; raw[2 * j + 1] = v.y;
    }
  }
  // 16 bits: the last element of the last row may lie in a dword that ends behind the range and reads as 0
  uint32_t tail = 0;
  if (HALF && TAIL && (N & 1))
    tail = buffer_load_u16(range, row < rows && first < N && first + VE >= N ? (uint32_t)row * row_bytes + row_bytes - 2u : kOutside, 0);
  float w[NE];
  if (!HALF) {
#pragma unroll
    for (int q = 0; q < NE; ++q) w[q] = __uint_as_float(raw[HALF ? 0 : q]);
  } else if (a.wtype == SQUANT_W_BF16) {
#pragma unroll
    for (int r = 0; r < NE / 2; ++r) widen_pair(raw[r], true, w[2 * r], w[2 * r + 1]);
  } else {
#pragma unroll
    for (int r = 0; r < NE / 2; ++r) widen_pair(raw[r], false, w[2 * r], w[2 * r + 1]);
  }
  if (TAIL) {
    const int left = N - first;  // elements of the last vector inside the row
#pragma unroll
    for (int e = 0; e < VE; ++e) {
      float& v = w[NE - VE + e];
      if (HALF && (e & 1) == 0 && (N & 1) && left == e + 1) v = a.wtype == SQUANT_W_BF16 ? widen_bf16(tail) : widen_f16(tail);
      v = e < left ? v : 0.0f;
    }
  }

  const float amax = team_max_f32<TEAM>(k1_absmax(w));
  uint32_t code[NE / 4], B[NE];
  int32_t esum;
  const float s = k1_quantize<NE, kChannelStage, HALF>(w, amax, (float)a.qmax, a.rcp_qmax, code, B, esum);
  if (kChannelStage) {
    uint32_t sm;
    const uint32_t need = umin2(k1_rows_flips<TEAM>(esum, sm), (uint32_t)N);
    if (__ballot(need != 0) != 0ull) {
      K1RowsLds<NE>& lds = *reinterpret_cast<K1RowsLds<NE>*>(smem + wave * kK1RowsLds);
      const uint32_t flip = k1_rows_select<TEAM, NE, VE>(B, sm, need, N, lds, lists + wave * (kWave / 16));
#pragma unroll
      for (int i = 0; i < NE / 4; ++i) {
        const uint32_t b = (((flip >> (4 * i)) & 15u) * 0x204081u) & 0x01010101u;  // bit e to byte e
        code[i] -= (b ^ sm) - sm;
      }
    }
  }

  // what depends on the lane alone is computed again, not kept in registers through the search
  const int lane_out = k1_tid<true>(), l_out = lane_out & (TEAM - 1), row_out = lane_out / TEAM;
  const int first_out = VE * (l_out + (NL - 1) * TEAM);
  if (l_out == 0 && row_out < rows) d.scales[c0 + row_out] = s;
  const int format = a.out_format;
  if (format == SQUANT_OUT_INT8) k1_rows_emit<NE, VE, SQUANT_OUT_INT8, TEAM>(code, d.out, c0, rows, row_out, l_out, N, s);
  else if (format == SQUANT_OUT_INT4) k1_rows_emit<NE, VE, SQUANT_OUT_INT4, TEAM>(code, d.out, c0, rows, row_out, l_out, N, s);
  else if (format == SQUANT_OUT_BF16) k1_rows_emit<NE, VE, SQUANT_OUT_BF16, TEAM>(code, d.out, c0, rows, row_out, l_out, N, s);
  else k1_rows_emit<NE, VE, SQUANT_OUT_F32, TEAM>(code, d.out, c0, rows, row_out, l_out, N, s);
  // the elements after the last whole vector of a row, one by one
  if (TAIL && row_out < rows && first_out < N && first_out + VE > N) {
    uint32_t lo = code[(NE - VE) / 4], hi = VE == 8 ? code[NE / 4 - 1] : 0u;
    const size_t m = (size_t)(c0 + row_out);
#pragma unroll 1
    for (int e = 0; e < N - first_out; ++e) {
      const uint32_t byte = lo & 255u;
      const float v = ((float)byte - 128.0f) * s;
      lo = __builtin_amdgcn_alignbit(hi, lo, 8);
      hi >>= 8;
      const size_t at = m * N + first_out + e;
      if (format == SQUANT_OUT_INT8) static_cast<uint8_t*>(d.out)[at] = (uint8_t)(byte ^ 0x80u);
      else if (format == SQUANT_OUT_BF16) static_cast<uint16_t*>(d.out)[at] = (uint16_t)bf16_bits(v);
      else if (format == SQUANT_OUT_F32) static_cast<float*>(d.out)[at] = v;
      else if ((e & 1) == 0)  // with the next element's nibble: past the end its code is 0
        static_cast<uint8_t*>(d.out)[m * ((N + 1) / 2) + (first_out + e) / 2] = (uint8_t)((byte & 15u) | (lo << 4));
    }
  }
}

// For the mixed kernel.
template <int MODE, int TEAM, bool HALF, bool TAIL>
__device__ __forceinline__ void k1_rows_dispatch(const LaunchArgs& a, const TensorDesc& d, int item, unsigned char* smem,
                                                 K1RowsList* lists) {
  if (HALF) {
    if (k1_rows_nv(d.N) <= 6) k1_rows_channels<MODE, TEAM, 24, 8, true, TAIL>(a, d, item, smem, lists);
    else k1_rows_channels<MODE, TEAM, 32, 8, true, TAIL>(a, d, item, smem, lists);
  } else {
    switch (k1_rows_nv(d.N)) {
      case 5: k1_rows_channels<MODE, TEAM, 20, 4, false, TAIL>(a, d, item, smem, lists); break;
      case 6: k1_rows_channels<MODE, TEAM, 24, 4, false, TAIL>(a, d, item, smem, lists); break;
      case 7: k1_rows_channels<MODE, TEAM, 28, 4, false, TAIL>(a, d, item, smem, lists); break;
      default: k1_rows_channels<MODE, TEAM, 32, 4, false, TAIL>(a, d, item, smem, lists); break;
    }
  }
}

// One kernel per team size and vector count (four elements each).  LDS: a K1RowsLds per wave, then the lists.
template <int MODE, int TEAM, int NV, bool HALF, bool TAIL>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) squant_channel_k1_rows(LaunchArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  int item;
  const TensorDesc d = locate(a, blockIdx.x, item);
  K1RowsList* lists = reinterpret_cast<K1RowsList*>(smem + blockDim.x / kWave * kK1RowsLds);
  k1_rows_channels<MODE, TEAM, 4 * NV, k1_ve<NV, HALF>(), HALF, TAIL>(a, d, item, smem, lists);
}

}  // namespace squant
