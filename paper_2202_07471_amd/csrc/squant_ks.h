// SQuant kernel for small convolution kernels other than 3x3 (1x3, 3x1, 1x7, 7x1, 2x2, 1x5,
// 4x4, 5x5, 7x7: K = kh*kw elements, 2 <= K <= kKsMaxK), built like the 3x3 kernel: one workgroup per
// output channel, every thread holds KPT whole kernels in registers (thread t the kernels
// t, t+G, ..., G = cin / KPT), SQuant-E, SQuant-K and the Algorithm 3 candidate are register
// arithmetic, LDS holds the histogram of SQuant-C and the channel's biased codes for the write-out.
//
// Up to seven elements the arithmetic is the 3x3 kernel's (squant_k9.h): rounding by a magic addition, codes
// packed as they come, biased perturbations, unique keys, a mask of flips that SQuant-C toggles, all with a selection
// network of its own per K.  Larger kernels step through their keys from the top.
// The version before ranked all pairs of keys (three instructions a pair), clamped and converted every
// code, stored it by itself and flipped SQuant-C's through LDS atomics.  20 M weights in channels of 192 kernels, to int8, us before and
// now: 1x7 29.1 and 22.0, 1x5 28.9 and 24.2, 1x3 33.0 and 28.6, 2x2 30.5 and 24.7; 16 x [1024, 192, 1, 7] binary16 with E&C 34.2
// and 21.6, with E&K 24.6 and 19.0; an InceptionV3-style set of 1.39 times the width, binary16, E&C 74.7 and 67.6.
#pragma once

#include "squant_common.h"
#include "squant_io.h"
#include "squant_k1.h"  // push_compares_signed
#include "squant_k9.h"  // K9Shared, rounding constants
#include "squant_plan.h"
#include "squant_select.h"

namespace squant {

// K consecutive weights (binary32 or 16-bit, at any alignment) into w[K*q .. K*q+K-1], in 16-byte
// pieces and shorter ones; a kernel behind the channel's end reads as zeros.
template <int K, int NW>
__device__ __forceinline__ void ks_load_kernel(float (&w)[NW], int q, rsrc_t row, uint32_t lane_off, uint32_t off) {
  constexpr int V4 = K / 4, R = K % 4;
#pragma unroll
  for (int j = 0; j < V4; ++j) {
    const vu4 v = buffer_load_u4(row, lane_off + 16u * j, off);
#pragma unroll
    for (int e = 0; e < 4; ++e) w[K * q + 4 * j + e] = __uint_as_float(v[e]);
  }
  if (R == 3) {
    const vu3 v = buffer_load_u3(row, lane_off + 16u * V4, off);
#pragma unroll
    for (int e = 0; e < 3; ++e) w[K * q + 4 * V4 + e] = __uint_as_float(v[e]);
  } else if (R == 2) {
    const vu2 v = buffer_load_u2(row, lane_off + 16u * V4, off);
    w[K * q + 4 * V4] = __uint_as_float(v.x); w[K * q + 4 * V4 + 1] = __uint_as_float(v.y);
  } else if (R == 1) {
    w[K * q + 4 * V4] = __uint_as_float(buffer_load_u1(row, lane_off + 16u * V4, off));
  }
}
// The dwords of K 16-bit weights; the type is looked at once, after all loads of a thread are on their way.
template <int K>
__device__ __forceinline__ void ks_load_kernel16(uint32_t (&d)[(K + 1) / 2], rsrc_t row, uint32_t lane_off, uint32_t off) {
  constexpr int V8 = K / 8;
#pragma unroll
  for (int j = 0; j < V8; ++j) {
    const vu4 v = buffer_load_u4(row, lane_off + 16u * j, off);
#pragma unroll
    for (int e = 0; e < 4; ++e) d[4 * j + e] = v[e];
  }
  if (K & 4) {
    const vu2 v = buffer_load_u2(row, lane_off + 16u * V8, off);
    d[4 * V8] = v.x; d[4 * V8 + 1] = v.y;
  }
  if (K & 2) d[(K & ~3) / 2] = buffer_load_u1(row, lane_off + 2u * (K & ~3), off);
  if (K & 1) d[K / 2] = buffer_load_u16(row, lane_off + 2u * (K - 1), off);
}
template <int K, int KPT, bool BF16>
__device__ __forceinline__ void ks_widen16(const uint32_t (&d)[KPT][(K + 1) / 2], float (&w)[K * KPT]) {
#pragma unroll
  for (int q = 0; q < KPT; ++q)
#pragma unroll
    for (int i = 0; i < K; ++i) {
      float lo, hi;
      widen_pair(d[q][i / 2], BF16, lo, hi);
      w[K * q + i] = i & 1 ? hi : lo;
    }
}

// Bits of a key's index tie-break.
template <int K>
constexpr int ks_index_bits() { return K <= 16 ? 4 : K <= 32 ? 5 : 6; }

// The k-th largest key (0x7fffffff: k = 0) and the one of rank `want`, by the keys in descending order as far as any
// kernel of the wave needs them (k is rarely above three): with keys within 2^30 of each other, key - m wraps to a huge
// number for the keys below m and to a small one for the others, so the largest difference names the next key.
// 1.5 instructions an element and step; all pairs of 25 elements took 900 and spilled.  FENCED: eight at a time, for registers.
template <int K, bool FENCED, int KP>
__device__ __forceinline__ void ks_step_keys(const int32_t (&key)[KP], int32_t k, int32_t want, int32_t& last, int32_t& ck) {
  int32_t m = key[0];
#pragma unroll
  for (int i = 1; i < K; ++i) m = imax2(m, key[i]);
  last = 0x7fffffff;
#pragma unroll 1
  for (int32_t rank = 0;; ++rank) {
    if (rank == k - 1) last = m;
    if (rank == want) ck = m;
    if (__ballot(rank < want) == 0ull) break;
    uint32_t z = 0;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      z = umax2(z, (uint32_t)key[i] - (uint32_t)m);
      if (FENCED && i % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
    m = (int32_t)((uint32_t)m + z);
  }
}

// The Algorithm 3 candidate from its key: the word and the element index.
template <int IB>
__device__ __forceinline__ void ks_candidate(int32_t ck, bool over, int32_t smask, uint32_t& cand_w, int& cand_i) {
  constexpr int IM = (1 << IB) - 1;
  const uint32_t mag = (uint32_t)ck >> IB;  // |p| of that element before any flip (if same-sign)
  const uint32_t absv = over ? (uint32_t)kOne - mag : mag;
  const uint32_t neg = (over ? ~(uint32_t)smask : (uint32_t)smask) & (1u << 23);
  cand_w = ck >= (1 << IB) ? (absv | neg) : kNoCandidate;
  cand_i = IM - (ck & IM);
}

// The sign a kernel whose perturbations P add up to 0 exactly takes, that of its largest |p| (lowest index first):
// see k9_zero_sum_sign.
template <int K, int KP>
__device__ __forceinline__ int32_t ks_zero_sum_sign(const int32_t (&P)[KP]) {
  constexpr int IB = ks_index_bits<K>(), IM = (1 << IB) - 1;
  int32_t pos = 0, neg = 0;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const int32_t p = P[i] << IB;
    pos = imax2(pos, p + (IM - i));
    neg = imax2(neg, (IM - i) - p);
  }
  return neg > pos ? -1 : 0;
}

// Cold path for kernels of 16 elements and more: the candidate of a kernel whose perturbations add up to 0, from its
// weights read once more.  Settled before the keys take the place of the perturbations, as for short kernels, it costs
// registers in every launch: 7x7, 868 a channel, 20 M binary32 weights with E&C 41.1 us so and 31.4 with this, 5x5, 300 a
// channel, binary16 23.1 and 18.3.  With E&K&C the keys are kept anyway, and 16-bit weights meet such kernels often (with one
// load after the other for each, 5x5, 192 a channel, 2 M bfloat16 weights 9.2 us, settled before 6.7): there, and for 16 elements,
// whose registers suffice, 16-bit kernels settle it before (kHere in ks_channel_long).
template <int K, bool HALF>
__device__ __forceinline__ void ks_zero_sum_candidate(rsrc_t row, uint32_t lane_off, bool bf16, float s, float qmaxf, uint32_t& cand_w,
                                                      int& cand_i) {
  int32_t best = 0, bv = 0;
  cand_i = 0;
  auto offer = [&](float w, int i) {
    int32_t P;
    round_and_perturb(w, s, qmaxf, P);
    const int32_t ap = P < 0 ? -P : P;
    if (ap > best) { best = ap; bv = P; cand_i = i; }
  };
  if (HALF) {
    uint32_t raw[(K + 1) / 2];
    ks_load_kernel16<K>(raw, row, lane_off, 0);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const uint32_t h = i & 1 ? raw[i / 2] >> 16 : raw[i / 2] & 0xFFFFu;
      offer(bf16 ? widen_bf16(h) : widen_f16(h), i);
      __builtin_amdgcn_sched_barrier(0);  // one after the other: registers
    }
  } else {
#pragma unroll 1
    for (int i = 0; i < K; ++i) offer(__uint_as_float(buffer_load_u1(row, lane_off + 4u * i, 0)), i);
  }
  cand_w = candidate_word(bv);
}

// SQuant-E, SQuant-K and the candidate update for one kernel held in registers (straight-line code, as
// for 3x3); zero: its perturbations add up to 0, the candidate is not settled.
template <int K, bool FAST, int MODE, bool HERE>
__device__ __forceinline__ void ks_solve(const float (&w)[K], float s, float rs, float qmaxf,
                                         float (&cf)[K], int32_t& esum, uint32_t& cand_w, int& cand_i, bool& zero) {
  constexpr int IB = ks_index_bits<K>(), IM = (1 << IB) - 1;
  float c[K];
  int32_t P[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const float x = FAST ? div_by_reciprocal(w[i], s, rs) : quotient(w[i], s);
    const float xc = __builtin_amdgcn_fmed3f(x, -qmaxf, qmaxf);
    c[i] = rintf(xc);
    const float p = c[i] - xc;  // exact
    // Q23 through the low mantissa bits of p * 2^23 + 1.5 * 2^23 (one rounding, half to even)
    P[i] = __float_as_int(__builtin_fmaf(p, 8388608.0f, 12582912.0f)) - 0x4B400000;
  }
  cand_w = kNoCandidate;
  cand_i = 0;
  if (MODE == SQUANT_MODE_E) {
#pragma unroll
    for (int i = 0; i < K; ++i) cf[i] = c[i] + 128.0f;
    return;
  }

  // ---- SQuant-K (Algorithm 2 on one kernel) ----
  int32_t E = 0;
#pragma unroll
  for (int i = 0; i < K; ++i) E += P[i];
  int32_t smask = E >> 31;
  const int32_t A = (E ^ smask) - smask;
  const int32_t k = (MODE == SQUANT_MODE_EC) ? 0 : (int32_t)((uint32_t)(A + kHalf - 1) >> 23);
  const int32_t r = A - (k << 23);  // |sum| left after k flips, < 0: over SQuant
  esum += (r ^ smask) - smask;
  if (!HERE) zero = E == 0;
  else if (__builtin_expect(__ballot(E == 0) != 0ull, 0)) smask = E == 0 ? ks_zero_sum_sign<K>(P) : smask;

  // unique keys: 2^IB |p| + (IM - i) >= 2^IB for the elements with the sign of the sum, below
  // 2^IB for all others; |P| <= 2^22 fits the 24-bit multiply
  int32_t key[K];
#pragma unroll
  for (int i = 0; i < K; ++i) key[i] = __mul24(P[i], smask ? -(1 << IB) : (1 << IB)) + (IM - i);
  const bool over = r < 0;
  const int32_t want = over ? k - 1 : k;  // the candidate's rank: last flipped resp. first un-flipped (k <= K/2 < K)
  const float flip = smask ? 129.0f : 127.0f;  // code -= sign(E)
  int32_t ck = 0;  // the candidate's key
  int32_t last;
  ks_step_keys<K, false>(key, k, want, last, ck);
#pragma unroll
  for (int i = 0; i < K; ++i) cf[i] = c[i] + (key[i] >= last ? flip : 128.0f);
  if (MODE == SQUANT_MODE_EK) return;

  // ---- perturbation update (Algorithm 3): the kernel's candidate for SQuant-C ----
  ks_candidate<IB>(ck, over, smask, cand_w, cand_i);
}

// The same for one kernel of more elements, one per thread.  Its perturbations take the place of the weights and its
// codes + 128 are packed as they come (`code`), so a 7x7 kernel lives in 75 registers.  5x5 kernels take it where SQuant-K
// flips nothing: 4 x [512, 300, 5, 5] in binary16 24.7 us above and 19.9 here with E&C, 12.1 and 11.4 with E, but [512, 200, 5, 5]
// 14.7 and 15.4 with E&K&C, 12.7 and 13.0 with E&K.
template <int K, int MODE>
constexpr bool ks_packed() { return K > 25 || K == 16 || (K == 25 && (MODE == SQUANT_MODE_E || MODE == SQUANT_MODE_EC)); }
template <int K, bool FAST, int MODE, bool HERE>
__device__ __forceinline__ void ks_solve_long(const float (&w)[K], float s, float rs, float qmaxf,
                                              uint32_t (&code)[(K + 3) / 4], int32_t& esum, uint32_t& cand_w, int& cand_i,
                                              bool& zero) {
  constexpr int IB = ks_index_bits<K>(), IM = (1 << IB) - 1;
  constexpr int KP = (K + 3) / 4 * 4;
  int32_t key[KP];  // first the perturbations
  uint32_t tb[KP];
#pragma unroll
  for (int i = 0; i < KP; ++i) {
    if (i < K) {
      const float x = FAST ? div_by_reciprocal(w[i], s, rs) : quotient(w[i], s);
      const float xc = __builtin_amdgcn_fmed3f(x, -qmaxf, qmaxf);
      const float t = xc + kRoundMagic;  // see squant_k9.h
      const float c = t - kRoundMagic;
      const float p = c - xc;  // exact
      key[i] = __float_as_int(__builtin_fmaf(p, 8388608.0f, kQ23Magic)) - (int32_t)kQ23Bias;
      tb[i] = __float_as_uint(t);
    } else {
      tb[i] = 128;
      key[i] = 0;
    }
    if (i % 4 == 3) {
      code[i / 4] = pack_low_bytes(tb[i - 3], tb[i - 2], tb[i - 1], tb[i]);
      __builtin_amdgcn_sched_barrier(0);  // one group at a time: registers
    }
  }
  cand_w = kNoCandidate;
  cand_i = 0;
  if (MODE == SQUANT_MODE_E) return;

  // ---- SQuant-K (Algorithm 2 on one kernel) ----
  int32_t E = 0;
#pragma unroll
  for (int i = 0; i < K; ++i) E += key[i];
  int32_t smask = E >> 31;
  const int32_t A = (E ^ smask) - smask;
  const int32_t k = (MODE == SQUANT_MODE_EC) ? 0 : (int32_t)((uint32_t)(A + kHalf - 1) >> 23);
  const int32_t r = A - (k << 23);  // |sum| left after k flips, < 0: over SQuant
  esum += (r ^ smask) - smask;
  if (!HERE) zero = E == 0;
  else if (__builtin_expect(__ballot(E == 0) != 0ull, 0)) smask = E == 0 ? ks_zero_sum_sign<K>(key) : smask;

  // unique keys: 2^IB |p| + (IM - i) >= 2^IB for the elements with the sign of the sum, below
  // 2^IB for all others; |P| <= 2^22 fits the 24-bit multiply
#pragma unroll
  for (int i = 0; i < KP; ++i) key[i] = i < K ? __mul24(key[i], smask ? -(1 << IB) : (1 << IB)) + (IM - i) : INT32_MIN / 4;
  const bool over = r < 0;
  const int32_t want = over ? k - 1 : k;  // the candidate's rank: last flipped resp. first un-flipped (k <= K/2 < K)
  int32_t ck = 0, last;
  if (MODE == SQUANT_MODE_EC) {  // nothing flips: the candidate is the largest
    ck = key[0];
#pragma unroll
    for (int i = 1; i < K; ++i) ck = imax2(ck, key[i]);
  } else {
    ks_step_keys<K, true>(key, k, want, last, ck);
#pragma unroll
    for (int base = 0; base < KP; base += 32) {
      constexpr int kGroup = 32;
      uint32_t flips = 0;
#pragma unroll
      for (int q = (KP - base < kGroup ? KP - base : kGroup) - 4; q >= 0; q -= 4) push_compares_signed(flips, last, &key[base + q]);
#pragma unroll
      for (int q = 0; q < kGroup && base + q < KP; q += 4) {
        const uint32_t b = (((flips >> q) & 15u) * 0x204081u) & 0x01010101u;  // bit e to byte e
        code[(base + q) / 4] -= (b ^ (uint32_t)smask) - (uint32_t)smask;
      }
    }
  }
  if (MODE == SQUANT_MODE_EK) return;
  ks_candidate<IB>(ck, over, smask, cand_w, cand_i);
}

// The kernel of a thread: SQuant-E, SQuant-K and its candidate, codes into its bytes of the channel.
template <int K, bool FAST, int MODE, bool HERE>
__device__ __forceinline__ void ks_solve_kernel(const float (&w)[K], float s, float rs, float qmaxf, uint8_t* code8, int32_t& esum,
                                                uint32_t& cand_w, int& cand_i, bool& zero) {
  if constexpr (ks_packed<K, MODE>()) {
    uint32_t code[(K + 3) / 4];
    ks_solve_long<K, FAST, MODE, HERE>(w, s, rs, qmaxf, code, esum, cand_w, cand_i, zero);
#pragma unroll
    for (int i = 0; i < K / 4; ++i) __builtin_memcpy(code8 + 4 * i, &code[i], 4);
#pragma unroll
    for (int i = K / 4 * 4; i < K; ++i) code8[i] = (uint8_t)(code[i / 4] >> (8 * (i & 3)));
  } else {
    float cf[K];
    ks_solve<K, FAST, MODE, HERE>(w, s, rs, qmaxf, cf, esum, cand_w, cand_i, zero);
#pragma unroll
    for (int i = 0; i < K; ++i) code8[i] = (uint8_t)(int)cf[i];
  }
}

// ---- kernels of up to seven elements: the 3x3 kernel's arithmetic ----
template <int K>
constexpr bool ks_short() { return K <= 7; }

// The K / 2 + 1 largest of K unique keys, largest first: k <= K / 2 elements flip and the next one may be wanted.  Three
// are sorted, the others inserted: a median of three gives each place.
template <int K>
__device__ __forceinline__ void ks_top(const uint32_t (&x)[K], uint32_t (&t)[K / 2 + 1]) {
  if constexpr (K == 2) {
    t[0] = umax2(x[0], x[1]);
    t[1] = umin2(x[0], x[1]);
  } else {
    constexpr int R = K / 2 + 1;
    uint32_t top[4] = {umax3(x[0], x[1], x[2]), umed3(x[0], x[1], x[2]), umin3(x[0], x[1], x[2]), 0};
#pragma unroll
    for (int i = 3; i < K; ++i) {
      uint32_t next[4];
      next[0] = umax2(top[0], x[i]);
      next[1] = umed3(top[0], top[1], x[i]);
      next[2] = umed3(top[1], top[2], x[i]);
      next[3] = i == 3 ? umin2(top[2], x[i]) : umed3(top[2], top[3], x[i]);
#pragma unroll
      for (int r = 0; r < 4; ++r) top[r] = next[r];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) t[r] = top[r];
  }
}

// SQuant-E on one kernel: see k9_round.
template <int K, bool CLAMP>
__device__ __forceinline__ void ks_round(const float (&w)[K], float s, float rs, float qmaxf, K9Kernel& kk, uint32_t (&pb)[K]) {
  uint32_t tb[8];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const float x = div_by_reciprocal(w[i], s, rs);  // the IEEE quotient
    const float xc = CLAMP ? __builtin_amdgcn_fmed3f(x, -qmaxf, qmaxf) : x;
    const float t = xc + kRoundMagic;
    pb[i] = __float_as_uint(__builtin_fmaf((t - kRoundMagic) - xc, 8388608.0f, kQ23Magic));
    tb[i] = __float_as_uint(t);
  }
  kk.d0 = K == 2 ? __builtin_amdgcn_perm(tb[1], tb[0], 0x0c0c0400u) : pack_low_bytes(tb[0], tb[1], tb[2], tb[K > 3 ? 3 : 2]);
  if (K == 5) kk.d1 = tb[4];  // its upper bytes are not codes
  if (K == 7) kk.d1 = pack_low_bytes(tb[4], tb[5], tb[6], tb[6]);
}

// See k9_zero_sum_sign.
template <int K>
__device__ __forceinline__ uint32_t ks_zero_sum_bits(const uint32_t (&pb)[K]) {
  int32_t P[K];
#pragma unroll
  for (int i = 0; i < K; ++i) P[i] = (int32_t)(pb[i] - kQ23Bias);
  return (uint32_t)ks_zero_sum_sign<K>(P);
}

// SQuant-K and the perturbation update for one kernel: see k9_flip, whose words these are.
template <int MODE, int K>
__device__ __forceinline__ void ks_flip(const uint32_t (&pb)[K], K9Kernel& kk, int32_t& esum, lanemask_t real) {
  constexpr bool kCand = MODE == SQUANT_MODE_EKC || MODE == SQUANT_MODE_EC;
  constexpr int R = K / 2 + 1;
  uint32_t eb = 0;
#pragma unroll
  for (int i = 0; i < K; ++i) eb += pb[i];
  const int32_t E = (int32_t)(eb - (uint32_t)K * kQ23Bias);
  uint32_t sm = (uint32_t)(E >> 31);
  const uint32_t A = ((uint32_t)E ^ sm) - sm;
  if (kCand) {
    const lanemask_t zero = lanes_eq(A, 0u) & real;
    if (__builtin_expect(zero != 0, 0)) sm = vsel(zero, ks_zero_sum_bits<K>(pb), sm);
  }
  kk.sm = sm;
  uint32_t key[K];
#pragma unroll
  for (int i = 0; i < K; ++i) key[i] = ((pb[i] ^ sm) << 5) | (uint32_t)(31 - i);
  const uint32_t base = (kQ23Bias << 5) + (sm & (((~kQ23Bias) << 5) - (kQ23Bias << 5)));

  if (MODE == SQUANT_MODE_EC) {
    esum += E;
    uint32_t ck = key[0];
#pragma unroll
    for (int i = 1; i < K; i += 2) ck = umax3(ck, key[i], key[i + 1 < K ? i + 1 : i]);
    const int32_t rel = (int32_t)(ck - base);
    kk.cand = vsel(lanes_sge(rel, 32), ((uint32_t)rel >> 5) | (sm & (1u << 23)), kNoCandidate);
    kk.cand_bit = 0x80000000u >> (ck & 31u);
    return;
  }

  const uint32_t tt = A + (uint32_t)(kHalf - 1);  // k = tt >> 23
  const int32_t r = (int32_t)(tt & 0x7FFFFFu) - (kHalf - 1);
  esum += (int32_t)(((uint32_t)r ^ sm) - sm);
  uint32_t top[R];
  ks_top<K>(key, top);
  uint32_t mask = 0x80000000u >> (top[0] & 31u);
  lanemask_t at_least = lanes_uge(tt, 1u << 23);
  uint32_t flips = vsel0(at_least, mask), thr = top[0], nxt = 0;  // thr: the k-th largest, k >= 1; nxt: the next one
  if (kCand) nxt = vsel(at_least, top[1], top[0]);
#pragma unroll
  for (int k = 2; k < R; ++k) {
    at_least = lanes_uge(tt, (uint32_t)k << 23);
    mask |= 0x80000000u >> (top[k - 1] & 31u);
    flips = vsel(at_least, mask, flips);
    if (kCand) {
      thr = vsel(at_least, top[k - 1], thr);
      nxt = vsel(at_least, top[k], nxt);
    }
  }
  kk.flips = flips;
  if (!kCand) return;

  const lanemask_t over = lanes_slt(r, 0);
  const uint32_t ck = vsel(over, thr, nxt);
  const int32_t rel = (int32_t)(ck - base);
  const uint32_t mag = (uint32_t)rel >> 5, sbit = sm & (1u << 23);
  const uint32_t word = vsel(over, ((2u << 23) - sbit) - mag, mag | sbit);
  kk.cand = vsel(lanes_sge(rel, 32), word, kNoCandidate);
  kk.cand_bit = 0x80000000u >> (ck & 31u);
}

template <int K>
__device__ __forceinline__ void ks_apply_flips(K9Kernel& kk) {
  const uint32_t b0 = ((kk.flips & 15u) * 0x204081u) & 0x01010101u;  // bit e to byte e
  kk.d0 -= (b0 ^ kk.sm) - kk.sm;
  if (K > 4) {
    const uint32_t b1 = ((kk.flips >> 4) * 0x204081u) & 0x01010101u;
    kk.d1 -= (b1 ^ kk.sm) - kk.sm;
  }
}

// SQuant-E and SQuant-K on all the kernels of a thread: see k9_solve_all.
template <int MODE, int K, int KPT, bool GENERAL>
__device__ __forceinline__ void ks_solve_short(const float (&w)[K * KPT], float s, float rs, float qmaxf, float f1, float f2,
                                               K9Kernel (&kk)[KPT], int32_t& esum, const lanemask_t (&real)[KPT]) {
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    kk[q].d0 = kk[q].d1 = kk[q].flips = kk[q].sm = kk[q].cand_bit = 0;
    kk[q].cand = kNoCandidate;
    if (__float_as_uint(s) + (uint32_t)q == 0xFFFFFFF0u) continue;  // never: a basic block for each kernel
    float x[K];
#pragma unroll
    for (int i = 0; i < K; ++i) x[i] = GENERAL ? w[K * q + i] * f1 * f2 : w[K * q + i];
    uint32_t pb[K];
    ks_round<K, GENERAL>(x, s, rs, qmaxf, kk[q], pb);
    if (MODE != SQUANT_MODE_E) {
      ks_flip<MODE, K>(pb, kk[q], esum, real[q]);
      if (MODE == SQUANT_MODE_EK) ks_apply_flips<K>(kk[q]);
    }
  }
}

// A channel of such kernels from its weights in w on: codes into `code8`.  As in k9_channel.
template <int MODE, int K, int KPT>
__device__ __forceinline__ void ks_channel_short(const float (&w)[K * KPT], float amax, float s, bool normal, float qmaxf, int N, int t,
                                                 int G, uint32_t owned, uint8_t* code8, K9Shared& sh) {
  constexpr bool kChannelStage = MODE == SQUANT_MODE_EKC || MODE == SQUANT_MODE_EC;
  K9Kernel kk[KPT];
  int32_t esum = 0;
  lanemask_t real[KPT];
#pragma unroll
  for (int q = 0; q < KPT; ++q) real[q] = __ballot((owned >> q) & 1u);
  const float rs0 = reciprocal(s);
  if (normal && div_by_reciprocal(amax, s, rs0) <= qmaxf) {
    ks_solve_short<MODE, K, KPT, false>(w, s, rs0, qmaxf, 1.0f, 1.0f, kk, esum, real);
  } else {  // a quotient beyond qmax, or an absmax outside the range of the reciprocal: scaled by powers of two
    const float f1 = normal ? 1.0f : amax < 1.0f ? 0x1p64f : 0x1p-64f;
    const float a1 = amax * f1;
    const float f2 = normal ? 1.0f : a1 < 0x1p-60f ? 0x1p64f : a1 > 0x1p60f ? 0x1p-64f : 1.0f;
    const float s2 = s > 0.0f ? s * f1 * f2 : 0x1p-40f;
    ks_solve_short<MODE, K, KPT, true>(w, s2, reciprocal(s2), qmaxf, f1, f2, kk, esum, real);
  }
  if (kChannelStage) {
#pragma unroll
    for (int q = 0; q < KPT; ++q)
      if ((owned >> q) & 1u) count_candidate(sh.sel, kk[q].cand);
    // after SQuant-K a kernel's sum is at most a half, eight of a thread 2^25; without it up to 3.5
    const int64_t ws = MODE == SQUANT_MODE_EC ? wave_sum_dpp(owned ? esum : 0) : wave_sum_rows(owned ? esum : 0);
    const int64_t ec = k9_block_sum<0>(ws, sh.red_i);
    k9_channel_flip<KPT, true>(kk, ec, N, t, G, owned, reinterpret_cast<uint32_t*>(code8), sh.sel);
#pragma unroll
    for (int q = 0; q < KPT; ++q) ks_apply_flips<K>(kk[q]);
  }
  // with SQuant-E alone, one kernel of two or three elements a thread: the few bytes one by one (3x1, 64 a channel, 20 M
  // weights to bfloat16 34.8 us as dwords, 34.4 so)
  store_kernel_codes<K, KPT == 1>(code8, t, G, owned, kk, !(MODE == SQUANT_MODE_E && K <= 3 && KPT == 1));
}

// The same for larger kernels, one a thread; `row`, `lane_off`: where the kernel's weights lie.
template <int MODE, int K, bool HALF>
__device__ __forceinline__ void ks_channel_long(const float (&w)[K], float s, bool normal, float qmaxf, int N, int t, bool active,
                                                uint8_t* code8, K9Shared& sh, rsrc_t row, uint32_t lane_off, bool bf16) {
  constexpr bool kChannelStage = MODE == SQUANT_MODE_EKC || MODE == SQUANT_MODE_EC;
  constexpr bool kHere = HALF && (MODE == SQUANT_MODE_EKC || K == 16);  // see ks_zero_sum_candidate
  int32_t esum = 0;
  uint32_t cv[1] = {kNoCandidate};
  int ci = 0;
  bool zero = false;
  if (active) {
    if (normal) ks_solve_kernel<K, true, MODE, kHere>(w, s, reciprocal(s), qmaxf, code8 + K * t, esum, cv[0], ci, zero);  // uniform
    else ks_solve_kernel<K, false, MODE, kHere>(w, s, 0.0f, qmaxf, code8 + K * t, esum, cv[0], ci, zero);
  }
  if (kChannelStage) {
    if (active) {
      if (!kHere && zero) ks_zero_sum_candidate<K, HALF>(row, lane_off, bf16, s, qmaxf, cv[0], ci);
      count_candidate(sh.sel, cv[0]);
    }
    const int64_t ec = block_sum_dpp1(esum, sh.red_i);
    const int sgn = sign_of(ec);
    const int64_t kc = flips_for(ec < 0 ? -ec : ec);
    if (kc > 0) {
      const int cpos[1] = {K * t + ci}, cn[1] = {t};
      channel_stage<1, 1>(cv, cpos, cn, sgn, (uint32_t)(kc > N ? N : kc), reinterpret_cast<uint32_t*>(code8), sh.sel);
    }
  }
}

// One workgroup per output channel of N kernels, any N and any alignment; thread t takes kernels
// t, t + G, ..., G = ceil(N / KPT) in whole fours.  HALF: 16-bit weights.  (One routine for both widths waits for the weights
// before it clears the histogram, see squant_k9.h: 7x7 kernels, 192 a channel, 20 M binary32 weights with E 28.3 us and
// 25.5 so; 1x2, 64 a channel, 20 M bfloat16 to 4 bit 69.1 and 63.9)
template <int MODE, int K, int KPT, bool HALF>
__device__ __forceinline__ void ks_channel(const LaunchArgs& a, const TensorDesc& d, int m,
                                           unsigned char* smem, K9Shared& sh) {
  constexpr bool kChannelStage = MODE == SQUANT_MODE_EKC || MODE == SQUANT_MODE_EC;
  const int T = blockDim.x, tid = threadIdx.x;
  const float qmaxf = (float)a.qmax;
  uint8_t* code8 = reinterpret_cast<uint8_t*>(smem);  // biased codes: code + 128

  const int N = d.N, G = KPT == 1 ? N : ((N + KPT - 1) / KPT + 3) & ~3;  // whole quads: see store_kernel_codes
  const int L = K * N;
  const bool active = tid < G;
  const int t = tid;
  uint32_t owned = active ? ~0u : 0u;  // bit q: kernel t + q * G exists and is this thread's
  if (active) {
#pragma unroll
    for (int q = KPT == 1 ? 1 : 0; q < KPT; ++q) owned &= t + q * G < N ? ~0u : ~(1u << q);
  }
  float w[K * KPT];
  uint32_t raw[KPT][(K + 1) / 2];
  constexpr uint32_t each = K * (HALF ? 2u : 4u);  // bytes of a kernel
  const rsrc_t row = make_rsrc(static_cast<const uint8_t*>(d.w) + (size_t)m * N * each, each * (uint32_t)N);
  const uint32_t lane_off = active ? each * (uint32_t)t : 0x40000000u;  // idle threads: out of range
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    if (HALF) ks_load_kernel16<K>(raw[q], row, lane_off, each * (uint32_t)(q * G));
    else ks_load_kernel<K>(w, q, row, lane_off, each * (uint32_t)(q * G));
  }
  if (kChannelStage) select_reset(sh.sel);  // before the first barrier, and while the weights are on their way
  if (HALF) {
    if (a.wtype == SQUANT_W_BF16) ks_widen16<K, KPT, true>(raw, w);
    else ks_widen16<K, KPT, false>(raw, w);
    weights_are_here();
  }

  float amax = 0.0f;
#pragma unroll
  for (int j = 0; j < K * KPT; ++j) amax = fmaxf(amax, fabsf(w[j]));
  amax = block_max_dpp1(amax, sh.red_f);
  const bool normal = scale_is_normal(amax);
  const float s = channel_scale(amax, qmaxf, a.rcp_qmax, normal);
  if (tid == 0) d.scales[m] = s;

  if constexpr (ks_short<K>()) {
    ks_channel_short<MODE, K, KPT>(w, amax, s, normal, qmaxf, N, t, G, owned, code8, sh);
  } else {
    static_assert(KPT == 1, "larger kernels: one a thread");
    ks_channel_long<MODE, K, HALF>(w, s, normal, qmaxf, N, t, active, code8, sh, row, lane_off, a.wtype == SQUANT_W_BF16);
  }
  if (tid == 0) code8[L] = 128;  // the element a packed row of odd length is short of
  __syncthreads();

  emit_row(code8, L, d.out, m, s, a.out_format, tid, T);
}

// Up to 256 threads: compiled for five waves per SIMD (measured 1-3.5 % faster than the
// compiler's own choice of four for 1x3, 1x7 and 2x2 kernels; six costs 5x5 27 %, eight spills), for three with 7x7
// kernels, which leave a few registers to scratch memory even so.  4x4 and 7x7 kernels went through the generic
// routine before: 2 x [162, 184, 7, 7] 106 -> 10.2 us, 16 x [256, 64, 7, 7] 234 -> 16.0, 4 x [256, 512, 7, 7] in
// binary16 941 -> 30, 16 x [512, 64, 4, 4] 49.9 -> 11.1, 2 x [512, 1000, 4, 4] 129 -> 22.3, all to int8.
template <int MAX_THREADS, int MODE, int K, int KPT, bool HALF>
__global__ void __launch_bounds__(MAX_THREADS)
    __attribute__((amdgpu_waves_per_eu(K == 16 ? 8 : K == 25 ? 5 : MAX_THREADS > 256 ? 1 : K == 49 ? 3 : 5))) squant_channel_ks(LaunchArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];  // K*N bytes of codes
  __shared__ K9Shared sh;
  int m;
  const TensorDesc d = locate(a, blockIdx.x, m);
  ks_channel<MODE, K, KPT, HALF>(a, d, m, smem, sh);
}

// The routine for a channel of N kernels of K elements in a workgroup of T threads: as few kernels
// per thread as T allows.
template <int MODE, int K, bool HALF>
__device__ __forceinline__ void ks_channel_fit(const LaunchArgs& a, const TensorDesc& d, int m, unsigned char* smem,
                                               K9Shared& sh) {
  constexpr int top = ks_max_kpt_log2(K);
  const int N = d.N, T = blockDim.x;
  if (N <= T || top < 1) { ks_channel<MODE, K, 1, HALF>(a, d, m, smem, sh); return; }
  if constexpr (top >= 1)
    if (N <= 2 * T) { ks_channel<MODE, K, 2, HALF>(a, d, m, smem, sh); return; }
  if constexpr (top >= 2)
    if (N <= 4 * T) { ks_channel<MODE, K, 4, HALF>(a, d, m, smem, sh); return; }
  if constexpr (top >= 3) ks_channel<MODE, K, 8, HALF>(a, d, m, smem, sh);
}

// For the mixed kernel.
template <int MODE, bool HALF>
__device__ __forceinline__ void ks_dispatch(const LaunchArgs& a, const TensorDesc& d, int m, unsigned char* smem,
                                            K9Shared& sh) {
  switch (d.K) {
    case 2: ks_channel_fit<MODE, 2, HALF>(a, d, m, smem, sh); break;
    case 3: ks_channel_fit<MODE, 3, HALF>(a, d, m, smem, sh); break;
    case 4: ks_channel_fit<MODE, 4, HALF>(a, d, m, smem, sh); break;
    case 5: ks_channel_fit<MODE, 5, HALF>(a, d, m, smem, sh); break;
    case 7: ks_channel_fit<MODE, 7, HALF>(a, d, m, smem, sh); break;
    case 16: ks_channel_fit<MODE, 16, HALF>(a, d, m, smem, sh); break;
    case 25: ks_channel_fit<MODE, 25, HALF>(a, d, m, smem, sh); break;
    default: break;  // the host puts no other tensor here
  }
}

}  // namespace squant
