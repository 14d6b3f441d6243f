// SQuant kernels for 1x1 convolutions and fully connected layers (K = kh*kw = 1).
//
// With one element per kernel SQuant-K has nothing to do (k = round(|p|) = 0 for |p| <= 0.5,
// Section 3.4), every element is its own kernel, and its rounding perturbation is its
// SQuant-C candidate (Algorithm 3, "under SQuant" with k = 0).  A TEAM of threads owns an
// output channel: a whole workgroup (squant_channel_k1) or, for channels of up to 2048
// elements, a single wave (squant_k1_wave.h).  A thread holds NE elements in vectors of VE
// (16 bytes: four binary32 or eight 16-bit weights; 8 bytes where an odd number of four-element
// vectors is wanted): vector j of thread t is vector t + j*T of the channel, so every load
// instruction of a wave reads 1 KB of consecutive weights.  The weights never touch LDS, the
// codes never leave the registers until they are stored.
//
// The kernels are bound by the vector instructions issued per weight (a wave64 instruction
// occupies its SIMD for two to four cycles), so everything per element is counted:
//   * loads and stores are buffer instructions on a descriptor of the channel's row: one
//     address register for all vectors, and the hardware's range check takes the place of the
//     per-vector bounds checks (out-of-range dwords read as 0 and are not written);
//   * SQuant-E is 9.75 instructions an element: three for the exact quotient (two for 16-bit weights, whose quotients
//     by the scales they can have are exact so: six linear layers in bfloat16 118.4 -> 117.0 us, 16 x [4096, 2048] 87.8 -> 86.2), rounding by a
//     magic addition that leaves code + 128 in the sum's low byte (squant_k9.h), the biased
//     Q23 perturbation by one FMA.  While the scale is a normal number the clamp to +-qmax can
//     only move the element that set it, by one rounding, so it is left out and such elements are
//     mended afterwards in the few channels that have one (channels of an absmax outside
//     [2^-60, 2^60] take a clamp: a subnormal scale has few significant bits);
//   * SQuant-C needs the `need` = round(|sum|) elements with the largest perturbation of one
//     sign, a handful in thousands.  It is found by threshold search: two instructions an
//     element (compare into the carry, add-with-carry) give a mask of the elements at or above
//     a threshold, a population count says how many they are.  The first threshold comes from
//     the density of evenly spread perturbations and aims a little below the need-th largest;
//     on Gaussian or heavy-tailed weights it is the only one (1.0 to 1.1 passes on average at 3
//     bits and more, about 2 where few weights are left outside the centre).  The elements
//     between the best bounds found, at most kListCap, go to a list in LDS and are ranked there.
// The version before counted every element into an LDS histogram (three instructions and an LDS
// atomic), took two passes of two instructions over it and checked bounds per vector.  Vector
// instructions per wave, before and after, and time:
//   bfloat16 -> packed 4 bit, cin 4096, one wave of 64 elements a lane: 1958 -> 1352
//     (six linear layers, 201 M weights: 254 -> 119 us, 2.0 -> 4.2 TB/s)
//   binary16 -> int8, cin 512, four channels a wave: 1499 -> 1046
//     (64 x [2048, 512], 67 M weights: 81 -> 59 us, 2.5 -> 3.4 TB/s)
#pragma once

#include <type_traits>

#include "squant_common.h"
#include "squant_io.h"
#include "squant_k9.h"  // rounding constants, pack_low_bytes
#include "squant_select.h"

namespace squant {

// ---- what differs between a workgroup on one channel and a wave on a channel of its own ----
// WAVE: the "threads" are the wave's lanes and a barrier only has to keep the compiler from
// moving LDS accesses across it (the LDS handles a wave's instructions in order).
template <bool WAVE>
__device__ __forceinline__ int k1_tid() {
  if (!WAVE) return (int)threadIdx.x;
  // The wave kernel calls from inside its loop over channels.  The empty statement keeps the
  // compiler from computing everything that depends on the lane once before that loop, where
  // it does not fit the registers and comes back from scratch memory in every round.
  int lane = (int)(threadIdx.x & (kWave - 1));
  asm volatile("" : "+v"(lane));
  return lane;
}
template <bool WAVE>
__device__ __forceinline__ int k1_team() { return WAVE ? kWave : (int)blockDim.x; }
template <bool WAVE>
__device__ __forceinline__ void k1_sync() {
  if (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// LDS of a team: the ranking list and, for a workgroup, what its waves exchange.
struct alignas(16) K1List {
  uint64_t list[kListCap + 8];  // padding: the ranking reads entries in eights
};
struct alignas(16) K1Shared : K1List {
  float red_f[16];
  int64_t red_i[16];
  uint32_t cnt[2][16];  // counts per wave, two sets in turn
  uint32_t list_count;
};

// ---------------------------------------------------------------------------
// loads
// ---------------------------------------------------------------------------
// The raw dwords of a thread's vectors.  N elements from `src`; HALF: 16-bit elements, where
// the last dword of an odd row is only half inside and reads as 0: `tail` takes its element.
// TAIL: N need not be a multiple of VE.
template <int NE, int VE, bool HALF, bool TAIL>
__device__ __forceinline__ void k1_load(const void* src, int N, int tid, int T,
                                        uint32_t (&raw)[HALF ? NE / 2 : NE], uint32_t& tail) {
  constexpr int NL = NE / VE;
  const rsrc_t row = make_rsrc(src, HALF ? 2u * ((uint32_t)N & ~1u) : 4u * (uint32_t)N);
  constexpr int kBytes = VE * (HALF ? 2 : 4);
  const uint32_t at = (uint32_t)tid * kBytes;
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const uint32_t step = (uint32_t)(j * kBytes) * (uint32_t)T;
    if (kBytes == 16) {
      const vu4 v = buffer_load_u4_stream(row, at, step);
      raw[4 * j] = v.x; raw[4 * j + 1] = v.y; raw[4 * j + 2] = v.z; raw[4 * j + 3] = v.w;
    } else {
      const vu2 v = buffer_load_u2_stream(row, at, step);
      raw[2 * j] = v.x; raw[2 * j + 1] = v.y;
    }
  }
  tail = 0;
  if (HALF && TAIL && (N & 1)) tail = static_cast<const uint16_t*>(src)[N - 1];
}

// Vector and thread that hold element n (uniform).
struct K1Place { int j, thread; };
template <int VE>
__device__ __forceinline__ K1Place k1_place(int n, int T) {
  const int v = n / VE, j = v / T;
  return {j, v - j * T};
}

// The raw dwords as binary32 weights.
template <int NE, int VE, bool HALF, bool TAIL>
__device__ __forceinline__ void k1_widen(uint32_t (&raw)[HALF ? NE / 2 : NE], uint32_t tail, bool bf16, int N,
                                         int tid, int T, float (&w)[NE]) {
  if (!HALF) {
#pragma unroll
    for (int q = 0; q < NE; ++q) w[q] = __uint_as_float(raw[q]);
    return;
  }
  if (TAIL && (N & 1)) {
    const K1Place p = k1_place<VE>(N - 1, T);
    const int at = p.j * (VE / 2) + ((N - 1) % VE) / 2;
#pragma unroll
    for (int r = 0; r < NE / 2; ++r)
      if (r == at) raw[r] = tid == p.thread ? tail : raw[r];
  }
  if (bf16) {
#pragma unroll
    for (int r = 0; r < NE / 2; ++r) widen_pair(raw[r], true, w[2 * r], w[2 * r + 1]);
  } else {
#pragma unroll
    for (int r = 0; r < NE / 2; ++r) widen_pair(raw[r], false, w[2 * r], w[2 * r + 1]);
  }
}

// ---------------------------------------------------------------------------
// SQuant-E
// ---------------------------------------------------------------------------
// x = w / s for the NE elements of a thread: the packed biased codes (code + 128, four to a
// dword) and, WITH_P, the Q23 perturbations in biased form (kQ23Bias + P).  `over` (uniform):
// the quotient of the absmax element exceeds qmax.  Returns the sum of the P.
// HALF: 16-bit weights.
template <int NE, bool WITH_P, bool HALF>
__device__ __forceinline__ int32_t k1_round_all(const float (&w)[NE], float s, float rs, float qmaxf,
                                                float xmax, uint32_t (&code)[NE / 4], uint32_t (&B)[NE]) {
  uint32_t biased = 0;
  const float rl = HALF ? reciprocal_low(s, rs) : 0.0f;
#pragma unroll
  for (int i = 0; i < NE / 4; ++i) {
    uint32_t tb[4];
    float x[4];  // the IEEE quotients
    // The two operations of 16-bit weights in stages of four elements: left alone the compiler takes one element to its end
    // before it begins the next, every instruction waits for the one before, and with the two to four waves a SIMD that long
    // rows have nothing hides that.  64 M weights bfloat16 to int8, us with three operations, with two one element after
    // the other, and so: cin 24576 52.7, 50.3, 48.0, 32768 49.1, 50.5, 48.3, 50176 79.2, 80.7, 78.6; binary16 to 4 bit 40960 65.6, 65.5, 63.1.
    if (HALF) {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = w[4 * i + e] * rl;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = __builtin_fmaf(w[4 * i + e], rs, x[e]);  // half_quotient
      __builtin_amdgcn_sched_barrier(0);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = div_by_reciprocal(w[4 * i + e], s, rs);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float t = x[e] + kRoundMagic;  // round half to even; code + 128 in the low byte
      tb[e] = __float_as_uint(t);
      if (WITH_P) {
        const float c = t - kRoundMagic;
        const float p = c - x[e];  // exact
        const uint32_t pb = __float_as_uint(__builtin_fmaf(p, 8388608.0f, kQ23Magic));
        biased += pb;
        B[4 * i + e] = pb;
      }
    }
    code[i] = pack_low_bytes(tb[0], tb[1], tb[2], tb[3]);
    // keeps the scheduler from interleaving the vectors of the thread, which costs tens of
    // registers and with them occupancy
    __builtin_amdgcn_sched_barrier(0);
  }
  if (WITH_P && xmax > qmaxf) {
    // The clamp (Section 2.2), after the fact: an element whose quotient is +-xmax rounded to
    // +-qmax all the same, but its perturbation is that of +-qmax itself, 0.  No other element
    // with that code has the perturbation of xmax.
    const uint32_t d = __float_as_uint(__builtin_fmaf(qmaxf - xmax, 8388608.0f, kQ23Magic));  // P of +xmax
    const uint32_t top = 128u + (uint32_t)qmaxf, bottom = 128u - (uint32_t)qmaxf;
#pragma unroll
    for (int q = 0; q < NE; ++q) {
      const uint32_t c = (code[q / 4] >> (8 * (q & 3))) & 255u;
      const bool hit = (c == top && B[q] == d) || (c == bottom && B[q] == 2u * kQ23Bias - d);
      biased += hit ? kQ23Bias - B[q] : 0u;
      B[q] = hit ? kQ23Bias : B[q];
    }
  }
  return (int32_t)(biased - (uint32_t)NE * kQ23Bias);
}

// ---------------------------------------------------------------------------
// SQuant-C: among the elements whose P has the sign of the channel sum, the `need` with the
// largest |P|, lowest index first on ties (Algorithm 2 on the channel, Eq. 7).  u = P (sum > 0)
// or ~P (sum < 0) orders the wanted side "larger is better": its elements are those with u > 0
// resp. u >= 0.  Elements past the channel's end hold P = 0 and are on neither side.
// ---------------------------------------------------------------------------
// Order within the channel, and the owner, of element q of thread t: vector, thread, element.
template <int VE>
__device__ __forceinline__ uint32_t k1_owner_word(int tid, int q) {
  return ((uint32_t)(q / VE) << 13) | ((uint32_t)tid << 3) | (uint32_t)(q % VE);
}

// Ranks the entries (order of u above ~owner word, so all different and not 0) of the list and
// sets the bits of the `need` largest in their owners' masks: bit q % 32 of word
// owner[(q / 32) * T + thread].  Four threads share an entry, each comparing it with every fourth
// pair; the eight entries after the last are 0.  After a barrier that follows the last push;
// another must follow before the masks are read.
template <bool WAVE, int VE>
__device__ __forceinline__ void k1_rank(const uint64_t* list, uint32_t* owner, uint32_t count, uint32_t need) {
  const uint32_t tid = (uint32_t)k1_tid<WAVE>(), T = (uint32_t)k1_team<WAVE>();
  auto pick = [&](uint64_t entry) {
    const uint32_t n = ~(uint32_t)entry;
    const uint32_t q = (n >> 13) * VE + (n & 7u), t = (n >> 3) & 1023u;
    atomicOr(&owner[(q >> 5) * T + t], 1u << (q & 31u));
  };
  const uint32_t sub = tid & 3u;
  for (uint32_t i0 = 0; i0 < count; i0 += T >> 2) {
    const uint32_t i = umin2(i0 + (tid >> 2), count);  // past the end: an entry of 0, never picked
    const uint64_t own = list[i];
    int rank = 0;
    for (uint32_t g = 0; g < count; g += 8) {
      const ulonglong2 two = *reinterpret_cast<const ulonglong2*>(list + (g + 2 * sub));
      rank += two.x > own ? 1 : 0;
      rank += two.y > own ? 1 : 0;
    }
    rank += __builtin_amdgcn_update_dpp(0, rank, 0xB1, 0xf, 0xf, true);  // quad_perm [1,0,3,2]
    rank += __builtin_amdgcn_update_dpp(0, rank, 0x4E, 0xf, 0xf, true);  // quad_perm [2,3,0,1]
    if (sub == 0 && (uint32_t)rank < need) pick(own);
  }
}

// Sum over the team of one count per wave (uniform over the wave); one barrier, for callers that
// alternate `set`.
template <bool WAVE, typename Sh>
__device__ __forceinline__ uint32_t k1_team_count(Sh& sh, uint32_t wave_total, int set) {
  if constexpr (WAVE) {
    return wave_total;
  } else {
    const int wid = threadIdx.x / kWave, nw = (blockDim.x + kWave - 1) / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) sh.cnt[set][wid] = wave_total;
    __syncthreads();
    uint32_t r = 0;
    for (int i = 0; i < nw; ++i) r += sh.cnt[set][i];
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)r);
  }
}

// Shifts the four results b[i] >= t (AT_LEAST) or b[i] <= t into m, b[3] first, so that b[0]
// ends up in bit 0: four compares and four additions with carry.  Ordered so that at least two
// instructions lie between a compare and the addition that reads its result, which this
// hardware asks for where the compiler does not see the pair.
#define SQ_PUSH(CMP, T)                               \
  asm(CMP " %1, %5, %9\n\t"                           \
      CMP " %2, %5, %8\n\t"                           \
      CMP " %3, %5, %7\n\t"                           \
      "v_addc_co_u32_e64 %0, %1, %0, %0, %1\n\t"      \
      CMP " %4, %5, %6\n\t"                           \
      "v_addc_co_u32_e64 %0, %2, %0, %0, %2\n\t"      \
      "v_addc_co_u32_e64 %0, %3, %0, %0, %3\n\t"      \
      "v_addc_co_u32_e64 %0, %4, %0, %0, %4"          \
      : "+v"(m), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3) \
      : T(t), "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]))
template <bool AT_LEAST>
__device__ __forceinline__ void push_compares(uint32_t& m, uint32_t t, const uint32_t* b) {
  uint64_t c0, c1, c2, c3;
  if (AT_LEAST) SQ_PUSH("v_cmp_le_u32_e64", "s");
  else SQ_PUSH("v_cmp_ge_u32_e64", "s");
}
// b[i] >= t with a threshold of the lane's own.
__device__ __forceinline__ void push_compares_lanes(uint32_t& m, uint32_t t, const uint32_t* b) {
  uint64_t c0, c1, c2, c3;
  SQ_PUSH("v_cmp_le_u32_e64", "v");
}
// The same for signed words.
__device__ __forceinline__ void push_compares_signed(uint32_t& m, int32_t t, const int32_t* b) {
  uint64_t c0, c1, c2, c3;
  SQ_PUSH("v_cmp_le_i32_e64", "v");
}
#undef SQ_PUSH

// Moves the bounds of the search onto elements: lo to the smallest u >= lo, hi behind the largest
// u < hi (uniform).  Four instructions an element, two passes' worth.  One barrier; that of a pass of
// the search lies between two calls.
template <int NE, bool WAVE, typename Sh>
__device__ __forceinline__ void k1_close_in(const uint32_t (&B)[NE], int32_t sm, int32_t& lo, int32_t& hi, Sh& sh) {
  // the empty statement keeps the compiler from computing B[q] ^ sm once before the search's loop,
  // in a register for each
  asm volatile("" : "+s"(sm));
  const uint32_t base = (kQ23Bias ^ (uint32_t)sm) - (uint32_t)sm;  // B[q] ^ sm = base + u
  const uint32_t from = base + (uint32_t)lo, to = base + (uint32_t)(hi - 1);
  uint32_t above = ~0u, below = ~0u;  // distances from the bounds; elements outside wrap to larger ones
#pragma unroll
  for (int q = 0; q < NE; q += 2) {
    const uint32_t x0 = B[q] ^ (uint32_t)sm, x1 = B[q + 1] ^ (uint32_t)sm;
    above = umin3(above, x0 - from, x1 - from);
    below = umin3(below, to - x0, to - x1);
    __builtin_amdgcn_sched_barrier(0);  // one pair at a time: registers are short here
  }
  above = ~(uint32_t)__builtin_amdgcn_readlane((int)wave_prefix_max_u32(~above), kWave - 1);
  below = ~(uint32_t)__builtin_amdgcn_readlane((int)wave_prefix_max_u32(~below), kWave - 1);
  if constexpr (!WAVE) {
    const int wid = threadIdx.x / kWave, nw = (blockDim.x + kWave - 1) / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) sh.red_i[wid] = (int64_t)(((uint64_t)below << 32) | above);
    __syncthreads();
#pragma unroll 1
    for (int i = 0; i < nw; ++i) {
      const uint64_t two = (uint64_t)sh.red_i[i];
      above = umin2(above, (uint32_t)two);
      below = umin2(below, (uint32_t)(two >> 32));
    }
    above = (uint32_t)__builtin_amdgcn_readfirstlane((int)above);
    below = (uint32_t)__builtin_amdgcn_readfirstlane((int)below);
  }
  // weights that are not finite leave elements beyond both bounds: the interval never turns over
  above = umin2(above, (uint32_t)(hi - lo - 1));
  below = umin2(below, (uint32_t)(hi - lo - 1) - above);
  lo += (int32_t)above;
  hi -= (int32_t)below;
}

// The next threshold after one, `thr`, that only n < need elements reach, while no lower bound is known;
// it aims at need + extra.
// Widen the distance from the top in proportion.  Where outliers set the scale the rest
// crowds around 0 and that lands far below the need-th element.  About half the row lies on the
// wanted side, so (0, N / 2) and the count just taken give a line through logarithms; the
// nearer of the two is taken, a quarter further from the top at least.  Passes on average without
// and with that line, 2 bits: 1 % outliers 4.5 and 3.3 (N = 2024), Student-t 3.4 and 2.8.  Six linear
// layers, 49 M weights with outliers, 2 bits: binary32 62.5 -> 56.6 us, bfloat16 55.4 -> 49.4.
__device__ __forceinline__ int32_t k1_lower_threshold(int32_t thr, uint32_t n, uint32_t need, float extra, int N) {
  // The empty statement keeps what depends on N alone from being computed before the loop.
  uint32_t half = (uint32_t)N >> 1;
  asm volatile("" : "+s"(half));
  const float few = (float)need, from_top = (float)((1 << 22) + 1 - thr);
  float wider = from_top * ((few * 1.25f + 4.0f) * __builtin_amdgcn_rcpf(fmaxf((float)n, 0.5f)));
  const float want = few + extra;
  if (want < (float)half) {
    const float base = __builtin_amdgcn_logf(fmaxf((float)n, 0.5f));
    const float part = (__builtin_amdgcn_logf(want) - base) * __builtin_amdgcn_rcpf(__builtin_amdgcn_logf((float)half) - base);
    wider = fminf(wider, fmaxf(1.25f * from_top, from_top + part * (float)thr));
  }
  return (1 << 22) - (int32_t)fminf(wider, 4194304.0f);
}

// B[q] = kQ23Bias + P; sm: 0 for a positive channel sum, -1 for a negative one.  All threads of the
// team call this; the owners' masks are zero, and the list counter, and a barrier has passed since.
// Returns the mask of this thread's elements that flip (bit q).
template <int NE, int VE, bool WAVE, typename MaskT, typename Sh>
__device__ __forceinline__ MaskT k1_channel_stage(const uint32_t (&B)[NE], int32_t sm, uint32_t need, int N, Sh& sh,
                                                  uint32_t* owner) {
  static_assert(NE <= 8 * (int)sizeof(MaskT), "one mask bit per element");
  const int T = k1_team<WAVE>(), tid = k1_tid<WAVE>();
  // mask of the elements with u >= thr, bit q for element q
  auto at_least = [&](int32_t thr) {
    MaskT all = 0;
#pragma unroll
    for (int base = (NE - 1) / 32 * 32; base >= 0; base -= 32) {  // 32 elements to a mask word
      uint32_t m = 0;
      const uint32_t t = kQ23Bias + (uint32_t)(thr ^ sm);  // P >= thr resp. P <= ~thr
      if (sm == 0) {
#pragma unroll
        for (int q = (NE - base < 32 ? NE - base : 32) - 4; q >= 0; q -= 4) push_compares<true>(m, t, &B[base + q]);
      } else {
#pragma unroll
        for (int q = (NE - base < 32 ? NE - base : 32) - 4; q >= 0; q -= 4) push_compares<false>(m, t, &B[base + q]);
      }
      all |= (MaskT)m << (base & (8 * (int)sizeof(MaskT) - 1));
    }
    return all;
  };
  auto population = [](MaskT m) {
    return (uint32_t)__popc((uint32_t)m) + (sizeof(MaskT) > 4 ? (uint32_t)__popc((uint32_t)((uint64_t)m >> 32)) : 0u);
  };

  // ---- threshold search ----
  // Bounds: fewer than `need` elements have u >= hi (n_hi of them, mask m_hi); at least `need`
  // have u >= lo (n_lo, mask m_lo) once `found`.  Until then the distance from the top grows by a
  // quarter at least with every pass; afterwards the interval shrinks with every pass and every
  // fourth one halves it, so the search ends whatever the distribution.
  // Weights of few levels (requantised, ternary) pile thousands of equal u onto a few values, and a
  // threshold between two of them learns nothing.  A count that the lower bound has already says so:
  // the bounds then close in on elements, which skips the gap, or ends the search where one value is
  // left.  Passes on average (a closing-in counted as two), without and with: 4-bit grids 29 and 8,
  // ternary 31 and 7, 8-bit grids at 4 bits 10 and 4.5; continuous weights as before.  Times:
  // 16 x [2048, 512] binary16 in 4-bit levels at 2 bits 102 -> 47 us, ternary 111 -> 31 us;
  // [1024, 50176] binary32 in 4-bit levels 275 -> 118 us.
  // the step of u per element when the perturbations are spread evenly
  const int32_t step = __builtin_amdgcn_readfirstlane((int32_t)(8388608.0f * __builtin_amdgcn_rcpf((float)N)));
  // The list is ranked in steps of T / 4 entries by eight, each a round trip to LDS, so the search
  // goes on until the bounds hold a list of a few steps: with lists of up to 128 entries ranked by
  // a wave the slowest channels of a launch took 3 us longer than the others (1x1 layers of the
  // MobileNetV2 set 10.6 -> 8.6 us).  With 64 elements a thread a pass costs more than it saves
  // (six linear layers 119 -> 139 us).
  const uint32_t cap = NE > 32 ? kListCap : umin2(16u + (uint32_t)T / 8u, kListCap);
  int32_t lo = 1 + sm, hi = (1 << 22) + 1;
  uint32_t n_lo = 0, n_hi = 0, incl = 0;
  MaskT m_lo = 0, m_hi = 0;
  bool found = false;
  // elements wanted at or above the first threshold
  const uint32_t aim = umin2(need + (need >> 2) + 4u, need + kListCap / 4);
  int32_t thr = (1 << 22) - (int32_t)aim * step;
  for (int pass = 1;; ++pass) {
    thr = thr < lo ? lo : thr > hi - 1 ? hi - 1 : thr;
    const MaskT m = at_least(thr);
    const uint32_t run = wave_prefix_sum(population(m));
    const uint32_t n = k1_team_count<WAVE>(sh, (uint32_t)__builtin_amdgcn_readlane((int)run, kWave - 1), pass & 1);
    const bool gap = n == n_lo;  // no element lies between the threshold and the lower bound
    if (n >= need) {
      lo = thr; n_lo = n; m_lo = m; incl = run; found = true;
      if (n == need) return m;
    } else {
      if (thr == lo && !found) return m;  // fewer candidates of the wanted sign than flips: all flip
      hi = thr; n_hi = n; m_hi = m;
    }
    if (found) {
      if (__builtin_expect(n_lo - n_hi <= cap || hi - lo == 1, 1)) break;
      if (__builtin_expect(gap, 0)) {
        k1_close_in<NE, WAVE>(B, sm, lo, hi, sh);
        if (hi - lo == 1) break;
      }
      if ((pass & 3) == 0) {
        thr = lo + ((hi - lo) >> 1);
      } else {
        // interpolate between the bounds; once the lower one is close, from the other side of `need`
        float want = n_lo - need > cap - (cap >> 2) - 2u ? (float)need + 0.125f * (float)cap
                                                         : (float)need - 0.25f * (float)cap;
        if (want <= (float)n_hi + 0.5f) want = 0.5f * (float)(n_hi + need);
        float part = (want - (float)n_hi) * __builtin_amdgcn_rcpf((float)(n_lo - n_hi));
        if (n < need) {
          // The last threshold was too high: the elements crowd towards the lower bound, as they do
          // where outliers set the scale, and a straight line creeps up on them from one side.
          // A line through the logarithms of the counts meets them from the other side (six linear
          // layers, 49 M binary32 weights with outliers: 77.9 -> 65.0 us at 2 bits, 61.7 -> 59.7 at 4).
          const float base = __builtin_amdgcn_logf(fmaxf((float)n_hi, 0.5f));
          part = (__builtin_amdgcn_logf(want) - base) * __builtin_amdgcn_rcpf(__builtin_amdgcn_logf((float)n_lo) - base);
        }
        thr = __builtin_amdgcn_readfirstlane(hi - (int32_t)(part * (float)(hi - lo)));
        thr = thr <= lo ? lo + 1 : thr;
      }
    } else {
      thr = __builtin_amdgcn_readfirstlane(k1_lower_threshold(thr, n, need, 0.25f * (float)cap, N));
    }
  }
  // those with u >= hi flip; `want` of the `count` with lo <= u < hi
  const MaskT live = m_lo & (MaskT)~m_hi;
  const uint32_t count = n_lo - n_hi, want = need - n_hi;

  if (count <= (uint32_t)kListCap) {
    if (n_hi != 0) incl = wave_prefix_sum(population(live));
    uint32_t slot = incl - population(live);
    if constexpr (!WAVE) {  // the order within the list does not matter
      uint32_t base = 0;
      if ((tid & (kWave - 1)) == kWave - 1 && incl != 0) base = atomicAdd(&sh.list_count, incl);
      slot += (uint32_t)__builtin_amdgcn_readlane((int)base, kWave - 1);
    }
    if (tid < 8) sh.list[count + tid] = 0;
    uint64_t* put = sh.list + slot;
    const uint32_t me = ~((uint32_t)tid << 3);  // ~k1_owner_word(tid, q) = me - k1_owner_word(0, q)
#pragma unroll
    for (int j = NE / 4 - 1; j >= 0; --j) {
      uint32_t bits = (uint32_t)(live >> (4 * j)) << 28;  // the vector's four, in the top bits
      if (__ballot(bits != 0) == 0ull) continue;  // few vectors hold a member
#pragma unroll
      for (int e = 3; e >= 0; --e) {
        const int q = 4 * j + e;
        if (__builtin_add_overflow(bits, bits, &bits))
          *put++ = ((uint64_t)(B[q] ^ (uint32_t)sm) << 32) | (me - k1_owner_word<VE>(0, q));
      }
    }
    k1_sync<WAVE>();
    k1_rank<WAVE, VE>(sh.list, owner, count, want);
    k1_sync<WAVE>();
    MaskT mine = owner[tid];
    if (sizeof(MaskT) > 4) mine |= (MaskT)owner[T + tid] << (8 * sizeof(MaskT) - 32);
    return m_hi | mine;
  }

  // more than kListCap elements with the same u: the lowest indices flip.  The VE elements of a
  // vector are consecutive and vectors ascend with the thread, so inside round j an exclusive
  // prefix count over the threads ranks them; the rounds follow each other.
  MaskT flip = m_hi;
  uint32_t done = 0;
#pragma unroll 1
  for (int round = 0; round < NE / VE && done < want; ++round) {
    const uint32_t bits = (uint32_t)(live >> (VE * round)) & ((1u << VE) - 1u);
    const uint32_t mine = (uint32_t)__popc(bits);
    const uint32_t run = wave_prefix_sum(mine);
    uint32_t rank = done + run - mine, total = (uint32_t)__builtin_amdgcn_readlane((int)run, kWave - 1);
    if constexpr (!WAVE) {
      const int wid = tid / kWave, nw = (T + kWave - 1) / kWave;
      __syncthreads();
      if ((tid & (kWave - 1)) == 0) sh.cnt[0][wid] = total;
      __syncthreads();
      total = 0;
      for (int w = 0; w < nw; ++w) {
        const uint32_t c = sh.cnt[0][w];
        if (w < wid) rank += c;
        total += c;
      }
    }
#pragma unroll
    for (int e = 0; e < VE; ++e)
      if (bits & (1u << e)) {
        if (rank < want) flip |= (MaskT)1 << (VE * round + e);
        ++rank;
      }
    done += total;
  }
  return flip;
}

// ---------------------------------------------------------------------------
// The whole solve of one channel whose weights are in w: scale, codes.  Returns the scale.
// ---------------------------------------------------------------------------
// Sum over a wave of per-thread sums of NE perturbations each.
template <int NE>
__device__ __forceinline__ int64_t k1_wave_sum(int32_t v) {
  return NE < 32 ? wave_sum_rows(v) : wave_sum_dpp(v);  // a row of 16 lanes: 16 * NE * 2^22 < 2^31
}

template <int NE>
__device__ __forceinline__ float k1_absmax(const float (&w)[NE]) {
  float amax = 0.0f;
#pragma unroll
  for (int q = 0; q < NE; q += 2) amax = fmaxf(fmaxf(amax, fabsf(w[q])), fabsf(w[q + 1]));
  return amax;
}

// SQuant-E with the scale of a channel of absmax `amax` (the channel's, in each of its lanes); w is used up.
// Codes and B as from k1_round_all; esum: the sum of the thread's P.  Returns the scale.
template <int NE, bool WITH_P, bool HALF>
__device__ __forceinline__ float k1_quantize(float (&w)[NE], float amax, float qmaxf, float rcp_qmax,
                                             uint32_t (&code)[NE / 4], uint32_t (&B)[NE], int32_t& esum) {
  // The quotients go through the reciprocal of s, which is proven exact for an absmax within
  // [2^-60, 2^60]; a channel outside is first scaled by a power of two (see squant_k9.h).  There a
  // subnormal scale may be far below absmax / qmax, with many quotients beyond qmax, or be 0, with
  // every one infinite (2^-40 in its place makes them at least 2^19): the weights of such a channel
  // give way to their clamped quotients, which are then rounded with a scale of 1.
  float s = div_by_reciprocal(amax, qmaxf, rcp_qmax);
  float s2 = s;
  if (__builtin_expect(!(amax >= 0x1p-60f && amax <= 0x1p60f), 0)) {
    s = amax > 0.0f ? amax / qmaxf : 1.0f;
    const float f1 = amax >= 1.0f ? 0x1p-64f : amax > 0.0f ? 0x1p64f : 1.0f;
    const float a1 = amax * f1;
    const float f2 = a1 > 0x1p60f ? 0x1p-64f : a1 < 0x1p-60f && amax > 0.0f ? 0x1p64f : 1.0f;
    const float sp = s > 0.0f ? s * f1 * f2 : 0x1p-40f, rp = reciprocal(sp);
#pragma unroll
    for (int q = 0; q < NE; ++q)
      w[q] = __builtin_amdgcn_fmed3f(div_by_reciprocal(w[q] * f1 * f2, sp, rp), -qmaxf, qmaxf);
    s2 = 1.0f;
    amax = 0.0f;  // no quotient beyond qmax is left
  }
  const float rs = reciprocal(s2);
  esum = k1_round_all<NE, WITH_P, HALF>(w, s2, rs, qmaxf, div_by_reciprocal(amax, s2, rs), code, B);
  return s;
}

template <int MODE, int NE, int VE, bool WAVE, bool HALF, typename Sh>
__device__ __forceinline__ float k1_solve(float (&w)[NE], int N, float qmaxf, float rcp_qmax, Sh& sh, uint32_t* owner,
                                          uint32_t (&code)[NE / 4]) {
  constexpr bool kChannelStage = MODE == SQUANT_MODE_EKC || MODE == SQUANT_MODE_EC;
  typedef typename std::conditional<(NE > 32), uint64_t, uint32_t>::type MaskT;
  const int T = k1_team<WAVE>(), tid = k1_tid<WAVE>();
  if (kChannelStage) {  // before the first barrier
    owner[tid] = 0;
    if (NE > 32) owner[T + tid] = 0;
    if constexpr (!WAVE)
      if (tid == 0) sh.list_count = 0;
  }
  float amax = k1_absmax(w);
  if constexpr (WAVE) amax = wave_max_dpp(amax);
  else amax = block_max_dpp1(amax, sh.red_f);

  uint32_t B[NE];
  int32_t esum;
  const float s = k1_quantize<NE, kChannelStage, HALF>(w, amax, qmaxf, rcp_qmax, code, B, esum);

  if (kChannelStage) {
    int64_t ec = k1_wave_sum<NE>(esum);
    if constexpr (!WAVE) {
      const int nw = (T + kWave - 1) / kWave;
      if ((tid & (kWave - 1)) == 0) sh.red_i[tid / kWave] = ec;
      __syncthreads();
      ec = 0;
      for (int i = 0; i < nw; ++i) ec += sh.red_i[i];
      ec = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(ec >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)ec));
    }
    // scalar arithmetic throughout; |ec| <= 2^16 * 2^22
    const int32_t sm = (int32_t)(ec >> 63);
    const uint32_t kc = (uint32_t)(((uint64_t)((ec ^ sm) - sm) + (uint64_t)(kHalf - 1)) >> 23);  // flips_for(|ec|)
    if (kc > 0) {
      if (WAVE) k1_sync<true>();  // the owners' masks are reset
      const MaskT flip = k1_channel_stage<NE, VE, WAVE, MaskT>(B, sm, umin2(kc, (uint32_t)N), N, sh, owner);
      // one step against the channel sum for the marked elements: on the biased bytes a +-1
      // never carries into the neighbouring code
#pragma unroll
      for (int i = 0; i < NE / 4; ++i) {
        const uint32_t f4 = (uint32_t)(flip >> (4 * i)) & 15u;
        const uint32_t b = (f4 * 0x204081u) & 0x01010101u;  // bit e to byte e
        code[i] -= (b ^ (uint32_t)sm) - (uint32_t)sm;
      }
    }
  }
  return s;
}

// ---------------------------------------------------------------------------
// stores
// ---------------------------------------------------------------------------
// The row of output channel m in one format (squant_output_t): whole vectors by buffer stores
// whose range ends with the last of them, the VE - 1 or fewer elements after it one by one.
template <int NE, int VE, int FORMAT>
__device__ __forceinline__ void k1_emit(const uint32_t (&code)[NE / 4], void* out_base, int m, int N, float s,
                                        int tid, int T) {
  constexpr int kUnit = FORMAT == SQUANT_OUT_INT8 ? VE : FORMAT == SQUANT_OUT_INT4 ? VE / 2
                        : FORMAT == SQUANT_OUT_BF16 ? 2 * VE : 4 * VE;  // bytes of a vector
  const int full = N / VE;
  const size_t row_bytes = FORMAT == SQUANT_OUT_INT8 ? (size_t)N : FORMAT == SQUANT_OUT_INT4 ? (size_t)(N + 1) / 2
                           : FORMAT == SQUANT_OUT_BF16 ? 2 * (size_t)N : 4 * (size_t)N;
  uint8_t* out = static_cast<uint8_t*>(out_base) + (size_t)m * row_bytes;
  const rsrc_t row = make_rsrc(out, (uint32_t)full * kUnit);
  const uint32_t at = (uint32_t)tid * kUnit;
#pragma unroll
  for (int j = 0; j < NE / VE; ++j) {
    const uint32_t step = (uint32_t)(j * kUnit) * (uint32_t)T;
    const uint32_t c0 = code[j * VE / 4], c1 = code[j * VE / 4 + VE / 4 - 1];
    if (FORMAT == SQUANT_OUT_INT8) {
      if (VE == 4) buffer_store_u1_stream(c0 ^ 0x80808080u, row, at, step);
      else buffer_store_u2_stream(vu2{c0 ^ 0x80808080u, c1 ^ 0x80808080u}, row, at, step);
    } else if (FORMAT == SQUANT_OUT_INT4) {
      if (VE == 4) buffer_store_u16_stream((uint16_t)pack_nibbles4(c0), row, at, step);
      else buffer_store_u1_stream(pack_nibbles8(c0, c1), row, at, step);
    } else if (FORMAT == SQUANT_OUT_BF16) {
      const vf4 v = dequant4(c0, s);
      const uint32_t o0 = bf16_bits(v.x) | (bf16_bits(v.y) << 16), o1 = bf16_bits(v.z) | (bf16_bits(v.w) << 16);
      if (VE == 4) {
        buffer_store_u2_stream(vu2{o0, o1}, row, at, step);
      } else {
        const vf4 u = dequant4(c1, s);
        buffer_store_u4_stream(vu4{o0, o1, bf16_bits(u.x) | (bf16_bits(u.y) << 16),
                                   bf16_bits(u.z) | (bf16_bits(u.w) << 16)}, row, at, step);
      }
    } else if (VE == 4) {
      buffer_store_u4_stream(__builtin_bit_cast(vu4, dequant4(c0, s)), row, at, step);
    } else {
      const int lane = tid & (kWave - 1);
      const vu2 c = team_interleave<kWave>(c0, c1, lane);
      const uint32_t piece = (uint32_t)(tid - lane) * kUnit + (uint32_t)lane * 16u;
      buffer_store_u4_stream(__builtin_bit_cast(vu4, dequant4(c.x, s)), row, piece, step);
      buffer_store_u4_stream(__builtin_bit_cast(vu4, dequant4(c.y, s)), row, piece + 16u * kWave, step);
    }
  }
}

// The elements after the last whole vector, one by one.
template <int NE, int VE>
__device__ __forceinline__ void k1_emit_tail(int format, const uint32_t (&code)[NE / 4], void* out_base, int m, int N,
                                             float s, int tid, int T) {
  const int rem = N % VE, first = N - rem;
  const K1Place p = k1_place<VE>(first, T);
  uint32_t c[VE / 4] = {};
#pragma unroll
  for (int j = 0; j < NE / VE; ++j)
    if (j == p.j) {
#pragma unroll
      for (int i = 0; i < VE / 4; ++i) c[i] = code[j * VE / 4 + i];
    }
  if (tid != p.thread) return;
#pragma unroll 1
  for (int e = 0; e < rem; ++e) {
    const uint32_t byte = c[0] & 255u;
    const float v = ((float)byte - 128.0f) * s;
    c[0] = VE == 4 ? c[0] >> 8 : __builtin_amdgcn_alignbit(c[VE / 4 - 1], c[0], 8);
    if (VE == 8) c[VE / 4 - 1] >>= 8;
    const size_t at = (size_t)m * N + first + e;
    if (format == SQUANT_OUT_INT8) static_cast<uint8_t*>(out_base)[at] = (uint8_t)(byte ^ 0x80u);
    else if (format == SQUANT_OUT_BF16) static_cast<uint16_t*>(out_base)[at] = (uint16_t)bf16_bits(v);
    else if (format == SQUANT_OUT_F32) static_cast<float*>(out_base)[at] = v;
    else if ((e & 1) == 0)  // with the next element's nibble: past the end its code is 0
      static_cast<uint8_t*>(out_base)[(size_t)m * ((N + 1) / 2) + (first + e) / 2] =
          (uint8_t)((byte & 15u) | (c[0] << 4));
  }
}

template <int NE, int VE, bool TAIL>
__device__ __forceinline__ void k1_emit_as(int format, const uint32_t (&code)[NE / 4], void* out_base, int m, int N,
                                           float s, int tid, int T) {
  // the format is chosen once, outside the loop over the vectors
  if (format == SQUANT_OUT_INT8) k1_emit<NE, VE, SQUANT_OUT_INT8>(code, out_base, m, N, s, tid, T);
  else if (format == SQUANT_OUT_INT4) k1_emit<NE, VE, SQUANT_OUT_INT4>(code, out_base, m, N, s, tid, T);
  else if (format == SQUANT_OUT_BF16) k1_emit<NE, VE, SQUANT_OUT_BF16>(code, out_base, m, N, s, tid, T);
  else k1_emit<NE, VE, SQUANT_OUT_F32>(code, out_base, m, N, s, tid, T);
  if (TAIL && N % VE != 0) k1_emit_tail<NE, VE>(format, code, out_base, m, N, s, tid, T);
}

// Elements per vector with NV four-element vectors per thread.
template <int NV, bool HALF>
constexpr int k1_ve() { return HALF && NV % 2 == 0 ? 8 : 4; }

template <int MODE, int NV, int VE, bool HALF, bool TAIL>
__device__ __forceinline__ void k1_channel(const LaunchArgs& a, const TensorDesc& d, int m, unsigned char* smem,
                                           K1Shared& sh) {
  constexpr int NE = 4 * NV;
  const int T = blockDim.x, tid = threadIdx.x, N = d.N;
  uint32_t raw[HALF ? NE / 2 : NE], tail, code[NE / 4];
  k1_load<NE, VE, HALF, TAIL>(static_cast<const uint8_t*>(d.w) + (size_t)m * N * (HALF ? 2 : 4), N, tid, T, raw, tail);
  float w[NE];
  k1_widen<NE, VE, HALF, TAIL>(raw, tail, a.wtype == SQUANT_W_BF16, N, tid, T, w);
  const float s = k1_solve<MODE, NE, VE, false, HALF>(w, N, (float)a.qmax, a.rcp_qmax, sh, reinterpret_cast<uint32_t*>(smem), code);
  if (tid == 0) d.scales[m] = s;
  k1_emit_as<NE, VE, TAIL>(a.out_format, code, d.out, m, N, s, tid, T);
}

// One kernel per vector count serves every workgroup size.  Up to seven vectors per thread fit
// the 64 VGPRs of eight waves per SIMD, eight the 72 of seven, ten to sixteen the 128 of
// four.  The steps matter because
// whole workgroups must fit: at 64 VGPRs a compute unit has 32 wave slots, so two workgroups of
// 1024 threads or eight of 256 run side by side; at 80 it has 24.
template <int MODE, int NV, bool HALF, bool TAIL>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(NV <= 7 ? 8 : NV <= 8 ? 7 : 4)))
    squant_channel_k1(LaunchArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];  // the owners' masks
  __shared__ K1Shared sh;
  int m;
  const TensorDesc d = locate(a, blockIdx.x, m);
  k1_channel<MODE, NV, k1_ve<NV, HALF>(), HALF, TAIL>(a, d, m, smem, sh);
}

}  // namespace squant
