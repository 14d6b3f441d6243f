// Global-memory access helpers and the output stage shared by the SQuant kernels that keep
// a channel's codes in LDS as biased bytes (code + 128, four to a dword).
#pragma once

#include "squant_common.h"

namespace squant {

typedef float vf3 __attribute__((ext_vector_type(3)));
typedef float vf4 __attribute__((ext_vector_type(4)));
typedef uint32_t vu4 __attribute__((ext_vector_type(4)));
typedef uint32_t vu2 __attribute__((ext_vector_type(2)));
typedef uint32_t vu3 __attribute__((ext_vector_type(3)));

// 16-byte load / store through the global (not flat) address space
__device__ __forceinline__ vf4 load_global_f4(const float* p) {
#if defined(__HIP_DEVICE_COMPILE__)
  return *reinterpret_cast<const __attribute__((address_space(1))) vf4*>(reinterpret_cast<uintptr_t>(p));
#else
  return *reinterpret_cast<const vf4*>(p);
#endif
}
__device__ __forceinline__ vf3 load_global_f3(const float* p) {
#if defined(__HIP_DEVICE_COMPILE__)
  // plain loads: the three 12-byte loads of a kernel share cache lines, and with the
  // non-temporal hint a line is gone by the second touch (measured 6-20 % slower)
  return *reinterpret_cast<const __attribute__((address_space(1))) vf3*>(reinterpret_cast<uintptr_t>(p));
#else
  return *reinterpret_cast<const vf3*>(p);
#endif
}
__device__ __forceinline__ void store_global_u4(void* p, vu4 v) {
#if defined(__HIP_DEVICE_COMPILE__)
  // codes are written once: non-temporal stores (measured 1 % faster)
  __builtin_nontemporal_store(
      v, reinterpret_cast<__attribute__((address_space(1))) vu4*>(reinterpret_cast<uintptr_t>(p)));
#else
  *reinterpret_cast<vu4*>(p) = v;
#endif
}
__device__ __forceinline__ void store_global_u1(void* p, uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_nontemporal_store(
      v, reinterpret_cast<__attribute__((address_space(1))) uint32_t*>(reinterpret_cast<uintptr_t>(p)));
#else
  *reinterpret_cast<uint32_t*>(p) = v;
#endif
}

__device__ __forceinline__ void store_global_f4(void* p, vf4 v) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_nontemporal_store(
      v, reinterpret_cast<__attribute__((address_space(1))) vf4*>(reinterpret_cast<uintptr_t>(p)));
#else
  *reinterpret_cast<vf4*>(p) = v;
#endif
}
__device__ __forceinline__ void store_global_u16(void* p, uint16_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  *reinterpret_cast<__attribute__((address_space(1))) uint16_t*>(reinterpret_cast<uintptr_t>(p)) = v;
#else
  *reinterpret_cast<uint16_t*>(p) = v;
#endif
}

// ---- buffer access: a descriptor of `bytes` bytes at p (uniform over the wave) ----
// The hardware checks every dword (every unit of a narrower access) against the range: one that
// does not lie inside as a whole reads as 0 and is not written, so rows of any length need no
// bounds checks; any byte alignment is taken.  Offsets: per lane, and uniform.
#if defined(__HIP_DEVICE_COMPILE__)
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
constexpr int kNonTemporal = 2;  // the non-temporal bit of the cache policy: rows are touched once
__device__ __forceinline__ vu4 buffer_load_u4_stream(rsrc_t r, uint32_t lane_off, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)off, kNonTemporal);
}
__device__ __forceinline__ uint32_t buffer_load_u1(rsrc_t r, uint32_t lane_off, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, (int)lane_off, (int)off, 0);
}
__device__ __forceinline__ vu2 buffer_load_u2(rsrc_t r, uint32_t lane_off, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane_off, (int)off, 0);
}
__device__ __forceinline__ vu3 buffer_load_u3(rsrc_t r, uint32_t lane_off, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b96(r, (int)lane_off, (int)off, 0);
}
__device__ __forceinline__ vu4 buffer_load_u4(rsrc_t r, uint32_t lane_off, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)off, 0);
}
__device__ __forceinline__ uint32_t buffer_load_u16(rsrc_t r, uint32_t lane_off, uint32_t off) {
  return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)lane_off, (int)off, 0);
}
__device__ __forceinline__ vu2 buffer_load_u2_stream(rsrc_t r, uint32_t lane_off, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane_off, (int)off, kNonTemporal);
}
// The uniform offset joins the lane's here and not the instruction's scalar operand: a 16-byte
// store with one is still reading its data when the next instruction may write those registers,
// and the compiler only keeps the two apart where there is none (first components of some lanes
// came out as the next vector's).
__device__ __forceinline__ void buffer_store_u4_stream(vu4 v, rsrc_t r, uint32_t lane_off, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)(lane_off + off), 0, kNonTemporal);
}
__device__ __forceinline__ void buffer_store_u2_stream(vu2 v, rsrc_t r, uint32_t lane_off, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b64(v, r, (int)lane_off, (int)off, kNonTemporal);
}
__device__ __forceinline__ void buffer_store_u1_stream(uint32_t v, rsrc_t r, uint32_t lane_off, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b32(v, r, (int)lane_off, (int)off, kNonTemporal);
}
__device__ __forceinline__ void buffer_store_u16_stream(uint16_t v, rsrc_t r, uint32_t lane_off, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b16(v, r, (int)lane_off, (int)off, kNonTemporal);
}
__device__ __forceinline__ void buffer_store_u8(uint32_t v, rsrc_t r, uint32_t lane_off) {
  __builtin_amdgcn_raw_buffer_store_b8((uint8_t)v, r, (int)lane_off, 0, 0);
}
// Says that no load is under way any more.  After weights that are widened in one of two branches the compiler is not sure,
// and a register of theirs that is written again later, behind the scale's store, makes the wave wait for that store to
// reach memory (SQuant-E alone, binary16 to int8: 100 M weights in channels of 100 kernels 73.5 us, 62 so).
__device__ __forceinline__ void weights_are_here() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0)
#else  // the host pass only parses the kernels
struct rsrc_t {};
__device__ void weights_are_here();
__device__ void buffer_store_u8(uint32_t, rsrc_t, uint32_t);
__device__ rsrc_t make_rsrc(const void*, uint32_t);
__device__ uint32_t buffer_load_u1(rsrc_t, uint32_t, uint32_t);
__device__ vu2 buffer_load_u2(rsrc_t, uint32_t, uint32_t);
__device__ vu3 buffer_load_u3(rsrc_t, uint32_t, uint32_t);
__device__ vu4 buffer_load_u4(rsrc_t, uint32_t, uint32_t);
__device__ uint32_t buffer_load_u16(rsrc_t, uint32_t, uint32_t);
__device__ vu4 buffer_load_u4_stream(rsrc_t, uint32_t, uint32_t);
__device__ vu2 buffer_load_u2_stream(rsrc_t, uint32_t, uint32_t);
__device__ void buffer_store_u4_stream(vu4, rsrc_t, uint32_t, uint32_t);
__device__ void buffer_store_u2_stream(vu2, rsrc_t, uint32_t, uint32_t);
__device__ void buffer_store_u1_stream(uint32_t, rsrc_t, uint32_t, uint32_t);
__device__ void buffer_store_u16_stream(uint16_t, rsrc_t, uint32_t, uint32_t);
#endif

// ---- binary16 / bfloat16 weights: widened exactly to binary32 on load ----
__device__ __forceinline__ float widen_f16(uint32_t bits) {  // low 16 bits
  return (float)__builtin_bit_cast(_Float16, (uint16_t)bits);
}
__device__ __forceinline__ float widen_bf16(uint32_t bits) {  // low 16 bits
  return __uint_as_float(bits << 16);
}
// Both halves of a dword, low half first.
__device__ __forceinline__ void widen_pair(uint32_t d, bool bf16, float& lo, float& hi) {
  if (bf16) {
    lo = __uint_as_float(d << 16);
    hi = __uint_as_float(d & 0xFFFF0000u);
  } else {
    lo = widen_f16(d);
    hi = widen_f16(d >> 16);
  }
}
__device__ __forceinline__ uint32_t load_global_u1(const uint32_t* p) {
#if defined(__HIP_DEVICE_COMPILE__)
  return *reinterpret_cast<const __attribute__((address_space(1))) uint32_t*>(reinterpret_cast<uintptr_t>(p));
#else
  return *p;
#endif
}
// Element i of a weight tensor of the given squant_wtype_t.
__device__ __forceinline__ float load_weight(const void* w, size_t i, int wtype) {
  if (wtype == SQUANT_W_F32) return static_cast<const float*>(w)[i];
  const uint32_t h = static_cast<const uint16_t*>(w)[i];
  return wtype == SQUANT_W_BF16 ? widen_bf16(h) : widen_f16(h);
}

// Low nibbles of the bytes of lo and hi, gathered into 32 bits (byte 0 of lo in bits 0-3).  The
// +128 bias of a code byte does not reach its low nibble, which is the code's 4-bit
// two's complement.  Even and odd bytes apart, one shift and one select of bits: four instructions for eight codes, where
// masking and folding each dword took eleven (32 x [512, 512, 3, 3] to 4 bit 56.6 -> 55.6 us, [512, 255, 3, 3] binary16 28.4 -> 27.5).
__device__ __forceinline__ uint32_t pack_nibbles8(uint32_t lo, uint32_t hi) {
  const uint32_t even = __builtin_amdgcn_perm(hi, lo, 0x06040200u), odd = __builtin_amdgcn_perm(hi, lo, 0x07050301u);
  return (even & 0x0F0F0F0Fu) | ((odd << 4) & 0xF0F0F0F0u);
}
// The same of one dword, in the low 16 bits.
__device__ __forceinline__ uint32_t pack_nibbles4(uint32_t c) { return pack_nibbles8(c, 0u); }

// The four biased code bytes of c as dequantised weights code * s (Algorithm 1 returns
// C * s; one binary32 multiply per element).
__device__ __forceinline__ vf4 dequant4(uint32_t c, float s) {
  vf4 v;
  v.x = ((float)(c & 0xFFu) - 128.0f) * s;
  v.y = ((float)((c >> 8) & 0xFFu) - 128.0f) * s;
  v.z = ((float)((c >> 16) & 0xFFu) - 128.0f) * s;
  v.w = ((float)(c >> 24) - 128.0f) * s;
  return v;
}

// binary32 to bfloat16 bits, round to nearest, ties to even (finite inputs).
__device__ __forceinline__ uint32_t bf16_bits(float v) {
  const uint32_t b = __float_as_uint(v);
  return (b + 0x7FFFu + ((b >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ void store_global_u2(void* p, vu2 v) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_nontemporal_store(
      v, reinterpret_cast<__attribute__((address_space(1))) vu2*>(reinterpret_cast<uintptr_t>(p)));
#else
  *reinterpret_cast<vu2*>(p) = v;
#endif
}

// Eight elements a lane go to binary32 as two stores of 16 bytes.  With its own eight elements each store of a lane
// would leave a gap of 16 bytes to its neighbour's, and no line would be written as a whole.  So the TEAM lanes of a row
// exchange their dwords of codes: dword p of the team (two a lane, in order) goes with the first store of lane p,
// p < TEAM, or the second of lane p - TEAM, and each store of the team is consecutive.  The lane's dwords from its c0, c1.
// bfloat16 to binary32, each lane storing its own, 64 consecutive bytes a quad, and so: 16 x [1024, 4096] 132.7, 90.5 and
// 74.1 us (5.4 TB/s), 16 x [1024, 12268] 440, 384 and 235, 48 x [1024, 320] 29.2, 23.4 and 20.6.
template <int TEAM>
__device__ __forceinline__ vu2 team_interleave(uint32_t c0, uint32_t c1, int lane) {
  const int from = 4 * ((lane & (kWave - TEAM)) + ((lane & (TEAM - 1)) >> 1));
  const uint32_t a0 = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)c0), a1 = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)c1);
  const uint32_t b0 = (uint32_t)__builtin_amdgcn_ds_bpermute(from + 2 * TEAM, (int)c0);
  const uint32_t b1 = (uint32_t)__builtin_amdgcn_ds_bpermute(from + 2 * TEAM, (int)c1);
  return lane & 1 ? vu2{a1, b1} : vu2{a0, b0};
}

// The K codes (biased bytes in d0, d1, d2) of a thread's kernels tid, tid + G, ... of a channel into the channel's
// bytes in LDS.  A store that is not aligned to its size costs the LDS dearly (a wave's 8 bytes at 9 n and one more byte 43 ns,
// nine single bytes 17, aligned dwords 2 each), so where the four lanes of a quad hold four consecutive kernels from a
// multiple of four on, whose 4 K bytes are K dwords, each lane puts together the dwords that begin in its
// kernel: its own bytes and, behind them, the first of the next lane's.  owned, bit q: the thread has kernel q.
// Whole quads call this.  A row's last dword may take up to three bytes behind it, from the next lane's kernel:
// 128, as a kernel without weights has.
// ALL: a thread has all of its kernels or none.
template <int K, bool ALL, int KPT, typename Kernel>
__device__ __forceinline__ void store_kernel_codes(uint8_t* code8, int tid, int G, uint32_t owned, const Kernel (&kk)[KPT],
                                                   bool quads = true) {
  static_assert(K == 2 || K == 3 || K == 4 || K == 5 || K == 7 || K == 9, "kernel sizes with a pattern of dwords");
  if (!quads || (K != 4 && KPT > 1 && (G & 3) != 0)) {
#pragma unroll
    for (int q = 0; q < KPT; ++q) {
      if (!((owned >> q) & 1u)) continue;
      uint8_t* dst = code8 + K * (tid + q * G);
      if (K > 4) {
        const uint64_t lo = (uint64_t)kk[q].d0 | ((uint64_t)kk[q].d1 << 32);
        __builtin_memcpy(dst, &lo, K < 8 ? 4 : 8);
      }
      const uint32_t rest = K == 9 ? kk[q].d2 : K > 4 ? kk[q].d1 : kk[q].d0;
#pragma unroll
      for (int i = 0; i < K % 4; ++i) dst[K / 4 * 4 + i] = (uint8_t)(rest >> (8 * i));
    }
    return;
  }
  const uint32_t i = (uint32_t)tid & 3u, before = (4u - i) & 3u;  // the lane within its quad
  // where the lane's first whole dword begins: `before` bytes into its kernel (9, 5), or i bytes (7, 3)
  const uint32_t first = K == 9 ? 2 * i + (i > 0 ? 1 : 0) : K == 7 ? 2 * i : K == 5 ? i + (i > 0 ? 1 : 0) : K == 2 ? i >> 1 : i;
  uint8_t* base = K == 4 ? code8 + 4 * tid : code8 + K * (tid & ~3) + 4 * first;
  uint32_t w0[KPT], w1[KPT], last[KPT];
#pragma unroll
  for (int q = 0; q < KPT; ++q) {
    const uint32_t d0 = kk[q].d0, d1 = kk[q].d1;
    const uint32_t next = (uint32_t)__builtin_amdgcn_mov_dpp((int)d0, 0xF9, 0xf, 0xf, true);  // quad_perm [1, 2, 3, 3]
    w1[q] = last[q] = 0;
    if (K == 9) {
      last[q] = __builtin_amdgcn_perm(next, kk[q].d2, 0x06050400u);
      w0[q] = __builtin_amdgcn_alignbyte(d1, d0, before);
      w1[q] = __builtin_amdgcn_alignbyte(last[q], d1, before);
    } else if (K == 7) {
      const uint32_t end = __builtin_amdgcn_perm(next, d1, 0x04020100u);
      w0[q] = __builtin_amdgcn_alignbyte(end, d0, i);
      w1[q] = __builtin_amdgcn_alignbyte(next >> 8, end, i);
    } else if (K == 5) {
      last[q] = __builtin_amdgcn_perm(next, d1, 0x06050400u);
      w0[q] = __builtin_amdgcn_alignbyte(last[q], d0, before);
    } else if (K == 4) {
      w0[q] = d0;
    } else if (K == 3) {
      w0[q] = __builtin_amdgcn_alignbyte(next >> 8, __builtin_amdgcn_perm(next, d0, 0x04020100u), i);
    } else {
      w0[q] = __builtin_amdgcn_perm(next, d0, 0x05040100u);
    }
  }
  auto at = [&](int q) { return reinterpret_cast<uint32_t*>(base + q * (K * G)); };
  auto put = [&](int q) {
    at(q)[0] = w0[q];
    if (K == 9) at(q)[1] = w1[q];
  };
  const bool begins = (K != 3 || i < 3) && (K != 2 || (i & 1u) == 0);  // a dword begins in the lane's kernel
  if (ALL) {
    if (owned != 0 && begins) {
#pragma unroll
      for (int q = 0; q < KPT; ++q) put(q);
    }
  } else {
#pragma unroll
    for (int q = 0; q < KPT; ++q)
      if (((owned >> q) & 1u) && begins) put(q);
  }
  const bool more = K == 7 ? i < 3 : (K == 9 || K == 5) && i == 0;
  if (owned != 0 && more) {
#pragma unroll
    for (int q = 0; q < KPT; ++q)
      if (ALL || ((owned >> q) & 1u)) at(q)[K == 9 ? 2 : 1] = K == 7 ? w1[q] : last[q];
  }
}

// Writes output channel m of a tensor from its biased codes in LDS (nvec dwords, so the
// channel has 4 * nvec elements) in the requested format (squant_output_t).  Called by the
// whole workgroup after a barrier; 16-byte stores where the channel's row is aligned.
__device__ __forceinline__ void emit_channel(const uint32_t* code32, int nvec, void* out_base,
                                             int m, float s, int format, int tid, int T) {
  const size_t L = 4 * (size_t)nvec;
  const vu4* src4 = reinterpret_cast<const vu4*>(code32);
  if (format == SQUANT_OUT_INT8) {
    uint8_t* out = static_cast<uint8_t*>(out_base) + (size_t)m * L;
    if ((nvec & 3) == 0 && (reinterpret_cast<uintptr_t>(out) & 15u) == 0) {
      for (int j = tid; j < (nvec >> 2); j += T) store_global_u4(out + 16 * j, src4[j] ^ 0x80808080u);
    } else {
      for (int j = tid; j < nvec; j += T) store_global_u1(out + 4 * j, code32[j] ^ 0x80808080u);
    }
  } else if (format == SQUANT_OUT_INT4) {
    uint8_t* out = static_cast<uint8_t*>(out_base) + (size_t)m * (L / 2);
    if ((nvec & 7) == 0 && (reinterpret_cast<uintptr_t>(out) & 15u) == 0) {
      for (int j = tid; j < (nvec >> 3); j += T) {
        const vu4 a = src4[2 * j], b = src4[2 * j + 1];
        vu4 o;
        o.x = pack_nibbles8(a.x, a.y);
        o.y = pack_nibbles8(a.z, a.w);
        o.z = pack_nibbles8(b.x, b.y);
        o.w = pack_nibbles8(b.z, b.w);
        store_global_u4(out + 16 * j, o);
      }
    } else {
      for (int j = tid; j < nvec; j += T) store_global_u16(out + 2 * j, (uint16_t)pack_nibbles4(code32[j]));
    }
  } else if (format == SQUANT_OUT_BF16) {
    uint16_t* out = static_cast<uint16_t*>(out_base) + (size_t)m * L;
    if ((reinterpret_cast<uintptr_t>(out) & 7u) == 0) {
      for (int j = tid; j < nvec; j += T) {
        const vf4 v = dequant4(code32[j], s);
        vu2 o;
        o.x = bf16_bits(v.x) | (bf16_bits(v.y) << 16);
        o.y = bf16_bits(v.z) | (bf16_bits(v.w) << 16);
        store_global_u2(out + 4 * j, o);
      }
    } else {
      for (int j = tid; j < nvec; j += T) {
        const vf4 v = dequant4(code32[j], s);
        out[4 * j] = (uint16_t)bf16_bits(v.x); out[4 * j + 1] = (uint16_t)bf16_bits(v.y);
        out[4 * j + 2] = (uint16_t)bf16_bits(v.z); out[4 * j + 3] = (uint16_t)bf16_bits(v.w);
      }
    }
  } else {  // SQUANT_OUT_F32
    float* out = static_cast<float*>(out_base) + (size_t)m * L;
    if ((reinterpret_cast<uintptr_t>(out) & 15u) == 0) {
      for (int j = tid; j < nvec; j += T) store_global_f4(out + 4 * j, dequant4(code32[j], s));
    } else {
      for (int j = tid; j < nvec; j += T) {
        const vf4 v = dequant4(code32[j], s);
        out[4 * j] = v.x; out[4 * j + 1] = v.y; out[4 * j + 2] = v.z; out[4 * j + 3] = v.w;
      }
    }
  }
}

// The same for a channel of any length L whose row starts anywhere: 16 (8 for bfloat16) bytes a
// store, whatever their alignment; the range of the row's descriptor cuts the last one at a whole
// dword, and the up to three bytes after it go one by one.  The codes' area is a multiple of 32
// bytes and holds 128 (code 0) in the byte behind an odd channel.
__device__ __forceinline__ void emit_row(const uint8_t* code8, int L, void* out_base, int m, float s, int format,
                                         int tid, int T) {
  const uint32_t* code32 = reinterpret_cast<const uint32_t*>(code8);
  const vu4* src4 = reinterpret_cast<const vu4*>(code8);
  if (format == SQUANT_OUT_INT8) {
    uint8_t* out = static_cast<uint8_t*>(out_base) + (size_t)m * L;
    const int whole = L & ~3;
    const rsrc_t row = make_rsrc(out, (uint32_t)whole);
    for (int j = tid; 16 * j < whole; j += T) buffer_store_u4_stream(src4[j] ^ 0x80808080u, row, 16u * j, 0);
    if (tid < L - whole) out[whole + tid] = code8[whole + tid] ^ 0x80u;
  } else if (format == SQUANT_OUT_INT4) {
    const int bytes = (L + 1) >> 1, whole = bytes & ~3;
    uint8_t* out = static_cast<uint8_t*>(out_base) + (size_t)m * bytes;
    const rsrc_t row = make_rsrc(out, (uint32_t)whole);
    for (int j = tid; 16 * j < whole; j += T) {
      const vu4 a = src4[2 * j], b = src4[2 * j + 1];
      const vu4 o = {pack_nibbles8(a.x, a.y), pack_nibbles8(a.z, a.w), pack_nibbles8(b.x, b.y), pack_nibbles8(b.z, b.w)};
      buffer_store_u4_stream(o, row, 16u * j, 0);
    }
    if (tid < bytes - whole) {
      const int e = 2 * (whole + tid);
      out[whole + tid] = (uint8_t)((code8[e] & 15u) | (code8[e + 1] << 4));
    }
  } else if (format == SQUANT_OUT_BF16) {
    uint16_t* out = static_cast<uint16_t*>(out_base) + (size_t)m * L;
    const rsrc_t row = make_rsrc(out, 2u * (uint32_t)(L & ~1));
    for (int j = tid; 4 * j < L; j += T) {
      const vf4 v = dequant4(code32[j], s);
      const vu2 o = {bf16_bits(v.x) | (bf16_bits(v.y) << 16), bf16_bits(v.z) | (bf16_bits(v.w) << 16)};
      buffer_store_u2_stream(o, row, 8u * j, 0);
    }
    if ((L & 1) && tid == 0) out[L - 1] = (uint16_t)bf16_bits(((float)code8[L - 1] - 128.0f) * s);
  } else {  // SQUANT_OUT_F32
    float* out = static_cast<float*>(out_base) + (size_t)m * L;
    const rsrc_t row = make_rsrc(out, 4u * (uint32_t)L);
    for (int j = tid; 4 * j < L; j += T)
      buffer_store_u4_stream(__builtin_bit_cast(vu4, dequant4(code32[j], s)), row, 16u * j, 0);
  }
}

// The same output stage for the generic kernel, whose LDS holds plain int8 codes and whose
// channel length L is arbitrary.  A packed row has (L + 1) / 2 bytes; the unused high
// nibble of an odd row's last byte is 0.
__device__ __forceinline__ void emit_channel_bytes(const int8_t* code, int L, void* out_base, int m,
                                                   float s, int format, int tid, int T) {
  if (format == SQUANT_OUT_INT8) {
    int8_t* out = static_cast<int8_t*>(out_base) + (size_t)m * L;
    if ((reinterpret_cast<uintptr_t>(out) & 3u) == 0) {
      const int L4 = L >> 2;
      const uint32_t* src = reinterpret_cast<const uint32_t*>(code);
      uint32_t* dst = reinterpret_cast<uint32_t*>(out);
      for (int j = tid; j < L4; j += T) dst[j] = src[j];
      for (int j = (L4 << 2) + tid; j < L; j += T) out[j] = code[j];
    } else {
      for (int j = tid; j < L; j += T) out[j] = code[j];
    }
  } else if (format == SQUANT_OUT_INT4) {
    const int row = (L + 1) >> 1;
    uint8_t* out = static_cast<uint8_t*>(out_base) + (size_t)m * row;
    for (int j = tid; j < row; j += T) {
      const uint32_t lo = (uint32_t)code[2 * j] & 0xFu;
      const uint32_t hi = (2 * j + 1 < L) ? ((uint32_t)code[2 * j + 1] & 0xFu) : 0u;
      out[j] = (uint8_t)(lo | (hi << 4));
    }
  } else if (format == SQUANT_OUT_BF16) {
    uint16_t* out = static_cast<uint16_t*>(out_base) + (size_t)m * L;
    for (int j = tid; j < L; j += T) out[j] = (uint16_t)bf16_bits((float)code[j] * s);
  } else {  // SQUANT_OUT_F32
    float* out = static_cast<float*>(out_base) + (size_t)m * L;
    for (int j = tid; j < L; j += T) out[j] = (float)code[j] * s;
  }
}

}  // namespace squant
