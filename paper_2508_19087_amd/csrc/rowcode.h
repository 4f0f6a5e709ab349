// rowcode.h - one lane's share of a row of activation codes or fp16
// activations, turned into bipolar words and bit-planes on gfx950 (APT-LLM,
// arXiv 2508.19087: Sec. III-A conversion and the bipolar form of a linear
// quantizer; Sec. IV-A decomposition into bit-planes).  Shared by the packer
// (pack.hip), which stores the plane words in the packed layout, and by the
// XOR route's fused decode form (gemm_xor.h), which stores them in LDS.
//
// A lane takes 16 consecutive elements of a row.  CodeRow reads signed b-bit
// codes (one byte each) and HalfRow fp16 values, which it quantizes with the
// row's bipolar scale (see Quantizer).  words() gives the 16 bipolar words u,
// one per byte; transpose8x8 leaves plane i of 8 elements in byte i; and
// plane_word gives, for a pair of planes, the 32-bit plane word that this lane
// and its neighbour (lanes 2m, 2m + 1, 32 consecutive elements) hold between
// them: the even lane gets plane i, the odd lane plane i + 1.
#pragma once

#include "apt_internal.h"

namespace apt {
namespace rowcode {

constexpr int kLaneElems = 16;
constexpr uint32_t kRawBufferFlags = 0x00020000u;

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t any_u32x4_t __attribute__((ext_vector_type(4), aligned(1)));  // at any byte

// Largest value and sum over the wave's 64 lanes, uniform: four DPP steps give
// every 16-lane row its result, four lane reads the wave's.
template <class Op>
__device__ __forceinline__ uint32_t wave_fold(uint32_t v, Op op) {
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));   // lane ^ 1
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));   // lane ^ 2
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));  // the row's half mirrored
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));  // the row mirrored
  const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
  const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
  return op(op(a, b), op(c, d));
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  return wave_fold(v, [](uint32_t x, uint32_t y) { return max(x, y); });
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
  return wave_fold(v, [](uint32_t x, uint32_t y) { return x + y; });
}

// The same conversions with the bit width in a register (the few-token GEMM
// is not instantiated per activation width).
__device__ __forceinline__ void code_words(const uint32_t d[4], int b, uint32_t u[4]) {
  const uint32_t field = ((1u << b) - 1u) * 0x01010101u;
  const uint32_t flip = (1u << (b - 1)) * 0x01010101u;
#pragma unroll
  for (int t = 0; t < 4; ++t) u[t] = (d[t] & field) ^ flip;
}

// A row's quantizer: its scale from the largest magnitude's fp16 bits, and the
// words of 16 of its values.
//
// Short form (a normal scale): with h = x / (2 s), the word is u = floor(h) +
// 2^(b-1), and no clamp is needed (|h| <= (2^b - 1)/2 (1 + 2^-11)).  One fma per
// value gives f = x / (2 s) + 2^(b-1) + 128 rounded to multiples of 2^-16, whose
// bits 16..22 are u (b = 8: + 256, multiples of 2^-15, bits 15..22): the reciprocal's rounding moves h by at most
// 2^-18, so an integer h rounds back to itself, and h is never close below an
// integer, since x and s have 11-bit significands: for |h| >= 1/2 a non-integer
// h is at least 2^-12 away from every integer.  Negative
// values above -s, where h comes arbitrarily close below 0, are first replaced
// by -s (same word: h in [-1/2, 0)), as signed 16-bit integers, and -0 by +0.
// The long form takes the exact quotient: h0 = fma(x, r / 2, 0), e = fma(-h0, 2 s,
// x), h = fma(e, r / 2, h0) with r = RN(1 / s), the quotient correction of
// Markstein's division with a correctly rounded reciprocal, floor and clamp.
// Both give the same words for every finite input (checked over all of them on
// the CPU); a row with an infinity or a NaN takes the long form, whose words stay
// in range.
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

// Largest and smallest of a lane's fp16 values (two dwords per packed
// three-operand instruction), and from them the largest magnitude's bits.
struct HalfExtremes {
  half2_t hi = {(_Float16)0.0f, (_Float16)0.0f}, lo = {(_Float16)0.0f, (_Float16)0.0f};
  __device__ __forceinline__ void fold(const uint32_t d[8]) {
#pragma unroll
    for (int t = 0; t < 8; t += 2) {
      const half2_t x = __builtin_bit_cast(half2_t, d[t]), y = __builtin_bit_cast(half2_t, d[t + 1]);
      hi = __builtin_elementwise_maximum(__builtin_elementwise_maximum(hi, x), y);
      lo = __builtin_elementwise_minimum(__builtin_elementwise_minimum(lo, x), y);
    }
  }
  __device__ __forceinline__ uint32_t largest_magnitude() const {
    const uint32_t h = __builtin_bit_cast(uint32_t, hi) & 0x7FFF7FFFu, l = __builtin_bit_cast(uint32_t, lo) & 0x7FFF7FFFu;
    return max(max(h & 0xFFFFu, h >> 16), max(l & 0xFFFFu, l >> 16));
  }
};

struct Quantizer {
  uint16_t scale;
  int b;
  bool quick;
  float rh, s2, base;
  uint32_t least;  // -s in both halves of a dword

  __device__ static __forceinline__ float base_of(int b) { return (float)((b == 8 ? 256 : 128) + (1 << (b - 1))); }

  __device__ __forceinline__ void set(uint32_t absmax_bits, int bits) {
    b = bits;
    const float absmax = __half2float(__ushort_as_half((unsigned short)absmax_bits));
    const __half s16 = __float2half_rn(__fdiv_rn(absmax, (float)((1 << b) - 1)));
    const float s = __half2float(s16);
    scale = __half_as_ushort(s16);
    rh = s > 0.0f ? __fdiv_rn(1.0f, s) * 0.5f : 0.0f;
    s2 = s * 2.0f;
    quick = scale - 0x0400u < 0x7800u;  // normal and finite (uniform where the row is)
    base = base_of(b);
    least = (0x8000u | scale) * 0x00010001u;
  }

  // The same quantizer, read back from LDS for a row that the whole wave shares:
  // its fields in scalar registers.
  __device__ __forceinline__ Quantizer uniform(int bits) const {
    auto first = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
    Quantizer r;
    r.scale = (uint16_t)first(scale);
    r.b = bits;
    r.quick = first(quick) != 0u;
    r.rh = __builtin_bit_cast(float, first(__builtin_bit_cast(uint32_t, rh)));
    r.s2 = __builtin_bit_cast(float, first(__builtin_bit_cast(uint32_t, s2)));
    r.base = base_of(bits);
    r.least = first(least);
    return r;
  }

  // Short form: f[j], whose bits 16..23 are the word of value j.
  template <bool kEight, int kDwords = 8>  // b == 8
  __device__ __forceinline__ void quick_bits(const uint32_t* d, uint32_t* f) const {
    typedef short short2_t __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int t = 0; t < kDwords; ++t) {
      const half2_t x0 = __builtin_bit_cast(half2_t, d[t]) + half2_t{(_Float16)0.0f, (_Float16)0.0f};
      const half2_t x = __builtin_bit_cast(
          half2_t, __builtin_elementwise_max(__builtin_bit_cast(short2_t, x0), __builtin_bit_cast(short2_t, least)));
      f[2 * t] = __builtin_bit_cast(uint32_t, __builtin_fmaf((float)x.x, rh, base)) << (kEight ? 1 : 0);
      f[2 * t + 1] = __builtin_bit_cast(uint32_t, __builtin_fmaf((float)x.y, rh, base)) << (kEight ? 1 : 0);
    }
  }
  // The words (bits 16..23) of four values in one dword.
  __device__ static __forceinline__ uint32_t gather(const uint32_t f[4]) {
    return __builtin_amdgcn_perm(f[1], f[0], 0x0C0C0602u) | __builtin_amdgcn_perm(f[3], f[2], 0x06020C0Cu);
  }

  // The 16 words of a lane, element 4 t + i in byte i of u[t].
  __device__ __forceinline__ void words(const uint32_t d[8], uint32_t u[4]) const {
    if (quick) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        uint32_t f[4];
        if (b == 8) quick_bits<true, 2>(d + 2 * t, f);
        else quick_bits<false, 2>(d + 2 * t, f);
        u[t] = gather(f);
      }
    } else {
      exact_words(d, u);
    }
  }

  __device__ __forceinline__ void exact_words(const uint32_t d[8], uint32_t u[4]) const {
#pragma clang fp contract(off)
    const int clo = -(1 << (b - 1)), chi = (1 << (b - 1)) - 1;
    const uint32_t field = ((1u << b) - 1u) * 0x01010101u;
    const uint32_t flip = (1u << (b - 1)) * 0x01010101u;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      uint32_t acc = 0u;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = 4 * t + q;
        const uint32_t bits = (d[j / 2] >> (16 * (j % 2))) & 0xFFFFu;
        const float x = __half2float(__ushort_as_half((unsigned short)bits));
        const float h0 = __builtin_fmaf(x, rh, 0.0f);
        const float e = __builtin_fmaf(-h0, s2, x);
        const float h = __builtin_fmaf(e, rh, h0);  // RN(x / s) / 2
        int c;
        asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(c) : "v"(h));
        c = min(max(c, clo), chi);
        const uint32_t sel = q == 1 ? 0x03020400u : q == 2 ? 0x03040100u : 0x04020100u;
        acc = q == 0 ? (uint32_t)c : __builtin_amdgcn_perm((uint32_t)c, acc, sel);
      }
      u[t] = (acc & field) ^ flip;
    }
  }
};

// Signed b-bit codes, one byte each.
template <bool kVec, int B>
struct CodeRow {
  static constexpr int kDwords = kLaneElems / 4;
  static constexpr int kElemBytes = 1;
  static constexpr bool kVector = kVec;
  static constexpr bool kScaled = false;

  // The lane's 16 codes from element k0 on.
  __device__ static void load(__amdgpu_buffer_rsrc_t rsrc, int k0, uint32_t d[kDwords]) {
    if (kVector) {
      // K % 16 == 0: the lane's 16 codes are all in the row or all past it.
      const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (uint32_t)k0, 0, 0);
#pragma unroll
      for (int t = 0; t < 4; ++t) d[t] = v[t];
    } else {
#pragma unroll
      for (int t = 0; t < kDwords; ++t) {
        uint32_t w = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          w |= (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rsrc, (uint32_t)(k0 + 4 * t + q), 0, 0)
               << (8 * q);
        d[t] = w;
      }
    }
  }
  // 16 codes at any byte.
  __device__ static void wide(const uint8_t* p, uint32_t d[kDwords]) {
    const any_u32x4_t v = *reinterpret_cast<const any_u32x4_t*>(p);
#pragma unroll
    for (int t = 0; t < 4; ++t) d[t] = v[t];
  }
  // The same from a row of K codes at `row`: where rows start at any byte, whole
  // groups are one unaligned 16-byte load and only the group across the row's end
  // takes byte loads.  W3A8 333 x 5003 x 2999 from codes, the GEMM's row stores at
  // any alignment included: 30.3 us with 16 byte loads per group and single
  // stores, 25.9 us so.
  __device__ static void load_row(__amdgpu_buffer_rsrc_t rsrc, const uint8_t* row, int K, int k0, uint32_t d[kDwords]) {
    if (kVector) {
      load(rsrc, k0, d);
    } else if (k0 + kLaneElems <= K) {
      wide(row + k0, d);
    } else if (k0 < K) {
      load(rsrc, k0, d);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) d[t] = 0u;
    }
  }
  // Bipolar words u = (x mod 2^b) XOR 2^(b-1), one per byte (Sec. III-A).
  __device__ static void words(const uint32_t d[kDwords], const Quantizer&, uint32_t u[4]) {
    constexpr uint32_t field = ((1u << B) - 1u) * 0x01010101u;
    constexpr uint32_t flip = (1u << (B - 1)) * 0x01010101u;
#pragma unroll
    for (int t = 0; t < 4; ++t) u[t] = (d[t] & field) ^ flip;
  }
};

// fp16 activations, quantized with the row's scale.
template <bool kVec, int B>
struct HalfRow {
  static constexpr int kDwords = kLaneElems / 2;
  static constexpr int kElemBytes = 2;
  static constexpr bool kVector = kVec;
  static constexpr bool kScaled = true;

  // The lane's 16 values from element k0 on (fp16 bits, two per dword).
  __device__ static void load(__amdgpu_buffer_rsrc_t rsrc, int k0, uint32_t d[kDwords]) {
    const uint32_t off = (uint32_t)k0 * 2u;
    if (kVector) {
      const u32x4_t v0 = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0);
      const u32x4_t v1 = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + 16u, 0, 0);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        d[t] = v0[t];
        d[4 + t] = v1[t];
      }
    } else {
#pragma unroll
      for (int t = 0; t < kDwords; ++t) {
        const uint32_t h0 = __builtin_amdgcn_raw_buffer_load_b16(rsrc, off + 4u * t, 0, 0);
        const uint32_t h1 = __builtin_amdgcn_raw_buffer_load_b16(rsrc, off + 4u * t + 2u, 0, 0);
        d[t] = (h0 & 0xFFFFu) | (h1 << 16);
      }
    }
  }
  // As CodeRow's.
  __device__ static void wide(const uint8_t* p, uint32_t d[kDwords]) {
    const any_u32x4_t v0 = reinterpret_cast<const any_u32x4_t*>(p)[0], v1 = reinterpret_cast<const any_u32x4_t*>(p)[1];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      d[t] = v0[t];
      d[4 + t] = v1[t];
    }
  }
  __device__ static void load_row(__amdgpu_buffer_rsrc_t rsrc, const uint8_t* row, int K, int k0, uint32_t d[kDwords]) {
    if (kVector) {
      load(rsrc, k0, d);
    } else if (k0 + kLaneElems <= K) {
      wide(row + (int64_t)k0 * 2, d);
    } else if (k0 < K) {
      load(rsrc, k0, d);
    } else {
#pragma unroll
      for (int t = 0; t < 8; ++t) d[t] = 0u;
    }
  }
  __device__ static void words(const uint32_t d[kDwords], const Quantizer& qz, uint32_t u[4]) { qz.words(d, u); }
};

// Delta swaps of an 8x8 bit-matrix transpose (bit 8r + c <-> bit 8c + r of a
// 64-bit value, rows r = bytes): distance 7 and 14 stay inside each dword,
// distance 28 moves nibbles between the dwords.  The three commute.
__device__ __forceinline__ uint32_t swap7(uint32_t x) {
  const uint32_t t = (x ^ (x >> 7)) & 0x00AA00AAu;
  return x ^ t ^ (t << 7);
}
__device__ __forceinline__ uint32_t swap14(uint32_t x) {
  const uint32_t t = (x ^ (x >> 14)) & 0x0000CCCCu;
  return x ^ t ^ (t << 14);
}

// Transposes the bytes lo (rows 0..3) and hi (rows 4..7): afterwards bit j of
// byte i is bit i of the former byte j.  With b <= 4 every byte is below 16:
// the distance-28 swap just moves hi's low nibbles up into lo (hi becomes 0).
template <int B>
__device__ __forceinline__ void transpose8x8(uint32_t& lo, uint32_t& hi) {
  if (B <= 4) {
    lo = swap14(swap7(lo | (hi << 4)));
    hi = 0u;
  } else {
    lo = swap14(swap7(lo));
    hi = swap14(swap7(hi));
    const uint32_t t = (lo ^ (hi << 4)) & 0xF0F0F0F0u;
    lo ^= t;
    hi ^= t >> 4;
  }
}

// This lane's word of plane pair (i, i + 1) after transpose8x8 of its two
// 8-element groups (lo/hi of elements 0..7 in sa, of 8..15 in sb): the even
// lane of a pair gets the 32 bits of plane i, the odd lane those of plane i + 1
// (one DPP swap between neighbours).
__device__ __forceinline__ uint32_t plane_word(uint32_t sa, uint32_t sb, int bi, bool odd) {
  // y = [a_i, b_i, a_i+1, b_i+1]: this lane's 16 bits of plane i, then of plane i+1
  const uint32_t y = __builtin_amdgcn_perm(
      sb, sa, (uint32_t)(bi | (4 + bi) << 8 | (bi + 1) << 16 | (5 + bi) << 24));
  const uint32_t z = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)y, 0xB1, 0xF, 0xF, false);  // lane ^ 1
  return __builtin_amdgcn_perm(z, y, odd ? 0x03020706u : 0x05040100u);
}

}  // namespace rowcode
}  // namespace apt
