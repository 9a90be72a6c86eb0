// Device helpers for residues as bytes and as packed 16-bit pairs.  Include
// from .hip sources only.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "ozaki2_internal.h"

namespace oz2 {

// Rounding to an integer and reading an integer without the FP64 round and
// convert instructions (which issue at a fraction of the FMA rate): with
// kRound = 1.5 * 2^52, fma(x, y, kRound) is kRound plus the exact product
// x*y rounded to the nearest integer (ties to even) whenever |x*y| < 2^51,
// since doubles in [2^52, 2^53) are the integers; and for an integer-valued
// |x| < 2^31 the low 32 bits of x + kRound are x in two's complement.
constexpr double kRound = 0x1.8p52;

typedef unsigned short v2u16 __attribute__((ext_vector_type(2)));

// 16-bit pairs: the low halves of a (low half) and b; a * b + c in each half
// (one packed instruction); a value in both halves.
__device__ __forceinline__ uint32_t pair16(uint32_t a, uint32_t b) {
  return __builtin_amdgcn_perm(b, a, 0x05040100u);
}
__device__ __forceinline__ uint32_t pk_mad(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_bit_cast(uint32_t, __builtin_bit_cast(v2u16, a) * __builtin_bit_cast(v2u16, b) +
                                          __builtin_bit_cast(v2u16, c));
}
__device__ __forceinline__ uint32_t pk_add(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_bit_cast(v2u16, a) + __builtin_bit_cast(v2u16, b));
}
__device__ __forceinline__ uint32_t pk_sub(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_bit_cast(v2u16, a) - __builtin_bit_cast(v2u16, b));
}
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(v2u16, a),
                                                                __builtin_bit_cast(v2u16, b)));
}
__device__ __forceinline__ uint32_t both16(int x) {
  return ((uint32_t)x & 0xFFFF) * 0x10001u;
}

// The low bytes of the four halves of two pairs (elements 0, 1 and 2, 3).
__device__ __forceinline__ uint32_t bytes_of_pairs(uint32_t x01, uint32_t x23) {
  return __builtin_amdgcn_perm(x23, x01, 0x06040200u);
}

// mod(x, p) in the symmetric INT8 range of Section 1.2 ([-(p-1)/2, (p-1)/2]
// for odd p, [-128, 127] for p = 256: [hi + 1 - p, hi] with hi = (p - 1) / 2)
// for |x| < 2^14.  The FP32 quotient x (1/p) is within 2^-9 of x/p there, so
// its rounding is within one of the nearest integer to x/p, and one
// correction either way lands r in the range (checked exhaustively for every
// p <= 256 and |x| < 2^14).
__device__ inline int mod_small(int x, int p, float pinv, int hi) {
  int r = x - (int)rintf((float)x * pinv) * p;
  r -= r > hi ? p : 0;
  r += r < hi + 1 - p ? p : 0;
  return r;
}

// Signed byte i of a 32-bit word.
__device__ inline int sbyte(uint32_t w, int i) { return (int)(w << (24 - 8 * i)) >> 24; }

// mod_small for modulus l of a constant table, placed as byte i of a word.
struct SmallMod {
  int p, hi;
  float pinv;
  __device__ explicit SmallMod(const CrtConsts& cc, int l)
      : p(cc.mod[l].p), hi((cc.mod[l].p - 1) / 2), pinv((float)cc.mod[l].pinv) {}
  __device__ uint32_t byte(int x, int i) const {
    return (uint32_t)(mod_small(x, p, pinv, hi) & 0xFF) << (8 * i);
  }
};

}  // namespace oz2
