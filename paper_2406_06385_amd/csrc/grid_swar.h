// The float32 decisions of the grid pass (which its host test runs too).
#pragma once

#include "common.h"

namespace lrqat {

// Four Q8 codes (one per byte of w) rounded to n or n + 1 as the bits of `carry`
// (bit 0 of each byte) say, n = floor(code / 2^f).  Returns the codes as two's
// complement, in the low nibble of each byte for b <= 4 and as whole signed
// bytes for b >= 5; clip marks (bit 7 of a byte) the codes that would leave the
// grid (n = hi with a carry).
__host__ __device__ __forceinline__ uint32_t swar_carry_q8(uint32_t w, uint32_t carry, int f, int b, uint32_t& clip) {
  const uint32_t ones = 0x01010101u;
  const uint32_t mn = ones * ((1u << b) - 1);
  const uint32_t nu = (w >> f) & mn;                       // n as a b-bit pattern per byte
  const uint32_t e = nu ^ (ones * ((1u << (b - 1)) - 1));   // zero where n = hi
  clip |= ~(((e + 0x7F7F7F7Fu) | e) & 0x80808080u) & (carry << 7);
  uint32_t qu = (nu + carry) & mn;
  if (b < 4) qu |= (qu & (ones << (b - 1))) * ((16u - (1u << b)) >> (b - 1));        // sign-extend to 4 bits
  else if (b > 4) qu |= (qu & (ones << (b - 1))) * ((256u - (1u << b)) >> (b - 1));  // to 8 bits
  return qu;
}

// Q8 code v (0..3) of a word, Phi0 = n + cf 2^-f: w of u = Phi0 + delta = n + 1/2 + w, delta = acc c.  The
// bracket is exact, so the one rounding keeps the sign of w at any size of delta; with |delta| < 1/2 the
// nearest integer to u is n + [w > 0], certain where |w| exceeds the error bound of delta.
__host__ __device__ __forceinline__ float grid_w(uint32_t word, int v, int f, float acc, float c) {
  const float sf = __builtin_bit_cast(float, uint32_t(127 - f) << 23);  // 2^-f
  const uint32_t fw = word & (0x01010101u * uint32_t((1 << f) - 1));
  return __builtin_fmaf(acc, c, __builtin_fmaf(float((fw >> (8 * v)) & 0xffu), sf, -0.5f));
}

// u + kGridMagic is u rounded half to even, the integer v as two's complement in its low bits (|v| < 2^22).
constexpr float kGridMagic = 12582912.f;  // 1.5 2^23

// v is certain where |u - v| is below this: u no nearer to a half-integer than the error bound tz of delta and
// the rounding of u, below 2^-24 (|v| + 1/2), more than doubled.  vab: |v|, or the largest of several.
// Values far off the grid are never certain.
__host__ __device__ __forceinline__ float grid_certain(float tz, float vab) {
  return vab < 32768.f ? 0.5f - (tz + __builtin_fmaf(0x1p-22f, vab, 0x1p-21f)) : -1.f;
}

}  // namespace lrqat
