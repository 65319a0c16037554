// 64-bit Hamming terms on the matrix cores: the bits of two descriptor words as FP4 (E2M1)
// digits, whose products the matrix instructions sum exactly in fp32.
#pragma once

#include "dev_common.hpp"

namespace ocsr {
namespace dev {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

// A product's operand is 32 FP4 numbers (16 bytes) per lane. Lane l of the 32 x 32 x 64
// form holds row (column) l & 31, digits 32 (l >> 5) ..; of the 16 x 16 x 128 form row
// (column) l & 15, digits 32 (l >> 4) ... Lane l's results are column l & 31 (l & 15) of
// rows 8 (r / 4) + 4 (l >> 5) + r % 4 (4 (l >> 4) + r).
__device__ __forceinline__ v16f mfma_fp4(v4i a, v4i b, v16f c) {
  const v8i A = {a.x, a.y, a.z, a.w, 0, 0, 0, 0}, B = {b.x, b.y, b.z, b.w, 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A, B, c, 4, 4, 0, 0, 0, 0);
}
__device__ __forceinline__ v4f mfma_fp4(v4i a, v4i b, v4f c) {
  const v8i A = {a.x, a.y, a.z, a.w, 0, 0, 0, 0}, B = {b.x, b.y, b.z, b.w, 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A, B, c, 4, 4, 0, 0, 0, 0);
}

// FP4 codes: the sign bit and, repeated eight times, the magnitudes 1, 2 and 4.
constexpr uint32_t kSign = 0x88888888u, kOne = 0x22222222u, kTwo = 0x44444444u, kFour = 0x66666666u;
// (w & sign) | mag and 2 w: v_bitop3_b32 and v_add_u32 issue up to 1.6 times as fast as the
// and-or and the left shift that the compiler would take (operands in vector registers).
// A product may read a vector instruction's result two wait states later at the earliest, and
// the compiler keeps that distance only for instructions that it knows: what feeds a product is
// a builtin, never inline asm (as asm, 53 of the dense kernels' 72 products followed their
// digits too closely). Doubled words are operands of and_or alone.
__device__ __forceinline__ uint32_t and_or(uint32_t w, uint32_t sign, uint32_t mag) {
  return __builtin_amdgcn_bitop3_b32(w, sign, mag, 0xea);
}
__device__ __forceinline__ uint32_t twice(uint32_t w) {
  uint32_t r;
  asm("v_add_u32 %0, %1, %1" : "=v"(r) : "v"(w));
  return r;
}
// 32 bits of a word as 32 numbers of one magnitude (bit 1: negative), seven instructions. sign,
// mag: kSign and the magnitude's codes, or both 0 for a word whose terms do not count. With
// +-1, p . q = 64 - 2 popcount(p ^ q).
__device__ __forceinline__ v4i fp4_signs(uint32_t w, uint32_t sign, uint32_t mag) {
  const uint32_t w2 = twice(w), w4 = twice(w2), w8 = twice(w4);
  v4i f;
  f.x = (int)and_or(w, sign, mag);
  f.y = (int)and_or(w2, sign, mag);
  f.z = (int)and_or(w4, sign, mag);
  f.w = (int)and_or(w8, sign, mag);
  return f;
}

// A cheaper code for words that meet one fixed word p many times (four instructions, no
// shifts): bits 0, 1 and 2 of each nibble stay where they are, as 0 or 1/2, 1, 2, and bit 3
// is a sign of +-1. The fixed word's digits (fp4_fixed) weigh them to 2 q (1 - 2 p) and
// -(1 - 2 p)(1 - 2 q), so that p . q = 2 popcount(p ^ q) - 2 popcount(p & 0x7777...) - 16 per
// 64 bits, between -112 and 112: what is left out depends on the fixed word alone.
__device__ __forceinline__ v4i fp4_bits(uint32_t w, uint32_t sign, uint32_t one) {
  v4i f;
  f.x = (int)(w & 0x11111111u);
  f.y = (int)(w & 0x22222222u);
  f.z = (int)(w & 0x44444444u);
  f.w = (int)((w & sign) | one);
  return f;
}
constexpr int kBitsMax = 112;   // largest |p . q| of a 64-bit word
// sign, one, two, four: the constants above, or all 0 for a point that does not count
__device__ __forceinline__ v4i fp4_fixed(uint32_t w, uint32_t sign, uint32_t one, uint32_t two,
                                         uint32_t four) {
  v4i f;
  f.x = (int)(((w << 3) & sign) | four);
  f.y = (int)(((w << 2) & sign) | two);
  f.z = (int)(((w << 1) & sign) | one);
  f.w = (int)((~w & sign) | one);
  return f;
}
// 2 popcount(p ^ q) - p . q of a fixed word p
__device__ __forceinline__ int fp4_fixed_rest(uint64_t w) {
  return 2 * __popcll(w & 0x7777777777777777ull) + 16;
}

}  // namespace dev
}  // namespace ocsr
