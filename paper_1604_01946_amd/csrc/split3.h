// fp32 operands on the bf16 matrix cores: every value is cut into three bf16 parts, x = h + m + l.
//
// fp32 matrix instructions reach 155 TFLOP/s on this chip, bf16 ones 1900 (measured, random operands).  h is x rounded to
// bf16 (8 significant bits), m the remainder rounded, l what is left: it has at most 8 significant bits, so the three
// parts hold all 24 bits of x exactly.  Of the nine products of two such numbers the six largest are formed, hh, hm, mh,
// mm, hl, lh, each exactly and accumulated in fp32.  The three left out: for 1 <= |x| < 2, |m| <= 2^-8 and |l| <= 2^-17, so
// ml and lm are up to 2^-25 of a product each and ll up to 2^-34, together the half unit in the last place that one
// rounding of an fp32 multiplication may cost; over random operands their rms is 2^-27.5, and their signs are random.
//
// Splitting is Dekker's (1971); bf16 triples for fp32 products are in Henry, Tang and Heinecke, ARITH 2019.
//
// Range: bf16 numbers of full precision end at 2^-126 like fp32 ones, and the last part of x lies 16 binades below x.  So
// operands are multiplied by 2^24 before they are cut (kUp) and sums by 2^-48 (kDown), both exactly: the smallest fp32
// number is then 2^-125 and every part is a multiple of the last place of x, so all fp32 numbers are held exactly, subnormal
// ones included.  The top end is below instead.
//
// Infinities, NaN, large numbers: an infinite x has h = inf and m = x - h = NaN, a finite x that rounds to bf16's
// infinity after scaling (above 2.02e31) has h = inf and m = -inf, and a sum of 2^80 (1.2e24) or more overflows, so every
// sum that such an operand enters comes out NaN or infinite, never finite.  The kernels look for that and work such sums
// out again on the fp32 matrix instructions.
#pragma once
#include "internal.h"

namespace lstm {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

constexpr float kUp = 0x1p24f, kDown = 0x1p-48f;

// The parts of two values (multiplied by kUp already), each pair packed into one register (first value in the low half).
struct Split2 {
  unsigned h, m, l;
};
__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  const floatx2 v = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ Split2 split3(float a, float b) {
  Split2 s;
  s.h = pack_bf16(a, b);
  a -= __builtin_bit_cast(float, s.h << 16);
  b -= __builtin_bit_cast(float, s.h & 0xffff0000u);
  s.m = pack_bf16(a, b);
  a -= __builtin_bit_cast(float, s.m << 16);
  b -= __builtin_bit_cast(float, s.m & 0xffff0000u);
  s.l = pack_bf16(a, b);
  return s;
}

// The parts of eight values (multiplied by kUp already) with consecutive k: what a lane feeds to a matrix instruction.
__device__ __forceinline__ void split8(const float (&v)[8], bf16x8 (&p)[3]) {
  uintx4 o[3];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const Split2 s = split3(v[2 * j], v[2 * j + 1]);
    o[0][j] = s.h;
    o[1][j] = s.m;
    o[2][j] = s.l;
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) p[q] = __builtin_bit_cast(bf16x8, o[q]);
}

// acc += A * B for 16 (32x32 tile) k: the six products of the parts, smallest first
__device__ __forceinline__ floatx16 mfma_split3(const bf16x8 (&a)[3], const bf16x8 (&b)[3], floatx16 acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[2], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], acc, 0, 0, 0);
}

}  // namespace lstm
