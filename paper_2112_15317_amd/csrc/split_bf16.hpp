// split_bf16.hpp -- fp32 products on the bf16 MFMA.
//
// An fp32 value v is the exact sum of three bf16 values, high, mid and low
// (8 significant bits each): h = bf16(v), m = bf16(v - h), l = v - h - m, both
// differences exact.  Of the nine products of two such triples the six whose
// weights are at least 2^-16 of the leading one are formed,
//   a * b = ah*bh + (ah*bm + am*bh) + (ah*bl + am*bm + al*bh),
// on v_mfma_f32_16x16x32_bf16 with fp32 accumulation; the three left out are
// below 2^-24 of |a * b|, half an fp32 rounding.  The six MFMAs of a block of
// 32 reduction terms run from zero and their sum is added to the block's
// accumulator on the vector ALU, so a long sum is rounded once per 32 terms.
// Against 64 bits the results are closer than the fp32 MFMA's: the VGG-16
// stack's output is 4.6e-7 off instead of 6.9e-7; added straight into the
// accumulator, six roundings per 32 terms, it was 7.8e-7, for 3 % less time.
//
// Six bf16 MFMAs of 16x16x32 take 0.38 of the cycles of the fp32 MFMAs of the
// same product.  Power then limits the matrix pipe: independent chains of the
// 32x32x16 form run at 2.4 PFLOP/s over zeros and at 1.8 over random normals.
//
// Values the triple cannot carry.  An infinite or NaN operand, or one that
// rounds to infinity (above 3.39e38), makes a NaN of every sum it enters.  bf16
// ends at 2^-133 (the MFMA keeps subnormals, of operands, products and sums), so
// an operand below 2^-110 may have bits that no part holds; they are left in
// the remainder after the third part, whose low 16 bits are zero otherwise.  A
// block whose sums are not all finite, or whose operands lose bits, redoes its
// output tile on the fp32 MFMA from the operands in memory, so infinities, NaNs
// and tiny values come out as from fp32 sums, at 3 to 7 times the call's time.
#pragma once

#include "sb_internal.hpp"

namespace sb {

typedef short s8 __attribute__((ext_vector_type(8)));
typedef float f8v __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// D(16x16) += A(16x32) * B(32x16).  Lane l supplies A[l%16][8*(l/16) + j] and
// B[8*(l/16) + j][l%16] (j = 0..7) and receives D[4*(l/16) + v][l%16] in
// element v.
__device__ __forceinline__ f4 mfma16x16x32(s8 a, s8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The six products (part of A, part of B), ordered so that consecutive ones
// share an operand.
constexpr int kSplitA[6] = {2, 1, 1, 0, 0, 0}, kSplitB[6] = {0, 0, 1, 1, 2, 0};

// A fragment's (or an LDS piece's) eight values as three bf16 pieces.
struct Split8 { s8 p[3]; };   // high, mid, low

// The triples of two values, packed as bf16 pairs (lo in bits 0..15).  (The
// remainders as bf16 pair dot products with (-1, 0) and (0, -1) would be 7
// instructions instead of 11, but those run slower: FC products 35 -> 38 us.)
// lost: low 16 bits set if a value has bits below 2^-133.
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& h, uint32_t& m,
                                           uint32_t& l, uint32_t& lost) {
  h = f32x2_to_bf16x2(a, b);
  float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
  m = f32x2_to_bf16x2(ra, rb);
  ra -= __uint_as_float(m << 16);
  rb -= __uint_as_float(m & 0xffff0000u);
  l = f32x2_to_bf16x2(ra, rb);
  lost |= __float_as_uint(ra) | __float_as_uint(rb);
}

__device__ __forceinline__ Split8 split8(f8v v, uint32_t& lost) {
  u32x4 h, m, l;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t a, b, c;
    split_pair(v[2 * j], v[2 * j + 1], a, b, c, lost);
    h[j] = a; m[j] = b; l[j] = c;
  }
  return Split8{{__builtin_bit_cast(s8, h), __builtin_bit_cast(s8, m), __builtin_bit_cast(s8, l)}};
}

// The triple of a stored operand, from which split_value gets the value back
// exactly.  A value that the triple cannot carry is stored as a NaN, so that
// every sum it enters asks for the fp32 MFMA, and its own bits.
constexpr u16 kSplitRaw = 0x7fff;
__device__ __forceinline__ void split_stored(float v, u16& h, u16& m, u16& l) {
  h = f32_to_bf16(v);
  const float r = v - bf16_to_f32(h);
  m = f32_to_bf16(r);
  const float q = r - bf16_to_f32(m);
  l = f32_to_bf16(q);
  if ((h & 0x7f80u) == 0x7f80u || (__float_as_uint(q) & 0xffffu)) {
    const uint32_t bits = __float_as_uint(v);
    h = kSplitRaw;
    m = (u16)(bits >> 16);
    l = (u16)bits;
  }
}
__device__ __forceinline__ float split_value(u16 h, u16 m, u16 l) {
  return h == kSplitRaw ? __uint_as_float((uint32_t)m << 16 | l)
                        : bf16_to_f32(h) + (bf16_to_f32(m) + bf16_to_f32(l));
}

// Whether a wave's sums are not all finite.
template <int I, int J>
__device__ __forceinline__ bool split_suspect(const f4 (&acc)[I][J]) {
  float z[4] = {0.f, 0.f, 0.f, 0.f};               // stays 0 over finite values
#pragma unroll
  for (int i = 0; i < I; ++i)
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) z[v] = fmaf(acc[i][j][v], 0.f, z[v]);
  return !((z[0] + z[1]) + (z[2] + z[3]) == 0.f);
}

}  // namespace sb
