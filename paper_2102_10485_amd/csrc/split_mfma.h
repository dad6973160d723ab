// MFMA operand types, and fp32 values as sums of bf16 parts.
#pragma once

#include "common.h"

namespace gan {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ inline void mma16B(floatx16& acc, const uint4& a, const uint4& b, bf16_t) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

// fp32 storage on the bf16 matrix cores.  x = h + m + l with h, m, l of eight significant bits each (h = bf16(x),
// m = bf16(x - h), l = x - h - m: both differences are exact, and l needs eight bits), so a product of two fp32 values is nine
// bf16 products, each exact in the MFMA.  The six down to 2^-16 of the product are taken, h*h into one fp32 accumulator and the
// five smaller ones into a second that is added at the end; the three left out are below 2^-24 of it and of either sign.
// Why: v_mfma_f32_32x32x2_f32 takes sixteen times the matrix-pipe time of the bf16 MFMA, six of which replace it.  Forward-type
// kernel, 20 x 64 samples, 128 -> 256 channels at side 8: 100 TFLOP/s before, 172 now; weight gradient of the same layer 95 and
// 126.  What bounds it now is the matrix pipe (1.0 PFLOP/s of bf16) and the 5.5 vector instructions that split a value (without
// them, 15 % less time).
// Error against 64-bit sums (relative, 64 .. 512 channels, sides 2 .. 16): 0.31-0.38 of the fp32 MFMA's on normal and on positive
// inputs, 0.35-0.56 on inputs after a ReLU, because a bf16 MFMA rounds its accumulator once for several products and the small
// terms have an accumulator of their own.  (All six into one accumulator: 0.85, but 1.1-1.4 after a ReLU, where half the products are zero
// and the fp32 MFMA has nothing to round; not taken, although its 128 x 64 wave tiles were 8 % faster.)
// What has no split -- infinities, NaN, values that round to a bf16 infinity -- leaves a NaN in the accumulators; a block that
// finds one computes its tile again with the fp32 MFMAs.  (Below 2^-110 the parts fall under the smallest bf16 and are lost.)
struct Split8 { u32x4 h, m, l; };
__device__ __forceinline__ void split_pair(float x0, float x1, unsigned& h, unsigned& m, unsigned& l) {
  h = pack2_bf16(x0, x1);
  const float r0 = x0 - __uint_as_float(h << 16), r1 = x1 - __uint_as_float(h & 0xffff0000u);
  m = pack2_bf16(r0, r1);
  l = pack2_bf16(r0 - __uint_as_float(m << 16), r1 - __uint_as_float(m & 0xffff0000u));
}
// eight values of one operand row (or column): elements 0..3 in lo, 4..7 in hi
__device__ __forceinline__ Split8 split8(const u32x4& lo, const u32x4& hi) {
  Split8 s;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const u32x4& v = i < 2 ? lo : hi;
    const int j = 2 * (i & 1);
    unsigned h, m, l;
    split_pair(__uint_as_float(v[j]), __uint_as_float(v[j + 1]), h, m, l);
    s.h[i] = h; s.m[i] = m; s.l[i] = l;
  }
  return s;
}
__device__ inline void mma_u4(floatx16& acc, const u32x4& a, const u32x4& b) {
  mma16B(acc, __builtin_bit_cast(uint4, a), __builtin_bit_cast(uint4, b), bf16_t());
}

}  // namespace gan
