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
// Values are split after a multiplication by 2^24, which the sum is rid of at the end: without it the parts of a value below 2^-109
// fall under the smallest bf16 (at 1e-36 the error was 2.6e-5); with it the lowest bit of every fp32 value, 2^-149, is a normal bf16.
// It costs one vector instruction a value (2.5 in 100 of the 10-pair 28x28 step, 4.5 of the 20-pair 32x32 one; a test for
// small values would cost the same and send them to the fp32 MFMAs).
// Why: v_mfma_f32_32x32x2_f32 takes sixteen times the matrix-pipe time of the bf16 MFMA, six of which replace it.  Forward-type
// kernel, 20 x 64 samples, 128 -> 256 channels at side 8: 100 TFLOP/s with the fp32 MFMAs, 157 when every block splits both
// operands, 180 with the weights split once by the update that writes them; weight gradient of the same layer 95, 152 when every wave
// splits what it multiplies, a tenth more with each chunk split once by its block (1035 -> 942 us).  What bounds the forward-type kernel now is
// the matrix pipe (1.1 PFLOP/s of bf16) together with the 6.5 vector instructions that split a value of the rows and the loads (6 bytes a weight).
// Error against 64-bit sums as a share of the fp32 MFMA's (64 .. 512 channels, sides 2 .. 16, six seeds each), 2-norm: 0.31-0.35 on normal
// and on gradient-sized inputs, 0.16-0.40 on positive ones, 0.34-0.55 on inputs after a ReLU, 0.38-0.44 on inputs spread over many
// magnitudes, where the weight gradient's is 0.64-0.87; the largest single error there is 0.6-1.0 on average over the seeds, and the
// worst seed's is up to 1.3 times the fp32 MFMA's worst (8e-5 of the root mean square).  It is this good because a bf16 MFMA
// rounds its accumulator once for several products and the small terms have an accumulator of their own.  (All six into one
// accumulator: 0.85, but 1.1-1.4 after a ReLU, where half the products are zero and the fp32 MFMA has nothing to round; not taken,
// although its 128 x 64 wave tiles were 8 % faster.)
// What leaves the range -- infinities, NaN, values from 2^104 and sums from 2^80 -- leaves an infinity or NaN in the accumulators; a
// block that finds one computes its tile again with the fp32 MFMAs.
struct Split8 { u32x4 h, m, l; };
constexpr float SPLIT_SCALE = 0x1p24f, SPLIT_UNSCALE = 0x1p-48f;      // of both operands; of their products' sum
__device__ __forceinline__ void split_pair(float x0, float x1, unsigned& h, unsigned& m, unsigned& l) {
  x0 *= SPLIT_SCALE;
  x1 *= SPLIT_SCALE;
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
// four neighbouring values of a row
struct Split4 { uint2 h, m, l; };
__device__ __forceinline__ Split4 split4(const u32x4& v) {
  Split4 s;
  split_pair(__uint_as_float(v[0]), __uint_as_float(v[1]), s.h.x, s.m.x, s.l.x);
  split_pair(__uint_as_float(v[2]), __uint_as_float(v[3]), s.h.y, s.m.y, s.l.y);
  return s;
}
__device__ inline void mma_u4(floatx16& acc, const u32x4& a, const u32x4& b) {
  mma16B(acc, __builtin_bit_cast(uint4, a), __builtin_bit_cast(uint4, b), bf16_t());
}

}  // namespace gan
