// fp32 products on the bf16 matrix cores: an fp32 value is the exact sum of three
// bf16 values (8 + 8 + 8 significant bits, each the nearest to what is left), and
// a product x y is formed from the six partial products that are not below its
// rounding, accumulated in fp32, the smallest first:
//   x1 y3 + x3 y1 + x2 y2 + x1 y2 + x2 y1 + x1 y1
// (the dropped ones are at most 2^-25 of |x y| and of either sign). Six
// v_mfma_f32_16x16x32_bf16 replace eight v_mfma_f32_16x16x4_f32 of twice the time
// each: measured issue rates 2026 and 138 TFLOP/s, so 2.4 times the fp32 rate. The
// error against 64 bits is smaller: 0.37e-7, 0.94e-7 and 2.2e-7 relative for
// contractions of 32, 64 and 220 terms, 1.0e-7, 1.5e-7 and 2.7e-7 with the fp32
// instruction, which rounds with every product (one bf16 instruction sums 32 terms at
// once); 3x3 convolutions of 8 channels 0.54e-7 and 1.5e-7. The split needs no scaling
// (bf16 has fp32's exponent range; below 2^-110 its last part loses bits).
//
// An operand that is infinite, or finite but beyond the largest bf16 value, leaves NaN
// in every result that it takes part in. Width 220 forms results that are not finite
// again with fp32 instructions from the joined parts (all_finite, join8, pick), which
// gives infinities and overflow as fp32 has them and leaves the other examples' bits.
// The convolutions have no registers to spare for that (the check and the second form
// made the 28 x 28 solves 3 to 7 % slower, other sizes up to 30 %): their activations pass the
// NaN on, so that state and residual show it.
//
// The accumulation rounds towards minus infinity by a small part of its last place
// (the mean error of sums of positive terms is -0.8e-9, -3.5e-9 and -7.7e-9 for 32, 96
// and 224 terms; the fp32 instruction has none), which adds up over layers, pixels
// and examples in sums that nearly cancel. So a product is formed with the sign of
// its layer, layer_sign(n) K_n v, and the sign is taken back afterwards: the errors
// of the layers then cancel instead (the bias gradients of 64 convolution layers of
// 500 images: error 7e-7 to 2.2e-6 without the sign, 2e-7 to 6e-7 with it and
// with the fp32 instruction). The sign depends on the fine layer index alone, so that
// every level and every kernel evaluates a layer the same way bit for bit.
#pragma once

#include <float.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "lp_layer_sign.h"

namespace lp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float split_f32x4 __attribute__((ext_vector_type(4)));

// Eight values of a lane, split.
struct Split8 {
  bf16x8 p[3];
};

// x minus its leading bf16 values, which are taken from the packed words they were
// converted to (converting them back one by one would convert each value twice)
__device__ __forceinline__ f32x8 split_rest(f32x8 x, const bf16x8& p) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 w = __builtin_bit_cast(u32x4, p);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[2 * i] -= __builtin_bit_cast(float, w[i] << 16);
    x[2 * i + 1] -= __builtin_bit_cast(float, w[i] & 0xffff0000u);
  }
  return x;
}

__device__ __forceinline__ Split8 split8(f32x8 x) {
  Split8 s;
  s.p[0] = __builtin_convertvector(x, bf16x8);
  x = split_rest(x, s.p[0]);
  s.p[1] = __builtin_convertvector(x, bf16x8);
  x = split_rest(x, s.p[1]);
  s.p[2] = __builtin_convertvector(x, bf16x8);
  return s;
}

__device__ __forceinline__ Split8 split8(split_f32x4 a, split_f32x4 b) {
  return split8(__builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// The values of a split (what is beyond bf16's range comes back as the largest float).
__device__ __forceinline__ f32x8 join8(const Split8& s) {
  f32x8 x;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float a = (float)s.p[0][i], b = (float)s.p[1][i], c = (float)s.p[2][i];
    x[i] = fabsf(a) < INFINITY ? a + (b + c) : b != b ? a : copysignf(FLT_MAX, a);
  }
  return x;
}

// Whether every value of the wave whose sum a lane passes is finite (a sum that
// overflows says no, which costs time only).
__device__ __forceinline__ bool all_finite(split_f32x4 sum) {
  return !__any(!(fabsf((sum[0] + sum[1]) + (sum[2] + sum[3])) < INFINITY));
}

// z where it is finite, else f
__device__ __forceinline__ split_f32x4 pick(split_f32x4 z, split_f32x4 f) {
#pragma unroll
  for (int r = 0; r < 4; ++r) z[r] = fabsf(z[r]) < INFINITY ? z[r] : f[r];
  return z;
}

// The four products of two A and two B fragments, their chains' instructions in turn.
__device__ __forceinline__ void mma_split4(const Split8& a0, const Split8& a1, const Split8& b0, const Split8& b1,
                                           split_f32x4& c00, split_f32x4& c10, split_f32x4& c01,
                                           split_f32x4& c11) {
  constexpr int ia[6] = {0, 2, 1, 0, 1, 0}, ib[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    c00 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0.p[ia[k]], b0.p[ib[k]], c00, 0, 0, 0);
    c10 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1.p[ia[k]], b0.p[ib[k]], c10, 0, 0, 0);
    c01 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0.p[ia[k]], b1.p[ib[k]], c01, 0, 0, 0);
    c11 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1.p[ia[k]], b1.p[ib[k]], c11, 0, 0, 0);
  }
}

}  // namespace lp
