// fp32 products on the bf16 matrix cores (gfx950).
//
// A bf16 MFMA does sixteen times the work of an fp32 one in the same time (measured on loops of MFMAs alone: 2250
// against 146 TFLOP/s), and vector instructions issue beside it, which they do not beside an fp32 MFMA.  An fp32
// number is the exact sum of three bf16 numbers (24 significant bits = 3 x 8):
//     x = hi + mid + lo,   hi = bf16(x), mid = bf16(x - hi), lo = bf16(x - hi - mid)   (the differences are exact)
// so x * w is nine products of bf16 numbers, each exact in the fp32 accumulator of an MFMA.  The three smallest,
// mid * lo, lo * mid and lo * lo, are below 2^-25 |x w| and are left out: six MFMAs, smallest products first.
// Measured against 64-bit sums on N(0, 1) data, relative error (2-norm) for K = 64 / 1024 / 4096: 1.1e-7 / 4.6e-7 /
// 9.9e-7 here and 1.5e-7 / 5.8e-7 / 1.15e-6 with fp32 MFMAs (the same with all nine products): what is left is the
// rounding of the running sum, and a bf16 MFMA rounds it once for 16 products where an fp32 one rounds it for 2.
//
// Numbers that the split cannot carry: an infinity or a NaN, or a finite number that rounds to an infinite bf16
// (above 3.39e38), makes every sum it enters infinite or NaN (inf - inf, inf * 0), also where the fp32 sum would be a
// plain infinity or finite.  Kernels that use the split therefore look at their finished sums and take those that
// are not finite again, in fp32, from the operands.  Below 2^-110 a number's lo, then mid part is smaller than the
// smallest normal bf16 and is flushed: products lose what is below 2^-126 |w|.
#pragma once
#include <cstdint>

#include <hip/hip_runtime.h>

namespace distdl {

typedef __bf16 split_bf16x2 __attribute__((ext_vector_type(2)));
typedef float split_f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t split_u32x4 __attribute__((ext_vector_type(4)));

__device__ inline uint32_t pack_bf16(float a, float b) {  // round to nearest even, one instruction
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(split_f32x2{a, b}, split_bf16x2));
}

// two numbers -> their hi, mid and lo parts, packed (eleven vector instructions)
__device__ inline void split_pair(float a, float b, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  hi = pack_bf16(a, b);
  a -= __uint_as_float(hi << 16);
  b -= __uint_as_float(hi & 0xffff0000u);
  mid = pack_bf16(a, b);
  a -= __uint_as_float(mid << 16);
  b -= __uint_as_float(mid & 0xffff0000u);
  lo = pack_bf16(a, b);
}

// eight numbers -> three MFMA operand pieces
__device__ inline void split_eight(const float (&x)[8], split_u32x4& hi, split_u32x4& mid, split_u32x4& lo) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t a, b, c;
    split_pair(x[2 * j], x[2 * j + 1], a, b, c);
    hi[j] = a;
    mid[j] = b;
    lo[j] = c;
  }
}

__device__ inline bool not_finite(float v) { return (__float_as_uint(v) & 0x7f800000u) == 0x7f800000u; }

}  // namespace distdl
