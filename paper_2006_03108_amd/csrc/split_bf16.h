// fp32 products on the bf16 matrix cores (gfx950).
//
// A bf16 MFMA does sixteen times the work of an fp32 one in the same time (measured on loops of MFMAs alone: 2250
// against 146 TFLOP/s), and vector instructions issue beside it, which they do not beside an fp32 MFMA.  An fp32
// number is the exact sum of three bf16 numbers (24 significant bits = 3 x 8; Henry, Tang and Heinecke, "Leveraging the
// bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", ARITH 2019):
//     x = hi + mid + lo,   hi = bf16(x), mid = bf16(x - hi), lo = bf16(x - hi - mid)   (the differences are exact)
// so x * w is nine products of bf16 numbers.  The three smallest, mid * lo, lo * mid and lo * lo, are below 2^-25 |x w|
// and are left out: six MFMAs, smallest products first.  (With all nine the error of a sum of 64 terms is 1.12e-7, with six
// 1.13e-7, with fp32 MFMAs 1.53e-7.)
//
// What an MFMA does with them (measured): a product of two bf16 numbers has 16 bits, but bits that lie far below the
// largest operand of the instruction, the accumulator among them, are dropped towards minus infinity, where fp32 MFMAs
// round to nearest.  The five small products feel that most: beside the hi * hi products in one accumulator they bias the
// sum (22 000 terms, N(0, 1): mean error -8e-7 of the sum's rms, fp32 MFMAs -3e-9).  So a kernel either keeps them in an
// accumulator of their own, or changes the sign of one operand and of the accumulator now and then, which turns the bias
// round.  Relative error (2-norm) against 64 bits of each kernel that uses the split, fp32 MFMAs in brackets:
//   gemm_split     8192 terms 2.7e-7 (8.1e-7), 17 terms 5.0e-8 (8.1e-8)
//   conv_any       891 terms 1.7e-7 (5.4e-7), weight gradient over 32768 positions a partial 8.2e-7 (2.2e-6)
//   conv_wsplit    32768 positions 3.1e-7 (1.1e-6)
//   conv_split     4000 terms 3.9e-7 (1.1e-6); see there for its two ways
//
// Range.  The operands are multiplied by 2^24 as they are split, and the sums by 2^-48: so the lo part of every normal
// fp32 number is itself a normal bf16 (it would be flushed for numbers below 2^-110).  In exchange numbers from 2^103,
// sums from 2^80, infinities and NaNs make the sums that they enter infinite or NaN.  Kernels that use the split look at
// their finished sums; a workgroup with one that is not finite makes its whole tile again with fp32 MFMAs from operands
// staged as they are, so that these too are what fp32 products give.
#pragma once
#include <cstdint>

#include <hip/hip_runtime.h>

namespace distdl {

typedef __bf16 split_bf16x2 __attribute__((ext_vector_type(2)));
typedef float split_f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t split_u32x4 __attribute__((ext_vector_type(4)));
typedef float split_f32x16 __attribute__((ext_vector_type(16)));

constexpr float kSplitScale = 16777216.f;                      // 2^24, of either operand
constexpr float kUnsplit = 1.f / kSplitScale / kSplitScale;    // of the sums

__device__ inline uint32_t pack_bf16(float a, float b) {  // round to nearest even, one instruction
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(split_f32x2{a, b}, split_bf16x2));
}

// two numbers -> the hi, mid and lo parts, packed, of their multiples (thirteen vector instructions); scale: +-kSplitScale
__device__ inline void split_pair(float a, float b, float scale, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  a *= scale;
  b *= scale;
  hi = pack_bf16(a, b);
  a -= __uint_as_float(hi << 16);
  b -= __uint_as_float(hi & 0xffff0000u);
  mid = pack_bf16(a, b);
  a -= __uint_as_float(mid << 16);
  b -= __uint_as_float(mid & 0xffff0000u);
  lo = pack_bf16(a, b);
}

// eight numbers -> three MFMA operand pieces
__device__ inline void split_eight(const float (&x)[8], float scale, split_u32x4& hi, split_u32x4& mid, split_u32x4& lo) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t a, b, c;
    split_pair(x[2 * j], x[2 * j + 1], scale, a, b, c);
    hi[j] = a;
    mid[j] = b;
    lo[j] = c;
  }
}

// The other way to stage numbers, for a tile that is made again: their upper and their lower halves.
__device__ inline void halve_pair(uint32_t a, uint32_t b, uint32_t& upper, uint32_t& lower) {
  upper = __builtin_amdgcn_perm(b, a, 0x07060302u);
  lower = __builtin_amdgcn_perm(b, a, 0x05040100u);
}
__device__ inline void halve_eight(const float (&x)[8], split_u32x4& upper, split_u32x4& lower) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t a, b;
    halve_pair(__float_as_uint(x[2 * j]), __float_as_uint(x[2 * j + 1]), a, b);
    upper[j] = a;
    lower[j] = b;
  }
}
// the numbers of a lane's operand pieces
struct Eight {
  float v[8];
};
__device__ inline Eight join_halves(split_u32x4 upper, split_u32x4 lower) {
  Eight o;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    o.v[2 * j] = __uint_as_float(__builtin_amdgcn_perm(upper[j], lower[j], 0x05040100u));
    o.v[2 * j + 1] = __uint_as_float(__builtin_amdgcn_perm(upper[j], lower[j], 0x07060302u));
  }
  return o;
}
// c += a b over the 16 k of two operand pieces: element e of the lanes is k e and 8 + e
__device__ inline split_f32x16 multiply_fp32(const Eight& a, const Eight& b, split_f32x16 c) {
#pragma unroll
  for (int e = 0; e < 8; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[e], b.v[e], c, 0, 0, 0);
  return c;
}

// (fp32 bits) an infinity or a NaN
__device__ inline bool not_finite(float v) { return (__float_as_uint(v) & 0x7f800000u) == 0x7f800000u; }
// 0, or NaN if v or `seen` is not finite: one instruction a sum
__device__ inline float note_not_finite(float v, float seen) { return fmaf(v, 0.f, seen); }
// the same for all lanes, so that what depends on it branches for whole waves
__device__ inline bool any_not_finite(float seen) { return __builtin_amdgcn_ballot_w64(seen != 0.f) != 0; }

}  // namespace distdl
