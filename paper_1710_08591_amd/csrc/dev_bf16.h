// FP32 operands on the BF16 matrix cores (gfx950), as three BF16 terms.
//
// x = hi + mid + lo with hi = bf16(x), mid = bf16(x - hi), lo = x - hi - mid:
// round to nearest leaves 16 and then 8 significant bits in the residuals, so
// the three terms hold all 24 bits of an FP32 number.  A product of two such
// sums takes six matrix products,
//   x y ~ hi hi' + hi mid' + mid hi' + hi lo' + lo hi' + mid mid',
// accumulated in FP32; the three that are left out (mid lo', lo mid', lo lo')
// are below 2^-24 of the product, about 2^-27 in the mean and of either sign.
// v_mfma_f32_16x16x32_bf16 does the work of eight v_mfma_f32_16x16x4_f32 in
// half of one's time, so six of them take 3/8 of the FP32 instructions' time.
// Values that are not finite, or that round to infinity in BF16, make every
// sum they enter NaN or infinite: the kernels look at their sums and form
// those again with the FP32 instructions from the same operands (the three
// terms of a weight add up to it exactly).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fftbf {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// two values as BF16, round to nearest even: a in the low half
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ float bf16_lo(uint32_t v) { return __builtin_bit_cast(float, v << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t v) { return __builtin_bit_cast(float, v & 0xFFFF0000u); }

// the three terms of (a, b), packed
__device__ __forceinline__ void split3(float a, float b, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  hi = pack_bf16(a, b);
  a -= bf16_lo(hi);
  b -= bf16_hi(hi);
  mid = pack_bf16(a, b);
  lo = pack_bf16(a - bf16_lo(mid), b - bf16_hi(mid));
}

__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// c + a b over 32 products, smallest terms first: a and b hold the terms hi, mid, lo
__device__ __forceinline__ f32x4 mfma_bf16x3(const u32x4 (&a)[3], const u32x4 (&b)[3], f32x4 c) {
  c = mfma_bf16(a[1], b[1], c);
  c = mfma_bf16(a[0], b[2], c);
  c = mfma_bf16(a[2], b[0], c);
  c = mfma_bf16(a[0], b[1], c);
  c = mfma_bf16(a[1], b[0], c);
  return mfma_bf16(a[0], b[0], c);
}

}  // namespace fftbf
