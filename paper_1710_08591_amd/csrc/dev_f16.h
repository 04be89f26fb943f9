// FP16 operand helpers for the matrix-core kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fftbf {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2 __attribute__((ext_vector_type(2)));

// Two floats into FP16 high and low terms: hi = fp16(v) (round to nearest
// even), lo = fp16(v - hi); the residual v - hi is exact in FP32 and comes
// from one mixed-precision fused multiply-add per value (the factor 1 is kept
// from the compiler, which would convert and subtract instead).
// No instruction here or elsewhere is written as inline assembly: the compiler
// does not see what such an instruction reads and writes, and leaves out the
// waits that it needs beside a matrix or dot product (an overwritten operand
// of a product still running, or a result read too early).
__device__ __forceinline__ void split2(float v0, float v1, uint32_t& hi, uint32_t& lo) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  const half2 h = __builtin_convertvector(f32x2{v0, v1}, half2);
  float one = 1.f;
  asm("" : "+s"(one));
  const f32x2 r = {fmaf(-(float)h[0], one, v0), fmaf(-(float)h[1], one, v1)};
  hi = __builtin_bit_cast(uint32_t, h);
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, half2));
}

}  // namespace fftbf
