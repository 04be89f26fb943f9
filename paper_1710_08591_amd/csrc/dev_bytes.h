// Byte-lane helpers of the int8 matrix-core kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fftbf {

typedef int v4i __attribute__((ext_vector_type(4)));

// y[k] = byte k of w0, w1, w2, w3
__device__ __forceinline__ void transpose_bytes(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t* y) {
  const uint32_t a01 = __builtin_amdgcn_perm(w1, w0, 0x05010400u), b01 = __builtin_amdgcn_perm(w1, w0, 0x07030602u);
  const uint32_t a23 = __builtin_amdgcn_perm(w3, w2, 0x05010400u), b23 = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
  y[0] = __builtin_amdgcn_perm(a23, a01, 0x05040100u);
  y[1] = __builtin_amdgcn_perm(a23, a01, 0x07060302u);
  y[2] = __builtin_amdgcn_perm(b23, b01, 0x05040100u);
  y[3] = __builtin_amdgcn_perm(b23, b01, 0x07060302u);
}

// the negatives of four int8 in [-127, 127]
__device__ __forceinline__ int neg_bytes(int z) {
  return (int)((((uint32_t)z ^ 0x7F7F7F7Fu) + 0x01010101u) ^ 0x80808080u);
}

// the four signed base-256 digits of v (each in [-128, 127]), lowest byte first
__device__ __forceinline__ uint32_t signed_digits(int v) { return ((uint32_t)v + 0x80808080u) ^ 0x80808080u; }

// a wavefront's LDS operations execute in the order it issues them, so data
// that stays within one wavefront needs the compiler's order only
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace fftbf
