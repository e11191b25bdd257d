// bf16 scalar helpers shared by the decoder-layer kernels and the projection
// with the gated product in its epilogue.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pgsr {
namespace {

__device__ inline float lo_bf16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float hi_bf16(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// fp32 -> bf16 bits, round to nearest even (finite inputs; NaN stays NaN).
__device__ inline uint32_t f32_to_bf16(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7F800000u) == 0x7F800000u) return (u >> 16) | ((u & 0xFFFFu) ? 0x40u : 0u);
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// SiLU(g) = g / (1 + e^-g)
__device__ inline float silu_f32(float g) { return g / (1.f + expf(-g)); }

}  // namespace
}  // namespace pgsr
