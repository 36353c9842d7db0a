// Pieces shared by the summary builds: key conversion, quantisers, the zero-mode floor.
#pragma once

#include "locks_internal.h"

namespace locks {
namespace {

constexpr float kZeroRel = 1e-6f;
constexpr float kZeroAbs = 1e-10f;

// Elements of a 16-byte chunk of bf16 or fp32 keys as floats.
template <typename KT>
__device__ __forceinline__ void chunk_to_f(const uint4& w, float* out);
template <>
__device__ __forceinline__ void chunk_to_f<uint16_t>(const uint4& w, float* out) {
  const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    out[2 * e] = __uint_as_float(u[e] << 16);
    out[2 * e + 1] = __uint_as_float(u[e] & 0xffff0000u);
  }
}
template <>
__device__ __forceinline__ void chunk_to_f<float>(const uint4& w, float* out) {
  out[0] = __uint_as_float(w.x); out[1] = __uint_as_float(w.y);
  out[2] = __uint_as_float(w.z); out[3] = __uint_as_float(w.w);
}

__device__ __forceinline__ float f16_scale(float amax, float qmax) {
  float s = fminf(amax / qmax, 65504.0f);
  return (float)(_Float16)s;
}

// 1 / s for a code scale s (0 when s is 0: every code is then 0)
__device__ __forceinline__ float inv_scale(float s) { return s > 0.0f ? 1.0f / s : 0.0f; }
// code of x at scale 1 / inv: nearest integer, clamped to +-qmax (x inv may differ
// from x / s in the last bit, which moves a code only at an exact half)
__device__ __forceinline__ int quant(float x, float inv, int qmax) {
  float c = rintf(x * inv);
  c = fminf(fmaxf(c, (float)-qmax), (float)qmax);
  return (int)c;
}

// code of x at scale s by a correctly rounded division
__device__ __forceinline__ int quant_div(float x, float s, int qmax) {
  if (!(s > 0.0f)) return 0;
  return (int)fminf(fmaxf(rintf(x / s), (float)-qmax), (float)qmax);
}

// Nearest bfloat16 (ties to even) of a finite float, as its 16-bit pattern.
__device__ __forceinline__ uint32_t bf16_rne_bits(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

__device__ __forceinline__ uint16_t f16_bits(float s) {
  _Float16 h = (_Float16)s;
  return *reinterpret_cast<uint16_t*>(&h);
}

}  // namespace
}  // namespace locks
