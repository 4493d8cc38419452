// Backward functions of the surrogates (Section 2.1.1), at x = V - theta with slope k.
#pragma once
#include "common.hpp"

namespace snn {

template <int SURR> __device__ __forceinline__ float surr(float k, float x) {
  if (SURR == 0) { float d = 1.0f + k * fabsf(x); return 1.0f / (d * d); }
  if (SURR == 1) { float u = 1.5707963267948966f * k * x; return (0.5f * k) / (1.0f + u * u); }
  if (SURR == 2) { float s = 1.0f / (1.0f + __expf(-k * x)); return k * s * (1.0f - s); }
  if (SURR == 3) return fmaxf(0.0f, 1.0f - fabsf(k * x));
  if (SURR == 4) return fabsf(k * x) <= 1.0f ? 0.5f : 0.0f;      // boxcar
  return 1.0f;                                                   // straight-through
}

// The surrogates with the hardware reciprocal (1 ulp) instead of an IEEE division: for the
// kernels where the surrogate's arithmetic, not memory, is what a step waits for (the one-launch
// layer reverse: the division alone took 1.6 us per block of 64 steps; the recurrent reverse
// kernels).
template <int SURR> __device__ __forceinline__ float surr_rcp(float k, float x) {
  if (SURR == 0) { const float d = 1.0f + k * fabsf(x); return __builtin_amdgcn_rcpf(d * d); }
  if (SURR == 1) { const float u = 1.5707963267948966f * k * x; return (0.5f * k) * __builtin_amdgcn_rcpf(1.0f + u * u); }
  if (SURR == 2) { const float s = __builtin_amdgcn_rcpf(1.0f + __expf(-k * x)); return k * s * (1.0f - s); }
  return surr<SURR>(k, x);
}

}  // namespace snn
