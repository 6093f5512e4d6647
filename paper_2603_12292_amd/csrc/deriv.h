// Values and partial derivatives of the operators on one case (the adjoint
// kernels and the folding of constants).
#pragma once

#include "beagle_device.h"
#include "trig.h"

namespace bgl {

// binary operator O of (a, b)
template <uint32_t O>
__device__ __forceinline__ float gbinop(float a, float b) {
  if constexpr (O == B_ADD) return a + b;
  if constexpr (O == B_SUB) return a - b;
  if constexpr (O == B_MUL) return a * b;
  if constexpr (O == B_DIV) return op_div(a, b);
  if constexpr (O == B_RSUB) return b - a;
  if constexpr (O == B_RDIV) return op_div(b, a);
  return 0.0f;
}

// partial derivatives of binop<O>(A, B): (d/dA, d/dB); 0 where a protected
// division replaces the quotient by 1
template <uint32_t O>
__device__ __forceinline__ void dbinop(float A, float B, float& dA, float& dB) {
  if constexpr (O == B_ADD) { dA = 1.0f; dB = 1.0f; }
  if constexpr (O == B_SUB) { dA = 1.0f; dB = -1.0f; }
  if constexpr (O == B_MUL) { dA = B; dB = A; }
  if constexpr (O == B_DIV) {
    const bool nz = B != 0.0f;
    const float r = __builtin_amdgcn_rcpf(nz ? B : 1.0f);
    dA = nz ? r : 0.0f;
    dB = nz ? -A * r * r : 0.0f;
  }
  if constexpr (O == B_RSUB) { dA = -1.0f; dB = 1.0f; }
  if constexpr (O == B_RDIV) {
    const bool nz = A != 0.0f;
    const float r = __builtin_amdgcn_rcpf(nz ? A : 1.0f);
    dA = nz ? -B * r * r : 0.0f;
    dB = nz ? r : 0.0f;
  }
}

// sin (COS = false) or cos of one value per lane, the interpreter's functions
template <bool COS>
__device__ __forceinline__ float trig1(float x) {
  float v[1] = {x};
  trig_tile<COS, 1>(v);
  return v[0];
}

// d/dx of unary operator u at operand x with value y
__device__ __forceinline__ float dunary(uint32_t u, float x, float y) {
  switch (u) {
    case 0: return trig1<true>(x);
    case 1: return -trig1<false>(x);
    case 2: return (x > 80.0f || x < -80.0f) ? 0.0f : y;
    case 3: return x != 0.0f ? __builtin_amdgcn_rcpf(x) : 0.0f;
    case 4: return x != 0.0f ? copysignf(0.5f, x) * __builtin_amdgcn_rcpf(y) : 0.0f;
    case 5: return 2.0f * x;
    case 6: return -(y * y);
    case 7: return 1.0f + y * y;
    case 8: return rsqrtf((1.0f - x) * (1.0f + x));
    case 9: return -rsqrtf((1.0f - x) * (1.0f + x));
    case 10: return 1.0f / (1.0f + x * x);
    default: {
      // tanh: sech^2 x = 4e / (1 + e)^2 with e = exp(-2|x|) (1 - y^2 cancels
      // where tanh saturates)
      const float e = op_exp(-2.0f * __builtin_fabsf(x));
      const float ep = 1.0f + e;
      return (4.0f * e) / (ep * ep);
    }
  }
}

}  // namespace bgl
