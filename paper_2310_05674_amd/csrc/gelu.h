// GELU and its derivative for the epilogues of the encoder's products: erf by Abramowitz & Stegun 7.1.26 (1.5e-7).
#pragma once
#include "common.h"

namespace sama {

// The correctly rounded 1 / y of a y in [1, 2^100]: the hardware's approximation and one Newton step, a third of the
// instructions of the general division.  Compared on an MI355X with __frcp_rn for each of the 838860801 floats of that range: no
// difference (profiles/gelu_reciprocal.md).
__device__ __forceinline__ float recip_rn(float y) {
  const float r = __builtin_amdgcn_rcpf(y);
  return fmaf(fmaf(-y, r, 1.f), r, r);
}
// For |z| so large that y would leave the range, exp(-z^2) is 0 and so is whatever it is multiplied by.
__device__ __forceinline__ void erf_and_gauss(float z, float& erfz, float& ez2) {
  const float az = fabsf(z);
  const float t = recip_rn(fminf(fmaf(0.3275911f, az, 1.f), 0x1p100f));
  ez2 = __expf(-az * az);
  const float poly = t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f), -0.284496736f), 0.254829592f);
  const float e = 1.f - poly * ez2;
  erfz = z < 0.f ? -e : e;
}
__device__ __forceinline__ float gelu_f(float x) {
  float e, g;
  erf_and_gauss(x * 0.70710678118654752f, e, g);
  return 0.5f * x * (1.f + e);
}
__device__ __forceinline__ float dgelu_f(float x) {
  float e, g;
  erf_and_gauss(x * 0.70710678118654752f, e, g);
  return fmaf(x * 0.39894228040143268f, g, 0.5f * (1.f + e));
}

}  // namespace sama
