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
__device__ __forceinline__ float gelu_cdf_f(float x) {   // gelu(x) = x times this
  float e, g;
  erf_and_gauss(x * 0.70710678118654752f, e, g);
  return 0.5f * (1.f + e);
}
__device__ __forceinline__ float gelu_f(float x) { return x * gelu_cdf_f(x); }
__device__ __forceinline__ float dgelu_f(float x) {
  float e, g;
  erf_and_gauss(x * 0.70710678118654752f, e, g);
  return fmaf(x * 0.39894228040143268f, g, 0.5f * (1.f + e));
}

// Both as functions of a bf16 value, out of a table.  Both epilogues take them of a value already rounded to bf16, and from 2^-25
// to 16 there are only 3713 of those for each sign; below, the factor of gelu is that of 2^-25 and the derivative 1/2 to the
// last bit, above both are 1 (0 for negative values).  An entry is what the functions above give, so a tile that looks up and
// one that computes have the same bits.  Entry i of a sign, at byte 4 i + 2^14 sign: the value of bits GELU_TAB_FIRST + i.
constexpr int GELU_TAB_FIRST = 0x32ff, GELU_TAB_LAST = 0x4180, GELU_TAB_ENTRIES = GELU_TAB_LAST - GELU_TAB_FIRST + 1;
constexpr int GELU_TAB_BYTES = 31 * 1024;   // of one table, in whole 1 KB loads
static_assert((1 << 14) + 4 * GELU_TAB_ENTRIES <= GELU_TAB_BYTES && 4 * GELU_TAB_ENTRIES <= 1 << 14, "table size");
// byte offsets of the entries of a packed pair, also packed
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t gelu_tab_offsets(uint32_t pk) {
  const u16x2 first = {GELU_TAB_FIRST, GELU_TAB_FIRST}, most = {GELU_TAB_ENTRIES - 1, GELU_TAB_ENTRIES - 1};
  const u16x2 i = __builtin_elementwise_min(__builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, pk & 0x7fff7fffu), first), most);
  return (__builtin_bit_cast(uint32_t, i) << 2) | ((pk & 0x80008000u) >> 1);   // 4 i < 2^14: nothing leaves its half
}

}  // namespace sama
