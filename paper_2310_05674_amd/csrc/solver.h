// One element of the base solver's update: for the passes over all parameters and for the gradient launches that update what they compute.
#pragma once
#include "common.h"
#include "kernels.h"

namespace sama {

// Adam: m' = b1 m + (1-b1) g ; v' = b2 v + (1-b2) g^2 ; theta' = theta - lr c1 m' / (c2 sqrt(v') + eps)
// with c1 = 1/(1-b1^t), c2 = 1/sqrt(1-b2^t) computed on the host in double.
__device__ __forceinline__ void adam_one(float g, float& m, float& v, float& th, const AdamArgs& a) {   // g includes the L2 term
  m = fmaf(a.beta1, m, a.one_m_beta1 * g);
  v = fmaf(a.beta2, v, a.one_m_beta2 * g * g);
  th = th - a.lr_c1 * m / (fmaf(a.c2, sqrtf(v), a.eps));
}

// SGD with heavy-ball momentum: b' = mu b + g, theta' = theta - lr b' in one rounding (b' is g itself without momentum, and b not read).
__device__ __forceinline__ void sgd_one(float g, float& b, float& th, float lr, float mu) {   // g includes the L2 term
  b = mu != 0.f ? fmaf(mu, b, g) : g;
  th = fmaf(-lr, b, th);
}

}  // namespace sama
