// Operands of the fp32 MFMA (v_mfma_f32_16x16x4_f32) straight from global memory, for the kernels whose products are too
// small for LDS staging to pay.
#pragma once
#include "common.h"

namespace sama {

typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int FCH = 16;       // contraction indices per chunk (one wave, four MFMAs deep)
constexpr int FWAVES = 8;     // waves of a workgroup, each with every FWAVES-th chunk

// four consecutive contraction indices k .. k+3 of row `row` of an operand with element (row, k) at p[row * s_row + k * s_k];
// out-of-range rows / indices read as 0
__device__ __forceinline__ float4v load_k4(const float* __restrict__ p, int64_t s_row, int64_t s_k, int row, int nrows, int k, int K,
                                            bool vec_ok) {
  float4v v = {0.f, 0.f, 0.f, 0.f};
  if (row >= nrows) return v;
  const float* q = p + (int64_t)row * s_row + (int64_t)k * s_k;
  if (vec_ok && k + 3 < K) return *reinterpret_cast<const float4v*>(q);
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (k + c < K) v[c] = q[(int64_t)c * s_k];
  return v;
}

}  // namespace sama
