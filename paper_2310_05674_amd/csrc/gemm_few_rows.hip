// The forward products of a pass over very few token rows (scoring one text): C[M x N] = A [M][K] . (B + B2) [N][K]^T in bf16
// with fp32 accumulation.
//
// Such a product is a sweep over the weights: 768 x 3072, hi + lo, is 9.4 MB against 0.6 MB of everything else.  The tiles of
// gemm_bf16.hip leave it to a few dozen workgroups that walk the contraction slab by slab (12 x 768, 128 rows: 17 us for
// K = 3072).  Here a workgroup owns 32 rows and 16 columns, its eight waves split the contraction, every wave fetching its
// operands from global memory straight into the 16x16x32 MFMA layout, four or six k-steps at a time, and the eight partial tiles are
// added in wave order through LDS.
#include "common.h"
#include "gelu.h"
#include "kernels.h"

namespace sama {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int FR_ROWS = 32, FR_COLS = 16, FR_WAVES = 8, FR_STEP = 32;

// AHEAD: pairs of k-steps of a wave fetched together
template <bool HILO, int AHEAD>
__global__ __launch_bounds__(64 * FR_WAVES, AHEAD > 2 ? 2 : 4) void k_gemm_few_rows(GemmBf16Args a) {
  __shared__ float s_red[FR_WAVES][FR_ROWS][FR_COLS + 1];
  // the rows in use are not waited for: those behind them are fetched and multiplied like the others, and not stored
  const int rows = a.rows != nullptr ? *a.rows : a.M;
  const int i0 = blockIdx.y * FR_ROWS, j0 = blockIdx.x * FR_COLS;
  const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pairs = a.K / (2 * FR_STEP);   // a wave takes two k-steps in a row: whole 128-byte lines
  const bf16_t* const A0 = a.A + (int64_t)min(i0 + r, a.M - 1) * a.lda + 8 * q;
  const bf16_t* const A1 = a.A + (int64_t)min(i0 + 16 + r, a.M - 1) * a.lda + 8 * q;
  const int64_t ob = (int64_t)min(j0 + r, a.N - 1) * a.ldb + 8 * q;
  const int row = threadIdx.x / FR_COLS, col = threadIdx.x % FR_COLS, i = i0 + row, j = j0 + col;   // this thread's output, of 32 x 16
  const int64_t o = (int64_t)i * a.ldc + j;
  const bool inside = i < a.M && j < a.N;
  const float bias = a.bias != nullptr && inside ? a.bias[j] : 0.f, res = a.res32 != nullptr && inside ? a.res32[o] : 0.f;
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  for (int p0 = wave; p0 < pairs; p0 += FR_WAVES * AHEAD) {
    bf16x8 x[AHEAD][2][2], hi[AHEAD][2], lo[AHEAD][2];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      const int p = min(p0 + u * FR_WAVES, pairs - 1);   // behind the end: fetched, not used
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int at = (2 * p + k) * FR_STEP;
        hi[u][k] = *reinterpret_cast<const bf16x8*>(a.B + ob + at);
        if (HILO) lo[u][k] = *reinterpret_cast<const bf16x8*>(a.B2 + ob + at);
        x[u][k][0] = *reinterpret_cast<const bf16x8*>(A0 + at);
        x[u][k][1] = *reinterpret_cast<const bf16x8*>(A1 + at);
      }
    }
    __builtin_amdgcn_sched_barrier(0);   // every load before the first product
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      if (p0 + u * FR_WAVES >= pairs) break;
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[u][k][t], hi[u][k], acc[t], 0, 0, 0);
          if (HILO) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[u][k][t], lo[u][k], acc[t], 0, 0, 0);
        }
    }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) s_red[wave][16 * t + 4 * q + e][r] = acc[t][e];
  __syncthreads();
  if (i >= rows || j >= a.N) return;
  float c = s_red[0][row][col];
#pragma unroll
  for (int w = 1; w < FR_WAVES; ++w) c += s_red[w][row][col];
  c += bias;
  c += res;
  if (a.act == GEMM_ACT_GELU_FWD) c = gelu_f(bf16_to_f32(f32_to_bf16(c)));   // as gemm_bf16.hip takes it
  if (a.C32 != nullptr) a.C32[o] = c;
  if (a.C16 != nullptr) a.C16[o] = f32_to_bf16(c);
}
}  // namespace

void launch_gemm_few_rows(hipStream_t st, const GemmBf16Args& a) {
  const char* e = check_gemm_bf16(a);
  if (e == nullptr && (a.a_trans || !a.b_trans || a.bsign != 0.f || a.C16_pre != nullptr || a.act == GEMM_ACT_GELU_BWD)) e = "few rows: forward products without a backward pass only";
  if (e != nullptr) { note_launch_error(e); return; }
  ProfScope ps(st, a.B2 ? F_GEMM_NT_HILO : F_GEMM_NT, 2.0 * a.M * a.N * a.K * (a.B2 ? 2.0 : 1.0));
  const dim3 grid((a.N + FR_COLS - 1) / FR_COLS, (a.M + FR_ROWS - 1) / FR_ROWS);
  const bool deep = (int64_t)grid.x * grid.y <= 256;   // a workgroup per CU: more of it in flight; else room for a second one
  if (a.B2) launch_kernel(ps, deep ? k_gemm_few_rows<true, 3> : k_gemm_few_rows<true, 2>, grid, 64 * FR_WAVES, 0, st, a);
  else launch_kernel(ps, deep ? k_gemm_few_rows<false, 3> : k_gemm_few_rows<false, 2>, grid, 64 * FR_WAVES, 0, st, a);
}

}  // namespace sama
