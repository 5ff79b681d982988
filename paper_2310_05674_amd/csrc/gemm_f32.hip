// fp32 contraction for the fp32 base learners (logistic regression, small MLPs): forward, dgrad and wgrad of a
// linear layer are the same kernel with different strides.  The matrix cores are used in their fp32 form
// (v_mfma_f32_16x16x4_f32), so results carry plain fp32 rounding.  Shapes are arbitrary: every global access is
// bounds-checked.
//
// These problems are tiny (a batch of 128 rows, a few hundred columns) and latency-bound, so the kernel is built for
// short dependency chains rather than for reuse: a workgroup owns one output tile, its eight waves split the
// contraction between them in interleaved chunks of 16 and fetch their operands from global memory straight into the
// MFMA operand layout (lane (r, q) holds row r and the four contraction indices 4q .. 4q+3 of a chunk: one 16-byte
// load where the contraction index is the contiguous one) -- no LDS staging, no barrier inside the loop, FDEPTH chunks
// of loads in flight ahead of the MFMAs.  The eight partial tiles are added in wave order through LDS, so the result does
// not depend on timing.  Measured on a 128 x 256 x 784 layer: 6.0 us, against 14.9 us with 32 x 32 tiles, four waves and one
// chunk ahead (32 workgroups on 256 CUs).
//
// Independent problems share a launch (a layer's weight gradient with its column sums and its input gradient; the + and
// the - pass of Eq. 5): a dependent launch costs ~4 us here, more than most of these products.
// The +-eps v passes read the weight operand as B + s * Bv (s = +-eps from device memory), so no perturbed copy of theta
// is ever written.
#include "common.h"
#include "kernels.h"
#include "mfma_f32.h"

namespace sama {
namespace {

struct GemmF32Batch { GemmF32Args j[GEMM_F32_MAX_JOBS]; int first_block[GEMM_F32_MAX_JOBS + 1]; int count; };

// XM x XN output tiles of 16 x 16 per workgroup; FDEPTH chunks in flight per wave
template <int XM, int XN, int FDEPTH>
__global__ __launch_bounds__(64 * FWAVES) void k_gemm_f32(GemmF32Batch batch) {
  constexpr int TM = 16 * XM, TN = 16 * XN;
  __shared__ float red[FWAVES][TM][TN + 1];
  __shared__ float rsum[FWAVES][TM];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, q = lane >> 4;
  int job = 0;
#pragma unroll
  for (int k = 1; k < GEMM_F32_MAX_JOBS; ++k)
    if (k < batch.count && (int)blockIdx.x >= batch.first_block[k]) job = k;
  const GemmF32Args a = batch.j[job];
  const int local = blockIdx.x - batch.first_block[job], nbx = (a.N + TN - 1) / TN;
  const int i0 = (local / nbx) * TM, j0 = (local % nbx) * TN;
  const float bscale = (a.Bv != nullptr && a.beps != nullptr) ? a.bsign * (*a.beps) : 0.f;
  const bool rows = a.rowsum != nullptr && j0 == 0;   // this workgroup also sums its rows of A over the contraction
  // 16-byte loads along the contraction index need it contiguous and every row start aligned
  const bool a_vec = a.sa_k == 1 && (a.sa_i & 3) == 0 && ((uintptr_t)a.A & 15) == 0;
  const bool b_vec = a.sb_k == 1 && (a.sb_j & 3) == 0 && ((uintptr_t)a.B & 15) == 0 && (a.Bv == nullptr || ((uintptr_t)a.Bv & 15) == 0);

  float4v acc[XM][XN];
  float rs[XM];
#pragma unroll
  for (int x = 0; x < XM; ++x) {
    rs[x] = 0.f;
#pragma unroll
    for (int y = 0; y < XN; ++y) acc[x][y] = (float4v){0.f, 0.f, 0.f, 0.f};
  }

  float4v av[FDEPTH][XM], bv[FDEPTH][XN], pv[FDEPTH][XN];
  auto fetch = [&](int k0, int buf) {
    const int k = k0 + 4 * q;
#pragma unroll
    for (int x = 0; x < XM; ++x) av[buf][x] = load_k4(a.A, a.sa_i, a.sa_k, i0 + 16 * x + r, a.M, k, a.K, a_vec);
#pragma unroll
    for (int y = 0; y < XN; ++y) {
      bv[buf][y] = load_k4(a.B, a.sb_j, a.sb_k, j0 + 16 * y + r, a.N, k, a.K, b_vec);
      if (bscale != 0.f) pv[buf][y] = load_k4(a.Bv, a.sb_j, a.sb_k, j0 + 16 * y + r, a.N, k, a.K, b_vec);
    }
  };
  // chunks wave, wave + FWAVES, ...; FDEPTH of them are requested before the first is used
  for (int kb = wave * FCH; kb < a.K; kb += FDEPTH * FWAVES * FCH) {
#pragma unroll
    for (int u = 0; u < FDEPTH; ++u)
      if (kb + u * FWAVES * FCH < a.K) fetch(kb + u * FWAVES * FCH, u);
#pragma unroll
    for (int u = 0; u < FDEPTH; ++u) {
      if (kb + u * FWAVES * FCH >= a.K) break;
      if (bscale != 0.f) {
#pragma unroll
        for (int y = 0; y < XN; ++y)
#pragma unroll
          for (int c = 0; c < 4; ++c) bv[u][y][c] = fmaf(bscale, pv[u][y][c], bv[u][y][c]);
      }
      if (rows) {
#pragma unroll
        for (int x = 0; x < XM; ++x) rs[x] += (av[u][x][0] + av[u][x][1]) + (av[u][x][2] + av[u][x][3]);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int x = 0; x < XM; ++x)
#pragma unroll
          for (int y = 0; y < XN; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u][x][c], bv[u][y][c], acc[x][y], 0, 0, 0);
    }
  }
  // partial tiles -> LDS, added in wave order
#pragma unroll
  for (int x = 0; x < XM; ++x) {
#pragma unroll
    for (int y = 0; y < XN; ++y)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[wave][16 * x + 4 * q + e][16 * y + r] = acc[x][y][e];
    if (rows) {
      float s = rs[x];
      s += __shfl_xor(s, 16, 64);
      s += __shfl_xor(s, 32, 64);
      if (q == 0) rsum[wave][16 * x + r] = s;
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < TM * TN; t += 64 * FWAVES) {
    const int li = t / TN, lj = t % TN, gi = i0 + li, gj = j0 + lj;
    if (gi >= a.M || gj >= a.N) continue;
    float bias = 0.f;
    if (a.bias != nullptr) {
      bias = a.bias[gj];
      if (bscale != 0.f && a.bias_v != nullptr) bias = fmaf(bscale, a.bias_v[gj], bias);
    }
    const float gate = a.gate != nullptr ? a.gate[(int64_t)gi * a.ldc + gj] : 1.f;
    float c = red[0][li][lj];
#pragma unroll
    for (int w = 1; w < FWAVES; ++w) c += red[w][li][lj];
    c += bias;
    if (a.relu) c = fmaxf(c, 0.f);
    a.C[(int64_t)gi * a.ldc + gj] = gate > 0.f ? c : 0.f;
  }
  if (rows && (int)threadIdx.x < TM && i0 + (int)threadIdx.x < a.M) {
    float c = rsum[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < FWAVES; ++w) c += rsum[w][threadIdx.x];
    a.rowsum[i0 + threadIdx.x] = c;
  }
}

int64_t tiles(const GemmF32Args* a, int count, int tm, int tn) {
  int64_t n = 0;
  for (int k = 0; k < count; ++k) n += (int64_t)((a[k].N + tn - 1) / tn) * ((a[k].M + tm - 1) / tm);
  return n;
}
template <int XM, int XN, int FDEPTH>
void launch_tile_f32(ProfScope& ps, hipStream_t st, const GemmF32Args* a, int count) {
  GemmF32Batch b{};
  b.count = count;
  int nb = 0;
  for (int k = 0; k < count; ++k) {
    b.j[k] = a[k];
    b.first_block[k] = nb;
    nb += (int)tiles(a + k, 1, 16 * XM, 16 * XN);
  }
  for (int k = count; k <= GEMM_F32_MAX_JOBS; ++k) b.first_block[k] = nb;
  launch_kernel(ps, k_gemm_f32<XM, XN, FDEPTH>, nb, 64 * FWAVES, 0, st, b);
}
}  // namespace

void launch_gemm_f32_batch(hipStream_t st, const GemmF32Args* a, int count) {
  double flops = 0.0;
  for (int k = 0; k < count; ++k) {
    if (a[k].M <= 0 || a[k].N <= 0) { note_launch_error("empty fp32 GEMM"); return; }
    flops += 2.0 * a[k].M * a[k].N * a[k].K;
  }
  ProfScope ps(st, F_GEMM_F32, flops);
  // The smallest tile gives the shortest chain and the most workgroups; it reads every operand row once per 16 columns, and as
  // soon as some CU has two of its workgroups to run the next larger tile is the faster one.  us, 16 x 16 / 32 x 32: 256 tiles
  // (512 x 128 x 784) 5.8 / 9.3, 384 (512 x 192 x 784) 9.7 / 9.4, 384 (512 x 192 x 256) 6.7 / 5.5; 32 x 32 / 64 x 32: 256 tiles
  // (1024 x 256 x 784) 9.6 / 15.3, 320 (1024 x 320 x 784) 16.8 / 15.3.  Over 408 products and pairs (32 to 2048 rows, widths to
  // 320, K to 1024) these lines take 1.2% longer than the fastest tile of each, lines at 512 3.6% (geometric means).
  constexpr int CUS = 256;
  if (tiles(a, count, 16, 16) <= CUS) launch_tile_f32<1, 1, 8>(ps, st, a, count);
  else if (tiles(a, count, 32, 32) <= CUS) launch_tile_f32<2, 2, 4>(ps, st, a, count);
  else launch_tile_f32<4, 2, 2>(ps, st, a, count);
}

}  // namespace sama
