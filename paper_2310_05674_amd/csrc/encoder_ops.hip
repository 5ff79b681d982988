// Non-GEMM pieces of the post-LN encoder base learner (Sec. 4.1 uses BERT / RoBERTa-shaped models):
// embedding gather + LayerNorm, LayerNorm forward / backward, fused attention forward / backward on the matrix
// cores, classifier head backward, column sums, embedding gradients.  All reductions run in a fixed order.
#include "common.h"
#include "kernels.h"

namespace sama {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float LN_EPS = 1e-5f;

// =========================================================================================== rows of a padded batch
// Every block works out where all the sequences go (at most 128 of them); thread i then places token row i of the padded
// batch, and marks row i of the plan where no sequence has it.
__global__ __launch_bounds__(256) void k_row_plan(const int32_t* __restrict__ ids, const int32_t* __restrict__ lens, int B, int S, RowSelect sel,
                                                  RowPlan out) {
  __shared__ int s_kept[MAX_SEQ], s_start[MAX_SEQ + 1];
  for (int b = threadIdx.x; b < B; b += 256) s_kept[b] = min(max(lens[b], 1), S);
  __syncthreads();
  for (int j = threadIdx.x; j < sel.n_mask; j += 256) {
    const int r = sel.mask_base + min(max(sel.mask_rows[j], 0), sel.mask_total - 1);
    atomicMax(&s_kept[r / S], r % S + 1);
  }
  __syncthreads();
  if (threadIdx.x < 64) {   // prefix sums: two sequences per lane, then across the wave
    const int b = 2 * threadIdx.x;
    const int k0 = b < B ? (s_kept[b] + ROW_GROUP - 1) / ROW_GROUP * ROW_GROUP : 0, k1 = b + 1 < B ? (s_kept[b + 1] + ROW_GROUP - 1) / ROW_GROUP * ROW_GROUP : 0;
    int sum = k0 + k1;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(sum, o, 64);
      if ((int)threadIdx.x >= o) sum += t;
    }
    if (b < B) { s_start[b] = sum - k0 - k1; s_start[b + 1] = sum - k1; }
    if (b + 1 < B) s_start[b + 2] = sum;
  }
  __syncthreads();
  const int total = s_start[B], i = blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.x == 0) {
    for (int b = threadIdx.x; b <= B; b += 256) out.start[b] = s_start[b];
    if (threadIdx.x == 0) *out.rows = (total + 63) / 64 * 64;
  }
  if (i >= B * S) return;
  const int b = i / S, pos = i - b * S, kept = s_start[b + 1] - s_start[b];
  if (pos < kept) {
    out.src[s_start[b] + pos] = i;
    out.ids[s_start[b] + pos] = ids[i];
  }
  if (pos % ROW_GROUP == 0) out.group[i / ROW_GROUP] = pos < kept ? (s_start[b] + pos) / ROW_GROUP : -1;
  if (i >= total) { out.src[i] = -1; out.ids[i] = 0; }
}

// One load brings a line of 128 bytes into the caches; the value is not used.
__device__ __forceinline__ void fetch_ahead(const WeightsAhead& w, const int32_t* __restrict__ rows, int block, int threads) {
  if (rows != nullptr && *rows >= w.max_rows) return;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (w.p[k] == nullptr) continue;
#pragma unroll 4
    for (int64_t i = ((int64_t)block * threads + threadIdx.x) * 64; i < w.n; i += (int64_t)AHEAD_BLOCKS * threads * 64) {
      const uint32_t v = *reinterpret_cast<const uint32_t*>(w.p[k] + i);
      asm volatile("" ::"v"(v));
    }
  }
}

// =========================================================================================== LayerNorm forward
// One wave per row; the row lives in registers, NV 16-byte pieces per lane (d <= 256 NV).  Statistics in fp32 with a centred
// second pass.
template <int NV>
__global__ __launch_bounds__(256) void k_ln_fwd(LnFwdArgs a) {
  const int block = (int)blockIdx.x - (a.ahead.n > 0 ? AHEAD_BLOCKS : 0);
  if (block < 0) return fetch_ahead(a.ahead, a.rows, blockIdx.x, 256);
  const int lane = threadIdx.x & 63, row = block * 4 + (threadIdx.x >> 6);
  const int r = a.pass_rows > 0 ? row % a.pass_rows : row;   // within its pass
  if (row >= a.M || (a.rows != nullptr && r >= *a.rows)) return;
  const int nq = a.d >> 2;  // float4 chunks per row
  const float sc = a.pv.scale_row(row);
  const int pos = a.x != nullptr ? 0 : (a.src != nullptr ? max(a.src[r], 0) : r) % a.S;
  float4 xr[NV];
  float sum = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int q = lane + 64 * j;
    xr[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (q < nq) {
      if (a.x != nullptr) {
        xr[j] = reinterpret_cast<const float4*>(a.x + (int64_t)row * a.d)[q];
      } else {
        const int id = min(max(a.ids[r], 0), a.V - 1);   // ids outside [0, V) are clamped
        const int64_t to = a.tok_off + (int64_t)id * a.d + 4 * q, po = a.pos_off + (int64_t)pos * a.d + 4 * q;
        float4 t = *reinterpret_cast<const float4*>(a.pv.theta + to), p = *reinterpret_cast<const float4*>(a.pv.theta + po);
        if (sc != 0.f) {
          const float4 tv = *reinterpret_cast<const float4*>(a.pv.vdir + to), pvv = *reinterpret_cast<const float4*>(a.pv.vdir + po);
          t.x = fmaf(sc, tv.x, t.x); t.y = fmaf(sc, tv.y, t.y); t.z = fmaf(sc, tv.z, t.z); t.w = fmaf(sc, tv.w, t.w);
          p.x = fmaf(sc, pvv.x, p.x); p.y = fmaf(sc, pvv.y, p.y); p.z = fmaf(sc, pvv.z, p.z); p.w = fmaf(sc, pvv.w, p.w);
        }
        xr[j] = make_float4(t.x + p.x, t.y + p.y, t.z + p.z, t.w + p.w);
        if (a.x_out != nullptr) reinterpret_cast<float4*>(a.x_out + (int64_t)row * a.d)[q] = xr[j];
      }
      sum += (xr[j].x + xr[j].y) + (xr[j].z + xr[j].w);
    }
  }
  const float mu = wave_sum(sum) / (float)a.d;
  float sq = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    if (lane + 64 * j < nq) {
      const float e0 = xr[j].x - mu, e1 = xr[j].y - mu, e2 = xr[j].z - mu, e3 = xr[j].w - mu;
      sq += (e0 * e0 + e1 * e1) + (e2 * e2 + e3 * e3);
    }
  }
  const float rstd = rsqrtf(wave_sum(sq) / (float)a.d + LN_EPS);
  if (lane == 0) {
    if (a.mean != nullptr) a.mean[row] = mu;
    if (a.rstd != nullptr) a.rstd[row] = rstd;
  }
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int q = lane + 64 * j;
    if (q < nq) {
      float4 g = *reinterpret_cast<const float4*>(a.pv.theta + a.g_off + 4 * q), b = *reinterpret_cast<const float4*>(a.pv.theta + a.b_off + 4 * q);
      if (sc != 0.f) {
        const float4 gv = *reinterpret_cast<const float4*>(a.pv.vdir + a.g_off + 4 * q), bv = *reinterpret_cast<const float4*>(a.pv.vdir + a.b_off + 4 * q);
        g.x = fmaf(sc, gv.x, g.x); g.y = fmaf(sc, gv.y, g.y); g.z = fmaf(sc, gv.z, g.z); g.w = fmaf(sc, gv.w, g.w);
        b.x = fmaf(sc, bv.x, b.x); b.y = fmaf(sc, bv.y, b.y); b.z = fmaf(sc, bv.z, b.z); b.w = fmaf(sc, bv.w, b.w);
      }
      const float4 o = make_float4(fmaf((xr[j].x - mu) * rstd, g.x, b.x), fmaf((xr[j].y - mu) * rstd, g.y, b.y),
                                   fmaf((xr[j].z - mu) * rstd, g.z, b.z), fmaf((xr[j].w - mu) * rstd, g.w, b.w));
      uint2 pk;
      pk.x = pack_bf16x2(o.x, o.y);
      pk.y = pack_bf16x2(o.z, o.w);
      *reinterpret_cast<uint2*>(a.y + (int64_t)row * a.d + 4 * q) = pk;
      if (a.y32 != nullptr) reinterpret_cast<float4*>(a.y32 + (int64_t)row * a.d)[q] = o;
    }
  }
}

// =========================================================================================== LayerNorm backward
// dx = rstd (dy g - mean(dy g) - xh mean(dy g xh)); per-block partial sums of dgamma = dy xh, dbeta = dy and of
// dx itself (the bias gradient of the linear layer feeding this LayerNorm).  A block owns LN_BWD_ROWS rows, a wave one of them; what
// the sums are made of goes through LDS, 1024 columns at a time, and is added in pairs of rows, the pairs in order.
// Bound by memory where there is much of it (8192 rows of 768: 16.1 us, 6.1 TB/s) and by the chain from the loads through two sums
// over the row where there is little: two rows to a wave and sums by shuffles took 8.4 us for 2048 rows of 1024, now 6.5, and 5.7
// for 512 of 768, now 4.2.
template <int NV>
__global__ __launch_bounds__(64 * LN_BWD_ROWS) void k_ln_bwd(LnBwdArgs a) {
  constexpr int G = 4;   // pieces of a lane in a turn
  static_assert(NV % G == 0 && LN_BWD_ROWS == 8, "turns; four pairs of rows");
  __shared__ float4 s_a[LN_BWD_ROWS][64 * G], s_b[LN_BWD_ROWS][64 * G];
  const int block = (int)blockIdx.x - (a.ahead.n > 0 ? AHEAD_BLOCKS : 0);
  if (block < 0) return fetch_ahead(a.ahead, a.rows, blockIdx.x, 64 * LN_BWD_ROWS);
  const int M = a.rows != nullptr ? __builtin_amdgcn_readfirstlane(*a.rows) : a.M;
  if (block * LN_BWD_ROWS >= M) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = block * LN_BWD_ROWS + wave;
  const int nq = a.d >> 2;
  const bool live = row < M;
  float4 xh[NV], dy[NV], dx[NV];   // dx: gamma, then dy g, then dx
  float mu = 0.f, rstd = 0.f;
  if (live) { mu = a.mean[row]; rstd = a.rstd[row]; }
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int q = lane + 64 * j;
    xh[j] = dy[j] = dx[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (live && q < nq) {
      xh[j] = reinterpret_cast<const float4*>(a.x + (int64_t)row * a.d)[q];
      dy[j] = reinterpret_cast<const float4*>(a.dy + (int64_t)row * a.d)[q];
      dx[j] = reinterpret_cast<const float4*>(a.gamma)[q];
    }
  }
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    if (lane + 64 * j >= nq) continue;
    xh[j] = make_float4((xh[j].x - mu) * rstd, (xh[j].y - mu) * rstd, (xh[j].z - mu) * rstd, (xh[j].w - mu) * rstd);
    dx[j] = make_float4(dy[j].x * dx[j].x, dy[j].y * dx[j].y, dy[j].z * dx[j].z, dy[j].w * dx[j].w);
    s1 += (dx[j].x + dx[j].y) + (dx[j].z + dx[j].w);
    s2 += (dx[j].x * xh[j].x + dx[j].y * xh[j].y) + (dx[j].z * xh[j].z + dx[j].w * xh[j].w);
  }
  const float m1 = wave_sum(s1) / (float)a.d, m2 = wave_sum(s2) / (float)a.d;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int q = lane + 64 * j;
    dx[j].x = rstd * (dx[j].x - m1 - xh[j].x * m2); dx[j].y = rstd * (dx[j].y - m1 - xh[j].y * m2);
    dx[j].z = rstd * (dx[j].z - m1 - xh[j].z * m2); dx[j].w = rstd * (dx[j].w - m1 - xh[j].w * m2);
    if (live && q < nq) {
      if (a.dx32 != nullptr) reinterpret_cast<float4*>(a.dx32 + (int64_t)row * a.d)[q] = dx[j];
      if (a.dx16 != nullptr) {
        uint2 pk;
        pk.x = pack_bf16x2(dx[j].x, dx[j].y);
        pk.y = pack_bf16x2(dx[j].z, dx[j].w);
        *reinterpret_cast<uint2*>(a.dx16 + (int64_t)row * a.d + 4 * q) = pk;
      }
    }
  }
  float4* const out = reinterpret_cast<float4*>(a.partial + (int64_t)block * 3 * a.d);
  const int tid = threadIdx.x;
  auto pairs_in_order = [](auto pair) {
    float4 t = pair(0);
#pragma unroll
    for (int r = 2; r < LN_BWD_ROWS; r += 2) { const float4 u = pair(r); t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w; }
    return t;
  };
#pragma unroll
  for (int j0 = 0; j0 < NV; j0 += G) {
    if (64 * j0 >= nq) break;
    if (j0 > 0) __syncthreads();
#pragma unroll
    for (int j = 0; j < G; ++j) { s_a[wave][lane + 64 * j] = xh[j0 + j]; s_b[wave][lane + 64 * j] = dy[j0 + j]; }
    __syncthreads();
    // half of the threads dgamma, the other half dbeta
    const int c = tid & (64 * G - 1), q = 64 * j0 + c;
    static_assert(64 * LN_BWD_ROWS == 2 * 64 * G, "a thread per quad of columns and sum");
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    if (q < nq) {
      if (tid < 64 * G) t = pairs_in_order([&](int r) {
        const float4 x0 = s_a[r][c], d0 = s_b[r][c], x1 = s_a[r + 1][c], d1 = s_b[r + 1][c];
        return make_float4(fmaf(d1.x, x1.x, d0.x * x0.x), fmaf(d1.y, x1.y, d0.y * x0.y), fmaf(d1.z, x1.z, d0.z * x0.z), fmaf(d1.w, x1.w, d0.w * x0.w));
      });
      else t = pairs_in_order([&](int r) {
        const float4 d0 = s_b[r][c], d1 = s_b[r + 1][c];
        return make_float4(d0.x + d1.x, d0.y + d1.y, d0.z + d1.z, d0.w + d1.w);
      });
      out[(tid < 64 * G ? 0 : nq) + q] = t;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < G; ++j) s_a[wave][lane + 64 * j] = dx[j0 + j];
    __syncthreads();
    if (tid < 64 * G && q < nq)
      out[2 * nq + q] = pairs_in_order([&](int r) {
        const float4 d0 = s_a[r][c], d1 = s_a[r + 1][c];
        return make_float4(d0.x + d1.x, d0.y + d1.y, d0.z + d1.z, d0.w + d1.w);
      });
  }
}

// out_v[c] = sum_r partial[r*stride + v*vstride + c] for up to three vectors v per job, several jobs per launch.
// A block owns 32 columns of one vector of one job; eight row groups walk the rows with stride 8 (independent
// loads), then are added in a fixed order.
struct ReduceRowsMulti { ReduceRowsJob j[REDUCE_MAX_JOBS]; int first_block[REDUCE_MAX_JOBS + 1]; int count; };
__global__ __launch_bounds__(256) void k_reduce_rows(ReduceRowsMulti m) {
  __shared__ float s_part[8][33];
  __shared__ int s_group[MAX_TOKENS / ROW_GROUP];
  int job = 0;
#pragma unroll
  for (int k = 1; k < REDUCE_MAX_JOBS; ++k)
    if (k < m.count && (int)blockIdx.x >= m.first_block[k]) job = k;
  const ReduceRowsJob& a = m.j[job];
  const int local = blockIdx.x - m.first_block[job], nbx = (a.N + 31) / 32;
  const int cl = threadIdx.x & 31, rg = threadIdx.x >> 5, c = (local % nbx) * 32 + cl, v = local / nbx;
  float acc = 0.f;
  if (a.group != nullptr) {
    for (int g = threadIdx.x; g * a.group_blocks < a.nrows; g += 256) s_group[g] = a.group[g];
    __syncthreads();
  }
  if (c < a.N) {
    const float* p = a.partial + (int64_t)v * a.vstride + c;
    if (a.group != nullptr) {
#pragma unroll 4
      for (int r = rg; r < a.nrows; r += 8) {
        const int g = s_group[r / a.group_blocks];
        const float v = p[(int64_t)(max(g, 0) * a.group_blocks + r % a.group_blocks) * a.stride];
        acc += g >= 0 ? v : 0.f;
      }
    } else if (a.seq_blocks > 0) {
      for (int r = rg; r < a.nrows; r += 8) {
        const int s = r / a.seq_blocks, o = r - s * a.seq_blocks;
        if (o < a.kept_blocks) acc += p[(int64_t)(s * a.kept_blocks + o) * a.stride];
      }
    } else {
#pragma unroll 4
      for (int r = rg; r < a.nrows; r += 8) acc += p[(int64_t)r * a.stride];
    }
  }
  s_part[rg][cl] = acc;
  __syncthreads();
  if (rg == 0 && c < a.N) {
    float t = s_part[0][cl];
#pragma unroll
    for (int g = 1; g < 8; ++g) t += s_part[g][cl];
    a.out[v][c] = t;
  }
}

// partial[rb][c] = sum of COLSUM_ROWS rows of column c of a bf16 matrix, up to two matrices per launch
struct ColsumMulti { ColsumJob j[2]; int first_block[3]; int count; };
__global__ __launch_bounds__(256) void k_colsum_partial_bf16(ColsumMulti m) {
  // a thread owns 8 adjacent columns (one 16-byte load per row); N is a multiple of 8
  const int job = (m.count > 1 && (int)blockIdx.x >= m.first_block[1]) ? 1 : 0;
  const ColsumJob& a = m.j[job];
  const int local = blockIdx.x - m.first_block[job], nbx = (a.N + 2047) / 2048;
  const int c = ((local % nbx) * 256 + threadIdx.x) * 8, rb = local / nbx;
  const int r0 = rb * COLSUM_ROWS, M = __builtin_amdgcn_readfirstlane(a.rows != nullptr ? *a.rows : a.M);
  if (c >= a.N || r0 >= M) return;
  float s[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) s[e] = 0.f;
  uint4 v[COLSUM_ROWS];
#pragma unroll
  for (int r = 0; r < COLSUM_ROWS; ++r)
    v[r] = (r0 + r < M) ? *reinterpret_cast<const uint4*>(a.X + (int64_t)(r0 + r) * a.N + c) : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
  for (int r = 0; r < COLSUM_ROWS; ++r) {
    const uint32_t w[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] += bf16_to_f32((bf16_t)(w[e >> 1] >> ((e & 1) * 16)));
  }
  float* out = a.partial + (int64_t)rb * a.N + c;
  *reinterpret_cast<float4*>(out) = make_float4(s[0], s[1], s[2], s[3]);
  *reinterpret_cast<float4*>(out + 4) = make_float4(s[4], s[5], s[6], s[7]);
}

// =========================================================================================== attention
// Sequence length S = 32 NT (NT = 2, 4 or 8 tiles of 32 positions), head width 64.
constexpr int AD = 64;  // head width

// four values as an operand
__device__ __forceinline__ s16x4 pack4(float a, float b, float c, float d) {
  return __builtin_bit_cast(s16x4, make_uint2(pack_bf16x2(a, b), pack_bf16x2(c, d)));
}

// A [ROWS x 64] bf16 matrix of a head (row stride ld in memory) is staged in LDS in dense rows of 128 bytes, the 16-byte chunk
// index of row r XORed with chunk_swz(r).  It is read in two ways, both without bank conflicts:
//   rows_operand: lane l takes 8 consecutive values of row base + l % 32 (sixteen rows at one chunk: sixteen 16-byte slots)
//   ld_transposed: for the 32x32x8 MFMA, lane l gets S[k0 + 4 (l / 32) + 0..3][e32 + l % 32] through ds_read_b64_tr_b16 (the
//     four rows one read touches lie in four different 64-byte windows)
// The matrices that a tile's products walk over come from there: fetched from global memory between those dependent products,
// each operand costs the latency of the L2 or beyond (S = 128, 384 heads: backward 37.6 us that way, 23.6 from LDS).  What a wave
// holds for a whole tile -- the queries of the forward pass, the own rows of the backward pass -- is read by one wave only, once
// a tile, and comes from global memory.
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
__device__ __forceinline__ int chunk_swz(int row) { return (((row >> 1) & 1) << 2) | ((row >> 2) & 3); }
// Rows from `kept` on are zeros: what lies behind a sequence's rows may be anything.  They are read from the last row that is there, so that
// all loads are under way at once: with a branch around each, every one waited for the one before it (one text of 128 positions, 12 heads
// 9.2 -> 5.8 us).
template <int THREADS, int ROWS>
struct Staged {
  static constexpr int N = ROWS * 8 / THREADS;
  static_assert(ROWS * 8 % THREADS == 0 && THREADS % 8 == 0, "whole pieces");
  uint4 v[N];
  __device__ __forceinline__ void load(const bf16_t* __restrict__ src, int ld, int kept) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int row = i * (THREADS / 8) + (threadIdx.x >> 3);
      v[i] = *reinterpret_cast<const uint4*>(src + (uint32_t)(min(row, kept - 1) * ld + (threadIdx.x & 7) * 8));
    }
  }
  __device__ __forceinline__ void store(bf16_t* __restrict__ S, int kept) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int row = i * (THREADS / 8) + (threadIdx.x >> 3);
      const uint32_t m = row < kept ? ~0u : 0u;
      *reinterpret_cast<uint4*>(S + row * AD + ((threadIdx.x & 7) ^ chunk_swz(row)) * 8) = make_uint4(v[i].x & m, v[i].y & m, v[i].z & m, v[i].w & m);
    }
  }
};
struct RowsOperand { bf16x8 k[4]; };   // the four k-steps (of 16 features) of 32 rows
__device__ __forceinline__ RowsOperand rows_operand(const bf16_t* __restrict__ S, int base, int lane) {
  RowsOperand o;
  const int row = base + (lane & 31), s = chunk_swz(row);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) o.k[ks] = *reinterpret_cast<const bf16x8*>(S + row * AD + ((2 * ks + (lane >> 5)) ^ s) * 8);
  return o;
}
__device__ __forceinline__ s16x4 ld_transposed(const bf16_t* __restrict__ S, int e32, int k0, int lane) {
  const int g = lane >> 4, j = lane & 15, row = k0 + 4 * (g >> 1) + (j >> 2), e = e32 + 16 * (g & 1) + 4 * (j & 3);
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(S + row * AD + ((e >> 3) ^ chunk_swz(row)) * 8 + (e & 7)));
}

// X^T-style product tile: acc[32 x 32] = sum_e R[row][e] * C[column][e].  Result lane layout: column = cbase + l%32,
// rows rbase + 8(r/4) + 4(l/32) + r%4 = rbase + tile_row(r) + own_row(l).
__device__ __forceinline__ constexpr int tile_row(int r) { return 8 * (r >> 2) + (r & 3); }
__device__ __forceinline__ int own_row(int lane) { return 4 * (lane >> 5); }
__device__ __forceinline__ f32x16 rows_dot_rows(const RowsOperand& R, const RowsOperand& C) {
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(R.k[ks], C.k[ks], acc, 0, 0, 0);
  return acc;
}

// A tile g^T[64 features][own] to row `row`: lanes 32 apart, which have neighbouring halves of eight features, exchange them first, so that
// each stores 16 bytes of one eight.
__device__ __forceinline__ void store_row(const f32x16 (&g)[2], bf16_t* __restrict__ row, int lane) {
#pragma unroll
  for (int et = 0; et < 2; ++et)
#pragma unroll
    for (int c = 0; c < 4; c += 2) {
      uint32_t p[2][2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int k = 0; k < 2; ++k) p[i][k] = pack_bf16x2(g[et][4 * (c + i) + 2 * k], g[et][4 * (c + i) + 2 * k + 1]);
      const u32x2 x = __builtin_amdgcn_permlane32_swap(p[0][0], p[1][0], false, false), y = __builtin_amdgcn_permlane32_swap(p[0][1], p[1][1], false, false);
      *reinterpret_cast<uint4*>(row + 32 * et + 8 * (c + (lane >> 5))) = make_uint4(x[0], y[0], x[1], y[1]);
    }
}

// exp(x / 8 - m).  The difference comes before the factor of 2^x: with that folded into one multiply-add the rounding of m log2 e, which
// grows with the scores, stays in the result, and from 10^10 on the largest score's own weight is 0 or infinite.
// (A score of NO_WEIGHT gives 0: key 0 of a sequence is always real.  It is put in place of scores and not 0 in place of the result, around
// which the compiler makes a branch.)
constexpr float NO_WEIGHT = -__builtin_inff();
__device__ __forceinline__ float exp_score(float x, float m) { return __expf(fmaf(x, 0.125f, -m)); }

// The rows of sequence b, of which `kept` are there, and its real tokens (keys at positions beyond get no weight).
struct SeqRows { int row0, kept, len; };
template <bool PADDED>
__device__ __forceinline__ SeqRows seq_rows(const int32_t* __restrict__ lens, const RowPlan& plan, int pass, int b, int B, int S) {
  if (!PADDED) return SeqRows{(pass * B + b) * S, S, S};
  const int n = lens[b], r0 = plan.start[b];
  return SeqRows{pass * B * S + r0, plan.start[b + 1] - r0, n < 1 ? 1 : (n > S ? S : n)};
}
// zeros into the rows of the plan that belong to no sequence, 64 columns at `out` of row 0 of the pass
template <int THREADS>
__device__ __forceinline__ void zero_tail(const RowPlan& plan, int B, bf16_t* __restrict__ out, int64_t ld) {
  const int r0 = plan.start[B], n = *plan.rows - r0;
  for (int c = threadIdx.x; c < n * 8; c += THREADS) *reinterpret_cast<uint4*>(out + (int64_t)(r0 + (c >> 3)) * ld + (c & 7) * 8) = make_uint4(0u, 0u, 0u, 0u);
}

// Forward.  A wave owns a tile of 32 queries (S = 64: two of the four waves only stage).  S^T[key][q] tiles leave each lane
// with one query column, so the softmax over keys is an in-lane reduction plus one exchange between the halves, and the
// probability tile is already an operand of the MFMA for O^T[e][q] = sum_key V^T[e][key] P^T[key][q].
// Bound by memory where the heads fill the chip (1024 heads of 128 positions, 67 MB: 22.9 -> 16.2 us, 4.1 TB/s of the 5.9 of a plain copy) and by the
// chain of a tile where they do not (12 padded heads 9.1 -> 6.2, 384 10.7 -> 8.4, 228 padded of 256 positions 14.9 -> 11.9).  What shortened it: no load
// waits for another, masks without branches, stores of 16 bytes, and 128 registers, which let four workgroups share a CU.
// A probability is divided by the row's sum and then rounded to bf16, and a tile's products are added eight keys at a time.  (Divided after the product, by
// the sum of the rounded ones, with 32x32x16 products and one multiply-add for a score, the kernels are 3% faster and the hypergradients of
// deep encoders others: 2% to 10% in the worst of two dozen, most below 0.2%.)
// With a loop over the tiles of a wave, even one that never turns, the 16 NT comparisons of keys with the length are kept as lane
// masks across it, hundreds of scalar registers of which most spill.
template <int NT> struct AttnFwd { static constexpr int WAVES = NT < 8 ? 4 : 8, THREADS = 64 * WAVES, PER_SIMD = NT < 8 ? 4 : 2; };
template <int NT, bool PADDED>   // PADDED = false: no lengths given, the comparisons against len fold away
__global__ __launch_bounds__(AttnFwd<NT>::THREADS, AttnFwd<NT>::PER_SIMD) void k_attn_fwd(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ out, float* __restrict__ lse,
                                                  int heads, int d, const int32_t* __restrict__ lens, RowPlan plan, int B) {
  constexpr int S = 32 * NT, THREADS = AttnFwd<NT>::THREADS;
  static_assert(NT <= AttnFwd<NT>::WAVES, "a tile of queries per wave");
  __shared__ __attribute__((aligned(16))) bf16_t Ks[S * AD];
  __shared__ __attribute__((aligned(16))) bf16_t Vs[S * AD];
  const int h = blockIdx.x, b = blockIdx.y, pass = blockIdx.z, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int ld = 3 * d;
  const SeqRows sr = seq_rows<PADDED>(lens, plan, pass, b, B, S);
  const bf16_t* Q = qkv + (int64_t)sr.row0 * ld + h * AD;
  const int len = sr.len, kept = sr.kept, nk = PADDED ? (len + 31) / 32 : NT, nq = PADDED ? (kept + 31) / 32 : NT;
  const int qt = wave;
  // the queries of a tile are used by one wave only: from global memory, beside the staging
  RowsOperand q;
  {
    const bf16_t* p = Q + (uint32_t)((32 * (qt < nq ? qt : 0) + (lane & 31)) * ld + 8 * (lane >> 5));
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) q.k[ks] = *reinterpret_cast<const bf16x8*>(p + 16 * ks);
  }
  Staged<THREADS, S> k, v;
  k.load(Q + d, ld, kept);
  v.load(Q + 2 * d, ld, kept);
  if (PADDED && b == 0) zero_tail<THREADS>(plan, B, out + (int64_t)pass * B * S * d + h * AD, d);
  k.store(Ks, kept);
  v.store(Vs, kept);
  __syncthreads();
  if (qt >= nq) return;
  f32x16 s[NT];
#pragma unroll
  for (int kt = 0; kt < NT; ++kt)
    if (kt < nk) s[kt] = rows_dot_rows(rows_operand(Ks, 32 * kt, lane), q);   // nk: tiles with a real key
  float mx = NO_WEIGHT;
#pragma unroll
  for (int kt = 0; kt < NT; ++kt)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (PADDED) s[kt][r] = kt < nk && 32 * kt + tile_row(r) < len - own_row(lane) ? s[kt][r] : NO_WEIGHT;
      mx = fmaxf(mx, s[kt][r]);
    }
  mx = join32(mx, [](float a, float b) { return fmaxf(a, b); });
  mx *= 0.125f;
  float sum = 0.f;
#pragma unroll
  for (int kt = 0; kt < NT; ++kt)
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[kt][r] = exp_score(s[kt][r], mx); sum += s[kt][r]; }
  sum = join32(sum, [](float a, float b) { return a + b; });
  const float inv = 1.f / sum;
  if (lane < 32 && lse != nullptr) lse[((int64_t)b * heads + h) * S + 32 * qt + lane] = mx + __logf(sum);
  f32x16 o[2];
#pragma unroll
  for (int et = 0; et < 2; ++et)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[et][r] = 0.f;
#pragma unroll
  for (int kt = 0; kt < NT; ++kt) {
    if (kt >= nk) break;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const s16x4 p = pack4(s[kt][4 * c] * inv, s[kt][4 * c + 1] * inv, s[kt][4 * c + 2] * inv, s[kt][4 * c + 3] * inv);
#pragma unroll
      for (int et = 0; et < 2; ++et) o[et] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(ld_transposed(Vs, 32 * et, 32 * kt + 8 * c, lane), p, o[et], 0, 0, 0);
    }
  }
  if (PADDED && 32 * qt + (lane & 31) >= kept) return;
  store_row(o, out + ((int64_t)sr.row0 + 32 * qt + (lane & 31)) * d + h * AD, lane);
}

// Backward.  Probabilities are recomputed from q, k and the saved log-sum-exp; a wave owns 32 queries or keys at a time.
//   dQ: dS^T[key][q] -> dQ^T[e][q] = sum_key K^T[e][key] dS^T[key][q]
//   dK: dS[q][key]   -> dK^T[e][key] = sum_q Q^T[e][q] dS[q][key]
//   dV: P[q][key]    -> dV^T[e][key] = sum_q dO^T[e][q] P[q][key]
// dS = P (dP - D) / 8 with D[q] = sum_e dO[q][e] O[q][e].
// A workgroup (blockIdx.z) forms one of the three, or (PARTS 2) dQ or the other two: it stages the two matrices it walks over, and
// its waves hold the rows of their own tile and 32 or 64 accumulators.  Bound by the latency of a tile's chain (LDS, product,
// exponentials, product) and by the requests for the rows it stages and holds.
//   Three parts: the scores are formed three times instead of twice, but 4 workgroups share a CU (35 KB of LDS at S = 128, 128
//   registers; 2 of eight waves at S = 256, with 68 KB) where one that formed all three, with 64 KB, had it alone.
//   Two parts: a round of three workgroups to a CU instead of four, with a longer chain each, so only once there are more heads than CUs.  us two / three,
//   heads of 128 positions: 60 9.8 / 7.4, 192 12.8 / 11.8, 252 14.7 / 14.5, 324 17.2 / 17.3, 512 24.0 / 25.7, 1024 49.1 / 54.5; padded 60 8.7 / 8.0, 132 9.6 / 9.2, 252 11.9 /
//   12.8, 384 14.3 / 14.7, 1024 34.1 / 37.0.  At S = 64 the two were equal; at S = 256 the registers left one workgroup to a CU (padded 52 against 47 us).
// No form keeps anything in scratch: of the rows' values four are read at a time, the lane is found anew behind the loops, and S = 64 has three waves to a
// SIMD and 130 registers (padded, with 128 and 20 bytes of scratch, 768 heads 13.7 / 12.1 us, 1536 25.3 / 23.5).
// All staged rows are requested at once and masks take no branch around exponentials and pieces: 384 heads of 128 positions 21.7 -> 18.0 us, padded 21.9 -> 14.6,
// 256 heads 16.6 -> 13.5, 228 padded of 256 28.8 -> 21.7.  (The times below are of kernels before that.)
// A wave has one tile and no loop around it: with one, the padded forms kept lane masks and eight-wave forms values across it in
// scratch (384 heads, S = 128 padded 22.0 -> 20.7 us; S = 256 52 -> 48 us, padded 52 -> 47 us).
// The own rows and D's are fetched behind the staged ones, whose lines they share: ahead of them, with 2 or 32 lines to an
// instruction each, they held those up (384 heads 20.8 -> 24.4 us).
template <int NT, bool PADDED, int PARTS>
__global__ __launch_bounds__(64 * NT, PARTS == 2 || NT == 2 ? 3 : 4) void k_attn_bwd(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ out,
                                                                      const bf16_t* __restrict__ dout, const float* __restrict__ lse,
                                                                      bf16_t* __restrict__ dqkv, int heads, int d, const int32_t* __restrict__ lens,
                                                                      RowPlan plan, int B) {
  constexpr int S = 32 * NT, THREADS = 64 * NT;
  enum { DK = 0, DQ = 1, DV = 2 };   // of two parts the first is both dK and dV
  __shared__ __attribute__((aligned(16))) bf16_t s_r[S * AD];   // dQ: K; dK and dV: Q
  __shared__ __attribute__((aligned(16))) bf16_t s_t[S * AD];   // dQ: V; dK and dV: dO
  __shared__ __attribute__((aligned(16))) float s_D[S], s_lse[S];
  const int h = blockIdx.x, b = blockIdx.y, part = blockIdx.z, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ld = 3 * d;
  const SeqRows sr = seq_rows<PADDED>(lens, plan, 0, b, B, S);
  const int len = sr.len, kept = sr.kept, nk = PADDED ? (len + 31) / 32 : NT, nq = PADDED ? (kept + 31) / 32 : NT;
  const bf16_t* Q = qkv + (int64_t)sr.row0 * ld + h * AD;
  const bf16_t* O = out + (int64_t)sr.row0 * d + h * AD;
  const bf16_t* dO = dout + (int64_t)sr.row0 * d + h * AD;
  // rows 32 tile + lane % 32 of a matrix, as rows_operand() would give them
  auto own_rows = [&](const bf16_t* X, int stride, int tile) {
    RowsOperand o;
    const bf16_t* p = X + (uint32_t)((32 * tile + (lane & 31)) * stride + 8 * (lane >> 5));
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) o.k[ks] = *reinterpret_cast<const bf16x8*>(p + 16 * ks);
    return o;
  };
  Staged<THREADS, S> r, t;
  r.load(part == DQ ? Q + d : Q, ld, kept);
  t.load(part == DQ ? Q + 2 * d : dO, part == DQ ? ld : d, kept);
  // two threads per query
  static_assert(THREADS == 2 * S, "one turn");
  const int dq = threadIdx.x >> 1, dhalf = threadIdx.x & 1;
  const bool with_d = !(PARTS == 3 && part == DV);
  uint4 o4[4], d4[4];
  if (with_d) {
    const uint32_t at = (uint32_t)(min(dq, kept - 1) * d + dhalf * 32);
#pragma unroll
    for (int i = 0; i < 4; ++i) { o4[i] = *reinterpret_cast<const uint4*>(O + at + 8 * i); d4[i] = *reinterpret_cast<const uint4*>(dO + at + 8 * i); }
  }
  const float dlse = lse[((int64_t)b * heads + h) * S + min(dq, kept - 1)];
  if (PADDED && b == 0) {
    zero_tail<THREADS>(plan, B, dqkv + (part == DQ ? 0 : (part == DK ? d : 2 * d)) + h * AD, ld);
    if (PARTS == 2 && part != DQ) zero_tail<THREADS>(plan, B, dqkv + 2 * d + h * AD, ld);
  }
  r.store(s_r, kept);
  t.store(s_t, kept);
  float D = 0.f;
  if (with_d) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t ow[4] = {o4[i].x, o4[i].y, o4[i].z, o4[i].w}, dw[4] = {d4[i].x, d4[i].y, d4[i].z, d4[i].w};
#pragma unroll
      for (int e = 0; e < 8; ++e)
        D = fmaf(bf16_to_f32((bf16_t)(ow[e >> 1] >> ((e & 1) * 16))), bf16_to_f32((bf16_t)(dw[e >> 1] >> ((e & 1) * 16))), D);
    }
    D += __shfl_xor(D, 1, 64);
  }
  if (dhalf == 0) { s_D[dq] = D * 0.125f; s_lse[dq] = dlse; }   // of rows that are not there: not used
  __syncthreads();

  if (wave >= nq) return;                                          // a wave owns a tile of queries (dQ) or keys
  const int own = wave;
  f32x16 g[2], gv[2];                                            // dQ, or dK and dV
#pragma unroll
  for (int et = 0; et < 2; ++et)
#pragma unroll
    for (int r = 0; r < 16; ++r) g[et][r] = gv[et][r] = 0.f;
  const int col = 32 * own + (lane & 31);                        // this lane's query or key
  // g^T[e][own] += sum over the 32 rows of `tile` of T^T[e][row] w[row][own]
  auto accumulate = [&](f32x16 (&g)[2], const bf16_t* T, int tile, const f32x16& w) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const s16x4 wb = pack4(w[4 * c], w[4 * c + 1], w[4 * c + 2], w[4 * c + 3]);
#pragma unroll
      for (int et = 0; et < 2; ++et)
        g[et] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(ld_transposed(T, 32 * et, 32 * tile + 8 * c, lane), wb, g[et], 0, 0, 0);
    }
  };
  // of a lane's rows 8 c .. 8 c + 3 in a tile of queries (four at a time: all sixteen of both values took registers that there were not)
  auto of_queries = [&](const float* x, int qt, int c) { return *reinterpret_cast<const f32x4*>(x + 32 * qt + own_row(lane) + 8 * c); };
  auto there = [&](int r, int qt) { return !PADDED || tile_row(r) < kept - own_row(lane) - 32 * qt; };
  if (part == DQ) {
    const float lq = s_lse[col], Dq = s_D[col];
    const RowsOperand qop = own_rows(Q, ld, own), dop = own_rows(dO, d, own);
#pragma unroll 1
    for (int kt = 0; kt < nk; ++kt) {
      f32x16 st = rows_dot_rows(rows_operand(s_r, 32 * kt, lane), qop);          // S^T[key][q]
      const f32x16 dp = rows_dot_rows(rows_operand(s_t, 32 * kt, lane), dop);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (PADDED) st[r] = tile_row(r) < len - own_row(lane) - 32 * kt ? st[r] : NO_WEIGHT;
        st[r] = exp_score(st[r], lq) * fmaf(dp[r], 0.125f, -Dq);                 // dS^T
      }
      accumulate(g, s_r, kt, st);
    }
  } else if (PARTS == 3 && part == DV) {
    if (own < nk) {
      const RowsOperand kop = own_rows(Q + d, ld, own);
#pragma unroll 1
      for (int qt = 0; qt < nq; ++qt) {
        f32x16 st = rows_dot_rows(rows_operand(s_r, 32 * qt, lane), kop);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const f32x4 l = of_queries(s_lse, qt, c);
#pragma unroll
          for (int r = 4 * c; r < 4 * c + 4; ++r) st[r] = exp_score(there(r, qt) ? st[r] : NO_WEIGHT, l[r & 3]);
        }
        accumulate(g, s_t, qt, st);
      }
    }
  } else if (own < nk) {                                         // otherwise keys without weight
    const RowsOperand kop = own_rows(Q + d, ld, own), vop = own_rows(Q + 2 * d, ld, own);
#pragma unroll 1
    for (int qt = 0; qt < nq; ++qt) {
      f32x16 st = rows_dot_rows(rows_operand(s_r, 32 * qt, lane), kop);          // S[q][key]
      f32x16 dp = rows_dot_rows(rows_operand(s_t, 32 * qt, lane), vop);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const f32x4 l = of_queries(s_lse, qt, c), D8 = of_queries(s_D, qt, c);
#pragma unroll
        for (int r = 4 * c; r < 4 * c + 4; ++r) {
          st[r] = exp_score(there(r, qt) ? st[r] : NO_WEIGHT, l[r & 3]);         // P
          dp[r] = st[r] * fmaf(dp[r], 0.125f, -D8[r & 3]);                       // dS
        }
      }
      if constexpr (PARTS == 2) accumulate(gv, s_t, qt, st);
      accumulate(g, s_r, qt, dp);
    }
  }
  const int lane_now = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), col_now = 32 * own + (lane_now & 31);   // not kept over the loops
  if (PADDED && part != DQ && col_now >= len) {                  // a key without weight
#pragma unroll
    for (int et = 0; et < 2; ++et)
#pragma unroll
      for (int r = 0; r < 16; ++r) g[et][r] = gv[et][r] = 0.f;
  }
  if (PADDED && col_now >= kept) return;
  auto store = [&](const f32x16 (&g)[2], int to) {   // to: where the result goes among the columns of dqkv
    store_row(g, dqkv + ((int64_t)sr.row0 + col_now) * ld + to + h * AD, lane_now);
  };
  store(g, part == DQ ? 0 : (part == DK ? d : 2 * d));
  if (PARTS == 2 && part != DQ) store(gv, 2 * d);
}

// =========================================================================================== classifier head
// Blocks [0, wblocks): dWc, dbc; the others: rows of dx, dlogits[b] . Wc at row b S (or start[b]) and, without `start`, zeros in
// the rows in between and up to `rows`.  Bound by the launch: one instead of three (fill, weights, rows), 19.4 -> 5.3 us for 32
// samples of 768.
__global__ __launch_bounds__(256) void k_head_bwd(const float* __restrict__ x, int S, const int32_t* __restrict__ start, int d, int B, int C,
                                                  const float* __restrict__ dlogits, const float* __restrict__ Wc, float* __restrict__ gWc,
                                                  float* __restrict__ gbc, float* __restrict__ dx, int rows, int wblocks) {
  if ((int)blockIdx.x < wblocks) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < C * d) {
      const int c = i / d, k = i - c * d;
      float s = 0.f;
#pragma unroll 8
      for (int b = 0; b < B; ++b) s = fmaf(dlogits[b * C + c], x[(int64_t)(start != nullptr ? start[b] : b * S) * d + k], s);
      gWc[i] = s;
    }
    if (i < C) {
      float s = 0.f;
#pragma unroll 8
      for (int b = 0; b < B; ++b) s += dlogits[b * C + i];
      gbc[i] = s;
    }
    return;
  }
  const int64_t i = (int64_t)(blockIdx.x - wblocks) * 256 + threadIdx.x;
  const int r = (int)(i / d), k = (int)(i - (int64_t)r * d);
  if (start != nullptr) {
    if (r >= B) return;
    float s = 0.f;
    for (int c = 0; c < C; ++c) s = fmaf(dlogits[r * C + c], Wc[(int64_t)c * d + k], s);
    dx[(int64_t)start[r] * d + k] = s;
    return;
  }
  if (r >= rows) return;
  float s = 0.f;
  if (r % S == 0 && r / S < B)
    for (int c = 0; c < C; ++c) s = fmaf(dlogits[(r / S) * C + c], Wc[(int64_t)c * d + k], s);
  dx[i] = s;
}

// =========================================================================================== rows that are read
__global__ __launch_bounds__(256) void k_select_rows(RowSelect s, int pass_rows, int d, const bf16_t* __restrict__ a16,
                                                     const float* __restrict__ x32, bf16_t* __restrict__ a16_out, float* __restrict__ x32_out) {
  const int r = selected_row(s, blockIdx.x), nq = d >> 2;
  const int64_t from = (int64_t)blockIdx.y * pass_rows + max(r, 0), to = (int64_t)blockIdx.y * s.n + blockIdx.x;
  for (int q = threadIdx.x; q < nq; q += 256) {
    reinterpret_cast<uint2*>(a16_out + to * d)[q] = r >= 0 ? reinterpret_cast<const uint2*>(a16 + from * d)[q] : make_uint2(0u, 0u);
    if (x32 != nullptr)
      reinterpret_cast<float4*>(x32_out + to * d)[q] = r >= 0 ? reinterpret_cast<const float4*>(x32 + from * d)[q] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
}
__global__ __launch_bounds__(256) void k_spread_rows(RowSelect s, RowPlan plan, int d, const bf16_t* __restrict__ a16, const float* __restrict__ x32,
                                                     bf16_t* __restrict__ a16_out, float* __restrict__ x32_out) {
  const int64_t to = blockIdx.x;
  if (plan.rows != nullptr && (int)blockIdx.x >= *plan.rows) return;
  const int o = plan.src != nullptr ? plan.src[blockIdx.x] : (int)blockIdx.x;
  const int b = o / s.S, p = o % s.S, nq = d >> 2;
  const bool kept = o >= 0 && p < SELECT_SEQ_ROWS;
  const int64_t from = kept ? b * SELECT_SEQ_ROWS + p : 0;
  for (int q = threadIdx.x; q < nq; q += 256) {
    reinterpret_cast<uint2*>(a16_out + to * d)[q] = kept ? reinterpret_cast<const uint2*>(a16 + from * d)[q] : make_uint2(0u, 0u);
    reinterpret_cast<float4*>(x32_out + to * d)[q] = kept ? reinterpret_cast<const float4*>(x32 + from * d)[q] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
}

// =========================================================================================== embedding gradients
// A block per position m and TOK_COLS columns.  The block lists, in ascending order, every position holding the same token id;
// only those of the first occurrence go on, and write the ordered sum of those rows.  What bounds it is the most frequent
// id (position 0 of every sequence, the head of the Zipf law: hundreds of rows), a serial chain of fetches and what one CU takes in: so its
// columns are spread over workgroups, and TOK_AHEAD rows are fetched together, without a branch between them (the list goes
// on with its last entry, which counts as zeros), and added in list order.  Such ids are seen early: the positions from TOK_SPLIT
// on have one block for all columns, since every block looks through all positions (three for each of 4096: 41 us).
// With the position gradients, all columns and 8 rows together -> now: 4096 positions of 768, 62 -> 24 us, 8192 118 -> 59, 2048 of
// 1024 24 -> 14, 4096 of 256 26 -> 23.
constexpr int TOK_COLS = 256, TOK_AHEAD = 64, TOK_SPLIT = 512, TOK_SCAN = 4;   // TOK_SCAN x 256 positions are looked at together
template <int R>   // rows fetched together
__device__ __forceinline__ void tok_rows(const float* __restrict__ demb, const uint16_t* __restrict__ list, int cnt, int d, int c, float* __restrict__ out) {
  const float* const col = demb + min(c, d - 1);
  float s = 0.f;
  for (int i = 0; i < cnt; i += R) {   // behind the end: zeros, which change no sum
    float v[R];
#pragma unroll
    for (int u = 0; u < R; u += 8) {
      const uint4 l = *reinterpret_cast<const uint4*>(list + i + u);
      const uint32_t w[4] = {l.x, l.y, l.z, l.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) v[u + e] = col[(int64_t)(w[e >> 1] >> (16 * (e & 1)) & 0xffffu) * d];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < R; ++u) s += i + u < cnt ? v[u] : 0.f;
  }
  if (c < d) out[c] = s;
}
__device__ __forceinline__ void tok_grad(const float* __restrict__ demb, const int32_t* __restrict__ ids, int m, int M, int c0, int c1, int d, int V,
                                         float* __restrict__ g_tok) {
  __shared__ __attribute__((aligned(16))) uint16_t s_list[MAX_TOKENS + TOK_AHEAD];
  static_assert(MAX_TOKENS <= 65536, "positions in 16 bits");
  __shared__ int s_wave[TOK_SCAN][4], s_earlier[4];
  const int id = min(max(ids[m], 0), V - 1), lane = threadIdx.x & 63, wave = threadIdx.x >> 6;   // clamped as in the forward pass
  int cnt = 0;
  for (int base = 0; base < M; base += 256 * TOK_SCAN) {
    int there[TOK_SCAN];
#pragma unroll
    for (int g = 0; g < TOK_SCAN; ++g) there[g] = ids[min(base + 256 * g + (int)threadIdx.x, M - 1)];
    unsigned long long hits[TOK_SCAN], earlier = 0;
#pragma unroll
    for (int g = 0; g < TOK_SCAN; ++g) {
      const int mm = base + 256 * g + threadIdx.x;
      hits[g] = __ballot(mm < M && min(max(there[g], 0), V - 1) == id);
      earlier |= hits[g] & __ballot(mm < m);
      if (lane == 0) s_wave[g][wave] = __popcll(hits[g]);
    }
    if (lane == 0) s_earlier[wave] = earlier != 0;
    __syncthreads();
    if (s_earlier[0] | s_earlier[1] | s_earlier[2] | s_earlier[3]) return;   // an earlier position holds this id
    int off = cnt;
#pragma unroll
    for (int g = 0; g < TOK_SCAN; ++g) {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (w == wave && (hits[g] >> lane & 1)) s_list[min(off + (int)__popcll(hits[g] & ((1ull << lane) - 1ull)), MAX_TOKENS - 1)] = (uint16_t)(base + 256 * g + threadIdx.x);
        off += s_wave[g][w];
      }
    }
    cnt = off;
    __syncthreads();
  }
  if (threadIdx.x < TOK_AHEAD) s_list[cnt + threadIdx.x] = s_list[cnt - 1];   // m itself is listed
  __syncthreads();
  float* out = g_tok + (int64_t)id * d;
  for (int c = c0 + threadIdx.x; c < c1; c += TOK_COLS) {
    if (cnt <= 8) tok_rows<8>(demb, s_list, cnt, d, c, out);
    else tok_rows<TOK_AHEAD>(demb, s_list, cnt, d, c, out);
  }
}
// Blocks [0, pblocks): position gradients; the others: TOK_COLS columns of a token position each.
__global__ __launch_bounds__(256) void k_embedding_grad(const float* __restrict__ demb, const int32_t* __restrict__ ids, int B, int S, int d, int V,
                                                        RowPlan plan, int pblocks, float* __restrict__ g_tok, float* __restrict__ g_pos) {
  if ((int)blockIdx.x >= pblocks) {
    const int M = plan.start != nullptr ? plan.start[B] : B * S, k = blockIdx.x - pblocks, chunks = (d + TOK_COLS - 1) / TOK_COLS;
    const int split = min(B * S, TOK_SPLIT);
    const bool all = k >= split * chunks;
    const int m = all ? k - split * chunks + split : k / chunks, c0 = all ? 0 : (k - m * chunks) * TOK_COLS;
    if (m < M) tok_grad(demb, plan.ids != nullptr ? plan.ids : ids, m, M, c0, all ? d : min(c0 + TOK_COLS, d), d, V, g_tok);
    return;
  }
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= S * d) return;
  float s = 0.f;
  if (plan.start == nullptr) {
#pragma unroll 8
    for (int b = 0; b < B; ++b) s += demb[(int64_t)b * S * d + i];
  } else {
    const int pos = i / d;
#pragma unroll 4
    for (int b = 0; b < B; ++b)
      if (pos < plan.start[b + 1] - plan.start[b]) s += demb[(int64_t)plan.start[b] * d + i];
  }
  g_pos[i] = s;
}
}  // namespace

void launch_ln_fwd(hipStream_t st, const LnFwdArgs& a) {
  ProfScope ps(st, F_LN_FWD, 6.0 * a.M * a.d);
  const int blocks = (a.M + 3) / 4 + (a.ahead.n > 0 ? AHEAD_BLOCKS : 0);
  if (a.d <= 1024) launch_kernel(ps, k_ln_fwd<4>, blocks, 256, 0, st, a);
  else launch_kernel(ps, k_ln_fwd<8>, blocks, 256, 0, st, a);
}
void launch_ln_bwd(hipStream_t st, const LnBwdArgs& a) {
  ProfScope ps(st, F_LN_BWD, 14.0 * a.M * a.d);
  const int blocks = (a.M + LN_BWD_ROWS - 1) / LN_BWD_ROWS + (a.ahead.n > 0 ? AHEAD_BLOCKS : 0);
  if (a.d <= 1024) launch_kernel(ps, k_ln_bwd<4>, blocks, 64 * LN_BWD_ROWS, 0, st, a);
  else launch_kernel(ps, k_ln_bwd<8>, blocks, 64 * LN_BWD_ROWS, 0, st, a);
}
void launch_reduce_rows_multi(hipStream_t st, const ReduceRowsJob* jobs, int count) {
  ReduceRowsMulti m{};
  m.count = count;
  int nb = 0;
  double bytes = 0.0;
  for (int k = 0; k < count; ++k) {
    m.j[k] = jobs[k];
    m.first_block[k] = nb;
    const int nv = jobs[k].out[2] ? 3 : (jobs[k].out[1] ? 2 : 1);
    nb += ((jobs[k].N + 31) / 32) * nv;
    bytes += 4.0 * jobs[k].nrows * jobs[k].N * nv;
  }
  for (int k = count; k <= REDUCE_MAX_JOBS; ++k) m.first_block[k] = nb;
  ProfScope ps(st, F_OTHER, bytes);
  launch_kernel(ps, k_reduce_rows, nb, 256, 0, st, m);
}
void launch_reduce_rows(hipStream_t st, const float* partial, int nrows, int64_t stride, int64_t vstride, int N, float* out0,
                        float* out1, float* out2) {
  const ReduceRowsJob j{partial, nrows, stride, vstride, N, {out0, out1, out2}};
  launch_reduce_rows_multi(st, &j, 1);
}
void launch_colsum_partial_multi(hipStream_t st, const ColsumJob* jobs, int count) {
  ColsumMulti m{};
  m.count = count;
  int nb = 0;
  double bytes = 0.0;
  for (int k = 0; k < count; ++k) {
    m.j[k] = jobs[k];
    m.first_block[k] = nb;
    nb += ((jobs[k].N + 2047) / 2048) * ((jobs[k].M + COLSUM_ROWS - 1) / COLSUM_ROWS);
    bytes += 2.0 * jobs[k].M * jobs[k].N;
  }
  for (int k = count; k < 3; ++k) m.first_block[k] = nb;
  ProfScope ps(st, F_OTHER, bytes);
  launch_kernel(ps, k_colsum_partial_bf16, nb, 256, 0, st, m);
}
void launch_colsum_bf16(hipStream_t st, const bf16_t* X, int M, int N, float* partial, float* out) {
  const int nrb = (M + COLSUM_ROWS - 1) / COLSUM_ROWS;
  const ColsumJob j{X, M, N, partial};
  launch_colsum_partial_multi(st, &j, 1);
  launch_reduce_rows(st, partial, nrb, N, 0, N, out, nullptr, nullptr);
}
// (S = 32 would fit the kernels, but the weight-gradient GEMMs contract over batch * S token rows in slabs of 64)
bool attention_supports(int S) { return S == 64 || S == 128 || S == 256; }
void launch_attention_fwd(hipStream_t st, const bf16_t* qkv, bf16_t* out, float* lse, int nw, int B, int S, int heads, int d,
                          const int32_t* lens, const RowPlan& plan) {
  ProfScope ps(st, F_ATTN_FWD, 4.0 * nw * B * heads * (double)S * S * 64.0);
  const dim3 grid(heads, B, nw);
  switch (S) {
    case 64:
      if (lens) launch_kernel(ps, k_attn_fwd<2, true>, grid, AttnFwd<2>::THREADS, 0, st, qkv, out, lse, heads, d, lens, plan, B);
      else launch_kernel(ps, k_attn_fwd<2, false>, grid, AttnFwd<2>::THREADS, 0, st, qkv, out, lse, heads, d, lens, plan, B);
      break;
    case 128:
      if (lens) launch_kernel(ps, k_attn_fwd<4, true>, grid, AttnFwd<4>::THREADS, 0, st, qkv, out, lse, heads, d, lens, plan, B);
      else launch_kernel(ps, k_attn_fwd<4, false>, grid, AttnFwd<4>::THREADS, 0, st, qkv, out, lse, heads, d, lens, plan, B);
      break;
    case 256:
      if (lens) launch_kernel(ps, k_attn_fwd<8, true>, grid, AttnFwd<8>::THREADS, 0, st, qkv, out, lse, heads, d, lens, plan, B);
      else launch_kernel(ps, k_attn_fwd<8, false>, grid, AttnFwd<8>::THREADS, 0, st, qkv, out, lse, heads, d, lens, plan, B);
      break;
    default: break;   // make_encoder admits no other length
  }
}
void launch_attention_bwd(hipStream_t st, const bf16_t* qkv, const bf16_t* out, const bf16_t* dout, const float* lse,
                          bf16_t* dqkv, int B, int S, int heads, int d, const int32_t* lens, const RowPlan& plan) {
  ProfScope ps(st, F_ATTN_BWD, 10.0 * B * heads * (double)S * S * 64.0);
  auto launch = [&](auto tiles, auto parts) {
    constexpr int NT = decltype(tiles)::value, PARTS = decltype(parts)::value;
    auto kernel = lens ? k_attn_bwd<NT, true, PARTS> : k_attn_bwd<NT, false, PARTS>;
    launch_kernel(ps, kernel, dim3(heads, B, PARTS), 64 * NT, 0, st, qkv, out, dout, lse, dqkv, heads, d, lens, plan, B);
  };
  const std::integral_constant<int, 2> two;
  const std::integral_constant<int, 3> three;
  switch (S) {
    case 64: launch(two, three); break;
    case 128: (int64_t)heads * B > 256 ? launch(std::integral_constant<int, 4>(), two) : launch(std::integral_constant<int, 4>(), three); break;
    case 256: launch(std::integral_constant<int, 8>(), three); break;
    default: break;
  }
}
void launch_head_bwd(hipStream_t st, const float* x, int S, const int32_t* start, int d, int B, int C, const float* theta, int64_t wc_off,
                     int64_t bc_off, const float* dlogits, float* grad, float* dx, int rows) {
  ProfScope ps(st, F_OTHER, 0.0);
  if (start != nullptr) launch_fill_f32(st, dx, 0.f, (int64_t)rows * d);
  const int wblocks = (C * d + 255) / 256, xblocks = (int)(((int64_t)(start != nullptr ? B : rows) * d + 255) / 256);
  launch_kernel(ps, k_head_bwd, wblocks + xblocks, 256, 0, st, x, S, start, d, B, C, dlogits, theta + wc_off, grad + wc_off, grad + bc_off, dx, rows, wblocks);
}
void launch_row_plan(hipStream_t st, const int32_t* ids, const int32_t* lens, int B, int S, const RowSelect& sel, const RowPlan& out) {
  ProfScope ps(st, F_OTHER, 16.0 * B * S);
  launch_kernel(ps, k_row_plan, (B * S + 255) / 256, 256, 0, st, ids, lens, B, S, sel, out);
}
void launch_select_rows(hipStream_t st, const RowSelect& s, int nw, int pass_rows, int d, const bf16_t* a16, const float* x32,
                        bf16_t* a16_out, float* x32_out) {
  ProfScope ps(st, F_OTHER, 12.0 * nw * s.n * d);
  launch_kernel(ps, k_select_rows, dim3(s.n, nw), 256, 0, st, s, pass_rows, d, a16, x32, a16_out, x32_out);
}
void launch_spread_rows(hipStream_t st, const RowSelect& s, const RowPlan& plan, int M, int d, const bf16_t* a16, const float* x32, bf16_t* a16_out, float* x32_out) {
  ProfScope ps(st, F_OTHER, 6.0 * (M + s.n) * d);
  launch_kernel(ps, k_spread_rows, M, 256, 0, st, s, plan, d, a16, x32, a16_out, x32_out);
}
void launch_embedding_bwd(hipStream_t st, const float* demb, const int32_t* ids, int B, int S, int d, int V, float* g_tok, float* g_pos,
                          const RowPlan& plan) {
  ProfScope ps(st, F_OTHER, 4.0 * B * S * d);
  const int pblocks = (S * d + 255) / 256;
  launch_kernel(ps, k_embedding_grad, pblocks + B * S + std::min(B * S, TOK_SPLIT) * ((d + TOK_COLS - 1) / TOK_COLS - 1), TOK_COLS, 0, st, demb, ids, B, S, d, V, plan, pblocks, g_tok, g_pos);
}

}  // namespace sama
