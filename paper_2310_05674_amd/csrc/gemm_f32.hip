// fp32 contraction for the fp32 base learners (logistic regression, small MLPs): forward, dgrad and wgrad of a
// linear layer are the same kernel with different strides.  The matrix cores are used in their fp32 form
// (v_mfma_f32_16x16x4_f32), so results carry plain fp32 rounding.  Shapes are arbitrary: rows
// beyond an operand's are clamped, contraction indices beyond the end read as zeros.
//
// These problems are tiny (a batch of 128 rows, a few hundred columns) and latency-bound, so the kernel is built for
// short dependency chains rather than for reuse: a workgroup owns one output tile, its eight waves split the
// contraction between them in interleaved chunks of 16 and fetch their operands from global memory straight into the
// MFMA operand layout (lane (r, q) holds row r and the four contraction indices 4q .. 4q+3 of a chunk) -- no LDS staging, no
// barrier inside the loop, FDEPTH chunks of loads in flight ahead of the MFMAs.  The eight partial tiles are added in wave order
// through LDS, so the result does not depend on timing.  Forward products that fill the chip have no chain to shorten; they go through
// LDS, a wave with the whole contraction (k_gemm_f32_lds), and add in the same order.
// Loads are as wide as the storage allows, whatever the alignment (gfx950 takes a 16-byte load at any float): along the
// contraction index 16 bytes, across the rows the two or four that a lane's tiles need of one index; and the loop has
// no branches that depend on the operands' edges: rows are clamped, and the chunk that is not whole is apart.  us for rows x
// columns x contraction, against scalar loads for odd widths and strided operands, every load behind its own bounds check:
// 203 x 173 x 301 6.1 -> 3.7, 1500 x 173 x 301 14.3 -> 8.2, 2048 x 256 x 784 16.8 -> 14.0, 128 x 256 x 784 5.7 -> 5.0, both gradients of
// a layer of 320 x 1024 over 512 rows 20.1 -> 16.1; over 150 products and pairs 1.37 times as fast (geometric mean).
//
// Independent problems share a launch (a layer's weight gradient with its column sums and its input gradient; the + and
// the - pass of Eq. 5): a dependent launch costs ~4 us here, more than most of these products.
// The +-eps v passes read the weight operand as B + s * Bv (s = +-eps from device memory), so no perturbed copy of theta
// is ever written.
#include "common.h"
#include "kernels.h"
#include "mfma_f32.h"
#include "solver.h"

namespace sama {
namespace {

// what a product is of a layer by the storage of its operands: both with the contraction index the contiguous one, only A, neither
enum { F32_FORWARD, F32_DGRAD, F32_WGRAD };
int storage_of(const GemmF32Args& a) {   // -1: none of them (a matrix of one column is of either kind)
  if (a.rowsum == nullptr && a.sa_k == 1 && a.sb_k == 1) return F32_FORWARD;
  if (a.Bv != nullptr || a.sb_j != 1) return -1;
  if (a.rowsum == nullptr && a.sa_k == 1) return F32_DGRAD;
  return a.sa_i == 1 ? F32_WGRAD : -1;
}
static_assert(GEMM_F32_MAX_JOBS == 2, "one or two problems");
struct GemmF32Batch { GemmF32Args j[2]; int blocks[2], storage[2]; };   // blocks: multiples of 8; none of a problem that is not there

// How an operand lies: a row's contraction indices side by side, or (an operand of a weight gradient, the weights of an input
// gradient) the rows at one contraction index.  A lane's X tiles of 16 rows are then rows r, 16 + r, ... or, of the second kind,
// the X adjacent rows X r .. X r + X - 1, so that one load has them all.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // a vector load wants no more than a float's alignment
typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
template <int X, bool KC>
__device__ __forceinline__ int tile_row(int x, int r) { return KC ? 16 * x + r : X * r + x; }

// Of one operand the chunk of contraction indices k .. k + 3 (k: this lane's first): v[x][c] is row `row(x)` at index k + c.
template <int X, bool KC, bool FULL>
struct F32Operand {
  const float* p[KC || !FULL ? X : 1];   // rows beyond the end are clamped: their products are never stored
  int64_t s_k;
  __device__ __forceinline__ void init(const float* base, int64_t s_row, int64_t s_k_, int row0, int nrows, int r) {
    s_k = s_k_;
#pragma unroll
    for (int x = 0; x < (KC || !FULL ? X : 1); ++x) p[x] = base + (int64_t)min(row0 + tile_row<X, KC>(x, r), nrows - 1) * s_row;
  }
  __device__ __forceinline__ void load(int k, float4v (&v)[X]) const {
    if constexpr (KC) {
#pragma unroll
      for (int x = 0; x < X; ++x) v[x] = *reinterpret_cast<const f4u*>(p[x] + k);
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int64_t o = (int64_t)(k + c) * s_k;
        if constexpr (FULL && X == 4) {
          const f4u t = *reinterpret_cast<const f4u*>(p[0] + o);
#pragma unroll
          for (int x = 0; x < X; ++x) v[x][c] = t[x];
        } else if constexpr (FULL && X == 2) {
          const f2u t = *reinterpret_cast<const f2u*>(p[0] + o);
          v[0][c] = t[0]; v[X - 1][c] = t[1];
        } else {
#pragma unroll
          for (int x = 0; x < X; ++x) v[x][c] = p[x][o];
        }
      }
    }
  }
  // zeros from K on
  __device__ __forceinline__ void load_tail(int k, int K, float4v (&v)[X]) const {
#pragma unroll
    for (int x = 0; x < X; ++x)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int64_t kk = min(k + c, K - 1);
        const float t = KC ? p[x][kk] : FULL ? p[0][kk * s_k + x] : p[KC || !FULL ? x : 0][kk * s_k];
        v[x][c] = k + c < K ? t : 0.f;
      }
  }
};

// XM x XN output tiles of 16 x 16 per workgroup; FDEPTH chunks in flight per wave.  FULL: all rows of an operand that is not KC exist.
// PV: B is perturbed.
template <int XM, int XN, int FDEPTH, bool A_KC, bool B_KC, bool FULL, bool PV>
__device__ __forceinline__ void gemm_f32_tile(const GemmF32Args& a, int i0, int j0, float bscale, float* __restrict__ red_, float* __restrict__ rsum_) {
  constexpr int TM = 16 * XM, TN = 16 * XN;
  float (*red)[TM][TN + 1] = reinterpret_cast<float (*)[TM][TN + 1]>(red_);
  float (*rsum)[TM] = reinterpret_cast<float (*)[TM]>(rsum_);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, q = lane >> 4;
  const bool rows = !A_KC && a.rowsum != nullptr && j0 == 0;   // this workgroup also sums its rows of A over the contraction
  F32Operand<XM, A_KC, FULL> oa;
  F32Operand<XN, B_KC, FULL> ob, ov;
  oa.init(a.A, a.sa_i, a.sa_k, i0, a.M, r);
  ob.init(a.B, a.sb_j, a.sb_k, j0, a.N, r);
  if (PV) ov.init(a.Bv, a.sb_j, a.sb_k, j0, a.N, r);

  float4v acc[XM][XN];
  float rs[XM];
#pragma unroll
  for (int x = 0; x < XM; ++x) {
    rs[x] = 0.f;
#pragma unroll
    for (int y = 0; y < XN; ++y) acc[x][y] = (float4v){0.f, 0.f, 0.f, 0.f};
  }
  float4v av[FDEPTH][XM], bv[FDEPTH][XN], pv[PV ? FDEPTH : 1][XN];
  // chunks wave, wave + FWAVES, ... of those that are whole
  constexpr int STEP = FWAVES * FCH;
  const int nfull = a.K / FCH, n = nfull > wave ? (nfull - wave + FWAVES - 1) / FWAVES : 0, k_lane = wave * FCH + 4 * q;
  auto fetch = [&](int i, int u) {   // the i-th of them
    oa.load(k_lane + i * STEP, av[u]);
    ob.load(k_lane + i * STEP, bv[u]);
    if constexpr (PV) ov.load(k_lane + i * STEP, pv[u]);
  };
  auto multiply = [&](const float4v (&av)[XM], float4v (&bv)[XN], const float4v (&pv)[XN]) {
    if constexpr (PV) {
#pragma unroll
      for (int y = 0; y < XN; ++y)
#pragma unroll
        for (int c = 0; c < 4; ++c) bv[y][c] = fmaf(bscale, pv[y][c], bv[y][c]);
    }
    if (rows) {
#pragma unroll
      for (int x = 0; x < XM; ++x) rs[x] += (av[x][0] + av[x][1]) + (av[x][2] + av[x][3]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int x = 0; x < XM; ++x)
#pragma unroll
        for (int y = 0; y < XN; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[x][c], bv[y][c], acc[x][y], 0, 0, 0);
  };
  auto use = [&](int u) { multiply(av[u], bv[u], pv[PV ? u : 0]); };
  // FDEPTH chunks are in flight; a buffer's next chunk is requested as soon as its last one has been used.  (No load is conditional
  // in the loop: the waits count loads.)  What is left of the contraction is the last chunk of its wave, and requested first.
  const bool tail = a.K % FCH != 0 && nfull % FWAVES == wave;
  float4v at[XM], bt[XN], pt[XN];
  if (tail) {
    const int k = nfull * FCH + 4 * q;
    oa.load_tail(k, a.K, at);
    ob.load_tail(k, a.K, bt);
    if constexpr (PV) ov.load_tail(k, a.K, pt);
  }
  if (FDEPTH < 8 && n >= FDEPTH) {
#pragma unroll
    for (int u = 0; u < FDEPTH; ++u) fetch(u, u);
    int i = 0;
    for (; i + 2 * FDEPTH <= n; i += FDEPTH) {
#pragma unroll
      for (int u = 0; u < FDEPTH; ++u) { use(u); fetch(i + FDEPTH + u, u); }
    }
#pragma unroll
    for (int u = 0; u < FDEPTH; ++u) {
      use(u);
      if (i + FDEPTH + u < n) fetch(i + FDEPTH + u, u);
    }
#pragma unroll
    for (int u = 0; u < FDEPTH; ++u)
      if (i + FDEPTH + u < n) use(u);
  } else {
    for (int i = 0; i < n; i += FDEPTH) {
#pragma unroll
      for (int u = 0; u < FDEPTH; ++u)
        if (i + u < n) fetch(i + u, u);
#pragma unroll
      for (int u = 0; u < FDEPTH; ++u)
        if (i + u < n) use(u);
    }
  }
  if (tail) multiply(at, bt, pt);
  // partial tiles -> LDS, added in wave order
#pragma unroll
  for (int x = 0; x < XM; ++x) {
#pragma unroll
    for (int y = 0; y < XN; ++y)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[wave][tile_row<XM, A_KC>(x, 4 * q + e)][tile_row<XN, B_KC>(y, r)] = acc[x][y][e];
    if (rows) {
      const auto add = [](float s, float t) { return s + t; };
      const float s = join32(join16(rs[x], add), add);
      if (q == 0) rsum[wave][tile_row<XM, A_KC>(x, r)] = s;
    }
  }
}

// a = second ? b : a, both read: an index into the kernel's arguments that is computed first costs another trip to them, 0.2 us
// (128 x 256 x 784: 4.95 us; with the index 5.27)
template <typename T>
__device__ __forceinline__ void pick(T& a, T b, bool second) {
  asm("" : "+s"(a));
  asm("" : "+s"(b));
  a = second ? b : a;
}

// What the update of an element reads, and the update.
struct Element { float m, v, t; };
__device__ __forceinline__ Element state_of(const BaseUpdate& u, int64_t k) {
  return Element{u.solver == 1 || u.mu != 0.f ? u.m[k] : 0.f, u.solver == 1 ? u.v[k] : 0.f, u.theta[k]};
}
__device__ __forceinline__ void update(const BaseUpdate& u, int64_t k, float g, Element s, bool store_g) {
  const float ge = fmaf(u.wd, s.t, g);
  if (store_g || u.wd != 0.f) u.g[k] = ge;   // the gradient the solver was given, kept for the adaptation
  if (u.solver == 1) {
    adam_one(ge, s.m, s.v, s.t, u.adam);
    u.v[k] = s.v;
  } else {
    sgd_one(ge, s.m, s.t, u.lr, u.mu);
  }
  if (u.solver == 1 || u.mu != 0.f) u.m[k] = s.m;
  u.theta[k] = s.t;
}
struct NoUpdate {};

// PAIR: there are two problems.  UPDATE: a BaseUpdate, or NoUpdate
template <int XM, int XN, int FDEPTH, bool PAIR, typename UPDATE>
__global__ __launch_bounds__(64 * FWAVES) void k_gemm_f32(GemmF32Batch batch, UPDATE upd) {
  constexpr bool UPD = std::is_same<UPDATE, BaseUpdate>::value;
  constexpr int TM = 16 * XM, TN = 16 * XN;
  __shared__ float red[FWAVES][TM][TN + 1];
  __shared__ float rsum[FWAVES][TM];
  const bool second = PAIR && (int)blockIdx.x >= batch.blocks[0];
  GemmF32Args a = batch.j[0];
  if constexpr (UPD) {
    if (upd.solver == 1 && upd.adam.dev != nullptr) { upd.adam.lr_c1 = upd.adam.dev[0]; upd.adam.c2 = upd.adam.dev[1]; }
    if ((int)blockIdx.x >= batch.blocks[0]) {   // the parameters whose gradients earlier launches left: all but these M x N and M
      const int64_t w0 = a.C - upd.g, b0 = a.rowsum - upd.g, nw = (int64_t)a.M * a.N;   // (dense, the vector behind the matrix), and those set apart between them
      int64_t k = ((int64_t)blockIdx.x - batch.blocks[0]) * (64 * FWAVES) + threadIdx.x;
      if (k >= w0) k += nw;
      if (k >= upd.apart) k += upd.apart_count;
      if (k >= b0) k += a.M;
      if (k < upd.n) update(upd, k, upd.g[k], state_of(upd, k), false);
      return;
    }
  }
  if (PAIR) {
    const GemmF32Args& b = batch.j[1];
    pick(a.A, b.A, second); pick(a.sa_i, b.sa_i, second); pick(a.sa_k, b.sa_k, second);
    pick(a.B, b.B, second); pick(a.sb_k, b.sb_k, second); pick(a.sb_j, b.sb_j, second);
    pick(a.Bv, b.Bv, second); pick(a.beps, b.beps, second); pick(a.bsign, b.bsign, second);
    pick(a.C, b.C, second); pick(a.ldc, b.ldc, second); pick(a.M, b.M, second); pick(a.N, b.N, second); pick(a.K, b.K, second);
    pick(a.bias, b.bias, second); pick(a.bias_v, b.bias_v, second); pick(a.gate, b.gate, second); pick(a.relu, b.relu, second); pick(a.rowsum, b.rowsum, second);
  }
  const int storage = second ? batch.storage[1] : batch.storage[0], blocks = second ? batch.blocks[1] : batch.blocks[0];
  // Workgroups are dealt round-robin to the 8 XCDs (a problem starts at a multiple of 8); each gets a run of a problem's tiles, so
  // that their rows of A come into its L2 once: 2048 x 256 x 784 15.8 -> 14.1 us
  const int nth = second ? blockIdx.x - batch.blocks[0] : blockIdx.x, local = (nth & 7) * (blocks >> 3) + (nth >> 3), nbx = (a.N + TN - 1) / TN;
  const int i0 = (local / nbx) * TM, j0 = (local % nbx) * TN;
  if (i0 >= a.M) return;
  const float bscale = (a.Bv != nullptr && a.beps != nullptr) ? a.bsign * (*a.beps) : 0.f;
  const bool rows = a.rowsum != nullptr && j0 == 0, full = (storage != F32_WGRAD || i0 + TM <= a.M) && j0 + TN <= a.N;
  float* const r0 = &red[0][0][0]; float* const r1 = &rsum[0][0];
  // of the elements this thread will finish, and one row's
  constexpr int NE = (TM * TN + 64 * FWAVES - 1) / (64 * FWAVES);
  Element es[UPD ? NE : 1], er{};
  if constexpr (UPD) {
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const int t = threadIdx.x + e * 64 * FWAVES, gi = min(i0 + t / TN, a.M - 1), gj = min(j0 + t % TN, a.N - 1);
      es[e] = state_of(upd, a.C - upd.g + (int64_t)gi * a.ldc + gj);
    }
    er = state_of(upd, a.rowsum - upd.g + min(i0 + (int)(threadIdx.x % TM), a.M - 1));
  }
  if (storage == F32_FORWARD) {
    if (bscale != 0.f) gemm_f32_tile<XM, XN, FDEPTH, true, true, true, true>(a, i0, j0, bscale, r0, r1);
    else gemm_f32_tile<XM, XN, FDEPTH, true, true, true, false>(a, i0, j0, 0.f, r0, r1);
  } else if (storage == F32_DGRAD) {
    if (full) gemm_f32_tile<XM, XN, FDEPTH, true, false, true, false>(a, i0, j0, 0.f, r0, r1);
    else gemm_f32_tile<XM, XN, FDEPTH, true, false, false, false>(a, i0, j0, 0.f, r0, r1);
  } else {
    if (full) gemm_f32_tile<XM, XN, FDEPTH, false, false, true, false>(a, i0, j0, 0.f, r0, r1);
    else gemm_f32_tile<XM, XN, FDEPTH, false, false, false, false>(a, i0, j0, 0.f, r0, r1);
  }
  __syncthreads();
  auto finish = [&](int t, const Element& el) {
    const int li = t / TN, lj = t % TN, gi = i0 + li, gj = j0 + lj;
    if (gi >= a.M || gj >= a.N) return;
    float bias = 0.f;
    if (a.bias != nullptr) {
      bias = a.bias[gj];
      if (bscale != 0.f && a.bias_v != nullptr) bias = fmaf(bscale, a.bias_v[gj], bias);
    }
    const float gate = a.gate != nullptr ? a.gate[(int64_t)gi * a.ldc + gj] : 1.f;
    float c = red[0][li][lj];
#pragma unroll
    for (int w = 1; w < FWAVES; ++w) c += red[w][li][lj];
    if constexpr (UPD) {
      update(upd, a.C - upd.g + (int64_t)gi * a.ldc + gj, c, el, true);
    } else {
      c += bias;
      if (a.relu) c = fmaxf(c, 0.f);
      a.C[(int64_t)gi * a.ldc + gj] = gate > 0.f ? c : 0.f;
    }
  };
  if constexpr (UPD) {
#pragma unroll
    for (int e = 0; e < NE; ++e)
      if (TM * TN % (64 * FWAVES) == 0 || (int)threadIdx.x + e * 64 * FWAVES < TM * TN) finish(threadIdx.x + e * 64 * FWAVES, es[e]);
  } else {
    for (int t = threadIdx.x; t < TM * TN; t += 64 * FWAVES) finish(t, er);
  }
  if (rows && (int)threadIdx.x < TM && i0 + (int)threadIdx.x < a.M) {
    float c = rsum[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < FWAVES; ++w) c += rsum[w][threadIdx.x];
    if constexpr (UPD) update(upd, a.rowsum - upd.g + i0 + threadIdx.x, c, er, true);
    else a.rowsum[i0 + threadIdx.x] = c;
  }
}

// Forward products that fill the chip.  There is no chain to shorten any more, and splitting the contraction over the waves has its price: a load
// touches 64 bytes of each of 16 rows, two chunks a wave are all that the registers hold in flight, and the partial tiles meet in LDS
// at the end.  Here a wave owns 32 x 16 of a workgroup's 64 x 32 and walks the whole contraction.  Slabs of 64 of the operands' rows come as whole lines,
// whatever their alignment, through registers (two slabs on their way) into three LDS stages with one barrier a slab; a wave fetches the next chunk's
// operands ahead of a chunk's products, also across the barrier.  Chunk c adds to accumulator c % 8, and the eight are added in
// order: the sums of the other tiles, to the bit.  Rows are 68 floats apart, so that the 16 rows of a fetch lie in 16 different places of the banks.
// Bound by the matrix cores in the loop (2048 x 256 x 768: 12.7 thousand clk of MFMAs, 17.2 as it is; with a slab's fetches, stores and loads ahead of its
// products instead of between them 23.9, with two workgroups of four 16 x 16 waves to a CU 18.5).  us a launch, 64 x 32 tile with the contraction
// split / this: 2048 x 256 x 784 15.2 / 11.4, 2048 x 256 x 256 7.9 / 5.8; scoring 2048 samples with 784-256-256-10 28.5 / 24.9.
constexpr int LDS_K = 64, LDS_ROW = LDS_K + 4, LDS_M = 64, LDS_N = 32;
__global__ __launch_bounds__(256, 2) void k_gemm_f32_lds(GemmF32Args a, int blocks) {
  constexpr int NP = (LDS_M + LDS_N) / 16, XM = 2;
  __shared__ __attribute__((aligned(16))) float sm[3][LDS_M + LDS_N][LDS_ROW];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 15, q = lane >> 4;
  const int nbx = (a.N + LDS_N - 1) / LDS_N, local = (blockIdx.x & 7) * (blocks >> 3) + (blockIdx.x >> 3);   // as above
  const int i0 = (local / nbx) * LDS_M, j0 = (local % nbx) * LDS_N;
  if (i0 >= a.M) return;
  const int nfull = a.K / LDS_K, rest = a.K % LDS_K;   // nfull > 0
  // a thread has 16 bytes of every sixteenth row of a slab, A's, then B's; rows beyond the end are clamped
  const int row = tid >> 4, col = 4 * (tid & 15);
  const float* p[NP];
#pragma unroll
  for (int u = 0; u < NP; ++u)
    p[u] = (u < LDS_M / 16 ? a.A + (int64_t)min(i0 + row + 16 * u, a.M - 1) * a.sa_i : a.B + (int64_t)min(j0 + row + 16 * u - LDS_M, a.N - 1) * a.sb_j) + col;
  float4v st[2][NP], tail[NP];   // slabs on their way, by parity; what is not a whole slab, with zeros from K on
  auto load = [&](int s, int u) {   // (of the last slab again behind it: no load in the loop is conditional, because the waits count them)
    return *reinterpret_cast<const f4u*>(p[u] + min(s, nfull - 1) * LDS_K);
  };
  float (*const to)[LDS_ROW] = reinterpret_cast<float (*)[LDS_ROW]>(&sm[0][row][col]);
  auto store = [&](int stage, int u, const float4v& v) { *reinterpret_cast<float4v*>(to[stage * (LDS_M + LDS_N) + 16 * u]) = v; };
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int u = 0; u < NP; ++u) st[i][u] = load(i, u);
#pragma unroll
  for (int u = 0; u < NP; ++u) tail[u] = (float4v){0.f, 0.f, 0.f, 0.f};
  if (rest > 0) {
    const int k = nfull * LDS_K;
    if (col + 4 <= rest) {
#pragma unroll
      for (int u = 0; u < NP; ++u) tail[u] = *reinterpret_cast<const f4u*>(p[u] + k);
    } else {
#pragma unroll
      for (int u = 0; u < NP; ++u)
#pragma unroll
        for (int e = 0; e < 3; ++e)
          if (col + e < rest) tail[u][e] = p[u][k + e];
    }
  }
  const int wi = (wave >> 1) * 16 * XM + r, wj = LDS_M + (wave & 1) * 16 + r, gj = j0 + wj - LDS_M;
  const float bias = a.bias != nullptr ? a.bias[min(gj, a.N - 1)] : 0.f;
  float4v acc[XM][8], op[2][XM + 1];   // operands of a chunk: B's, A's
#pragma unroll
  for (int x = 0; x < XM; ++x)
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[x][c] = (float4v){0.f, 0.f, 0.f, 0.f};
  const float (*const fa)[LDS_ROW] = reinterpret_cast<const float (*)[LDS_ROW]>(&sm[0][wi][4 * q]);
  const float (*const fb)[LDS_ROW] = reinterpret_cast<const float (*)[LDS_ROW]>(&sm[0][wj][4 * q]);
  auto fetch = [&](int stage, int c, int i) {
    return *reinterpret_cast<const float4v*>(&(i == 0 ? fb : fa)[stage * (LDS_M + LDS_N) + (i == 0 ? 0 : 16 * (i - 1))][16 * c]);
  };
  auto fetch_all = [&](int stage, int c, float4v (&v)[XM + 1]) {
#pragma unroll
    for (int i = 0; i <= XM; ++i) v[i] = fetch(stage, c, i);
  };
  // The products of a slab whose first chunk has been fetched.  Between them: the fetches for the next chunk, the slab after the next on its
  // way to its stage, the requests for the one after those.  Each goes behind a product of its own, because with one wave to a SIMD nothing
  // else multiplies while an LDS or address unit takes its time.
  auto slab = [&](int s, int st0, int st1, int st2, auto odd) {
    constexpr int P = decltype(odd)::value;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int m = 0; m < 4 * XM; ++m) {
        const int e = m / XM, x = m % XM;
        __builtin_amdgcn_sched_barrier(0);
        acc[x][4 * P + c] = __builtin_amdgcn_mfma_f32_16x16x4f32(op[c & 1][1 + x][e], op[c & 1][0][e], acc[x][4 * P + c], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (m <= XM) op[(c + 1) & 1][m] = c < 3 ? fetch(st0, c + 1, m) : fetch(st1, 0, m);
        else if (c < 3 && m < XM + 3) store(st2, 2 * c + m - XM - 1, st[P][2 * c + m - XM - 1]);
        else if (c < 3 && m < XM + 5) st[P][2 * c + m - XM - 3] = load(s + 4, 2 * c + m - XM - 3);
      }
    }
    __syncthreads();
  };
  static_assert(NP == 6 && XM == 2, "places between the products");
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int u = 0; u < NP; ++u) { store(i, u, st[i][u]); st[i][u] = load(2 + i, u); }
  __syncthreads();
  fetch_all(0, 0, op[0]);
  int s = 0, s0 = 0, s1 = 1, s2 = 2;   // stages of this slab and the next two
  auto next = [&]() { const int t = s0; s0 = s1; s1 = s2; s2 = t; };
  for (; s + 1 < nfull; s += 2) {
    slab(s, s0, s1, s2, even); next();
    slab(s + 1, s0, s1, s2, odd); next();
  }
  if (s < nfull) { slab(s, s0, s1, s2, even); next(); }
  if (rest > 0) {
#pragma unroll
    for (int u = 0; u < NP; ++u) store(s1, u, tail[u]);   // (of s0 the first chunk may still be being fetched)
    __syncthreads();
    auto last = [&](auto odd) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (c * FCH >= rest) break;
        fetch_all(s1, c, op[0]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int x = 0; x < XM; ++x)
            acc[x][4 * decltype(odd)::value + c] = __builtin_amdgcn_mfma_f32_16x16x4f32(op[0][1 + x][e], op[0][0][e], acc[x][4 * decltype(odd)::value + c], 0, 0, 0);
      }
    };
    if (nfull & 1) last(odd);
    else last(even);
  }
  if (gj >= a.N) return;
#pragma unroll
  for (int x = 0; x < XM; ++x)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int gi = i0 + (wave >> 1) * 16 * XM + 16 * x + 4 * q + e;
      if (gi >= a.M) return;
      float c = acc[x][0][e];
#pragma unroll
      for (int w = 1; w < 8; ++w) c += acc[x][w][e];
      c += bias;
      if (a.relu) c = fmaxf(c, 0.f);
      a.C[(int64_t)gi * a.ldc + gj] = c;
    }
}

int64_t tiles(const GemmF32Args* a, int count, int tm, int tn) {
  int64_t n = 0;
  for (int k = 0; k < count; ++k) n += (int64_t)((a[k].N + tn - 1) / tn) * ((a[k].M + tm - 1) / tm);
  return n;
}
template <int XM, int XN, int FDEPTH>
void launch_tile_f32(ProfScope& ps, hipStream_t st, const GemmF32Args* a, int count, const BaseUpdate* u) {
  GemmF32Batch b{};
  for (int k = 0; k < count; ++k) {
    b.j[k] = a[k];
    b.storage[k] = storage_of(a[k]);
    b.blocks[k] = (int)(tiles(a + k, 1, 16 * XM, 16 * XN) + 7) / 8 * 8;
  }
  if (u != nullptr) {
    const int64_t rest = u->n - (int64_t)a[0].M * a[0].N - a[0].M - u->apart_count;
    launch_kernel(ps, k_gemm_f32<XM, XN, FDEPTH, false, BaseUpdate>, b.blocks[0] + (int)((rest + 64 * FWAVES - 1) / (64 * FWAVES)), 64 * FWAVES, 0, st, b, *u);
  } else if (count == 2) {
    launch_kernel(ps, k_gemm_f32<XM, XN, FDEPTH, true, NoUpdate>, b.blocks[0] + b.blocks[1], 64 * FWAVES, 0, st, b, NoUpdate{});
  } else {
    launch_kernel(ps, k_gemm_f32<XM, XN, FDEPTH, false, NoUpdate>, b.blocks[0], 64 * FWAVES, 0, st, b, NoUpdate{});
  }
}

void launch(hipStream_t st, const GemmF32Args* a, int count, const BaseUpdate* u) {
  double flops = 0.0;
  for (int k = 0; k < count; ++k) {
    if (a[k].M <= 0 || a[k].N <= 0) { note_launch_error("empty fp32 GEMM"); return; }
    if (storage_of(a[k]) < 0) { note_launch_error("fp32 GEMM: operand storage"); return; }
    flops += 2.0 * a[k].M * a[k].N * a[k].K;
  }
  ProfScope ps(st, F_GEMM_F32, flops);
  // The smallest tile gives the shortest chain and the most workgroups, but reads every operand row once per 16 columns.  us, 16 x 16 /
  // 32 x 32: 256 tiles of 16 x 16 (512 x 128 x 784) 5.4 / 8.7, 512 (512 x 256 x 784) 8.1 / 8.8, 640 (512 x 320 x 1024) 14.5 / 11.0;
  // 32 x 32 / 64 x 32: 256 tiles of 32 x 32 (1024 x 256 x 784) 9.0 / 14.3, 320 (a weight gradient over 512 rows, 320 x 1024)
  // 11.7 / 9.4.  Over 150 products and pairs (16 to 2048 rows, widths to 320, K to 1024) these
  // lines take 1.4% longer than the fastest tile of each, lines at 256 and 256 3.9% (geometric means).
  // The line at 256 holds for k_gemm_f32_lds too.  Up to it (56 forward products of 160 to 256 tiles of 32 x 32, K from 64 to 1024) that takes 5 to 30% longer than
  // 32 x 32: 1024 x 256 x 64 4.3 / 4.5, x 256 5.8 / 6.6, x 784 10.0 / 12.6.  Beyond (72 products) it takes 3 to 30% less than 64 x 32 with the contraction
  // split: 1536 x 192 x 64 5.1 / 4.6, x 191 8.0 / 6.7, x 784 14.9 / 13.4, 2048 x 130 x 64 5.1 / 4.3, 2048 x 320 x 1024 31.1 / 23.2.
  constexpr int CUS = 256;
  if (tiles(a, count, 16, 16) <= 2 * CUS) launch_tile_f32<1, 1, 8>(ps, st, a, count, u);
  else if (tiles(a, count, 32, 32) <= CUS) launch_tile_f32<2, 2, 4>(ps, st, a, count, u);
  // (the first slab has to be a whole one; the pair of a perturbed forward pass, which large batches have, stays with the tile whose waves
  // form theta +- eps v as they load, and a gate belongs to a gradient)
  else if (count == 1 && storage_of(a[0]) == F32_FORWARD && a[0].Bv == nullptr && a[0].gate == nullptr && a[0].K >= LDS_K) {
    const int blocks = (int)(tiles(a, 1, LDS_M, LDS_N) + 7) / 8 * 8;
    launch_kernel(ps, k_gemm_f32_lds, blocks, 256, 0, st, a[0], blocks);
  }
  else launch_tile_f32<4, 2, 2>(ps, st, a, count, u);
}
}  // namespace

void launch_gemm_f32_batch(hipStream_t st, const GemmF32Args* a, int count) { launch(st, a, count, nullptr); }
void launch_gemm_f32_update(hipStream_t st, const GemmF32Args& a, const BaseUpdate& u) {
  // the forms the kernel is for: a dense weight gradient with its bias gradient behind it, both in u.g
  if (storage_of(a) != F32_WGRAD || a.ldc != a.N || a.rowsum == nullptr || a.C < u.g || a.rowsum < a.C + (int64_t)a.M * a.N || a.rowsum + a.M > u.g + u.n ||
      (u.apart_count != 0 && (u.apart_count < 0 || u.apart < a.C + (int64_t)a.M * a.N - u.g || u.apart + u.apart_count > a.rowsum - u.g)) ||
      a.bias != nullptr || a.gate != nullptr || a.relu) { note_launch_error("fp32 GEMM with an update: not a weight gradient"); return; }
  launch(st, &a, 1, &u);
}

}  // namespace sama
