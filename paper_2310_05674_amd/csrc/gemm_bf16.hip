// bf16 x bf16 -> fp32 contraction on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16) for the encoder's linear
// layers: forward (X W^T), dgrad (dY W) and wgrad (dY^T X) are one kernel template over the storage of its two
// operands.
//
//   operand slabs go global -> LDS directly (global_load_lds_dwordx4, 1 KB per wave instruction) into dense,
//   XOR-swizzled stages, NSTAGE - 1 slabs in flight, one barrier per slab; no staging registers
//   most tiles have waves that do nothing but issue those loads: a wave that issues a slab's loads itself waits for the
//   address units to take them, a third of the slab's matrix time, before it multiplies.  Against the same tile without them:
//   256 x 128 hi + lo 6%, 128 x 128 10%, 128 x 96 11%, 128 x 64 4% faster, 128 x 128 single-term TN 16% (geometric means
//   over 65 and 51 problems); four such waves are 4% faster than two, eight the same as four
//   an operand whose contraction index is contiguous in memory is staged [row][k] and fetched with 16-byte reads;
//   one whose contraction index is the strided one (dgrad's W, both operands of wgrad) is staged as it lies in
//   memory, [k][row], and fetched with the transposing LDS read (ds_read_b64_tr_b16)
//   the MFMA operands of k-step t + 1 are fetched while the MFMAs of step t issue, also across the slab boundary
//   measured on MI355X: a CU takes in 56 B/clk where L2 holds the slabs, 40 from the last-level cache and 26 where the weights
//   come from memory, and at the MFMA peak 256 x 256 tiles need 32 B/clk, 256 x 128 48, 128 x 128 64: small tiles are bound by
//   this, and the weights of a product of few rows are fetched by the launch before it (k_ln_fwd, k_ln_bwd).  The loops of the largest
//   tiles are bound by power: without any loads a launch of 256 x 128 hi + lo tiles of 111 us takes 96 in as many clocks, at 1.73 GHz
//   instead of 1.50, with the matrix cores busy 65 % of the time (profiles/gemm_bounds.md)
//   workgroup ids are remapped so that each XCD (own L2) works on a compact patch of tiles
//   the accumulators leave through LDS so that every global access of the epilogue is a full row segment
//
// For the theta +- eps v passes of Eq. 5 and the direct-gradient pass the weight operand is hi + lo (two bf16
// halves).  DUAL tiles stage the A slab once together with the hi and the lo slab of B and issue two MFMAs per A
// operand, so A is neither loaded nor fetched twice.
//
// Several independent problems of one storage class can share a launch (the + and - pass of Eq. 5, the four weight
// gradients of a layer): more tiles per launch for the small per-layer shapes.
//
// Fused epilogues: + bias (fp32, optionally perturbed), + residual (fp32), GELU forward (writes both the
// pre-activation and the activation), GELU backward (multiplies by gelu'(pre)), fp32 and/or bf16 stores.  The large hi + lo
// tiles look the GELU factors up in a table that their loading waves bring into LDS during the last slab.
#include <type_traits>
#include "common.h"
#include "gelu.h"
#include "kernels.h"

namespace sama {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void gvoid;
constexpr int LDS_MAX = 160 * 1024;

// PW: waves that only load (0: the multiplying waves load for themselves).  SB: see the kernel.
template <int BM_, int BN_, int BK_, int WGM_, int WGN_, int NSTAGE_, bool DUAL_, int PW_ = 0, bool SB_ = false>
struct Tile {
  static constexpr int PW = PW_;
  static constexpr bool SB = SB_;
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WGM = WGM_, WGN = WGN_, NSTAGE = NSTAGE_;
  static constexpr bool DUAL = DUAL_;
  static constexpr int WAVES = WGM * WGN, LW = PW > 0 ? PW : WAVES, THREADS = (WAVES + PW) * 64;   // multiplying, loading
  static constexpr int WM = BM / WGM, WN = BN / WGN, XT = WM / 32, YT = WN / 32;
  static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE_BYTES = A_BYTES + (DUAL ? 2 : 1) * B_BYTES;
  static constexpr int NLA = A_BYTES / 1024 / LW, NLB = B_BYTES / 1024 / LW;   // 1 KB loads of a loading wave per slab
  static constexpr int NL = NLA + (DUAL ? 2 : 1) * NLB;
  static_assert(LDS_MAX >= NSTAGE * STAGE_BYTES, "stages exceed the 160 KB of LDS");
  static constexpr int LDS_MAIN = NSTAGE * STAGE_BYTES;
  static constexpr int EPI_LD = WN + 8;   // 4 rows apart = 32 banks apart: the two lane halves of a staging write do not collide
  static constexpr int LDS_EPI = WAVES * 32 * EPI_LD * 4;
  static constexpr int LDS_BYTES = LDS_MAIN > LDS_EPI ? LDS_MAIN : LDS_EPI;
  // Whether the GELU epilogues look their values up (gelu.h).  The table comes into a stage that the last slab does not use, while
  // that slab is multiplied, and stays clear of the epilogue's staging.  Computed, a value is 26 quarter-rate vector instructions
  // in which the matrix cores stand still; looked up it is seven and an LDS read.  us computed / looked up, forward: 2048 x 4096 x
  // 1024 (256 x 128 tiles) 37.3 / 34.5, 4096 x 3072 x 768 (256 x 192) 47.1 / 40.8; backward 40.1 / 37.7, 50.9 / 45.7; with 128 x 128
  // tiles, 1024 x 3072 x 768, 19.6 / 18.0.  The 128 x 64 and smaller tiles compute: the table would be as much to load as a slab
  // of them or more.  The 128 x 96 ones compute too, though looking up is 1.1 to 3.2 us faster in each of twelve products timed both
  // ways (1024 x 3072 x 768 forward 19.2 / 17.9: profiles/gemm_bounds.md); in ten of them another tile is faster than either.
  static constexpr bool TAB = DUAL && PW > 0 && BM * BN >= 128 * 128;
  static_assert(!TAB || (NSTAGE >= 2 && STAGE_BYTES >= GELU_TAB_BYTES && LDS_MAIN - GELU_TAB_BYTES >= LDS_EPI), "room for the table");
  static_assert(A_BYTES % (1024 * LW) == 0 && B_BYTES % (1024 * LW) == 0, "slab must split into whole wave loads");
  static_assert(NL * (NSTAGE - 2) <= 63, "vmcnt range");
};

// Byte offset (relative to the slab's first element in global memory) of the 16-byte piece that belongs at byte
// `ldsoff` of an operand's dense LDS stage.
//   KC (contraction contiguous, storage [rows][k]): stage [R][BK]; the 16-byte chunk index within a row is XORed
//     with (row / RP) % NCH so that 16 consecutive rows at one logical chunk fill all 64 banks.
//   KS (contraction strided, storage [k][rows]): stage [BK][R]; the 64-byte chunk index within a k-row is XORed with
//     chunk_swizzle(k-row) so that the four k-rows one transposing read touches fill all 64 banks.
// Rows past `nrows` are clamped (their products land in outputs the epilogue never stores).
// A k-row of R values is R / 32 chunks; four consecutive k-rows have to put one chunk each into the four quarters of the
// banks.  Rows a multiple of four chunks long all start at the same bank, rows of two chunks pairwise, rows of six at
// alternating halves; rows of one or three chunks are spread already.
template <int R>
__device__ __forceinline__ int chunk_swizzle(int kr) {
  constexpr int NC = R / 32;
  static_assert(NC % 4 == 0 || NC == 1 || NC == 2 || NC == 3 || NC == 6, "tile width");
  return NC % 4 == 0 ? (kr & 3) : (NC == 2 || NC == 6) ? ((kr >> 1) & 1) : 0;
}
template <bool KC, int R, int BK>
__device__ __forceinline__ uint32_t piece_offset(int ldsoff, int row0, int nrows, int64_t ld) {
  if (KC) {
    constexpr int RB = BK * 2, RP = 256 / RB, NCH = RB / 16;
    const int r = ldsoff / RB, p = (ldsoff % RB) / 16;
    const int c = p ^ ((r / RP) % NCH);
    return (uint32_t)(((int64_t)min(row0 + r, nrows - 1) * ld + c * 8) * 2);
  } else {
    constexpr int RBS = R * 2;
    const int kr = ldsoff / RBS, q16 = (ldsoff % RBS) / 16;
    const int ql = (((q16 >> 2) ^ chunk_swizzle<R>(kr)) << 2) | (q16 & 3);
    return (uint32_t)(((int64_t)kr * ld + min(row0 + ql * 8, nrows - 8)) * 2);
  }
}

// MFMA operand (8 contraction values k = ks*16 + 8*(lane/32) + 0..7 of tile row tb + lane%32) out of a swizzled stage.
// `lo` is the lane-dependent part precomputed by fetch_lane_offset, `tb` the first row of the 32-row tile.
template <bool KC, int R, int BK>
__device__ __forceinline__ int fetch_lane_offset(int lane, int ks_or_tile) {
  if (KC) {
    constexpr int RB = BK * 2, RP = 256 / RB, NCH = RB / 16;
    const int rl = lane & 31, hi = lane >> 5;
    const int s = (rl / RP) % NCH;
    return rl * RB + (((2 * ks_or_tile + hi) ^ s) * 16);                  // per ks
  } else {
    constexpr int RBS = R * 2;
    const int g = lane >> 4, j = lane & 15;
    const int cc = ks_or_tile;                                            // 64-byte chunk of the tile = tile_row0 / 32
    const int kr = 8 * (g >> 1) + (j >> 2);                               // the swizzle is the same for kr + 4 and kr + 16
    return kr * RBS + ((cc ^ chunk_swizzle<R>(kr)) * 64) + (16 * (g & 1) + 4 * (j & 3)) * 2;   // per tile
  }
}

// Waits until all but the `younger` (at most W) last slabs of NL loads each of this wave have landed.
template <int NL, int W>
__device__ __forceinline__ void wait_loads(int younger) {
  if constexpr (W == 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
    if (younger >= W) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL * W) : "memory");
    else wait_loads<NL, W - 1>(younger);
  }
}

struct GemmBatch {
  GemmBf16Args p[GEMM_MAX_BATCH];
  int first_tile[GEMM_MAX_BATCH + 1];   // tile ids [first_tile[k], first_tile[k + 1]) belong to problem k
  int count, group;
};

struct LoopArgs {
  const bf16_t *A, *B, *B2;
  int64_t lda, ldb;
  int M, N, K, act;
  const float* gelu_tab;
  const int32_t* rows;
  __device__ __forceinline__ void pin() {   // keeps the reads where they are
    asm("" : "+s"(A), "+s"(B), "+s"(B2), "+s"(lda), "+s"(ldb), "+s"(M), "+s"(N), "+s"(K), "+s"(act), "+s"(gelu_tab), "+s"(rows));
  }
};
__device__ __forceinline__ LoopArgs loop_args(const GemmBf16Args& a) { return LoopArgs{a.A, a.B, a.B2, a.lda, a.ldb, a.M, a.N, a.K, a.act, a.gelu_tab, a.rows}; }

template <typename T, bool A_KC, bool B_KC>
__global__ __launch_bounds__(T::THREADS) void k_gemm_bf16(GemmBatch batch, int ntiles, int tiles_per_xcd) {
  constexpr int BM = T::BM, BN = T::BN, BK = T::BK, XT = T::XT, YT = T::YT, NSTAGE = T::NSTAGE, WAVES = T::WAVES;
  constexpr bool DUAL = T::DUAL;
  // Whether the operands of a k-step are fetched right before it (fewer registers, the order left to the compiler) instead of
  // during the step before.  With the transposing reads of a strided operand the three-stage tiles are 7-9% faster that way.
  constexpr bool SB = T::SB || (!B_KC && T::PW > 0 && NSTAGE == 3);
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = (wave / T::WGN) * T::WM, wc = (wave % T::WGN) * T::WN;
  // XCD-aware order: workgroups are dealt round-robin to the 8 XCDs; each XCD gets a contiguous run of tile ids, and
  // tile ids walk down `group` tile rows before moving one tile column to the right, so that the tiles in flight on
  // one XCD form a compact patch (few distinct A and B panels in its L2).
  // Where the rows in use are known on the device only, the launch has the tiles of all rows, and the order is made here over
  // those in use (the problems of a batch then have the same rows).
  const int32_t* const in_use = batch.p[0].rows;
  const int rows = in_use != nullptr ? __builtin_amdgcn_readfirstlane(*in_use) : 0;
  const bool fewer_tiles = A_KC && in_use != nullptr;
  int pid, prob = 0;
  if (fewer_tiles) {
    const int gy = (rows + BM - 1) / BM;
    int n = 0;
    for (int k = 0; k < batch.count; ++k) n += gy * ((batch.p[k].N + BN - 1) / BN);
    const int per_xcd = (n + 7) / 8;
    pid = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || pid >= n) return;
    for (int k = 0; k + 1 < batch.count; ++k) {
      const int t = gy * ((batch.p[k].N + BN - 1) / BN);
      if (pid < t) break;
      pid -= t;
      prob = k + 1;
    }
  } else {
    pid = (blockIdx.x & 7) * tiles_per_xcd + (blockIdx.x >> 3);
    if (pid >= ntiles) return;
    int before = 0;
#pragma unroll
    for (int k = 1; k < GEMM_MAX_BATCH; ++k)
      if (k < batch.count && pid >= batch.first_tile[k]) { prob = k; before = batch.first_tile[k]; }
    pid -= before;
  }
  // What the loop needs of problem 0 is read with the kernel's first arguments: an index into them that is computed first costs another
  // trip to memory, 0.2 us, and most launches have one problem.
  const GemmBf16Args& a = batch.p[prob];   // for the epilogue
  LoopArgs la = loop_args(batch.p[0]);
  la.pin();
  if (prob != 0) la = loop_args(a);
  const int group = batch.group;
  const int Mrows = fewer_tiles ? rows : la.M;
  const int gx = (la.N + BN - 1) / BN, gy = (Mrows + BM - 1) / BM;
  const int width = group * gx, grp = pid / width, first = grp * group;
  const int gsz = min(gy - first, group);
  const int ti = first + (pid % width) % gsz, tj = (pid % width) / gsz;
  const int i0 = ti * BM, j0 = tj * BN;

  f32x16 acc[XT][YT];
#pragma unroll
  for (int x = 0; x < XT; ++x)
#pragma unroll
    for (int y = 0; y < YT; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;

  const int nk = (!A_KC && la.rows != nullptr ? __builtin_amdgcn_readfirstlane(*la.rows) : la.K) / BK;
  // The operand pointers live in registers for the whole k loop (read through `a` they would be re-fetched from the
  // kernel-argument segment after every inline-assembly load, a scalar-memory round trip per slab).
  const char* const pA = reinterpret_cast<const char*>(la.A);
  const char* const pB = reinterpret_cast<const char*>(la.B);
  const char* const pB2 = reinterpret_cast<const char*>(la.B2);
  const int iters = (!DUAL && pB2 != nullptr) ? 2 * nk : nk;   // non-DUAL tiles contract with hi, then with lo

  // the GELU table's place: at the top, or at the bottom (and the staging of the epilogue above it) if the last slab is at the top
  const bool look_up = T::TAB && la.act != GEMM_ACT_NONE;
  const bool tab_low = (iters - 1) % NSTAGE == NSTAGE - 1;
  const int tab_at = tab_low ? 0 : T::LDS_MAIN - GELU_TAB_BYTES;
  const int lw = T::PW > 0 ? wave - WAVES : wave;            // number among the loading waves
  const bool loader = T::PW == 0 || wave >= WAVES;
  // per-lane global offsets of this wave's loads
  uint32_t offA[T::NLA], offB[T::NLB];
#pragma unroll
  for (int q = 0; q < T::NLA; ++q) offA[q] = piece_offset<A_KC, BM, BK>((q * T::LW + lw) * 1024 + lane * 16, i0, Mrows, la.lda);
#pragma unroll
  for (int q = 0; q < T::NLB; ++q) offB[q] = piece_offset<B_KC, BN, BK>((q * T::LW + lw) * 1024 + lane * 16, j0, la.N, la.ldb);
  const int64_t stepA = A_KC ? (int64_t)BK * 2 : (int64_t)BK * la.lda * 2;   // bytes per slab
  const int64_t stepB = B_KC ? (int64_t)BK * 2 : (int64_t)BK * la.ldb * 2;

  // Direct global -> LDS loads: lane l of a wave-level load lands at (m0) + 16 l.  Written as inline assembly so
  // that the only waits on them are the explicit vmcnt waits below.
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void*)smem_raw;
  // All NL loads of a slab are issued together right after the barrier that frees their stage (in waves that also
  // multiply, spreading them over the k-steps measured 3-8% slower: it shortens the prefetch distance).
  constexpr int KS = BK / 16;
  auto issue = [&](int sl) {
    if (sl >= iters || !loader) return;
    const int stage = sl % NSTAGE;
    const int kq = sl >= nk ? sl - nk : sl;
    const char* ap = pA + kq * stepA;
    const char* bp = (sl >= nk ? pB2 : pB) + kq * stepB;
    const char* b2p = pB2 + kq * stepB;
    const uint32_t sa = lds0 + stage * T::STAGE_BYTES + lw * 1024;
    const uint32_t sb = sa + T::A_BYTES;
#pragma unroll
    for (int t = 0; t < T::NL; ++t) {
      if (t < T::NLA) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(sa + t * T::LW * 1024), "v"(offA[t]), "s"(ap) : "memory", "m0");
      } else if (t < T::NLA + T::NLB) {
        const int q = t - T::NLA;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(sb + q * T::LW * 1024), "v"(offB[q]), "s"(bp) : "memory", "m0");
      } else {
        const int q = t - T::NLA - T::NLB;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(sb + T::B_BYTES + q * T::LW * 1024), "v"(offB[q]), "s"(b2p) : "memory", "m0");
      }
    }
  };

  // lane-dependent parts of the operand fetch addresses
  int fa[A_KC ? BK / 16 : XT], fb[B_KC ? BK / 16 : YT];
  if (A_KC) {
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) fa[ks] = fetch_lane_offset<true, BM, BK>(lane, ks) + wr * BK * 2;
  } else {
#pragma unroll
    for (int x = 0; x < XT; ++x) fa[x] = fetch_lane_offset<false, BM, BK>(lane, (wr >> 5) + x);
  }
  if (B_KC) {
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) fb[ks] = fetch_lane_offset<true, BN, BK>(lane, ks) + wc * BK * 2;
  } else {
#pragma unroll
    for (int y = 0; y < YT; ++y) fb[y] = fetch_lane_offset<false, BN, BK>(lane, (wc >> 5) + y);
  }

  auto fetchA = [&](const unsigned char* sa, int x, int ks) -> bf16x8 {
    if (A_KC) return *reinterpret_cast<const bf16x8*>(sa + fa[ks] + x * 32 * BK * 2);
    const unsigned char* p = sa + fa[x] + ks * 16 * BM * 2;
    union { bf16x8 v; s16x4 h[2]; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * BM * 2));
    return u.v;
  };
  auto fetchB = [&](const unsigned char* sb, int y, int ks) -> bf16x8 {
    if (B_KC) return *reinterpret_cast<const bf16x8*>(sb + fb[ks] + y * 32 * BK * 2);
    const unsigned char* p = sb + fb[y] + ks * 16 * BN * 2;
    union { bf16x8 v; s16x4 h[2]; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * BN * 2));
    return u.v;
  };

  // ---- pipeline: NSTAGE - 1 slabs in flight; the k-steps of all slabs form one stream in which the operands of
  // step t + 1 are fetched from LDS before the MFMAs of step t are issued (also across the slab boundary, so the
  // LDS latency after a barrier hides behind the last MFMAs of the previous slab)
#pragma unroll
  for (int s = 0; s < NSTAGE - 1; ++s) issue(s);

  static_assert(KS % 2 == 0, "operand double buffer parity");
  bf16x8 av[2][XT], bv[2][YT], bw[2][DUAL ? YT : 1];
  // make slab `sl` visible: a loading wave's own loads landed, then everyone's; afterwards the stage of slab sl - 1 is free
  auto arrive = [&](int sl) {
    const int younger = iters - 1 - sl;
    if (loader) wait_loads<T::NL, NSTAGE - 2>(younger);
    __builtin_amdgcn_s_barrier();
    issue(sl + NSTAGE - 1);
  };
  auto fetch = [&](int sl, int ks, int buf) {
    const unsigned char* sa = smem_raw + (sl % NSTAGE) * T::STAGE_BYTES;
    const unsigned char* sb = sa + T::A_BYTES;
#pragma unroll
    for (int x = 0; x < XT; ++x) av[buf][x] = fetchA(sa, x, ks);
#pragma unroll
    for (int y = 0; y < YT; ++y) bv[buf][y] = fetchB(sb, y, ks);
    if (DUAL) {
#pragma unroll
      for (int y = 0; y < YT; ++y) bw[buf][y] = fetchB(sb + T::B_BYTES, y, ks);
    }
  };
  if (T::PW > 0 && loader) {   // the barriers of the others, and the loads
    for (int i = 0; i < iters; ++i) arrive(i);
    if constexpr (T::TAB) {
      if (look_up) {   // all slabs but the last have been read
        const char* const tab = reinterpret_cast<const char*>(la.gelu_tab) + (la.act == GEMM_ACT_GELU_BWD ? GELU_TAB_BYTES : 0);
#pragma unroll
        for (int q = 0; q < (GELU_TAB_BYTES / 1024 + T::LW - 1) / T::LW; ++q) {
          const int piece = q * T::LW + lw;
          if (piece < GELU_TAB_BYTES / 1024)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds0 + tab_at + piece * 1024), "v"(lane * 16), "s"(tab + piece * 1024) : "memory", "m0");
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
    }
    __syncthreads();
    return;
  }
  arrive(0);
  auto mfma_step = [&](int cur) {
    if (!SB) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int x = 0; x < XT; ++x)
#pragma unroll
      for (int y = 0; y < YT; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[cur][x], bv[cur][y], acc[x][y], 0, 0, 0);
    if (DUAL) {
#pragma unroll
      for (int x = 0; x < XT; ++x)
#pragma unroll
        for (int y = 0; y < YT; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[cur][x], bw[cur][y], acc[x][y], 0, 0, 0);
    }
    if (!SB) __builtin_amdgcn_sched_barrier(0);
  };
  if (SB) {
    for (int i = 0; i < iters; ++i) {
      if (i > 0) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave's reads of slab i - 1 are complete
        arrive(i);
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) { fetch(i, ks, 0); mfma_step(0); }
    }
  } else {
    fetch(0, 0, 0);
    for (int i = 0; i + 1 < iters; ++i) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int cur = ks & 1;
        if (ks + 1 < KS) {
          fetch(i, ks + 1, cur ^ 1);
        } else {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave's reads of slab i are complete
          arrive(i + 1);
          fetch(i + 1, 0, cur ^ 1);
        }
        mfma_step(cur);
      }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {   // last slab
      if (ks + 1 < KS) fetch(iters - 1, ks + 1, (ks & 1) ^ 1);
      mfma_step(ks & 1);
    }
  }
  __syncthreads();

  // ---- epilogue: accumulators -> LDS (per wave, 32 x WN fp32 at a time) -> row-contiguous global accesses
  constexpr int EPI_LD = T::EPI_LD, LPR = T::WN / 4, RPP = 64 / LPR;   // lanes per row, rows per pass
  float* epi = reinterpret_cast<float*>(smem_raw + (look_up && tab_low ? GELU_TAB_BYTES : 0)) + wave * 32 * EPI_LD;
  const unsigned char* const tab = smem_raw + tab_at;
  const int cg = lane % LPR, rq = lane / LPR;
  const int gj = j0 + wc + 4 * cg;
  const bool col_ok = gj < a.N && (LPR * RPP == 64 || lane < LPR * RPP);   // 96-wide wave tiles: 24 lanes a row, two rows
  float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
  if (col_ok && a.bias != nullptr) {
    bias = *reinterpret_cast<const float4*>(a.bias + gj);
    if (a.bias_v != nullptr && a.beps != nullptr && a.bsign != 0.f) {
      const float s = a.bsign * (*a.beps);
      const float4 bv = *reinterpret_cast<const float4*>(a.bias_v + gj);
      bias.x = fmaf(s, bv.x, bias.x); bias.y = fmaf(s, bv.y, bias.y); bias.z = fmaf(s, bv.z, bias.z); bias.w = fmaf(s, bv.w, bias.w);
    }
  }
  const float* const res32 = a.res32; const bf16_t* const aux16 = a.aux16;
  bf16_t* const C16_pre = a.C16_pre; bf16_t* const C16 = a.C16; float* const C32 = a.C32;
  const int act = a.act;
  const int64_t ldc = a.ldc, base = (int64_t)(i0 + wr) * ldc + j0 + wc;   // of the wave's tile
  const uint32_t lane_off = (uint32_t)(rq * ldc) + 4u * cg;               // a step is a uniform distance plus this (rq < 8)
  constexpr int NIT = 32 / RPP;
  // A slice of 32 rows goes through LDS at a time and is finished four steps (of RPP rows) at a time, each operation for the
  // four together; the side inputs (an fp32 residual or a saved pre-activation, an epilogue has one of them at most) of the next
  // four steps are requested before the current ones are finished, across the slices.
  constexpr int CH = 4, PER = NIT / CH, NCH = XT * PER;
  static_assert(NIT % CH == 0, "steps of a slice");
  const bool side = res32 != nullptr || act == GEMM_ACT_GELU_BWD;
  auto entry = [&](uint32_t offset) { return *reinterpret_cast<const float*>(tab + offset); };   // of the GELU table
  auto epilogue = [&](auto all_rows) {   // all_rows: every row of the tile exists
    auto exists = [&](int row) { return decltype(all_rows)::value || i0 + wr + row < Mrows; };   // row: within the wave's tile
    auto step = [&](int q, int u) { return base + (int64_t)((q / PER) * 32 + RPP * ((q % PER) * CH + u)) * ldc; };
    auto row_of = [&](int q, int u) { return rq + RPP * ((q % PER) * CH + u); };   // within the slice
    auto load_side = [&](int q, uint4 (&sv)[CH]) {
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        if (!exists((q / PER) * 32 + row_of(q, u))) continue;
        if (res32 != nullptr) {
          sv[u] = *reinterpret_cast<const uint4*>(res32 + step(q, u) + lane_off);
        } else {
          const uint2 t = *reinterpret_cast<const uint2*>(aux16 + step(q, u) + lane_off);
          sv[u].x = t.x; sv[u].y = t.y;
        }
      }
    };
    constexpr bool AHEAD = XT * YT <= 4;   // more accumulators leave no registers for two sets of side inputs
    uint4 sv[AHEAD ? 2 : 1][CH] = {};
    if (AHEAD && side && col_ok) load_side(0, sv[0]);
#pragma unroll
    for (int q = 0; q < NCH; ++q) {
      const int x = q / PER;
      if (!AHEAD && side && col_ok) load_side(q, sv[0]);
      if (q % PER == 0) {
        // the staging region is private to the wave: LDS operations of one wave complete in order, no block barrier
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
#pragma unroll
        for (int y = 0; y < YT; ++y)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            epi[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * EPI_LD + y * 32 + (lane & 31)] = acc[x][y][r];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
      if (!col_ok) continue;
      if (AHEAD && side && q + 1 < NCH) load_side(q + 1, sv[AHEAD ? (q + 1) & 1 : 0]);
      float c[CH][4];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
        const float4 v = *reinterpret_cast<const float4*>(epi + row_of(q, u) * EPI_LD + 4 * cg);
        c[u][0] = v.x + bias.x; c[u][1] = v.y + bias.y; c[u][2] = v.z + bias.z; c[u][3] = v.w + bias.w;
      }
      if (res32 != nullptr) {
#pragma unroll
        for (int u = 0; u < CH; ++u) {
          const uint4 r = sv[AHEAD ? q & 1 : 0][u];
          c[u][0] += __uint_as_float(r.x); c[u][1] += __uint_as_float(r.y); c[u][2] += __uint_as_float(r.z); c[u][3] += __uint_as_float(r.w);
        }
      }
      if (act == GEMM_ACT_GELU_FWD) {
        // the backward pass sees the rounded pre-activation, so the activation is taken from it too
#pragma unroll
        for (int u = 0; u < CH; ++u) {
          const uint2 pk = make_uint2(pack_bf16x2(c[u][0], c[u][1]), pack_bf16x2(c[u][2], c[u][3]));
          if (C16_pre != nullptr && exists(x * 32 + row_of(q, u))) *reinterpret_cast<uint2*>(C16_pre + step(q, u) + lane_off) = pk;   // forward-only passes do not keep it
          c[u][0] = bf16_to_f32((bf16_t)pk.x); c[u][1] = bf16_to_f32((bf16_t)(pk.x >> 16));
          c[u][2] = bf16_to_f32((bf16_t)pk.y); c[u][3] = bf16_to_f32((bf16_t)(pk.y >> 16));
          if constexpr (T::TAB) {
            const uint32_t o0 = gelu_tab_offsets(pk.x), o1 = gelu_tab_offsets(pk.y);
            c[u][0] *= entry(o0 & 0xffffu); c[u][1] *= entry(o0 >> 16); c[u][2] *= entry(o1 & 0xffffu); c[u][3] *= entry(o1 >> 16);
          }
        }
        if constexpr (!T::TAB) {
#pragma unroll
          for (int u = 0; u < CH; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) c[u][e] = gelu_f(c[u][e]);
        }
      } else if (act == GEMM_ACT_GELU_BWD) {
#pragma unroll
        for (int u = 0; u < CH; ++u) {
          const uint4 r = sv[AHEAD ? q & 1 : 0][u];
          const float x[4] = {bf16_to_f32((bf16_t)r.x), bf16_to_f32((bf16_t)(r.x >> 16)), bf16_to_f32((bf16_t)r.y), bf16_to_f32((bf16_t)(r.y >> 16))};
          if constexpr (T::TAB) {   // + 0 x: of an infinity or a NaN the derivative is NaN
            const uint32_t o0 = gelu_tab_offsets(r.x), o1 = gelu_tab_offsets(r.y);
            c[u][0] *= fmaf(x[0], 0.f, entry(o0 & 0xffffu)); c[u][1] *= fmaf(x[1], 0.f, entry(o0 >> 16));
            c[u][2] *= fmaf(x[2], 0.f, entry(o1 & 0xffffu)); c[u][3] *= fmaf(x[3], 0.f, entry(o1 >> 16));
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) c[u][e] *= dgelu_f(x[e]);
          }
        }
      }
      if (C32 != nullptr) {
#pragma unroll
        for (int u = 0; u < CH; ++u)
          if (exists(x * 32 + row_of(q, u))) *reinterpret_cast<float4*>(C32 + step(q, u) + lane_off) = make_float4(c[u][0], c[u][1], c[u][2], c[u][3]);
      }
      if (C16 != nullptr) {
#pragma unroll
        for (int u = 0; u < CH; ++u)
          if (exists(x * 32 + row_of(q, u))) *reinterpret_cast<uint2*>(C16 + step(q, u) + lane_off) = make_uint2(pack_bf16x2(c[u][0], c[u][1]), pack_bf16x2(c[u][2], c[u][3]));
      }
    }
  };
  if (i0 + wr >= Mrows) return;
  if (i0 + BM <= Mrows) epilogue(std::true_type{});
  else epilogue(std::false_type{});
}

template <typename T, bool A_KC, bool B_KC>
void launch_tile(ProfScope& ps, hipStream_t st, const GemmBf16Args* p, int count, int group) {
  static bool configured = false;      // per instantiation: raise the dynamic LDS limit once
  if (!configured) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_bf16<T, A_KC, B_KC>), hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
    configured = true;
  }
  GemmBatch b{};
  b.count = count; b.group = group;
  int nt = 0;
  for (int k = 0; k < count; ++k) {
    b.p[k] = p[k];
    b.first_tile[k] = nt;
    nt += ((p[k].N + T::BN - 1) / T::BN) * ((p[k].M + T::BM - 1) / T::BM);
  }
  for (int k = count; k <= GEMM_MAX_BATCH; ++k) b.first_tile[k] = nt;
  const int per_xcd = (nt + 7) / 8;
  launch_kernel(ps, k_gemm_bf16<T, A_KC, B_KC>, 8 * per_xcd, T::THREADS, T::LDS_BYTES, st, b, nt, per_xcd);
}

// Tiles <BM, BN, BK, multiplying waves in M, in N, stages, hi + lo, loading waves, operands fetched one step at a time>
// The 32 x 32 ones are for products of few rows (scoring one text), which a larger tile leaves to a few dozen workgroups that walk
// the contraction slab by slab: with twice as many and five slabs in flight, 128 rows of 768 x 3072 take 14.1 us hi + lo
// (64 x 32: 17.9) and 10.7 single-term (64 x 64: 17.2).  Splitting the contraction over the waves of a workgroup was
// 0.8 us faster, but sums in another order, so that a text scored alone came out otherwise than in a batch.
typedef Tile<256, 256, 64, 2, 4, 2, false> S1;
typedef Tile<256, 192, 64, 4, 2, 2, false, 4, true> S2;
typedef Tile<256, 128, 64, 4, 2, 3, false, 4, true> S3;
typedef Tile<128, 128, 64, 4, 2, 4, false, 4> S4;
typedef Tile<128, 64, 64, 4, 2, 4, false, 4> S5;
typedef Tile<64, 64, 64, 2, 2, 4, false> S6;         // two workgroups per CU
typedef Tile<128, 128, 64, 4, 2, 2, false> S7;       // two workgroups per CU
typedef Tile<32, 32, 64, 1, 1, 6, false, 2> S8;      // three workgroups per CU
typedef Tile<256, 192, 64, 4, 2, 2, true, 4, true> D1;
typedef Tile<256, 128, 64, 4, 2, 2, true, 4> D2;
typedef Tile<128, 128, 64, 4, 2, 3, true, 4> D3;
typedef Tile<128, 96, 64, 4, 1, 3, true, 4> D4;
typedef Tile<128, 64, 64, 4, 2, 4, true, 4> D5;
typedef Tile<64, 64, 64, 2, 2, 4, true, 2> D6;
typedef Tile<64, 64, 64, 2, 2, 3, true, 2> D7;       // two workgroups per CU
typedef Tile<64, 32, 64, 2, 1, 4, true, 1> D8;       // two workgroups per CU
typedef Tile<32, 32, 64, 1, 1, 6, true, 2> D9;       // two workgroups per CU

// What a launch costs with a tile, in us, beyond what it costs with any: per round, epilogue + 64-deep slabs x time of a slab.
// A round is up to `per_cu` tiles on each of the 256 CUs; a slab takes `few` with a handful of tiles on the chip, `one` with one
// on every CU and, where two fit, `two` as soon as some CU holds two and `all` when every one does; in between in proportion.
// The numbers are robust least-squares fits of the logarithms over 2561 timed problems (widths 192 to 2048, FFN 2 and 4 times that,
// 64 to 8192 rows: NT, NN, pairs of NT, a layer's four TN problems in a launch; the vocabulary head's products over 8192 to
// 50304 tokens; weights cold), taken when the GELU epilogues computed their factors and averaged over the kinds of epilogue.  On the
// times of the kernels as they are, picking by them takes 0.9% (hi + lo) and 1.2% (single-term) longer in total than the fastest
// tile of each problem, a fit of these 0.6% and 1.2%; GELU backward 1.7%, the head's products 0.4 to 3.3%: profiles/gemm_tile_costs.md.
struct TileCost { int id, bm, bn, per_cu; double few, one, two, all, epilogue; };
constexpr TileCost SINGLE[] = {
    {1, 256, 256, 1, 1.282, 1.816, 0, 0, 8.26}, {2, 256, 192, 1, 1.060, 1.218, 0, 0, 8.62},
    {3, 256, 128, 1, 0.561, 0.923, 0, 0, 6.42}, {4, 128, 128, 1, 0.427, 0.600, 0, 0, 3.55},
    {5, 128, 64, 1, 0.322, 0.419, 0, 0, 2.08},  {6, 64, 64, 2, 0.257, 0.282, 0.470, 0.486, 1.36},
    {7, 128, 128, 2, 0.714, 0.828, 0.828, 1.167, 3.94}, {8, 32, 32, 3, 0.160, 0.202, 0.282, 0.381, 1.03}};
constexpr TileCost HILO[] = {
    {11, 256, 192, 1, 1.425, 2.186, 0, 0, 12.13}, {12, 256, 128, 1, 1.072, 1.533, 0, 0, 7.70},
    {13, 128, 128, 1, 0.672, 0.928, 0, 0, 4.58},  {14, 128, 96, 1, 0.671, 0.782, 0, 0, 4.52},
    {15, 128, 64, 1, 0.491, 0.603, 0, 0, 2.46},   {16, 64, 64, 1, 0.435, 0.435, 0, 0, 1.66},
    {17, 64, 64, 2, 0.449, 0.469, 0.723, 0.723, 1.59}, {18, 64, 32, 2, 0.320, 0.341, 0.528, 0.528, 1.42},
    {19, 32, 32, 2, 0.236, 0.255, 0.381, 0.381, 1.28}};

int g_force_shape = 0, g_group = 8;

// Cost of a launch with `share` quarters of a padded batch's rows in use.
double launch_cost(const TileCost& c, const GemmBf16Args* p, int count, int share) {
  int64_t tiles = 0;
  double slabs = 0.0;                                    // of all tiles
  for (int k = 0; k < count; ++k) {
    const int64_t part = p[k].rows != nullptr ? share : 4, M = p[k].a_trans ? p[k].M : (p[k].M * part + 3) / 4, K = p[k].a_trans ? (p[k].K * part + 3) / 4 : p[k].K;
    const int64_t t = ((M + c.bm - 1) / c.bm) * ((p[k].N + c.bn - 1) / c.bn);
    tiles += t;
    slabs += (double)t * K / 64.0;
  }
  slabs /= (double)tiles;
  const int64_t cap = 256 * c.per_cu, rest = tiles % cap;
  double cost = (double)(tiles / cap) * (slabs * (c.per_cu > 1 ? c.all : c.one) + c.epilogue);
  if (rest > 0) {
    const double slab = rest <= 256 ? c.few + (c.one - c.few) * (double)rest / 256.0 : c.two + (c.all - c.two) * (double)(rest - 256) / (double)(cap - 256);
    cost += slabs * slab + c.epilogue;
  }
  return cost;
}

// How many rows of a padded batch are in use only the device knows, and how long texts are is the caller's: the tile is the one
// that costs least in total over batches a quarter, half, three quarters and all in use.  Longer than the fastest tile of a
// product at each of these (geometric means over the same timed problems): 16, 6, 7 and 9%; choosing for one share in between, two
// thirds, 30, 11, 5 and 8%, for all rows 37, 16, 5 and 2%.
template <int N>
int pick_tile(const TileCost (&costs)[N], const GemmBf16Args* p, int count) {
  bool padded = false;
  for (int k = 0; k < count; ++k) padded = padded || p[k].rows != nullptr;
  int best = 0;
  double best_cost = 0.0;
  for (const TileCost& c : costs) {
    double cost = 0.0;
    for (int share = padded ? 1 : 4; share <= 4; ++share) cost += launch_cost(c, p, count, share);
    if (best == 0 || cost < best_cost) { best = c.id; best_cost = cost; }
  }
  return best;
}

template <bool A_KC, bool B_KC>
void launch_class(ProfScope& ps, hipStream_t st, const GemmBf16Args* p, int count) {
  const bool dual = p[0].B2 != nullptr;
  int shape = g_force_shape;
  if (shape >= 11 && !dual) shape = 0;   // hi + lo tiles read B2
  if (shape == 0) shape = dual ? pick_tile(HILO, p, count) : pick_tile(SINGLE, p, count);
  switch (shape) {
    case 1: launch_tile<S1, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 2: launch_tile<S2, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 3: launch_tile<S3, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 4: launch_tile<S4, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 5: launch_tile<S5, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 6: launch_tile<S6, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 8: launch_tile<S8, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 11: launch_tile<D1, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 12: launch_tile<D2, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 13: launch_tile<D3, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 14: launch_tile<D4, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 15: launch_tile<D5, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 16: launch_tile<D6, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 17: launch_tile<D7, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 18: launch_tile<D8, A_KC, B_KC>(ps, st, p, count, g_group); break;
    case 19: launch_tile<D9, A_KC, B_KC>(ps, st, p, count, g_group); break;
    default: launch_tile<S7, A_KC, B_KC>(ps, st, p, count, g_group); break;
  }
}
}  // namespace

__global__ __launch_bounds__(256) void k_gelu_tables(float* __restrict__ tab) {
  const int i = blockIdx.x * 256 + threadIdx.x, sign = blockIdx.y;
  if (i >= GELU_TAB_ENTRIES) return;
  const float x = bf16_to_f32((bf16_t)((GELU_TAB_FIRST + i) | sign << 15));
  tab[(sign << 12) + i] = gelu_cdf_f(x);
  tab[GELU_TAB_BYTES / 4 + (sign << 12) + i] = dgelu_f(x);
}
size_t gelu_table_bytes() { return 2 * GELU_TAB_BYTES; }
void launch_gelu_tables(hipStream_t st, float* tab) {
  ProfScope ps(st, F_OTHER, 0.0);
  launch_kernel(ps, k_gelu_tables, dim3((GELU_TAB_ENTRIES + 255) / 256, 2), 256, 0, st, tab);
}

const char* check_gemm_bf16(const GemmBf16Args& a) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) return "empty GEMM";
  if (a.K % 64 != 0) return "K must be a multiple of 64";
  if (a.M % 8 != 0 || a.N % 8 != 0) return "M and N must be multiples of 8";
  if (a.lda % 8 != 0 || a.ldb % 8 != 0 || a.ldc % 4 != 0) return "leading dimensions must be multiples of 8 (A, B) and 4 (C)";
  if (((uintptr_t)a.A | (uintptr_t)a.B | (uintptr_t)a.B2 | (uintptr_t)a.bias | (uintptr_t)a.bias_v | (uintptr_t)a.C32 |
       (uintptr_t)a.res32) & 15) return "operands, bias, fp32 residual and fp32 output must be 16-byte aligned";
  if (((uintptr_t)a.C16 | (uintptr_t)a.C16_pre | (uintptr_t)a.aux16) & 7) return "bf16 epilogue tensors must be 8-byte aligned";
  if (a.act != GEMM_ACT_NONE && (a.gelu_tab == nullptr || ((uintptr_t)a.gelu_tab & 15) != 0)) return "the GELU epilogues need their 16-byte aligned table";
  if (a.res32 != nullptr && a.act == GEMM_ACT_GELU_BWD) return "a residual and the GELU backward exclude each other";
  if (a.lda < (a.a_trans ? a.M : a.K) || a.ldb < (a.b_trans ? a.K : a.N) || a.ldc < a.N) return "leading dimension too small";
  const int64_t abytes = (int64_t)(a.a_trans ? a.K : a.M) * a.lda * 2, bbytes = (int64_t)(a.b_trans ? a.N : a.K) * a.ldb * 2;
  if (abytes >= ((int64_t)1 << 31) || bbytes >= ((int64_t)1 << 31)) return "operands must be smaller than 2 GiB";
  return nullptr;
}

void gemm_bf16_force_shape(int s) { g_force_shape = s % 100; g_group = s >= 100 ? s / 100 : 8; }

const char* check_gemm_bf16_batch(const GemmBf16Args* p, int count) {
  if (count < 1 || count > GEMM_MAX_BATCH) return "batch of 1 to 4 problems";
  for (int k = 0; k < count; ++k) {
    if (const char* e = check_gemm_bf16(p[k])) return e;
    if (p[k].a_trans != p[0].a_trans || p[k].b_trans != p[0].b_trans || (p[k].B2 != nullptr) != (p[0].B2 != nullptr))
      return "the problems of a batch must share operand storage and the hi + lo form";
  }
  return nullptr;
}

static const char* g_launch_error = nullptr;
void note_launch_error(const char* what) { if (g_launch_error == nullptr) g_launch_error = what; }
const char* take_launch_error() { const char* e = g_launch_error; g_launch_error = nullptr; return e; }

void launch_gemm_bf16_batch(hipStream_t st, const GemmBf16Args* p, int count) {
  if (const char* e = check_gemm_bf16_batch(p, count)) { note_launch_error(e); return; }   // never run a shape the tiles cannot cover
  double flops = 0.0;
  for (int k = 0; k < count; ++k) flops += 2.0 * p[k].M * p[k].N * p[k].K * (p[k].B2 ? 2.0 : 1.0);   // hi + lo contracts over 2K
  const bool hilo = p[0].B2 != nullptr;
  ProfScope ps(st, p[0].a_trans ? F_GEMM_TN : (p[0].b_trans ? (hilo ? F_GEMM_NT_HILO : F_GEMM_NT) : (hilo ? F_GEMM_NN_HILO : F_GEMM_NN)), flops);
  // a_trans = 0: A is [M][K], contraction contiguous.  b_trans = 1: B is [N][K], contraction contiguous.
  if (!p[0].a_trans && p[0].b_trans) launch_class<true, true>(ps, st, p, count);
  else if (!p[0].a_trans && !p[0].b_trans) launch_class<true, false>(ps, st, p, count);
  else if (p[0].a_trans && !p[0].b_trans) launch_class<false, false>(ps, st, p, count);
  else launch_class<false, true>(ps, st, p, count);
}

void launch_gemm_bf16(hipStream_t st, const GemmBf16Args& a) { launch_gemm_bf16_batch(st, &a, 1); }

}  // namespace sama
