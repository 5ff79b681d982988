// bf16 x bf16 -> fp32 contraction on the gfx950 matrix cores (v_mfma_f32_16x16x32_bf16) for the encoder's linear
// layers: forward (X W^T), dgrad (dY W) and wgrad (dY^T X) are one kernel template over the storage of its two
// operands.
//
//   16 x 16 x 32 and not 32 x 32 x 16: the large tiles are bound by power, and an issue loop fed from registers (256 workgroups of 8 waves,
//   normal values) holds 2030 TFLOP/s at 1.98 GHz with the one and 1790 at 1.76 with the other.  Both add 16 products at a time in
//   order and agree bit for bit.  us per launch, 32 x 32 x 16 / 16 x 16 x 32: 8192 x 1024 x 4096 hi + lo (256 x 128 tiles) 110 / 97,
//   8192 x 4096 x 1024 123 / 115
//   operand slabs go global -> LDS directly (global_load_lds_dwordx4, 1 KB per wave instruction) into dense,
//   XOR-swizzled stages, NSTAGE - 1 slabs in flight, one barrier per slab; no staging registers
//   most tiles have waves that do nothing but issue those loads: a wave that issues a slab's loads itself waits for the
//   address units to take them, a third of the slab's matrix time, before it multiplies.  Against the same tile without them:
//   256 x 128 hi + lo 6%, 128 x 128 10%, 128 x 96 11%, 128 x 64 4% faster, 128 x 128 single-term TN 16% (geometric means
//   over 65 and 51 problems); four such waves are 4% faster than two, eight the same as four
//   an operand whose contraction index is contiguous in memory is staged [row][k] and fetched with 16-byte reads;
//   one whose contraction index is the strided one (dgrad's W, both operands of wgrad) is staged as it lies in
//   memory, [k][row], and fetched with the transposing LDS read (ds_read_b64_tr_b16)
//   the MFMA operands of the next piece of a slab are fetched between the MFMAs of the current one, also across the slab boundary
//   measured on MI355X: a CU takes in 56 B/clk where L2 holds the slabs, 40 from the last-level cache and 26 where the weights
//   come from memory, and at the MFMA peak 256 x 256 tiles need 32 B/clk, 256 x 128 48, 128 x 128 64: small tiles are bound by
//   this, and the weights of a product of few rows are fetched by the launch before it (k_ln_fwd, k_ln_bwd).  (profiles/gemm_bounds.md)
//   workgroup ids are remapped so that each XCD (own L2) works on a compact patch of tiles
//   what runs before a workgroup's first load and behind its last product is short straight code
//
// For the theta +- eps v passes of Eq. 5 and the direct-gradient pass the weight operand is hi + lo (two bf16
// halves).  DUAL tiles stage the A slab once together with the hi and the lo slab of B, and an MFMA contracts 16 values of A with those of hi,
// then with those of lo.  That order of the sums is kept: a hypergradient, a difference of two nearly equal gradients, has moved by up to 10% of its
// size where it was given up.  It costs a second read of every fragment of A from LDS: with 32 values of hi and then 32 of lo, which needs none,
// products take 0.5% (256 x 192 tiles) to 5% (input gradients, 128 x 64) less.  Read once and doubled in registers (v_permlane32_swap) they
// take longer: scoring 8192 rows of 24 x 1024 9.41 ms, this way 8.88.
// How a tile is cut into waves decides what is read per product: 64 x 32 of a wave in 128 x 128 and 128 x 64 tiles, where it was 32 x 64 and 32 x 32:
// 4096 x 1024 x 4096 NT 61.4 / 60.0, NN 67.3 / 65.4, 2048 x 1024 x 4096 NT 36.8 / 35.9, NN 38.3 / 36.8; 128 x 96 tiles with 64 x 32 for 32 x 96 NT 0.7% faster,
// NN 2.7% slower (geometric means of 29 and 30 problems).
//
// Several independent problems of one storage class can share a launch (the + and - pass of Eq. 5, the four weight
// gradients of a layer): more tiles per launch for the small per-layer shapes.
//
// Fused epilogues: + bias (fp32, optionally perturbed), + residual (fp32), GELU forward (writes both the
// pre-activation and the activation), GELU backward (multiplies by gelu'(pre)), fp32 and/or bf16 stores.  The large hi + lo
// tiles look the GELU factors up in a table that their loading waves bring into LDS during the last slab.
#include <algorithm>
#include <atomic>
#include <type_traits>
#include <utility>
#include "common.h"
#include "gelu.h"
#include "kernels.h"

namespace sama {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void gvoid;
constexpr int LDS_MAX = 160 * 1024;

// PW: waves that only load (0: the multiplying waves load for themselves).  YP: 16-column fragments of B per piece of a k-step, 0: all.
// RD: how the fetches of a piece lie between the products of the one before: n: over the first 1 / n of them; 0: with a strided operand right
// before its own products (fewer registers, the order left to the compiler: 2 to 8% faster with three stages and for 256 x 256), else all
// ahead of those products.
template <int BM_, int BN_, int BK_, int WGM_, int WGN_, int NSTAGE_, bool DUAL_, int PW_ = 0, int YP_ = 0, int RD_ = 2, int TW_ = 0>
struct Tile {
  static constexpr int PW = PW_, RD = RD_, TW = TW_;
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WGM = WGM_, WGN = WGN_, NSTAGE = NSTAGE_;
  static constexpr bool DUAL = DUAL_;
  static constexpr int WAVES = WGM * WGN, LW = PW > 0 ? PW : WAVES, THREADS = (WAVES + PW + TW) * 64;   // multiplying, loading
  // TW: 1: a wave that touches the weights ahead of the loads (see the kernel)
  static_assert(TW == 0 || PW > 0, "a touching wave only beside loading ones");
  static constexpr int WM = BM / WGM, WN = BN / WGN, XT = WM / 16, YT = WN / 16;
  static constexpr int YP = YP_ > 0 ? YP_ : YT, NP = YT / YP;               // pieces of a k-step
  static_assert(WM % 16 == 0 && WN % 32 == 0 && YT % YP == 0, "wave tiles");
  static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE_BYTES = A_BYTES + (DUAL ? 2 : 1) * B_BYTES;
  static constexpr int NLA = A_BYTES / 1024 / LW, NLB = B_BYTES / 1024 / LW;   // 1 KB loads of a loading wave per slab
  static constexpr int NL = NLA + (DUAL ? 2 : 1) * NLB;
  static constexpr int LDS_BYTES = NSTAGE * STAGE_BYTES;
  static_assert(LDS_MAX >= LDS_BYTES, "stages exceed the 160 KB of LDS");
  // Whether the GELU epilogues look their values up (gelu.h).  The table comes into a stage that the last slab does not use, while
  // that slab is multiplied.  Computed, a value is 26 quarter-rate vector instructions in which the matrix cores stand still; looked up it
  // is seven and an LDS read.  us computed / looked up, forward: 2048 x 4096 x 1024 (256 x 128 tiles) 37.3 / 34.5, 4096 x 3072 x 768 (256 x
  // 192) 47.1 / 40.8, 1024 x 3072 x 768 (128 x 128) 19.6 / 18.0, (128 x 96) 19.2 / 17.9 (with 32 x 32 x 16 MFMAs and the epilogue through LDS).  The 128 x 64 and smaller tiles compute: the table
  // would be as much to load as a slab of them or more.
  static constexpr bool TAB = DUAL && PW > 0 && BM * BN >= 128 * 96;
  static_assert(!TAB || (NSTAGE >= 2 && STAGE_BYTES >= GELU_TAB_BYTES), "room for the table");
  static_assert(A_BYTES % (1024 * LW) == 0 && B_BYTES % (1024 * LW) == 0, "slab must split into whole wave loads");
  static_assert(NL * (NSTAGE - 2) <= 63, "vmcnt range");
};

// Byte offset (relative to the slab's first element in global memory) of the 16-byte piece that belongs at byte
// `ldsoff` of an operand's dense LDS stage.
//   KC (contraction contiguous, storage [rows][k]): stage [R][BK]; the 16-byte chunk index within a row is XORed
//     with (row / RP) % NCH so that 16 consecutive rows at one logical chunk fill all 64 banks.
//   KS (contraction strided, storage [k][rows]): stage [BK][R]; the 32-byte chunk index within a k-row is XORed with
//     chunk_swizzle(k-row) so that the eight k-rows that half a wave of a transposing read touches fill all 64 banks.
// Rows past `nrows` are clamped (their products land in outputs the epilogue never stores).
// A k-row of R values is R / 16 chunks of 32 bytes.  Half a wave reads one chunk of the k-rows 0..3 and 8..11 (or these plus 4, 16 or
// 20), and the eight have to lie in eight different eighths of the banks.  Rows a multiple of eight chunks long all start at the same
// bank; rows of four or twelve chunks at two alternating halves, so that two bits have to tell the four k-rows of one parity apart; rows of two
// or six chunks spread four neighbours, and one bit tells k-rows eight apart.
template <int R>
__device__ __forceinline__ int chunk_swizzle(int kr) {
  constexpr int NC = R / 16;
  static_assert(NC % 8 == 0 || NC == 4 || NC == 12 || NC == 2 || NC == 6, "tile width");
  return NC % 8 == 0 ? (kr & 3) | ((kr >> 1) & 4) : NC % 4 == 0 ? ((kr >> 1) & 1) | ((kr >> 2) & 2) : (kr >> 3) & 1;
}
template <bool KC, int R, int BK>
__device__ __forceinline__ uint32_t piece_offset(uint32_t ldsoff, uint32_t row0, uint32_t nrows, uint32_t ld) {
  if (KC) {
    constexpr uint32_t RB = BK * 2, RP = 256 / RB, NCH = RB / 16;
    const uint32_t r = ldsoff / RB, p = (ldsoff % RB) / 16;
    const uint32_t c = p ^ ((r / RP) % NCH);
    return min(row0 + r, nrows - 1) * ld * 2 + c * 16;
  } else {
    constexpr uint32_t RBS = R * 2;
    const uint32_t kr = ldsoff / RBS, q16 = (ldsoff % RBS) / 16;
    const uint32_t ql = (((q16 >> 1) ^ (uint32_t)chunk_swizzle<R>((int)kr)) << 1) | (q16 & 1);
    return kr * ld * 2 + min(row0 + ql * 8, nrows - 8) * 2;
  }
}
// The offsets of the NLOADS loads of wave `lw` of LW, which lie LW KB apart in the stage.  Where the swizzle repeats after P loads and no row
// is clamped, load q is load q - P a uniform distance further on: few instructions, because all of them run before a workgroup's first load.
template <bool KC, int R, int BK, int LW, int NLOADS>
__device__ __forceinline__ void load_offsets(uint32_t (&off)[NLOADS], uint32_t lw, uint32_t lane, uint32_t row0, uint32_t nrows, uint32_t ld) {
  constexpr uint32_t ROW = KC ? BK * 2 : R * 2;     // bytes of a row of the stage
  auto repeats = [](int p) { return p * LW * 1024 % ROW == 0 && p * LW * 1024 / ROW % 16 == 0; };
  constexpr int P = repeats(1) ? 1 : repeats(2) ? 2 : repeats(3) ? 3 : NLOADS;
#pragma unroll
  for (int q = 0; q < NLOADS && q < P; ++q) off[q] = piece_offset<KC, R, BK>((q * LW + lw) * 1024 + lane * 16, row0, nrows, ld);
  if constexpr (P < NLOADS) {
    if (!KC || row0 + R <= nrows) {   // (of a strided operand the columns are clamped, the same in each load)
      const uint32_t step = P * LW * 1024 / ROW * ld * 2;
#pragma unroll
      for (int q = P; q < NLOADS; ++q) off[q] = off[q - P] + step;
    } else {
#pragma unroll
      for (int q = P; q < NLOADS; ++q) off[q] = piece_offset<KC, R, BK>((q * LW + lw) * 1024 + lane * 16, row0, nrows, ld);
    }
  }
}

// MFMA operand out of a swizzled stage: the lane-dependent part of its address, for a k-step (KC) or for a 16-row fragment of the tile
// (KS).  A lane has 8 contraction values of tile row tb + lane % 16: of a single-term product k = 32 ks + 8 (lane / 16) + 0..7; of a hi + lo
// one 16 ks + 8 (lane / 16 % 2) + 0..7, lanes 0..31 of the hi half of B and 32..63 of the lo half, and A the same in both: the matrix core adds
// the 32 products of an instruction 16 at a time in order, so that one instruction is 16 of hi, then 16 of lo.
template <bool KC, int R, int BK, bool HALVES>
__device__ __forceinline__ int fetch_lane_offset(int lane, int ks_or_frag) {
  const int part = HALVES ? (lane >> 4) & 1 : lane >> 4;
  if (KC) {
    constexpr int RB = BK * 2, RP = 256 / RB, NCH = RB / 16;
    static_assert(16 % RP == 0 && (16 / RP) % NCH == 0, "the swizzle repeats from fragment to fragment");
    const int rl = lane & 15;
    const int s = (rl / RP) % NCH;
    return rl * RB + ((((HALVES ? 2 : 4) * ks_or_frag + part) ^ s) * 16);
  } else {
    constexpr int RBS = R * 2;
    const int j = lane & 15;
    const int kr = 8 * part + (j >> 2);                                   // the swizzle is the same for kr + 4, kr + 16 and kr + 32
    return kr * RBS + ((ks_or_frag ^ chunk_swizzle<R>(kr)) * 32) + 8 * (j & 3);
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

// What the loop needs of a problem.
struct LoopArgs {
  const bf16_t *A, *B, *B2;
  uint32_t lda, ldb;
  int M, N, K, act;
  const int32_t* rows;
  const float* gelu_tab;
};
__host__ __device__ __forceinline__ LoopArgs loop_args(const GemmBf16Args& a) {
  return LoopArgs{a.A, a.B, a.B2, (uint32_t)a.lda, (uint32_t)a.ldb, a.M, a.N, a.K, a.act, a.rows, a.gelu_tab};
}
struct GemmBatch {
  LoopArgs first;      // of problem 0
  int ntiles, tiles_per_xcd, count, group;
  int first_tile[GEMM_MAX_BATCH + 1];   // tile ids [first_tile[k], first_tile[k + 1]) belong to problem k
  int kind[GEMM_MAX_BATCH];             // of each epilogue
  uint64_t choice;                      // k_gemm_rows: four bits for each sixteenth of the rows, the tile to take where as many are in use
  GemmBf16Args p[GEMM_MAX_BATCH];
};
enum { EPI_ANY, EPI_C16, EPI_C32, EPI_RES32, EPI_GELU_FWD, EPI_GELU_BWD, EPI_LN32 };

template <typename F, int... I>
__device__ __forceinline__ void static_for_each(std::integer_sequence<int, I...>, F f) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>   // f(0), ..., f(N - 1) with constants
__device__ __forceinline__ void static_for(F f) { static_for_each(std::make_integer_sequence<int, N>{}, f); }

// a / b for a below 2^20 and b > 0, both the same in every lane: (a + 1/2) / b is at least 1 / (2 b) from any whole number, a relative
// distance above 2^-21, and the approximate quotient is closer to it than that.
__device__ __forceinline__ uint32_t small_quotient(uint32_t a, uint32_t b) {
  return __builtin_amdgcn_readfirstlane((uint32_t)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)b)));
}
constexpr int SMALL_TILES = 1 << 20;

// What runs before a workgroup's first load is short, and the loading waves run nothing else: with 400 instructions of signed index arithmetic
// (two integer divisions, a bounds check for each offset), scalar loads that waited for each other and a branch every dozen of them (a taken one
// is 35 clk) it took 1.8 to 2.7 us from a workgroup's start to its first load; with the 150 here 0.5 to 0.6 us.  us per launch before / after,
// hi + lo: 128 x 3072 x 768 7.4 / 6.5, 2048 x 1024 x 1024 11.1 / 10.4, 2048 x 4096 x 1024 30.9 / 29.3.
// LN: the residual is a LayerNorm's output and made here of its input; a kernel of its own, because with one more kind of epilogue the others of the 256 x 128 tile kept 52 bytes
// a lane in scratch, small products took 1% longer, and the compiler gave up on k_gemm_rows.
template <typename T, bool A_KC, bool B_KC, bool LN = false>
__device__ __forceinline__ void gemm_tile(const GemmBatch& batch) {
  constexpr int BM = T::BM, BN = T::BN, BK = T::BK, XT = T::XT, YT = T::YT, NSTAGE = T::NSTAGE, WAVES = T::WAVES;
  constexpr bool DUAL = T::DUAL;
  static_assert(!LN || (DUAL && A_KC && B_KC), "forward hi + lo products");
  constexpr int RD = (DUAL && !B_KC && NSTAGE == 3) || (T::RD == 0 && !(A_KC && B_KC)) ? 0 : T::RD == 0 ? 9 : T::RD;   // see Tile
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // XCD-aware order: workgroups are dealt round-robin to the 8 XCDs; each XCD gets a contiguous run of tile ids, and
  // tile ids walk down `group` tile rows before moving one tile column to the right, so that the tiles in flight on
  // one XCD form a compact patch (few distinct A and B panels in its L2).
  // Where the rows in use are known on the device only, the launch has the tiles of all rows, and the order is made here over
  // those in use (the problems of a batch then have the same rows).
  // What the loop needs of problem 0 is read with the kernel's first arguments: an index into them that is computed first costs another
  // trip to memory, 0.2 us, and most launches have one problem.
  LoopArgs la = batch.first;
  const uint32_t ntiles = batch.ntiles, count = batch.count, group = batch.group;
  uint32_t per_xcd = batch.tiles_per_xcd;
  asm("" : "+s"(la.A), "+s"(la.B), "+s"(la.B2), "+s"(la.lda), "+s"(la.ldb), "+s"(la.M), "+s"(la.N), "+s"(la.K), "+s"(la.act), "+s"(la.rows));
  auto in_use = [](const int32_t* rows) { return (uint32_t)*(const __attribute__((address_space(4))) int32_t*)rows; };   // nobody writes it now: a scalar load
  const bool fewer_tiles = A_KC && la.rows != nullptr;
  uint32_t Mrows = 0;
  if (fewer_tiles) Mrows = in_use(la.rows);
  uint32_t pid, prob = 0;
  if (fewer_tiles) {
    const uint32_t gy = (Mrows + BM - 1) / BM;
    uint32_t n = gy * (((uint32_t)la.N + BN - 1) / BN);
    for (uint32_t k = 1; k < count; ++k) n += gy * (((uint32_t)batch.p[k].N + BN - 1) / BN);
    per_xcd = (n + 7) / 8;
    pid = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per_xcd || pid >= n) return;
    for (uint32_t k = 0; k + 1 < count; ++k) {
      const uint32_t t = gy * (((uint32_t)batch.p[k].N + BN - 1) / BN);
      if (pid < t) break;
      pid -= t;
      prob = k + 1;
    }
  } else {
    pid = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (pid >= ntiles) return;
    if (count > 1) {
      uint32_t before = 0;
#pragma unroll
      for (uint32_t k = 1; k < GEMM_MAX_BATCH; ++k)
        if (k < count && pid >= (uint32_t)batch.first_tile[k]) { prob = k; before = batch.first_tile[k]; }
      pid -= before;
    }
  }
  const GemmBf16Args& a = batch.p[prob];   // for the epilogue
  if (prob != 0) la = loop_args(a);
  const uint32_t rows_of = fewer_tiles ? Mrows : (uint32_t)la.M;
  const uint32_t gx = ((uint32_t)la.N + BN - 1) / BN, gy = (rows_of + BM - 1) / BM, width = group * gx;
  uint32_t grp, tj, ti;
  if (ntiles < SMALL_TILES) {
    grp = small_quotient(pid, width);
    const uint32_t gsz = min(gy - grp * group, group), rest = pid - grp * width;
    tj = small_quotient(rest, gsz); ti = grp * group + rest - tj * gsz;
  } else {
    grp = pid / width;
    const uint32_t gsz = min(gy - grp * group, group), rest = pid - grp * width;
    tj = rest / gsz; ti = grp * group + rest - tj * gsz;
  }
  const uint32_t i0 = ti * BM, j0 = tj * BN;

  int nk = la.K / BK;
  if (!A_KC && la.rows != nullptr) nk = (int)in_use(la.rows) / BK;   // the problems of a launch need not agree in this
  const int iters = (!DUAL && la.B2 != nullptr) ? 2 * nk : nk;   // non-DUAL tiles contract with hi, then with lo

  // the GELU table's place: at the bottom, or at the top if the last slab is at the bottom
  const bool look_up = T::TAB && la.act != GEMM_ACT_NONE;
  const int tab_at = (iters - 1) % NSTAGE == 0 ? T::LDS_BYTES - GELU_TAB_BYTES : 0;
  const uint32_t lw = T::PW > 0 ? wave - WAVES : wave;            // number among the loading waves
  const bool loader = T::PW == 0 || wave >= WAVES;
  if constexpr (T::TW > 0) {
    if (wave == WAVES + T::PW) {
      // Lines of the weights' next eight slabs, a word of each: an eighth of them for each of the up to eight workgroups of an XCD that read them.
      // Weights in memory come slowly a slab at a time, 128 bytes of a row (or a few hundred of a k-row) here and there, however many slabs are
      // in flight; a kilobyte of a row at once comes faster, and the slabs then find it in L2.  us without / with, weights cold (1.2 GB in turn):
      // hi + lo 2048 x 1024 x 4096 NT 36.5 / 34.4, NN 42.1 / 36.5 (128 x 64 tiles), 1024 x 1024 x 4096 NT 27.6 / 23.7, NN 36.3 / 25.0 (64 x 64);
      // weights warm 33.1 / 33.2, 34 / 34.6, 20.8 / 22.8, 24.8 / 23.3.  With fewer than 32 slabs there is no time for it (2048 x 1024 x 1024
      // 10.1 / 10.9); done by a multiplying wave it costs all tiles 1 to 2 us; 128 x 128 tiles gain 2 us of 49 here and lose 1.5 of 41 there.
      // Whole calls without it: scoring 2048 rows of 24 x 1024 +2.9%, base step of 1536 +1.2%, and where the caches hold the weights -1.9 to +0.5%; told
      // so by the encoder and left out there, calls gained up to 1.8 and lost up to 3.4%.
      constexpr int TS = 8, TN = (BN + 63) / 64;   // slabs of a chunk, loads for an eighth of its lines
      static_assert(!T::TAB, "no barrier for the table");
      if (iters < 4 * TS) return;
      uint32_t off[TN], got = 0;
      const uint32_t part = ti & 7;
#pragma unroll
      for (int u = 0; u < TN; ++u) {
        if (B_KC) off[u] = min(j0 + part * (BN / 8) + u * 8 + lane / 8, (uint32_t)la.N - 1) * la.ldb * 2 + lane % 8 * 128;   // a line is a row's 64 values
        else off[u] = (part * 64 + lane) * la.ldb * 2 + min(j0 + u * 64, (uint32_t)la.N - 8) * 2;                             // or 64 columns of a k-row
      }
      const uint32_t step = B_KC ? TS * BK * 2 : TS * BK * la.ldb * 2;
      auto touch = [&](int chunk) {
        if ((chunk + 1) * TS > iters) return;
        const uint64_t at = (uint64_t)chunk * step;
#pragma unroll
        for (int u = 0; u < TN; ++u) asm volatile("global_load_dword %0, %1, %2" : "+v"(got) : "v"(off[u]), "s"(reinterpret_cast<const char*>(la.B) + at) : "memory");
        if (DUAL) {
#pragma unroll
          for (int u = 0; u < TN; ++u) asm volatile("global_load_dword %0, %1, %2" : "+v"(got) : "v"(off[u]), "s"(reinterpret_cast<const char*>(la.B2) + at) : "memory");
        }
      };
      touch(0);
      for (int i = 0; i < iters; ++i) {
        __builtin_amdgcn_s_barrier();
        if (i % TS == 0) touch(i / TS + 1);
      }
      asm volatile("s_waitcnt vmcnt(0)" : "+v"(got)::"memory");   // into a register nobody else has until then
      return;
    }
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void*)smem_raw;

  // ---- loads.  Direct global -> LDS: lane l of a wave-level load lands at (m0) + 16 l.  Written as inline assembly so
  // that the only waits on them are the explicit vmcnt waits below.  All NL loads of a slab are issued together right after the barrier that
  // frees their stage (in waves that also multiply, spreading them over the k-steps measured 3-8% slower: it shortens the prefetch distance).
  uint32_t offA[T::NLA], offB[T::NLB];          // of each lane, from the slab's first element
  const char *ap = reinterpret_cast<const char*>(la.A), *bp = reinterpret_cast<const char*>(la.B), *b2p = reinterpret_cast<const char*>(la.B2);   // of the next slab
  const uint32_t stepA = A_KC ? BK * 2 : BK * la.lda * 2, stepB = B_KC ? BK * 2 : BK * la.ldb * 2;   // bytes per slab
  int next = 0;                                 // slab
  uint32_t next_at = lds0 + lw * 1024;          // its stage
  auto load = [&](uint32_t to, uint32_t off, const char* from) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(to), "v"(off), "s"(from) : "memory", "m0");
  };
  auto issue = [&]() {
    if (next >= iters) return;
    if (!DUAL && next == nk) { ap = reinterpret_cast<const char*>(la.A); bp = b2p; }
#pragma unroll
    for (int q = 0; q < T::NLA; ++q) load(next_at + q * T::LW * 1024, offA[q], ap);
#pragma unroll
    for (int q = 0; q < T::NLB; ++q) load(next_at + T::A_BYTES + q * T::LW * 1024, offB[q], bp);
    if (DUAL) {
#pragma unroll
      for (int q = 0; q < T::NLB; ++q) load(next_at + T::A_BYTES + T::B_BYTES + q * T::LW * 1024, offB[q], b2p);
      b2p += stepB;
    }
    ap += stepA; bp += stepB;
    next_at = (next + 1) % NSTAGE == 0 ? lds0 + lw * 1024 : next_at + T::STAGE_BYTES;
    ++next;
  };
  // make slab `sl` visible: a loading wave's own loads landed, then everyone's; afterwards the stage of slab sl - 1 is free
  auto arrive = [&](int sl) {
    if (loader) wait_loads<T::NL, NSTAGE - 2>(iters - 1 - sl);
    __builtin_amdgcn_s_barrier();
    if (loader) issue();
  };
  if (loader) {
    load_offsets<A_KC, BM, BK, T::LW, T::NLA>(offA, lw, lane, i0, rows_of, la.lda);
    load_offsets<B_KC, BN, BK, T::LW, T::NLB>(offB, lw, lane, j0, la.N, la.ldb);
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; ++s) issue();
  }
  if (T::PW > 0 && loader) {   // the barriers of the others, and the loads
    for (int i = 0; i < iters; ++i) arrive(i);
    if constexpr (T::TAB) {
      if (look_up) {   // all slabs but the last have been read
        const char* const tab = reinterpret_cast<const char*>(la.gelu_tab) + (la.act == GEMM_ACT_GELU_BWD ? GELU_TAB_BYTES : 0);
#pragma unroll
        for (int q = 0; q < (GELU_TAB_BYTES / 1024 + T::LW - 1) / T::LW; ++q) {
          const uint32_t piece = q * T::LW + lw;
          if (piece < GELU_TAB_BYTES / 1024) load(lds0 + tab_at + piece * 1024, lane * 16, tab + piece * 1024);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
      }
    }
    return;
  }

  const int wr = (int)(wave / T::WGN) * T::WM, wc = (int)(wave % T::WGN) * T::WN;
  // the epilogue's arguments, read while the first slab is on its way
  const float *res32 = a.res32, *bias_at = a.bias;
  const bf16_t* aux16 = a.aux16;
  bf16_t *C16_pre = a.C16_pre, *C16 = a.C16;
  float* C32 = a.C32;
  int64_t ldc = a.ldc;
  int kind = batch.kind[prob];
  asm("" : "+s"(res32), "+s"(bias_at), "+s"(aux16), "+s"(C16_pre), "+s"(C16), "+s"(C32), "+s"(ldc), "+s"(kind));
  const float bs = (bias_at != nullptr && a.bias_v != nullptr && a.beps != nullptr && a.bsign != 0.f) ? a.bsign * *(const __attribute__((address_space(4))) float*)a.beps : 0.f;
  f32x4 acc[XT][YT];
#pragma unroll
  for (int x = 0; x < XT; ++x)
#pragma unroll
    for (int y = 0; y < YT; ++y) acc[x][y] = (f32x4){0.f, 0.f, 0.f, 0.f};

  constexpr int KD = DUAL ? 16 : 32, KS = BK / KD;   // depth of a k-step, steps of a slab
  // lane-dependent parts of the operand fetch addresses
  const int lo_half = DUAL ? (int)(lane >> 5) * T::B_BYTES : 0;
  int fa[A_KC ? KS : XT], fb[B_KC ? KS : YT];
  if (A_KC) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fa[ks] = fetch_lane_offset<true, BM, BK, DUAL>(lane, ks) + wr * BK * 2;
  } else {
#pragma unroll
    for (int x = 0; x < XT; ++x) fa[x] = fetch_lane_offset<false, BM, BK, DUAL>(lane, (wr >> 4) + x);
  }
  if (B_KC) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fb[ks] = fetch_lane_offset<true, BN, BK, DUAL>(lane, ks) + wc * BK * 2 + lo_half;
  } else {
#pragma unroll
    for (int y = 0; y < YT; ++y) fb[y] = fetch_lane_offset<false, BN, BK, DUAL>(lane, (wc >> 4) + y) + lo_half;
  }

  auto fetchA = [&](const unsigned char* sa, int x, int ks) -> bf16x8 {
    if (A_KC) return *reinterpret_cast<const bf16x8*>(sa + fa[ks] + x * 16 * BK * 2);
    const unsigned char* p = sa + fa[x] + ks * KD * BM * 2;
    union { bf16x8 v; s16x4 h[2]; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * BM * 2));
    return u.v;
  };
  auto fetchB = [&](const unsigned char* sb, int y, int ks) -> bf16x8 {
    if (B_KC) return *reinterpret_cast<const bf16x8*>(sb + fb[ks] + y * 16 * BK * 2);
    const unsigned char* p = sb + fb[y] + ks * KD * BN * 2;
    union { bf16x8 v; s16x4 h[2]; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * BN * 2));
    return u.v;
  };

  // ---- pipeline: NSTAGE - 1 slabs in flight; a k-step is cut into pieces of YP fragments of B, and
  // the pieces of all slabs form one stream in which the operands of piece t + 1 are fetched from LDS before the MFMAs of piece t are
  // issued (also across the slab boundary, so the LDS latency after a barrier hides behind the last MFMAs of the previous slab)
  constexpr int YP = T::YP, NP = T::NP, NT = KS * NP;   // NT: pieces of a slab
  static_assert(KS % 2 == 0 && NT % 2 == 0, "operand double buffer parity");
  bf16x8 av[2][XT], bv[2][YP];
  // D = B-fragment x A-fragment: a lane gets four neighbouring columns of one row
  constexpr int NM = XT * YP;
  auto mfma = [&](auto t, auto m) {
    constexpr int T_ = t, ks = T_ / NP, y0 = T_ % NP * YP, x = m / YP, yy = m % YP, y = (x & 1) ? YP - 1 - yy : yy;
    acc[x][y0 + y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv[T_ & 1][y], av[ks & 1][x], acc[x][y0 + y], 0, 0, 0);
  };
  // operand r of the piece t of the slab at `at`: first what its first products need
  constexpr int MOST = YP + XT;
  auto operands = [](int t) { return YP + (t % NP == 0 ? XT : 0); };
  auto read = [&](const unsigned char* at, auto t, auto r) {
    constexpr int T_ = t, R_ = r, ks = T_ / NP, p = T_ % NP, wa = p == 0 ? 1 : 0;
    const unsigned char* const sb = at + T::A_BYTES;
    if constexpr (wa == 1 && R_ == 0) av[ks & 1][0] = fetchA(at, 0, ks);
    else if constexpr (R_ - wa < YP) bv[T_ & 1][R_ - wa] = fetchB(sb, p * YP + R_ - wa, ks);
    else av[ks & 1][R_ - YP] = fetchA(at, R_ - YP, ks);
  };
  auto read_all = [&](const unsigned char* at, auto t) {
    static_for<MOST>([&](auto r) { if constexpr (decltype(r)::value < operands(decltype(t)::value)) read(at, t, r); });
  };
  auto multiply = [&](auto t) {
    if (RD != 0) __builtin_amdgcn_sched_barrier(0);
    static_for<NM>([&](auto m) { mfma(t, m); });
    if (RD != 0) __builtin_amdgcn_sched_barrier(0);
  };
  // the products of piece t with the reads of piece tn of the slab at `at` between them
  auto multiply_reading = [&](auto t, const unsigned char* at, auto tn) {
    constexpr int nr = operands(decltype(tn)::value);
    constexpr auto before = [](int m) { const int b = (m * nr * RD + NM - 1) / NM; return b < nr ? b : nr; };   // reads ahead of product m - 1
    __builtin_amdgcn_sched_barrier(0);
    static_for<NM>([&](auto m) {
      static_for<MOST>([&](auto r) { if constexpr (decltype(r)::value >= before(decltype(m)::value) && decltype(r)::value < before(decltype(m)::value + 1)) read(at, tn, r); });
      __builtin_amdgcn_sched_barrier(0);
      mfma(t, m);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  auto stage_of = [&](int sl) { return smem_raw + (sl % NSTAGE) * T::STAGE_BYTES; };

  arrive(0);
  if constexpr (RD == 0) {
    for (int i = 0; i + 1 < iters; ++i) {
      if (i > 0) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave's reads of slab i - 1 are complete
        arrive(i);
      }
      const unsigned char* const at = stage_of(i);
      static_for<NT>([&](auto t) { read_all(at, t); multiply(t); });
    }
  } else {
    read_all(stage_of(0), std::integral_constant<int, 0>{});
    for (int i = 0; i + 1 < iters; ++i) {
      const unsigned char* const at = stage_of(i);
      static_for<NT - 1>([&](auto t) { multiply_reading(t, at, std::integral_constant<int, decltype(t)::value + 1>{}); });
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave's reads of slab i are complete
      arrive(i + 1);
      multiply_reading(std::integral_constant<int, NT - 1>{}, stage_of(i + 1), std::integral_constant<int, 0>{});
    }
  }
  // ---- epilogue: a lane has four neighbouring columns of row lane % 16 of each fragment.  fp32 goes out from there, 64 bytes of a row at a
  // time; of two neighbouring fragments in bf16, lanes 16 apart exchange halves first, so that a lane has eight neighbouring columns of
  // one of them.  Nothing goes through LDS.
  // A unit is a pair of fragments side by side.  Whole tiles of the usual kinds go through
  // code of their own for each kind, without a branch in it; what a unit needs from memory (bias, an fp32 residual or a saved
  // pre-activation, an epilogue has one of these at most) is requested DEPTH - 1 units before it, for the first ones while the last slab
  // is multiplied.
  // The units of a column of them follow each other, but for bf16 outputs of wave tiles 64 rows tall those of a row: a unit is half a 128-byte line
  // there, and halves stored four units apart leave L2 one by one.  MiB written of 12 by 2048 x 3072 x 1024, before / along rows: 256 x 128 tiles 12.7 /
  // 12.0, 256 x 192 14.8 / 12.0 (with the offsets of the lanes computed behind the last slab, which take 12 registers to scratch ahead of it and 4
  // here); us 8192 x 3072 x 1024 with 256 x 192 tiles NT 76.4 / 73.7, 8192 x 2304 x 768 54.8 / 52.6.  Wave tiles 32 rows tall have two units to a column
  // and write no more than their output; of 128 rows (256 x 256, single-term) the fp32 weight gradients would take 2 to 3 % longer.
  constexpr int PAIRS = YT / 2, UNITS = PAIRS * XT, DEPTH = XT * YT > 16 ? 2 : XT * YT == 16 ? 3 : 4;
  const uint32_t wave_row = i0 + wr, wave_col = j0 + wc;
  const bool fast = kind != EPI_ANY && wave_row + T::WM <= rows_of && wave_col + T::WN <= (uint32_t)la.N;   // this wave's part of the tile is whole
  int g;                    // columns of the lane's values: 4 g, after the exchange pair_col
  uint32_t off32, off16;    // (ldc < 2^24 where they are used)
  auto lane_offsets = [&](uint32_t lane_) {
    g = (int)lane_ >> 4;
    const int pair_col = 16 * (g & 1) + 8 * (g >> 1);
    off32 = ((lane_ & 15) * (uint32_t)ldc + 4 * g) * 4; off16 = ((lane_ & 15) * (uint32_t)ldc + pair_col) * 2;
  };
  const int64_t tile0 = ((int64_t)i0 + wr) * ldc + j0 + wc;
  constexpr bool ALONG = XT == 4;   // bf16 outputs
  constexpr auto unit_x = [](bool bf16, int unit) { return ALONG && bf16 ? unit / PAIRS : unit % XT; };
  constexpr auto unit_h = [](bool bf16, int unit) { return ALONG && bf16 ? unit % PAIRS : unit / XT; };
  auto of_unit = [&](bool bf16, int unit) { return tile0 + (int64_t)(unit_x(bf16, unit) * 16) * ldc + unit_h(bf16, unit) * 32; };
  uint4 sv[DEPTH][2] = {};
  constexpr int NBIAS = ALONG ? PAIRS : 2;
  float4 bias[NBIAS][2] = {};
  auto at_columns = [&](const float* base, const float* v, int col) {   // four of the bias, or of a gain or shift, perturbed
    float4 t = *reinterpret_cast<const float4*>(base + col);
    if (bs != 0.f) {
      const float4 d = *reinterpret_cast<const float4*>(v + col);
      t.x = fmaf(bs, d.x, t.x); t.y = fmaf(bs, d.y, t.y); t.z = fmaf(bs, d.z, t.z); t.w = fmaf(bs, d.w, t.w);
    }
    return t;
  };
  auto load_bias = [&](int h) {
    if (bias_at == nullptr) return;
#pragma unroll
    for (int u = 0; u < 2; ++u) bias[h % NBIAS][u] = at_columns(bias_at, a.bias_v, wave_col + 32 * h + 16 * u + 4 * g);
  };
  // The LayerNorm's output is not stored and read again, but made here of its input: of each row the mean and the reciprocal deviation, of each
  // column gain and shift; the same operations, so the same bits.
  const float* ln_mean = nullptr;
  int ln_rstd = 0, ln_g = 0, ln_b = 0;
  if constexpr (LN) {
    ln_mean = a.ln_mean; ln_rstd = a.ln_rstd; ln_g = a.ln_g; ln_b = a.ln_b;
    asm("" : "+s"(ln_mean), "+s"(ln_rstd), "+s"(ln_g), "+s"(ln_b));
  }
  constexpr int LN_XT = LN ? XT : 1, LN_BUF = PAIRS < 2 ? 1 : 2;
  float row_mean[LN_XT], row_rstd[LN_XT];
  float4 gain[LN_BUF][2], shift[LN_BUF][2];
  auto load_ln_columns = [&](int h) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int col = wave_col + 32 * h + 16 * u + 4 * g;
      gain[h % LN_BUF][u] = at_columns(bias_at + ln_g, a.bias_v + ln_g, col);
      shift[h % LN_BUF][u] = at_columns(bias_at + ln_b, a.bias_v + ln_b, col);
      bias[h % LN_BUF][u] = at_columns(bias_at, a.bias_v, col);
    }
  };
  auto load_ln = [&]() {
    if (!fast) return;
    const uint32_t row = wave_row + (lane & 15);
#pragma unroll
    for (int x = 0; x < LN_XT; ++x) { row_mean[x] = ln_mean[row + 16 * x]; row_rstd[x] = ln_mean[ln_rstd + row + 16 * x]; }
    load_ln_columns(0);
  };
  auto load_side = [&](int unit) {
    uint4 (&v)[2] = sv[unit % DEPTH];
    if (LN || kind == EPI_RES32) {
      const char* const p = reinterpret_cast<const char*>(res32 + of_unit(false, unit));
      v[0] = *reinterpret_cast<const uint4*>(p + off32);
      v[1] = *reinterpret_cast<const uint4*>(p + off32 + 64);
    } else if (kind == EPI_GELU_BWD) {
      v[0] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(aux16 + of_unit(true, unit)) + off16);
    }
  };
  auto load_first = [&]() {
    if (!fast) return;
    if constexpr (!LN) static_for<ALONG ? PAIRS : 1>([&](auto h) { load_bias(h); });
    static_for<DEPTH - 1>([&](auto u) { if constexpr (decltype(u)::value < UNITS) load_side(u); });
  };
  constexpr bool EARLY = XT * YT != 24;   // the 64 x 96 tiles of a wave leave no registers for it
  constexpr bool LN_EARLY = XT * YT <= 12;   // the larger ones have none for the statistics and gains either
  if (EARLY) { lane_offsets(lane); load_first(); }
  if constexpr (LN && LN_EARLY) load_ln();
  // the last slab
  {
    if (RD == 0 && iters > 1) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      arrive(iters - 1);
    }
    const unsigned char* const at = stage_of(iters - 1);
    if constexpr (RD == 0) {
      static_for<NT>([&](auto t) { read_all(at, t); multiply(t); });
    } else {
      static_for<NT - 1>([&](auto t) { multiply_reading(t, at, std::integral_constant<int, decltype(t)::value + 1>{}); });
      multiply(std::integral_constant<int, NT - 1>{});
    }
  }
  if (!EARLY) {
    uint32_t lane_ = lane;
    asm volatile("" : "+v"(lane_));   // computed here and not kept over the last slab
    lane_offsets(lane_); load_first();
  }
  if (look_up) __syncthreads();   // the table has come
  if (wave_row >= rows_of || wave_col >= (uint32_t)la.N) return;
  const unsigned char* const tab = smem_raw + tab_at;
  auto entry = [&](uint32_t offset) { return *reinterpret_cast<const float*>(tab + offset); };
  auto exchange = [](uint2 (&v)[2]) {   // its own inverse
    u32x2 r = __builtin_amdgcn_permlane16_swap(v[0].x, v[1].x, false, false); v[0].x = r[0]; v[1].x = r[1];
    r = __builtin_amdgcn_permlane16_swap(v[0].y, v[1].y, false, false); v[0].y = r[0]; v[1].y = r[1];
  };
  auto packed = [](const float (&c)[4]) { return make_uint2(pack_bf16x2(c[0], c[1]), pack_bf16x2(c[2], c[3])); };
  auto gelu = [&](float (&c)[4], uint2 pk) {   // of the rounded pre-activation, which is what the backward pass sees
    c[0] = bf16_to_f32((bf16_t)pk.x); c[1] = bf16_to_f32((bf16_t)(pk.x >> 16)); c[2] = bf16_to_f32((bf16_t)pk.y); c[3] = bf16_to_f32((bf16_t)(pk.y >> 16));
    if constexpr (T::TAB) {
      const uint32_t o0 = gelu_tab_offsets(pk.x), o1 = gelu_tab_offsets(pk.y);
      c[0] *= entry(o0 & 0xffffu); c[1] *= entry(o0 >> 16); c[2] *= entry(o1 & 0xffffu); c[3] *= entry(o1 >> 16);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) c[e] = gelu_f(c[e]);
    }
  };
  auto dgelu = [&](float (&c)[4], uint2 pk) {
    const float x[4] = {bf16_to_f32((bf16_t)pk.x), bf16_to_f32((bf16_t)(pk.x >> 16)), bf16_to_f32((bf16_t)pk.y), bf16_to_f32((bf16_t)(pk.y >> 16))};
    if constexpr (T::TAB) {   // + 0 x: of an infinity or a NaN the derivative is NaN
      const uint32_t o0 = gelu_tab_offsets(pk.x), o1 = gelu_tab_offsets(pk.y);
      c[0] *= fmaf(x[0], 0.f, entry(o0 & 0xffffu)); c[1] *= fmaf(x[1], 0.f, entry(o0 >> 16)); c[2] *= fmaf(x[2], 0.f, entry(o1 & 0xffffu)); c[3] *= fmaf(x[3], 0.f, entry(o1 >> 16));
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) c[e] *= dgelu_f(x[e]);
    }
  };
  auto add = [](float (&c)[4], uint4 r) { c[0] += __uint_as_float(r.x); c[1] += __uint_as_float(r.y); c[2] += __uint_as_float(r.z); c[3] += __uint_as_float(r.w); };
  auto add_ln = [](float (&c)[4], uint4 r, float mu, float rs, float4 gn, float4 sh) {
    c[0] += fmaf((__uint_as_float(r.x) - mu) * rs, gn.x, sh.x); c[1] += fmaf((__uint_as_float(r.y) - mu) * rs, gn.y, sh.y);
    c[2] += fmaf((__uint_as_float(r.z) - mu) * rs, gn.z, sh.z); c[3] += fmaf((__uint_as_float(r.w) - mu) * rs, gn.w, sh.w);
  };
  if (fast) {
    auto of_kind = [&](auto k) {
      constexpr int KIND = k;
      if constexpr (KIND == EPI_LN32 && !LN_EARLY) load_ln();
      static_for<UNITS>([&](auto unit_) {
        constexpr bool BF16 = KIND != EPI_C32 && KIND != EPI_RES32 && KIND != EPI_LN32;
        constexpr int unit = unit_, x = unit_x(BF16, unit), h = unit_h(BF16, unit);
        if constexpr (!LN && !ALONG && x == 0 && h + 1 < PAIRS) load_bias(h + 1);
        if constexpr (KIND == EPI_LN32 && x == 0 && h + 1 < PAIRS) load_ln_columns(h + 1);
        if constexpr ((KIND == EPI_RES32 || KIND == EPI_LN32 || KIND == EPI_GELU_BWD) && unit + DEPTH - 1 < UNITS) load_side(unit + DEPTH - 1);
        const uint4 (&cur)[2] = sv[unit % DEPTH];
        float c[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const f32x4 v = acc[x][2 * h + u];
          const float4 b = bias[KIND == EPI_LN32 ? h % LN_BUF : h % NBIAS][u];
          c[u][0] = v[0] + b.x; c[u][1] = v[1] + b.y; c[u][2] = v[2] + b.z; c[u][3] = v[3] + b.w;
        }
        if constexpr (KIND == EPI_RES32) { add(c[0], cur[0]); add(c[1], cur[1]); }
        if constexpr (KIND == EPI_LN32) {
#pragma unroll
          for (int u = 0; u < 2; ++u) add_ln(c[u], cur[u], row_mean[x], row_rstd[x], gain[h % LN_BUF][u], shift[h % LN_BUF][u]);
        }
        if constexpr (KIND == EPI_GELU_FWD) {
          uint2 pk[2] = {packed(c[0]), packed(c[1])};
          gelu(c[0], pk[0]); gelu(c[1], pk[1]);
          if (C16_pre != nullptr) {   // forward-only passes do not keep it
            exchange(pk);
            *reinterpret_cast<uint4*>(reinterpret_cast<char*>(C16_pre + of_unit(BF16, unit)) + off16) = make_uint4(pk[0].x, pk[0].y, pk[1].x, pk[1].y);
          }
        }
        if constexpr (KIND == EPI_GELU_BWD) {
          uint2 pk[2] = {make_uint2(cur[0].x, cur[0].y), make_uint2(cur[0].z, cur[0].w)};
          exchange(pk);
          dgelu(c[0], pk[0]); dgelu(c[1], pk[1]);
        }
        if (KIND == EPI_C32 || KIND == EPI_RES32 || KIND == EPI_LN32 || (KIND != EPI_C16 && C32 != nullptr)) {
          char* const p = reinterpret_cast<char*>(C32 + of_unit(BF16, unit));
          *reinterpret_cast<float4*>(p + off32) = make_float4(c[0][0], c[0][1], c[0][2], c[0][3]);
          *reinterpret_cast<float4*>(p + off32 + 64) = make_float4(c[1][0], c[1][1], c[1][2], c[1][3]);
        } else {
          uint2 pk[2] = {packed(c[0]), packed(c[1])};
          exchange(pk);
          *reinterpret_cast<uint4*>(reinterpret_cast<char*>(C16 + of_unit(BF16, unit)) + off16) = make_uint4(pk[0].x, pk[0].y, pk[1].x, pk[1].y);
        }
      });
    };
    if constexpr (LN) {
      return of_kind(std::integral_constant<int, EPI_LN32>{});
    } else {
      switch (kind) {
        case EPI_C16: return of_kind(std::integral_constant<int, EPI_C16>{});
        case EPI_C32: return of_kind(std::integral_constant<int, EPI_C32>{});
        case EPI_RES32: return of_kind(std::integral_constant<int, EPI_RES32>{});
        case EPI_GELU_FWD: return of_kind(std::integral_constant<int, EPI_GELU_FWD>{});
        default: return of_kind(std::integral_constant<int, EPI_GELU_BWD>{});
      }
    }
  }
  // any combination, any alignment the operands may have, tiles at the edges
  const int row0 = (int)i0 + wr + (int)(lane & 15), col0 = (int)j0 + wc + 4 * g, nrows = (int)rows_of, ncols = la.N, act = la.act;
  static_for<UNITS>([&](auto unit_) {
    constexpr int unit = unit_, x = unit % XT, h = unit / XT;
    const int row = row0 + 16 * x;
    if (row >= nrows) return;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int col = col0 + 32 * h + 16 * u;
      if (col >= ncols) continue;
      const int64_t at = (int64_t)row * ldc + col;
      float c[4] = {acc[x][2 * h + u][0], acc[x][2 * h + u][1], acc[x][2 * h + u][2], acc[x][2 * h + u][3]};
      if (bias_at != nullptr) {
        const float4 b = at_columns(bias_at, a.bias_v, col);
        c[0] += b.x; c[1] += b.y; c[2] += b.z; c[3] += b.w;
      }
      if constexpr (LN) add_ln(c, *reinterpret_cast<const uint4*>(res32 + at), ln_mean[row], ln_mean[ln_rstd + row], at_columns(bias_at + ln_g, a.bias_v + ln_g, col), at_columns(bias_at + ln_b, a.bias_v + ln_b, col));
      else if (res32 != nullptr) add(c, *reinterpret_cast<const uint4*>(res32 + at));
      if (act == GEMM_ACT_GELU_FWD) {
        const uint2 pk = packed(c);
        if (C16_pre != nullptr) *reinterpret_cast<uint2*>(C16_pre + at) = pk;
        gelu(c, pk);
      } else if (act == GEMM_ACT_GELU_BWD) {
        dgelu(c, *reinterpret_cast<const uint2*>(aux16 + at));
      }
      if (C32 != nullptr) *reinterpret_cast<float4*>(C32 + at) = make_float4(c[0], c[1], c[2], c[3]);
      if (C16 != nullptr) *reinterpret_cast<uint2*>(C16 + at) = packed(c);
    }
  });
}

template <typename T, bool A_KC, bool B_KC, bool LN>
__global__ __launch_bounds__(T::THREADS) void k_gemm_bf16(GemmBatch batch) { gemm_tile<T, A_KC, B_KC, LN>(batch); }

// What a whole tile's epilogue does, where it is one of the usual things on usual alignments.
int epilogue_kind(const GemmBf16Args& a) {
  if (a.ldc % 8 != 0 || a.ldc >= (1 << 24) || (((uintptr_t)a.C16 | (uintptr_t)a.C16_pre | (uintptr_t)a.aux16) & 15) != 0) return EPI_ANY;
  if ((a.C32 != nullptr) == (a.C16 != nullptr)) return EPI_ANY;
  if (a.act != GEMM_ACT_NONE) return a.res32 != nullptr ? EPI_ANY : a.act == GEMM_ACT_GELU_FWD ? EPI_GELU_FWD : EPI_GELU_BWD;
  if (a.res32 != nullptr) return a.C32 == nullptr ? EPI_ANY : a.ln_mean != nullptr ? EPI_LN32 : EPI_RES32;
  return a.C32 != nullptr ? EPI_C32 : EPI_C16;
}

GemmBatch make_batch(const GemmBf16Args* p, int count, int group, int bm, int bn) {
  GemmBatch b{};
  b.first = loop_args(p[0]);
  b.count = count; b.group = group;
  int nt = 0;
  for (int k = 0; k < count; ++k) {
    b.p[k] = p[k];
    b.kind[k] = epilogue_kind(p[k]);
    b.first_tile[k] = nt;
    nt += ((p[k].N + bn - 1) / bn) * ((p[k].M + bm - 1) / bm);
  }
  for (int k = count; k <= GEMM_MAX_BATCH; ++k) b.first_tile[k] = nt;
  b.ntiles = nt; b.tiles_per_xcd = (nt + 7) / 8;
  return b;
}

template <typename T, bool A_KC, bool B_KC, bool LN = false>
void launch_tile(ProfScope& ps, hipStream_t st, const GemmBf16Args* p, int count, int group) {
  static bool configured = false;      // per instantiation: raise the dynamic LDS limit once
  if (!configured) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_bf16<T, A_KC, B_KC, LN>), hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
    configured = true;
  }
  const GemmBatch b = make_batch(p, count, group, T::BM, T::BN);
  launch_kernel(ps, k_gemm_bf16<T, A_KC, B_KC, LN>, 8 * b.tiles_per_xcd, T::THREADS, T::LDS_BYTES, st, b);
}

// Tiles <BM, BN, BK, multiplying waves in M, in N, stages, hi + lo, loading waves, fragments of a piece, fetches (see Tile)>
// The 32 x 32 ones are for products of few rows (scoring one text), which a larger tile leaves to a few dozen workgroups that walk
// the contraction slab by slab: with twice as many and five slabs in flight, 128 rows of 768 x 3072 take 12.1 us hi + lo (64 x 32: 13.9;
// one multiplying wave instead of two 13.0; slabs of 128 11.4) and 10.7 single-term (64 x 64: 17.2).  Splitting the contraction over the
// waves of a workgroup was 0.8 us faster, but sums in another order, so that a text scored alone came out otherwise than in a batch.
typedef Tile<256, 256, 64, 2, 4, 2, false, 0, 2, 0> S1;
typedef Tile<256, 192, 64, 4, 2, 2, false, 4, 2, 1> S2;
typedef Tile<256, 128, 64, 4, 2, 3, false, 4, 2, 2> S3;
typedef Tile<128, 128, 64, 4, 2, 4, false, 4, 0, 1> S4;
typedef Tile<128, 64, 64, 4, 2, 4, false, 4, 0, 1> S5;
typedef Tile<64, 64, 64, 2, 2, 4, false, 0, 0, 1> S6;         // two workgroups per CU
typedef Tile<128, 128, 64, 4, 2, 2, false, 0, 0, 1> S7;       // two workgroups per CU
typedef Tile<32, 32, 64, 1, 1, 6, false, 2, 0, 1> S8;      // three workgroups per CU
typedef Tile<256, 192, 64, 4, 2, 2, true, 4, 2, 1> D1;
typedef Tile<256, 128, 64, 4, 2, 2, true, 4, 2, 2> D2;
typedef Tile<128, 128, 64, 2, 4, 3, true, 4, 0, 1> D3;
// (64 x 32 of a wave forward, 32 x 96 for input gradients: above)
template <bool B_KC> using D4 = std::conditional_t<B_KC, Tile<128, 96, 64, 2, 3, 3, true, 4, 0, 1>, Tile<128, 96, 64, 4, 1, 3, true, 4, 0, 2>>;
typedef Tile<128, 64, 64, 2, 2, 4, true, 4, 0, 1, 1> D5;
typedef Tile<64, 64, 64, 2, 2, 4, true, 2, 0, 1, 1> D6;
typedef Tile<64, 64, 64, 2, 2, 3, true, 2, 0, 1, 1> D7;       // two workgroups per CU
typedef Tile<64, 32, 64, 4, 1, 4, true, 2, 0, 1> D8;       // two workgroups per CU
typedef Tile<32, 32, 64, 2, 1, 6, true, 2, 0, 0> D9;       // two workgroups per CU
typedef Tile<32, 32, 128, 2, 1, 3, true, 2, 0, 1> D10;     // two workgroups per CU; contractions of a multiple of 128

// A hi + lo product of a padded batch: the tile is chosen here, by the rows in use, among four of one workgroup to a CU.  (The waves that a
// tile does not have end at once; the bodies are those of the launches with one tile, but for the touching waves, for which 168 registers a wave
// leave no room.)
typedef Tile<128, 64, 64, 2, 2, 4, true, 4, 0, 1> R5;
constexpr int ROWS_THREADS = D1::THREADS, ROWS_SHARES = 16;
static_assert(D2::THREADS <= ROWS_THREADS && D4<true>::THREADS <= ROWS_THREADS && D4<false>::THREADS <= ROWS_THREADS && R5::THREADS <= ROWS_THREADS, "waves");
template <typename T, bool B_KC, bool LN>
__device__ __forceinline__ void gemm_rows_tile(const GemmBatch& batch) {
  if (T::THREADS == ROWS_THREADS || (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x) < (uint32_t)T::THREADS) gemm_tile<T, true, B_KC, LN>(batch);
}
template <bool B_KC, bool LN>
__global__ __launch_bounds__(ROWS_THREADS) void k_gemm_rows(GemmBatch batch) {
  const uint32_t in_use = *(const __attribute__((address_space(4))) int32_t*)batch.first.rows;
  const uint32_t share = small_quotient(ROWS_SHARES * in_use - 1, batch.first.M);   // 0 < in_use <= M
  switch ((uint32_t)(batch.choice >> (4 * share)) & 15) {
    case 1:
      if constexpr (!LN) return gemm_rows_tile<D1, B_KC, LN>(batch);
      [[fallthrough]];   // (with LN the host chooses the next one instead)
    case 2: return gemm_rows_tile<D2, B_KC, LN>(batch);
    case 4: return gemm_rows_tile<D4<B_KC>, B_KC, LN>(batch);
    default: return gemm_rows_tile<R5, B_KC, LN>(batch);
  }
}

// What a launch costs with a tile, in us, beyond what it costs with any: per round, epilogue + 64-deep slabs x time of a slab.
// A round is up to `per_cu` tiles on each of the 256 CUs; a slab takes `few` with a handful of tiles on the chip, `one` with one
// on every CU and, where two fit, `two` as soon as some CU holds two and `all` when every one does; in between in proportion.
// The numbers are robust least-squares fits of the logarithms over timed problems (widths 192 to 2048, FFN 2 and 4 times that,
// 64 to 8192 rows: NT, NN, pairs of NT, a layer's four TN problems in a launch; the vocabulary head's products over 8192 to
// 50304 tokens; weights cold): HILO_NN of the kernels before 128 x 128 and 128 x 64 tiles were cut into 64 x 32 waves (up to 2% longer), SINGLE and HILO of still earlier ones (32 x 32 x 16 MFMAs, the epilogue through LDS), which took 1.3
// to 1.5 times as long; HILO's last entry was set by hand beside the one before it.  On times of the former, picking by them takes
// 0.4% (NT), 0.3% (pairs), 0.5% (NN) and 0.5% (TN) longer in total than the fastest tile of each problem, the head's products 1 to 2%; by
// HILO for NN too, NN takes 2.6% and the head's NN 7%.  On times of the present kernels it is 0.8% (NT), 0.7% (pairs) and 1.3% (NN): profiles/gemm_tile_costs.md.
struct TileCost { int id, bm, bn, per_cu; double few, one, two, all, epilogue; int bk = 64; };
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
    {19, 32, 32, 2, 0.236, 0.255, 0.381, 0.381, 1.28}, {20, 32, 32, 2, 0.220, 0.240, 0.360, 0.360, 1.28, 128}};

constexpr TileCost HILO_NN[] = {   // the strided weights of an input gradient
    {11, 256, 192, 1, 1.203, 1.828, 0, 0, 8.00},  {12, 256, 128, 1, 0.998, 1.366, 0, 0, 3.68},
    {13, 128, 128, 1, 0.693, 0.886, 0, 0, 2.39},  {14, 128, 96, 1, 0.587, 0.720, 0, 0, 1.74},
    {15, 128, 64, 1, 0.364, 0.497, 0, 0, 0.95},   {16, 64, 64, 1, 0.247, 0.339, 0, 0, 0.52},
    {17, 64, 64, 2, 0.299, 0.373, 0.557, 0.642, 0.60}, {18, 64, 32, 2, 0.217, 0.309, 0.450, 0.498, 0.11},
    {19, 32, 32, 2, 0.178, 0.268, 0.376, 0.422, 0.19}, {20, 32, 32, 2, 0.235, 0.335, 0.347, 0.446, 0.00, 128}};

int g_force_shape = 0, g_group = 8;
uint64_t g_force_rows = 0;
std::atomic<int64_t> g_launches[GEMM_COUNTS];

// Tiles, and cost, of a launch with `share` of `of` parts of a padded batch's rows in use.
double launch_cost(const TileCost& c, const GemmBf16Args* p, int count, int share, int of, int64_t* ntiles = nullptr) {
  int64_t tiles = 0;
  double slabs = 0.0;                                    // of all tiles
  for (int k = 0; k < count; ++k) {
    const int64_t part = p[k].rows != nullptr ? share : of, M = p[k].a_trans ? p[k].M : (p[k].M * part + of - 1) / of, K = p[k].a_trans ? (p[k].K * part + of - 1) / of : p[k].K;
    const int64_t t = ((M + c.bm - 1) / c.bm) * ((p[k].N + c.bn - 1) / c.bn);
    tiles += t;
    slabs += (double)t * K / 64.0;
  }
  if (ntiles != nullptr) *ntiles = tiles;
  slabs /= (double)tiles;
  const int64_t cap = 256 * c.per_cu, rest = tiles % cap;
  double cost = (double)(tiles / cap) * (slabs * (c.per_cu > 1 ? c.all : c.one) + c.epilogue);
  if (rest > 0) {
    const double slab = rest <= 256 ? c.few + (c.one - c.few) * (double)rest / 256.0 : c.two + (c.all - c.two) * (double)(rest - 256) / (double)(cap - 256);
    cost += slabs * slab + c.epilogue;
  }
  return cost;
}

// How many rows of a padded batch are in use only the device knows, and how long texts are is the caller's: where one tile has to do for
// the launch, it is the one that costs least in total over batches a quarter, half, three quarters and all in use.  Longer than the fastest
// tile of a product at each of these (geometric means): 16, 6, 7 and 9%; choosing for one share in between, two thirds, 30, 11, 5 and 8%, for
// all rows 37, 16, 5 and 2%.
template <int N>
int pick_tile(const TileCost (&costs)[N], const GemmBf16Args* p, int count, bool padded, double* total) {
  bool deep = true;   // whole slabs of 128
  for (int k = 0; k < count; ++k) deep = deep && p[k].K % 128 == 0 && (!p[k].a_trans || p[k].rows == nullptr);
  int best = 0;
  for (const TileCost& c : costs) {
    if ((c.bk == 128 && !deep) || (c.id == 11 && p[0].ln_mean != nullptr)) continue;
    double cost = 0.0;
    for (int share = padded ? 1 : 4; share <= 4; ++share) cost += launch_cost(c, p, count, share, 4);
    if (best == 0 || cost < *total) { best = c.id; *total = cost; }
  }
  return best;
}

// The same for k_gemm_rows: the tile of least cost for each sixteenth of the rows; returns whether that is worth more over the quarters than
// the 0.4 us a launch that the choice takes (0.3 in forward products, whose table is in longer microseconds; at 0.6 and 1.0 the choices are 0.01 and 0.07%
// further from the fastest tiles).  Entry 15 stands for R5 here, which touches no weights and takes 1.07 times as long in input gradients over 2048 and more: a
// price of its own there made padded base steps of 24 x 1024 up to 5.7% shorter and those of 6 x 1024 with FFN 2048 up to 3.4% longer, 0.2%
// shorter in the mean of 12 models.
template <int N>
bool pick_by_rows(const TileCost (&costs)[N], const GemmBf16Args* p, int count, double one_tile, uint64_t* choice, int64_t* most_tiles) {
  double total = 0.0;
  *choice = 0; *most_tiles = 0;
  for (int share = 1; share <= ROWS_SHARES; ++share) {
    int best = 0;
    double best_cost = 0.0;
    int64_t best_tiles = 0;
    for (const TileCost& c : costs) {
      if (c.id != 11 && c.id != 12 && c.id != 14 && c.id != 15) continue;   // those of k_gemm_rows
      if (c.id == 11 && p[0].ln_mean != nullptr) continue;   // has no registers for it: 284 bytes a lane in scratch
      int64_t tiles;
      const double cost = launch_cost(c, p, count, share, ROWS_SHARES, &tiles);
      if (best == 0 || cost < best_cost) { best = c.id - 10; best_cost = cost; best_tiles = tiles; }
    }
    *choice |= (uint64_t)best << (4 * (share - 1));
    *most_tiles = std::max(*most_tiles, best_tiles);
    if (share % (ROWS_SHARES / 4) == 0) total += best_cost + 0.4;
  }
  return total < one_tile;
}

// Tiles of the largest launch by a given choice.
template <int N>
int64_t most_tiles_of(const TileCost (&costs)[N], const GemmBf16Args* p, int count, uint64_t choice) {
  int64_t most = 0;
  for (int share = 1; share <= ROWS_SHARES; ++share)
    for (const TileCost& c : costs) {
      int64_t tiles = 0;
      if (c.id == 10 + (int)((choice >> (4 * (share - 1))) & 15)) launch_cost(c, p, count, share, ROWS_SHARES, &tiles);
      most = std::max(most, tiles);
    }
  return most;
}

template <bool B_KC, bool LN>
void launch_rows(ProfScope& ps, hipStream_t st, const GemmBf16Args* p, int count, uint64_t choice, int64_t most_tiles) {
  static bool configured = false;
  constexpr int LDS = std::max({D1::LDS_BYTES, D2::LDS_BYTES, D4<B_KC>::LDS_BYTES, R5::LDS_BYTES});
  if (!configured) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_rows<B_KC, LN>), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    configured = true;
  }
  g_launches[B_KC ? GEMM_ROWS_NT : GEMM_ROWS_NN].fetch_add(1, std::memory_order_relaxed);
  GemmBatch b = make_batch(p, count, g_group, 64, 64);
  b.choice = choice;
  b.tiles_per_xcd = (int)((most_tiles + 7) / 8);
  launch_kernel(ps, k_gemm_rows<B_KC, LN>, 8 * b.tiles_per_xcd, ROWS_THREADS, LDS, st, b);
}

// LN (here and in the kernels): every problem has a LayerNorm's residual
template <bool A_KC, bool B_KC, bool LN = false>
void launch_class(ProfScope& ps, hipStream_t st, const GemmBf16Args* p, int count) {
  const bool dual = p[0].B2 != nullptr;
  int shape = g_force_shape;
  if ((shape >= 11 && !dual) || (LN && shape <= 11)) shape = 0;   // hi + lo tiles read B2
  for (int k = 0; k < count; ++k)
    if (shape == 20 && (p[k].K % 128 != 0 || (p[k].a_trans && p[k].rows != nullptr))) shape = 0;
  if (shape == 0) {
    bool padded = false;
    for (int k = 0; k < count; ++k) padded = padded || p[k].rows != nullptr;
    double total = 0.0;
    shape = !dual ? pick_tile(SINGLE, p, count, padded, &total) : B_KC ? pick_tile(HILO, p, count, padded, &total) : pick_tile(HILO_NN, p, count, padded, &total);
    if constexpr (A_KC) {
      uint64_t choice = g_force_rows;
      int64_t tiles;
      for (int share = 0; LN && share < ROWS_SHARES; ++share)
        if ((choice >> (4 * share) & 15) == 1) choice ^= (uint64_t)(1 ^ 2) << (4 * share);
      if (choice != 0 && padded && dual) return launch_rows<B_KC, LN>(ps, st, p, count, choice, most_tiles_of(HILO, p, count, choice));
      if (padded && dual && (B_KC ? pick_by_rows(HILO, p, count, total, &choice, &tiles) : pick_by_rows(HILO_NN, p, count, total, &choice, &tiles)))
        return launch_rows<B_KC, LN>(ps, st, p, count, choice, tiles);
    }
  }
  switch (shape) {
    case 12: return launch_tile<D2, A_KC, B_KC, LN>(ps, st, p, count, g_group);
    case 13: return launch_tile<D3, A_KC, B_KC, LN>(ps, st, p, count, g_group);
    case 14: return launch_tile<D4<B_KC>, A_KC, B_KC, LN>(ps, st, p, count, g_group);
    case 15: return launch_tile<D5, A_KC, B_KC, LN>(ps, st, p, count, g_group);
    case 16: return launch_tile<D6, A_KC, B_KC, LN>(ps, st, p, count, g_group);
    case 17: return launch_tile<D7, A_KC, B_KC, LN>(ps, st, p, count, g_group);
    case 18: return launch_tile<D8, A_KC, B_KC, LN>(ps, st, p, count, g_group);
    case 19: return launch_tile<D9, A_KC, B_KC, LN>(ps, st, p, count, g_group);
    case 20: return launch_tile<D10, A_KC, B_KC, LN>(ps, st, p, count, g_group);
    default: break;
  }
  if constexpr (LN) {
    launch_tile<D2, A_KC, B_KC, LN>(ps, st, p, count, g_group);
  } else {
    switch (shape) {
      case 1: launch_tile<S1, A_KC, B_KC>(ps, st, p, count, g_group); break;
      case 2: launch_tile<S2, A_KC, B_KC>(ps, st, p, count, g_group); break;
      case 3: launch_tile<S3, A_KC, B_KC>(ps, st, p, count, g_group); break;
      case 4: launch_tile<S4, A_KC, B_KC>(ps, st, p, count, g_group); break;
      case 5: launch_tile<S5, A_KC, B_KC>(ps, st, p, count, g_group); break;
      case 6: launch_tile<S6, A_KC, B_KC>(ps, st, p, count, g_group); break;
      case 8: launch_tile<S8, A_KC, B_KC>(ps, st, p, count, g_group); break;
      case 11: launch_tile<D1, A_KC, B_KC>(ps, st, p, count, g_group); break;
      default: launch_tile<S7, A_KC, B_KC>(ps, st, p, count, g_group); break;
    }
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
  if (a.ln_mean != nullptr && (a.res32 == nullptr || a.bias == nullptr || a.B2 == nullptr || a.a_trans || !a.b_trans)) return "a LayerNorm's residual belongs to a forward hi + lo product with a bias";
  if (a.ln_mean != nullptr && ((a.ln_g | a.ln_b) & 3) != 0) return "gains and shifts must be 16-byte aligned";
  if (a.lda < (a.a_trans ? a.M : a.K) || a.ldb < (a.b_trans ? a.K : a.N) || a.ldc < a.N) return "leading dimension too small";
  const int64_t abytes = (int64_t)(a.a_trans ? a.K : a.M) * a.lda * 2, bbytes = (int64_t)(a.b_trans ? a.N : a.K) * a.ldb * 2;
  if (abytes >= ((int64_t)1 << 31) || bbytes >= ((int64_t)1 << 31)) return "operands must be smaller than 2 GiB";
  return nullptr;
}

bool gemm_bf16_force_rows(uint64_t choice) {
  for (uint64_t c = choice; c != 0; c >>= 4)
    if ((c & 15) != 1 && (c & 15) != 2 && (c & 15) != 4 && (c & 15) != 5) return false;
  if (choice != 0 && choice >> 60 == 0) return false;   // a tile for each sixteenth
  g_force_rows = choice;
  return true;
}
void gemm_bf16_take_counts(int64_t* counts) {
  for (int k = 0; k < GEMM_COUNTS; ++k) counts[k] = g_launches[k].exchange(0, std::memory_order_relaxed);
}
void gemm_bf16_force_shape(int s) { g_force_shape = s % 100; g_group = s >= 100 ? s / 100 : 8; }

const char* check_gemm_bf16_batch(const GemmBf16Args* p, int count) {
  if (count < 1 || count > GEMM_MAX_BATCH) return "batch of 1 to 4 problems";
  for (int k = 0; k < count; ++k) {
    if (const char* e = check_gemm_bf16(p[k])) return e;
    if (p[k].a_trans != p[0].a_trans || p[k].b_trans != p[0].b_trans || (p[k].B2 != nullptr) != (p[0].B2 != nullptr) || (p[k].ln_mean != nullptr) != (p[0].ln_mean != nullptr))
      return "the problems of a batch must share operand storage, the hi + lo form and whether a LayerNorm's output is added";
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
  if (p[0].ln_mean != nullptr) launch_class<true, true, true>(ps, st, p, count);
  else if (!p[0].a_trans && p[0].b_trans) launch_class<true, true>(ps, st, p, count);
  else if (!p[0].a_trans && !p[0].b_trans) launch_class<true, false>(ps, st, p, count);
  else if (p[0].a_trans && !p[0].b_trans) launch_class<false, false>(ps, st, p, count);
  else launch_class<false, true>(ps, st, p, count);
}

void launch_gemm_bf16(hipStream_t st, const GemmBf16Args& a) { launch_gemm_bf16_batch(st, &a, 1); }

}  // namespace sama
