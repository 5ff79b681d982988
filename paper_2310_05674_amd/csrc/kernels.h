// Host-side launchers of every gfx950 kernel in libsama.  Internal; the C ABI is include/sama.h.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include <tuple>
#include <utility>
#include "common.h"

namespace sama {
namespace detail {
template <typename Tuple, size_t... I>
inline void arg_pointers(Tuple& t, void** out, std::index_sequence<I...>) {
  ((out[I] = const_cast<void*>(static_cast<const void*>(&std::get<I>(t)))), ...);
}
}  // namespace detail

// ------------------------------------------------------------------ optional per-launch timing (profile.hip)
enum Family {
  F_GEMM_NT = 0, F_GEMM_NN, F_GEMM_TN, F_GEMM_NT_HILO, F_GEMM_NN_HILO, F_GEMM_F32, F_ATTN_FWD, F_ATTN_BWD, F_LN_FWD, F_LN_BWD, F_ADAM, F_ADAPT_NORM,
  F_PERTURB, F_RESIDUAL, F_NUDGE, F_SAMPLE_STAGE, F_MLM_SOFTMAX, F_OTHER, F_COUNT
};
// While profiling is enabled every launch made through launch_kernel carries a start and a stop event that take the
// kernel's own begin and end timestamps (hipExtLaunchKernel), so a recorded duration is the kernel's execution time as
// a kernel trace shows it, without the dispatch gap in front of it.  A scope names the family and the work of what its
// launcher enqueues; `units` = algorithmic flops (GEMM, attention) or algorithmic bytes (everything else), credited to
// the scope's first launch.
struct ProfScope {
  ProfScope(hipStream_t st, int family, double units);
  bool on() const { return on_; }
  void next_events(hipEvent_t* start, hipEvent_t* stop);   // registers one more launch of this scope (profiling on only)
  hipStream_t st_;
  int family_;
  double units_;
  bool on_;
};
// kernel<<<grid, block, lds, st>>>(args...), timed when the scope is live.  The actual arguments are converted to the
// kernel's formal parameter types first, as the launch syntax would.
template <typename... P, typename... A>
inline void launch_kernel(ProfScope& ps, void (*kernel)(P...), dim3 grid, dim3 block, unsigned lds, hipStream_t st, A&&... a) {
  static_assert(sizeof...(P) == sizeof...(A), "argument count");
  std::tuple<P...> params(std::forward<A>(a)...);
  void* ptrs[sizeof...(P) > 0 ? sizeof...(P) : 1];
  detail::arg_pointers(params, ptrs, std::index_sequence_for<P...>{});
  if (ps.on()) {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    ps.next_events(&e0, &e1);
    (void)hipExtLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs, lds, st, e0, e1, 0);
  } else {
    (void)hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs, lds, st);
  }
}
void prof_enable(bool on);
bool prof_read(int family, const char** name, int64_t* launches, double* total_ms, double* units);

constexpr int EW_MAX_BLOCKS = 65536;  // grid cap of the elementwise kernels (also the size of the norm partials)
// A launcher that is handed a shape its kernel cannot run records the reason here and launches nothing; the C entry
// points report it as an error (take_launch_error returns and clears it, null = none).
void note_launch_error(const char* what);
const char* take_launch_error();

constexpr int MAX_BATCH = 2048;
constexpr int MAX_TOKENS = 8192;   // encoder: token rows of one batch (the token-gradient kernel lists them in LDS)
constexpr int MAX_WNET_HIDDEN = 256;
constexpr int MAX_CORR_HIDDEN = 128;   // label corrector: hidden width and number of classes it supports
constexpr int MAX_CORR_CLASSES = 16;

// ------------------------------------------------------------------ elementwise chain (elementwise.hip)
struct AdamArgs {
  float beta1, one_m_beta1, beta2, one_m_beta2;
  float lr_c1;  // lr / (1 - beta1^t)
  float c2;     // 1 / sqrt(1 - beta2^t)
  float eps, weight_decay;
  const float* dev;  // non-null: lr_c1 = dev[0], c2 = dev[1] read on the device (launch_step_scalars), the two fields above unused
  bf16_t* lo;        // non-null: also lo[k] = bf16(theta'[k] - float(bf16(theta'[k]))) for the first n16 elements (what
                     // launch_residual_lo would compute afterwards)
};
struct AdaptArgs {
  int mode;  // 0: Adam closed form, 1: scalar
  float scalar;
  float one_m_beta1, one_m_beta2;
  float lr_c1_c2;  // lr c1 c2
  float c2, eps;
  const float* dev;  // non-null: lr_c1_c2 = dev[2], c2 = dev[3] read on the device
};
// The step-dependent scalars of Adam and of its adaptation, kept on the device so that a captured sequence of launches
// stays valid from replay to replay: t = (counters[0] += advance); step[0..3] = {lr / (1 - beta1^t),
// 1 / sqrt(1 - beta2^t), lr c1 c2, c2} in double arithmetic (left alone while t < 1).  A base step advances them in its
// per-sample stage; launch_step_scalars is the form on its own.
struct StepScalars { int64_t* counters; int advance; float lr, beta1, beta2; float* step; };
__device__ __forceinline__ void step_scalars(const StepScalars& s) {
  const int64_t t = s.counters[0] + s.advance;
  if (s.advance != 0) s.counters[0] = t;
  if (t < 1) return;
  const double c1 = 1.0 / (1.0 - ipow((double)s.beta1, t));
  const double c2 = 1.0 / sqrt(1.0 - ipow((double)s.beta2, t));
  s.step[0] = (float)((double)s.lr * c1); s.step[1] = (float)c2;
  s.step[2] = (float)((double)s.lr * c1 * c2); s.step[3] = (float)c2;
}
void launch_step_scalars(hipStream_t, const StepScalars&);
// With a non-zero weight decay the L2 term is added to g in place (g then is the gradient the solver was given).
void launch_adam(hipStream_t, float* g, float* m, float* v, float* theta, bf16_t* theta16, int64_t n, int64_t n16,
                 const AdamArgs&);
// SGD with heavy-ball momentum mu (velocity in buf, untouched when mu = 0); lo as in AdamArgs (may be null)
void launch_sgd(hipStream_t, float* g, float* buf, float* theta, bf16_t* theta16, bf16_t* lo, int64_t n, int64_t n16, float lr,
                float wd, float mu);
// v = D . gmeta, then eps = alpha/||v|| -> scalars[0], ||v|| -> scalars[1], status[0] = (norm unusable)
void launch_adapt_norm(hipStream_t, const float* g, const float* m, const float* v, const float* gmeta, float* vdir,
                       double* partial /*[EW_MAX_BLOCKS]*/, int64_t n, const AdaptArgs&, float alpha, float* scalars,
                       int64_t* status);
// The same in pieces: v = D . gmeta over one range, its per-block sums of squares into partial[0 .. returned count)
// (at most max_blocks), and, once every range is done, eps and the status word from all the partials in index order.
// A range that is the only one may be given `fin` (a ticket as in last_block): if it is small enough its last block also
// does the second step, which *finished tells.
struct EpsFinish { float alpha; float* scalars; int64_t* status; uint32_t* ticket; };
int launch_adapt_slice(hipStream_t, const float* g, const float* m, const float* v, const float* gmeta, float* vdir,
                       double* partial, int64_t n, const AdaptArgs&, int max_blocks, const EpsFinish& fin = EpsFinish{},
                       bool* finished = nullptr);
void launch_eps_from_partials(hipStream_t, const double* partial, int count, float alpha, float* scalars, int64_t* status);
void launch_perturb_lo(hipStream_t, const float* theta, const float* vdir, const float* eps_ptr, bf16_t* lo_p,
                       bf16_t* lo_m, int64_t n16);
// perturb_lo and the nudge of the first n16 elements (n16 % 4 == 0) in one pass: theta, theta16 <- theta - eps v,
// lo_p / lo_m = low halves of theta_old +- eps v against the NEW theta16
void launch_perturb_nudge(hipStream_t, float* theta, const float* vdir, const float* eps_ptr, bf16_t* theta16, bf16_t* lo_p,
                          bf16_t* lo_m, int64_t n16);
// lo[k] = bf16(theta[k] - float(bf16(theta[k]))): the part of the master weights the bf16 working copy cannot hold
void launch_residual_lo(hipStream_t, const float* theta, bf16_t* lo, int64_t n16);
// theta <- theta - eps v; theta16 / lo (either may be null) receive the rounded copy and its residual half over the first
// n16 elements; nothing happens when eps = 0 or *status != 0 (status may be null)
void launch_nudge(hipStream_t, float* theta, const float* vdir, const float* eps_ptr, const int64_t* status, bf16_t* theta16,
                  bf16_t* lo, int64_t n, int64_t n16);
// undoes launch_perturb_nudge's nudge of the first n16 elements when *status != 0 although eps > 0 (early exit otherwise)
void launch_unnudge(hipStream_t, float* theta, const float* vdir, const float* eps_ptr, const int64_t* status, bf16_t* theta16,
                    bf16_t* lo, int64_t n16);
void launch_fill_f32(hipStream_t, float* p, float val, int64_t n);
void launch_copy_f32(hipStream_t, float* dst, const float* src, int64_t n);
void launch_to_bf16(hipStream_t, bf16_t* dst, const float* src, int64_t n);
void launch_fill_i64x4(hipStream_t, int64_t* p, int64_t a, int64_t b, int64_t c, int64_t d, int mask);

// ------------------------------------------------------------------ per-sample stage (sample_stage.hip)
enum { STAGE_BASE = 0, STAGE_META = 1, STAGE_GLAM = 2, STAGE_EVAL = 3 };   // EVAL: BASE's losses and weights only
constexpr int STAGE_MAX_BLOCKS = 64;
int stage_blocks(int B);   // most workgroups a stage over B samples uses per pass (the number of its partials)
// h from the two lambda-gradients (Eq. 5) and, with do_update, Adam on lambda
struct MetaUpdateArgs {
  double* glam_p; double* glam_m;   // [nl] out: the two lambda-gradients
  const float* scalars;   // [0] = eps
  int64_t* counters;      // [1] = meta step count, [2] = status
  float* hypergrad;       // [nl] out
  float* hypergrad_user;  // optional
  float* eps_user;        // optional
  float* glam_p_f32; float* glam_m_f32;  // fp32 copies for inspection
  float* lambda; float* meta_m; float* meta_v;
  int nl, do_update;
  float lr, beta1, beta2, eps;
};
// The classifier: logits[i][c] = x[i * stride + :] . W[c] + b[c], W and b inside theta, contraction over k features.  The
// second pass of Eq. 5 reads its features pass_stride behind and sees the opposite perturbation.
struct HeadView {
  const float* x; int64_t stride, pass_stride;
  int k;
  ParamView pv; int64_t w_off, b_off;
  const int32_t* start;   // null, or row (of k values) of each sample instead of i * stride / k
  bool dots;   // few rows of many features: each logit a dot product of one wave; otherwise fp32 matrix-core tiles
};
struct SampleStageArgs {
  HeadView head;
  int C, B, H, mode;
  float* logits;        // [B x C] out, or null
  const int32_t* y;
  const uint8_t* mask;  // may be null
  const float* lambda;  // [3H+1] weighting net, then the corrector [Hc*2C + Hc + C*Hc + C] when Hc > 0
  int Hc; float kappa;  // label corrector (BASE and GLAM): Hc = 0 turns it off
  float* losses;        // [B] out (may be null in EVAL)
  float* weights;       // [B] out, w(l_i; lambda), or null
  float* dlogits;       // [B x C] out, row stride C (BASE, META)
  float* loss_scalar;   // out: sum_i coef_i l_i
  float* loss_user;     // optional second destination
  // GLAM: both passes of Eq. 5 in one launch, then the combine and the update of `mu` (which may write `lambda`)
  MetaUpdateArgs mu;
  double* part;         // partials: 2 * stage_blocks(B) * n_lambda (GLAM), stage_blocks(B) (BASE, META)
  uint32_t* ticket;     // zero; zero again after the launch
  StepScalars step;     // counters != null: also advances the base solver's step-dependent scalars
  // Sequence mode (pos_loss != null; BASE or GLAM): sample i is sequence i of B, its loss the mean of pos_loss[j] over
  // the positions with pos_row[j] / S == i (0 without any); head, y, dlogits are unused.  The - pass of GLAM reads pos_loss
  // pos_pass_stride behind the + pass.  BASE writes
  // pos_coef[j] = mask_i w_i / (B_eff count_i) and ADDS sum_i coef_i l_i to *loss_scalar (and *loss_user).
  const float* pos_loss; const int32_t* pos_row; int n_pos, S; int64_t pos_pass_stride;
  float* pos_coef;
};
void launch_sample_stage(hipStream_t, const SampleStageArgs&);

// ------------------------------------------------------------------ fp32 GEMM (gemm_f32.hip)
// C[M x N] = sum_k A(i,k) B(k,j), A(i,k) = A[i*sa_i + k*sa_k], B(k,j) = Bh[k*sb_k + j*sb_j] (+ bscale * Bv[same]),
// bscale = bsign * (*beps) when Bv != null.  Epilogue: + bias(j) (a ParamView index bias_off + j), then
// relu, or multiplication by (gate[i*ldc + j] > 0).
struct GemmF32Args {
  const float* A; int64_t sa_i, sa_k;
  const float* B; const float* Bv; const float* beps; float bsign; int64_t sb_k, sb_j;
  float* C; int64_t ldc;
  int M, N, K;
  const float* bias; const float* bias_v;  // null = no bias; perturbed with the same bscale
  const float* gate;                       // null = none
  int relu;
  float* rowsum;                           // null, or [M] out: rowsum[i] = sum_k A(i,k) (the bias gradient beside a weight gradient)
};
constexpr int GEMM_F32_MAX_JOBS = 2;
// The base solver's update of all n parameters, for a launch that computes the last of their gradients.
struct BaseUpdate {
  int solver;                             // 0: none, 1: Adam, 2: SGD
  AdamArgs adam; float lr, wd, mu;
  float *g, *m, *v, *theta; int64_t n;
  int64_t apart, apart_count;             // the first, and how many, of those that the launch leaves alone: behind its product's C, before its rowsum
};
// A weight gradient (C and rowsum inside u.g) in one launch with the update of every parameter: the launch's own results are updated as
// they are stored, the other gradients (but for those set apart) by workgroups beside those of the product.  us a base step with the update in a launch of its own /
// with the last gradient, Adam: 66 parameters 13.4 / 11.6, 63 thousand 29.9 / 27.4, 269 thousand 33.3 / 30.7, 531 thousand 58.9 / 54.7,
// 1.6 million 80 / 70; SGD 12.9 / 11.4, 29.4 / 27.0, 32.5 / 30.1, 56.7 / 53.8, 74.7 / 69.8.
void launch_gemm_f32_update(hipStream_t, const GemmF32Args& a, const BaseUpdate& u);
// one or two independent problems in one launch
void launch_gemm_f32_batch(hipStream_t, const GemmF32Args* p, int count);

// ------------------------------------------------------------------ bf16 MFMA GEMM (gemm_bf16.hip)
enum { GEMM_ACT_NONE = 0, GEMM_ACT_GELU_FWD = 1, GEMM_ACT_GELU_BWD = 2 };
// C[M x N] = A . (B + B2).  a_trans = 0: A stored [M][K]; 1: stored [K][M].  b_trans = 1: B stored [N][K]
// (a weight matrix [out x in] used forward); 0: stored [K][N].  B2 (same storage as B) may be null.
// Epilogue, in this order: + bias[j] (+ bsign * *beps * bias_v[j]); + res32 [i*ldc + j] (not with GELU_BWD);
// GELU_FWD: C16_pre = bf16(c) (stored when C16_pre is given), c = gelu(that);  GELU_BWD: c *= gelu'(aux16[i*ldc + j]);  stores to C32 and/or C16.
struct GemmBf16Args {
  const bf16_t* A; int64_t lda; int a_trans;
  const bf16_t* B; const bf16_t* B2; int64_t ldb; int b_trans;
  int M, N, K;
  int64_t ldc;
  const float* bias; const float* bias_v; const float* beps; float bsign;
  const float* res32;
  // null, or res32 is the input of a LayerNorm whose output is the residual (forward hi + lo products): the mean of each row, 1 / deviation ln_rstd behind it,
  // and gain and shift of each column ln_g and ln_b from the bias (from bias_v what perturbs them)
  const float* ln_mean; int32_t ln_rstd, ln_g, ln_b;
  int act; const bf16_t* aux16; bf16_t* C16_pre;
  const float* gelu_tab;   // the GELU epilogues: what launch_gelu_tables() wrote
  float* C32; bf16_t* C16;
  const int32_t* rows;   // null, or (device) the token rows in use: a multiple of 64 that replaces M (a_trans = 0) or K (a_trans = 1)
};
// The factors of gelu and gelu' for every bf16 value (gelu.h), gelu_table_bytes() bytes, 16-byte aligned.
size_t gelu_table_bytes();
void launch_gelu_tables(hipStream_t, float* tab);
const char* check_gemm_bf16(const GemmBf16Args&);  // null if the shapes / alignments are supported
void launch_gemm_bf16(hipStream_t, const GemmBf16Args&);
// Up to GEMM_MAX_BATCH independent problems in one launch; they must agree in a_trans, b_trans and in whether B2 is
// given (shapes, K and epilogues may differ).
constexpr int GEMM_MAX_BATCH = 4;
const char* check_gemm_bf16_batch(const GemmBf16Args* p, int count);
void launch_gemm_bf16_batch(hipStream_t, const GemmBf16Args* p, int count);
void encoder_side_sink(bool on);         // tuning hook: per-layer gradient consumers on that stream (default on)
void encoder_side_stream(int mode);     // tuning hook: weight-gradient launches on a second stream: 0 never, 2 always, else (default) by size
// tuning hooks: the choice of k_gemm_rows (0: the heuristic; false: not four bits of 1, 2, 4 or 5 for each sixteenth), and how often which launch was made
// since the last call
bool gemm_bf16_force_rows(uint64_t choice);
enum { GEMM_ROWS_NT, GEMM_ROWS_NN, GEMM_COUNTS };
void gemm_bf16_take_counts(int64_t* counts);
void gemm_bf16_force_shape(int shape);  // tuning hook: 0 = heuristic, else 100 * tile-order group + tile configuration id

// ------------------------------------------------------------------ encoder ops (encoder_ops.hip)
constexpr int LN_MAX_D = 2048;       // LayerNorm kernels keep a row in registers (4 or 8 16-byte pieces per lane)
constexpr int LN_BWD_ROWS = 8;       // rows per block in the LayerNorm backward (size of its partial sums)
constexpr int COLSUM_ROWS = 16;      // rows per block in the column-sum kernel
// Where the token rows of a padded batch lie.  Of each sequence only the positions that can influence a result are there, its
// real tokens (and masked positions), rounded up to 16 so that the groups of 16 rows the matrix cores add at a time are those of
// the padded batch and every sum over rows keeps its order; the sequences follow one another.  All null: nothing is left out,
// position p of sequence b is row b S + p.
constexpr int ROW_GROUP = 16;
constexpr int MAX_SEQ = MAX_TOKENS / 64;
struct RowPlan {
  int32_t* start;   // [B + 1] row of each sequence's position 0; start[B] = rows of all sequences
  int32_t* rows;    // [1] start[B] rounded up to a multiple of 64
  int32_t* ids;     // [M] token of each row (0 behind start[B])
  int32_t* src;     // [M] b S + p of each row (-1 behind start[B])
  int32_t* group;   // [M / 16] where each group of 16 rows of the padded batch went, in groups, or -1
};
struct RowSelect;
// lens [B]: real tokens; sel.n_mask > 0: masked positions to keep as well
void launch_row_plan(hipStream_t, const int32_t* ids, const int32_t* lens, int B, int S, const RowSelect& sel, const RowPlan& out);
// Weights that the products behind a LayerNorm will read: workgroups of its launch beside those of the rows fetch them.
struct WeightsAhead {
  const bf16_t* p[4]; int64_t n;   // up to four arrays of n values each (a multiple of 64), or null; n = 0: none
  int max_rows;                    // no longer worth it with this many rows in use
};
constexpr int AHEAD_BLOCKS = 256;
struct LnFwdArgs {
  const float* x;          // [M x d] input, or null: embedding mode (x = tok_emb[id] + pos_emb[m % S])
  const int32_t* ids; int S; int64_t tok_off, pos_off; float* x_out;  // embedding mode; x_out [M x d] may be null
  int V;                   // embedding mode: vocabulary size, ids are clamped into [0, V)
  int pass_rows;           // rows of one of the stacked passes (0: not stacked); they share the ids
  const int32_t* rows;     // null, or rows in use of each pass (RowPlan); embedding mode then takes src's positions
  const int32_t* src;
  ParamView pv; int64_t g_off, b_off;                                 // gamma / beta inside theta
  bf16_t* y; float* y32; float* mean; float* rstd;                    // y32 (fp32 copy for the residual path), mean, rstd may be null
  int M, d;
  WeightsAhead ahead;
};
void launch_ln_fwd(hipStream_t, const LnFwdArgs&);
struct LnBwdArgs {
  const float* dy; const float* x; const float* mean; const float* rstd; const float* gamma;
  float* dx32; bf16_t* dx16;
  float* partial;          // [ceil(M / LN_BWD_ROWS)][3][d]: dgamma, dbeta, column sums of dx
  int M, d;
  const int32_t* rows;     // null, or rows in use
  WeightsAhead ahead;
};
void launch_ln_bwd(hipStream_t, const LnBwdArgs&);
// out_v[c] = sum_r partial[r*stride + v*vstride + c] for the non-null outputs v = 0, 1, 2, in a fixed order
void launch_reduce_rows(hipStream_t, const float* partial, int nrows, int64_t stride, int64_t vstride, int N, float* out0,
                        float* out1, float* out2);
// the same for up to REDUCE_MAX_JOBS independent reductions in one launch (a job with fewer than three outputs
// leaves the trailing out[] null)
constexpr int REDUCE_MAX_JOBS = 4;
// A matrix of selected rows (SELECT_SEQ_ROWS of every row_step token rows) is reduced in the order of its token rows: `nrows`
// counts them all, in blocks of row_step / blocks_per_seq, and those of the rows left out are skipped.
struct ReduceRowsJob {
  const float* partial; int nrows; int64_t stride, vstride; int N; float* out[3];
  int seq_blocks, kept_blocks;              // 0, or: of each seq_blocks blocks the first kept_blocks are there
  const int32_t* group; int group_blocks;   // null, or RowPlan's, and blocks per group
};
void launch_reduce_rows_multi(hipStream_t, const ReduceRowsJob* jobs, int count);
// first stage of the column sums of up to two bf16 matrices [M x N] (ld = N): partial [ceil(M / COLSUM_ROWS)][N]
struct ColsumJob { const bf16_t* X; int M, N; float* partial; const int32_t* rows; };   // rows: null, or rows in use
void launch_colsum_partial_multi(hipStream_t, const ColsumJob* jobs, int count);
// column sums of a bf16 matrix [M x N] (ld = N) through partial [ceil(M / COLSUM_ROWS)][N]
void launch_colsum_bf16(hipStream_t, const bf16_t* X, int M, int N, float* partial, float* out);
// softmax(q k^T / 8) v for S in {64, 128, 256} (attention_supports), head width 64; qkv [B*S x 3d] bf16; out [B*S x d]
// bf16; lse [nw B][heads][S]; nw stacked passes of B sequences.  lens (device, or null = all S): sequence b has lens[b] real
// tokens (clamped into [1, S]); keys beyond get no weight; its rows lie where the plan says.  Rows of the plan that belong to
// no sequence get zeros.
bool attention_supports(int S);
void launch_attention_fwd(hipStream_t, const bf16_t* qkv, bf16_t* out, float* lse, int nw, int B, int S, int heads, int d,
                          const int32_t* lens, const RowPlan& plan);
void launch_attention_bwd(hipStream_t, const bf16_t* qkv, const bf16_t* out, const bf16_t* dout, const float* lse,
                          bf16_t* dqkv, int B, int S, int heads, int d, const int32_t* lens, const RowPlan& plan);
// The token rows whose last hidden state is read, side by side in a compact matrix of n rows (a multiple of 64; rows without a
// token are zero).  Either the first SELECT_SEQ_ROWS positions of each of n_cls sequences -- the classifier reads the first of
// them, and sums over token rows keep the composition of the groups of 16 that the matrix cores add at a time --, or
// (n_mask > 0) the masked positions.
constexpr int SELECT_SEQ_ROWS = 16;
struct RowSelect {
  int n, S, n_cls;
  int n_mask;
  const int32_t* mask_rows;                 // [n_mask] token row among the mask_total rows from mask_base on, clamped into range
  int mask_base, mask_total;
  const int32_t* start;                     // RowPlan's (null: nothing left out)
};
// token row of compact row i (i < s.n), or -1 where there is none
__device__ __forceinline__ int selected_row(const RowSelect& s, int i) {
  if (s.n_mask > 0) {
    if (i >= s.n_mask) return -1;
    const int r = s.mask_base + min(max(s.mask_rows[i], 0), s.mask_total - 1);
    return s.start != nullptr ? s.start[r / s.S] + r % s.S : r;
  }
  const int b = i / SELECT_SEQ_ROWS;
  if (b >= s.n_cls) return -1;
  return (s.start != nullptr ? s.start[b] : b * s.S) + i % SELECT_SEQ_ROWS;
}
// compact row i of pass k <- row of token i (passes pass_rows apart in the sources, n in the results); x32 / x32_out may be null
void launch_select_rows(hipStream_t, const RowSelect&, int nw, int pass_rows, int d, const bf16_t* a16, const float* x32, bf16_t* a16_out,
                        float* x32_out);
// The adjoint for a selection by sequence: each of the M token rows = its compact row, or zero
void launch_spread_rows(hipStream_t, const RowSelect&, const RowPlan&, int M, int d, const bf16_t* a16, const float* x32, bf16_t* a16_out, float* x32_out);
// dWc, dbc into grad; dx[r][:] = dlogits[b] . Wc for r = b S, or r = start[b] when start is given, zeros in the others of its `rows`
void launch_head_bwd(hipStream_t, const float* x, int S, const int32_t* start, int d, int B, int C, const float* theta, int64_t wc_off,
                     int64_t bc_off, const float* dlogits, float* grad, float* dx, int rows);
// embedding gradients from demb [B*S x d]: pos_emb rows summed over the batch; tok_emb rows summed over the
// occurrences of each id in ascending position order (the tok_emb part of grad must be zero on entry)
// (ids outside [0, V) are clamped into it, here and in the forward pass)
// with a plan: demb by its rows, ids the plan's
void launch_embedding_bwd(hipStream_t, const float* demb, const int32_t* ids, int B, int S, int d, int V, float* g_tok, float* g_pos,
                          const RowPlan& plan);


// ------------------------------------------------------------------ masked-token head (mlm_head.hip)
// ids_out = [ids_ft | ids_pt] ([n x S] token rows), y_out = [y_ft | 0], mask_out = [mask_ft (null = ones) | 0]
void launch_aux_cat(hipStream_t, const int32_t* ids_ft, const int32_t* y_ft, const uint8_t* mask_ft, int n_ft,
                    const int32_t* ids_pt, int n_pt, int S, int32_t* ids_out, int32_t* y_out, uint8_t* mask_out,
                    const int32_t* len_ft, const int32_t* len_pt, int32_t* len_out);
// row j of pass k of X (passes pass_stride apart) as the two-term split hi = bf16(x), lo = bf16(x - hi) in row k P + j;
// rows n_mask..P-1 of a pass are zero
void launch_split_rows(hipStream_t, const float* X, int64_t pass_stride, int n_mask, int P, int d, int nw, bf16_t* hi, bf16_t* lo);
// loss_pos[k P + j] = logsumexp(Z[k P + j][:V]) - Z[k P + j][tgt[j]], lse_pos likewise (V % 4 == 0)
void launch_mlm_ce(hipStream_t, const float* Z, int V, int P, const int32_t* tgt, int n_mask, int nw, float* loss_pos,
                   float* lse_pos);
// dZ [P x V] bf16 = coef_pos[j] (softmax(Z[j]) - onehot(tgt[j])), zero rows from n_mask on
void launch_mlm_dz(hipStream_t, const float* Z, int V, const int32_t* tgt, const float* coef_pos, const float* lse_pos,
                   int n_mask, int P, bf16_t* dZ);
// dx[selected_row(sel, j)][:] += sum_{k < nparts} part[k * part_stride + j * d + :] for the masked positions j; they are distinct
void launch_scatter_add_rows(hipStream_t, const float* part, int nparts, int64_t part_stride, const RowSelect& sel, int d, float* dx);

}  // namespace sama
