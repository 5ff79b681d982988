// Post-LN transformer encoder classifier in bf16 with fp32 accumulation: the explicit forward / backward kernel
// sequence (no autograd).  x0 = LN(tok[ids] + pos); per layer x <- LN1(x + Attn(x)), x <- LN2(x + FFN(x));
// logits = x_L[:, 0] Wc^T + bc.  Residual sums and every LayerNorm input stay fp32; GEMM operands are bf16.
#include <algorithm>
#include <cmath>
#include "kernels.h"
#include "model.h"

namespace sama {
static int g_side_stream = 1;   // 0 never, 2 always, else the rule below
static bool g_side_sink = true;
void encoder_side_stream(int mode) { g_side_stream = mode; }
void encoder_side_sink(bool on) { g_side_sink = on; }
namespace {
// Whether a backward pass over `rows` token rows (of a padded batch: all of them) puts a layer's weight gradients and what follows
// them on the second stream.  They run beside the next layer's chain, so a single layer gains nothing and pays for the join
// (8192 rows of 1 x 512: 1151 us an iteration of one base step on two streams, 1071 on one).  With several layers it is worth it once
// the chain's kernels are long enough, and the layers many enough, for what it costs: with an iteration's two backward passes 100 us of
// host time for each layer and, at their ends, 65 to 120 us of the GPU's (what a single layer loses).  The line lies where rows x
// parameters of the layers x sqrt(rows / 1024) do; in 1e9, us on two streams / one: 1.9 (512 rows, 12 x 192) 2948 / 2806, 7.2 (1024,
// 4 x 384) 1468 / 1408, 7.7 (512, 12 x 384) 3750 / 3686, 9.1 (2048, 4 x 256) 1318 / 1313, 10.2 (2048, 2 x 384) 960 / 926, 10.9 (256,
// 12 x 768) 5536 / 5560, 12.9 (4096, 2 x 256) 878 / 898, 14.5 (4096, 4 x 192) 1481 / 1548, 20.5 (2048, 4 x 384) 1750 / 1764, 36 (2048,
// 4 x 512) 2056 / 2124, 43 (4096, 12 x 192) 4334 / 4698.  Of 172 shapes (1 to 24 layers of 192 to 1024, 256 to 8192 rows, 16 of them
// padded) four take more than 1 % longer than on the other side, at most 3.2 %; by the plain product of rows and parameters 19
// (6.9 %), by that of one layer 18 (6.2 %).  With the products faster (16x16x32 MFMAs) 16 do, at most 3.3 %; lines from 8 to 30 are no better
// than this one: profiles/second_stream.md.
inline bool side_wanted(int64_t rows, int layers, int64_t layer_params) {
  if (g_side_stream == 0 || g_side_stream == 2) return g_side_stream == 2;
  return layers > 1 && (double)rows * (double)(layers * layer_params) * std::sqrt((double)rows / 1024.0) >= 1.05e10;
}

struct LayerOff { int64_t Wqkv, Wo, W1, W2, bqkv, bo, ln1g, ln1b, b1, b2, ln2g, ln2b; };

class EncoderModel : public Model {
 public:
  EncoderModel(const sama_config& c, const std::vector<TensorInfo>& lay) {
    L_ = c.dims[0]; d_ = c.dims[1]; heads_ = c.dims[2]; ffn_ = c.dims[3]; S_ = c.dims[4]; V_ = c.dims[5]; C_ = c.dims[6];
    auto find = [&](const std::string& nm) { for (auto& t : lay) if (t.name == nm) return t.offset; return (int64_t)-1; };
    for (int l = 0; l < L_; ++l) {
      const std::string p = "l" + std::to_string(l) + ".";
      off_.push_back({find(p + "Wqkv"), find(p + "Wo"), find(p + "W1"), find(p + "W2"), find(p + "bqkv"), find(p + "bo"),
                      find(p + "ln1_g"), find(p + "ln1_b"), find(p + "b1"), find(p + "b2"), find(p + "ln2_g"), find(p + "ln2_b")});
    }
    tok_ = find("tok_emb"); pos_ = find("pos_emb"); eg_ = find("emb_ln_g"); eb_ = find("emb_ln_b"); wc_ = find("Wc"); bc_ = find("bc");
    wm_ = find("Wmlm"); bm_ = find("bmlm");
    Pmax_ = wm_ >= 0 ? (c.max_aux_masked + 63) / 64 * 64 : 0;
  }
  int n_classes() const override { return C_; }
  bool has_mlm() const override { return wm_ >= 0; }
  int mlm_stride() const override { return P_; }

  void plan(BumpAlloc& ws, int max_b) override {
    const size_t sel = std::max(((size_t)max_b * SELECT_SEQ_ROWS + 63) / 64 * 64, (size_t)Pmax_);   // most selected rows
    const size_t M = (size_t)max_b * S_;                                                            // >= sel
    X_.resize(L_ + 1); qkv_.resize(L_); lse_.resize(L_); ao_.resize(L_); pre1_.resize(L_); mean1_.resize(L_); rstd1_.resize(L_);
    x1_.resize(L_); fpre_.resize(L_); fact_.resize(L_); pre2_.resize(L_); mean2_.resize(L_); rstd2_.resize(L_);
    // Forward-only passes run in activation slot 0 and ping-pong between X_[0] / X_[1]; the + and the - pass of
    // Eq. 5 run stacked (2M rows), so those buffers are twice as tall.
    for (int l = 0; l <= L_; ++l) X_[l] = ws.take<bf16_t>((l < 2 ? 2 : 1) * M * d_);
    for (int l = 0; l < L_; ++l) {
      const size_t R = (l == 0 ? 2 : 1) * M;
      qkv_[l] = ws.take<bf16_t>(R * 3 * d_); lse_[l] = ws.take<float>((size_t)max_b * heads_ * S_);
      ao_[l] = ws.take<bf16_t>(R * d_); pre1_[l] = ws.take<float>(R * d_); mean1_[l] = ws.take<float>(M); rstd1_[l] = ws.take<float>(M);
      x1_[l] = ws.take<bf16_t>(R * d_); fpre_[l] = ws.take<bf16_t>(R * ffn_); fact_[l] = ws.take<bf16_t>(R * ffn_);
      pre2_[l] = ws.take<float>(R * d_); mean2_[l] = ws.take<float>(M); rstd2_[l] = ws.take<float>(M);
    }
    gelu_tab_ = (float*)ws.take<char>(gelu_table_bytes());
    plan_.start = ws.take<int32_t>(MAX_SEQ + 1); plan_.rows = ws.take<int32_t>(1); plan_.ids = ws.take<int32_t>(M); plan_.src = ws.take<int32_t>(M);
    plan_.group = ws.take<int32_t>(M / ROW_GROUP);
    pre0_ = ws.take<float>(M * d_); mean0_ = ws.take<float>(M); rstd0_ = ws.take<float>(M);
    dX_[0] = ws.take<float>(M * d_); dX_[1] = ws.take<float>(M * d_);
    res_[0] = ws.take<float>(2 * M * d_); res_[1] = ws.take<float>(2 * M * d_);
    ds32_ = ws.take<float>(M * d_); do_ = ws.take<bf16_t>(M * d_);
    ao_sel_ = ws.take<bf16_t>(2 * sel * d_); res_sel_ = ws.take<float>(2 * sel * d_); do_sel_ = ws.take<bf16_t>(sel * d_);
    // What a layer's weight-gradient launches read exists twice (layer parity): they run on a second stream while the
    // next layer's backward chain already writes the other set.
    for (int p = 0; p < 2; ++p) {
      ds16_[p][0] = ws.take<bf16_t>(M * d_); ds16_[p][1] = ws.take<bf16_t>(M * d_);
      dpre_[p] = ws.take<bf16_t>(M * ffn_); dqkv_[p] = ws.take<bf16_t>(M * 3 * d_);
    }
    const size_t nblk = (M + LN_BWD_ROWS - 1) / LN_BWD_ROWS, nrb = (M + COLSUM_ROWS - 1) / COLSUM_ROWS;
    const size_t wide = (size_t)(3 * d_ > ffn_ ? 3 * d_ : ffn_);
    for (int p = 0; p < 2; ++p) {
      lnpart_[p][0] = ws.take<float>(nblk * 3 * d_); lnpart_[p][1] = ws.take<float>(nblk * 3 * d_);
      cspart_[p][0] = ws.take<float>(nrb * wide); cspart_[p][1] = ws.take<float>(nrb * wide);
    }
    if (has_mlm()) {   // masked-token head: up to Pmax_ positions, two stacked passes
      const size_t P = Pmax_;
      hm_ = ws.take<bf16_t>(2 * P * d_); hm_lo_ = ws.take<bf16_t>(2 * P * d_); zt_ = ws.take<float>(2 * P * V_); lse_pos_ = ws.take<float>(2 * P);
      dzt_ = ws.take<bf16_t>(P * V_); dhm_ = ws.take<float>((size_t)GEMM_MAX_BATCH * P * d_);
      cs_mlm_ = ws.take<float>((P + COLSUM_ROWS - 1) / COLSUM_ROWS * V_);
    }
  }

  void prepare(hipStream_t st) override { launch_gelu_tables(st, gelu_tab_); }

  struct LnOff { int64_t g, b; };   // gain and shift of a LayerNorm inside theta
  struct RowStats { float *mean, *rstd; };
  struct LnInput { const float* x; RowStats st; LnOff off; };   // what a LayerNorm's output is made of
  // One linear layer of `nw` stacked passes (pass k owns rows [k M, (k + 1) M) of every activation): the same
  // epilogue `e` (its pointers are those of pass 0) for each pass, with that pass's weights, those of the LayerNorm `ln` where the residual is its output.
  void fwd_linear(hipStream_t st, const PassWeights* w, int nw, const bf16_t* A, int K, int64_t woff, int N, int64_t boff, int M,
                  const GemmBf16Args& e, const int32_t* rows = nullptr, LnOff ln = {}) const {
    GemmBf16Args g[2];
    for (int k = 0; k < nw; ++k) {
      g[k] = e;
      const int64_t ro = (int64_t)k * M * N;
      g[k].A = A + (int64_t)k * M * K; g[k].lda = K; g[k].a_trans = 0;
      g[k].B = w[k].hi + woff; g[k].B2 = w[k].lo ? w[k].lo + woff : nullptr; g[k].ldb = K; g[k].b_trans = 1;
      g[k].M = M; g[k].N = N; g[k].K = K; g[k].ldc = N; g[k].rows = rows;
      g[k].bias = w[k].theta + boff;
      if (w[k].sign != 0.f) { g[k].bias_v = w[k].vdir + boff; g[k].beps = w[k].eps_ptr; g[k].bsign = w[k].sign; }
      if (e.res32) g[k].res32 = e.res32 + ro;
      if (e.ln_mean) { g[k].ln_mean = e.ln_mean + (int64_t)k * M; g[k].ln_g = (int32_t)(ln.g - boff); g[k].ln_b = (int32_t)(ln.b - boff); }
      if (e.C32) g[k].C32 = e.C32 + ro;
      if (e.C16) g[k].C16 = e.C16 + ro;
      if (e.C16_pre) g[k].C16_pre = e.C16_pre + ro;
    }
    launch_gemm_bf16_batch(st, g, nw);
  }

  // What follows the last attention is row by row, and of its result only position 0 of each sequence (the classifier) or
  // the masked positions are read, so the last layer's output projection, LayerNorms and FFN, 9/12 of its matrix work, run on
  // those rows alone, side by side; the other rows have no influence on a result and their gradients are zero.  A pass that
  // keeps what the backward of both heads needs (n = 0) stays on all rows: the masked ones lie in nearly every group of 16 rows.
  RowSelect select(const sama_batch& b, bool keep, const MlmBatch* mb) const {
    RowSelect s{};
    s.S = S_; s.start = b.seq_len != nullptr ? plan_.start : nullptr;
    if (mb != nullptr) {
      if (keep) return s;
      s.n_mask = mb->n_mask; s.mask_rows = mb->rows; s.mask_base = mb->row_base; s.mask_total = mb->rows_in_batch;
      s.n = (mb->n_mask + 63) / 64 * 64;
    } else {
      s.n_cls = b.n;
      s.n = (b.n * SELECT_SEQ_ROWS + 63) / 64 * 64;
    }
    return s;
  }

  // The next weights for the LayerNorm of a pass over `rows` rows to fetch, where that pays: the products of few rows are bound by weights
  // that come from memory, and a LayerNorm leaves most of its bandwidth unused.  With the rows of a long product there is
  // time for both, and fetching ahead only delays the LayerNorm; and what the last-level cache (256 MB) holds from one pass to the
  // next needs no fetching: when scoring, the two halves of the weights; in training, with the optimizer's state, 20 bytes each.
  // us without it / with it, where the rule has it: 12 x 768 scoring 128 rows 678 / 647, 512 828 / 738, 2048 1378 / 1237, base step of 1024 rows
  // 3039 / 2831, of 2048 3918 / 3659; 24 x 1024 base step of 512 rows 6828 / 6422; 12 x 768 iteration of 1024 rows 7670 / 7163; base step of
  // 2048 rows of 8 x 384 (260 MB with the state) 1436 / 1390.  Without it / with it, where the rule leaves it out: 12 x 768 scoring 4096 rows
  // 1893 / 1864, base step of 4096 5471 / 5454; 24 x 1024 base step of 2048 rows 10418 / 10350; scoring 128 rows of 12 x 576
  // (177 MB) 542 / 551.  The stacked passes count the rows of both: left out of them, as the rule does at 24 x 1024 and 1024 rows, an
  // iteration takes 18867 us, with it there too 18928.
  // Padded batches go on to twice as many rows in use: the tiles that are chosen on the device have no wave that touches weights ahead.  Without it /
  // with it, 4096 rows, about 2900 in use: base step of 12 x 768 4515 / 4354, 12 x 960 5680 / 5621, 12 x 1024 6138 / 6088; 24 x 1024 base step of 3584 rows
  // 12034 / 11661, scoring 3072 3736 / 3549, iteration of 3584 31847 / 30669, of 2048 23534 / 23699 (the most that any of 130 calls loses, 1.2 % on
  // another card); 12 x 896 and narrower than 768 within 0.7 %.  Without lengths nothing changes at 4096 rows (5512 / 5507), and at 24 x 1024 2048 rows
  // lose (27180 / 27540).
  WeightsAhead weights_ahead(const PassWeights* w, int nw, bool scoring, int64_t off, int64_t n, int rows, const int32_t* in_use) const {
    WeightsAhead a{};
    a.max_rows = ((in_use != nullptr ? 4 : 2) << 20) / (nw * d_);
    const int64_t params = L_ * ((int64_t)4 * d_ * d_ + (int64_t)2 * ffn_ * d_);
    if (params * (scoring ? 4 : 20) < 256000000 || (in_use == nullptr && rows >= a.max_rows)) return a;
    for (int k = 0; k < nw; ++k) { a.p[2 * k] = w[k].hi + off; a.p[2 * k + 1] = w[k].lo != nullptr ? w[k].lo + off : nullptr; }
    a.n = n;
    return a;
  }

  // nw = 1: one pass with weights w[0].  nw = 2: the theta + eps v and theta - eps v passes of Eq. 5 on the same
  // batch, stacked along the row dimension (forward only, keep must be false).
  HeadView run_forward(hipStream_t st, const PassWeights* w, int nw, const sama_batch& b, bool keep, const MlmBatch* mb) {
    const int B = b.n, M = B * S_;
    const RowSelect sel = select(b, keep, mb);
    const RowPlan rp = b.seq_len != nullptr ? plan_ : RowPlan{};   // a padded batch: only the rows that matter
    const bool scoring = nw == 1 && !keep;
    if (b.seq_len != nullptr) launch_row_plan(st, (const int32_t*)b.x, b.seq_len, B, S_, mb ? masked(b, *mb) : RowSelect{}, rp);
    // The residual is made by the product that adds it, from the input and the statistics of the LayerNorm, which saves the LayerNorm's
    // fp32 output, 4 of 10 bytes an element that it reads and writes; the bits are the same.  (The last LayerNorm's, and that of the one before the rows are
    // selected, have other readers; so have all of a pass on the bf16 weights alone, whose tiles do without.)
    // It pays once the LayerNorm is bound by memory; a smaller product's epilogue is a chain that gets longer.  us stored / made: scoring 128 rows of 12 x 768 551 / 549 to 560,
    // 1024 rows of 6 x 768 427 / 429, 1024 of 6 x 1024 545 / 541, 2048 759 / 753, 4096 of 6 x 768 860 / 849, 8192 of 8 x 384 836 / 822; base step of 2048 rows of
    // 8 x 384 1316 / 1319, 4096 1740 / 1728, 2048 of 6 x 1024 2780 / 2772.
    // All rows count, also of a padded batch: how many are in use only the device knows, and with few of them it does not lose either.  4096 rows,
    // 15 %, 30 % and 60 % in use: scoring 6 x 1024 684 / 673, 782 / 764, 959 / 935, 6 x 384 300 / 293, 314 / 308, 367 / 357; base step of 6 x 768 1425 / 1415,
    // 1580 / 1571, 1943 / 1916; meta step of 6 x 768 2171 / 2138, 2472 / 2440, 3180 / 3141.  Of 105 such calls from 1536 rows on three take longer, by at most 0.6 % (the stacked
    // passes of 1536 and 2048 rows of 6 x 384).
    constexpr int64_t MAKE_RES = 1 << 20;
    const bool make_res = w[0].lo != nullptr && (int64_t)nw * M * d_ >= MAKE_RES;
    const bool far = eb_ - off_[0].bo > INT32_MAX;   // beyond a product's offsets: two billion embedding weights lie between
    auto others_read = [&](int l) { return !make_res || l == L_ - 1 || (l == L_ - 2 && sel.n > 0) || (l < 0 && far); };   // what leaves layer l (-1: the embeddings)
    // A pass that is not kept needs the input and the statistics of a LayerNorm until that product only: they pass through memory that
    // nobody reads then, the embeddings through that of the residual, statistics (the embeddings' and a layer's last ones in turn) through that of the backward pass.
    auto passing = [&](int k) { return make_res ? RowStats{dX_[0] + (int64_t)4 * k * M, dX_[0] + (int64_t)(4 * k + 2) * M} : RowStats{nullptr, nullptr}; };
    float* const emb = keep ? pre0_ : res_[0];
    LnInput before{emb, keep ? RowStats{mean0_, rstd0_} : passing(0), {eg_, eb_}};   // of what comes into the layer
    ParamView pv{w[0].theta, w[0].vdir, w[0].eps_ptr, w[0].sign, nw == 2 ? M : 0};   // flips behind the first pass's rows
    LnFwdArgs e{};
    e.x = nullptr; e.ids = rp.ids ? rp.ids : (const int32_t*)b.x; e.src = rp.src; e.rows = rp.rows; e.pass_rows = M; e.S = S_; e.V = V_; e.tok_off = tok_; e.pos_off = pos_; e.x_out = keep || !others_read(-1) ? emb : nullptr;
    e.pv = pv; e.g_off = eg_; e.b_off = eb_; e.y = X_[0]; e.y32 = others_read(-1) ? res_[0] : nullptr; e.mean = before.st.mean; e.rstd = before.st.rstd;
    e.M = nw * M; e.d = d_; e.ahead = weights_ahead(w, nw, scoring, off_[0].Wqkv, (int64_t)4 * d_ * d_, M, rp.rows);
    launch_ln_fwd(st, e);
    for (int l = 0; l < L_; ++l) {
      const int s = keep ? l : 0;                       // activation slot: forward-only passes reuse slot 0
      const bf16_t* xin = keep ? X_[l] : X_[l & 1];
      bf16_t* xout = keep ? X_[l + 1] : X_[(l + 1) & 1];
      const LayerOff& o = off_[l];
      GemmBf16Args g{};
      g.C16 = qkv_[s];
      fwd_linear(st, w, nw, xin, d_, o.Wqkv, 3 * d_, o.bqkv, M, g, rp.rows);
      launch_attention_fwd(st, qkv_[s], ao_[s], keep ? lse_[s] : nullptr, nw, B, S_, heads_, d_, b.seq_len, rp);
      const bool last = l == L_ - 1 && sel.n > 0;
      const int rows = last ? sel.n : M;            // of one pass, from here on
      const int32_t* const in_use = last ? nullptr : rp.rows;
      if (last) {
        launch_select_rows(st, sel, nw, M, d_, ao_[s], res_[0], ao_sel_, res_sel_);
        if (nw == 2) pv.flip_row = rows;
      }
      g = GemmBf16Args{};
      g.res32 = last ? res_sel_ : res_[0]; g.C32 = pre1_[s];          // the residual stream stays fp32
      LnOff ln{};
      if (!last && !others_read(l - 1)) {
        g.res32 = before.x; g.ln_mean = before.st.mean; g.ln_rstd = (int32_t)(before.st.rstd - before.st.mean);
        ln = before.off;
      }
      fwd_linear(st, w, nw, last ? ao_sel_ : ao_[s], d_, o.Wo, d_, o.bo, rows, g, in_use, ln);
      const RowStats s1 = keep ? RowStats{mean1_[s], rstd1_[s]} : passing(1), s2 = keep ? RowStats{mean2_[s], rstd2_[s]} : passing(0);
      LnFwdArgs n1{};
      n1.x = pre1_[s]; n1.pv = pv; n1.g_off = o.ln1g; n1.b_off = o.ln1b; n1.y = x1_[s]; n1.y32 = make_res ? nullptr : res_[1];
      n1.mean = s1.mean; n1.rstd = s1.rstd; n1.M = nw * rows; n1.d = d_; n1.pass_rows = rows; n1.rows = in_use;
      n1.ahead = weights_ahead(w, nw, scoring, o.W1, (int64_t)2 * ffn_ * d_, rows, in_use);
      launch_ln_fwd(st, n1);
      g = GemmBf16Args{};
      g.act = GEMM_ACT_GELU_FWD; g.gelu_tab = gelu_tab_; g.C16_pre = keep ? fpre_[s] : nullptr; g.C16 = fact_[s];   // only a backward pass reads the pre-activation
      fwd_linear(st, w, nw, x1_[s], d_, o.W1, ffn_, o.b1, rows, g, in_use);
      g = GemmBf16Args{};
      g.res32 = res_[1]; g.C32 = pre2_[s];
      if (make_res) { g.res32 = pre1_[s]; g.ln_mean = s1.mean; g.ln_rstd = (int32_t)(s1.rstd - s1.mean); }
      fwd_linear(st, w, nw, fact_[s], ffn_, o.W2, d_, o.b2, rows, g, in_use, {o.ln1g, o.ln1b});
      LnFwdArgs n2{};
      n2.x = pre2_[s]; n2.pv = pv; n2.g_off = o.ln2g; n2.b_off = o.ln2b; n2.y = xout; n2.y32 = others_read(l) ? res_[0] : nullptr;
      n2.mean = s2.mean; n2.rstd = s2.rstd; n2.M = nw * rows; n2.d = d_; n2.pass_rows = rows; n2.rows = in_use;
      if (l + 1 < L_) n2.ahead = weights_ahead(w, nw, scoring, off_[l + 1].Wqkv, (int64_t)4 * d_ * d_, M, rp.rows);
      launch_ln_fwd(st, n2);
      before = LnInput{pre2_[s], s2, {o.ln2g, o.ln2b}};
    }
    HeadView h{};                                   // position 0 of the fp32 output of the last LayerNorm
    h.x = res_[0]; h.stride = (int64_t)(sel.n > 0 ? SELECT_SEQ_ROWS : S_) * d_; h.pass_stride = (int64_t)(sel.n > 0 ? sel.n : M) * d_; h.k = d_;
    h.pv = ParamView{w[0].theta, w[0].vdir, w[0].eps_ptr, w[0].sign, 0};
    h.w_off = wc_; h.b_off = bc_; h.dots = true;
    h.start = sel.n > 0 ? nullptr : rp.start;
    return h;
  }

  HeadView forward(hipStream_t st, const PassWeights& w, const sama_batch& b, bool keep, const MlmBatch* mb) override {
    if (mb) mask_sel_ = masked(b, *mb);
    return run_forward(st, &w, 1, b, keep, mb);
  }
  HeadView forward_pair(hipStream_t st, const PassWeights& wp, const PassWeights& wm, const sama_batch& b, const MlmBatch* mb) override {
    const PassWeights w[2] = {wp, wm};
    return run_forward(st, w, 2, b, false, mb);
  }

  // (called with the batch of the last forward() or forward_pair())
  void mlm_forward(hipStream_t st, const PassWeights* w, int nw, bool kept, const MlmBatch& mb, float* loss_pos) override {
    P_ = (mb.n_mask + 63) / 64 * 64;
    // A kept pass (base step) contracts the bf16 hidden states like every other layer.  The +- passes of Eq. 5 feed
    // a loss whose difference is the signal: their hidden states enter as the two-term split of the fp32 LayerNorm
    // output, x_hi (W_hi + W_lo) + x_lo W_hi, so that the rounding of x to bf16 does not bury that difference.
    if (kept) launch_select_rows(st, mask_sel_, 1, 0, d_, X_[L_], nullptr, hm_, nullptr);
    else launch_split_rows(st, res_[0], (int64_t)P_ * d_, mb.n_mask, P_, d_, nw, hm_, hm_lo_);   // such a pass ends on the masked rows
    GemmBf16Args g{};
    g.C32 = zt_;
    fwd_linear(st, w, nw, hm_, d_, wm_, V_, bm_, P_, g);
    if (!kept) {
      GemmBf16Args lo[2];
      for (int k = 0; k < nw; ++k) {
        lo[k] = GemmBf16Args{};
        lo[k].A = hm_lo_ + (int64_t)k * P_ * d_; lo[k].lda = d_; lo[k].a_trans = 0;
        lo[k].B = w[k].hi + wm_; lo[k].ldb = d_; lo[k].b_trans = 1;
        lo[k].M = P_; lo[k].N = V_; lo[k].K = d_; lo[k].ldc = V_;
        lo[k].res32 = zt_ + (int64_t)k * P_ * V_; lo[k].C32 = zt_ + (int64_t)k * P_ * V_;   // in place: an element is read and written by the same thread
      }
      launch_gemm_bf16_batch(st, lo, nw);
    }
    launch_mlm_ce(st, zt_, V_, P_, mb.tgt, mb.n_mask, nw, loss_pos, lse_pos_);
  }

  RowSelect masked(const sama_batch& b, const MlmBatch& mb) const { return select(b, false, &mb); }

  // dW[N x K] = dY^T . X into `out`
  GemmBf16Args wgrad(const bf16_t* dY, int N, const bf16_t* X, int K, int M, float* out, const int32_t* rows = nullptr) const {
    GemmBf16Args g{};
    g.A = dY; g.lda = N; g.a_trans = 1;
    g.B = X; g.ldb = K; g.b_trans = 0;
    g.M = N; g.N = K; g.K = M; g.ldc = K; g.C32 = out; g.rows = rows;
    return g;
  }
  // dX[M x K] = dY[M x N] . W[N x K]
  GemmBf16Args dgrad(const PassWeights& w, const bf16_t* dY, int N, int64_t woff, int K, int M, const int32_t* rows) const {
    GemmBf16Args g{};
    g.A = dY; g.lda = N; g.a_trans = 0;
    g.B = w.hi + woff; g.B2 = w.lo ? w.lo + woff : nullptr; g.ldb = K; g.b_trans = 0;
    g.M = M; g.N = K; g.K = N; g.ldc = K; g.rows = rows;
    return g;
  }

  void backward(hipStream_t st, const PassWeights& w, const sama_batch& b, const float* dlogits, float* grad) override {
    run_backward(st, w, b, dlogits, grad, nullptr, nullptr);
  }
  void backward_mlm(hipStream_t st, const PassWeights& w, const sama_batch& b, const float* dlogits, float* grad,
                    const MlmBatch& mb, const float* coef_pos) override {
    run_backward(st, w, b, dlogits, grad, &mb, coef_pos);
  }

  // The masked-token head's backward: dZ = coef (softmax - onehot) in bf16; the hidden-state gradient dZ . Wmlm has a
  // small output and a vocabulary-long contraction, so it runs as up to GEMM_MAX_BATCH K-chunks in one launch whose
  // partial results the scatter adds into the token rows of dx; then dWmlm = dZ^T . H and dbmlm = column sums of dZ.
  void mlm_backward(hipStream_t st, const PassWeights& w, const MlmBatch& mb, const float* coef_pos, float* grad, float* dx) {
    launch_mlm_dz(st, zt_, V_, mb.tgt, coef_pos, lse_pos_, mb.n_mask, P_, dzt_);
    const int slabs = V_ / 64, np = slabs < GEMM_MAX_BATCH ? slabs : GEMM_MAX_BATCH;
    GemmBf16Args g[GEMM_MAX_BATCH];
    for (int k = 0; k < np; ++k) {
      const int64_t k0 = (int64_t)(slabs * k / np) * 64, k1 = (int64_t)(slabs * (k + 1) / np) * 64;
      g[k] = GemmBf16Args{};
      g[k].A = dzt_ + k0; g[k].lda = V_; g[k].a_trans = 0;
      g[k].B = w.hi + wm_ + k0 * d_; g[k].B2 = w.lo ? w.lo + wm_ + k0 * d_ : nullptr; g[k].ldb = d_; g[k].b_trans = 0;
      g[k].M = P_; g[k].N = d_; g[k].K = (int)(k1 - k0); g[k].ldc = d_;
      g[k].C32 = dhm_ + (int64_t)k * P_ * d_;
    }
    launch_gemm_bf16_batch(st, g, np);
    launch_scatter_add_rows(st, dhm_, np, (int64_t)P_ * d_, mask_sel_, d_, dx);
    launch_gemm_bf16(st, wgrad(dzt_, V_, hm_, d_, P_, grad + wm_));
    launch_colsum_bf16(st, dzt_, P_, V_, cs_mlm_, grad + bm_);
  }

  void run_backward(hipStream_t st, const PassWeights& w, const sama_batch& b, const float* dlogits, float* grad,
                    const MlmBatch* mb, const float* coef_pos) {
    const int B = b.n, M = B * S_;
    const RowSelect sel = select(b, true, mb);
    const RowPlan rp = b.seq_len != nullptr ? plan_ : RowPlan{};   // of the kept forward pass
    float* dx = dX_[0];
    float* dx_next = dX_[1];
    launch_head_bwd(st, res_[0], sel.n > 0 ? SELECT_SEQ_ROWS : S_, sel.n > 0 ? nullptr : rp.start, d_, B, C_, w.theta, wc_, bc_, dlogits, grad, dx, sel.n > 0 ? sel.n : M);
    if (mb) mlm_backward(st, w, *mb, coef_pos, grad, dx);
    else if (has_mlm()) {   // a loss without masked-token terms leaves the head's gradient at zero
      launch_fill_f32(st, grad + wm_, 0.f, (int64_t)V_ * d_);
      launch_fill_f32(st, grad + bm_, 0.f, V_);
    }
    // The layer's four weight gradients, its two bias column sums and its four small reductions leave in three
    // launches at the end of the layer, on a second stream of the same priority: nothing in the backward chain
    // depends on them, and the chain's launches (small dgrad tiles, LayerNorm, attention) leave room on the CUs.
    // Their inputs alternate between two buffer sets; the chain waits for the launches of two layers ago before it
    // overwrites a set, and the pass ends with both streams joined.
    const bool two = side_wanted(M, L_, (int64_t)4 * d_ * d_ + (int64_t)2 * ffn_ * d_) && ensure_side();
    hipStream_t ss = two ? side_ : st;
    bool sink_used = false;
    for (int l = L_ - 1; l >= 0; --l) {
      const LayerOff& o = off_[l];
      const int p = l & 1;
      if (two && side_busy_[p]) { (void)hipStreamWaitEvent(st, ev_side_[p], 0); side_busy_[p] = false; }
      bf16_t* const ds2 = ds16_[p][0]; bf16_t* const ds1 = ds16_[p][1]; bf16_t* const dpre = dpre_[p]; bf16_t* const dqkv = dqkv_[p];
      GemmBf16Args wg[4];
      auto ahead = [&](int64_t off, int64_t n) { return weights_ahead(&w, 1, false, off, n, M, rp.rows); };   // as below: W2, W1; Wo, Wqkv
      const bool last = l == L_ - 1 && sel.n > 0;  // the gradient arrives, and stays down to the output projection, on the selected rows
      const int rows = last ? sel.n : M;
      const int32_t* const in_use = last ? nullptr : rp.rows;
      // LN2
      LnBwdArgs n2{dx, pre2_[l], mean2_[l], rstd2_[l], w.theta + o.ln2g, ds32_, ds2, lnpart_[p][0], rows, d_, in_use, ahead(o.W1, (int64_t)2 * ffn_ * d_)};
      launch_ln_bwd(st, n2);
      // FFN
      wg[0] = wgrad(ds2, d_, fact_[l], ffn_, rows, grad + o.W2, in_use);
      GemmBf16Args g = dgrad(w, ds2, d_, o.W2, ffn_, rows, in_use);
      g.act = GEMM_ACT_GELU_BWD; g.gelu_tab = gelu_tab_; g.aux16 = fpre_[l]; g.C16 = dpre;
      launch_gemm_bf16(st, g);
      wg[1] = wgrad(dpre, ffn_, x1_[l], d_, rows, grad + o.W1, in_use);
      g = dgrad(w, dpre, ffn_, o.W1, d_, rows, in_use);
      g.res32 = ds32_; g.C32 = dx_next;                       // + the residual branch
      launch_gemm_bf16(st, g);
      // LN1
      LnBwdArgs n1{dx_next, pre1_[l], mean1_[l], rstd1_[l], w.theta + o.ln1g, ds32_, ds1, lnpart_[p][1], rows, d_, in_use, ahead(o.Wqkv, (int64_t)4 * d_ * d_)};
      launch_ln_bwd(st, n1);
      // attention
      wg[2] = wgrad(ds1, d_, last ? ao_sel_ : ao_[l], d_, rows, grad + o.Wo, in_use);
      g = dgrad(w, ds1, d_, o.Wo, d_, rows, in_use);
      g.C16 = last ? do_sel_ : do_;
      launch_gemm_bf16(st, g);
      const float* dres = ds32_;                              // the residual branch around the attention
      if (last) {
        launch_spread_rows(st, sel, rp, M, d_, do_sel_, ds32_, do_, dx_next);
        dres = dx_next;
      }
      launch_attention_bwd(st, qkv_[l], ao_[l], do_, lse_[l], dqkv, B, S_, heads_, d_, b.seq_len, rp);
      wg[3] = wgrad(dqkv, 3 * d_, X_[l], d_, M, grad + o.Wqkv, rp.rows);
      g = dgrad(w, dqkv, 3 * d_, o.Wqkv, d_, M, rp.rows);
      g.res32 = dres; g.C32 = dx;                             // gradient w.r.t. the layer input
      if (two) {   // everything the side launches read is written by now (the last dgrad only reads dqkv)
        (void)hipEventRecord(ev_chain_[p], st);
        (void)hipStreamWaitEvent(side_, ev_chain_[p], 0);
      }
      launch_gemm_bf16(st, g);
      const bool sink_now = two && g_side_sink && sink_ != nullptr;
      if (sink_now) (void)hipEventRecord(ev_last_[p], st);   // behind the layer's last read of its own weights
      launch_gemm_bf16_batch(ss, wg, 4);
      const ColsumJob cj[2] = {{dpre, rows, ffn_, cspart_[p][0], in_use}, {dqkv, M, 3 * d_, cspart_[p][1], rp.rows}};
      launch_colsum_partial_multi(ss, cj, 2);
      const int nblk = M / LN_BWD_ROWS, nrb = M / COLSUM_ROWS;   // S is a multiple of 64
      const int ls = last ? S_ / LN_BWD_ROWS : 0, lk = SELECT_SEQ_ROWS / LN_BWD_ROWS, cs = last ? S_ / COLSUM_ROWS : 0, ck = SELECT_SEQ_ROWS / COLSUM_ROWS;
      const int32_t* const gr = last ? nullptr : rp.group;
      constexpr int lg = ROW_GROUP / LN_BWD_ROWS, cg = ROW_GROUP / COLSUM_ROWS;
      const ReduceRowsJob rj[4] = {
          {lnpart_[p][0], nblk, 3 * d_, d_, d_, {grad + o.ln2g, grad + o.ln2b, grad + o.b2}, ls, lk, gr, lg},
          {lnpart_[p][1], nblk, 3 * d_, d_, d_, {grad + o.ln1g, grad + o.ln1b, grad + o.bo}, ls, lk, gr, lg},
          {cspart_[p][0], nrb, ffn_, 0, ffn_, {grad + o.b1, nullptr, nullptr}, cs, ck, gr, cg},
          {cspart_[p][1], nrb, 3 * d_, 0, 3 * d_, {grad + o.bqkv, nullptr, nullptr}, 0, 0, rp.group, cg}};
      launch_reduce_rows_multi(ss, rj, 4);
      if (two && l == L_ - 1) launch_fill_f32(side_, grad + tok_, 0.f, (int64_t)V_ * d_);   // for the scatter at the end
      if (two) { (void)hipEventRecord(ev_side_[p], side_); side_busy_[p] = true; }
      if (sink_now) {   // this layer's gradients are final (matrices and vectors are one range each); a consumer may
        (void)hipStreamWaitEvent(side_, ev_last_[p], 0);   // overwrite the layer's weights once its last dgrad has read them
        sink_->ready(side_, o.Wqkv, (int64_t)4 * d_ * d_ + (int64_t)2 * ffn_ * d_);
        sink_->ready(side_, o.bqkv, (int64_t)9 * d_ + ffn_);
        sink_used = true;
      }
    }
    if (sink_used) { (void)hipEventRecord(ev_side_[0], side_); side_busy_[0] = true; }   // join behind the consumer's work too
    // The embeddings need nothing of the last layer's side launches, which end beside them (4 x 256 iteration 1735 -> 1634 us, 12 x 768
    // of 512 rows 6403 -> 6367): only what used lnpart_[1] is waited for first, and with one layer the cleared token rows.
    auto join = [&](int p) { if (two && side_busy_[p]) { (void)hipStreamWaitEvent(st, ev_side_[p], 0); side_busy_[p] = false; } };
    join(1);
    if (L_ == 1) join(0);
    LnBwdArgs n0{dx, pre0_, mean0_, rstd0_, w.theta + eg_, ds32_, nullptr, lnpart_[1][0], M, d_, rp.rows, {}};
    launch_ln_bwd(st, n0);
    const ReduceRowsJob r0{lnpart_[1][0], M / LN_BWD_ROWS, 3 * d_, d_, d_, {grad + eg_, grad + eb_, nullptr}, 0, 0, rp.group, ROW_GROUP / LN_BWD_ROWS};
    launch_reduce_rows_multi(st, &r0, 1);
    if (!two) launch_fill_f32(st, grad + tok_, 0.f, (int64_t)V_ * d_);
    launch_embedding_bwd(st, ds32_, (const int32_t*)b.x, B, S_, d_, V_, grad + tok_, grad + pos_, rp);
    join(0);
  }

  // second stream (default priority, created at the first backward pass that wants it) and the events that order it.  Both streams
  // are this GPU's and no host reads anything by these events, so they go without the system-scope fence, which writes the caches
  // back in the middle of the chain: 4 x 256 iteration 1967 -> 1923 us, 24 x 1024 29.42 -> 29.31 ms.
  bool ensure_side() {
    if (side_ != nullptr) return true;
    if (side_failed_) return false;
    bool ok = hipStreamCreateWithFlags(&side_, hipStreamNonBlocking) == hipSuccess;
    for (int p = 0; p < 2 && ok; ++p)
      ok = hipEventCreateWithFlags(&ev_chain_[p], hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess &&
           hipEventCreateWithFlags(&ev_side_[p], hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess &&
           hipEventCreateWithFlags(&ev_last_[p], hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess;
    if (!ok) { release_side(); side_failed_ = true; (void)hipGetLastError(); }
    return ok;
  }
  void release_side() {
    for (int p = 0; p < 2; ++p) {
      if (ev_chain_[p]) (void)hipEventDestroy(ev_chain_[p]);
      if (ev_side_[p]) (void)hipEventDestroy(ev_side_[p]);
      if (ev_last_[p]) (void)hipEventDestroy(ev_last_[p]);
      ev_chain_[p] = ev_side_[p] = ev_last_[p] = nullptr;
    }
    if (side_) (void)hipStreamDestroy(side_);
    side_ = nullptr;
  }
  ~EncoderModel() override { release_side(); }

 private:
  int L_, d_, heads_, ffn_, S_, V_, C_;
  std::vector<LayerOff> off_;
  int64_t tok_, pos_, eg_, eb_, wc_, bc_, wm_, bm_;
  int Pmax_ = 0, P_ = 0;   // masked-token head: most positions, and those of the last pass (multiples of 64)
  bf16_t* hm_ = nullptr; bf16_t* hm_lo_ = nullptr; float* zt_ = nullptr; float* lse_pos_ = nullptr; bf16_t* dzt_ = nullptr; float* dhm_ = nullptr;
  float* cs_mlm_ = nullptr;
  std::vector<bf16_t*> X_, qkv_, ao_, x1_, fpre_, fact_;
  std::vector<float*> lse_, pre1_, mean1_, rstd1_, pre2_, mean2_, rstd2_;
  float* gelu_tab_ = nullptr;
  RowPlan plan_{};            // of the last padded batch
  RowSelect mask_sel_{};      // masked positions of the last batch with any
  float *pre0_ = nullptr, *mean0_ = nullptr, *rstd0_ = nullptr;
  float* dX_[2] = {nullptr, nullptr};
  float* res_[2] = {nullptr, nullptr};   // fp32 LayerNorm outputs: the residual stream of the current forward pass
  float* ds32_ = nullptr; bf16_t* do_ = nullptr;
  bf16_t *ao_sel_ = nullptr, *do_sel_ = nullptr; float* res_sel_ = nullptr;   // compact rows of the last layer
  bf16_t* ds16_[2][2] = {}; bf16_t* dpre_[2] = {}; bf16_t* dqkv_[2] = {};   // [layer parity]
  float* lnpart_[2][2] = {}; float* cspart_[2][2] = {};
  hipStream_t side_ = nullptr; hipEvent_t ev_chain_[2] = {}, ev_side_[2] = {}, ev_last_[2] = {};
  bool side_busy_[2] = {false, false}, side_failed_ = false;
};
}  // namespace

Model* make_encoder(const sama_config& c, const std::vector<TensorInfo>& layout, std::string& err) {
  const int d = c.dims[1], heads = c.dims[2], ffn = c.dims[3], S = c.dims[4];
  if (!attention_supports(S)) { err = "the encoder kernels are built for S = 64, 128 or 256"; return nullptr; }
  if (d / heads != 64 || d % heads != 0) { err = "the attention kernels are built for head width d/heads = 64"; return nullptr; }
  if (d > LN_MAX_D) { err = "d must be <= 2048"; return nullptr; }
  if (ffn % 64 != 0) { err = "ffn must be a multiple of 64"; return nullptr; }
  const int tb = c.max_batch + (c.aux_mlm ? c.max_aux_batch : 0);
  const int mb = tb > c.max_meta_batch ? tb : c.max_meta_batch;
  if ((int64_t)mb * S > MAX_TOKENS) { err = "max batch (+ max auxiliary batch) * S must be <= 8192 tokens"; return nullptr; }
  if (c.aux_mlm && c.dims[5] % 64 != 0) { err = "the masked-token head needs a vocabulary size that is a multiple of 64"; return nullptr; }
  return new EncoderModel(c, layout);
}

}  // namespace sama
