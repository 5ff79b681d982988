// ReLU MLP / multinomial logistic regression base learner in fp32: each layer is one forward GEMM with a fused
// bias + ReLU epilogue; backward is one launch per layer: the wgrad GEMM with the bias gradient's column sums, and the
// dgrad GEMM with the ReLU gate fused; in a base step the last of them also updates the parameters.
#include "kernels.h"
#include "model.h"

namespace sama {
namespace {

class MlpModel : public Model {
 public:
  MlpModel(const sama_config& cfg, const std::vector<TensorInfo>& layout) {
    L_ = cfg.n_dims - 1;
    for (int i = 0; i < cfg.n_dims; ++i) dims_.push_back(cfg.dims[i]);
    for (int l = 0; l < L_; ++l) { woff_.push_back(layout[l].offset); boff_.push_back(layout[L_ + l].offset); }
  }
  void plan(BumpAlloc& ws, int max_b) override {
    act_.assign(L_ + 1, nullptr);
    int wmax = 0;
    for (int l = 1; l < L_; ++l) { act_[l] = ws.take<float>((size_t)2 * max_b * dims_[l]);   /* the + and the - pass run side by side */ wmax = dims_[l] > wmax ? dims_[l] : wmax; }
    d_[0] = ws.take<float>((size_t)max_b * (wmax > 0 ? wmax : 1));
    d_[1] = ws.take<float>((size_t)max_b * (wmax > 0 ? wmax : 1));
  }
  int n_classes() const override { return dims_[L_]; }

  // The hidden layers of one pass, or of the + and the - pass of Eq. 5 on the same batch side by side in each launch (rows
  // of pass k at k * b.n); the last layer is the head, which the per-sample stage evaluates.
  HeadView run_forward(hipStream_t st, const PassWeights* w, int nw, const sama_batch& b) {
    for (int l = 0; l + 1 < L_; ++l) {
      GemmF32Args g[2];
      for (int k = 0; k < nw; ++k) {
        g[k] = GemmF32Args{};
        const int64_t row = (int64_t)k * b.n;
        g[k].A = l == 0 ? (const float*)b.x : act_[l] + row * dims_[l]; g[k].sa_i = dims_[l]; g[k].sa_k = 1;
        g[k].B = w[k].theta + woff_[l]; g[k].sb_k = 1; g[k].sb_j = dims_[l];
        g[k].bias = w[k].theta + boff_[l];
        if (w[k].sign != 0.f) { g[k].Bv = w[k].vdir + woff_[l]; g[k].beps = w[k].eps_ptr; g[k].bsign = w[k].sign; g[k].bias_v = w[k].vdir + boff_[l]; }
        g[k].C = act_[l + 1] + row * dims_[l + 1]; g[k].ldc = dims_[l + 1];
        g[k].M = b.n; g[k].N = dims_[l + 1]; g[k].K = dims_[l];
        g[k].relu = 1;
      }
      launch_gemm_f32_batch(st, g, nw);
    }
    const int K = dims_[L_ - 1];
    HeadView h{};
    h.x = L_ == 1 ? (const float*)b.x : act_[L_ - 1]; h.stride = K; h.pass_stride = L_ == 1 ? 0 : (int64_t)b.n * K; h.k = K;
    h.pv = ParamView{w[0].theta, w[0].vdir, w[0].eps_ptr, w[0].sign, 0};
    h.w_off = woff_[L_ - 1]; h.b_off = boff_[L_ - 1];
    return h;
  }
  HeadView forward(hipStream_t st, const PassWeights& w, const sama_batch& b, bool /*keep*/, const MlmBatch*) override {
    return run_forward(st, &w, 1, b);
  }
  HeadView forward_pair(hipStream_t st, const PassWeights& wp, const PassWeights& wm, const sama_batch& b, const MlmBatch*) override {
    const PassWeights w[2] = {wp, wm};
    return run_forward(st, w, 2, b);
  }

  void backward(hipStream_t st, const PassWeights& w, const sama_batch& b, const float* dlogits, float* grad) override {
    const float* d = dlogits;
    for (int l = L_ - 1; l >= 0; --l) {
      GemmF32Args g[2] = {};  // dW[d_{l+1} x d_l] = d^T . in, and the bias gradient = row sums of d^T
      g[0].A = d; g[0].sa_i = 1; g[0].sa_k = dims_[l + 1];
      g[0].B = (l == 0) ? (const float*)b.x : act_[l]; g[0].sb_k = dims_[l]; g[0].sb_j = 1;
      g[0].C = grad + woff_[l]; g[0].ldc = dims_[l];
      g[0].M = dims_[l + 1]; g[0].N = dims_[l]; g[0].K = b.n;
      g[0].rowsum = grad + boff_[l];
      if (l > 0) {            // dprev[B x d_l] = (d . W_l) * (act_l > 0)
        g[1].A = d; g[1].sa_i = dims_[l + 1]; g[1].sa_k = 1;
        g[1].B = w.theta + woff_[l]; g[1].sb_k = dims_[l]; g[1].sb_j = 1;
        g[1].C = d_[l & 1]; g[1].ldc = dims_[l];
        g[1].M = b.n; g[1].N = dims_[l]; g[1].K = dims_[l + 1];
        g[1].gate = act_[l];
      }
      // The first layer's launch, the last one, reads no weights: with it goes the update of all of them, or of those it computes, which a
      // launch of its own would wait for.
      BaseUpdate u{};
      if (l == 0 && sink_ != nullptr && sink_->take_over(&u, (int64_t)g[0].M * g[0].N, boff_[0])) launch_gemm_f32_update(st, g[0], u);
      else launch_gemm_f32_batch(st, g, l > 0 ? 2 : 1);
      d = d_[l & 1];
    }
  }

 private:
  int L_;
  std::vector<int> dims_;
  std::vector<int64_t> woff_, boff_;
  std::vector<float*> act_;
  float* d_[2] = {nullptr, nullptr};
};
}  // namespace

Model* make_mlp(const sama_config& cfg, const std::vector<TensorInfo>& layout) { return new MlpModel(cfg, layout); }

}  // namespace sama
