// Classifier head and per-sample stage between the model's last hidden state and its backward pass (Sec. 4.1):
//   z_i = W x_i + b
//   l_i = logsumexp(z_i) - z_i[y_i];  w_i = sigmoid(W2 . relu(W1 l_i + b1) + b2);  B_eff = sum mask
//   BASE: coef_i = mask_i w_i / B_eff   META: coef_i = mask_i / B_eff   -> dz_i = coef_i (softmax(z_i) - e_{y_i})
//   GLAM: dL_base/dlambda = (1/B_eff) sum_i mask_i l_i dw(l_i; lambda)/dlambda   (weight-net backward only)
// With label correction (Sec. 4.1; Hc > 0) the BASE and GLAM modes compare the prediction with the corrected soft label
//   c_i = softmax(kappa e_{y_i} + W2c relu(W1c [e_{y_i}, softmax(z_i)] + b1c) + b2c),  l_i = -sum_k c_ik log softmax(z_i)_k,
//   BASE: dz_i = coef_i (softmax(z_i) - c_i)
//   GLAM: additionally d/dlambda_c = sum_i coef_i sum_k (-log p_ik) dc_ik/dlambda_c  (corrector backward; its inputs are constants)
// and the finite-difference combine + Adam step on lambda (Eq. 5, Table 4).
//
// Everything here is small and latency-bound, a launch of its own costing as much as most of these steps.  The logits of a
// workgroup's 32 samples come from the fp32 matrix cores, the eight waves splitting the contraction.  Sixteen lanes share a sample (classes, weight-net and corrector hidden
// units are split between them and joined across the lanes), a workgroup holds 32 samples at a time, and a batch is spread over
// up to STAGE_MAX_BLOCKS workgroups.  What a mode sums over the batch (the loss, the lambda-gradient) leaves each
// workgroup as a partial; the workgroup that finishes last adds the partials in workgroup order, so results do not depend on
// timing.  The + and the - pass of Eq. 5 are one launch (grid.y), and the last workgroup of that launch also combines them
// and updates lambda.  Arithmetic is in double so that the +-eps difference of Eq. 5 is not lost to rounding.
//
// What it costs is one chain of steps, each executed once: 0.5 us for a trip to memory that nothing runs beside, 0.5 to 1.5 us for
// an exponential or logarithm in double with its code coming in, 2 us for the hand-over to the last workgroup.  So loads are
// wide and without branches, what later steps need is requested before the head's operands, the corrector is converted to double
// once, a lane works on four hidden units at a time, and the last workgroup requests all partials and the state of lambda at once.
// us per launch (start of a kernel to that of the next), first with a load or a shuffle through LDS wherever one was needed, then as
// it is: logistic regression, 512 samples, base step 10.6 -> 6.9, both passes and the update 17.9 -> 10.5; 128 samples of 256
// features, H = 100 10.0 -> 8.3 and 15.1 -> 13.5; label correction, 203 samples, Hc = 64 19.8 -> 12.5 and 44.5 -> 29.9; an encoder's
// text alone 13.4 -> 7.0, 32 texts 17.6 -> 11.6 and 27.4 -> 18.5.
#include "common.h"
#include "kernels.h"
#include "mfma_f32.h"

namespace sama {
namespace {

constexpr int ST_THREADS = 512, ST_LANES = 16, ST_SAMPLES = ST_THREADS / ST_LANES;   // samples per trip
constexpr int ST_MAX_RUN = (MAX_BATCH + STAGE_MAX_BLOCKS - 1) / STAGE_MAX_BLOCKS < ST_SAMPLES ? ST_SAMPLES : (MAX_BATCH + STAGE_MAX_BLOCKS - 1) / STAGE_MAX_BLOCKS;
constexpr int MAX_CORR = MAX_CORR_HIDDEN * 2 * MAX_CORR_CLASSES + MAX_CORR_HIDDEN + MAX_CORR_CLASSES * MAX_CORR_HIDDEN + MAX_CORR_CLASSES;
constexpr int CQ = 4;                        // classes per lane: up to 64 over sixteen lanes
static_assert(ST_MAX_RUN == ST_SAMPLES && ST_SAMPLES == 32 && ST_THREADS == 64 * FWAVES, "one trip of 2 x 16 samples per workgroup");

constexpr int HEAD_LDS = 8192;   // floats of LDS for the head
static_assert(FWAVES * 32 * 17 <= HEAD_LDS, "partial tiles");
// s_z[i][c] = logits of samples i_begin + i (two 16-row MFMA tiles), c < C: wave w takes every FWAVES-th chunk of the
// contraction, requests four chunks at a time, and the partial tiles are added in wave order.
__device__ __forceinline__ void head_logits(const HeadView& h, int pass, int i_begin, int n_own, int C, float* __restrict__ red, double* __restrict__ s_z) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 15, q = lane >> 4;
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  const float s = pass == 0 ? h.pv.scale() : -h.pv.scale();
  // rows and classes beyond the end are clamped: their products are not read
  const float* const x0 = h.x + pass * h.pass_stride + (int64_t)(i_begin + min(r, n_own - 1)) * h.stride;
  const float* const x1 = h.x + pass * h.pass_stride + (int64_t)(i_begin + min(16 + r, n_own - 1)) * h.stride;
  constexpr int DEPTH = 4, STEP = FWAVES * FCH;
  const int nfull = h.k / FCH, n = nfull > wave ? (nfull - wave + FWAVES - 1) / FWAVES : 0;
  const bool tail = h.k % FCH != 0 && nfull % FWAVES == wave;
  for (int c0 = 0; c0 < C; c0 += 16) {
    const int own_c = c0 + (threadIdx.x & 15);
    const float bias = h.pv.at(h.b_off + min(own_c, C - 1), s);
    const int64_t wrow = h.w_off + (int64_t)min(c0 + r, C - 1) * h.k;
    const float* const W = h.pv.theta + wrow;
    const float* const Wv = h.pv.vdir + wrow;
    float4v acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    auto multiply = [&](const float4v& a0, const float4v& a1, const float4v& bw, const float4v& bp) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float b = s != 0.f ? fmaf(s, bp[c], bw[c]) : bw[c];
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[c], b, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[c], b, acc[1], 0, 0, 0);
      }
    };
    for (int i = 0; i < n; i += DEPTH) {
      float4v a0[DEPTH], a1[DEPTH], bw[DEPTH], bp[DEPTH];
#pragma unroll
      for (int u = 0; u < DEPTH; ++u) {
        if (i + u >= n) break;
        const int k = wave * FCH + (i + u) * STEP + 4 * q;
        a0[u] = *reinterpret_cast<const f4u*>(x0 + k);
        a1[u] = *reinterpret_cast<const f4u*>(x1 + k);
        bw[u] = *reinterpret_cast<const f4u*>(W + k);
        bp[u] = s != 0.f ? *reinterpret_cast<const f4u*>(Wv + k) : bw[u];
      }
#pragma unroll
      for (int u = 0; u < DEPTH; ++u)
        if (i + u < n) multiply(a0[u], a1[u], bw[u], bp[u]);
    }
    if (tail) {
      float4v t[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int k = nfull * FCH + 4 * q + c, kk = min(k, h.k - 1);
        t[0][c] = k < h.k ? x0[kk] : 0.f; t[1][c] = k < h.k ? x1[kk] : 0.f;
        t[2][c] = k < h.k ? W[kk] : 0.f; t[3][c] = k < h.k && s != 0.f ? Wv[kk] : 0.f;
      }
      multiply(t[0], t[1], t[2], t[3]);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[(wave * 32 + 16 * t + 4 * q + e) * 17 + r] = acc[t][e];
    __syncthreads();
    {
      const int i = threadIdx.x >> 4, c = threadIdx.x & 15;   // 512 threads: one of the 32 x 16 outputs each
      if (own_c < C) {
        double z = (double)bias;
#pragma unroll
        for (int w = 0; w < FWAVES; ++w) z += (double)red[(w * 32 + i) * 17 + c];
        s_z[i * 64 + own_c] = z;
      }
    }
    if (c0 + 16 < C) __syncthreads();
  }
}

// The same with a wave per sample: 64 strided partial sums in fp32, joined in a fixed tree.  The losses of the two passes of
// Eq. 5 differ in their last digits only, and a deep model's gradients follow those of its logits, so what the
// encoder's logits are rounded to is kept independent of how a workgroup's tiles split the features.
// W, as the pass sees it, comes through LDS, CU classes and 1024 features at a time, and a wave has that many features of its
// samples in registers: one trip to memory.  What is beyond the features or classes is zero.
template <int SU>
__device__ __forceinline__ void head_dots(const HeadView& h, int pass, int i_begin, int n_own, int C, float* __restrict__ s_w, double* __restrict__ s_z) {
  constexpr int CU = 8, KB = HEAD_LDS / CU, KT = KB / 64, WT = KB / ST_THREADS;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float s = pass == 0 ? h.pv.scale() : -h.pv.scale();
  const float* x[SU];   // sample wave + FWAVES u of the workgroup's is this wave's u-th
#pragma unroll
  for (int u = 0; u < SU; ++u) {
    const int i = i_begin + min(wave + FWAVES * u, n_own - 1);
    x[u] = h.x + pass * h.pass_stride + (h.start != nullptr ? (int64_t)h.start[i] * h.k : (int64_t)i * h.stride);
  }
  for (int c0 = 0; c0 < C; c0 += CU) {
    const float bias = h.pv.at(h.b_off + min(c0 + (lane & (CU - 1)), C - 1), s);   // of class c0 + lane
    float acc[SU][CU] = {};
    for (int k0 = 0; k0 < h.k; k0 += KB) {
      const int nk = min(KB, h.k - k0);
      float xk[SU][KT], w[CU][WT];
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int u = 0; u < SU; ++u) xk[u][t] = 64 * t + lane < nk ? x[u][k0 + 64 * t + lane] : 0.f;
#pragma unroll
      for (int c = 0; c < CU; ++c)
#pragma unroll
        for (int t = 0; t < WT; ++t) {
          const int k = t * ST_THREADS + tid;
          w[c][t] = c0 + c < C && k < nk ? h.pv.at(h.w_off + (int64_t)(c0 + c) * h.k + k0 + k, s) : 0.f;
        }
      if (c0 + k0 > 0) __syncthreads();
#pragma unroll
      for (int c = 0; c < CU; ++c)
#pragma unroll
        for (int t = 0; t < WT; ++t) s_w[c * KB + t * ST_THREADS + tid] = w[c][t];
      __syncthreads();
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int c = 0; c < CU; ++c) {
          const float w = s_w[c * KB + 64 * t + lane];
#pragma unroll
          for (int u = 0; u < SU; ++u) acc[u][c] = fmaf(xk[u][t], w, acc[u][c]);
        }
    }
#pragma unroll
    for (int c = 0; c < CU; ++c) {
      const float b = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(bias), c));
#pragma unroll
      for (int u = 0; u < SU; ++u) {
        const float z = wave_sum(acc[u][c]);
        if (lane == 0 && wave + FWAVES * u < n_own && c0 + c < C) s_z[(wave + FWAVES * u) * 64 + c0 + c] = (double)(z + b);
      }
    }
  }
}

// every lane of a group of sixteen gets the sum / maximum over the group
__device__ __forceinline__ double sum16(double x) { return join_group(x, [](double a, double b) { return a + b; }); }
__device__ __forceinline__ double max16(double x) { return join_group(x, [](double a, double b) { return fmax(a, b); }); }
// sum over the workgroup in a fixed order, for every thread; `red` holds ST_THREADS / 64 values
__device__ __forceinline__ double block_sum_d(double x, double* red) {
  x = wave_sum(x);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < ST_THREADS / 64; ++k) s += red[k];
  return s;
}

// h = -(glam+ - glam-) / (2 eps); then (optionally) Adam on lambda.  A raised status word (counters[2]) or a
// hypergradient with a non-finite component zeroes h and skips the update; the latter raises the status word itself.
// glam+ / glam- are the sums of the workgroups' partials in order.  A load of one takes a microsecond: a thread requests those of
// EL components and KC workgroups at once, and everything else it will need beside them.  One chunk of EL * ST_THREADS
// components stays in registers from the sums to the update; where there are more, the sums are read back.
template <int EL, int KC>
__device__ __forceinline__ void meta_update(const MetaUpdateArgs& a, const double* part, int nblk) {
  const int tid = threadIdx.x;
  const float eps = a.scalars[0];
  const int64_t t = a.counters[1] + 1;
  bool skip = (a.counters[2] != 0) || !(eps > 0.f);
  const bool one = a.nl <= EL * ST_THREADS;
  int bad = 0;
  double gp[EL], gm[EL], c1 = 0.0, c2 = 0.0;
  float m0[EL], v0[EL], l0[EL];
  auto state = [&](int i0) {
#pragma unroll
    for (int e = 0; e < EL; ++e) {
      const int i = i0 + e * ST_THREADS;
      m0[e] = v0[e] = l0[e] = 0.f;
      if (a.do_update && i < a.nl) { m0[e] = a.meta_m[i]; v0[e] = a.meta_v[i]; l0[e] = a.lambda[i]; }
    }
  };
  for (int i0 = tid; i0 < a.nl; i0 += EL * ST_THREADS) {
    if (one) state(i0);
#pragma unroll
    for (int e = 0; e < EL; ++e) gp[e] = gm[e] = 0.0;
    for (int k0 = 0; k0 < nblk; k0 += KC) {
      double p[KC][EL], m[KC][EL];
#pragma unroll
      for (int u = 0; u < KC; ++u)
#pragma unroll
        for (int e = 0; e < EL; ++e) {
          const bool there = k0 + u < nblk && i0 + e * ST_THREADS < a.nl;
          const double* q = part + (int64_t)(k0 + u) * a.nl + i0 + e * ST_THREADS;
          p[u][e] = there ? collect(q) : 0.0;
          m[u][e] = there ? collect(q + (int64_t)nblk * a.nl) : 0.0;
        }
      if (k0 == 0 && i0 == tid) {   // beside the first loads
        c1 = 1.0 / (1.0 - ipow((double)a.beta1, t));
        c2 = 1.0 / sqrt(1.0 - ipow((double)a.beta2, t));
      }
#pragma unroll
      for (int u = 0; u < KC; ++u)
#pragma unroll
        for (int e = 0; e < EL; ++e) { gp[e] += p[u][e]; gm[e] += m[u][e]; }
    }
#pragma unroll
    for (int e = 0; e < EL; ++e) {
      const int i = i0 + e * ST_THREADS;
      if (i >= a.nl) break;
      a.glam_p[i] = gp[e]; a.glam_m[i] = gm[e];
      if (!skip) {
        const double h = -(gp[e] - gm[e]) / (2.0 * (double)eps);
        if (!(fabs(h) <= 3.0e38)) bad = 1;   // NaN, infinite, or beyond what the fp32 outputs hold
      }
    }
  }
  if (__syncthreads_or(bad)) {   // every thread has read counters[2] above
    skip = true;
    if (tid == 0) a.counters[2] = 1;
  }
  for (int i0 = tid; i0 < a.nl; i0 += EL * ST_THREADS) {
    if (!one) {
      state(i0);
#pragma unroll
      for (int e = 0; e < EL; ++e) {   // written by this thread above
        const int i = i0 + e * ST_THREADS;
        gp[e] = i < a.nl ? a.glam_p[i] : 0.0; gm[e] = i < a.nl ? a.glam_m[i] : 0.0;
      }
    }
#pragma unroll
    for (int e = 0; e < EL; ++e) {
      const int i = i0 + e * ST_THREADS;
      if (i >= a.nl) break;
      const double h = skip ? 0.0 : -(gp[e] - gm[e]) / (2.0 * (double)eps);
      a.hypergrad[i] = (float)h;
      if (a.hypergrad_user) a.hypergrad_user[i] = (float)h;
      a.glam_p_f32[i] = (float)gp[e];
      a.glam_m_f32[i] = (float)gm[e];
      if (a.do_update && !skip) {
        const double m = (double)a.beta1 * m0[e] + (1.0 - (double)a.beta1) * h;
        const double v = (double)a.beta2 * v0[e] + (1.0 - (double)a.beta2) * h * h;
        a.meta_m[i] = (float)m;
        a.meta_v[i] = (float)v;
        a.lambda[i] = (float)((double)l0[e] - (double)a.lr * c1 * m / (c2 * sqrt(v) + (double)a.eps));
      }
    }
  }
  if (tid == 0) {
    if (a.eps_user) *a.eps_user = skip ? 0.f : eps;
    if (a.do_update && !skip) a.counters[1] = t;
  }
}

// CORR: label correction compiled in (its arrays make up most of the LDS)
template <bool CORR>
__global__ __launch_bounds__(ST_THREADS) void k_sample_stage(SampleStageArgs a, int run, int nblk) {
  __shared__ double s_l[ST_MAX_RUN];    // l_i of this workgroup's samples
  __shared__ double s_dz[ST_MAX_RUN];   // per-sample dL/dz of the weight net (GLAM)
  __shared__ float s_cnt[ST_MAX_RUN];   // sequence mode: positions per sequence
  __shared__ float s_lam[3 * MAX_WNET_HIDDEN + 1];
  __shared__ double red[ST_THREADS / 64];
  __shared__ int s_last;
  __shared__ double s_a[ST_SAMPLES * MAX_CORR_HIDDEN];   // relu(a_ij); before that, the head's
  static_assert(sizeof(s_a) >= HEAD_LDS * sizeof(float), "the head's share");
  float* const s_head = reinterpret_cast<float*>(s_a);
  __shared__ double s_z[ST_SAMPLES * 64];
  __shared__ double s_lc[CORR ? MAX_CORR : 1];           // the corrector, converted once
  __shared__ double s_t[CORR ? ST_SAMPLES * MAX_CORR_HIDDEN : 1];   // dL/da_ij
  __shared__ double s_p[CORR ? ST_SAMPLES * MAX_CORR_CLASSES : 1], s_ds[CORR ? ST_SAMPLES * MAX_CORR_CLASSES : 1];
  __shared__ int s_y[CORR ? ST_SAMPLES : 1];
  const int tid = threadIdx.x, lane = tid & (ST_LANES - 1), grp = tid / ST_LANES, H = a.H, B = a.B, C = a.C;
  if ((int)blockIdx.x == nblk) {   // the step-dependent scalars of the base solver (the update runs much later)
    if (tid == 0) step_scalars(a.step);
    return;
  }
  const int pass = blockIdx.y, i_begin = blockIdx.x * run, i_end = min(B, i_begin + run), n_own = i_end - i_begin;
  const bool seq_mode = a.pos_loss != nullptr;          // per-sequence losses from masked-token positions
  const int Hc = CORR ? a.Hc : 0;
  const float* pos_loss = a.pos_loss + pass * a.pos_pass_stride;
  float* losses = pass == (int)gridDim.y - 1 ? a.losses : nullptr;   // of the most recent pass

  // What the samples' steps will need is requested before the head's operands, and put in place behind the head.
  const bool weighs = a.mode != STAGE_META;             // the clean batch has unit weights
  float lam[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) lam[u] = weighs && tid + u * ST_THREADS < 3 * H + 1 ? a.lambda[tid + u * ST_THREADS] : 0.f;
  static_assert(3 * MAX_WNET_HIDDEN + 1 <= 2 * ST_THREADS, "two parameters a thread");
  const int i_own = min(i_begin + grp, i_end - 1);      // one trip: ST_SAMPLES samples at most
  const int y_own = seq_mode ? 0 : a.y[i_own];
  const bool masked_out = a.mask != nullptr && a.mask[i_own] == 0;
  const int nlc = Hc > 0 ? Hc * 2 * C + Hc + C * Hc + C : 0;
  if (CORR)
    for (int i = tid; i < nlc; i += 4 * ST_THREADS) {
      float t[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) t[u] = i + u * ST_THREADS < nlc ? a.lambda[3 * H + 1 + i + u * ST_THREADS] : 0.f;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i + u * ST_THREADS < nlc) s_lc[i + u * ST_THREADS] = (double)t[u];
    }
  double beff = (double)B;
  if (a.mask != nullptr) {
    double cnt = 0.0;
    for (int i = tid; i < B; i += ST_THREADS) cnt += a.mask[i] != 0 ? 1.0 : 0.0;
    beff = block_sum_d(cnt, red);
  }
  const double inv_beff = beff > 0.0 ? 1.0 / beff : 0.0;
  if (!seq_mode) {
    if (!a.head.dots) head_logits(a.head, pass, i_begin, n_own, C, s_head, s_z);
    else if (n_own <= FWAVES) head_dots<1>(a.head, pass, i_begin, n_own, C, s_head, s_z);
    else head_dots<ST_SAMPLES / FWAVES>(a.head, pass, i_begin, n_own, C, s_head, s_z);
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (tid + u * ST_THREADS < 3 * H + 1) s_lam[tid + u * ST_THREADS] = lam[u];
  __syncthreads();
  const float* W1 = s_lam; const float* b1 = s_lam + H; const float* W2 = s_lam + 2 * H;
  const double b2 = (double)s_lam[3 * H];
  const double* W1c = s_lc; const double* b1c = s_lc + Hc * 2 * C; const double* W2c = b1c + Hc; const double* b2c = W2c + C * Hc;

  if (seq_mode) {
    // wave w takes sequences w, w + waves, ...: its lanes stride over the positions (coalesced), keep the matching losses,
    // and a tree over the lanes adds the 64 partial sums in a fixed order
    for (int i = tid >> 6; i < n_own; i += ST_THREADS / 64) {
      double acc = 0.0, n_i = 0.0;
      for (int j = tid & 63; j < a.n_pos; j += 64) {
        int r = a.pos_row[j];
        r = r < 0 ? 0 : (r >= B * a.S ? B * a.S - 1 : r);
        if (r / a.S == i_begin + i) { acc += (double)pos_loss[j]; n_i += 1.0; }
      }
      acc = wave_sum(acc); n_i = wave_sum(n_i);
      if ((tid & 63) == 0) { s_l[i] = n_i > 0.0 ? acc / n_i : 0.0; s_cnt[i] = (float)n_i; }
    }
    __syncthreads();
  }
  double lsum = 0.0;
  constexpr int PAIRS = CORR ? (MAX_CORR_HIDDEN * MAX_CORR_CLASSES + ST_THREADS - 1) / ST_THREADS : 1;
  double gW2[PAIRS], gWp[PAIRS], gWy[PAIRS], gb2[PAIRS], gb1 = 0.0;   // corrector backward: thread owns (hidden unit, class) pairs
  const int pair_step = CORR ? min(ST_THREADS / Hc, C) : 1, pair_j = CORR ? tid % Hc : 0, pair_k = CORR ? tid / Hc : 0;
#pragma unroll
  for (int u = 0; u < PAIRS; ++u) gW2[u] = gWp[u] = gWy[u] = gb2[u] = 0.0;

  static_assert(ST_MAX_RUN <= ST_SAMPLES, "a sample for each group of lanes");
  {                                                       // every thread takes part (barriers with CORR)
    const int i = i_begin + grp;
    const bool live = i < i_end;
    const int ic = i_own;
    const double mk = live && !masked_out ? 1.0 : 0.0;
    double l, lse = 0.0, zc[CQ] = {0.0, 0.0, 0.0, 0.0};
    int yi = 0;
    double cs = 0.0;                                      // corrected soft label of class `lane` (Hc > 0)
    if (seq_mode) {
      l = s_l[ic - i_begin];
    } else {
      const double* z = s_z + (ic - i_begin) * 64;
      yi = min(max(y_own, 0), C - 1);   // labels outside [0, C) are clamped
#pragma unroll
      for (int q = 0; q < CQ; ++q) zc[q] = lane + ST_LANES * q < C ? z[lane + ST_LANES * q] : -1.0e300;
      const double zy = z[yi];
      if (a.logits != nullptr && live) {
#pragma unroll
        for (int q = 0; q < CQ; ++q)
          if (lane + ST_LANES * q < C) a.logits[(int64_t)i * C + lane + ST_LANES * q] = (float)z[lane + ST_LANES * q];
      }
      const double zmax = max16(fmax(fmax(zc[0], zc[1]), fmax(zc[2], zc[3])));
      double se = 0.0;
#pragma unroll
      for (int q = 0; q < CQ; ++q)
        if (lane + ST_LANES * q < C) se += exp(zc[q] - zmax);
      lse = log(sum16(se)) + zmax;
      if (CORR) {
        const bool own = lane < C;                        // C <= 16: lane k holds class k
        const double lp = zc[0] - lse, p = own ? exp(lp) : 0.0;
        s_p[grp * MAX_CORR_CLASSES + lane] = p;
        if (lane == 0) s_y[grp] = yi;
        __syncthreads();
        // A lane takes four hidden units and four classes at a time, so that its LDS reads and chains of additions overlap; units and
        // classes beyond the end add zeros.
        double sc[MAX_CORR_CLASSES];
#pragma unroll
        for (int k = 0; k < MAX_CORR_CLASSES; ++k) sc[k] = 0.0;
        for (int j0 = lane; j0 - lane < Hc; j0 += 4 * ST_LANES) {
          int jj[4];
          double aj[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            jj[u] = min(j0 + u * ST_LANES, Hc - 1);
            aj[u] = b1c[jj[u]] + W1c[jj[u] * 2 * C + yi];
          }
          for (int k0 = 0; k0 < C; k0 += 4) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int k = min(k0 + v, C - 1);
              const double pk = k0 + v < C ? s_p[grp * MAX_CORR_CLASSES + k] : 0.0;
#pragma unroll
              for (int u = 0; u < 4; ++u) aj[u] += (k0 + v < C ? W1c[jj[u] * 2 * C + C + k] : 0.0) * pk;
            }
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const bool there = j0 + u * ST_LANES < Hc;
            aj[u] = there && aj[u] > 0.0 ? aj[u] : 0.0;
            if (there) s_a[grp * MAX_CORR_HIDDEN + jj[u]] = aj[u];
          }
#pragma unroll
          for (int k0 = 0; k0 < MAX_CORR_CLASSES; k0 += 4) {
            if (k0 >= C) break;
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
              for (int u = 0; u < 4; ++u) sc[k0 + v] += (j0 + u * ST_LANES < Hc ? W2c[min(k0 + v, C - 1) * Hc + jj[u]] : 0.0) * aj[u];
          }
        }
        double s_own = 0.0;
#pragma unroll
        for (int k0 = 0; k0 < MAX_CORR_CLASSES; k0 += 4) {
          if (k0 >= C) break;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const double tot = sum16(sc[k0 + v]);
            if (k0 + v == lane && own) s_own = tot + b2c[lane] + (lane == yi ? (double)a.kappa : 0.0);
          }
        }
        const double smax = max16(own ? s_own : -1.0e300);
        cs = own ? exp(s_own - smax) : 0.0;
        cs /= sum16(cs);
        l = -sum16(own ? cs * lp : 0.0);
      } else {
        l = lse - zy;
      }
    }
    if (losses != nullptr && live && lane == 0) losses[i] = (float)l;
    double w = 1.0;
    if (a.mode != STAGE_META) {
      double zz = 0.0;
      for (int h = lane; h < H; h += ST_LANES) zz += (double)W2[h] * fmax((double)W1[h] * l + (double)b1[h], 0.0);
      w = 1.0 / (1.0 + exp(-(sum16(zz) + b2)));
    }
    if (a.weights != nullptr && live && lane == 0) a.weights[i] = (float)w;
    if (a.mode == STAGE_EVAL) return;
    const double coef = mk * w * inv_beff;
    if (a.mode == STAGE_GLAM) {
      if (live && lane == 0) { s_l[i - i_begin] = l; s_dz[i - i_begin] = w * (1.0 - w) * l * mk * inv_beff; }
      if (CORR) {
        // ds_ik = c_ik (dc_ik - sum_k' c_ik' dc_ik'), dc_ik = -coef_i log p_ik;  t_ij = [a_ij > 0] sum_k W2c[k][j] ds_ik
        const double dc = lane < C ? -coef * (zc[0] - lse) : 0.0;
        const double dot = sum16(cs * dc), ds = cs * (dc - dot);
        s_ds[grp * MAX_CORR_CLASSES + lane] = ds;
        __syncthreads();
        for (int j0 = lane; j0 - lane < Hc; j0 += 4 * ST_LANES) {
          int jj[4];
          double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int u = 0; u < 4; ++u) jj[u] = min(j0 + u * ST_LANES, Hc - 1);
          for (int k0 = 0; k0 < C; k0 += 4) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int k = min(k0 + v, C - 1);
              const double dk = k0 + v < C ? s_ds[grp * MAX_CORR_CLASSES + k] : 0.0;
#pragma unroll
              for (int u = 0; u < 4; ++u) t[u] += (k0 + v < C ? W2c[k * Hc + jj[u]] : 0.0) * dk;
            }
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (j0 + u * ST_LANES < Hc) s_t[grp * MAX_CORR_HIDDEN + jj[u]] = s_a[grp * MAX_CORR_HIDDEN + jj[u]] > 0.0 ? t[u] : 0.0;
        }
        __syncthreads();
        // thread: hidden unit pair_j, classes pair_k, pair_k + pair_step, ...; it shares what it reads of the unit between them
        if (pair_k < pair_step) {
          const int last = C - 1;
#pragma unroll 4
          for (int s = 0; s < n_own; ++s) {
            const double aj = s_a[s * MAX_CORR_HIDDEN + pair_j], t = s_t[s * MAX_CORR_HIDDEN + pair_j];
            const int ys = s_y[s];
#pragma unroll
            for (int u = 0; u < PAIRS; ++u) {
              if (u * pair_step >= C) break;   // the same for every thread
              const int k = min(pair_k + u * pair_step, last);
              const double d = s_ds[s * MAX_CORR_CLASSES + k];
              gW2[u] += d * aj;
              gWp[u] += t * s_p[s * MAX_CORR_CLASSES + k];
              gWy[u] += ys == k ? t : 0.0;
              gb2[u] += d;      // kept for pair_j == 0
            }
            gb1 += t;           // kept for pair_k == 0
          }
        }
      }
    } else if (seq_mode) {
      if (lane == 0) {
        if (live) s_dz[i - i_begin] = coef;
        lsum += coef * l;
      }
    } else {
      if (lane == 0) lsum += coef * l;
#pragma unroll
      for (int q = 0; q < CQ; ++q) {
        const int c = lane + ST_LANES * q;
        if (live && c < C) {
          const double target = CORR ? cs : (c == yi ? 1.0 : 0.0);
          a.dlogits[(int64_t)i * C + c] = (float)(coef * (exp(zc[q] - lse) - target));
        }
      }
    }
  }

  const int total = nblk * gridDim.y;      // workgroups whose partials make the result
  if (a.mode != STAGE_GLAM) {
    if (seq_mode) {
      __syncthreads();
      for (int j = tid; j < a.n_pos; j += ST_THREADS) {
        int r = a.pos_row[j];
        r = r < 0 ? 0 : (r >= B * a.S ? B * a.S - 1 : r);
        const int i = r / a.S;
        if (i >= i_begin && i < i_end) a.pos_coef[j] = (float)(s_dz[i - i_begin] / (double)s_cnt[i - i_begin]);   // s_cnt >= 1: position j itself
      }
    }
    double L = block_sum_d(lsum, red);
    if (total > 1) {
      if (tid == 0) publish(a.part + blockIdx.x, L);
      if (!last_block(a.ticket, total, &s_last)) return;
      static_assert(STAGE_MAX_BLOCKS <= 64, "a partial per lane");
      if (tid < 64) L = wave_sum(tid < nblk ? collect(a.part + tid) : 0.0);
    }
    if (tid == 0) {
      if (a.loss_scalar) *a.loss_scalar = seq_mode ? *a.loss_scalar + (float)L : (float)L;
      if (a.loss_user) *a.loss_user = seq_mode ? *a.loss_user + (float)L : (float)L;
    }
    return;
  }
  __syncthreads();
  double* glam = a.part + (int64_t)(pass * nblk + blockIdx.x) * a.mu.nl;
  // weight-net backward: hidden unit h is shared by nch consecutive lanes of a wave (the largest power of two <=
  // ST_THREADS / H, at most 64), each walking a contiguous run of the samples in order; the nch partial sums of a unit
  // are then added pairwise across the lanes (fixed order, no atomics)
  {
    int nch = 1;
    while (2 * nch * H <= ST_THREADS && nch < 64) nch *= 2;
    const int per = (n_own + nch - 1) / nch;
    const int h = tid / nch, c = tid % nch;              // ST_THREADS / nch >= H units in one trip
    double part[3] = {0.0, 0.0, 0.0};                    // dW1, db1, dW2
    if (h < H) {
      const double w1 = W1[h], bb = b1[h], w2 = W2[h];
      const int i1 = (c + 1) * per < n_own ? (c + 1) * per : n_own;
      for (int i = c * per; i < i1; ++i) {
        const double l = s_l[i], dz = s_dz[i];
        const double pre = w1 * l + bb;
        if (pre > 0.0) {
          const double da = dz * w2;
          part[0] += da * l;
          part[1] += da;
          part[2] += dz * pre;
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) part[q] = run_sum(part[q], nch);
    if (h < H && c == 0) { publish(glam + h, part[0]); publish(glam + H + h, part[1]); publish(glam + 2 * H + h, part[2]); }
  }
  double dsum = 0.0;
  for (int i = tid; i < n_own; i += ST_THREADS) dsum += s_dz[i];
  const double db2 = block_sum_d(dsum, red);
  if (tid == 0) publish(glam + 3 * H, db2);
  if (CORR) {
    double* gc = glam + 3 * H + 1;
    const int j = pair_j;
    if (pair_k < pair_step) {
#pragma unroll
      for (int u = 0; u < PAIRS; ++u) {
        const int k = pair_k + u * pair_step;
        if (k >= C) break;
        publish(gc + j * 2 * C + k, gWy[u]);
        publish(gc + j * 2 * C + C + k, gWp[u]);
        publish(gc + Hc * 2 * C + Hc + k * Hc + j, gW2[u]);
        if (j == 0) publish(gc + Hc * 2 * C + Hc + C * Hc + k, gb2[u]);
      }
      if (pair_k == 0) publish(gc + Hc * 2 * C + j, gb1);
    }
  }
  if (!last_block(a.ticket, total, &s_last)) return;
  if (CORR) meta_update<5, 4>(a.mu, a.part, nblk);   // lambda is that of the corrector for the most part
  else meta_update<1, 16>(a.mu, a.part, nblk);
}
}  // namespace

int stage_blocks(int B) {
  const int n = (B + ST_SAMPLES - 1) / ST_SAMPLES;
  return n < STAGE_MAX_BLOCKS ? n : STAGE_MAX_BLOCKS;
}
void launch_sample_stage(hipStream_t st, const SampleStageArgs& a) {
  ProfScope ps(st, F_SAMPLE_STAGE, 0.0);
  const bool corr = a.Hc > 0 && a.mode != STAGE_META && a.pos_loss == nullptr;   // the clean batch keeps its hard labels
  const int run = (a.B + stage_blocks(a.B) - 1) / stage_blocks(a.B), nblk = (a.B + run - 1) / run;
  const dim3 grid(nblk + (a.step.counters != nullptr ? 1 : 0), a.mode == STAGE_GLAM ? 2 : 1);   // a base step's scalars: one workgroup more
  if (corr) launch_kernel(ps, k_sample_stage<true>, grid, ST_THREADS, 0, st, a, run, nblk);
  else launch_kernel(ps, k_sample_stage<false>, grid, ST_THREADS, 0, st, a, run, nblk);
}

}  // namespace sama
