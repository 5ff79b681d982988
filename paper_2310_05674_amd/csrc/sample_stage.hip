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
// units are split between them and joined by shuffles), a workgroup holds 32 samples at a time, and a batch is spread over
// up to STAGE_MAX_BLOCKS workgroups.  What a mode sums over the batch (the loss, the lambda-gradient) leaves each
// workgroup as a partial; the workgroup that finishes last adds the partials in workgroup order, so results do not depend on
// timing.  The + and the - pass of Eq. 5 are one launch (grid.y), and the last workgroup of that launch also combines them
// and updates lambda.  Arithmetic is in double so that the +-eps difference of Eq. 5 is not lost to rounding.
//
// Measured against one workgroup per pass with a lane per sample and launches of their own for the head, the two passes, the
// update of lambda and the step scalars (kernel durations in a trace): label correction with 203 samples, Hc = 64, 10 classes
// 347 -> 21 us (base step) and 2 x 347 + 9 -> 43 us (both passes and the update); scoring 2048 samples 44 + 7 -> 8.5 us;
// reweighting with 128 samples, H = 100: 13 + 8 -> 10 us and 2 x (13 + 8) + 5 -> 15 us.
// Sums across lanes by vector instructions instead of shuffles through LDS, and the other workgroups' partials requested at once
// instead of one or four at a time: a logistic-regression iteration (512 samples, H = 16; three stages) 62.2 -> 55.5 us.
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

// s_z[i][c] = logits of samples i_begin + i (two 16-row MFMA tiles), c < C: wave w takes every FWAVES-th chunk of the
// contraction, requests four chunks at a time, and the partial tiles are added in wave order.  red: FWAVES x 32 x 17.
__device__ void head_logits(const HeadView& h, int pass, int i_begin, int n_own, int C, float* __restrict__ red, double* __restrict__ s_z) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, q = lane >> 4;
  const float* x = h.x + pass * h.pass_stride + i_begin * h.stride;
  const float* W = h.pv.theta + h.w_off;
  const float* Wv = h.pv.vdir + h.w_off;
  const float s = pass == 0 ? h.pv.scale() : -h.pv.scale();
  const bool x_vec = (h.stride & 3) == 0 && ((uintptr_t)x & 15) == 0;
  const bool w_vec = (h.k & 3) == 0 && (((uintptr_t)W | (s != 0.f ? (uintptr_t)Wv : 0)) & 15) == 0;
  constexpr int DEPTH = 4;
  for (int c0 = 0; c0 < C; c0 += 16) {
    float4v acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    for (int kb = wave * FCH; kb < h.k; kb += DEPTH * FWAVES * FCH) {
      float4v av[DEPTH][2], bv[DEPTH], pv[DEPTH];
#pragma unroll
      for (int u = 0; u < DEPTH; ++u) {
        const int k = kb + u * FWAVES * FCH + 4 * q;      // a chunk beyond the end reads as zeros
        av[u][0] = load_k4(x, h.stride, 1, r, n_own, k, h.k, x_vec);
        av[u][1] = load_k4(x, h.stride, 1, 16 + r, n_own, k, h.k, x_vec);
        bv[u] = load_k4(W, h.k, 1, c0 + r, C, k, h.k, w_vec);
        if (s != 0.f) pv[u] = load_k4(Wv, h.k, 1, c0 + r, C, k, h.k, w_vec);
      }
#pragma unroll
      for (int u = 0; u < DEPTH; ++u) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float b = s != 0.f ? fmaf(s, pv[u][c], bv[u][c]) : bv[u][c];
          acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u][0][c], b, acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u][1][c], b, acc[1], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[(wave * 32 + 16 * t + 4 * q + e) * 17 + r] = acc[t][e];
    __syncthreads();
    {
      const int i = threadIdx.x >> 4, c = threadIdx.x & 15;   // 512 threads: one of the 32 x 16 outputs each
      if (c0 + c < C) {
        double z = (double)h.pv.at(h.b_off + c0 + c, s);
#pragma unroll
        for (int w = 0; w < FWAVES; ++w) z += (double)red[(w * 32 + i) * 17 + c];
        s_z[i * 64 + c0 + c] = z;
      }
    }
    __syncthreads();
  }
}

// The same with a wave per sample: 64 strided partial sums in fp32, joined by a shuffle tree.  The losses of the two passes of
// Eq. 5 differ in their last digits only, and a deep model's gradients follow those of its logits, so what the
// encoder's logits are rounded to is kept independent of how a workgroup's tiles split the features.
// Up to four samples of a wave and four classes share each element of W that is read.
template <bool PERTURBED>
__device__ void head_dots(const HeadView& h, int pass, int i_begin, int n_own, int C, double* __restrict__ s_z) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float s = pass == 0 ? h.pv.scale() : -h.pv.scale();
  constexpr int CU = 4, SU = ST_SAMPLES / FWAVES;   // sample wave + FWAVES u of the workgroup's is this wave's u-th
  const float* x[SU];
#pragma unroll
  for (int u = 0; u < SU; ++u) {
    const int i = i_begin + min(wave + FWAVES * u, n_own - 1);
    x[u] = h.x + pass * h.pass_stride + (h.start != nullptr ? (int64_t)h.start[i] * h.k : (int64_t)i * h.stride);
  }
  if (wave < n_own) {
    for (int c0 = 0; c0 < C; c0 += CU) {
      float acc[SU][CU] = {};
#pragma unroll 8
      for (int k = lane; k < h.k; k += 64) {
        float w[CU], xk[SU];
#pragma unroll
        for (int c = 0; c < CU; ++c) {
          const int64_t o = h.w_off + (int64_t)min(c0 + c, C - 1) * h.k + k;
          w[c] = PERTURBED ? fmaf(s, h.pv.vdir[o], h.pv.theta[o]) : h.pv.theta[o];
        }
#pragma unroll
        for (int u = 0; u < SU; ++u) xk[u] = x[u][k];
#pragma unroll
        for (int u = 0; u < SU; ++u)
#pragma unroll
          for (int c = 0; c < CU; ++c) acc[u][c] = fmaf(xk[u], w[c], acc[u][c]);
      }
#pragma unroll
      for (int u = 0; u < SU; ++u)
#pragma unroll
        for (int c = 0; c < CU; ++c) {
          const float z = wave_sum(acc[u][c]);
          if (lane == 0 && c0 + c < C && wave + FWAVES * u < n_own) s_z[(wave + FWAVES * u) * 64 + c0 + c] = (double)(z + h.pv.at(h.b_off + c0 + c, s));
        }
    }
  }
  __syncthreads();
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
// glam+ / glam- are the sums of the workgroups' partials in order.
constexpr int COLLECT = 16;
__device__ void meta_update(const MetaUpdateArgs& a, const double* part, int nblk) {
  const float eps = a.scalars[0];
  bool skip = (a.counters[2] != 0) || !(eps > 0.f);
  int bad = 0;
  for (int i = threadIdx.x; i < a.nl; i += ST_THREADS) {
    double gp = 0.0, gm = 0.0;
    for (int k0 = 0; k0 < nblk; k0 += COLLECT) {   // a load of each takes a microsecond: COLLECT workgroups' at once
      double p[COLLECT], m[COLLECT];
#pragma unroll
      for (int u = 0; u < COLLECT; ++u) {
        p[u] = k0 + u < nblk ? collect(part + (int64_t)(k0 + u) * a.nl + i) : 0.0;
        m[u] = k0 + u < nblk ? collect(part + (int64_t)(nblk + k0 + u) * a.nl + i) : 0.0;
      }
#pragma unroll
      for (int u = 0; u < COLLECT; ++u) { gp += p[u]; gm += m[u]; }
    }
    a.glam_p[i] = gp; a.glam_m[i] = gm;
    if (!skip) {
      const double h = -(gp - gm) / (2.0 * (double)eps);
      if (!(fabs(h) <= 3.0e38)) bad = 1;   // NaN, infinite, or beyond what the fp32 outputs hold
    }
  }
  const int64_t t = a.counters[1] + 1;
  if (__syncthreads_or(bad)) {   // every thread has read counters[2] above
    skip = true;
    if (threadIdx.x == 0) a.counters[2] = 1;
  }
  const double c1 = 1.0 / (1.0 - ipow((double)a.beta1, t));
  const double c2 = 1.0 / sqrt(1.0 - ipow((double)a.beta2, t));
  for (int i = threadIdx.x; i < a.nl; i += ST_THREADS) {
    const double gp = a.glam_p[i], gm = a.glam_m[i];   // written by this thread above
    const double h = skip ? 0.0 : -(gp - gm) / (2.0 * (double)eps);
    a.hypergrad[i] = (float)h;
    if (a.hypergrad_user) a.hypergrad_user[i] = (float)h;
    a.glam_p_f32[i] = (float)gp;
    a.glam_m_f32[i] = (float)gm;
    if (a.do_update && !skip) {
      const double m = (double)a.beta1 * a.meta_m[i] + (1.0 - (double)a.beta1) * h;
      const double v = (double)a.beta2 * a.meta_v[i] + (1.0 - (double)a.beta2) * h * h;
      a.meta_m[i] = (float)m;
      a.meta_v[i] = (float)v;
      a.lambda[i] = (float)((double)a.lambda[i] - (double)a.lr * c1 * m / (c2 * sqrt(v) + (double)a.eps));
    }
  }
  if (threadIdx.x == 0) {
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
  __shared__ float s_hred[FWAVES * 32 * 17];
  __shared__ double s_z[ST_SAMPLES * 64];
  __shared__ float s_lc[CORR ? MAX_CORR : 1];
  __shared__ double s_a[CORR ? ST_SAMPLES * MAX_CORR_HIDDEN : 1], s_t[CORR ? ST_SAMPLES * MAX_CORR_HIDDEN : 1];   // relu(a_ij), dL/da_ij
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

  for (int i = tid; i < 3 * H + 1; i += ST_THREADS) s_lam[i] = a.lambda[i];
  const int nlc = Hc > 0 ? Hc * 2 * C + Hc + C * Hc + C : 0;
  if (CORR)
    for (int i = tid; i < nlc; i += ST_THREADS) s_lc[i] = a.lambda[3 * H + 1 + i];
  double beff = (double)B;
  if (a.mask != nullptr) {
    double cnt = 0.0;
    for (int i = tid; i < B; i += ST_THREADS) cnt += a.mask[i] != 0 ? 1.0 : 0.0;
    beff = block_sum_d(cnt, red);
  }
  const double inv_beff = beff > 0.0 ? 1.0 / beff : 0.0;
  __syncthreads();
  if (!seq_mode) {
    if (a.head.dots && a.head.pv.scale() != 0.f) head_dots<true>(a.head, pass, i_begin, n_own, C, s_z);
    else if (a.head.dots) head_dots<false>(a.head, pass, i_begin, n_own, C, s_z);
    else head_logits(a.head, pass, i_begin, n_own, C, s_hred, s_z);
  }
  const float* W1 = s_lam; const float* b1 = s_lam + H; const float* W2 = s_lam + 2 * H;
  const double b2 = (double)s_lam[3 * H];
  const float* W1c = s_lc; const float* b1c = s_lc + Hc * 2 * C; const float* W2c = b1c + Hc; const float* b2c = W2c + C * Hc;

  if (seq_mode) {
    // wave w takes sequences w, w + waves, ...: its lanes stride over the positions (coalesced), keep the matching losses,
    // and a shuffle tree adds the 64 partial sums in a fixed order
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
  double gW2[PAIRS], gWp[PAIRS], gWy[PAIRS], gb1[PAIRS], gb2[PAIRS];   // corrector backward: thread owns (hidden unit, class) pairs
#pragma unroll
  for (int u = 0; u < PAIRS; ++u) gW2[u] = gWp[u] = gWy[u] = gb1[u] = gb2[u] = 0.0;

  for (int i0 = i_begin; i0 < i_end; i0 += ST_SAMPLES) {   // every thread takes part in every trip (barriers with CORR)
    const int i = i0 + grp;
    const bool live = i < i_end;
    const int ic = live ? i : i_end - 1;
    const double mk = (live && (a.mask == nullptr || a.mask[ic] != 0)) ? 1.0 : 0.0;
    double l, lse = 0.0, zc[CQ] = {0.0, 0.0, 0.0, 0.0};
    int yi = 0;
    double cs = 0.0;                                      // corrected soft label of class `lane` (Hc > 0)
    if (seq_mode) {
      l = s_l[ic - i_begin];
    } else {
      const double* z = s_z + (ic - i_begin) * 64;
      yi = min(max(a.y[ic], 0), C - 1);   // labels outside [0, C) are clamped
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
        double sc[MAX_CORR_CLASSES];
#pragma unroll
        for (int k = 0; k < MAX_CORR_CLASSES; ++k) sc[k] = 0.0;
        for (int j = lane; j < Hc; j += ST_LANES) {
          double aj = (double)b1c[j] + (double)W1c[j * 2 * C + yi];
          for (int k = 0; k < C; ++k) aj += (double)W1c[j * 2 * C + C + k] * s_p[grp * MAX_CORR_CLASSES + k];
          aj = aj > 0.0 ? aj : 0.0;
          s_a[grp * MAX_CORR_HIDDEN + j] = aj;
#pragma unroll
          for (int k = 0; k < MAX_CORR_CLASSES; ++k)
            if (k < C) sc[k] += (double)W2c[k * Hc + j] * aj;
        }
        double s_own = 0.0;
#pragma unroll
        for (int k = 0; k < MAX_CORR_CLASSES; ++k) {
          if (k < C) {   // the same for every lane
            const double tot = sum16(sc[k]);
            if (k == lane) s_own = tot + (double)b2c[k] + (k == yi ? (double)a.kappa : 0.0);
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
    if (a.mode == STAGE_EVAL) {
      if (CORR) __syncthreads();                          // s_p is rewritten by the next trip
      continue;
    }
    const double coef = mk * w * inv_beff;
    if (a.mode == STAGE_GLAM) {
      if (live && lane == 0) { s_l[i - i_begin] = l; s_dz[i - i_begin] = w * (1.0 - w) * l * mk * inv_beff; }
      if (CORR) {
        // ds_ik = c_ik (dc_ik - sum_k' c_ik' dc_ik'), dc_ik = -coef_i log p_ik;  t_ij = [a_ij > 0] sum_k W2c[k][j] ds_ik
        const double dc = lane < C ? -coef * (zc[0] - lse) : 0.0;
        const double dot = sum16(cs * dc), ds = cs * (dc - dot);
        s_ds[grp * MAX_CORR_CLASSES + lane] = ds;
        __syncthreads();
        for (int j = lane; j < Hc; j += ST_LANES) {
          double t = 0.0;
          for (int k = 0; k < C; ++k) t += (double)W2c[k * Hc + j] * s_ds[grp * MAX_CORR_CLASSES + k];
          s_t[grp * MAX_CORR_HIDDEN + j] = s_a[grp * MAX_CORR_HIDDEN + j] > 0.0 ? t : 0.0;
        }
        __syncthreads();
        const int ns = min(ST_SAMPLES, i_end - i0);
#pragma unroll
        for (int u = 0; u < PAIRS; ++u) {
          const int pr = tid + u * ST_THREADS, j = pr % Hc, k = pr / Hc;
          if (k >= C) continue;
          for (int s = 0; s < ns; ++s) {
            const double aj = s_a[s * MAX_CORR_HIDDEN + j], t = s_t[s * MAX_CORR_HIDDEN + j], d = s_ds[s * MAX_CORR_CLASSES + k];
            gW2[u] += d * aj;
            gWp[u] += t * s_p[s * MAX_CORR_CLASSES + k];
            gWy[u] += s_y[s] == k ? t : 0.0;
            gb1[u] += t;      // kept by the pairs with k == 0
            gb2[u] += d;      // kept by the pairs with j == 0
          }
        }
        __syncthreads();
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
      if (CORR) __syncthreads();
    }
  }
  if (a.mode == STAGE_EVAL) return;

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
#pragma unroll
    for (int u = 0; u < PAIRS; ++u) {
      const int pr = tid + u * ST_THREADS, j = pr % Hc, k = pr / Hc;
      if (k >= C) continue;
      publish(gc + j * 2 * C + k, gWy[u]);
      publish(gc + j * 2 * C + C + k, gWp[u]);
      publish(gc + Hc * 2 * C + Hc + k * Hc + j, gW2[u]);
      if (k == 0) publish(gc + Hc * 2 * C + j, gb1[u]);
      if (j == 0) publish(gc + Hc * 2 * C + Hc + C * Hc + k, gb2[u]);
    }
  }
  if (!last_block(a.ticket, total, &s_last)) return;
  meta_update(a.mu, a.part, nblk);
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
