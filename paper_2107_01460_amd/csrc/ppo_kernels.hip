// Clipped-PPO minibatch update: each network's forward pass over the gathered minibatch, loss and backward pass (fused_train.h,
// split_net.h, bf16_net.h; fp32 networks above 320 units layer by layer on gemm.h), gradients as copies added in a fixed order,
// global-norm clipping and Adam.
#include <algorithm>
#include <cmath>

#include "bf16_net.h"
#include "fused_train.h"
#include "gemm.h"
#include "heads.h"
#include "ppo_common.h"
#include "split_net.h"

namespace marl {

// implemented in policy_kernels.hip
void mlp_hidden_forward(const RowSrc& X, int64_t S, int Din, int H, const float* W1, const float* b1, const float* W2,
                        const float* b2, float* h1, float* h2, hipStream_t s);
const float* effective_params(const marl_config& c, const float* params, float* scratch, hipStream_t s, WeightUse use);
void stage_bf16_weights(const marl_config& c, const float* params, float* scratch, hipStream_t s);
int64_t effective_param_floats(const marl_config& c, bool update);
Bf16NetWeights effective_bf16_weights(const marl_config& c, const float* eff, int net);

namespace {

struct UpdateWsView {
  float *eff_params, *grad;
  Scalars* sc;        // two sets: optimiser step k accumulates into set k % 2 while its Adam kernel zeroes the other
  double* adv_stats;  // [n_epochs * n_minibatches][2]: sum and sum of squares of every minibatch's advantages
  int32_t* ident;
  float *h1a, *h2a, *dz1a;
  float *h1c, *h2c, *dz1c;
  float* partial;  // per-workgroup copies of one network's gradient (two-stage reduction of the fused training kernel)
  float* partial_head;  // networks that fused_train_kernel does not take: per-workgroup W3 / b3 gradients (and loss statistics)
  float* split_ws;      // theirs too: the k splits of a weight-gradient product, added in a fixed order
  int64_t split_floats;
  // bf16 configuration: one set of buffers, used by the actor and then by the critic
  bf16_t *bh1, *bdz2, *bdz1;
};

int64_t align256(int64_t x) { return (x + 255) & ~(int64_t)255; }

// floats of workspace for the k splits of dW2 (H x H + H) and dW1 (Din x H + H) of one network of S samples
int64_t split_ws_floats(int H, int Din, int64_t S) { return std::max(tn_copy_floats(H, H, S), tn_copy_floats(Din, H, S)); }

UpdateWsView carve_update_ws(const marl_config& c, void* ws, int64_t* total) {
  const Dims d = dims_of(c);
  const int64_t R = (int64_t)d.T * d.N, rows_mb = R / c.n_minibatches;
  const int64_t Sa = rows_mb * d.A, Sc = d.central ? rows_mb : Sa;
  char* p = static_cast<char*>(ws);
  int64_t off = 0;
  auto take = [&](int64_t bytes) {
    char* r = p + off;
    off += align256(bytes);
    return r;
  };
  UpdateWsView v{};
  v.eff_params = (float*)take(effective_param_floats(c, true) * 4);
  v.grad = (float*)take(d.P * 4);
  v.sc = (Scalars*)take(2 * sizeof(Scalars));
  v.adv_stats = (double*)take((int64_t)c.n_epochs * c.n_minibatches * 2 * sizeof(double));
  v.ident = (int32_t*)take(R * 4);
  if (!d.bf16) {
    v.h1a = (float*)take(Sa * d.Ha * 4);
    v.h2a = (float*)take(Sa * d.Ha * 4);
    v.dz1a = (float*)take(Sa * d.Ha * 4);
    v.h1c = (float*)take(Sc * d.Hc * 4);
    v.h2c = (float*)take(Sc * d.Hc * 4);
    v.dz1c = (float*)take(Sc * d.Hc * 4);
    int64_t copies = 0;
    if (fused_train_supported(d.Ha, d.D)) copies = std::max(copies, fused_train_partial_floats(d.Ha, d.D, Sa, d.Pa));
    if (fused_train_supported(d.Hc, d.Dc)) copies = std::max(copies, fused_train_partial_floats(d.Hc, d.Dc, Sc, d.P - d.Pa));
    if (fused_train_pair_supported(d.Ha, d.D, Sa, d.Hc, d.Dc, Sc)) copies = std::max(copies, fused_train_pair_partial_floats(Sa, d.Pa, d.P - d.Pa));
    v.partial = copies > 0 ? (float*)take(copies * 4) : nullptr;
    // the k splits of the weight gradients that are products of their own
    v.split_floats = 0;
    if (!fused_train_supported(d.Ha, d.D)) v.split_floats = std::max(v.split_floats, split_ws_floats(d.Ha, d.D, Sa));
    if (!fused_train_supported(d.Hc, d.Dc)) v.split_floats = std::max(v.split_floats, split_ws_floats(d.Hc, d.Dc, Sc));
    v.split_ws = v.split_floats > 0 ? (float*)take(v.split_floats * 4) : nullptr;
    auto head_floats = [](int H, int Din, int nout) -> int64_t {
      return fused_train_supported(H, Din) ? 0 : split_net_supported(H) ? split_net_partial_floats(H, nout) : loss_head_partial_floats(H, nout);
    };
    const int64_t head = std::max(head_floats(d.Ha, d.D, kActions), head_floats(d.Hc, d.Dc, 1));
    v.partial_head = (float*)take(head * 4);
  } else {
    const int64_t SH = std::max(Sa * d.Ha, Sc * d.Hc);
    v.bh1 = (bf16_t*)take(SH * 2);
    v.bdz2 = (bf16_t*)take(SH * 2);
    v.bdz1 = (bf16_t*)take(SH * 2);
    v.partial_head = (float*)take(std::max(bf16_net_grid(d.Ha) * copy_pitch(bf16_net_partial_floats(d.Ha, kActions)), bf16_net_grid(d.Hc) * copy_pitch(bf16_net_partial_floats(d.Hc, 1))) * 4);
    v.split_ws = (float*)take(std::max(std::max(bf16_wgrad_floats(false, d.Ha, d.Ha, Sa), bf16_wgrad_floats(true, d.D, d.Ha, Sa)),
                                       std::max(bf16_wgrad_floats(false, d.Hc, d.Hc, Sc), bf16_wgrad_floats(true, d.Dc, d.Hc, Sc))) * 4);
  }
  if (total) *total = off;
  return v;
}

// gW [rows][H] += A^T B, gb += column sums of B.  The k splits go to split_ws and are added in a fixed order, where the workspace
// has room and the bias gradient directly follows the weight gradient (its column sums ride along).
void weight_gradient(const RowSrc& A, const float* B, int64_t S, int rows, int H, float* gW, float* gb, float* split_ws, int64_t split_floats, hipStream_t s) {
  GemmArgs g{};
  g.A = A; g.B = B; g.ldb = H; g.C = gW; g.ldc = H;
  g.M = rows; g.N = H; g.K = S; g.colsum = gb;
  const int64_t count = (int64_t)rows * H + H, nz = tn_plan(rows, H, S).splits;
  if (split_ws != nullptr && gb == gW + (int64_t)rows * H && nz * count <= split_floats) {
    g.split_out = split_ws;
    g.split_count = count;
  }
  if (launch_gemm<GEMM_TN, EPI_ATOMIC_ADD>(g, s)) launch_reduce_partials(split_ws, (int)nz, count, gW, s);
}

// Backward through one network given dz2, the gradient of the second hidden layer's pre-activations.
void mlp_backward(const RowSrc& X, int64_t S, int Din, int H, const float* W2, const float* h1, const float* dz2, float* dz1, float* grad,
                  const NetOffsets& go, const UpdateWsView& w, hipStream_t s) {
  weight_gradient(RowSrc{h1, H, nullptr, 1, S}, dz2, S, H, H, grad + go.W2, grad + go.b2, w.split_ws, w.split_floats, s);
  GemmArgs g{};  // dz1 = (dz2 W2^T) * (1 - h1^2)
  g.A = RowSrc{dz2, H, nullptr, 1, S}; g.B = W2; g.ldb = H; g.C = dz1; g.ldc = H;
  g.aux_mat = h1; g.ldaux = H;
  g.M = S; g.N = H; g.K = H;
  launch_gemm<GEMM_NT, EPI_DTANH>(g, s);
  weight_gradient(X, dz1, S, Din, H, grad + go.W1, grad + go.b1, w.split_ws, w.split_floats, s);
}

// Forward, loss and backward of one fp32 network whose row tiles go through it in one kernel.
template <int NOUT, class LossFn>
int32_t train_net_split(const RowSrc& X, int64_t S, int Din, int H, const float* eff, const ParamMap& pm, int net, float* grad, const NetOffsets& go,
                        const LossFn& fn, const UpdateWsView& w, float* h1, float* dz2, float* dz1, hipStream_t s) {
  const NetOffsets o = padded_offsets(pm, net);
  SplitNetArgs a{};
  a.X = X; a.S = S; a.Din = Din; a.Kp = pm.kpad1[net]; a.W = eff + pm.sw_w1[net];
  a.b1 = eff + o.b1; a.b2 = eff + o.b2; a.W3 = eff + o.W3; a.b3 = eff + o.b3;
  a.h1 = h1; a.dz2 = dz2; a.dz1 = dz1; a.partial = w.partial_head;
  unsigned grid = 0;
  {
    TimedLaunch timed(KC_FUSED_TRAIN, 2.0 * (double)S * ((double)Din * H + 2.0 * (double)H * H), s);
    const int32_t rc = launch_split_net_rows<kSplitTrainRows, NOUT, true>(H, a, fn, &grid, s);
    if (rc != MARL_OK) return rc;
  }
  launch_reduce_partials(w.partial_head, (int)grid, (int64_t)H * NOUT + NOUT + 5, grad + go.W3, s, (int64_t)H * NOUT + NOUT, w.sc->acc);
  weight_gradient(RowSrc{h1, H, nullptr, 1, S}, dz2, S, H, H, grad + go.W2, grad + go.b2, w.split_ws, w.split_floats, s);
  weight_gradient(X, dz1, S, Din, H, grad + go.W1, grad + go.b1, w.split_ws, w.split_floats, s);
  return launch_status();
}

// Forward, loss and backward of one network in the bf16 configuration.
template <int NOUT, class LossFn>
int32_t train_net_bf16(const RowSrc& X, int64_t S, int Din, int H, const Bf16NetWeights& bw, const float* eff,
                       const NetOffsets& o, float* grad, const NetOffsets& go, const LossFn& fn, const UpdateWsView& w, hipStream_t s) {
  Bf16NetArgs a{};
  a.X = X; a.S = S; a.Din = Din; a.w = bw; a.b1 = eff + o.b1; a.b2 = eff + o.b2; a.W3 = eff + o.W3; a.b3 = eff + o.b3;
  a.h1 = w.bh1; a.dz2 = w.bdz2; a.dz1 = w.bdz1; a.partial = w.partial_head;
  unsigned grid = 0;
  int32_t rc;
  {
    TimedLaunch timed(KC_FUSED_TRAIN, 2.0 * (double)S * ((double)Din * H + 2.0 * (double)H * H), s);
    rc = launch_bf16_net_rows<64, NOUT, true>(H, a, fn, &grid, s);
  }
  if (rc != MARL_OK) return rc;
  launch_reduce_partials(w.partial_head, (int)grid, bf16_net_partial_floats(H, NOUT), grad + go.W3, s, (int64_t)H * NOUT + NOUT, w.sc->acc);
  Bf16WgradArgs g{};
  g.A = w.bh1; g.lda = H; g.B = w.bdz2; g.S = S; g.M = H; g.N = H; g.out = w.split_ws;
  if ((rc = launch_bf16_wgrad(false, g, grad + go.W2, s)) != MARL_OK) return rc;
  g.X = X; g.B = w.bdz1; g.M = Din;
  return launch_bf16_wgrad(true, g, grad + go.W1, s);
}

}  // namespace

int64_t update_workspace_bytes(const marl_config& c) {
  int64_t total = 0;
  carve_update_ws(c, nullptr, &total);
  return total;
}

namespace {
__global__ void advance_counters_kernel(marl_counters* counters, uint64_t steps, int64_t adam_steps) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    counters->step += steps;
    counters->adam_step += adam_steps;
  }
}
}  // namespace

int32_t launch_advance_counters(marl_counters* counters, uint64_t steps, int64_t adam_steps, hipStream_t s) {
  hipLaunchKernelGGL(advance_counters_kernel, dim3(1), dim3(64), 0, s, counters, steps, adam_steps);
  return launch_status();
}

int32_t launch_ppo_update(const marl_config& c, marl_traj tr, float* params, float* adam_m, float* adam_v,
                          int64_t adam_step0, const int32_t* perm, float* stats, float* grad_dump, void* workspace,
                          hipStream_t s, const int64_t* adam_step_base) {
  const Dims d = dims_of(c);
  const UpdateWsView w = carve_update_ws(c, workspace, nullptr);
  const int64_t R = (int64_t)d.T * d.N, rows_mb = R / c.n_minibatches;
  const int64_t Sa = rows_mb * d.A, Sc = d.central ? rows_mb : Sa;
  if (perm == nullptr)
    hipLaunchKernelGGL(iota_kernel, dim3((unsigned)((R + 255) / 256)), dim3(256), 0, s, w.ident, R);
  // ga/gc: blocks of the gradient (parameter-vector layout); oa/oc: blocks of the aligned working copy of the weights
  const NetOffsets ga = net_offsets(0, d.D, d.Ha, kActions), gc = net_offsets(d.Pa, d.Dc, d.Hc, 1);
  const ParamMap pm = param_map(d, true);
  const NetOffsets oa = padded_offsets(pm, 0), oc = padded_offsets(pm, 1);
  int64_t k = adam_step0;
  // Once per update: the gradient, both sets of scalars and the advantage statistics start at zero (afterwards every
  // Adam kernel zeroes the gradient and the scalars of the next step), and the advantage statistics of ALL minibatches
  // of all epochs are summed in one launch -- the row orders are known up front.
  const int n_steps = c.n_epochs * c.n_minibatches;
  hipLaunchKernelGGL(zero_step_kernel, dim3((unsigned)((d.P + 255) / 256)), dim3(256), 0, s, w.grad, d.P, w.sc, 2,
                     w.adv_stats, 2 * n_steps);
  if (c.normalize_adv) {
    const unsigned nb = (unsigned)std::min<int64_t>(std::max(1, 256 / c.n_minibatches), (Sa + 255) / 256);  // every workgroup ends with two atomics on its minibatch's two doubles
    hipLaunchKernelGGL(adv_stats_all_kernel, dim3(nb, (unsigned)n_steps), dim3(256), 0, s, tr.adv, perm ? perm : w.ident,
                       perm ? R : (int64_t)0, c.n_minibatches, rows_mb, d.A, w.adv_stats);
  }
  for (int e = 0; e < c.n_epochs; ++e) {
    for (int mb = 0; mb < c.n_minibatches; ++mb) {
      const int step = e * c.n_minibatches + mb;
      Scalars* const sck = w.sc + (step & 1);
      UpdateWsView wk = w;  // the view the helpers get: this step's scalars
      wk.sc = sck;
      const int32_t* rows = (perm ? perm + (int64_t)e * R : w.ident) + (int64_t)mb * rows_mb;
      const float* const eff = w.eff_params;
      if (step == 0) effective_params(c, params, w.eff_params, s, USE_UPDATE);
      else stage_bf16_weights(c, params, w.eff_params, s);  // (the rest of the copy: the last step's Adam kernel)
      LossCommon lc{};
      lc.rows = rows; lc.A = d.A; lc.ad = make_small_div(d.A); lc.rows_mb = rows_mb; lc.inv_B = (float)(1.0 / (double)(rows_mb * d.A));
      lc.sc = sck; lc.adv_stats = w.adv_stats + 2 * step; lc.normalize = c.normalize_adv; lc.clip_eps = c.clip_eps;
      lc.ent_coef = c.ent_coef; lc.vf_coef = c.vf_coef; lc.clip_value = c.clip_value;
      const RowSrc Xa{tr.obs, d.D, rows, d.A, Sa, make_small_div(d.A)};
      const RowSrc Xc{tr.obs, d.Dc, rows, d.central ? 1 : d.A, Sc, make_small_div(d.central ? 1 : d.A)};
      auto train_args = [&](const RowSrc& X, int64_t S, int net) {
        const NetOffsets& o = net == 0 ? oa : oc;
        FusedTrainArgs t{};
        t.X = X; t.S = S; t.Din = pm.din[net]; t.Kp = pm.kpad1[net]; t.W = eff + pm.sw_w1[net];
        t.b1 = eff + o.b1; t.b2 = eff + o.b2; t.W3 = eff + o.W3; t.b3 = eff + o.b3;
        t.grad = w.grad + (net == 0 ? ga : gc).W1; t.gcount = net == 0 ? d.Pa : d.P - d.Pa;
        t.stats = sck->acc; t.partial = w.partial;
        return t;
      };
      // ---- both networks in one launch (same shape, few tiles)
      const bool pair = !d.bf16 && Sa < ((int64_t)1 << 31) && fused_train_pair_supported(d.Ha, d.D, Sa, d.Hc, d.Dc, Sc);
      if (pair) {
        ActorLoss fa{lc, tr.action, tr.logp, tr.adv};
        CriticLoss fc{lc, tr.ret, tr.value, d.central ? d.A : 1};
        const FusedTrainArgs ta = train_args(Xa, Sa, 0), tc = train_args(Xc, Sc, 1);
        const int32_t rc = (launch_fused_train_pair<kActions, 1>(d.Ha, ta, fa, tc, fc, s));
        if (rc != MARL_OK) return rc;
      }
      // ---- actor
      if (!pair) {
        ActorLoss fn{lc, tr.action, tr.logp, tr.adv};
        if (d.bf16) {
          const int32_t rc = train_net_bf16<kActions>(Xa, Sa, d.D, d.Ha, effective_bf16_weights(c, eff, 0), eff, oa, w.grad, ga, fn, wk, s);
          if (rc != MARL_OK) return rc;
        } else if (fused_train_supported(d.Ha, d.D) && Sa < ((int64_t)1 << 31)) {
          const int32_t rc = launch_fused_train<kActions>(d.Ha, train_args(Xa, Sa, 0), fn, s);
          if (rc != MARL_OK) return rc;
        } else if (split_net_supported(d.Ha)) {
          const int32_t rc = train_net_split<kActions>(Xa, Sa, d.D, d.Ha, eff, pm, 0, w.grad, ga, fn, wk, w.h1a, w.h2a, w.dz1a, s);
          if (rc != MARL_OK) return rc;
        } else {
          mlp_hidden_forward(Xa, Sa, d.D, d.Ha, eff + oa.W1, eff + oa.b1, eff + oa.W2, eff + oa.b2, w.h1a, w.h2a, s);
          const int32_t rc = launch_loss_head<kActions, true>(w.h2a, Sa, d.Ha, eff + oa.W3, eff + oa.b3, fn, nullptr, w.grad + ga.W3,
                                                              w.partial_head, sck, s);
          if (rc != MARL_OK) return rc;
          mlp_backward(Xa, Sa, d.D, d.Ha, eff + oa.W2, w.h1a, w.h2a, w.dz1a, w.grad, ga, wk, s);
        }
      }
      // ---- critic
      if (!pair) {
        CriticLoss fn{lc, tr.ret, tr.value, d.central ? d.A : 1};
        if (d.bf16) {
          const int32_t rc = train_net_bf16<1>(Xc, Sc, d.Dc, d.Hc, effective_bf16_weights(c, eff, 1), eff, oc, w.grad, gc, fn, wk, s);
          if (rc != MARL_OK) return rc;
        } else if (fused_train_supported(d.Hc, d.Dc) && Sc < ((int64_t)1 << 31)) {
          const int32_t rc = launch_fused_train<1>(d.Hc, train_args(Xc, Sc, 1), fn, s);
          if (rc != MARL_OK) return rc;
        } else if (split_net_supported(d.Hc)) {
          const int32_t rc = train_net_split<1>(Xc, Sc, d.Dc, d.Hc, eff, pm, 1, w.grad, gc, fn, wk, w.h1c, w.h2c, w.dz1c, s);
          if (rc != MARL_OK) return rc;
        } else {
          mlp_hidden_forward(Xc, Sc, d.Dc, d.Hc, eff + oc.W1, eff + oc.b1, eff + oc.W2, eff + oc.b2, w.h1c, w.h2c, s);
          const int32_t rc = launch_loss_head<1, true>(w.h2c, Sc, d.Hc, eff + oc.W3, eff + oc.b3, fn, nullptr, w.grad + gc.W3,
                                                       w.partial_head, sck, s);
          if (rc != MARL_OK) return rc;
          mlp_backward(Xc, Sc, d.Dc, d.Hc, eff + oc.W2, w.h1c, w.h2c, w.dz1c, w.grad, gc, wk, s);
        }
      }
      // ---- clip + Adam
      hipLaunchKernelGGL(grad_norm_kernel, dim3(grad_norm_blocks(d.P)), dim3(256), 0, s,
                         w.grad, d.P, sck);
      ++k;
      AdamArgs a{};
      a.norm_blocks = (int)grad_norm_blocks(d.P);
      a.k_base = adam_step_base;
      a.k_local = (int)k;
      a.lr = c.lr; a.b1 = c.beta1; a.b2 = c.beta2; a.eps = c.adam_eps;
      a.bc1 = (float)(1.0 - std::pow((double)c.beta1, (double)k));
      a.bc2 = (float)(1.0 - std::pow((double)c.beta2, (double)k));
      a.max_norm = c.max_grad_norm; a.ent_coef = c.ent_coef; a.vf_coef = c.vf_coef;
      const bool last = (e == c.n_epochs - 1 && mb == c.n_minibatches - 1);
      hipLaunchKernelGGL(adam_kernel<StageNext>, dim3((unsigned)((d.P + 255) / 256)), dim3(256), 0, s, params, adam_m, adam_v,
                         w.grad, d.P, a, sck, stats + (int64_t)(e * c.n_minibatches + mb) * MARL_N_STATS,
                         (last ? grad_dump : nullptr), w.sc + ((step + 1) & 1),
                         StageNext{last ? nullptr : w.eff_params, pm, (int)d.bf16});
      const int32_t rc = launch_status();
      if (rc != MARL_OK) return rc;
    }
  }
  return MARL_OK;
}

}  // namespace marl
