// Actor / critic forward pass of the rollout, categorical sampling, and the rollout driver.
//
// A forward pass is one kernel per network (split_net.h, bf16_net.h; small fp32 calls one for both, fused_forward.h), and fp32
// networks above 320 units go layer by layer on gemm.h and the output-layer kernels of heads.h.  What the actor's kernel does with
// a sample's logits includes the draw of the action by Gumbel-max from Philox uniforms and its log-probability.
#include "bf16_net.h"
#include "fused_forward.h"
#include "gemm.h"
#include "heads.h"
#include "rollout_fused.h"
#include "split_net.h"
#include "stage_params.h"

namespace marl {

int64_t effective_param_floats(const marl_config& c, bool update);

namespace {

// clear[0 .. n_clear - 1] = 0 beside it, for a kernel behind this one
__global__ void stage_params_kernel(const float* __restrict__ src, float* __restrict__ dst, ParamMap pm, int for_rollout, int for_update, int32_t* clear, int n_clear) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t k = i; k < n_clear; k += (int64_t)gridDim.x * blockDim.x) clear[k] = 0;
  if (i >= pm.src[12]) return;
#pragma unroll
  for (int net = 0; net < 2; ++net) {  // zero rows of the copies of W1 (fewer than 32 rows: far fewer floats than parameters)
    const int H = pm.hidden[net];
    if (pm.fused[net] && i < (int64_t)(pm.kpad1[net] - pm.din[net]) * H) stage_element(dst, pm, net, pm.sw_w1[net], 0.f, pm.din[net] + i / H, i % H, for_rollout);
  }
  stage_param(dst, pm, i, src[i], false, for_rollout, for_update != 0);
}

// The same for the bf16 configuration, the networks' fragment copies (bf16_stage) in the first `frag_blocks` workgroups of the launch.
__global__ void __launch_bounds__(256) stage_bf16_params_kernel(const float* __restrict__ src, float* __restrict__ dst, ParamMap pm, Bf16StageNet a, Bf16StageNet b, unsigned frag_blocks) {
  if (blockIdx.x < frag_blocks) {
    bf16_stage(a, b, (int64_t)blockIdx.x * 256 + threadIdx.x);
    return;
  }
  const int64_t i = (int64_t)(blockIdx.x - frag_blocks) * 256 + threadIdx.x;
  if (i < pm.src[12]) stage_param(dst, pm, i, src[i], true, COPY_SPLIT, false);
}

// What the rollout does with a sample's outputs.
struct ActorRolloutFinish {
  float* logits_out;  // nullable
  SampleArgs sa;
  int do_sample;
  __device__ __forceinline__ void operator()(int64_t s, const float out[kActions], float*, float*) const {
    if (logits_out) {
#pragma unroll
      for (int k = 0; k < kActions; ++k) logits_out[s * kActions + k] = out[k];
    }
    if (do_sample) sample_and_store(out, s, sa);
  }
};
// Rows below `split` go to value_out, the rest (the rows of the post-rollout observation, when one pass covers all
// T + 1 slabs) to tail_out.
struct CriticRolloutFinish {
  float* value_out;
  int broadcast;
  int64_t split;
  float* tail_out;
  __device__ __forceinline__ void operator()(int64_t s, const float out[1], float*, float*) const {
    float* const dst = s < split ? value_out + s * broadcast : tail_out + (s - split) * broadcast;
    for (int k = 0; k < broadcast; ++k) dst[k] = out[0];
  }
};

FusedFwdArgs direct_args(const RowSrc& X, int64_t S, int Din, const float* params, const NetOffsets& o) {
  FusedFwdArgs a{};
  a.X = X; a.S = S; a.Din = Din;
  a.W1 = params + o.W1; a.b1 = params + o.b1; a.W2 = params + o.W2; a.b2 = params + o.b2; a.W3 = params + o.W3; a.b3 = params + o.b3;
  a.kpad1 = (Din + 15) / 16 * 16; a.px = fused_forward_px(Din);
  return a;
}

SplitNetArgs split_net_args(const RowSrc& X, int64_t S, int Din, const float* eff, const ParamMap& pm, int net) {
  const NetOffsets o = padded_offsets(pm, net);
  SplitNetArgs a{};
  a.X = X; a.S = S; a.Din = Din; a.Kp = pm.kpad1[net]; a.W = eff + pm.sw_w1[net];
  a.b1 = eff + o.b1; a.b2 = eff + o.b2; a.W3 = eff + o.W3; a.b3 = eff + o.b3;
  return a;
}

struct RolloutWsView {
  float *eff_params, *h1a, *h2a, *h1c, *h2c;  // activations: layer-by-layer fp32 networks
};

int64_t align256(int64_t x) { return (x + 255) & ~(int64_t)255; }

bool use_fused_rollout(const marl_config& c) {
  const Dims d = dims_of(c);
  return !d.bf16 && rollout_fused_supported(d.Ha, d.A);
}

}  // namespace

// What marl_rollout_static compares with MARL_STATIC_SCRATCH_BYTES: the working copy of the parameters and both hidden layers of one
// pass (in bf16 the packed inputs too) as kernels that go layer by layer hold them, all fp32 networks of 64, 128 and 256 units on chip
// with split copies of their weights.  A rule of its own, so that what the call takes does not move with the kernels; what these need
// (carve_rollout_ws) is far less, or, where split copies of the weights take the place of plain ones, up to 0.6 MB more.
int64_t rollout_static_need(const marl_config& c, int64_t n_rows) {
  const Dims d = dims_of(c);
  int64_t params = 0, layers = 0;
  auto add = [&](int64_t floats) { params += (floats + 63) / 64 * 64; };
  for (int k = 0; k < 2; ++k) {
    const int64_t H = k ? d.Hc : d.Ha, din = k ? d.Dc : d.D, out = k ? 1 : kActions, rows = k && d.central ? n_rows : n_rows * d.A;
    const bool on_chip = !d.bf16 && fused_forward_supported((int)H, (int)din);
    add(on_chip ? (din + 15) / 16 * 16 * H * 3 / 2 : din * H);
    add(H);
    add(on_chip ? H * H * 3 / 2 : H * H);
    add(H); add(H * out); add(out);
    if (d.bf16) layers += align256(rows * round_up64(din) * 2) + 2 * align256(rows * H * 2);
    else if (!on_chip) layers += 2 * align256(rows * H * 4);
  }
  if (d.bf16) params += (bf16_net_weight_elems(d.D, d.Ha) + bf16_net_weight_elems(d.Dc, d.Hc) + 1) / 2 + 192;
  return align256(params * 4) + layers;
}

namespace {

RolloutWsView carve_rollout_ws(const marl_config& c, int64_t n_rows, void* ws, int64_t* total) {
  const Dims d = dims_of(c);
  const int64_t S = n_rows * d.A, Sc = d.central ? n_rows : S;
  char* p = static_cast<char*>(ws);
  int64_t off = 0;
  auto take = [&](int64_t bytes) {
    char* r = p + off;
    off += align256(bytes);
    return r;
  };
  RolloutWsView v{};
  v.eff_params = (float*)take(effective_param_floats(c, false) * 4);
  const int H[2] = {d.Ha, d.Hc}, din[2] = {d.D, d.Dc};
  const int64_t rows[2] = {S, Sc};
  if (!d.bf16) {  // hidden activations of one pass: only the layer-by-layer path stores them
    float** const h[2][2] = {{&v.h1a, &v.h2a}, {&v.h1c, &v.h2c}};
    for (int n = 0; n < 2; ++n)
      if (!split_net_supported(H[n]))
        for (float** p2 : h[n]) *p2 = (float*)take(rows[n] * H[n] * 4);
  }
  // never less than the size that marl_rollout_static decides by
  off = std::max(off, rollout_static_need(c, n_rows));
  if (total) *total = off;
  return v;
}

}  // namespace

void mlp_hidden_forward(const RowSrc& X, int64_t S, int Din, int H, const float* W1, const float* b1, const float* W2,
                        const float* b2, float* h1, float* h2, hipStream_t s) {
  GemmArgs g{};
  g.A = X; g.B = W1; g.ldb = H; g.C = h1; g.ldc = H; g.aux_vec = b1;
  g.M = S; g.N = H; g.K = Din;
  launch_gemm<GEMM_NN, EPI_BIAS_TANH>(g, s);
  GemmArgs g2{};
  g2.A = RowSrc{h1, H, nullptr, 1, S}; g2.B = W2; g2.ldb = H; g2.C = h2; g2.ldc = H; g2.aux_vec = b2;
  g2.M = S; g2.N = H; g2.K = H;
  launch_gemm<GEMM_NN, EPI_BIAS_TANH>(g2, s);
}

// Floats of the working copy: the aligned fp32 copy, followed (bf16 configuration) by the bf16 weight matrices.
int64_t effective_param_floats(const marl_config& c, bool update) {
  const Dims d = dims_of(c);
  int64_t n = param_map(d, update).total;
  if (d.bf16) n += (bf16_net_weight_elems(d.D, d.Ha) + bf16_net_weight_elems(d.Dc, d.Hc) + 1) / 2 + 192;  // + alignment slack
  return n;
}

Bf16NetWeights effective_bf16_weights(const marl_config& c, const float* eff, int net) {
  const Dims d = dims_of(c);  // (the map is the same for an update and for a forward pass: no network is fused)
  bf16_t* base = reinterpret_cast<bf16_t*>(const_cast<float*>(eff) + ((param_map(d, false).total + 63) / 64) * 64);
  if (net == 0) return Bf16NetWeights{base, (int)round_up64(d.D)};
  return Bf16NetWeights{base + ((bf16_net_weight_elems(d.D, d.Ha) + 63) / 64) * 64, (int)round_up64(d.Dc)};
}

// What the bf16 networks' weight copies are made from.
std::pair<Bf16StageNet, Bf16StageNet> bf16_stage_nets(const marl_config& c, const float* params, const float* scratch) {
  const Dims d = dims_of(c);
  const NetOffsets oa = net_offsets(0, d.D, d.Ha, kActions), oc = net_offsets(d.Pa, d.Dc, d.Hc, 1);
  const Bf16NetWeights wa = effective_bf16_weights(c, scratch, 0), wc = effective_bf16_weights(c, scratch, 1);
  return {Bf16StageNet{params + oa.W1, params + oa.W2, wa.w, d.D, wa.Kp, d.Ha}, Bf16StageNet{params + oc.W1, params + oc.W2, wc.w, d.Dc, wc.Kp, d.Hc}};
}
// The copies by themselves (nothing for other configurations).
void stage_bf16_weights(const marl_config& c, const float* params, float* scratch, hipStream_t s) {
  if (c.precision != 1) return;
  const auto nets = bf16_stage_nets(c, params, scratch);
  launch_bf16_stage(nets.first, nets.second, s);
}

static const float* stage_working_copy(const marl_config& c, const float* params, float* scratch, hipStream_t s, WeightUse use, RolloutCopy actor, int32_t* clear, int n_clear) {
  const Dims d = dims_of(c);
  const ParamMap pm = param_map(d, use == USE_UPDATE);
  const unsigned blocks = (unsigned)((d.P + 255) / 256);
  if (d.bf16) {
    const auto nets = bf16_stage_nets(c, params, scratch);
    const unsigned frag = bf16_stage_blocks(nets.first, nets.second);
    hipLaunchKernelGGL(stage_bf16_params_kernel, dim3(frag + blocks), dim3(256), 0, s, params, scratch, pm, nets.first, nets.second, frag);
  } else {
    hipLaunchKernelGGL(stage_params_kernel, dim3(blocks), dim3(256), 0, s, params, scratch, pm,
                       (int)actor, (int)(use == USE_UPDATE), clear, n_clear);
  }
  return scratch;
}
const float* effective_params(const marl_config& c, const float* params, float* scratch, hipStream_t s, WeightUse use) {
  return stage_working_copy(c, params, scratch, s, use, COPY_SPLIT, nullptr, 0);
}

int64_t rollout_workspace_bytes(const marl_config& c, int64_t n_rows) {
  int64_t total = 0;
  carve_rollout_ws(c, n_rows, nullptr, &total);
  return total;
}

// One forward pass over n_rows observation rows.  Any of logits / value / sampling outputs may be absent.
// value_tail (nullable): the values of rows value_split .. n_rows go there instead (kernels that keep a row's activations on chip only).
static int32_t forward_rows(const marl_config& c, const float* eff, const float* obs, int64_t n_rows,
                            const RolloutWsView& w, bool want_actor, float* logits_out, const SampleArgs* sample,
                            float* value_out, hipStream_t s, int64_t value_split = -1, float* value_tail = nullptr) {
  const Dims d = dims_of(c);
  const int64_t S = n_rows * d.A;
  if (d.bf16) {
    auto args = [&](int net, int64_t rows, int Din) {
      const NetOffsets o = padded_offsets(param_map(d, false), net);
      Bf16NetArgs a{};
      a.X = RowSrc{obs, Din, nullptr, 1, rows}; a.S = rows; a.Din = Din; a.w = effective_bf16_weights(c, eff, net);
      a.b1 = eff + o.b1; a.b2 = eff + o.b2; a.W3 = eff + o.W3; a.b3 = eff + o.b3;
      return a;
    };
    const int64_t Sc = d.central ? n_rows : S;
    const ActorRolloutFinish fa{logits_out, sample ? *sample : SampleArgs{}, sample ? 1 : 0};
    const CriticRolloutFinish fc{value_out, d.central ? d.A : 1, value_tail ? value_split : Sc, value_tail};
    // both in one launch where they take the same kernel: the second network's tiles follow on the compute units as the first one's end
    if (want_actor && value_out && bf16_pair_supported(d.Ha, S, d.Hc, Sc))
      return launch_bf16_forward_pair<kActions, 1>(d.Ha, args(0, S, d.D), fa, args(1, Sc, d.Dc), fc, s);
    if (want_actor) {
      const int32_t rc = launch_bf16_forward<kActions>(d.Ha, args(0, S, d.D), fa, s);
      if (rc != MARL_OK) return rc;
    }
    if (value_out) {
      const int32_t rc = launch_bf16_forward<1>(d.Hc, args(1, Sc, d.Dc), fc, s);
      if (rc != MARL_OK) return rc;
    }
    return launch_status();
  }
  if (want_actor) {
    const NetOffsets o = padded_offsets(param_map(d, false), 0);
    const RowSrc X{obs, d.D, nullptr, 1, S};
    if (split_net_supported(d.Ha)) {
      ActorRolloutFinish fin{logits_out, sample ? *sample : SampleArgs{}, sample ? 1 : 0};
      const int32_t rc = launch_split_forward<kActions>(d.Ha, split_net_args(X, S, d.D, eff, param_map(d, false), 0), fin, s);
      if (rc != MARL_OK) return rc;
    } else {
      mlp_hidden_forward(X, S, d.D, d.Ha, eff + o.W1, eff + o.b1, eff + o.W2, eff + o.b2, w.h1a, w.h2a, s);
      launch_actor_head_rollout(w.h2a, S, d.Ha, eff + o.W3, eff + o.b3, logits_out, sample, s);
    }
  }
  if (value_out) {
    const NetOffsets o = padded_offsets(param_map(d, false), 1);
    const int64_t Sc = d.central ? n_rows : S;
    const RowSrc X{obs, d.Dc, nullptr, 1, Sc};
    if (split_net_supported(d.Hc)) {
      CriticRolloutFinish fin{value_out, d.central ? d.A : 1, value_tail ? value_split : Sc, value_tail};
      const int32_t rc = launch_split_forward<1>(d.Hc, split_net_args(X, Sc, d.Dc, eff, param_map(d, false), 1), fin, s);
      if (rc != MARL_OK) return rc;
    } else {
      mlp_hidden_forward(X, Sc, d.Dc, d.Hc, eff + o.W1, eff + o.b1, eff + o.W2, eff + o.b2, w.h1c, w.h2c, s);
      launch_critic_head_rollout(w.h2c, Sc, d.Hc, eff + o.W3, eff + o.b3, value_out, d.central ? d.A : 1, s);
    }
  }
  return launch_status();
}

int32_t launch_policy_forward(const marl_config& c, const float* params, const float* obs, int64_t n_rows,
                              float* logits, float* value, void* workspace, hipStream_t s) {
  const Dims d = dims_of(c);
  const int64_t S = n_rows * d.A;
  if (!d.bf16 && S <= kForwardSmall && fused_forward_supported(d.Ha, d.D) && fused_forward_supported(d.Hc, d.Dc)) {
    const int64_t Sc = d.central ? n_rows : S;
    auto direct = [&](int64_t rows, int Din, const NetOffsets& o) { return direct_args(RowSrc{obs, Din, nullptr, 1, rows}, rows, Din, params, o); };
    const ActorRolloutFinish fa{logits, SampleArgs{}, 0};
    const CriticRolloutFinish fc{value, d.central ? d.A : 1, Sc, nullptr};
    return launch_fused_forward_small<kActions, 1>(
        d.Ha, direct(logits != nullptr ? S : 0, d.D, net_offsets(0, d.D, d.Ha, kActions)), fa,
        d.Hc, direct(value != nullptr ? Sc : 0, d.Dc, net_offsets(d.Pa, d.Dc, d.Hc, 1)), fc, s);
  }
  const RolloutWsView w = carve_rollout_ws(c, n_rows, workspace, nullptr);
  const float* eff = effective_params(c, params, w.eff_params, s, USE_FORWARD);
  return forward_rows(c, eff, obs, n_rows, w, logits != nullptr, logits, nullptr, value, s);
}

int32_t launch_sample(const marl_config& c, const float* logits, const float* uniforms, const int32_t* forced,
                      int64_t n, uint64_t step, int32_t* action, int32_t* sampled, float* logp, hipStream_t s) {
  SampleArgs a{};
  a.uniforms = uniforms; a.forced = forced; a.action = action; a.sampled = sampled; a.logp = logp;
  a.step = step; a.k0 = (uint32_t)(c.seed & 0xffffffffu); a.k1 = (uint32_t)(c.seed >> 32);
  launch_sample_only(logits, n, a, s);
  return launch_status();
}

static int32_t launch_rollout_fused(const marl_config& c, bool eval, const RolloutArgs& a, hipStream_t s) {
  switch (c.view) {
    case 3: return launch_rollout_fused_v3(c.actor_hidden, eval, a, s);
    case 5: return launch_rollout_fused_v5(c.actor_hidden, eval, a, s);
    case 7: return launch_rollout_fused_v7(c.actor_hidden, eval, a, s);
    default: return MARL_E_CONFIG;
  }
}

// The actor's part of the arguments of the fused rollout and evaluation kernels.
static RolloutArgs rollout_fused_args(const marl_config& c, marl_env_state st, const float* eff) {
  const Dims d = dims_of(c);
  const ParamMap pm = param_map(d, false);
  const NetOffsets o = padded_offsets(pm, 0);
  RolloutArgs a{};
  a.p = env_params(c);
  a.st = st;
  a.W1 = eff + pm.sw_w1[0]; a.W2 = eff + pm.sw_w2[0];
  a.b1 = eff + o.b1; a.b2 = eff + o.b2; a.W3 = eff + o.W3; a.b3 = eff + o.b3;
  return a;
}

int32_t launch_rollout(const marl_config& c, marl_env_state st, const float* params, marl_traj tr,
                       uint64_t step_offset, const int32_t* forced_actions, const float* forced_uniforms,
                       void* workspace, hipStream_t s, const uint64_t* step_base) {
  const Dims d = dims_of(c);
  const RolloutWsView w = carve_rollout_ws(c, d.N, workspace, nullptr);
  const bool fused = use_fused_rollout(c);
  const int rows = fused ? rollout_rows(d.Ha, d.A, d.N) : 0;
  const float* eff = stage_working_copy(c, params, w.eff_params, s, USE_FORWARD, !fused ? COPY_SPLIT : rows == 16 ? COPY_FP32_16 : COPY_FP32, nullptr, 0);
  const int64_t NA = d.NA, slab = NA * d.D;
  int32_t rc;
  // The values do not steer the rollout (the parameters are constant during it): where the critic's forward pass
  // needs no per-row workspace (whole networks in one kernel), the values of all T steps and of the post-rollout observation
  // are computed in one pass over the stored observations afterwards instead of one small launch per step.
  const bool batch_values = d.bf16 || split_net_supported(d.Hc);
  if (fused) {
    // all T steps in one launch: a workgroup keeps its environments on chip and streams the trajectory out
    RolloutArgs a = rollout_fused_args(c, st, eff);
    a.T = d.T; a.rows = rows;
    a.obs = tr.obs; a.action = tr.action; a.logp = tr.logp; a.reward = tr.reward; a.done = tr.done;
    a.logits = tr.logits; a.sampled = tr.sampled; a.uniforms = forced_uniforms; a.forced = forced_actions;
    a.step0 = step_offset; a.step_base = step_base;
    {
      // booked with the algorithmic flops of the actor's two hidden layers over all T steps
      const double flops = 2.0 * (double)d.T * NA * ((double)d.D * d.Ha + (double)d.Ha * d.Ha);
      TimedLaunch timed(KC_ROLLOUT, flops, s);
      if ((rc = launch_rollout_fused(c, false, a, s)) != MARL_OK) return rc;
    }
    if (!batch_values) {
      for (int t = 0; t < d.T; ++t)
        if ((rc = forward_rows(c, eff, tr.obs + (int64_t)t * slab, d.N, w, false, nullptr, nullptr, tr.value + (int64_t)t * NA, s)) != MARL_OK)
          return rc;
    }
  } else {
    rc = launch_env_step(c, st, nullptr, tr.obs, nullptr, nullptr, /*do_step=*/false, s);
    if (rc != MARL_OK) return rc;
    for (int t = 0; t < d.T; ++t) {
      SampleArgs a{};
      a.uniforms = forced_uniforms ? forced_uniforms + (int64_t)t * NA * kActions : nullptr;
      a.forced = forced_actions ? forced_actions + (int64_t)t * NA : nullptr;
      a.action = tr.action + (int64_t)t * NA;
      a.sampled = tr.sampled ? tr.sampled + (int64_t)t * NA : nullptr;
      a.logp = tr.logp + (int64_t)t * NA;
      a.step = step_offset + (uint64_t)t;
      a.step_base = step_base;
      a.k0 = (uint32_t)(c.seed & 0xffffffffu);
      a.k1 = (uint32_t)(c.seed >> 32);
      rc = forward_rows(c, eff, tr.obs + (int64_t)t * slab, d.N, w, true,
                        tr.logits ? tr.logits + (int64_t)t * NA * kActions : nullptr, &a,
                        batch_values ? nullptr : tr.value + (int64_t)t * NA, s);
      if (rc != MARL_OK) return rc;
      rc = launch_env_step(c, st, a.action, tr.obs + (int64_t)(t + 1) * slab, tr.reward + (int64_t)t * NA,
                           tr.done + (int64_t)t * d.N, true, s);
      if (rc != MARL_OK) return rc;
    }
  }
  if (batch_values) {  // slabs 0 .. T in one launch: rows of slab T go to last_value
    const int64_t Sc_split = (int64_t)d.T * (d.central ? d.N : NA);
    return forward_rows(c, eff, tr.obs, (int64_t)(d.T + 1) * d.N, w, false, nullptr, nullptr, tr.value, s, Sc_split, tr.last_value);
  }
  return forward_rows(c, eff, tr.obs + (int64_t)d.T * slab, d.N, w, false, nullptr, nullptr, tr.last_value, s);
}

// ---- greedy evaluation block ---------------------------------------------------------------------------

namespace {

__global__ void eval_zero_kernel(marl_eval_stats out, int N) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n < N) {
    out.ret_sum[n] = 0.f;
    out.len_sum[n] = 0;
    out.episodes[n] = 0;
  }
}

// action = index of the largest logit, lowest index on exact ties
__global__ void __launch_bounds__(256) greedy_kernel(const float* __restrict__ logits, int32_t* __restrict__ action, int64_t S) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= S) return;
  int best = 0;
  float top = logits[i * kActions];
#pragma unroll
  for (int k = 1; k < kActions; ++k) {
    const float v = logits[i * kActions + k];
    if (v > top) {
      top = v;
      best = k;
    }
  }
  action[i] = best;
}

// Books one step into the statistics of the environments that are still inside their first n_episodes episodes:
// team reward = the agents' rewards added in ascending agent index, then added to the running sum (fp32).
__global__ void __launch_bounds__(256) eval_accumulate_kernel(const float* __restrict__ reward, const uint8_t* __restrict__ done,
                                                              marl_eval_stats out, int N, int A, int n_episodes) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const int e = out.episodes[n];
  if (e >= n_episodes) return;
  float team = 0.f;
  for (int a = 0; a < A; ++a) team += reward[(int64_t)n * A + a];
  out.ret_sum[n] += team;
  out.len_sum[n] += 1;
  if (done[n]) out.episodes[n] = e + 1;
}

struct EvalWsView {
  void* rollout_ws;
  float *obs, *logits, *reward;
  int32_t* action;
  uint8_t* done;
  EvalEpisodes eps;  // slots: as many as there is room for
};
// Episodes of an environment that there is room for: sixteen, and more while that is 32 768 of all environments together (2.2 MB, 4.3 with more than four
// agents or food; four times that at 8192 environments, the most that go side by side).  A block takes half of them at most, because the
// rows play the block's steps, however many episodes these are: enough where episodes last half as long as they may.
inline int eval_slots(int N) { return std::max(16, 32768 / N); }

EvalWsView carve_eval_ws(const marl_config& c, void* ws, int64_t* total) {
  const Dims d = dims_of(c);
  char* p = static_cast<char*>(ws);
  int64_t off = 0;
  auto take = [&](int64_t bytes) {
    char* r = p + off;
    off += align256(bytes);
    return r;
  };
  EvalWsView v;
  v.rollout_ws = take(rollout_workspace_bytes(c, d.N));
  v.obs = (float*)take(d.NA * d.D * 4);
  v.logits = (float*)take(d.NA * kActions * 4);
  v.reward = (float*)take(d.NA * 4);
  v.action = (int32_t*)take(d.NA * 4);
  v.done = (uint8_t*)take(d.N);
  v.eps = EvalEpisodes{};
  v.eps.slots = use_fused_rollout(c) && rollout_eval_places(d.Ha, d.A, d.F, d.V) / d.N >= 2 ? eval_slots(d.N) : 0;
  v.eps.len = (int32_t*)take((int64_t)v.eps.slots * d.N * 4);
  v.eps.record = (uint32_t*)take((int64_t)v.eps.slots * d.N * eval_record_words(std::max(d.A, d.F)) * 4);
  v.eps.next = (int32_t*)take(v.eps.slots > 0 ? (int64_t)d.N * 4 : 0);
  if (total) *total = off;
  return v;
}

}  // namespace

int64_t eval_workspace_bytes(const marl_config& c) {
  int64_t total = 0;
  carve_eval_ws(c, nullptr, &total);
  return total;
}

int32_t launch_evaluate(const marl_config& c, marl_env_state st, const float* params, int32_t n_episodes,
                        marl_eval_stats out, void* workspace, hipStream_t s) {
  const Dims d = dims_of(c);
  const EvalWsView e = carve_eval_ws(c, workspace, nullptr);
  const RolloutWsView w = carve_rollout_ws(c, d.N, e.rollout_ws, nullptr);
  const int copies = 2 * (int64_t)n_episodes <= e.eps.slots ? rollout_eval_copies(d.Ha, d.A, d.F, d.V, d.N, n_episodes) : 0;
  const float* eff = stage_working_copy(c, params, w.eff_params, s, USE_FORWARD, COPY_SPLIT, e.eps.next, copies > 0 ? d.N : 0);
  const int64_t steps = (int64_t)n_episodes * c.episode_cap;
  if (use_fused_rollout(c)) {  // the whole block in one launch, or in two (rollout_eval.h), statistics in registers
    RolloutArgs a = rollout_fused_args(c, st, eff);
    a.T = (int)steps;
    a.ev = out;
    a.n_episodes = n_episodes;
    if (copies > 0) {
      a.eps = e.eps;
      a.eps.copies = copies;
      a.eps.idle = std::max(0, (copies - n_episodes) / 4);
      a.eps.steps = (int)((steps + copies - a.eps.idle - 1) / (copies - a.eps.idle));
      a.eps.every = (c.episode_cap + 2) / 3;
      const int32_t rc = launch_rollout_fused(c, true, a, s);
      if (rc != MARL_OK) return rc;
      a.eps.copies = 0;
    }
    return launch_rollout_fused(c, true, a, s);
  }
  const unsigned nb_env = (unsigned)((d.N + 255) / 256), nb_s = (unsigned)((d.NA + 255) / 256);
  hipLaunchKernelGGL(eval_zero_kernel, dim3(nb_env), dim3(256), 0, s, out, d.N);
  int32_t rc = launch_env_step(c, st, nullptr, e.obs, nullptr, nullptr, /*do_step=*/false, s);
  if (rc != MARL_OK) return rc;
  for (int64_t t = 0; t < steps; ++t) {
    rc = forward_rows(c, eff, e.obs, d.N, w, true, e.logits, nullptr, nullptr, s);
    if (rc != MARL_OK) return rc;
    hipLaunchKernelGGL(greedy_kernel, dim3(nb_s), dim3(256), 0, s, e.logits, e.action, d.NA);
    rc = launch_env_step(c, st, e.action, e.obs, e.reward, e.done, true, s);
    if (rc != MARL_OK) return rc;
    hipLaunchKernelGGL(eval_accumulate_kernel, dim3(nb_env), dim3(256), 0, s, e.reward, e.done, out, d.N, d.A, (int)n_episodes);
  }
  return launch_status();
}

}  // namespace marl
