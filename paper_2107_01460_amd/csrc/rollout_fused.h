// The whole rollout as ONE kernel: a workgroup owns a block of environments for all T time steps.
//
// Environments never interact and the parameters are constant during a rollout, so nothing has to be exchanged
// between workgroups: each keeps the state of its BM / A environments in the registers of one lane per env-agent,
// paints the agents' observation windows straight into the LDS tile that is the A operand of the actor's first
// layer, runs both hidden layers on the matrix cores (weights from the operand-order copies in L2, as in
// fused_forward_kernel), the output layer and the Gumbel-max sampling on the ALUs, hands the actions to the env lanes
// through cross-lane reads, resolves the transition in registers, and paints the next observation -- only the
// trajectory (observations, actions, log-probabilities, rewards, dones) is streamed out.  The critic's values do not
// steer the rollout and are computed in one pass over the stored observations afterwards.
//
// Both layers run on split bf16 operands, transposed (gemm_phase_t): the windows hold small integers and halves, exact in
// bf16, so layer 1 takes half the products, h1 is split once, and the output layer starts from the registers that layer 2
// ends in.  A step is a chain of latencies: 128 steps of 3072 samples at 128 units 0.84 ms, with fp32 tiles 1.0 ms.
//
// The same kernel with EVAL = true is the greedy evaluation block: argmax actions, no trajectory, and the
// per-environment return / length / episode counts accumulated in registers.
#pragma once
#include "env_device.h"
#include "fused_forward.h"

namespace marl {

struct RolloutFusedArgs {
  EnvParams p;
  marl_env_state st;
  const float *W1s, *W2s, *b1, *b2, *W3, *b3;  // actor: split operand-order W1 / W2, aligned biases and output layer
  const float *W1o, *W2o;  // fp32 operand-order W1 / W2 (training rollouts; ParamMap)
  int kpad1, px;           // ... rows of W1o, pitch of an fp32 window
  int T;  // steps to take
  // training rollout
  float* obs;  // [T+1][N][A][D]
  int32_t* action;
  float* logp;
  float* reward;
  uint8_t* done;
  float* logits;     // nullable
  int32_t* sampled;  // nullable
  const float* uniforms;  // nullable [T][N][A][6]
  const int32_t* forced;  // nullable [T][N][A]
  uint64_t step0;
  const uint64_t* step_base;  // nullable
  // evaluation block
  marl_eval_stats ev;
  int n_episodes;
};

// log-softmax(lg)[a] with the hardware exp2 / log2 units (a value, not a decision: the relative error of about
// 1e-6 is far inside the tolerance of a log-probability)
__device__ __forceinline__ float log_softmax_fast(const float lg[kActions], int a) {
  float m = lg[0];
#pragma unroll
  for (int k = 1; k < kActions; ++k) m = fmaxf(m, lg[k]);
  float se = 0.f, la = 0.f;
#pragma unroll
  for (int k = 0; k < kActions; ++k) {
    se += __builtin_amdgcn_exp2f((lg[k] - m) * 1.4426950408889634f);
    la = (k == a) ? lg[k] : la;
  }
  return la - m - __builtin_amdgcn_logf(se) * 0.6931471805599453f;
}

}  // namespace marl
#include "rollout_fp32.h"
namespace marl {

// pitch of a window in LDS, in elements: the width rounded up to a k group, and an odd number of 16-byte units
constexpr int rollout_fused_px(int D) { return (D + 15) / 16 * 16 + 8; }

// OCC: workgroups per CU the registers are capped for
template <int H, int BM, int V, int CA, int KIND, bool EVAL, int OCC>
__global__ void __launch_bounds__(256, OCC) rollout_fused_kernel(RolloutFusedArgs a) {
  constexpr int D = 3 * V * V, PX = rollout_fused_px(D), PH = H + 8, HPLANE = BM * PH, NOUT = kActions;
  constexpr int NTN = H / 32, MT = BM / 32, TILES = MT * NTN;
  static_assert(TILES == 4, "one 32x32 MFMA tile per wavefront");
  static_assert(BM <= 64, "the env lanes are lanes of one wavefront");
  extern __shared__ __attribute__((aligned(16))) float lds[];
  bf16_t* const Xs2 = reinterpret_cast<bf16_t*>(lds);  // [2][BM][PX]  observation windows of two consecutive steps (exact in bf16),
                                                       //              k-contiguous; columns D .. PX stay zero
  bf16_t* const Hs = Xs2 + 2 * BM * PX;                // [3][BM][PH]  h1, split
  float* const red = reinterpret_cast<float*>(Hs + 3 * HPLANE);  // [NTN][NOUT][BM] shares of the output layer
  float* const W3s = red + NTN * NOUT * BM;            // [H][NOUT]
  float* const noise = W3s + H * NOUT;                 // [2][BM][8] log(-log u) of the step's uniforms, two steps alternating
  float* const b1s = noise + 2 * BM * 8;               // [H]
  float* const b2s = b1s + H;                          // [H]

  const EnvParams& p = a.p;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lo = lane & 31, hi = lane >> 5;
  const int mt = wave / NTN, nt = wave % NTN;
  const int srow = mt * 32 + lo, u0 = nt * 32 + 4 * hi;  // this lane's sample of the tile; its units are u0 + 8 j .. + 3
  const int A = p.A, N = p.N;
  const int epw = BM / A;  // envs of this workgroup
  const int64_t env0 = (int64_t)blockIdx.x * epw;
  const int envs_here = (int)min((int64_t)epw, (int64_t)N - env0);
  const int samples_here = envs_here * A;
  const int64_t NA = (int64_t)N * A;

  // ---- env lanes: lane l < BM of ONE wavefront is agent l % A of env env0 + l / A.  Which wavefront it is rotates
  // with the workgroup index, so that the workgroups of a CU keep their serial sections on different SIMDs.
  const int env_wave = blockIdx.x & 3;
  const bool is_env_wave = wave == env_wave;
  const int le = lane / A, ai = lane - le * A;
  const bool active = is_env_wave && lane < samples_here;
  const int64_t n = env0 + le;
  const size_t nn = active ? (size_t)n : 0;
  const int64_t s_glob = env0 * A + lane;  // this env lane's sample index
  // ---- the other three wavefronts draw the sampling noise of the NEXT step while the env lanes work: it depends on
  // (step, sample) only.  Thread j of them: sample slot j % BM, Philox call j / BM (call 0: actions 0..3, call 1: 4, 5).
  const int nz_j = ((wave - env_wave - 1) & 3) * 64 + lane;
  const bool nz_on = !EVAL && !is_env_wave && nz_j < 2 * BM && (nz_j % BM) < samples_here;
  const int nz_s = nz_j % BM, nz_call = nz_j / BM;
  uint32_t ag[CA], fd[CA];
  int t_ep = 0;
  uint32_t episode = 0;
  float ret_sum = 0.f;
  int len_sum = 0, episodes = 0;
  const uint64_t step_base = (!EVAL && a.step_base != nullptr) ? *a.step_base : 0;

  auto draw_noise = [&](int t) {  // noise of step t into buffer t & 1
    if (!nz_on) return;
    float* const dst = noise + ((t & 1) * BM + nz_s) * 8 + 4 * nz_call;
    const int64_t s = env0 * A + nz_s;
    float u[4];
    if (a.uniforms) {
      const float* src = a.uniforms + ((int64_t)t * NA + s) * NOUT + 4 * nz_call;
#pragma unroll
      for (int k = 0; k < 4; ++k) u[k] = (4 * nz_call + k < NOUT) ? src[k] : 0.5f;
    } else {
      const uint64_t step = a.step0 + step_base + (uint64_t)t;
      uint32_t o[4];
      philox4x32_10((uint32_t)step, (uint32_t)(step >> 32), (uint32_t)s * 2u + (uint32_t)nz_call, kStreamSample, p.k0, p.k1, o);
#pragma unroll
      for (int k = 0; k < 4; ++k) u[k] = rand_unit(o[k]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) dst[k] = logf(-logf(u[k]));  // the same fp32 operations as the per-step sampler
  };

  for (int i = tid; i < H * NOUT; i += 256) W3s[i] = a.W3[i];
  for (int i = tid; i < H; i += 256) {
    b1s[i] = a.b1[i];
    b2s[i] = a.b2[i];
  }
  for (int i = tid; i < BM * PX; i += 256) reinterpret_cast<uint32_t*>(Xs2)[i] = 0u;  // padding columns and unused rows stay zero for good
  if (is_env_wave) {
    load_env_state<CA, CA, KIND>(ag, fd, a.st, p, nn, active);
    t_ep = a.st.t_in_ep[nn];
    episode = a.st.episode_id[nn];
  }
  __syncthreads();
  if (active) {
    if (KIND == 0) forage_paint<V, CA, CA>(Xs2 + lane * PX, ag, fd, ai, p);
    else wh_paint<V, CA, CA>(Xs2 + lane * PX, ag, fd, ai, p);
  }
  if (a.T > 0) draw_noise(0);
  // the output layer's bias stays in registers for all T steps
  float b3r[NOUT];
#pragma unroll
  for (int k = 0; k < NOUT; ++k) b3r[k] = a.b3[k];
  // The windows of step t sit in tile t & 1: while the env lanes paint the windows of step t + 1 into the other tile, the
  // wavefronts that are idle then copy tile t & 1 out as slab t of the trajectory.  Thread j of them (0 .. 191).
  auto store_slab = [&](int t, int j, int nthreads) {
    const bf16_t* const Xt = Xs2 + (t & 1) * BM * PX;
    float* const out = a.obs + ((int64_t)t * N + env0) * A * D;
    const int count = samples_here * D;
    for (int i = j; i < count; i += nthreads) {
      const int r = i / D, c = i - r * D;
      out[i] = from_bf16(Xt[r * PX + c]);
    }
  };

  // the first weights of a layer are requested a phase ahead (buffer loads: one descriptor, one lane offset)
  constexpr int KG1 = (D + 15) / 16, KG2 = H / 16;
  const int wlane = (hi * H + nt * 32 + lo) * 4;
  const WeightRsrc rsW1 = split_weight_rsrc(a.W1s, 16 * KG1, H), rsW2 = split_weight_rsrc(a.W2s, H, H);
  PhaseW<KG1> pw1;
  phase_w_request<H, KG1>(pw1, rsW1, wlane, KG1);
  for (int t = 0;; ++t) {
    __syncthreads();  // the windows (and the noise) of step t are complete
    if (t == a.T) {
      if (!EVAL) store_slab(t, tid, 256);  // the post-rollout observation
      break;
    }
    const bf16_t* const Xs = Xs2 + (t & 1) * BM * PX;
    int uw = u0;  // the weights and biases in LDS are read in every step: kept across steps, they would take 96 registers
    asm volatile("" : "+v"(uw));
    // ---- layer 1: h1 = tanh(X W1 + b1) -> LDS.  Both layers are computed transposed (gemm_phase_t).
    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    gemm_phase_t<H, KG1, true>(Xs + srow * PX + 8 * hi, 0, rsW1, wlane, KG1, acc, pw1);
    PhaseW<KG2> pw2;  // layer 2's weights arrive during the tanh of layer 1
    phase_w_request<H, KG2>(pw2, rsW2, wlane, KG2);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float4 bs = *reinterpret_cast<const float4*>(&b1s[uw + 8 * j]);
      store_split4<false>(&Hs[srow * PH + u0 + 8 * j], HPLANE,
                          make_float4(tanh_f32(acc[4 * j] + bs.x), tanh_f32(acc[4 * j + 1] + bs.y), tanh_f32(acc[4 * j + 2] + bs.z), tanh_f32(acc[4 * j + 3] + bs.w)));
    }
    __syncthreads();  // h1 complete; every wavefront is past its reads of the windows
    // ---- layer 2: h2 = tanh(h1 W2 + b2), and this wavefront's units' share of the output layer
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    gemm_phase_t<H, KG2, false>(Hs + srow * PH + 8 * hi, HPLANE, rsW2, wlane, KG2, acc, pw2);
    phase_w_request<H, KG1>(pw1, rsW1, wlane, KG1);  // layer 1 of the next step
    {
      float part[NOUT];
#pragma unroll
      for (int k = 0; k < NOUT; ++k) part[k] = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float4 bs = *reinterpret_cast<const float4*>(&b2s[uw + 8 * j]);
        const float h[4] = {tanh_f32(acc[4 * j] + bs.x), tanh_f32(acc[4 * j + 1] + bs.y), tanh_f32(acc[4 * j + 2] + bs.z), tanh_f32(acc[4 * j + 3] + bs.w)};
        float wv[4 * NOUT];
#pragma unroll
        for (int q = 0; q < NOUT; ++q) {
          const float4 w4 = *reinterpret_cast<const float4*>(&W3s[(uw + 8 * j) * NOUT + 4 * q]);
          wv[4 * q] = w4.x; wv[4 * q + 1] = w4.y; wv[4 * q + 2] = w4.z; wv[4 * q + 3] = w4.w;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int k = 0; k < NOUT; ++k) part[k] = fmaf(h[e], wv[e * NOUT + k], part[k]);
        __builtin_amdgcn_sched_barrier(0);  // one quarter's weights in registers at a time
      }
#pragma unroll
      for (int k = 0; k < NOUT; ++k) {
        const float v = part[k] + __shfl_xor(part[k], 32);
        if (hi == 0) red[(nt * NOUT + k) * BM + srow] = v;
      }
    }
    __syncthreads();
    if (!is_env_wave) {
      if (t + 1 < a.T) draw_noise(t + 1);
      if (!EVAL) store_slab(t, ((wave - env_wave - 1) & 3) * 64 + lane, 192);
    } else {
      // ---- the env lanes: logits -> action -> transition -> next window.  The whole wavefront runs this, so that the
      // cross-lane reads below find their source lanes running.
      const int row = lane < BM ? lane : 0;
      float lg[NOUT];
#pragma unroll
      for (int k = 0; k < NOUT; ++k) {
        float v = b3r[k];
#pragma unroll
        for (int q = 0; q < NTN; ++q) v += red[(q * NOUT + k) * BM + row];
        lg[k] = v;
      }
      int my_act = 0;
      if (active) {
        if (EVAL) {  // largest logit, lowest index on exact ties
          float top = lg[0];
#pragma unroll
          for (int k = 1; k < NOUT; ++k)
            if (lg[k] > top) {
              top = lg[k];
              my_act = k;
            }
        } else {
          const int64_t o = (int64_t)t * NA + s_glob;
          if (a.logits) {
#pragma unroll
            for (int k = 0; k < NOUT; ++k) a.logits[o * NOUT + k] = lg[k];
          }
          // Gumbel-max: argmax_k lg[k] - log(-log u[k]), lowest k on exact ties
          const float* const g = noise + ((t & 1) * BM + lane) * 8;
          const float4 g0 = *reinterpret_cast<const float4*>(g);
          const float2 g1 = *reinterpret_cast<const float2*>(g + 4);
          const float gk[NOUT] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y};
          float best = -INFINITY;
#pragma unroll
          for (int k = 0; k < NOUT; ++k) {
            const float z = lg[k] - gk[k];
            if (z > best) {
              best = z;
              my_act = k;
            }
          }
          if (a.sampled) a.sampled[o] = my_act;
          if (a.forced) my_act = a.forced[o];
          a.action[o] = my_act;
          a.logp[o] = log_softmax_fast(lg, my_act);
        }
      }
      int act[CA];
#pragma unroll
      for (int b = 0; b < CA; ++b) {
        const int v = __shfl(my_act, min(le * A + b, 63));
        act[b] = (active && b < A) ? v : 0;
      }
      float rew;
      bool dn;
      if (KIND == 0) forage_transition<CA, CA>(ag, fd, act, ai, active, p, (uint32_t)n, t_ep, episode, rew, dn);
      else wh_transition<CA, CA>(ag, fd, act, ai, active, p, (uint32_t)n, t_ep, episode, rew, dn);
      if (EVAL) {
        // team reward = the agents' rewards added in ascending agent index, then added to the running sum (fp32)
        float team = 0.f;
#pragma unroll
        for (int b = 0; b < CA; ++b) {
          const float rb = __shfl(rew, min(le * A + b, 63));
          if (b < A) team += rb;
        }
        if (active && episodes < a.n_episodes) {
          ret_sum += team;
          len_sum += 1;
          if (dn) episodes += 1;
        }
      } else if (active) {
        a.reward[(int64_t)t * NA + s_glob] = rew;
        if (ai == 0) a.done[(int64_t)t * N + n] = dn ? 1 : 0;
      }
      if (active) {  // the windows of step t + 1 into the other tile
        bf16_t* const Xn = Xs2 + ((t + 1) & 1) * BM * PX;
        if (KIND == 0) forage_paint<V, CA, CA>(Xn + lane * PX, ag, fd, ai, p);
        else wh_paint<V, CA, CA>(Xn + lane * PX, ag, fd, ai, p);
      }
    }
  }
  if (active) {
    store_env_state<CA, CA, KIND>(ag, fd, a.st, p, (size_t)n, ai, /*dn=*/true, t_ep, episode);
    if (EVAL && ai == 0) {
      a.ev.ret_sum[n] = ret_sum;
      a.ev.len_sum[n] = len_sum;
      a.ev.episodes[n] = episodes;
    }
  }
}

// Networks and views the kernel is instantiated for: hidden width 64 (64-sample tiles) or 128 (32-sample tiles).
inline bool rollout_fused_supported(int H, int A) { return (H == 64 || H == 128) && A <= 8; }
// Workgroups up to which a training rollout is a chain of latencies (two per CU); beyond, rollout_fp32_kernel.
constexpr unsigned kRolloutSplitGrid = 512;
inline int rollout_fused_bm(int H) { return H == 64 ? 64 : 32; }

template <int H, int BM, int V, int CA, int KIND, bool EVAL, int OCC = (CA <= 4 && V <= 5) ? 2 : 1>
inline int32_t launch_rollout_fused_inst(const RolloutFusedArgs& a, hipStream_t s) {
  const int epw = BM / a.p.A;
  const unsigned grid = (unsigned)((a.p.N + epw - 1) / epw);
  if constexpr (!EVAL) {
    if (grid > kRolloutSplitGrid) {
      auto kern32 = rollout_fp32_kernel<H, BM, V, CA, KIND, ((H == 64 && CA <= 2) || (CA <= 4 && V <= 5)) ? 3 : 1>;
      const size_t bytes32 = (2 * (size_t)BM * a.px + (size_t)BM * (H + 4) + 256 * (size_t)kActions + (size_t)H * kActions + 2 * BM * 8) * sizeof(float);
      if (bytes32 > 64 * 1024 &&
          hipFuncSetAttribute(reinterpret_cast<const void*>(kern32), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
        return MARL_E_LAUNCH;
      hipLaunchKernelGGL(kern32, dim3(grid), dim3(256), bytes32, s, a);
      return launch_status();
    }
  }
  auto kern = rollout_fused_kernel<H, BM, V, CA, KIND, EVAL, OCC>;
  const size_t bytes = 2 * (size_t)BM * (2 * rollout_fused_px(3 * V * V) + 3 * (H + 8)) + sizeof(float) * ((H / 32) * kActions * BM + H * kActions + 2 * BM * 8 + 2 * H);
  static bool configured = false;  // per instantiation
  if (!configured) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
      return MARL_E_LAUNCH;
    configured = true;
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), bytes, s, a);
  return launch_status();
}

template <int V, int KIND, bool EVAL>
inline int32_t launch_rollout_fused_view(int H, const RolloutFusedArgs& a, hipStream_t s) {
  const int cap = a.p.A > a.p.F ? a.p.A : a.p.F;  // every loop over entities is unrolled to the capacity
  if constexpr (V == 3 && KIND == 0) {  // the small foraging shape (two agents, one food): half the unrolled entity loops
    if (cap <= 2 && H == 64) return launch_rollout_fused_inst<64, 64, V, 2, KIND, EVAL>(a, s);
  }
  if (H == 64) {
    if (cap <= 4) return launch_rollout_fused_inst<64, 64, V, 4, KIND, EVAL>(a, s);
    return launch_rollout_fused_inst<64, 64, V, 8, KIND, EVAL>(a, s);
  }
  if (cap <= 4) return launch_rollout_fused_inst<128, 32, V, 4, KIND, EVAL>(a, s);
  return launch_rollout_fused_inst<128, 32, V, 8, KIND, EVAL>(a, s);
}

// Defined in rollout_v3.hip / rollout_v5.hip / rollout_v7.hip (one translation unit per view size).
int32_t launch_rollout_fused_v3(int H, bool eval, const RolloutFusedArgs& a, hipStream_t s);
int32_t launch_rollout_fused_v5(int H, bool eval, const RolloutFusedArgs& a, hipStream_t s);
int32_t launch_rollout_fused_v7(int H, bool eval, const RolloutFusedArgs& a, hipStream_t s);

template <int V>
inline int32_t launch_rollout_fused_tu(int H, bool eval, const RolloutFusedArgs& a, hipStream_t s) {
  if (a.p.kind == 0) {
    if (eval) return launch_rollout_fused_view<V, 0, true>(H, a, s);
    return launch_rollout_fused_view<V, 0, false>(H, a, s);
  }
  if (eval) return launch_rollout_fused_view<V, 1, true>(H, a, s);
  return launch_rollout_fused_view<V, 1, false>(H, a, s);
}

}  // namespace marl
