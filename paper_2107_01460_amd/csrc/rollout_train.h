// The whole training rollout as ONE kernel: a workgroup owns a block of environments for all T time steps.
//
// Environments never interact and the parameters are constant during a rollout, so nothing has to be exchanged between
// workgroups: each keeps the state of its BM / A environments in the registers of one lane per env-agent, paints the
// agents' observation windows straight into the LDS tile that is the A operand of the actor's first layer, runs both
// hidden layers on the matrix cores (weights in operand order from the L2), the output layer and the Gumbel-max sampling on
// the ALUs, hands the actions to the env lanes through cross-lane reads, resolves the transition in registers, and paints
// the next observation -- only the trajectory (observations, actions, log-probabilities, rewards, dones) is streamed out.
// The critic's values do not steer the rollout and are computed in one pass over the stored observations afterwards.
//
// The products run on the fp32 instruction for every number of environments: a sampled action is a discrete choice, and with one arithmetic
// below some number of environments and another one above, an environment's run would depend on how many others share the launch.  (On split bf16
// operands as in rollout_eval.h, 128 steps of 3072 samples at 128 units took 0.83 ms where tiles of 32 samples took 1.02; tiles of 16 on the
// fp32 instruction, the same bits as 32, take 0.77.)
#pragma once
#include "rollout_common.h"

namespace marl {

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

// All B fragments of one product against weights, for this lane: KG groups of 16 along k, two 16-byte buffer loads each
// (ParamMap; lane_off is this lane's offset (hi * LDB + n) * 4 in floats).  The whole set is requested one phase ahead of the
// product that uses it.
template <int KG>
struct PhaseW32 {
  float4 w[KG][2];
};
template <int LDB, int KG>
__device__ __forceinline__ void phase_w32_request(PhaseW32<KG>& pw, WeightRsrc B, int lane_off) {
#pragma unroll
  for (int g = 0; g < KG; ++g)
#pragma unroll
    for (int u = 0; u < 2; ++u)
      pw.w[g][u] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(B, lane_off * 4, (16 * g + 8 * u) * LDB * 4, 0));
}
// acc += A B for this wavefront's 32x32 tile: A rows in LDS (As points at this lane's row, + 4 * hi; the fragments of
// the next group are read before the matrix instructions of the current one), B from pw.
template <int KG>
__device__ __forceinline__ void gemm_phase_w32(const float* __restrict__ As, floatx16& acc, const PhaseW32<KG>& pw) {
  float4 av[2][2];
  av[0][0] = *reinterpret_cast<const float4*>(As);
  av[0][1] = *reinterpret_cast<const float4*>(As + 8);
#pragma unroll
  for (int g = 0; g < KG; ++g) {
    const int gn = g + 1 < KG ? g + 1 : g;
    av[(g + 1) & 1][0] = *reinterpret_cast<const float4*>(As + 16 * gn);
    av[(g + 1) & 1][1] = *reinterpret_cast<const float4*>(As + 16 * gn + 8);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float af[4] = {av[g & 1][u].x, av[g & 1][u].y, av[g & 1][u].z, av[g & 1][u].w};
      const float bf[4] = {pw.w[g][u].x, pw.w[g][u].y, pw.w[g][u].z, pw.w[g][u].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[j], bf[j], acc, 0, 0, 0);
    }
  }
}

// The same for tiles of 16 samples, on v_mfma_f32_16x16x4_f32: NT column tiles of this wavefront, one 16-byte load each per group of 16 along k.  A chain of
// either instruction is a chain of fused multiply-adds in the order of its k, and the order here is the one above -- k, k + 4, k + 1, k + 5, ... of
// every eight -- so that a sample's sums have the same bits in tiles of either height.  A lane (quarter q of the wavefront) has k = step16_first(q) + 2 h of eight
// in the h-th of their two instructions; the weights' copy has those four of every 16 beside one another (rollout_order16).
__device__ __forceinline__ int step16_first(int q) { return 4 * (q & 1) + (q >> 1); }
template <int KG, int NT>
struct PhaseW16 {
  float4 w[KG][NT];
};
template <int LDB, int KG, int NT>
__device__ __forceinline__ void phase_w16_request(PhaseW16<KG, NT>& pw, WeightRsrc B, int lane_off) {
#pragma unroll
  for (int g = 0; g < KG; ++g)
#pragma unroll
    for (int c = 0; c < NT; ++c)
      pw.w[g][c] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(B, lane_off * 4, 16 * g * LDB * 4 + 16 * c * 16, 0));
}
// As points at this lane's row, + step16_first(q)
template <int KG, int NT>
__device__ __forceinline__ void gemm_phase_w16(const float* __restrict__ As, floatx4 (&acc)[NT], const PhaseW16<KG, NT>& pw) {
  float av[2][4];
  auto read = [&](int g) {
#pragma unroll
    for (int e = 0; e < 4; ++e) av[g & 1][e] = As[16 * g + 8 * (e / 2) + 2 * (e % 2)];
  };
  read(0);
#pragma unroll
  for (int g = 0; g < KG; ++g) {
    if (g + 1 < KG) read(g + 1);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int c = 0; c < NT; ++c) {
        const float4 w = pw.w[g][c];
        acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[g & 1][e], e == 0 ? w.x : e == 1 ? w.y : e == 2 ? w.z : w.w, acc[c], 0, 0, 0);
      }
  }
}

// pitch of a window in LDS, in floats: a multiple of four, with an odd number of 16-byte units
constexpr int rollout_train_px(int D) { return (D + 15) / 16 * 16 + 4; }

// OCC: workgroups per CU the registers are capped for
template <int H, int BM, int V, int CA, int KIND, int OCC>
__global__ void __launch_bounds__(256, OCC) rollout_train_kernel(RolloutArgs a) {
  constexpr int D = 3 * V * V, PX = rollout_train_px(D), KPAD = (D + 15) / 16 * 16, PH = H + 4, GROUPS = H / 16, NOUT = kActions;
  constexpr bool SMALL = BM == 16;  // 16 x 16 tiles, H / 64 per wavefront
  constexpr int NTN = H / 32, NT16 = H / 64;
  static_assert(SMALL || BM / 32 * NTN == 4, "one 32x32 MFMA tile per wavefront");
  static_assert(SMALL || GROUPS == 256 / BM, "one thread per sample and share of 16 units");
  extern __shared__ __attribute__((aligned(16))) float lds[];
  float* const Xs2 = lds;                      // [2][BM][PX]  observation windows of two consecutive steps, k-contiguous;
                                               //              columns D .. PX stay zero
  float* const Hs = Xs2 + 2 * BM * PX;         // [BM][PH]  h1, then h2
  float* const red = Hs + BM * PH;             // [GROUPS][BM][NOUT]
  float* const W3s = red + GROUPS * BM * NOUT; // [H][NOUT]
  float* const noise = W3s + H * NOUT;         // [2][BM][8] log(-log u) of the step's uniforms, two steps alternating

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lo = lane & 31, hi = lane >> 5;
  const int mt = wave / NTN, nt = wave % NTN;
  const int l15 = lane & 15, l4 = lane >> 4;
  RolloutEnvs<BM, V, CA, KIND> env(a, wave, lane);
  const int64_t NA = (int64_t)a.p.N * a.p.A;
  // ---- the other three wavefronts draw the sampling noise of the NEXT step while the env lanes work: it depends on
  // (step, sample) only.  Thread j of them: sample slot j % BM, Philox call j / BM (call 0: actions 0..3, call 1: 4, 5).
  const int nz_s = env.other % BM, nz_call = env.other / BM;
  const bool nz_on = !env.is_env_wave && nz_call < 2 && nz_s < env.samples_here;
  const uint64_t step_base = (a.step_base != nullptr) ? *a.step_base : 0;

  auto draw_noise = [&](int t) {  // noise of step t into buffer t & 1
    if (!nz_on) return;
    float* const dst = noise + ((t & 1) * BM + nz_s) * 8 + 4 * nz_call;
    const int64_t s = env.env0 * env.A + nz_s;
    float u[4];
    if (a.uniforms) {
      const float* src = a.uniforms + ((int64_t)t * NA + s) * NOUT + 4 * nz_call;
#pragma unroll
      for (int k = 0; k < 4; ++k) u[k] = (4 * nz_call + k < NOUT) ? src[k] : 0.5f;
    } else {
      const uint64_t step = a.step0 + step_base + (uint64_t)t;
      uint32_t o[4];
      philox4x32_10((uint32_t)step, (uint32_t)(step >> 32), (uint32_t)s * 2u + (uint32_t)nz_call, kStreamSample, a.p.k0, a.p.k1, o);
#pragma unroll
      for (int k = 0; k < 4; ++k) u[k] = rand_unit(o[k]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) dst[k] = logf(-logf(u[k]));  // the same fp32 operations as the per-step sampler
  };

  GroupCopy<H * NOUT, 256> w3;
  w3.request(tid, a.W3);
  for (int i = tid; i < 2 * BM * PX; i += 256) Xs2[i] = 0.f;  // padding columns and unused rows stay zero for good
  if (env.is_env_wave) env.load();
  w3.store(tid, [&](int e, float v) { W3s[e] = v; });
  __syncthreads();
  if (env.active) env.paint(Xs2 + lane * PX);
  if (a.T > 0) draw_noise(0);
  // the biases of this lane's column and of the output layer stay in registers for all T steps
  constexpr int NB = SMALL ? NT16 : 1;
  float bias1[NB], bias2[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) {
    const int n = SMALL ? 16 * (wave * NT16 + c) + l15 : nt * 32 + lo;
    bias1[c] = a.b1[n];
    bias2[c] = a.b2[n];
  }
  float b3r[NOUT];
#pragma unroll
  for (int k = 0; k < NOUT; ++k) b3r[k] = a.b3[k];
  // The windows of step t sit in tile t & 1: while the env lanes paint the windows of step t + 1 into the other tile, the
  // wavefronts that are idle then copy tile t & 1 out as slab t of the trajectory.  Thread j of them (0 .. 191).
  auto store_slab = [&](int t, int j, int nthreads) {
    const float* const Xt = Xs2 + (t & 1) * BM * PX;
    float* const out = a.obs + ((int64_t)t * a.p.N + env.env0) * env.A * D;
    const int count = env.samples_here * D;
    for (int i = j; i < count; i += nthreads) {
      const int r = i / D, c = i - r * D;
      out[i] = Xt[r * PX + c];
    }
  };

  // the weights of a whole layer are requested a phase ahead (buffer loads: one descriptor, one lane offset)
  constexpr int KG1 = KPAD / 16, KG2 = H / 16;
  const int wlane = SMALL ? (l4 * H + 16 * wave * NT16 + l15) * 4 : (hi * H + nt * 32 + lo) * 4;
  const WeightRsrc rsW1 = weight_rsrc(a.W1, KPAD * H), rsW2 = weight_rsrc(a.W2, H * H);
  std::conditional_t<SMALL, PhaseW16<KG1, NT16>, PhaseW32<KG1>> pw1;
  std::conditional_t<SMALL, PhaseW16<KG2, NT16>, PhaseW32<KG2>> pw2;
  auto request1 = [&]() {
    if constexpr (SMALL) phase_w16_request<H>(pw1, rsW1, wlane);
    else phase_w32_request<H, KG1>(pw1, rsW1, wlane);
  };
  auto request2 = [&]() {
    if constexpr (SMALL) phase_w16_request<H>(pw2, rsW2, wlane);
    else phase_w32_request<H, KG2>(pw2, rsW2, wlane);
  };
  floatx16 acc;
  floatx4 acc16[NT16];
  // this wavefront's part of A (rows of pitch `pitch`) times the weights in pw
  auto product = [&](const float* A, int pitch, const auto& pw) {
    if constexpr (SMALL) {
#pragma unroll
      for (int c = 0; c < NT16; ++c) acc16[c] = floatx4{0.f, 0.f, 0.f, 0.f};
      gemm_phase_w16(A + l15 * pitch + step16_first(l4), acc16, pw);
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
      gemm_phase_w32(A + (mt * 32 + lo) * pitch + 4 * hi, acc, pw);
    }
  };
  auto store_tanh = [&](const float (&bias)[NB]) {  // -> Hs
    if constexpr (SMALL) {
#pragma unroll
      for (int c = 0; c < NT16; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) Hs[(4 * l4 + r) * PH + 16 * (wave * NT16 + c) + l15] = tanh_f32(acc16[c][r] + bias[c]);
    } else {
      const int col = nt * 32 + lo;
#pragma unroll
      for (int r = 0; r < 16; ++r) Hs[(mt * 32 + 8 * (r / 4) + 4 * hi + (r % 4)) * PH + col] = tanh_f32(acc[r] + bias[0]);
    }
  };
  request1();
  for (int t = 0;; ++t) {
    loop_head_barrier();  // the windows (and the noise) of step t are complete
    if (t == a.T) {
      store_slab(t, tid, 256);  // the post-rollout observation
      break;
    }
    const float* const Xs = Xs2 + (t & 1) * BM * PX;
    // ---- layer 1: h1 = tanh(X W1 + b1) -> LDS
    product(Xs, PX, pw1);
    request2();  // layer 2's weights arrive during the tanh of layer 1
    store_tanh(bias1);
    __syncthreads();  // h1 complete; every wavefront is past its reads of the windows
    // ---- layer 2: h2 = tanh(h1 W2 + b2)
    product(Hs, PH, pw2);
    request1();  // layer 1 of the next step
    __syncthreads();  // every wavefront is past its last read of h1
    store_tanh(bias2);
    __syncthreads();
    // ---- output layer on the ALUs: thread -> (sample tid % BM, 16 of the hidden units and, in small tiles, some of the outputs)
    {
      constexpr int SPLIT = !SMALL ? 1 : GROUPS == 8 ? 2 : 3, KO = NOUT / SPLIT, PER = 16;
      const int s = tid % BM, grp = tid / BM % GROUPS, k0 = tid / (BM * GROUPS) * KO;
      if (!SMALL || k0 < NOUT) {
        float part[KO];
#pragma unroll
        for (int k = 0; k < KO; ++k) part[k] = 0.f;
#pragma unroll 2
        for (int i = grp * PER; i < (grp + 1) * PER; i += 4) {
          const float4 hv = *reinterpret_cast<const float4*>(&Hs[s * PH + i]);
          const float hh[4] = {hv.x, hv.y, hv.z, hv.w};
          float wv[4 * KO];
          if constexpr (!SMALL) {
#pragma unroll
            for (int q = 0; q < KO; ++q) {
              const float4 w4 = *reinterpret_cast<const float4*>(&W3s[i * NOUT + 4 * q]);
              wv[4 * q] = w4.x; wv[4 * q + 1] = w4.y; wv[4 * q + 2] = w4.z; wv[4 * q + 3] = w4.w;
            }
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
              for (int k = 0; k < KO; ++k) wv[j * KO + k] = W3s[(i + j) * NOUT + k0 + k];
          }
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int k = 0; k < KO; ++k) part[k] = fmaf(hh[j], wv[j * KO + k], part[k]);
        }
        if constexpr (!SMALL) {
#pragma unroll
          for (int k = 0; k < NOUT; k += 2) *reinterpret_cast<float2*>(&red[(grp * BM + s) * NOUT + k]) = make_float2(part[k], part[k + 1]);
        } else {
#pragma unroll
          for (int k = 0; k < KO; ++k) red[(grp * BM + s) * NOUT + k0 + k] = part[k];
        }
      }
    }
    __syncthreads();
    if (!env.is_env_wave) {
      if (t + 1 < a.T) draw_noise(t + 1);
      store_slab(t, env.other, 192);
    } else {
      // ---- the env lanes: logits -> action -> transition -> next window
      const int row = lane < BM ? lane : 0;
      float lg[NOUT];
      static_assert(NOUT % 2 == 0, "shares are read two at a time");
#pragma unroll
      for (int k = 0; k < NOUT; ++k) lg[k] = b3r[k];
#pragma unroll
      for (int gq = 0; gq < GROUPS; ++gq)
#pragma unroll
        for (int k = 0; k < NOUT; k += 2) {
          const float2 v = *reinterpret_cast<const float2*>(&red[(gq * BM + row) * NOUT + k]);
          lg[k] += v.x;
          lg[k + 1] += v.y;
        }
      // Where this step's records of the workgroup begin, and a lane's place there that the compiler does not know from before: otherwise it keeps a 64-bit
      // address of each array and lane across the steps, one of them in scratch memory, whose reload waited for all stores before it, 2000 cycles a step.
      const int64_t sample0 = (int64_t)t * NA + env.env0 * env.A, env_row0 = (int64_t)t * a.p.N + env.env0;
      uint32_t at = lane, at_env = env.le;
      asm volatile("" : "+v"(at), "+v"(at_env));
      int my_act = 0;
      if (env.active) {
        if (a.logits) {
#pragma unroll
          for (int k = 0; k < NOUT; ++k) (a.logits + sample0 * NOUT)[at * NOUT + k] = lg[k];
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
        if (a.sampled) (a.sampled + sample0)[at] = my_act;
        if (a.forced) {
          my_act = (a.forced + sample0)[at];
          asm volatile("" : "+v"(my_act));  // waited for here, not behind the branch
        }
        (a.action + sample0)[at] = my_act;
        (a.logp + sample0)[at] = log_softmax_fast(lg, my_act);
      }
      float rew;
      bool dn;
      env.step(my_act, rew, dn);
      if (env.active) {
        (a.reward + sample0)[at] = rew;
        if (env.ai == 0) (a.done + env_row0)[at_env] = dn ? 1 : 0;
        env.paint(Xs2 + ((t + 1) & 1) * BM * PX + lane * PX);  // the windows of step t + 1 into the other tile
      }
    }
  }
  if (env.active) env.store();
}

}  // namespace marl
