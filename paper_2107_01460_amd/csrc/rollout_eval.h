// The greedy evaluation block as ONE kernel, as rollout_train.h: argmax actions, no trajectory, and the per-environment
// return / length / episode counts accumulated in registers.
//
// Both layers run on split bf16 operands, transposed (gemm_phase_t): the windows hold small integers and halves, exact in
// bf16, so layer 1 takes half the products, h1 is split once, and the output layer starts from the registers that layer 2
// ends in.  A step is a chain of latencies: 200 steps of 384 samples at 128 units 1.2 ms, with fp32 tiles 1.48 ms.
//
// An environment's next episode starts from a layout that depends on the seed, the environment and the episode's number alone.  So while
// the chip has room, the block's episodes are played beside one another in a first launch (EvalEpisodes): the rows of an environment take them in order,
// the counted ones and those behind them, until they have taken as many steps as the block has.  A second launch adds the counted ones up in the order of
// time, finds the episode that the block's last step falls into and plays that one's part, from the third of it that was put down: nothing where every
// episode lasts as long as it may.  R rows take n episodes' steps in a chain of n / R + 1 caps at most, and a third behind it.  Of 2 n rows n / 4 may end early
// without another episode that may take a cap from there on, so that a few early ends cost nothing.
// Four episodes of 50 steps as above: 296 us in place of 1200.  Where episodes end early, in one chain / side by side: 128 environments, five robots, 60
// steps at most, 44 .. 47 on average, 128 units, two episodes 1340 / 1130, four 2670 / 1150, eight 5330 / 1090.  (Rows for the counted episodes alone, with
// the rest of the block in the second launch: 1850, 2430 and 3940.)
#pragma once
#include "rollout_common.h"

namespace marl {

// pitch of a window in LDS, in elements: the width rounded up to a k group, and an odd number of 16-byte units
constexpr int rollout_eval_px(int D) { return (D + 15) / 16 * 16 + 8; }

// OCC: workgroups per CU the registers are capped for
template <int H, int BM, int V, int CA, int KIND, int OCC>
__global__ void __launch_bounds__(256, OCC) rollout_eval_kernel(RolloutArgs a) {
  constexpr int D = 3 * V * V, PX = rollout_eval_px(D), PH = H + 8, HPLANE = BM * PH, NOUT = kActions;
  constexpr int NTN = H / 32, MT = BM / 32, TILES = MT * NTN;
  static_assert(TILES == 4, "one 32x32 MFMA tile per wavefront");
  extern __shared__ __attribute__((aligned(16))) float lds[];
  bf16_t* const Xs2 = reinterpret_cast<bf16_t*>(lds);  // [2][BM][PX]  observation windows of two consecutive steps (exact in bf16),
                                                       //              k-contiguous; columns D .. PX stay zero
  bf16_t* const Hs = Xs2 + 2 * BM * PX;                // [3][BM][PH]  h1, split
  float* const red = reinterpret_cast<float*>(Hs + 3 * HPLANE);  // [NTN][NOUT][BM] shares of the output layer
  float* const W3s = red + NTN * NOUT * BM;            // [H][NOUT]
  float* const b1s = W3s + H * NOUT;                   // [H]
  float* const b2s = b1s + H;                          // [H]
  int* const running = reinterpret_cast<int*>(b2s + H);  // does an environment still take a step

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lo = lane & 31, hi = lane >> 5;
  const int mt = wave / NTN, nt = wave % NTN;
  const int srow = mt * 32 + lo, u0 = nt * 32 + 4 * hi;  // this lane's sample of the tile; its units are u0 + 8 j .. + 3
  const EvalEpisodes& eps = a.eps;
  const bool apart = eps.copies > 0;  // episodes by themselves, or the steps that are left
  RolloutEnvs<BM, V, CA, KIND> env(a, wave, lane, max(eps.copies, 1));
  float ret_sum = 0.f;  // of the block; apart: of the episode (its rewards in the warehouse are whole numbers, whose sums are exact)
  int len_sum = 0, episodes = 0;
  constexpr int REC = eval_record_words(CA);
  int left = 0;                    // steps this lane's environment still takes; apart: is it playing
  int slot = env.copy, events = 0; // apart: the episode it plays and its steps with a reward
  int put_down = slot < a.n_episodes ? 0 : eps.every;  // apart: the step after which the entities are put down (0: of a counted episode, not at all)
  uint32_t episode0 = 0;

  GroupCopy<H * NOUT, 256> w3;
  GroupCopy<H, 256> b1, b2;
  w3.request(tid, a.W3);
  b1.request(tid, a.b1);
  b2.request(tid, a.b2);
  for (int i = tid; i < BM * PX; i += 256) reinterpret_cast<uint32_t*>(Xs2)[i] = 0u;  // padding columns and unused rows stay zero for good
  if (env.is_env_wave) {
    env.load();
    episode0 = env.episode;
    // an episode that began within its cap ends within it; a state of another kind is played from here in the last call
    const bool known = env.t_ep >= 0 && env.t_ep < env.p.cap;
    if (env.active && apart) {
      left = known;
      if (known && slot > 0) env.restart(episode0 + slot);
    } else if (env.active) {
      left = a.T;
      if (known && eps.slots > 0) {
        for (int e = 0; e < a.n_episodes; ++e) {
          const int64_t i = (int64_t)e * env.p.N + env.n;
          const int v = eps.len[i];
          const float4 r0 = *reinterpret_cast<const float4*>(eps.record + REC * i), r1 = *reinterpret_cast<const float4*>(eps.record + REC * i + 4);
          const float r[kEpisodeRewards] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
          len_sum += v & 0xffffff;
#pragma unroll
          for (int q = 0; q < kEpisodeRewards; ++q)
            if (q < v >> 24) ret_sum += r[q];
        }
        episodes = a.n_episodes;
        left -= len_sum;
        int e = a.n_episodes;  // the episode that holds the last step, or the first that was not played
        for (bool more = true; more && e < eps.slots;) {
          int v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] = eps.len[(int64_t)min(e + u, eps.slots - 1) * env.p.N + env.n];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            more = more && left > 0 && e < eps.slots && v[u] <= left;  // (what lies behind the last episode played is not looked at: left is zero there)
            if (more) {
              left -= v[u];
              ++e;
            }
          }
        }
        const int third = e < eps.slots ? min(left / eps.every, 2) : 0;
        if (third > 0) {
          env.recall(eps.record + REC * ((int64_t)e * env.p.N + env.n) + 2 * CA * (third - 1));
          env.episode = episode0 + e;
          env.t_ep = third * eps.every;
          left -= third * eps.every;
        } else {
          env.restart(episode0 + e);
        }
      }
    }
  }
  w3.store(tid, [&](int e, float v) { W3s[e] = v; });
  b1.store(tid, [&](int e, float v) { b1s[e] = v; });
  b2.store(tid, [&](int e, float v) { b2s[e] = v; });
  __syncthreads();
  if (left > 0) env.paint(Xs2 + lane * PX);
  if (env.is_env_wave) {
    const bool any = __builtin_amdgcn_ballot_w64(left > 0) != 0;
    if (lane == 0) *running = any;
  }
  // the output layer's bias stays in registers for all T steps
  float b3r[NOUT];
#pragma unroll
  for (int k = 0; k < NOUT; ++k) b3r[k] = a.b3[k];
  // the first weights of a layer are requested a phase ahead (buffer loads: one descriptor, one lane offset)
  constexpr int KG1 = (D + 15) / 16, KG2 = H / 16;
  const int wlane = (hi * H + nt * 32 + lo) * 4;
  const WeightRsrc rsW1 = split_weight_rsrc(a.W1, 16 * KG1, H), rsW2 = split_weight_rsrc(a.W2, H, H);
  constexpr int RING = 8;  // a layer's weights all at once where the registers allow: the groups follow one another faster than the L2 answers (layer 2: 4000 -> 2000 cycles)
  PhaseW<KG1, RING> pw1;
  phase_w_request<H>(pw1, rsW1, wlane, KG1);
  for (int t = 0;; ++t) {
    loop_head_barrier();  // the windows of step t are complete
    if (__builtin_amdgcn_readfirstlane(*running) == 0) break;  // uniform; written again two barriers from here
    const bf16_t* const Xs = Xs2 + (t & 1) * BM * PX;
    int uw = u0;  // the weights and biases in LDS are read in every step: kept across steps, they would take 96 registers
    asm volatile("" : "+v"(uw));
    // ---- layer 1: h1 = tanh(X W1 + b1) -> LDS.  Both layers are computed transposed (gemm_phase_t).
    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    gemm_phase_t<H, KG1, true>(Xs + srow * PX + 8 * hi, 0, rsW1, wlane, KG1, acc, pw1);
    PhaseW<KG2, RING> pw2;  // layer 2's weights arrive during the tanh of layer 1
    phase_w_request<H>(pw2, rsW2, wlane, KG2);
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
    phase_w_request<H>(pw1, rsW1, wlane, KG1);  // layer 1 of the next step
    {
      float part[NOUT];
#pragma unroll
      for (int k = 0; k < NOUT; ++k) part[k] = 0.f;
      float4 bs[2], wv[2][NOUT];  // a quarter's bias and weights, requested a quarter ahead
      auto request = [&](int j) {
        bs[j & 1] = *reinterpret_cast<const float4*>(&b2s[uw + 8 * j]);
#pragma unroll
        for (int q = 0; q < NOUT; ++q) wv[j & 1][q] = *reinterpret_cast<const float4*>(&W3s[(uw + 8 * j) * NOUT + 4 * q]);
      };
      request(0);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (j + 1 < 4) request(j + 1);
        const float4 bj = bs[j & 1];
        const float h[4] = {tanh_f32(acc[4 * j] + bj.x), tanh_f32(acc[4 * j + 1] + bj.y), tanh_f32(acc[4 * j + 2] + bj.z), tanh_f32(acc[4 * j + 3] + bj.w)};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int k = 0; k < NOUT; ++k) {
            const float4 w4 = wv[j & 1][(e * NOUT + k) / 4];
            const int c = (e * NOUT + k) % 4;
            part[k] = fmaf(h[e], c == 0 ? w4.x : c == 1 ? w4.y : c == 2 ? w4.z : w4.w, part[k]);
          }
        __builtin_amdgcn_sched_barrier(0);  // two quarters' weights in registers at a time
      }
#pragma unroll
      for (int k = 0; k < NOUT; ++k) {
        const float v = part[k] + __shfl_xor(part[k], 32);
        if (hi == 0) red[(nt * NOUT + k) * BM + srow] = v;
      }
    }
    __syncthreads();
    if (env.is_env_wave) {
      // ---- the env lanes: logits -> action -> transition -> next window
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
      float top = lg[0];  // largest logit, lowest index on exact ties
#pragma unroll
      for (int k = 1; k < NOUT; ++k)
        if (lg[k] > top) {
          top = lg[k];
          my_act = k;
        }
      if (left > 0) {  // the same in all lanes of an env
        float rew;
        bool dn;
        env.step(my_act, rew, dn);
        // team reward = the agents' rewards added in ascending agent index, then added to the running sum (fp32)
        float team = 0.f;
#pragma unroll
        for (int b = 0; b < CA; ++b) {
          const float rb = __shfl(rew, min(env.le * env.A + b, 63));
          if (b < env.A) team += rb;
        }
        if (apart) {
          const auto at = [&]() { return (int64_t)slot * env.p.N + env.n; };
          len_sum += 1;
          if (KIND == 0 && team != 0.f) {  // at most one for each food of an episode
            if (slot < a.n_episodes && env.ai == 0 && events < kEpisodeRewards) eps.record[REC * at() + events] = __float_as_uint(team);
            events += 1;
          }
          if (KIND != 0) ret_sum += team;
          if (dn) {
            const bool counted = slot < a.n_episodes;
            if (env.ai == 0) {
              if (KIND != 0 && counted) eps.record[REC * at()] = __float_as_uint(ret_sum);
              eps.len[at()] = len_sum | (!counted ? 0 : KIND != 0 ? 1 : events) << 24;
            }
            ret_sum = 0.f;
            len_sum = events = 0;
            slot = eps.slots;
            if (t + 1 < eps.steps) {
              int taken = 0;
              if (env.ai == 0) {
                const int k = atomicAdd(eps.next + env.n, 1) - eps.idle;
                taken = k < 0 ? eps.slots : eps.copies + k;
              }
              slot = __shfl(taken, env.le * env.A);
            }
            put_down = slot < a.n_episodes ? 0 : eps.every;
            if (slot < eps.slots) env.restart(episode0 + slot);
            else left = 0;
          } else if (len_sum == put_down) {
            if (env.ai == 0) env.save(eps.record + REC * at() + (put_down == eps.every ? 0 : 2 * CA));
            put_down += eps.every;
          }
        } else {
          left -= 1;
          if (episodes < a.n_episodes) {
            ret_sum += team;
            len_sum += 1;
            if (dn) episodes += 1;
          }
        }
        if (left > 0) env.paint(Xs2 + ((t + 1) & 1) * BM * PX + lane * PX);  // the windows of step t + 1 into the other tile
      }
      const bool any = __builtin_amdgcn_ballot_w64(left > 0) != 0;
      if (lane == 0) *running = any;
    }
  }
  if (env.active && !apart) {
    env.store();
    if (env.ai == 0) {
      a.ev.ret_sum[env.n] = ret_sum;
      a.ev.len_sum[env.n] = len_sum;
      a.ev.episodes[env.n] = episodes;
    }
  }
}

}  // namespace marl
