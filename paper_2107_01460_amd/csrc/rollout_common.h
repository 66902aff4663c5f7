// What the two rollout kernels share: the arguments, and the environments of a workgroup in the registers of one of its
// wavefronts.
#pragma once
#include "env_device.h"
#include "gemm.h"
#include "heads.h"

namespace marl {

// Episodes of an evaluation block that were played by themselves (rollout_eval.h), at most `slots` of an environment: the length of each (and above
// it, from bit 24 on, a counted one's number of steps with a reward) and a record, of a counted one those rewards in the order of time, of a later one its
// entities a third and two thirds of the cap into it.
constexpr int kEpisodeRewards = 8;
constexpr int eval_record_words(int capacity) { return capacity <= 4 ? 16 : 32; }  // two sets of entities
struct EvalEpisodes {
  int slots, copies;  // copies: rows of an environment, which take its episodes in order; 0 in the call that plays what is left
  int idle, steps;    // the first `idle` rows that are done before `steps` steps take no other episode; a row that has taken so many neither
  int every;          // a third of the cap, rounded up
  int32_t* len;       // [slots][N]
  uint32_t* record;   // [slots][N][eval_record_words]
  int32_t* next;      // [N] rows that were done before `steps` steps so far, zero before the launch
};

struct RolloutArgs {
  EnvParams p;
  marl_env_state st;
  const float *W1, *W2;  // the actor's weights in the order the kernel reads them: fp32 (training), split (evaluation)
  const float *b1, *b2, *W3, *b3;
  int T;  // steps to take
  // training rollout
  int rows;    // samples of a tile (rollout_rows): the order of W1 and W2 goes by it
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
  EvalEpisodes eps;
};

// Lane l < BM of ONE wavefront is agent l % A of env env0 + l / A.  Which wavefront it is rotates with the workgroup index, so
// that the workgroups of a CU keep their serial sections on different SIMDs.
template <int BM, int V, int CA, int KIND>
struct RolloutEnvs {
  static_assert(BM <= 64, "the env lanes are lanes of one wavefront");
  const EnvParams& p;
  const marl_env_state& st;
  int lane, A, le, ai, samples_here, other, copy = 0;
  int64_t env0, n;
  bool is_env_wave, active;
  uint32_t ag[CA], fd[CA];
  int t_ep = 0;
  uint32_t episode = 0;

  // copies: how often every environment appears, as rows copy * N + n
  __device__ __forceinline__ RolloutEnvs(const RolloutArgs& a, int wave, int lane_, int copies = 1) : p(a.p), st(a.st), lane(lane_), A(a.p.A) {
    const int epw = BM / A;  // envs of this workgroup
    env0 = (int64_t)blockIdx.x * epw;
    const int envs_here = (int)min((int64_t)epw, (int64_t)p.N * copies - env0);
    samples_here = envs_here * A;
    const int env_wave = blockIdx.x & 3;
    is_env_wave = wave == env_wave;
    other = ((wave - env_wave - 1) & 3) * 64 + lane;  // thread number among the other three wavefronts
    le = lane / A;
    ai = lane - le * A;
    active = is_env_wave && lane < samples_here;
    n = env0 + le;
    if (copies > 1) {
      copy = (int)((uint32_t)n / (uint32_t)p.N);
      n -= (int64_t)copy * p.N;
    }
  }
  __device__ __forceinline__ void load() {
    const size_t nn = active ? (size_t)n : 0;
    load_env_state<CA, CA, KIND>(ag, fd, st, p, nn, active);
    t_ep = st.t_in_ep[nn];
    episode = st.episode_id[nn];
  }
  // Start of episode e (all lanes of an env together).
  __device__ __forceinline__ void restart(uint32_t e) {
    episode = e;
    t_ep = 0;
    if (KIND == 0) reset_regs<CA, CA, true>(ag, fd, p, (uint32_t)n, e, ai);
    else wh_reset_regs<CA, CA, true>(ag, fd, p, (uint32_t)n, e, ai);
  }
  template <typename T>
  __device__ __forceinline__ void paint(T* window) const {
    if (KIND == 0) forage_paint<V, CA, CA, true>(window, ag, fd, ai, p);
    else wh_paint<V, CA, CA, true>(window, ag, fd, ai, p);
  }
  // The entities to and from 2 * CA words (16-byte aligned).
  __device__ __forceinline__ void save(uint32_t* d) const {
#pragma unroll
    for (int i = 0; i < CA; i += 2) reinterpret_cast<uint4*>(d)[i / 2] = make_uint4(ag[i], fd[i], ag[i + 1], fd[i + 1]);
  }
  __device__ __forceinline__ void recall(const uint32_t* d) {
#pragma unroll
    for (int i = 0; i < CA; i += 2) {
      const uint4 v = reinterpret_cast<const uint4*>(d)[i / 2];
      ag[i] = v.x; fd[i] = v.y; ag[i + 1] = v.z; fd[i + 1] = v.w;
    }
  }
  // All lanes of an env run this together, so that the cross-lane reads find their source lanes running.
  __device__ __forceinline__ void step(int my_act, float& rew, bool& dn) {
    int act[CA];
#pragma unroll
    for (int b = 0; b < CA; ++b) {
      const int v = __shfl(my_act, min(le * A + b, 63));
      act[b] = (active && b < A) ? v : 0;
    }
    if (KIND == 0) forage_transition<CA, CA>(ag, fd, act, ai, active, p, (uint32_t)n, t_ep, episode, rew, dn);
    else wh_transition<CA, CA>(ag, fd, act, ai, active, p, (uint32_t)n, t_ep, episode, rew, dn);
  }
  __device__ __forceinline__ void store() const { store_env_state<CA, CA, KIND>(ag, fd, st, p, (size_t)n, ai, /*dn=*/true, t_ep, episode); }
};

}  // namespace marl
