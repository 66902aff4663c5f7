// The GRU cell over a whole sequence in one launch each way: h' = (1 - z) n + z h for t = 0 .. T-1 and its gradient for
// t = T-1 .. 0.  Sequences are independent of one another, so a workgroup keeps SM * 16 of them (in an update, where
// gru_by_runs says so, of their runs between the beginnings of episodes, SeqRuns) from the first step to the last: the hidden state (forward) or its
// gradient (backward) never leaves the registers, the operand of the next step's product is handed over through LDS, and nothing but the
// per-step records goes through memory.
//
// The product with the hidden-to-hidden weights runs transposed, weights x state, on v_mfma_f32_16x16x32_bf16 with split
// operands (split_bf16.h): its result gives a lane four consecutive units of one sequence, so that every load and store of
// a record is 16 bytes wide.  The weights come split and in the order a lane feeds them to the instruction
// (gru_stage_weight below).
//   H <= 128 (RES): H / 16 wavefronts of 16 units; all of the weights, 18 H^2 bytes, stay in the registers (144 of 256 per
//     lane at H = 128).
//   H <= 256: H / 32 wavefronts of 32 units; 18 H^2 bytes no longer fit a compute unit, so the weights are streamed from
//     the L2 once per step, a contraction step or two ahead of their use.
// Measured against one launch per step and direction on the fp32 instruction (128 steps of 768 sequences, 128 units):
// forward 2.7 ms -> 0.25 ms, backward 3.6 ms -> 0.5 ms; a training iteration of 1024 environments 171 -> 51 ms.
// Bound there: a step is a chain of 72 matrix instructions per wavefront, a barrier and the gate arithmetic, 2.6 us forward and 3.4 us
// backward, and a launch takes as many as the longest run has: with episodes of at most 50 steps in place of 128-step rollouts 386 ->
// 174 us and 436 -> 185 us, the two networks' kernels beside each other 335 -> 217 us and 474 -> 240 us.  With enough sequences the bound
// is the records' way to memory (128 units, 1 048 576 steps: 1.00 and 1.09 ms, 4.3 TB/s) or, above 128 units, the weights' way from the L2
// (256 units, 262 144 steps: 1.28 and 1.50 ms, 15 TB/s; whole sequences in 128 workgroups 1.96 and 2.41 ms).
#pragma once
#include "gemm.h"
#include "heads.h"

namespace marl {

inline bool gru_seq_supported(int H) { return H % 32 == 0 && H <= 256; }
inline int64_t gru_weight_floats(int H) { return (((int64_t)H * H * 9 / 2 + 63) / 64) * 64; }  // one staged copy

// The element (k, c) of gate weights [H][3H] in the two staged copies: three planes of bf16, in 512-element fragments of 16 units by
// 32 along the contraction.
template <bool FWD, bool BWD>
__device__ __forceinline__ void gru_stage_weight(float v, int k, int c, int H, bf16_t* __restrict__ fwd, bf16_t* __restrict__ bwd) {
  const SplitPair s = split_pair_any(v, 0.f);
  const uint32_t part[3] = {s.h, s.m, s.l};
  const int KS = H / 32, g = c / H, u = c - g * H;
  const int64_t f = ((int64_t)((u / 16) * KS + k / 32) * 9 + g * 3) * 512 + ((u % 16) + 16 * ((k % 32) / 8)) * 8 + k % 8;
  const int64_t b = ((int64_t)((k / 16) * 3 * KS + g * KS + u / 32) * 3) * 512 + ((k % 16) + 16 * ((u % 32) / 8)) * 8 + u % 8;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    if (FWD) fwd[f + 512 * p] = (bf16_t)part[p];
    if (BWD) bwd[b + 512 * p] = (bf16_t)part[p];
  }
}

__device__ __forceinline__ float sigmoid_f32(float x) { return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x)); }

// The runs of a minibatch of sequences: a state is zeroed where an episode begins, so that the steps between two such places, a run, depend
// on nothing before them, and the runs of all sequences can go side by side.  A chain is then as long as an episode at most, not as
// the rollout.  Run i of `env[]` covers `y` steps from row x = t * (S1 / per) + environment on and stands for `per` sequences; the longest come first (that is
// for speed alone: lanes of a workgroup whose run has ended wait for the others, and the workgroups' shares come out alike).
struct SeqRuns {
  const int2* env;
  const int* count;
  int* next;  // streamed weights: groups taken beyond each workgroup's first, zero before the launch
  int turn;   // 1: the first round is dealt out from the last workgroup on
};
// The first sequence of a workgroup's k-th group of MT (whole workgroup, uniform).  With the weights in registers (DEALT) every round of gridDim.x groups is
// dealt out the other way round, so that who has the longest of one round has the shortest of the next, and a workgroup without a group in a round has none in
// later ones.  With streamed weights, whose steps are longer, a workgroup that is done takes the next one from a counter, so that who began with a long
// group takes fewer: 1536 sequences of 128 steps in runs of ten, 256 units, dealt out an update of 8.8 ms, from the counter 8.3–8.5.  (For resident weights the counter, 30 ns
// for each group, one after the other, is what bounds: runs of five steps of 3072 sequences, 32 units, 131 and 170 us forward and backward, dealt out 35 and 40.)
// The two networks, which run beside one another, begin at opposite ends (turn): where the groups are few, most workgroups leave at once and the working ones of
// both would come to lie on the same compute units (192 sequences x 128 steps, 64 units: an update of 1.17 of the time).
template <int MT, bool DEALT>
__device__ __forceinline__ int group_first(const SeqRuns& runs, int k, int* slot) {
  if (DEALT || k == 0) return MT * (int)(k * gridDim.x + ((k + runs.turn) & 1 ? gridDim.x - 1 - blockIdx.x : blockIdx.x));
  loop_head_barrier();  // every wavefront has read the last number
  if (threadIdx.x == 0) *slot = (int)gridDim.x + atomicAdd(runs.next, 1);
  __syncthreads();
  return MT * __builtin_amdgcn_readfirstlane(*slot);
}
// Sequence k's row of a step's S1 and steps; past the end: 0 steps of the first sequence's row.
__device__ __forceinline__ void run_of(const SeqRuns& runs, int per, int k, int total, int64_t& row, int& len) {
  const bool in = k < total;
  const int i = (in ? k : 0) / per, a = in ? k - i * per : 0;
  const int2 r = runs.env[i];
  row = (int64_t)r.x * per + a;
  len = in ? r.y : 0;
}
template <int SM>
__device__ __forceinline__ int longest_run(const int (&len)[SM]) {
  int n = 0;
#pragma unroll
  for (int m = 0; m < SM; ++m) n = max(n, len[m]);
#pragma unroll
  for (int o = 8; o > 0; o /= 2) n = max(n, __shfl_xor(n, o));
  return __builtin_amdgcn_readfirstlane(n);
}

// The records of a step, [S1][4H]: forward (h Wh_n + bh_n, r, z, n); the backward pass replaces them by the gradients of
// the pre-activations (of h Wh_n + bh_n, r, z, n), so that columns 0 .. 3H-1 are the gradient of the hidden products (new
// gate first) and columns H .. 4H-1 that of the input products.
struct GruFwdArgs {
  const float* Gi;       // [T][S1][3H] input products, no bias
  const bf16_t* W;       // staged weights
  const float *bi, *bh;  // [3H]
  const float* h_first;  // [S1][H] state before the first step; may be hs
  float* hs;             // [T][S1][H] state after every step
  float* rec;            // [T][S1][4H], nullable
  // Step 0 starts from a zero state where reset0[s / per] is set, step t > 0 where reset[(t - 1) * (S1 / per) + s / per] is.
  const uint8_t *reset0, *reset;  // reset0 nullable; reset is not read if T = 1
  int per;
  int64_t S1;
  int T;
  SeqRuns runs;  // SEG
};

// acc[i] += W[i] x B over 32 along the contraction, i-th of N independent tiles (small products first)
__device__ __forceinline__ floatx4 mfma16(const bf16x8& a, const bf16x8& b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// SEG: the runs of a.runs, a workgroup taking group after group; otherwise workgroup i has sequences i * MT .. for all T steps.
template <int KS, int SM, bool RES, bool SEG>
__global__ void __launch_bounds__(RES ? 128 * KS : 64 * KS, 2) gru_seq_fwd_kernel(GruFwdArgs a) {
  constexpr int H = 32 * KS, UB = RES ? 1 : 2, MT = 16 * SM, P = H + 8, PLANE = MT * P;
  constexpr int THREADS = RES ? 128 * KS : 64 * KS;
  __shared__ __attribute__((aligned(16))) bf16_t Hs[2][3 * PLANE];
  __shared__ __attribute__((aligned(16))) float bias[4][H];  // r and z: both biases; n: input, hidden
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lo = lane & 15, q = lane >> 4;
  const int total = SEG ? *a.runs.count * a.per : 0;
  __shared__ int group;  // SEG with streamed weights
  if (SEG && group_first<MT, RES>(a.runs, 0, &group) >= total) return;
  for (int j = tid; j < H; j += THREADS) {
    bias[0][j] = a.bi[j] + a.bh[j];
    bias[1][j] = a.bi[H + j] + a.bh[H + j];
    bias[2][j] = a.bi[2 * H + j];
    bias[3][j] = a.bh[2 * H + j];
  }
  int unit[UB];  // first of this lane's four units
#pragma unroll
  for (int b = 0; b < UB; ++b) unit[b] = 16 * (UB * wave + b) + 4 * q;

  const WeightRsrc wsrc = weight_rsrc(reinterpret_cast<const float*>(a.W), H * H * 9 / 2);
  int woff = UB * wave * KS * 9 * 1024 + lane * 16;  // this lane's bytes of its wavefront's fragments
  // Streamed: a wavefront starts its walk along the contraction at a step of its own, since the wavefronts' fragments are a
  // multiple of 4 KB apart and in step would all ask the same memory channels of the L2 at the same time (128 steps of 2048
  // sequences, 256 units: 3.45 -> 3.0 ms).  It depends on the wavefront, that is on the units, and on nothing else: a sequence's
  // sums are the same wherever in a batch of whatever size it is.  (The remainder tells the compiler the range, and with it that
  // the steps' offsets need no comparison each: an iteration of 16 384 environments 446 -> 432 ms.)
  const int rot = RES ? 0 : __builtin_amdgcn_readfirstlane(wave % KS);
  auto step_of = [&](int ks) { return RES ? ks : ks + rot < KS ? ks + rot : ks + rot - KS; };
  auto load_w = [&](int i, bf16x8 (&w)[9]) {
#pragma unroll
    for (int f = 0; f < 9; ++f)
      w[f] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wsrc, woff, ((i / KS * KS + step_of(i % KS)) * 9 + f) * 1024, 0));
  };
  // streamed: contraction steps in flight, a divisor of NI (the ring goes on into the next step)
  constexpr int NI = UB * KS, RING = RES ? NI : SM == 1 && NI % 4 == 0 ? 4 : 2;
  static_assert(NI % RING == 0, "ring");
  bf16x8 w[RING][9];
#pragma unroll
  for (int i = 0; i < (RES ? NI : RING - 1); ++i) load_w(i, w[i]);

  for (int k = 0;; ++k) {
    int64_t row[SM];  // of the current step
    int64_t env[SM];  // without SEG
    int len[SM], steps = a.T;  // a sequence past its last step stays at that row and stores nothing
    if (SEG) {
      const int first = group_first<MT, RES>(a.runs, k, &group);
      if (first >= total) return;  // uniform
#pragma unroll
      for (int m = 0; m < SM; ++m) run_of(a.runs, a.per, first + 16 * m + lo, total, row[m], len[m]);
      steps = longest_run(len);
    } else {
#pragma unroll
      for (int m = 0; m < SM; ++m) {
        const int64_t at = (int64_t)blockIdx.x * MT + 16 * m + lo;
        row[m] = min(at, a.S1 - 1);
        len[m] = at < a.S1 ? a.T : 0;
        env[m] = row[m] / a.per;
      }
    }
    const int64_t nenv = a.S1 / a.per;
    float4 h[UB][SM], gi[UB][SM][3];
    auto load_gi = [&](int b, const int64_t (&at)[SM]) {
#pragma unroll
      for (int m = 0; m < SM; ++m)
#pragma unroll
        for (int g = 0; g < 3; ++g) gi[b][m][g] = *reinterpret_cast<const float4*>(a.Gi + at[m] * 3 * H + g * H + unit[b]);
    };
    bool wild = false;  // was a state out of split_pair's range to begin with?  (One step's state is at most the last one's or 1.)
    auto hand_over = [&](int buf, int b, int m) {
      bf16_t* const dst = &Hs[buf][(16 * m + lo) * P + unit[b]];
      if (wild) store_split4<true>(dst, PLANE, h[b][m]);
      else store_split4<false>(dst, PLANE, h[b][m]);
    };
    int rs[SM];  // does the coming step start from a zero state
    auto load_reset = [&](int t) {
#pragma unroll
      for (int m = 0; m < SM; ++m) rs[m] = t > 0 ? a.reset[(t - 1) * nenv + env[m]] : (a.reset0 != nullptr ? a.reset0[env[m]] : 0);
    };
    if (!SEG) load_reset(0);
    float top = 0.f;
#pragma unroll
    for (int b = 0; b < UB; ++b) {
      load_gi(b, row);
#pragma unroll
      for (int m = 0; m < SM; ++m) {
        if (SEG) rs[m] = row[m] >= a.S1;  // a run that does not begin at step 0 begins where an episode does
        h[b][m] = *reinterpret_cast<const float4*>(a.h_first + (SEG && rs[m] ? 0 : row[m]) * H + unit[b]);
        if (rs[m]) h[b][m] = make_float4(0.f, 0.f, 0.f, 0.f);
        top = max_abs(top, h[b][m]);
      }
    }
    wild = split_out_of_range(top * 0x1p10f);  // room for a million steps' rounding
#pragma unroll
    for (int b = 0; b < UB; ++b)
#pragma unroll
      for (int m = 0; m < SM; ++m) hand_over(0, b, m);
    __syncthreads();

#pragma unroll 1
    for (int t = 0; t < steps; ++t) {
      if (!RES) asm volatile("" : "+v"(woff));  // the loads stay inside the loop: hoisted, they would be spilled
      const bf16_t* const frag = &Hs[t & 1][lo * P + 8 * q];
      if (!SEG && t + 1 < steps) load_reset(t + 1);
      int64_t next[SM];
#pragma unroll
      for (int m = 0; m < SM; ++m) next[m] = t + 1 < len[m] ? row[m] + a.S1 : row[m];
#pragma unroll
      for (int b = 0; b < UB; ++b) {
        floatx4 acc[3][SM];
#pragma unroll
        for (int g = 0; g < 3; ++g)
#pragma unroll
          for (int m = 0; m < SM; ++m) acc[g][m] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const int i = b * KS + ks, slot = i % RING;
          if (!RES) load_w((i + RING - 1) % NI, w[(i + RING - 1) % RING]);
          Split8 x[SM];
#pragma unroll
          for (int m = 0; m < SM; ++m) x[m] = frag_row(frag + 16 * m * P + 32 * step_of(ks), PLANE);
#define MARL_GRU_PRODUCT(WP, XP)            \
  _Pragma("unroll") for (int g = 0; g < 3; ++g) \
  _Pragma("unroll") for (int m = 0; m < SM; ++m) acc[g][m] = mfma16(w[slot][3 * g + WP], x[m].XP, acc[g][m]);
          MARL_GRU_PRODUCT(2, h)
          MARL_GRU_PRODUCT(0, l)
          MARL_GRU_PRODUCT(1, m)
          MARL_GRU_PRODUCT(1, h)
          MARL_GRU_PRODUCT(0, m)
          MARL_GRU_PRODUCT(0, h)
#undef MARL_GRU_PRODUCT
        }
        float4 bs[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) bs[k] = *reinterpret_cast<const float4*>(&bias[k][unit[b]]);
        float4 vr[SM], vz[SM], vn[SM], vh[SM], out[SM];
#pragma unroll
        for (int m = 0; m < SM; ++m) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            auto at = [e](const float4& v) { return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w; };
            auto put = [e](float4& v, float f) { (e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w) = f; };
            const float r = sigmoid_f32(at(gi[b][m][0]) + (acc[0][m][e] + at(bs[0])));
            const float z = sigmoid_f32(at(gi[b][m][1]) + (acc[1][m][e] + at(bs[1])));
            const float hn = acc[2][m][e] + at(bs[3]);
            const float n = tanh_f32((at(gi[b][m][2]) + at(bs[2])) + r * hn);
            put(vr[m], r); put(vz[m], z); put(vh[m], hn); put(vn[m], n);
            put(out[m], (1.0f - z) * n + z * at(h[b][m]));
          }
        }
        if (t + 1 < steps) load_gi(b, next);  // ahead of this step's stores: the counter that loads wait on is in order
#pragma unroll
        for (int m = 0; m < SM; ++m) {
          if (t < len[m]) {
            if (SEG || a.rec != nullptr) {
              float* const d = a.rec + row[m] * 4 * H + unit[b];
              *reinterpret_cast<float4*>(d) = vh[m];
              *reinterpret_cast<float4*>(d + H) = vr[m];
              *reinterpret_cast<float4*>(d + 2 * H) = vz[m];
              *reinterpret_cast<float4*>(d + 3 * H) = vn[m];
            }
            *reinterpret_cast<float4*>(a.hs + row[m] * H + unit[b]) = out[m];
          }
          h[b][m] = !SEG && rs[m] ? make_float4(0.f, 0.f, 0.f, 0.f) : out[m];
          hand_over((t + 1) & 1, b, m);
        }
      }
#pragma unroll
      for (int m = 0; m < SM; ++m) row[m] = next[m];
      lds_barrier();
    }
    if (!SEG) return;
  }
}

struct GruBwdArgs {
  const bf16_t* W;       // staged weights (backward copy)
  const float* W3;       // [H][NOUT] output layer
  const float* dl;       // [T][S1][NOUT] gradient of the outputs
  float* rec;            // [T][S1][4H] records, replaced by gradients
  const float* hs;       // [T][S1][H] state before every step (before a reset)
  const uint8_t* reset;  // [T - 1][S1 / per], as forward
  int per;
  int64_t S1;
  int T;
  SeqRuns runs;
};

// SEG as forward.
template <int KS, int SM, bool RES, bool SEG, int NOUT>
__global__ void __launch_bounds__(RES ? 128 * KS : 64 * KS, 2) gru_seq_bwd_kernel(GruBwdArgs a) {
  constexpr int H = 32 * KS, UB = RES ? 1 : 2, MT = 16 * SM, P = 3 * H + 8, PLANE = MT * P;
  constexpr int THREADS = RES ? 128 * KS : 64 * KS;
  __shared__ __attribute__((aligned(16))) bf16_t Gs[3 * PLANE];
  __shared__ __attribute__((aligned(16))) float W3s[H * NOUT];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lo = lane & 15, q = lane >> 4;
  const int total = SEG ? *a.runs.count * a.per : 0;
  __shared__ int group;  // SEG with streamed weights
  if (SEG && group_first<MT, RES>(a.runs, 0, &group) >= total) return;
  GroupCopy<H * NOUT, THREADS> w3;
  w3.request(tid, a.W3);
  w3.store(tid, [&](int e, float v) { W3s[e] = v; });
  int unit[UB];
#pragma unroll
  for (int b = 0; b < UB; ++b) unit[b] = 16 * (UB * wave + b) + 4 * q;

  constexpr int NI = 3 * KS, RING = RES ? NI : 3;  // NI is a multiple of 3
  const WeightRsrc wsrc = weight_rsrc(reinterpret_cast<const float*>(a.W), H * H * 9 / 2);
  int woff = UB * wave * NI * 3 * 1024 + lane * 16;
  auto load_w = [&](int i, bf16x8 (&w)[UB][3]) {
#pragma unroll
    for (int b = 0; b < UB; ++b)
#pragma unroll
      for (int p = 0; p < 3; ++p) w[b][p] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wsrc, woff, ((b * NI + i) * 3 + p) * 1024, 0));
  };
  bf16x8 w[RING][UB][3];
#pragma unroll
  for (int i = 0; i < (RES ? NI : RING - 1); ++i) load_w(i, w[i]);

  __syncthreads();  // W3s
  for (int k = 0;; ++k) {
    int64_t row[SM];  // of the current step; a sequence past its first step stays there and stores nothing
    int64_t env[SM];  // without SEG
    int len[SM], steps = a.T;
    int from_zero[SM];  // SEG: does the run's first step start from zero, else the current one (a byte that is looked at a step after its request)
    if (SEG) {
      const int first = group_first<MT, RES>(a.runs, k, &group);
      if (first >= total) return;  // uniform
#pragma unroll
      for (int m = 0; m < SM; ++m) {
        run_of(a.runs, a.per, first + 16 * m + lo, total, row[m], len[m]);
        from_zero[m] = row[m] >= a.S1;
        row[m] += max(len[m] - 1, 0) * a.S1;
      }
      steps = longest_run(len);
    } else {
#pragma unroll
      for (int m = 0; m < SM; ++m) {
        const int64_t at = (int64_t)blockIdx.x * MT + 16 * m + lo, s = min(at, a.S1 - 1);
        len[m] = at < a.S1 ? a.T : 0;
        env[m] = s / a.per;
        row[m] = (a.T - 1) * a.S1 + s;
      }
    }
    const int64_t nenv = a.S1 / a.per;
    float4 rec[UB][SM][4], hp[UB][SM], carry[UB][SM];
    float dl[SM][NOUT];
    auto load_step = [&](int b, int m) {
#pragma unroll
      for (int k = 0; k < 4; ++k) rec[b][m][k] = *reinterpret_cast<const float4*>(a.rec + row[m] * 4 * H + k * H + unit[b]);
      hp[b][m] = *reinterpret_cast<const float4*>(a.hs + row[m] * H + unit[b]);
    };
    auto load_row = [&](int t, int m) {
#pragma unroll
      for (int k = 0; k < NOUT; ++k) dl[m][k] = a.dl[row[m] * NOUT + k];
      if (!SEG) from_zero[m] = t > 0 ? a.reset[(t - 1) * nenv + env[m]] : 0;
    };
#pragma unroll
    for (int m = 0; m < SM; ++m) {
      load_row(steps - 1, m);
#pragma unroll
      for (int b = 0; b < UB; ++b) {
        load_step(b, m);
        carry[b][m] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }

#pragma unroll 1
    for (int t = 0; t < steps; ++t) {  // t-th step from the end of each run
      if (!RES) asm volatile("" : "+v"(woff));
      bool zero[SM];
#pragma unroll
      for (int m = 0; m < SM; ++m) {
        zero[m] = from_zero[m] != 0 && (!SEG || t + 1 == len[m]);
        const int64_t here = row[m];
        if (t + 1 < len[m]) row[m] -= a.S1;
#pragma unroll
        for (int b = 0; b < UB; ++b) {
          float4 gr, gz, gn, gh;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            auto at = [e](const float4& v) { return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w; };
            auto put = [e](float4& v, float f) { (e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w) = f; };
            float dh = at(carry[b][m]);
#pragma unroll
            for (int k = 0; k < NOUT; ++k) dh = fmaf(dl[m][k], W3s[(unit[b] + e) * NOUT + k], dh);
            const float hn = at(rec[b][m][0]), r = at(rec[b][m][1]), z = at(rec[b][m][2]), n = at(rec[b][m][3]);
            const float hprev = zero[m] ? 0.f : at(hp[b][m]);
            const float dpre_n = dh * (1.0f - z) * (1.0f - n * n);
            put(gr, dpre_n * hn * r * (1.0f - r));
            put(gz, dh * (hprev - n) * z * (1.0f - z));
            put(gn, dpre_n);
            put(gh, dpre_n * r);
            put(carry[b][m], dh * z);
          }
          if (t < len[m]) {
            float* const d = a.rec + here * 4 * H + unit[b];
            *reinterpret_cast<float4*>(d) = gh;
            *reinterpret_cast<float4*>(d + H) = gr;
            *reinterpret_cast<float4*>(d + 2 * H) = gz;
            *reinterpret_cast<float4*>(d + 3 * H) = gn;
          }
          bf16_t* const dst = &Gs[(16 * m + lo) * P + unit[b]];
          if (split_out_of_range(max_abs(max_abs(max_abs(0.f, gr), gz), gh))) {
            store_split4<true>(dst, PLANE, gr);
            store_split4<true>(dst + H, PLANE, gz);
            store_split4<true>(dst + 2 * H, PLANE, gh);
          } else {
            store_split4<false>(dst, PLANE, gr);
            store_split4<false>(dst + H, PLANE, gz);
            store_split4<false>(dst + 2 * H, PLANE, gh);
          }
          if (t + 1 < steps) load_step(b, m);
        }
        if (t + 1 < steps) load_row(steps - 2 - t, m);
      }
      if (t + 1 == steps) break;  // uniform: nothing flows into the initial state
      lds_barrier();
      floatx4 acc[UB][SM];
#pragma unroll
      for (int b = 0; b < UB; ++b)
#pragma unroll
        for (int m = 0; m < SM; ++m) acc[b][m] = floatx4{0.f, 0.f, 0.f, 0.f};
      const bf16_t* const frag = Gs + lo * P + 8 * q;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int slot = i % RING;
        if (!RES) load_w((i + RING - 1) % NI, w[(i + RING - 1) % RING]);
        Split8 x[SM];
#pragma unroll
        for (int m = 0; m < SM; ++m) x[m] = frag_row(frag + 16 * m * P + 32 * i, PLANE);
#define MARL_GRU_PRODUCT(WP, XP)             \
  _Pragma("unroll") for (int b = 0; b < UB; ++b) \
  _Pragma("unroll") for (int m = 0; m < SM; ++m) acc[b][m] = mfma16(w[slot][b][WP], x[m].XP, acc[b][m]);
        MARL_GRU_PRODUCT(2, h)
        MARL_GRU_PRODUCT(0, l)
        MARL_GRU_PRODUCT(1, m)
        MARL_GRU_PRODUCT(1, h)
        MARL_GRU_PRODUCT(0, m)
        MARL_GRU_PRODUCT(0, h)
#undef MARL_GRU_PRODUCT
      }
#pragma unroll
      for (int b = 0; b < UB; ++b)
#pragma unroll
        for (int m = 0; m < SM; ++m) {
          carry[b][m].x += acc[b][m][0];
          carry[b][m].y += acc[b][m][1];
          carry[b][m].z += acc[b][m][2];
          carry[b][m].w += acc[b][m][3];
          if (!SEG && zero[m]) carry[b][m] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
      lds_barrier();  // the tile has been read
    }
    if (!SEG) return;
  }
}

// ---- one rollout step of the actor: observation -> hidden state, logits, action ----------------------------------------
// The whole cell of 16 * SM samples in one workgroup: embedding, both gate products, gates, output layer, sampling.  All
// weights are streamed from the L2, split and in operand order, RING - 1 contraction steps ahead of their use; the hidden
// product runs before the barrier that publishes the embedding.  Replaces an embedding product, an input-gate product, a
// step of the cell and an output-layer kernel, whose intermediate results (5 H floats per sample) went through memory.
// Bound: the weights' way from the L2 (664 KB per workgroup at 128 units and 75 inputs, 64 bytes per clock: 4.3 us) up to
// one workgroup per compute unit, the matrix instructions beyond.  Measured: 3072 samples 12.6 us (four kernels: about 90),
// 65 536 samples 127 us.
struct GruActorArgs {
  const float* obs;      // [S][D]
  const bf16_t* We;      // staged embedding, K1 = D rounded up to 32 rows (gru_stage_embedding)
  const bf16_t *Wi, *Wh; // staged gate weights
  const float *be, *bi, *bh, *W3, *b3;
  const float* h_in;     // [S][H]
  float* h_out;          // [S][H], may be h_in
  const uint8_t* reset;  // nullable [S / per]
  int per;
  int64_t S;
  int D;
  float* logits;         // nullable [S][6]
  SampleArgs sample;
};
inline int64_t gru_embedding_floats(int D, int H) { return (int64_t)((D + 31) / 32 * 32) * H * 3 / 2; }

// element (k, u) of the embedding [D][H], zeros for D <= k
__device__ __forceinline__ void gru_stage_embedding(float v, int k, int u, int K1, bf16_t* __restrict__ dst) {
  const SplitPair s = split_pair_any(v, 0.f);
  const uint32_t part[3] = {s.h, s.m, s.l};
  const int64_t f = ((int64_t)(u / 16) * (K1 / 32) + k / 32) * 3 * 512 + ((u % 16) + 16 * ((k % 32) / 8)) * 8 + k % 8;
#pragma unroll
  for (int p = 0; p < 3; ++p) dst[f + 512 * p] = (bf16_t)part[p];
}

template <int KS, int SM>
__global__ void __launch_bounds__(KS <= 4 ? 128 * KS : 64 * KS, 2) gru_actor_step_kernel(GruActorArgs a) {
  constexpr int H = 32 * KS, UB = KS <= 4 ? 1 : 2, MT = 16 * SM, P = H + 8, PLANE = MT * P, NOUT = kActions;
  constexpr int THREADS = KS <= 4 ? 128 * KS : 64 * KS, WAVES = THREADS / 64;
  constexpr int PX = 160 + 8, XPLANE = MT * PX;  // up to 147 inputs
  static_assert(THREADS >= 2 * MT, "one thread per sample and Philox call");
  __shared__ __attribute__((aligned(16))) bf16_t Hs[3 * PLANE];
  __shared__ __attribute__((aligned(16))) bf16_t Xs[3 * XPLANE];  // inputs
  __shared__ __attribute__((aligned(16))) bf16_t Es[3 * PLANE];   // embedding
  __shared__ __attribute__((aligned(16))) float bias[5][H];  // embedding; r and z: both biases; n: input, hidden
  __shared__ __attribute__((aligned(16))) float W3s[H * NOUT];
  __shared__ float red[WAVES][MT][NOUT];
  __shared__ float noise[MT][8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lo = lane & 15, q = lane >> 4;
  const int64_t s0 = (int64_t)blockIdx.x * MT;
  const int rows = (int)min((int64_t)MT, a.S - s0);
  GroupCopy<H * NOUT, THREADS> w3;
  w3.request(tid, a.W3);
  const int K1 = (a.D + 31) / 32 * 32, KS1 = K1 / 32;

  constexpr int NI = UB * KS, RING = SM == 1 ? 4 : 2;
  const WeightRsrc rs_e = weight_rsrc(reinterpret_cast<const float*>(a.We), K1 * H * 3 / 2);
  const WeightRsrc rs_h = weight_rsrc(reinterpret_cast<const float*>(a.Wh), H * H * 9 / 2);
  const WeightRsrc rs_i = weight_rsrc(reinterpret_cast<const float*>(a.Wi), H * H * 9 / 2);
  const int woff = UB * wave * KS * 9 * 1024 + lane * 16;
  bf16x8 w[RING][9];
  auto load_w = [&](int i) {  // i < NI: hidden-to-hidden, then input-to-hidden
#pragma unroll
    for (int f = 0; f < 9; ++f)
      w[i % RING][f] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(i < NI ? rs_h : rs_i, woff, ((i % NI) * 9 + f) * 1024, 0));
  };

  int64_t srow[SM];
  bool live[SM];
  int unit[UB];
  float4 h[UB][SM];
#pragma unroll
  for (int b = 0; b < UB; ++b) unit[b] = 16 * (UB * wave + b) + 4 * q;
#pragma unroll
  for (int m = 0; m < SM; ++m) {
    live[m] = s0 + 16 * m + lo < a.S;
    srow[m] = live[m] ? s0 + 16 * m + lo : a.S - 1;
    const bool zero = a.reset != nullptr && a.reset[srow[m] / a.per];
#pragma unroll
    for (int b = 0; b < UB; ++b) {
      h[b][m] = *reinterpret_cast<const float4*>(a.h_in + srow[m] * H + unit[b]);
      if (zero) h[b][m] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  for (int i = tid; i < MT * (K1 / 2); i += THREADS) {  // two columns of a row; zeros past the ends
    const int r = i / (K1 / 2), c = 2 * (i - r * (K1 / 2));
    const float* const src = a.obs + (s0 + r) * a.D + c;
    const SplitPair v = split_pair_any(r < rows && c < a.D ? src[0] : 0.f, r < rows && c + 1 < a.D ? src[1] : 0.f);
    bf16_t* const dst = Xs + r * PX + c;
    *reinterpret_cast<uint32_t*>(dst) = v.h;
    *reinterpret_cast<uint32_t*>(dst + XPLANE) = v.m;
    *reinterpret_cast<uint32_t*>(dst + 2 * XPLANE) = v.l;
  }
  for (int j = tid; j < H; j += THREADS) {
    bias[0][j] = a.be[j];
    bias[1][j] = a.bi[j] + a.bh[j];
    bias[2][j] = a.bi[H + j] + a.bh[H + j];
    bias[3][j] = a.bi[2 * H + j];
    bias[4][j] = a.bh[2 * H + j];
  }
  w3.store(tid, [&](int e, float v) { W3s[e] = v; });
  const SampleArgs& sa = a.sample;
  if (tid < 2 * MT && (tid >> 1) < rows) {  // log(-log u) of sample tid / 2, Philox call tid % 2 (see sample_uniforms)
    const int64_t s = s0 + (tid >> 1);
    const int call = tid & 1;
    float u[4];
    if (sa.uniforms) {
#pragma unroll
      for (int k = 0; k < 4; ++k) u[k] = 4 * call + k < NOUT ? sa.uniforms[s * NOUT + 4 * call + k] : 0.5f;
    } else {
      const uint64_t step = sa.step + (sa.step_base != nullptr ? *sa.step_base : 0);
      uint32_t o[4];
      philox4x32_10((uint32_t)step, (uint32_t)(step >> 32), (uint32_t)s * 2u + (uint32_t)call, kStreamSample, sa.k0, sa.k1, o);
#pragma unroll
      for (int k = 0; k < 4; ++k) u[k] = rand_unit(o[k]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) noise[tid >> 1][4 * call + k] = logf(-logf(u[k]));
  }
#pragma unroll
  for (int b = 0; b < UB; ++b)
#pragma unroll
    for (int m = 0; m < SM; ++m) store_split4<true>(&Hs[(16 * m + lo) * P + unit[b]], PLANE, h[b][m]);
#pragma unroll
  for (int i = 0; i < RING - 1; ++i) load_w(i);
  __syncthreads();

  // ---- embedding
#pragma unroll
  for (int b = 0; b < UB; ++b) {
    floatx4 acc[SM];
#pragma unroll
    for (int m = 0; m < SM; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int eoff = (UB * wave + b) * KS1 * 3 * 1024 + lane * 16;
#pragma unroll 1
    for (int ks = 0; ks < KS1; ++ks) {
      bf16x8 e[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) e[p] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs_e, eoff, (ks * 3 + p) * 1024, 0));
#pragma unroll
      for (int m = 0; m < SM; ++m) {
        const Split8 x = frag_row(Xs + (16 * m + lo) * PX + 32 * ks + 8 * q, XPLANE);
        acc[m] = mfma16(e[2], x.h, acc[m]);
        acc[m] = mfma16(e[0], x.l, acc[m]);
        acc[m] = mfma16(e[1], x.m, acc[m]);
        acc[m] = mfma16(e[1], x.h, acc[m]);
        acc[m] = mfma16(e[0], x.m, acc[m]);
        acc[m] = mfma16(e[0], x.h, acc[m]);
      }
    }
    const float4 bs = *reinterpret_cast<const float4*>(&bias[0][unit[b]]);
#pragma unroll
    for (int m = 0; m < SM; ++m)
      store_split4<false>(&Es[(16 * m + lo) * P + unit[b]], PLANE,
                          make_float4(tanh_f32(acc[m][0] + bs.x), tanh_f32(acc[m][1] + bs.y), tanh_f32(acc[m][2] + bs.z), tanh_f32(acc[m][3] + bs.w)));
  }
  // ---- gates: r and z of both products in one accumulator, n of the hidden and of the input product
  floatx4 acc[UB][4][SM];
#pragma unroll
  for (int b = 0; b < UB; ++b)
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int m = 0; m < SM; ++m) acc[b][g][m] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 2 * NI; ++i) {
    const int b = (i % NI) / KS, ks = i % KS;
    if (i + RING - 1 < 2 * NI) load_w(i + RING - 1);
    if (i == NI) lds_barrier();  // the embedding is complete
    Split8 x[SM];
#pragma unroll
    for (int m = 0; m < SM; ++m) x[m] = frag_row((i < NI ? Hs : Es) + (16 * m + lo) * P + 32 * ks + 8 * q, PLANE);
#define MARL_GRU_PRODUCT(WP, XP)            \
  _Pragma("unroll") for (int g = 0; g < 3; ++g) \
  _Pragma("unroll") for (int m = 0; m < SM; ++m) acc[b][g == 2 && i >= NI ? 3 : g][m] = mfma16(w[i % RING][3 * g + WP], x[m].XP, acc[b][g == 2 && i >= NI ? 3 : g][m]);
    MARL_GRU_PRODUCT(2, h)
    MARL_GRU_PRODUCT(0, l)
    MARL_GRU_PRODUCT(1, m)
    MARL_GRU_PRODUCT(1, h)
    MARL_GRU_PRODUCT(0, m)
    MARL_GRU_PRODUCT(0, h)
#undef MARL_GRU_PRODUCT
  }
  float part[SM][NOUT];
#pragma unroll
  for (int m = 0; m < SM; ++m)
#pragma unroll
    for (int k = 0; k < NOUT; ++k) part[m][k] = 0.f;
#pragma unroll
  for (int b = 0; b < UB; ++b) {
#pragma unroll
    for (int m = 0; m < SM; ++m) {
      float out[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float hv = e == 0 ? h[b][m].x : e == 1 ? h[b][m].y : e == 2 ? h[b][m].z : h[b][m].w;
        const float r = sigmoid_f32(acc[b][0][m][e] + bias[1][unit[b] + e]);
        const float z = sigmoid_f32(acc[b][1][m][e] + bias[2][unit[b] + e]);
        const float n = tanh_f32((acc[b][3][m][e] + bias[3][unit[b] + e]) + r * (acc[b][2][m][e] + bias[4][unit[b] + e]));
        out[e] = (1.0f - z) * n + z * hv;
#pragma unroll
        for (int k = 0; k < NOUT; ++k) part[m][k] = fmaf(out[e], W3s[(unit[b] + e) * NOUT + k], part[m][k]);
      }
      if (live[m]) *reinterpret_cast<float4*>(a.h_out + srow[m] * H + unit[b]) = make_float4(out[0], out[1], out[2], out[3]);
    }
  }
#pragma unroll
  for (int m = 0; m < SM; ++m)
#pragma unroll
    for (int k = 0; k < NOUT; ++k) {  // the four lanes of a sample in this wavefront
      float v = part[m][k];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (q == 0) red[wave][16 * m + lo][k] = v;
    }
  lds_barrier();
  if (tid < rows) {
    const int64_t s = s0 + tid;
    float lg[NOUT], best = -INFINITY;
    int act = 0;
#pragma unroll
    for (int k = 0; k < NOUT; ++k) {
      float v = a.b3[k];
#pragma unroll
      for (int u = 0; u < WAVES; ++u) v += red[u][tid][k];
      lg[k] = v;
      if (a.logits != nullptr) a.logits[s * NOUT + k] = v;
      const float z = v - noise[tid][k];  // Gumbel-max, lowest index on exact ties
      if (z > best) {
        best = z;
        act = k;
      }
    }
    if (sa.sampled) sa.sampled[s] = act;
    if (sa.forced) act = sa.forced[s];
    sa.action[s] = act;
    sa.logp[s] = log_softmax_at(lg, act);
  }
}

// Sequences per workgroup without runs: 16 while that leaves compute units idle, 32 (the same weights for twice the work) beyond.
inline bool gru_seq_tiles16(int64_t S1) { return S1 <= 256 * 16; }
// Workgroups for runs of S steps in all: as many as are resident at once (256 registers, eight wavefronts a compute unit).  16 sequences each for any
// number of them: with 32 a minibatch's two directions take 0.30 + 0.34 ms where they take 0.17 + 0.18 (128 units, 98 304 steps), 1.02 + 1.20 where
// 1.00 + 1.09 (128 units, 1 048 576 steps).
inline int64_t gru_run_places(int waves) { return 256 * std::max(1, 8 / waves); }
inline dim3 gru_run_grid(int64_t S, int waves) { return dim3((unsigned)std::min<int64_t>((S + 15) / 16, gru_run_places(waves))); }
// Does an update of S1 sequences of T steps, episodes of at most `cap`, go run by run?  Where the sequences alone leave most of the chip idle and are long
// enough to be cut.  An update's time in runs over that in whole sequences, 32 .. 256 units, episodes of ten steps / of 50 / none ending: 128 steps of 64
// sequences 0.43 .. 0.61 / 0.45 .. 0.63 / 0.94 .. 1.00; of 512 sequences 0.69 .. 0.82 / 0.60 .. 0.68 / 0.94 .. 0.99; of 1024 0.84 .. 1.06 / 0.71 .. 0.83 /
// 0.95 .. 1.01; of 1536 0.88 .. 1.01 / 0.82 .. 0.94 / 0.94 .. 1.02; of 2048 0.95 .. 1.06 / 0.87 .. 1.02 / 0.98 .. 1.00, so that from there on the longest chain
// has to come out at two thirds or less (256 units, 2048 sequences beside 8192 of 128 units, episodes of 70 steps: an iteration of 387 ms in place of 397); of
// 3072 at 96 units and more 1.02 .. 1.06 / 0.97 .. 1.03 / 0.99 .. 1.01.  Shorter sequences have less to gain and as much to plan: 32 steps, episodes of
// three steps / of ten / none ending, 192 sequences 0.58 .. 0.87 / 0.94 .. 1.01 / 0.98 .. 1.01, 768 0.79 .. 0.94 / 0.91 .. 1.08 / 0.96 .. 1.02, with resident
// weights 1024 to 1536 of episodes of ten steps up to 1.13; 16 steps 0.95 .. 1.05.  Streamed weights, whose steps are longer: 16 steps of 192 sequences 0.88 .. 0.95 in
// episodes of three steps, 32 steps of 1024 0.74 .. 0.84 / 0.95 .. 1.11, 4096 in episodes of five steps 0.90, 8192 1.07 .. 1.11.  At 128
// units whole sequences in tiles of 32 spill registers: in runs 0.95 .. 1.00 of their time above 4096 sequences, of 16 steps as of 128.
inline bool gru_by_runs(int T, int cap, int64_t S1, int H) {
  if (!gru_seq_supported(H)) return false;
  if (H == 128 && !gru_seq_tiles16(S1)) return true;
  if (T < (H > 128 ? 16 : 24)) return false;
  if (S1 <= (H > 128 ? 1536 : 24 * std::min(T, 64))) return true;
  const int64_t chain = std::max<int64_t>(std::min(T, cap), T * S1 / (16 * gru_run_places(H <= 128 ? H / 16 : H / 32)));
  return S1 <= 3072 ? 2 * T >= 3 * chain : H > 128 && gru_seq_tiles16(S1);
}

template <int KS, bool SEG>
inline void launch_gru_fwd_ks(const GruFwdArgs& a, hipStream_t s) {
  constexpr bool RES = KS <= 4;
  constexpr int WAVES = RES ? 2 * KS : KS;
  if constexpr (SEG) hipLaunchKernelGGL((gru_seq_fwd_kernel<KS, 1, RES, true>), gru_run_grid(a.T * a.S1, WAVES), dim3(64 * WAVES), 0, s, a);
  else if (gru_seq_tiles16(a.S1)) hipLaunchKernelGGL((gru_seq_fwd_kernel<KS, 1, RES, false>), dim3((unsigned)((a.S1 + 15) / 16)), dim3(64 * WAVES), 0, s, a);
  else hipLaunchKernelGGL((gru_seq_fwd_kernel<KS, 2, RES, false>), dim3((unsigned)((a.S1 + 31) / 32)), dim3(64 * WAVES), 0, s, a);
}
template <int KS>
inline void launch_gru_actor_ks(const GruActorArgs& a, hipStream_t s) {
  const dim3 block(KS <= 4 ? 128 * KS : 64 * KS);
  if (gru_seq_tiles16(a.S)) hipLaunchKernelGGL((gru_actor_step_kernel<KS, 1>), dim3((unsigned)((a.S + 15) / 16)), block, 0, s, a);
  else hipLaunchKernelGGL((gru_actor_step_kernel<KS, 2>), dim3((unsigned)((a.S + 31) / 32)), block, 0, s, a);
}
template <int KS, bool SEG, int NOUT>
inline void launch_gru_bwd_ks(const GruBwdArgs& a, hipStream_t s) {
  constexpr bool RES = KS <= 4;
  constexpr int WAVES = RES ? 2 * KS : KS;
  if constexpr (SEG) hipLaunchKernelGGL((gru_seq_bwd_kernel<KS, 1, RES, true, NOUT>), gru_run_grid(a.T * a.S1, WAVES), dim3(64 * WAVES), 0, s, a);
  else if (KS == 4 || gru_seq_tiles16(a.S1))  // (128 units, more sequences: in runs)
    hipLaunchKernelGGL((gru_seq_bwd_kernel<KS, 1, RES, false, NOUT>), dim3((unsigned)((a.S1 + 15) / 16)), dim3(64 * WAVES), 0, s, a);
  else if constexpr (KS != 4) hipLaunchKernelGGL((gru_seq_bwd_kernel<KS, 2, RES, false, NOUT>), dim3((unsigned)((a.S1 + 31) / 32)), dim3(64 * WAVES), 0, s, a);
}

}  // namespace marl
