// Recurrent IPPO / MAPPO: a GRU cell in place of the second hidden layer of both networks.
//
//   e = tanh(x We + be);  r = sigma(e Wi_r + bi_r + h Wh_r + bh_r);  z likewise;
//   n = tanh(e Wi_n + bi_n + r (h Wh_n + bh_n));  h' = (1 - z) n + z h;  out = h' W3 + b3
//
// Every product with a weight matrix is an MFMA GEMM (gemm.h); the gate arithmetic is element-wise.  The products
// that do not depend on the hidden state (the embedding e and its gate pre-activations e Wi) run once over all
// T steps of a minibatch of sequences; h Wh and the gates are stepped through time by one kernel each way (gru_seq.h;
// above 256 units by a product and an element-wise kernel per step), and the weight gradients are again taken in one
// product over all steps.
#include <algorithm>
#include <cmath>

#include "gemm.h"
#include "gru_seq.h"
#include "heads.h"
#include "ppo_common.h"

namespace marl {

int32_t launch_env_step(const marl_config& c, marl_env_state st, const int32_t* actions, float* obs, float* reward,
                        uint8_t* done, bool do_step, hipStream_t s);

namespace {

// Offsets (in floats) of one recurrent network's blocks inside the flat parameter vector.
struct RecOffsets {
  int64_t We, be, Wi, bi, Wh, bh, W3, b3, end;
};
RecOffsets rec_offsets(int64_t base, int Din, int H, int Dout) {
  RecOffsets o;
  o.We = base;
  o.be = o.We + (int64_t)Din * H;
  o.Wi = o.be + H;
  o.bi = o.Wi + (int64_t)H * 3 * H;
  o.Wh = o.bi + 3 * H;
  o.bh = o.Wh + (int64_t)H * 3 * H;
  o.W3 = o.bh + 3 * H;
  o.b3 = o.W3 + (int64_t)H * Dout;
  o.end = o.b3 + Dout;
  return o;
}

// Working copy of the parameters with every block on a 64-float boundary (16-byte loads of weight rows).
struct RecParamMap {
  int64_t src[17], dst[17];  // 16 blocks (actor 8, critic 8) + end
  // per network the sequence kernels cover, after the blocks: Wh split and in operand order, for each direction
  int64_t wh_fwd[2], wh_bwd[2];
  int hidden[2];
  int64_t total;
};
RecParamMap rec_param_map(const Dims& d) {
  RecParamMap m;
  const RecOffsets a = rec_offsets(0, d.D, d.Ha, kActions), c = rec_offsets(d.Pa, d.Dc, d.Hc, 1);
  const int64_t src[17] = {a.We, a.be, a.Wi, a.bi, a.Wh, a.bh, a.W3, a.b3, c.We, c.be, c.Wi, c.bi, c.Wh, c.bh, c.W3, c.b3, c.end};
  int64_t off = 0;
  for (int i = 0; i < 17; ++i) {
    m.src[i] = src[i];
    m.dst[i] = off;
    if (i < 16) off += ((src[i + 1] - src[i] + 63) / 64) * 64;
  }
  m.hidden[0] = d.Ha;
  m.hidden[1] = d.Hc;
  for (int n = 0; n < 2; ++n) {
    const int64_t sz = gru_seq_supported(m.hidden[n]) ? gru_weight_floats(m.hidden[n]) : 0;
    m.wh_fwd[n] = off;
    off += sz;
    m.wh_bwd[n] = off;
    off += sz;
  }
  m.total = off;
  return m;
}
RecOffsets rec_padded(const RecParamMap& m, int net) {
  const int64_t* o = m.dst + 8 * net;
  return RecOffsets{o[0], o[1], o[2], o[3], o[4], o[5], o[6], o[7], o[8]};
}

__global__ void rec_stage_params_kernel(const float* __restrict__ src, float* __restrict__ dst, RecParamMap pm) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= pm.src[16]) return;
  int b = 0;
#pragma unroll
  for (int k = 1; k < 16; ++k) b += (i >= pm.src[k]) ? 1 : 0;
  const float v = src[i];
  const int64_t e = i - pm.src[b];
  dst[pm.dst[b] + e] = v;
  if (b == 4 || b == 12) {  // a Wh block [H][3H]
    const int net = b == 12, H = pm.hidden[net];
    if (H <= 256) {
      const int k = (int)(e / (3 * H)), c = (int)(e - (int64_t)k * (3 * H));
      gru_stage_weight<true, true>(v, k, c, H, reinterpret_cast<bf16_t*>(dst + pm.wh_fwd[net]), reinterpret_cast<bf16_t*>(dst + pm.wh_bwd[net]));
    }
  }
}

// dst[s][j] = src[s][j], 0 where reset[s / per] (nullable) is set.  dst may be src.
__global__ void mask_hidden_kernel(const float* src, float* dst, const uint8_t* __restrict__ reset, int64_t n_elems, int H, int per) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_elems) return;
  dst[i] = reset != nullptr && reset[i / H / per] ? 0.f : src[i];
}

// ---- one step at a time, for widths above 256: the arithmetic of gru_seq.h, one thread per (sample, hidden unit) -------
// Gi / Gh are the products without their biases, hprev the state the step starts from.
__global__ void __launch_bounds__(256) gru_forward_kernel(const float* __restrict__ Gi, const float* __restrict__ Gh,
                                                          const float* __restrict__ bi, const float* __restrict__ bh,
                                                          const float* __restrict__ hprev, float* __restrict__ rec,
                                                          float* __restrict__ hout, int64_t S, int H) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= S * H) return;
  const int64_t s = i / H;
  const int j = (int)(i - s * H);
  const float* gi = Gi + s * 3 * H;
  const float* gh = Gh + s * 3 * H;
  const float r = sigmoid_f32((gi[j] + bi[j]) + (gh[j] + bh[j]));
  const float z = sigmoid_f32((gi[H + j] + bi[H + j]) + (gh[H + j] + bh[H + j]));
  const float hn = gh[2 * H + j] + bh[2 * H + j];
  const float n = tanh_f32((gi[2 * H + j] + bi[2 * H + j]) + r * hn);
  if (rec != nullptr) {
    rec[s * 4 * H + j] = hn;
    rec[s * 4 * H + H + j] = r;
    rec[s * 4 * H + 2 * H + j] = z;
    rec[s * 4 * H + 3 * H + j] = n;
  }
  hout[i] = (1.0f - z) * n + z * hprev[i];
}

// dh = gradient from the next step (dh_next, absent at the last step; next_reset: that step started from zero) + the output
// layer's (dl W3^T).  Replaces the step's records by the gradients and writes dh * z, the direct part of the gradient with
// respect to the incoming state (the products with Wh^T are added by GEMMs).
template <int NOUT>
__global__ void __launch_bounds__(256) gru_backward_kernel(const float* __restrict__ dh_next, const uint8_t* __restrict__ next_reset,
                                                           const float* __restrict__ dl, const float* __restrict__ W3,
                                                           float* __restrict__ rec, const float* __restrict__ hs,
                                                           const uint8_t* __restrict__ reset, float* __restrict__ dhprev, int per,
                                                           int64_t S, int H) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= S * H) return;
  const int64_t s = i / H;
  const int j = (int)(i - s * H);
  float dh = dh_next != nullptr && !next_reset[s / per] ? dh_next[i] : 0.f;
#pragma unroll
  for (int k = 0; k < NOUT; ++k) dh = fmaf(dl[s * NOUT + k], W3[(int64_t)j * NOUT + k], dh);
  float* const q = rec + s * 4 * H + j;
  const float hn = q[0], r = q[H], z = q[2 * H], n = q[3 * H];
  const float hprev = reset != nullptr && reset[s / per] ? 0.f : hs[i];
  const float dpre_n = dh * (1.0f - z) * (1.0f - n * n);
  q[0] = dpre_n * r;
  q[H] = dpre_n * hn * r * (1.0f - r);
  q[2 * H] = dh * (hprev - n) * z * (1.0f - z);
  q[3 * H] = dpre_n;
  dhprev[i] = dh * z;
}

// The next minibatches of sequences of an update, blockIdx.y-th of them in every kernel here.  Minibatches planned at once: an epoch's, so that
// the same launches serve them all, but no more than these, so that the room for plans grows neither with the epochs nor with their minibatches.
constexpr int kPlanned = 32;
constexpr int kRunBins = 1024;  // lengths from here on count as one
constexpr int kRunHead = 8;     // ints before a minibatch's bins: number of runs, groups taken by each of its four kernels
struct SeqPlanArgs {
  const int32_t* envs;  // [N] the epoch's order, nullable: the identity
  const uint8_t* done;  // [T][N]
  int J, N, T;
  int first;            // minibatch of the epoch that is the plan's first
  int32_t *rows, *hrows;  // [minibatch of the plan][T * J]
  uint8_t* reset;
  int2* runs;
  int32_t* head;        // [minibatch of the plan][run_head_ints(T)], zero before the first pass
  __device__ __forceinline__ int env(int q, int j) const { const int place = (first + q) * J + j; return envs != nullptr ? envs[place] : place; }
};
__host__ __device__ inline int run_bins(int T) { return T < kRunBins ? T : kRunBins; }
__host__ __device__ inline int64_t run_head_ints(int T) { return (kRunHead + 2 * (int64_t)run_bins(T) + 3) / 4 * 4; }

// Index arrays: row r = t * J + j is trajectory row t * N + envs[j]; reset[r] = the step before t ended the episode of that environment (never at t = 0);
// hrows[r] = the state row that step t starts from, r, or the row of zeros behind the T + 1 slabs.
__global__ void __launch_bounds__(256) seq_index_kernel(SeqPlanArgs a) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x, TJ = (int64_t)a.T * a.J;
  if (r >= TJ) return;
  const int q = blockIdx.y, t = (int)(r / a.J), j = (int)(r - (int64_t)t * a.J), env = a.env(q, j);
  const bool z = t > 0 && a.done[(int64_t)(t - 1) * a.N + env];
  a.rows[q * TJ + r] = t * a.N + env;
  a.reset[q * TJ + r] = z;
  a.hrows[q * TJ + r] = z ? (a.T + 1) * a.J : (int32_t)r;
}

// Runs (SeqRuns), the longest first, in no order among those of one length (a run's results do not depend on which others it shares a workgroup
// with): the first pass counts them by length, the second one places them.  A wavefront takes a sequence, 64 steps a lane each: a lane whose step begins an
// episode ends the run before it.  Four pieces of 64 steps are requested together; a workgroup's counts meet in LDS, so that a few
// atomics per workgroup remain.  (A thread per sequence, with the index arrays among its stores: 128 steps of 32 sequences 76 us in place of 16 with the index arrays' kernel.)
template <bool PLACE, int PER>  // PER: sequences a wavefront takes
__global__ void __launch_bounds__(256) seq_runs_kernel(SeqPlanArgs a) {
  __shared__ int32_t bin[kRunBins], at[kRunBins], wave_sum[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q = blockIdx.y, B = run_bins(a.T);
  const int j0 = (blockIdx.x * 4 + wave) * PER, mine = max(0, min(PER, a.J - j0)), chunks = (a.T + 63) / 64;
  int32_t* const head = a.head + q * run_head_ints(a.T);
  int32_t *const count = head + kRunHead, *const taken = count + B;  // by length, B first
  for (int b = tid; b < B; b += 256) bin[b] = 0;
  __syncthreads();
  int env[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) env[i] = i < mine ? a.env(q, j0 + i) : 0;
  // visits the runs of this wavefront's sequences, at most one a lane at a time
  auto runs = [&](auto&& run) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (i >= mine) break;
      int begin = 0;
      for (int c = 0; c < chunks; c += 4) {
        bool z[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = 64 * (c + u) + lane;
          z[u] = t > 0 && t < a.T && a.done[(int64_t)(t - 1) * a.N + env[i]];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t0 = 64 * (c + u);
          const uint64_t mask = __builtin_amdgcn_ballot_w64(z[u]), below = mask & ((1ull << lane) - 1);
          if (z[u]) {
            const int from = below != 0 ? t0 + 63 - __builtin_clzll(below) : begin;
            run(j0 + i, from, t0 + lane - from);
          }
          if (mask != 0) begin = t0 + 63 - __builtin_clzll(mask);
        }
      }
      if (lane == 0) run(j0 + i, begin, a.T - begin);
    }
  };
  runs([&](int, int, int len) { atomicAdd(&bin[B - min(len, B)], 1); });
  __syncthreads();
  if (!PLACE) {
    for (int b = tid; b < B; b += 256)
      if (bin[b] > 0) atomicAdd(&count[b], bin[b]);
    return;
  }
  // where this workgroup's runs of each length begin: behind the longer ones and those other workgroups have placed
  constexpr int OWN = kRunBins / 256;  // bins a thread adds up
  int own[OWN], sum = 0;
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    const int b = OWN * tid + u;
    own[u] = b < B ? count[b] : 0;
    sum += own[u];
  }
  int before = sum;
#pragma unroll
  for (int o = 1; o < 64; o *= 2) {
    const int v = __shfl_up(before, o);
    if (lane >= o) before += v;
  }
  if (lane == 63) wave_sum[wave] = before;
  __syncthreads();
  before -= sum;
#pragma unroll
  for (int w = 0; w < 4; ++w) before += w < wave ? wave_sum[w] : 0;
  if (blockIdx.x == 0 && tid == 255) head[0] = before + sum;
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    const int b = OWN * tid + u;
    if (b < B) at[b] = before + (bin[b] > 0 ? atomicAdd(&taken[b], bin[b]) : 0);
    before += own[u];
  }
  __syncthreads();
  runs([&](int j, int begin, int len) { a.runs[q * (int64_t)a.T * a.J + atomicAdd(&at[B - min(len, B)], 1)] = make_int2(begin * a.J + j, len); });
}

// with_runs: the index arrays alone where no network takes the runs
void launch_seq_plan(const SeqPlanArgs& a, int minibatches, bool with_runs, hipStream_t s) {
  const unsigned my = (unsigned)minibatches;
  hipLaunchKernelGGL(seq_index_kernel, dim3((unsigned)(((int64_t)a.T * a.J + 255) / 256), my), dim3(256), 0, s, a);
  if (!with_runs) return;
  if (a.J <= 1024) {  // few sequences: a wavefront each, for the shortest chain
    hipLaunchKernelGGL((seq_runs_kernel<false, 1>), dim3((unsigned)((a.J + 3) / 4), my), dim3(256), 0, s, a);
    hipLaunchKernelGGL((seq_runs_kernel<true, 1>), dim3((unsigned)((a.J + 3) / 4), my), dim3(256), 0, s, a);
  } else {  // fewer workgroups that add to the same counts
    hipLaunchKernelGGL((seq_runs_kernel<false, 8>), dim3((unsigned)((a.J + 31) / 32), my), dim3(256), 0, s, a);
    hipLaunchKernelGGL((seq_runs_kernel<true, 8>), dim3((unsigned)((a.J + 31) / 32), my), dim3(256), 0, s, a);
  }
}

// dst[(j * per + a)][u] = h0[(envs[j] * per + a)][u]; zeros[0 .. per * H - 1] = 0
__global__ void gather_hidden_kernel(const float* __restrict__ h0, const int32_t* __restrict__ envs, int J, int per, int H,
                                     float* __restrict__ dst, float* __restrict__ zeros) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)J * per * H) return;
  if (i < per * H) zeros[i] = 0.f;
  const int64_t q = i / H;
  const int u = (int)(i - q * H);
  const int j = (int)(q / per), a = (int)(q - (int64_t)j * per);
  dst[i] = h0[((int64_t)envs[j] * per + a) * H + u];
}

int64_t align256(int64_t x) { return (x + 255) & ~(int64_t)255; }
unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

// gW [M][N] += A^T B over K samples, the column sums of B (the bias gradient) directly behind it.  Every k range stores its own copy in
// `split` and the copies are added in a fixed order; at 98 304 samples, 128 x 384 outputs: 341 ranges adding with atomics 186 us, 170
// copies 70 us.
void weight_gradient(const RowSrc& A, const float* B, int64_t ldb, int M, int N, int64_t K, int c_rot, float* gW, float* split, hipStream_t s) {
  GemmArgs g{};
  g.A = A; g.B = B; g.ldb = ldb; g.C = gW; g.ldc = N; g.c_rot = c_rot;
  g.M = M; g.N = N; g.K = K; g.colsum = gW + (int64_t)M * N;
  g.split_out = split; g.split_count = (int64_t)M * N + N;
  if (launch_gemm<GEMM_TN, EPI_ATOMIC_ADD>(g, s))
    launch_reduce_partials(split, (int)tn_plan(M, N, K).splits, g.split_count, gW, s);
}

const float* stage_params(const Dims& d, const float* params, float* scratch, hipStream_t s) {
  hipLaunchKernelGGL(rec_stage_params_kernel, dim3(blocks_for(d.P)), dim3(256), 0, s, params, scratch, rec_param_map(d));
  return scratch;
}

// e = tanh(X We + be) [S][H] and Gi = e Wi [S][3H] (bias added with the gates)
void embed_and_input_gates(const RowSrc& X, int64_t S, int Din, int H, const float* eff, const RecOffsets& o, float* E,
                           float* Gi, hipStream_t s) {
  GemmArgs g{};
  g.A = X; g.B = eff + o.We; g.ldb = H; g.C = E; g.ldc = H; g.aux_vec = eff + o.be;
  g.M = S; g.N = H; g.K = Din;
  launch_gemm<GEMM_NN, EPI_BIAS_TANH>(g, s);
  GemmArgs g2{};
  g2.A = RowSrc{E, H, nullptr, 1, S}; g2.B = eff + o.Wi; g2.ldb = 3 * H; g2.C = Gi; g2.ldc = 3 * H;
  g2.M = S; g2.N = 3 * H; g2.K = H;
  launch_gemm<GEMM_NN, EPI_STORE>(g2, s);
}

void hidden_gates(const float* hprev, int64_t S, int H, const float* eff, const RecOffsets& o, float* Gh, hipStream_t s) {
  GemmArgs g{};
  g.A = RowSrc{hprev, H, nullptr, 1, S}; g.B = eff + o.Wh; g.ldb = 3 * H; g.C = Gh; g.ldc = 3 * H;
  g.M = S; g.N = 3 * H; g.K = H;
  launch_gemm<GEMM_NN, EPI_STORE>(g, s);
}

// All steps of a, forward; SEG: run by run of a.runs.  GhT [S1][3H] and hm [S1][H] are used above 256 units only.
template <bool SEG>
void gru_forward(const GruFwdArgs& a, int H, const float* eff, const RecOffsets& o, float* GhT, float* hm, hipStream_t s) {
  if (gru_seq_supported(H)) {
    TimedLaunch timed(KC_GEMM_NN, 2.0 * (double)a.T * (double)a.S1 * H * 3.0 * H, s);
    switch (H / 32) {
      case 1: return launch_gru_fwd_ks<1, SEG>(a, s);
      case 2: return launch_gru_fwd_ks<2, SEG>(a, s);
      case 3: return launch_gru_fwd_ks<3, SEG>(a, s);
      case 4: return launch_gru_fwd_ks<4, SEG>(a, s);
      case 5: return launch_gru_fwd_ks<5, SEG>(a, s);
      case 6: return launch_gru_fwd_ks<6, SEG>(a, s);
      case 7: return launch_gru_fwd_ks<7, SEG>(a, s);
      default: return launch_gru_fwd_ks<8, SEG>(a, s);
    }
  }
  for (int t = 0; t < a.T; ++t) {
    const uint8_t* const reset = t > 0 ? a.reset + (int64_t)(t - 1) * (a.S1 / a.per) : a.reset0;
    hipLaunchKernelGGL(mask_hidden_kernel, dim3(blocks_for(a.S1 * H)), dim3(256), 0, s, t > 0 ? a.hs + (int64_t)(t - 1) * a.S1 * H : a.h_first,
                       hm, reset, a.S1 * H, H, a.per);
    hidden_gates(hm, a.S1, H, eff, o, GhT, s);
    hipLaunchKernelGGL(gru_forward_kernel, dim3(blocks_for(a.S1 * H)), dim3(256), 0, s, a.Gi + (int64_t)t * a.S1 * 3 * H, GhT, a.bi, a.bh, hm,
                       a.rec != nullptr ? a.rec + (int64_t)t * a.S1 * 4 * H : (float*)nullptr, a.hs + (int64_t)t * a.S1 * H, a.S1, H);
  }
}

// All steps of a, backward.  dhp [2][S1][H] is used above 256 units only.
template <bool SEG, int NOUT>
void gru_backward(const GruBwdArgs& a, int H, const float* eff, const RecOffsets& o, float* dhp, hipStream_t s) {
  if (gru_seq_supported(H)) {
    TimedLaunch timed(KC_GEMM_NT, 2.0 * (double)(a.T - 1) * (double)a.S1 * H * 3.0 * H, s);
    switch (H / 32) {
      case 1: return launch_gru_bwd_ks<1, SEG, NOUT>(a, s);
      case 2: return launch_gru_bwd_ks<2, SEG, NOUT>(a, s);
      case 3: return launch_gru_bwd_ks<3, SEG, NOUT>(a, s);
      case 4: return launch_gru_bwd_ks<4, SEG, NOUT>(a, s);
      case 5: return launch_gru_bwd_ks<5, SEG, NOUT>(a, s);
      case 6: return launch_gru_bwd_ks<6, SEG, NOUT>(a, s);
      case 7: return launch_gru_bwd_ks<7, SEG, NOUT>(a, s);
      default: return launch_gru_bwd_ks<8, SEG, NOUT>(a, s);
    }
  }
  const int64_t J = a.S1 / a.per;
  for (int t = a.T - 1; t >= 0; --t) {
    float* const out = dhp + (int64_t)(t & 1) * a.S1 * H;
    float* const rec = a.rec + (int64_t)t * a.S1 * 4 * H;
    const bool last = t == a.T - 1;
    hipLaunchKernelGGL(gru_backward_kernel<NOUT>, dim3(blocks_for(a.S1 * H)), dim3(256), 0, s,
                       last ? (const float*)nullptr : dhp + (int64_t)((t + 1) & 1) * a.S1 * H, last ? (const uint8_t*)nullptr : a.reset + t * J,
                       a.dl + (int64_t)t * a.S1 * NOUT, a.W3, rec, a.hs + (int64_t)t * a.S1 * H, t > 0 ? a.reset + (t - 1) * J : (const uint8_t*)nullptr,
                       out, a.per, a.S1, H);
    if (t == 0) break;
    // dL/dhprev += dgh Wh^T: the columns of r and z, then the one of the new gate, which the records hold first
    GemmArgs g{};
    g.A = RowSrc{rec + H, 4 * H, nullptr, 1, a.S1}; g.B = eff + o.Wh; g.ldb = 3 * H; g.C = out; g.ldc = H;
    g.M = a.S1; g.N = H; g.K = 2 * H;
    launch_gemm<GEMM_NT, EPI_ATOMIC_ADD>(g, s);
    g.A = RowSrc{rec, 4 * H, nullptr, 1, a.S1}; g.B = eff + o.Wh + 2 * H; g.K = H;
    launch_gemm<GEMM_NT, EPI_ATOMIC_ADD>(g, s);
  }
}

// ---- rollout ---------------------------------------------------------------------------------------------

// The critic's values do not steer the rollout: it runs over the stored observations afterwards, this many steps at a time: as
// many as keep a chunk at 32 768 samples, whose intermediate results take 20 H bytes each.  (At 1024 environments of three agents,
// 128 units, the workspace is 83 MB and the rollout takes 3.91 ms; chunks of 131 072 samples: 334 MB and 3.78 ms.  At 16 384
// environments with a central critic of 256 units: 207 MB and 34.0 ms, 710 MB and 33.2 ms.)
int64_t rec_critic_steps(const Dims& d) {
  const int64_t Sc = d.central ? d.N : d.NA;
  return std::max<int64_t>(1, std::min<int64_t>(d.T + 1, 32768 / Sc));
}

struct RecRolloutWs {
  float *eff, *we, *wi, *ha, *hm, *E, *Gi, *Gh, *Hs;
};
RecRolloutWs carve_rec_rollout(const marl_config& c, void* ws, int64_t* total) {
  const Dims d = dims_of(c);
  const int64_t Sc = d.central ? d.N : d.NA, chunk = rec_critic_steps(d) * Sc;
  const bool fused_actor = gru_seq_supported(d.Ha), stepped_critic = !gru_seq_supported(d.Hc);
  const int64_t one_a = fused_actor ? 0 : d.NA * d.Ha, one_c = stepped_critic ? Sc * d.Hc : 0;  // one step's buffers
  char* p = static_cast<char*>(ws);
  int64_t off = 0;
  auto take = [&](int64_t bytes) {
    char* r = p + off;
    off += align256(bytes);
    return (float*)r;
  };
  RecRolloutWs w;
  w.eff = take(rec_param_map(d).total * 4);
  w.we = take(fused_actor ? gru_embedding_floats(d.D, d.Ha) * 4 : 0);
  w.wi = take(fused_actor ? gru_weight_floats(d.Ha) * 4 : 0);
  w.ha = take(d.NA * d.Ha * 4);
  w.hm = take(std::max(one_a, one_c) * 4);
  w.Gh = take(3 * std::max(one_a, one_c) * 4);
  w.E = take(std::max(one_a, chunk * d.Hc) * 4);
  w.Gi = take(3 * std::max(one_a, chunk * d.Hc) * 4);
  w.Hs = take(chunk * d.Hc * 4);
  if (total) *total = off;
  return w;
}

// The actor's embedding [D][H] and input-gate weights [H][3H] for gru_actor_step_kernel.
__global__ void rec_stage_actor_kernel(const float* __restrict__ We, const float* __restrict__ Wi, int D, int K1, int H,
                                       bf16_t* __restrict__ we, bf16_t* __restrict__ wi) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < K1 * H) {
    const int k = i / H, u = i - k * H;
    gru_stage_embedding(k < D ? We[k * H + u] : 0.f, k, u, K1, we);
  } else if (i < K1 * H + 3 * H * H) {
    const int e = i - K1 * H, k = e / (3 * H);
    gru_stage_weight<true, false>(Wi[e], k, e - k * 3 * H, H, wi, nullptr);
  }
}

void launch_actor_step(const GruActorArgs& a, int H, hipStream_t s) {
  TimedLaunch timed(KC_GEMM_NN, 2.0 * (double)a.S * H * ((double)a.D + 6.0 * H), s);
  switch (H / 32) {
    case 1: return launch_gru_actor_ks<1>(a, s);
    case 2: return launch_gru_actor_ks<2>(a, s);
    case 3: return launch_gru_actor_ks<3>(a, s);
    case 4: return launch_gru_actor_ks<4>(a, s);
    case 5: return launch_gru_actor_ks<5>(a, s);
    case 6: return launch_gru_actor_ks<6>(a, s);
    case 7: return launch_gru_actor_ks<7>(a, s);
    default: return launch_gru_actor_ks<8>(a, s);
  }
}

}  // namespace

int64_t rec_rollout_workspace_bytes(const marl_config& c) {
  int64_t total = 0;
  carve_rec_rollout(c, nullptr, &total);
  return total;
}

int32_t launch_rollout_recurrent(const marl_config& c, marl_env_state st, const float* params, marl_traj tr,
                                 marl_rec_state rec, uint64_t step_offset, const int32_t* forced_actions,
                                 const float* forced_uniforms, void* workspace, hipStream_t s) {
  const Dims d = dims_of(c);
  const RecRolloutWs w = carve_rec_rollout(c, workspace, nullptr);
  const float* eff = stage_params(d, params, w.eff, s);
  const RecParamMap pm = rec_param_map(d);
  const RecOffsets oa = rec_padded(pm, 0), oc = rec_padded(pm, 1);
  const int64_t NA = d.NA, slab = NA * d.D;
  const int64_t Sc = d.central ? d.N : NA;
  const int per_c = d.central ? 1 : d.A;
  const bool fused_actor = gru_seq_supported(d.Ha);
  if (fused_actor) {
    const int K1 = (d.D + 31) / 32 * 32;
    hipLaunchKernelGGL(rec_stage_actor_kernel, dim3(blocks_for((int64_t)K1 * d.Ha + 3 * (int64_t)d.Ha * d.Ha)), dim3(256), 0, s, eff + oa.We,
                       eff + oa.Wi, d.D, K1, d.Ha, reinterpret_cast<bf16_t*>(w.we), reinterpret_cast<bf16_t*>(w.wi));
  }
  int32_t rc = launch_env_step(c, st, nullptr, tr.obs, nullptr, nullptr, /*do_step=*/false, s);
  if (rc != MARL_OK) return rc;
  for (int t = 0; t < d.T; ++t) {
    const uint8_t* ended = t > 0 ? tr.done + (int64_t)(t - 1) * d.N : (const uint8_t*)nullptr;  // a new episode starts from the zero state
    const float* obs_t = tr.obs + (int64_t)t * slab;
    const float* h_in = t > 0 ? w.ha : rec.ha0;
    float* const logits = tr.logits ? tr.logits + (int64_t)t * NA * kActions : (float*)nullptr;
    SampleArgs a{};
    a.uniforms = forced_uniforms ? forced_uniforms + (int64_t)t * NA * kActions : nullptr;
    a.forced = forced_actions ? forced_actions + (int64_t)t * NA : nullptr;
    a.action = tr.action + (int64_t)t * NA;
    a.sampled = tr.sampled ? tr.sampled + (int64_t)t * NA : nullptr;
    a.logp = tr.logp + (int64_t)t * NA;
    a.step = step_offset + (uint64_t)t;
    a.k0 = (uint32_t)(c.seed & 0xffffffffu);
    a.k1 = (uint32_t)(c.seed >> 32);
    if (fused_actor) {
      GruActorArgs g{};
      g.obs = obs_t; g.We = reinterpret_cast<const bf16_t*>(w.we); g.Wi = reinterpret_cast<const bf16_t*>(w.wi);
      g.Wh = reinterpret_cast<const bf16_t*>(eff + pm.wh_fwd[0]); g.be = eff + oa.be; g.bi = eff + oa.bi; g.bh = eff + oa.bh;
      g.W3 = eff + oa.W3; g.b3 = eff + oa.b3; g.h_in = h_in; g.h_out = w.ha; g.reset = ended; g.per = d.A; g.S = NA; g.D = d.D;
      g.logits = logits; g.sample = a;
      launch_actor_step(g, d.Ha, s);
    } else {
      embed_and_input_gates(RowSrc{obs_t, d.D, nullptr, 1, NA}, NA, d.D, d.Ha, eff, oa, w.E, w.Gi, s);
      GruFwdArgs g{};
      g.Gi = w.Gi; g.bi = eff + oa.bi; g.bh = eff + oa.bh; g.h_first = h_in; g.hs = w.ha; g.reset0 = ended; g.per = d.A; g.S1 = NA; g.T = 1;
      gru_forward<false>(g, d.Ha, eff, oa, w.Gh, w.hm, s);
      launch_actor_head_rollout(w.ha, NA, d.Ha, eff + oa.W3, eff + oa.b3, logits, &a, s);
    }
    rc = launch_env_step(c, st, a.action, tr.obs + (int64_t)(t + 1) * slab, tr.reward + (int64_t)t * NA,
                         tr.done + (int64_t)t * d.N, true, s);
    if (rc != MARL_OK) return rc;
  }
  const uint8_t* ended = tr.done + (int64_t)(d.T - 1) * d.N;
  hipLaunchKernelGGL(mask_hidden_kernel, dim3(blocks_for(NA * d.Ha)), dim3(256), 0, s, w.ha, rec.ha1, ended, NA * d.Ha, d.Ha, d.A);
  // the critic over the observations of steps 0 .. T; the last is the bootstrap value, and the hidden state of the next
  // rollout is the one before it
  const int64_t steps = rec_critic_steps(d);
  int64_t n_prev = 0;
  for (int64_t t0 = 0; t0 <= d.T; t0 += steps) {
    const int64_t n = std::min<int64_t>(steps, d.T + 1 - t0);
    embed_and_input_gates(RowSrc{tr.obs + t0 * slab, d.Dc, nullptr, 1, n * Sc}, n * Sc, d.Dc, d.Hc, eff, oc, w.E, w.Gi, s);
    GruFwdArgs g{};
    g.Gi = w.Gi; g.W = reinterpret_cast<const bf16_t*>(eff + pm.wh_fwd[1]); g.bi = eff + oc.bi; g.bh = eff + oc.bh;
    g.h_first = t0 > 0 ? w.Hs + (n_prev - 1) * Sc * d.Hc : rec.hc0; g.hs = w.Hs;
    g.reset0 = t0 > 0 ? tr.done + (t0 - 1) * d.N : (const uint8_t*)nullptr; g.reset = tr.done + t0 * d.N;
    g.per = per_c; g.S1 = Sc; g.T = (int)n;
    gru_forward<false>(g, d.Hc, eff, oc, w.Gh, w.hm, s);
    const int64_t nv = std::min<int64_t>(n, d.T - t0);  // steps with a value of their own
    if (nv > 0) launch_critic_head_rollout(w.Hs, nv * Sc, d.Hc, eff + oc.W3, eff + oc.b3, tr.value + t0 * NA, d.central ? d.A : 1, s);
    if (nv < n) launch_critic_head_rollout(w.Hs + nv * Sc * d.Hc, Sc, d.Hc, eff + oc.W3, eff + oc.b3, tr.last_value, d.central ? d.A : 1, s);
    if (t0 <= d.T - 1 && d.T - 1 < t0 + n)
      hipLaunchKernelGGL(mask_hidden_kernel, dim3(blocks_for(Sc * d.Hc)), dim3(256), 0, s, w.Hs + (d.T - 1 - t0) * Sc * d.Hc, rec.hc1, ended,
                         Sc * d.Hc, d.Hc, per_c);
    n_prev = n;
  }
  return launch_status();
}

// ---- sequence PPO update ------------------------------------------------------------------------------------

namespace {

// buffers of one network's forward and backward pass over a minibatch
struct RecNetWs {
  float *dl, *E, *G, *R, *Hs, *GhT, *hm, *dHp, *partial, *split;  // R: records [S][4H]; Hs: states, T + 1 slabs and one row of zeros
};
struct RecUpdateWs {
  float *eff, *grad;
  Scalars* sc;
  SeqPlanArgs plan;
  RecNetWs net[2];  // actor, critic: a set each, so that the two networks can run side by side
};

RecUpdateWs carve_rec_update(const marl_config& c, void* ws, int64_t* total) {
  const Dims d = dims_of(c);
  const int64_t J = d.N / c.n_minibatches, TJ = (int64_t)d.T * J;
  const int64_t Sa = TJ * d.A, Sc = d.central ? TJ : Sa;                // samples of a minibatch over all steps
  const int64_t S1a = J * d.A, S1c = d.central ? J : S1a;              // samples of one step
  char* p = static_cast<char*>(ws);
  int64_t off = 0;
  auto take = [&](int64_t bytes) {
    char* r = p + off;
    off += align256(bytes);
    return r;
  };
  RecUpdateWs w;
  w.eff = (float*)take(rec_param_map(d).total * 4);
  w.grad = (float*)take(d.P * 4);
  w.sc = (Scalars*)take(sizeof(Scalars));
  w.plan = SeqPlanArgs{};
  w.plan.J = (int)J; w.plan.N = d.N; w.plan.T = d.T;
  const int64_t planned = std::min(c.n_minibatches, kPlanned);
  w.plan.rows = (int32_t*)take(planned * TJ * 4);
  w.plan.hrows = (int32_t*)take(planned * TJ * 4);
  w.plan.reset = (uint8_t*)take(planned * TJ);
  w.plan.runs = (int2*)take(planned * TJ * 8);
  w.plan.head = (int32_t*)take(planned * run_head_ints(d.T) * 4);
  for (int k = 0; k < 2; ++k) {
    const int64_t SH = k == 0 ? Sa * d.Ha : Sc * d.Hc, S1H = k == 0 ? S1a * d.Ha : S1c * d.Hc;
    const int H = k == 0 ? d.Ha : d.Hc;
    RecNetWs& n = w.net[k];
    n.dl = (float*)take((k == 0 ? Sa * kActions : Sc) * 4);
    n.E = (float*)take(SH * 4);
    n.G = (float*)take(3 * SH * 4);
    n.R = (float*)take(4 * SH * 4);
    n.Hs = (float*)take((SH + S1H + (int64_t)(k == 0 || !d.central ? d.A * H : H)) * 4);
    const int64_t step = gru_seq_supported(H) ? 0 : S1H;  // one step's buffers
    n.GhT = (float*)take(3 * step * 4);
    n.hm = (float*)take(step * 4);
    n.dHp = (float*)take(2 * step * 4);
    n.partial = (float*)take(loss_head_partial_floats(H, k == 0 ? kActions : 1) * 4);
    n.split = (float*)take(std::max(tn_copy_floats(H, 3 * H, k == 0 ? Sa : Sc), tn_copy_floats(k == 0 ? d.D : d.Dc, H, k == 0 ? Sa : Sc)) * 4);
  }
  if (total) *total = off;
  return w;
}

// Forward over the T steps, loss, and back-propagation through time of one network on a minibatch of J sequences
// (`per` samples per environment row).  Samples are ordered [t][j][a].
template <int NOUT, class LossFn>
int32_t train_net_recurrent(const RowSrc& X, int T, int64_t J, int per, int Din, int H, const float* h0,
                            const int32_t* envs, const float* eff, const RecOffsets& o, const float* wh_fwd,
                            const float* wh_bwd, float* grad, const RecOffsets& go, const LossFn& fn, const RecNetWs& w,
                            const uint8_t* reset, const int32_t* hrows, bool by_runs, const SeqRuns& runs, Scalars* sc, hipStream_t s) {
  const int64_t S1 = J * per, S = (int64_t)T * S1;
  hipLaunchKernelGGL(gather_hidden_kernel, dim3(blocks_for(S1 * H)), dim3(256), 0, s, h0, envs, (int)J, per, H, w.Hs, w.Hs + (S + S1) * H);
  embed_and_input_gates(X, S, Din, H, eff, o, w.E, w.G, s);
  GruFwdArgs f{};
  f.Gi = w.G; f.W = reinterpret_cast<const bf16_t*>(wh_fwd); f.bi = eff + o.bi; f.bh = eff + o.bh;
  f.h_first = w.Hs; f.hs = w.Hs + S1 * H; f.rec = w.R; f.reset = reset + J; f.per = per; f.S1 = S1; f.T = T;
  f.runs = runs;
  if (by_runs) gru_forward<true>(f, H, eff, o, w.GhT, w.hm, s);
  else gru_forward<false>(f, H, eff, o, w.GhT, w.hm, s);
  // output layer, loss, dL/dout, W3 / b3 gradient over all steps
  const int32_t rc = launch_loss_head<NOUT, false>(w.Hs + S1 * H, S, H, eff + o.W3, eff + o.b3, fn, w.dl, grad + go.W3, w.partial, sc, s);
  if (rc != MARL_OK) return rc;
  GruBwdArgs bw{};
  bw.W = reinterpret_cast<const bf16_t*>(wh_bwd); bw.W3 = eff + o.W3; bw.dl = w.dl; bw.rec = w.R; bw.hs = w.Hs; bw.reset = reset + J;
  bw.per = per; bw.S1 = S1; bw.T = T;
  bw.runs = runs;
  bw.runs.next += 1;
  if (by_runs) gru_backward<true, NOUT>(bw, H, eff, o, w.dHp, s);
  else gru_backward<false, NOUT>(bw, H, eff, o, w.dHp, s);
  const float* const dgh = w.R;      // [S][4H], columns n, r, z
  const float* const dgi = w.R + H;  // [S][4H], columns r, z, n
  // gWh += (states the steps start from)^T dGh, the new gate's columns last; gWi += E^T dGi
  weight_gradient(RowSrc{w.Hs, H, hrows, per, S}, dgh, 4 * H, H, 3 * H, S, 2 * H, grad + go.Wh, w.split, s);
  weight_gradient(RowSrc{w.E, H, nullptr, 1, S}, dgi, 4 * H, H, 3 * H, S, 0, grad + go.Wi, w.split, s);
  {  // dE = (dGi Wi^T) * (1 - e^2), in place over e
    GemmArgs g{};
    g.A = RowSrc{dgi, 4 * H, nullptr, 1, S}; g.B = eff + o.Wi; g.ldb = 3 * H; g.C = w.E; g.ldc = H;
    g.aux_mat = w.E; g.ldaux = H; g.M = S; g.N = H; g.K = 3 * H;
    launch_gemm<GEMM_NT, EPI_DTANH>(g, s);
  }
  weight_gradient(X, w.E, H, Din, H, S, 0, grad + go.We, w.split, s);
  return MARL_OK;
}

}  // namespace

int64_t rec_update_workspace_bytes(const marl_config& c) {
  int64_t total = 0;
  carve_rec_update(c, nullptr, &total);
  return total;
}

int32_t launch_ppo_update_recurrent(const marl_config& c, marl_traj tr, marl_rec_state rec, float* params, float* adam_m,
                                    float* adam_v, int64_t adam_step0, const int32_t* perm, float* stats,
                                    float* grad_dump, void* workspace, hipStream_t s) {
  const Dims d = dims_of(c);
  const RecUpdateWs w = carve_rec_update(c, workspace, nullptr);
  const int64_t J = d.N / c.n_minibatches, TJ = (int64_t)d.T * J;
  const RecOffsets ga = rec_offsets(0, d.D, d.Ha, kActions), gc = rec_offsets(d.Pa, d.Dc, d.Hc, 1);
  const RecParamMap pm = rec_param_map(d);
  const RecOffsets oa = rec_padded(pm, 0), oc = rec_padded(pm, 1);
  const SideStream* const side = side_stream();
  const bool by_runs_a = gru_by_runs(d.T, c.episode_cap, J * d.A, d.Ha), by_runs_c = gru_by_runs(d.T, c.episode_cap, d.central ? J : J * d.A, d.Hc);
  SeqPlanArgs plan = w.plan;
  plan.done = tr.done;
  int64_t k = adam_step0;
  for (int e = 0; e < c.n_epochs; ++e) {
    for (int mb = 0; mb < c.n_minibatches; ++mb) {
      const int q = mb % kPlanned;
      int32_t *const rows = w.plan.rows + q * TJ, *const hrows = w.plan.hrows + q * TJ, *const head = w.plan.head + q * run_head_ints(d.T);
      const uint8_t* const reset = w.plan.reset + q * TJ;
      const SeqRuns runs_a{w.plan.runs + q * TJ, head, head + 1, 0}, runs_c{w.plan.runs + q * TJ, head, head + 3, 1};
      const float* eff = stage_params(d, params, w.eff, s);
      const int planned = q == 0 ? std::min(c.n_minibatches - mb, kPlanned) : 0;  // clears the heads of their plans too
      hipLaunchKernelGGL(zero_step_kernel, dim3(blocks_for(d.P)), dim3(256), 0, s, w.grad, d.P, w.sc, 1, (double*)(planned ? w.plan.head : nullptr),
                         (int)(planned * run_head_ints(d.T) / 2));
      if (planned) {
        plan.envs = perm != nullptr ? perm + (int64_t)e * d.N : nullptr;
        plan.first = mb;
        launch_seq_plan(plan, planned, by_runs_a || by_runs_c, s);
      }
      LossCommon lc{};
      lc.rows = rows; lc.A = d.A; lc.ad = make_small_div(d.A); lc.rows_mb = TJ; lc.inv_B = (float)(1.0 / (double)(TJ * d.A));
      lc.sc = w.sc; lc.adv_stats = &w.sc->adv_sum; lc.normalize = c.normalize_adv; lc.clip_eps = c.clip_eps; lc.ent_coef = c.ent_coef;
      lc.vf_coef = c.vf_coef; lc.clip_value = c.clip_value;
      if (c.normalize_adv) {
        const unsigned nb = (unsigned)std::min<int64_t>(256, (TJ * d.A + 255) / 256);
        hipLaunchKernelGGL(adv_stats_kernel, dim3(nb), dim3(256), 0, s, tr.adv, lc, w.sc);
      }
      // The two networks share nothing but their inputs and write disjoint parts of the gradient: the critic runs on the
      // second stream beside the actor.  A time step of either is a short chain of dependent matrix instructions on a
      // few hundred workgroups, so the two chains interleave on the compute units instead of following one another.
      hipStream_t s2 = s;
      if (side != nullptr && hipEventRecord(side->fork, s) == hipSuccess && hipStreamWaitEvent(side->stream, side->fork, 0) == hipSuccess)
        s2 = side->stream;
      int32_t rc_a, rc_c;
      {
        ActorLoss fn{lc, tr.action, tr.logp, tr.adv};
        rc_a = train_net_recurrent<kActions>(RowSrc{tr.obs, d.D, rows, d.A, TJ * d.A}, d.T, J, d.A, d.D, d.Ha, rec.ha0, rows,
                                             eff, oa, eff + pm.wh_fwd[0], eff + pm.wh_bwd[0], w.grad, ga, fn, w.net[0], reset,
                                             hrows, by_runs_a, runs_a, w.sc, s);
      }
      {
        CriticLoss fn{lc, tr.ret, tr.value, d.central ? d.A : 1};
        const int per = d.central ? 1 : d.A;
        rc_c = train_net_recurrent<1>(RowSrc{tr.obs, d.Dc, rows, per, TJ * per}, d.T, J, per, d.Dc, d.Hc, rec.hc0, rows, eff,
                                      oc, eff + pm.wh_fwd[1], eff + pm.wh_bwd[1], w.grad, gc, fn, w.net[1], reset, hrows, by_runs_c, runs_c, w.sc, s2);
      }
      if (s2 != s) {  // join also after an error, so that the caller's stream never runs ahead of work still queued beside it
        if (hipEventRecord(side->join, s2) != hipSuccess || hipStreamWaitEvent(s, side->join, 0) != hipSuccess) {
          (void)hipStreamSynchronize(s2);
          return MARL_E_LAUNCH;
        }
      }
      if (rc_a != MARL_OK) return rc_a;
      if (rc_c != MARL_OK) return rc_c;
      hipLaunchKernelGGL(grad_norm_kernel, dim3(grad_norm_blocks(d.P)), dim3(256), 0, s,
                         w.grad, d.P, w.sc);
      ++k;
      AdamArgs a{};
      a.norm_blocks = (int)grad_norm_blocks(d.P);
      a.lr = c.lr; a.b1 = c.beta1; a.b2 = c.beta2; a.eps = c.adam_eps;
      a.bc1 = (float)(1.0 - std::pow((double)c.beta1, (double)k));
      a.bc2 = (float)(1.0 - std::pow((double)c.beta2, (double)k));
      a.max_norm = c.max_grad_norm; a.ent_coef = c.ent_coef; a.vf_coef = c.vf_coef;
      const bool last = (e == c.n_epochs - 1 && mb == c.n_minibatches - 1);
      hipLaunchKernelGGL(adam_kernel<NoStage>, dim3(blocks_for(d.P)), dim3(256), 0, s, params, adam_m, adam_v, w.grad, d.P, a, w.sc,
                         stats + (int64_t)(e * c.n_minibatches + mb) * MARL_N_STATS, (last ? grad_dump : (float*)nullptr),
                         (Scalars*)nullptr, NoStage{});
      const int32_t rc = launch_status();
      if (rc != MARL_OK) return rc;
    }
  }
  return MARL_OK;
}

}  // namespace marl
