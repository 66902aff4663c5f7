// Pieces of the PPO update shared by the feed-forward and the recurrent drivers: per-minibatch device scalars,
// the actor and critic loss functors (loss terms and dL/d(output) of one sample), the output-layer + loss
// kernel of the layer-wise paths, advantage statistics, gradient-norm and Adam kernels.
#pragma once
#include <algorithm>
#include <cmath>

#include "gemm.h"
#include "heads.h"
#include "stage_params.h"

namespace marl {
namespace {

constexpr int kNormBlocks = 256;

// Device scalars of one minibatch step.
struct Scalars {
  double adv_sum, adv_sq;  // sum of the minibatch's advantages, sum of their squares
  float acc[8];            // 0 policy loss, 1 value loss, 2 entropy, 3 approx KL, 4 clip fraction
  double norm_part[kNormBlocks];  // |grad|^2 summed per workgroup of grad_norm_kernel; adam_kernel adds them in order
};

struct LossCommon {
  const int32_t* rows;  // [rows_mb] trajectory row of each minibatch row
  int A;
  SmallDiv ad;          // make_small_div(A)
  int64_t rows_mb;
  float inv_B;  // 1 / (rows_mb * A)
  const Scalars* sc;
  const double* adv_stats;  // sum and sum of squares of this minibatch's advantages
  int normalize;
  float clip_eps, ent_coef, vf_coef;
  int clip_value;
};

__global__ void iota_kernel(int32_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = (int32_t)i;
}

// Zeroes the gradient, `nsc` sets of scalars and `nextra` doubles (nullable).
__global__ void zero_step_kernel(float* grad, int64_t P, Scalars* sc, int nsc, double* extra, int nextra) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < P) grad[i] = 0.f;
  if (i < nsc) {
    sc[i].adv_sum = 0.0;
    sc[i].adv_sq = 0.0;
    for (int k = 0; k < 8; ++k) sc[i].acc[k] = 0.f;
  }
  if (extra != nullptr)
    for (int64_t j = i; j < nextra; j += (int64_t)gridDim.x * blockDim.x) extra[j] = 0.0;
}

__device__ __forceinline__ double block_sum_f64(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[wave] = v;
  __syncthreads();
  double t = 0;
  if (threadIdx.x == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
  return t;  // valid in thread 0
}

// Sum and sum of squares of the minibatch's advantages, both in fp64 (the variance is their difference: with fp32
// inputs and fp64 sums the cancellation costs nothing that matters until the spread is 1e-6 of the mean).
__global__ void __launch_bounds__(256) adv_stats_kernel(const float* __restrict__ adv, LossCommon lc, Scalars* sc) {
  __shared__ double red[2][4];
  const int64_t B = lc.rows_mb * lc.A;
  double sum = 0, sq = 0;
  for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < B; s += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = s / lc.A;
    const int a = (int)(s - row * lc.A);
    const double x = adv[(int64_t)lc.rows[row] * lc.A + a];
    sum += x;
    sq += x * x;
  }
  const double t0 = block_sum_f64(sum, red[0]);
  const double t1 = block_sum_f64(sq, red[1]);
  if (threadIdx.x == 0) {
    atomicAdd(&sc->adv_sum, t0);
    atomicAdd(&sc->adv_sq, t1);
  }
}

// The same for every minibatch of an update in one launch: blockIdx.y = e * n_minibatches + mb; the row order of
// epoch e starts at rows + e * epoch_stride, minibatch mb takes its rows mb * rows_mb .. ; out[2 (e * n_minibatches + mb)]
// gets the sum, the next double the sum of squares (zeroed before the launch).
__global__ void __launch_bounds__(256) adv_stats_all_kernel(const float* __restrict__ adv, const int32_t* __restrict__ rows,
                                                            int64_t epoch_stride, int n_minibatches, int64_t rows_mb, int A,
                                                            double* __restrict__ out) {
  __shared__ double red[2][4];
  const int m = blockIdx.y, e = m / n_minibatches, mb = m - e * n_minibatches;
  const int32_t* const r0 = rows + e * epoch_stride + (int64_t)mb * rows_mb;
  const int64_t B = rows_mb * A;
  double sum = 0, sq = 0;
  for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < B; s += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = s / A;
    const int a = (int)(s - row * A);
    const double x = adv[(int64_t)r0[row] * A + a];
    sum += x;
    sq += x * x;
  }
  const double t0 = block_sum_f64(sum, red[0]);
  const double t1 = block_sum_f64(sq, red[1]);
  if (threadIdx.x == 0) {
    atomicAdd(&out[2 * m], t0);
    atomicAdd(&out[2 * m + 1], t1);
  }
}

// exp and log on the hardware exp2 / log2 units (1 ulp each; the arguments here are O(1))
__device__ __forceinline__ float fast_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }
__device__ __forceinline__ float fast_log(float x) { return __builtin_amdgcn_logf(x) * 0.6931471805599453f; }

// Per-minibatch constants of a loss, computed once per thread instead of once per sample.
struct LossPrep {
  float mean, rstd;
};

struct ActorLoss {
  static constexpr unsigned kStats = 0b11101;  // the statistics that compute() adds to, by their index
  LossCommon lc;
  const int32_t* action;
  const float* logp_old;
  const float* adv;
  struct In {
    int act;
    float logp_old, adv;
  };
  // the trajectory values of minibatch sample s (separate from the arithmetic so that they can be fetched early);
  // row_entry / load_with split the dependent pair of loads so that the first can be issued a phase ahead
  // (FAST: the magic-number division of SmallDiv, for callers that have checked small_div_ok(lc.ad, samples))
  template <bool FAST = false>
  __device__ __forceinline__ int32_t row_entry(int64_t s) const { return lc.rows[lc.ad.div<FAST>(s, lc.A)]; }
  template <bool FAST = false>
  __device__ __forceinline__ In load_with(int64_t s, int32_t entry) const {
    const int a = (int)(s - lc.ad.div<FAST>(s, lc.A) * lc.A);
    const int64_t src = (int64_t)entry * lc.A + a;
    return In{action[src], logp_old[src], adv[src]};
  }
  __device__ __forceinline__ In load(int64_t s) const { return load_with(s, row_entry(s)); }
  __device__ __forceinline__ LossPrep prepare() const {
    LossPrep p{0.f, 1.f};
    if (lc.normalize) {
      const double B = (double)lc.rows_mb * lc.A;
      const double mean = lc.adv_stats[0] / B;
      p.mean = (float)mean;
      p.rstd = (float)(1.0 / (sqrt(fmax(lc.adv_stats[1] / B - mean * mean, 0.0)) + 1e-8));
    }
    return p;
  }
  // returns dL/dlogits in dl; adds this sample's terms to st[0..4]
  __device__ __forceinline__ void compute(const In& in, const LossPrep& prep, const float out[kActions], float dl[kActions],
                                          float st[5]) const {
    const int act = in.act;
    float m = out[0];
#pragma unroll
    for (int k = 1; k < kActions; ++k) m = fmaxf(m, out[k]);
    float ex[kActions], se = 0.f;
#pragma unroll
    for (int k = 0; k < kActions; ++k) {
      ex[k] = fast_exp(out[k] - m);
      se += ex[k];
    }
    const float lse = m + fast_log(se), rse = __builtin_amdgcn_rcpf(se);
    float lp[kActions], p[kActions], ent = 0.f, logp_new = 0.f;
#pragma unroll
    for (int k = 0; k < kActions; ++k) {
      lp[k] = out[k] - lse;
      p[k] = ex[k] * rse;
      ent -= p[k] * lp[k];
      logp_new = (k == act) ? lp[k] : logp_new;
    }
    float advn = in.adv;
    if (lc.normalize) advn = (advn - prep.mean) * prep.rstd;
    const float log_ratio = logp_new - in.logp_old;
    const float ratio = fast_exp(log_ratio);
    const float rc = fminf(fmaxf(ratio, 1.0f - lc.clip_eps), 1.0f + lc.clip_eps);
    const float s1 = ratio * advn, s2 = rc * advn;
    st[0] += -fminf(s1, s2) * lc.inv_B;
    st[2] += ent * lc.inv_B;
    st[3] += ((ratio - 1.0f) - log_ratio) * lc.inv_B;
    st[4] += (fabsf(ratio - 1.0f) > lc.clip_eps ? 1.0f : 0.0f) * lc.inv_B;
    const float dlogp = (s1 <= s2) ? -(advn * ratio) * lc.inv_B : 0.0f;
    const float ec = lc.ent_coef * lc.inv_B;
#pragma unroll
    for (int k = 0; k < kActions; ++k) dl[k] = dlogp * ((k == act ? 1.0f : 0.0f) - p[k]) + ec * p[k] * (lp[k] + ent);
  }
  __device__ __forceinline__ void operator()(int64_t s, const float out[kActions], float dl[kActions], float st[5]) const {
    compute(load(s), prepare(), out, dl, st);
  }
};

struct CriticLoss {
  static constexpr unsigned kStats = 0b00010;
  LossCommon lc;
  const float* ret;
  const float* v_old;
  int per_row;  // samples of the trajectory that share this prediction: A (central critic) or 1
  struct In {
    float ret[kMaxAgents], v_old[kMaxAgents];
  };
  template <bool FAST = false>
  __device__ __forceinline__ int32_t row_entry(int64_t s) const { return lc.rows[per_row == 1 ? lc.ad.div<FAST>(s, lc.A) : s]; }
  __device__ __forceinline__ In load(int64_t s) const { return load_with(s, row_entry(s)); }
  __device__ __forceinline__ LossPrep prepare() const { return LossPrep{0.f, 1.f}; }
  template <bool FAST = false>
  __device__ __forceinline__ In load_with(int64_t s, int32_t entry) const {
    In in;
    if (per_row == 1) {
      const int a = (int)(s - lc.ad.div<FAST>(s, lc.A) * lc.A);
      const int64_t src = (int64_t)entry * lc.A + a;
      in.ret[0] = ret[src];
      in.v_old[0] = v_old[src];
    } else {
      const int64_t src0 = (int64_t)entry * lc.A;
#pragma unroll
      for (int a = 0; a < kMaxAgents; ++a)
        if (a < lc.A) {
          in.ret[a] = ret[src0 + a];
          in.v_old[a] = v_old[src0 + a];
        }
    }
    return in;
  }
  __device__ __forceinline__ float term(float v, float r, float vo, float* loss) const {
    const float e = v - r;
    float l = 0.5f * e * e, g = e;
    if (lc.clip_value) {
      const float dvv = v - vo;
      const float vc = vo + fminf(fmaxf(dvv, -lc.clip_eps), lc.clip_eps);
      const float ec = vc - r, lcl = 0.5f * ec * ec;
      if (lcl > l) {
        l = lcl;
        g = (dvv > -lc.clip_eps && dvv < lc.clip_eps) ? ec : 0.0f;
      }
    }
    *loss += l * lc.inv_B;
    return g;
  }
  __device__ __forceinline__ void compute(const In& in, const LossPrep&, const float out[1], float dl[1], float st[5]) const {
    float g = 0.f;
#pragma unroll
    for (int a = 0; a < kMaxAgents; ++a)
      if (a < per_row) g += term(out[0], in.ret[a], in.v_old[a], &st[1]);
    dl[0] = g * lc.vf_coef * lc.inv_B;
  }
  __device__ __forceinline__ void operator()(int64_t s, const float out[1], float dl[1], float st[5]) const {
    compute(load(s), prepare(), out, dl, st);
  }
};

// Output layer + loss + gradient of the output layer, up to 512 hidden units (a multiple of 32).  Persistent over tiles of
// 32 samples whose activations sit in LDS at their whole width; a workgroup's share of the W3 / b3 gradient leaves it once,
// with plain stores, and is added in a fixed order by the launcher.  (With atomics the 2048 workgroups queued up on the same
// few cache lines: 460 us of the 480 us a launch on 98 304 samples took; 131 us for 1 048 576 now, 537 MB of activations.)
// DZ2: H2 is replaced by dz2 = (dL/dout W3^T)(1 - h2^2), the gradient of its pre-activations, which the tile in LDS gives
// without another pass over the activations (a kernel of its own took 76 us for 50 000 samples of 192 units).  Otherwise dL/dout
// goes to dl_out [S][NOUT] and H2 stays.
// Bound: memory and, per tile, a chain of three barriers, which the other workgroup of the compute unit and the next
// tile's loads, already in flight, cover.
constexpr int kLossHeadGrid = 512;
constexpr int kLossTile = 32;
inline int64_t loss_head_partial_floats(int H, int nout) { return kLossHeadGrid * copy_pitch(H * nout + nout); }
inline size_t loss_head_lds(int H, int nout) { return sizeof(float) * (kLossTile * (H + 4) + H * nout + 8 * nout * kLossTile + kLossTile * 8); }

// NQ: 16-byte pieces of a row per staging thread, at least H / 32 (the last piece again beyond that)
template <int NOUT, int NQ, bool DZ2, class LossFn>
__global__ void __launch_bounds__(256, 2) loss_head_kernel(float* H2, int64_t S, int H,
                                                           const float* __restrict__ W3, const float* __restrict__ b3,
                                                           LossFn fn, float* __restrict__ dl_out, float* __restrict__ partial,
                                                           Scalars* sc) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int P = H + 4;
  float* const tile = lds;                              // [32][P]
  float* const w3 = tile + kLossTile * P;               // [H][NOUT]
  float* const red = w3 + H * NOUT;                     // [8][NOUT][32]
  float* const dls = red + 8 * NOUT * kLossTile;        // [32][8]
  const int tid = threadIdx.x;
  const int row = tid >> 3, c0 = 4 * (tid & 7), nq = H / 32;  // staging: row, every eighth 16-byte piece of it
  const int smp = tid & 31, grp = tid >> 5;                   // output layer: sample, share of the units
  const int units = H <= 128 ? 128 : 256, parts = 256 / units, part = tid / units;  // W3 gradient: unit tid % units (+ units), share of the samples
  float gw[2][NOUT], gb[NOUT], st[5] = {0.f, 0.f, 0.f, 0.f, 0.f}, bias[NOUT];
#pragma unroll
  for (int k = 0; k < NOUT; ++k) {
    gw[0][k] = gw[1][k] = gb[k] = 0.f;
    bias[k] = b3[k];
  }
  const LossPrep prep = fn.prepare();
  for (int i = tid; i < H * NOUT; i += 256) w3[i] = W3[i];
  float wu[2][NOUT];  // DZ2: the output weights of this thread's units
  if (DZ2) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int k = 0; k < NOUT; ++k) wu[c][k] = W3[min(tid % units + c * units, H - 1) * NOUT + k];
  }
  const int64_t ntiles = (S + kLossTile - 1) / kLossTile;
  typedef float f4 __attribute__((ext_vector_type(4)));
  f4 v[NQ];
  typename LossFn::In in;
  auto fetch = [&](int64_t t) {
    const float* const src = H2 + min(t * kLossTile + row, S - 1) * H + c0;  // rows past the end: the last row, with a zero gradient
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = *reinterpret_cast<const f4*>(src + 32 * min(q, nq - 1));
    if (tid < kLossTile) in = fn.load(min(t * kLossTile + tid, S - 1));
  };
  if (blockIdx.x < ntiles) fetch(blockIdx.x);
  for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int64_t s0 = t * kLossTile;
#pragma unroll
    for (int q = 0; q < NQ; ++q) *reinterpret_cast<f4*>(&tile[row * P + c0 + 32 * min(q, nq - 1)]) = v[q];
    const typename LossFn::In cur = in;
    __syncthreads();
    if (t + gridDim.x < ntiles) fetch(t + gridDim.x);
    {
      float acc[NOUT];
#pragma unroll
      for (int k = 0; k < NOUT; ++k) acc[k] = 0.f;
      const int per = H / 8;  // a multiple of 4
#pragma unroll 2
      for (int i = grp * per; i < (grp + 1) * per; i += 4) {
        const float4 hv = *reinterpret_cast<const float4*>(&tile[smp * P + i]);
        const float hh[4] = {hv.x, hv.y, hv.z, hv.w};
        float wv[4 * NOUT];
#pragma unroll
        for (int q = 0; q < NOUT; ++q) {
          const float4 w = *reinterpret_cast<const float4*>(&w3[i * NOUT + 4 * q]);
          wv[4 * q] = w.x; wv[4 * q + 1] = w.y; wv[4 * q + 2] = w.z; wv[4 * q + 3] = w.w;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int k = 0; k < NOUT; ++k) acc[k] = fmaf(hh[j], wv[j * NOUT + k], acc[k]);
      }
#pragma unroll
      for (int k = 0; k < NOUT; ++k) red[(grp * NOUT + k) * kLossTile + smp] = acc[k];
    }
    __syncthreads();
    if (tid < kLossTile) {
      float out[NOUT], dl[NOUT];
#pragma unroll
      for (int k = 0; k < NOUT; ++k) {
        out[k] = bias[k];
        dl[k] = 0.f;
#pragma unroll
        for (int g = 0; g < 8; ++g) out[k] += red[(g * NOUT + k) * kLossTile + tid];
      }
      if (s0 + tid < S) {
        fn.compute(cur, prep, out, dl, st);
        if (!DZ2) {
#pragma unroll
          for (int k = 0; k < NOUT; ++k) dl_out[(s0 + tid) * NOUT + k] = dl[k];
        }
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) dls[tid * 8 + k] = k < NOUT ? dl[k < NOUT ? k : 0] : 0.f;
#pragma unroll
      for (int k = 0; k < NOUT; ++k) gb[k] += dl[k];
    }
    __syncthreads();
    // gW3[i][k] += sum_s H2[s][i] * dl[s][k]
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int i = tid % units + c * units;
      if (i < H) {
        const int n = kLossTile / parts, live = (int)min((int64_t)kLossTile, S - s0);
        float* const dst = H2 + s0 * H + i;
#pragma unroll 4
        for (int s = part * n; s < (part + 1) * n; ++s) {
          const float h = tile[s * P + i];
          float d = 0.f;
#pragma unroll
          for (int k = 0; k < NOUT; ++k) {
            const float dl = dls[s * 8 + k];
            gw[c][k] = fmaf(h, dl, gw[c][k]);
            if (DZ2) d = fmaf(dl, wu[c][k], d);
          }
          if (DZ2 && s < live) dst[s * H] = d * (1.0f - h * h);
        }
      }
    }
    __syncthreads();  // the tile has been read
  }
  float* const own = partial + blockIdx.x * copy_pitch(H * NOUT + NOUT);
  if (parts == 2) {  // H <= 128: the two halves of the samples
    if (part == 1) {
#pragma unroll
      for (int k = 0; k < NOUT; ++k) tile[(tid - units) * NOUT + k] = gw[0][k];
    }
    __syncthreads();
    if (part == 0) {
#pragma unroll
      for (int k = 0; k < NOUT; ++k) gw[0][k] += tile[tid * NOUT + k];
    }
  }
  if (part == 0) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
      if (tid + c * units < H) {
#pragma unroll
        for (int k = 0; k < NOUT; ++k) own[(tid + c * units) * NOUT + k] = gw[c][k];
      }
  }
  if (tid < 64) {  // one wavefront: reduce across its lanes (32 of them hold zeros)
#pragma unroll
    for (int k = 0; k < NOUT; ++k) {
      float g = gb[k];
      for (int o = 32; o > 0; o >>= 1) g += __shfl_xor(g, o);
      if (tid == 0) own[H * NOUT + k] = g;
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      float g = st[k];
      for (int o = 32; o > 0; o >>= 1) g += __shfl_xor(g, o);
      if (tid == 0 && g != 0.f) atomicAdd(&sc->acc[k], g);
    }
  }
}

// gW3: [H][NOUT], the gradient of b3 directly behind it; partial: loss_head_partial_floats
template <int NOUT, bool DZ2, class LossFn>
inline int32_t launch_loss_head(float* H2, int64_t S, int H, const float* W3, const float* b3, const LossFn& fn, float* dl,
                                float* gW3, float* partial, Scalars* sc, hipStream_t s) {
  auto kern = H <= 128 ? loss_head_kernel<NOUT, 4, DZ2, LossFn> : H <= 256 ? loss_head_kernel<NOUT, 8, DZ2, LossFn> : loss_head_kernel<NOUT, 16, DZ2, LossFn>;
  const size_t bytes = loss_head_lds(H, NOUT);
  if (bytes > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
    return MARL_E_LAUNCH;
  const unsigned nb = (unsigned)std::min<int64_t>(kLossHeadGrid, (S + kLossTile - 1) / kLossTile);
  hipLaunchKernelGGL(kern, dim3(nb), dim3(256), bytes, s, H2, S, H, W3, b3, fn, dl, partial, sc);
  launch_reduce_partials(partial, (int)nb, (int64_t)H * NOUT + NOUT, gW3, s);
  return MARL_OK;
}

// Squared gradient norm in two fixed-order stages (no atomics, so the clipping factor is the same bits in every run):
// workgroup b of at most kNormBlocks sums its grid-stride share in fp64 and stores it; adam_kernel (256 threads per
// workgroup = kNormBlocks) adds the shares.
__global__ void __launch_bounds__(256) grad_norm_kernel(const float* __restrict__ grad, int64_t P, Scalars* sc) {
  __shared__ double red[4];
  double part = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < P; i += (int64_t)gridDim.x * blockDim.x) {
    const double g = grad[i];
    part += g * g;
  }
  const double t = block_sum_f64(part, red);
  if (threadIdx.x == 0) sc->norm_part[blockIdx.x] = t;
}
inline unsigned grad_norm_blocks(int64_t P) { return (unsigned)std::min<int64_t>(kNormBlocks, (P + 255) / 256); }

struct AdamArgs {
  float lr, b1, b2, eps, bc1, bc2, max_norm, ent_coef, vf_coef;
  int norm_blocks;        // workgroups grad_norm_kernel ran with
  const int64_t* k_base;  // nullable: device-resident count of optimiser steps taken before this call; then the bias
  int k_local;            // corrections are computed on the device for step *k_base + k_local instead of bc1 / bc2
};

// What becomes of a new parameter besides its place in the parameter vector: nothing, or its places in the working copy that the next
// optimiser step of the same update reads (a launch less per step; the copy's padding rows stay as the first step's staging left them).
struct NoStage {
  __device__ __forceinline__ void operator()(int64_t, float) const {}
};
struct StageNext {
  float* dst;  // nullable: the update's last step
  ParamMap pm;
  int round;
  __device__ __forceinline__ void operator()(int64_t i, float v) const {
    if (dst != nullptr) stage_param(dst, pm, i, v, round != 0, false, true);
  }
};

// sc_next (nullable): the gradient and that set of scalars are zeroed for the next optimiser step, which accumulates
// into them (two sets of scalars alternate, so nobody reads the one being zeroed).
template <class Stage>
__global__ void __launch_bounds__(256) adam_kernel(float* __restrict__ params, float* __restrict__ m,
                                                   float* __restrict__ v, float* __restrict__ grad, int64_t P,
                                                   AdamArgs a, const Scalars* sc, float* __restrict__ stats_row,
                                                   float* __restrict__ grad_dump, Scalars* sc_next, Stage stage) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  // the workgroups' shares of |grad|^2, added by a fixed tree (the same in every workgroup and every run)
  __shared__ double nparts[kNormBlocks];
  nparts[threadIdx.x] = (int)threadIdx.x < a.norm_blocks ? sc->norm_part[threadIdx.x] : 0.0;
  __syncthreads();
  for (int o = kNormBlocks / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) nparts[threadIdx.x] += nparts[threadIdx.x + o];
    __syncthreads();
  }
  const float norm = sqrtf((float)nparts[0]);
  const float scale = a.max_norm > 0.f ? a.max_norm / fmaxf(norm, a.max_norm) : 1.0f;
  if (a.k_base != nullptr) {
    const double k = (double)(*a.k_base + a.k_local);
    a.bc1 = (float)(1.0 - pow((double)a.b1, k));
    a.bc2 = (float)(1.0 - pow((double)a.b2, k));
  }
  if (i < P) {
    const float g = grad[i] * scale;
    const float mi = a.b1 * m[i] + (1.0f - a.b1) * g;
    const float vi = a.b2 * v[i] + (1.0f - a.b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    const float p = params[i] - a.lr * (mi / a.bc1) / (sqrtf(vi / a.bc2) + a.eps);
    params[i] = p;
    stage(i, p);
    if (grad_dump) grad_dump[i] = g;
    if (sc_next != nullptr) grad[i] = 0.f;
  }
  if (i == 0 && sc_next != nullptr) {
    sc_next->adv_sum = 0.0;
    sc_next->adv_sq = 0.0;
    for (int k = 0; k < 8; ++k) sc_next->acc[k] = 0.f;
  }
  if (i == 0) {
    const float total = sc->acc[0] - a.ent_coef * sc->acc[2] + a.vf_coef * sc->acc[1];
    stats_row[0] = sc->acc[0];
    stats_row[1] = sc->acc[1];
    stats_row[2] = sc->acc[2];
    stats_row[3] = sc->acc[3];
    stats_row[4] = sc->acc[4];
    stats_row[5] = norm;
    stats_row[6] = total;
    stats_row[7] = (isfinite(total) && isfinite(norm)) ? 0.f : 1.f;
  }
}

}  // namespace
}  // namespace marl
