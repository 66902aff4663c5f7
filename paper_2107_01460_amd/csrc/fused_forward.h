// Forward pass of small calls: both hidden layers, the output layer and whatever consumes the outputs of both networks in one
// launch, on the caller's unstaged parameters and the fp32 instruction, with the first hidden activation kept in LDS.
//
// Such a call is a chain of latencies on a few compute units.  Workgroup = 16 samples, four wavefronts: each takes 64 columns with all samples, and
// where the layer is narrower a part of the contraction (the parts meet in LDS, where bias and tanh are shared by all threads).  The weights
// come straight from the parameters, 16 bytes a lane at any 4-byte boundary -- four columns of one row, which are the same lane's operands of four
// v_mfma_f32_16x16x4_f32 -- and the first groups of both layers, the biases and the inputs are all requested before anything is waited for.  One
// environment of three agents, 75 inputs, 128 / 128 units: 6.7 us; with 32 samples a workgroup, 4-byte loads of the weights three
// groups ahead and biases loaded where they are added 11.0 us.  2040 samples of 147 inputs, 256 / 256 units, with the sampling behind it: 39.6 -> 19.8 us.
#pragma once
#include "gemm.h"
#include "heads.h"

namespace marl {

struct FusedFwdArgs {
  RowSrc X;   // S rows of Din floats
  int64_t S;
  int Din;
  const float *W1, *b1, *W2, *b2, *W3, *b3;  // W[in][H], at any 4-byte boundary
  int kpad1;               // Din rounded up to a multiple of 16
  int px;                  // pitch of the X tile in LDS: a multiple of 4 with px / 4 odd, >= kpad1
};
constexpr int kSmallRows = 16;  // samples of a workgroup
inline size_t fused_forward_small_lds(int H, int px, int nout) {
  return sizeof(float) * (kSmallRows * (size_t)px + kSmallRows * (H + 4) + (256 / H) * kSmallRows * (size_t)(H + 4) + (size_t)H * nout);
}

// The kernel's body: tile `bid` of 16 samples.
template <int H, int NOUT, class Finish>
__device__ __forceinline__ void fused_forward_body(const FusedFwdArgs& a, const Finish& fin, const unsigned bid) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  constexpr int BM = kSmallRows, PH = H + 4, CB = H / 64, KW = 4 / CB, VPT = H / 16;
  static_assert(H == 64 || H == 128 || H == 256, "the wavefronts share columns and contraction evenly");
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int px = a.px;
  float* const Xs = lds;                 // [BM][px]      input rows; columns Din .. px are zero
  float* const Hs = Xs + BM * px;        // [BM][PH]      h1
  float* const Ps = Hs + BM * PH;        // [KW][BM][PH]  parts of a layer
  float* const W3s = Ps + KW * BM * PH;  // [H][NOUT]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = lane & 15, q = lane >> 4;
  const int cb = wave % CB, kw = wave / CB;         // this wavefront's columns and its part of the contraction: groups kw, kw + KW, ... of 16
  const int row = tid / 16, c0 = (tid % 16) * VPT;  // this thread's sample and units between the layers
  const int64_t s0 = (int64_t)bid * BM;
  // ---- requests: inputs, first weights, biases
  constexpr int XB = 6, R1 = 3, R2 = H / 16 / KW < 4 ? H / 16 / KW : 4;
  const float* const xrow = a.X.base + min(s0 + row, a.S - 1) * a.X.ld;  // rows past the end are the last one again: their results are never stored
  float x[XB];
#pragma unroll
  for (int u = 0; u < XB; ++u) x[u] = xrow[min(tid % 16 + 16 * u, a.Din - 1)];
  const int ng1 = a.kpad1 / 16;
  constexpr int NG2 = H / 16;
  const int col = 64 * cb + 4 * i;
  f4 w1[R1][4], w2[R2][4];
  auto load = [&](const float* W, int K, int g, f4 (&w)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = *reinterpret_cast<const f4u*>(W + (int64_t)min(16 * g + 4 * q + j, K - 1) * H + col);
  };
#pragma unroll
  for (int t = 0; t < R1; ++t) load(a.W1, a.Din, kw + KW * t, w1[t]);
  f4 bias1[VPT / 4], bias2[VPT / 4];
#pragma unroll
  for (int v = 0; v < VPT / 4; ++v) bias1[v] = *reinterpret_cast<const f4u*>(a.b1 + c0 + 4 * v);
  constexpr int W3T = (H * NOUT + 255) / 256;
  float w3[W3T];
#pragma unroll
  for (int u = 0; u < W3T; ++u) w3[u] = a.W3[min(tid + 256 * u, H * NOUT - 1)];
#pragma unroll
  for (int t = 0; t < R2; ++t) load(a.W2, H, kw + KW * t, w2[t]);
#pragma unroll
  for (int v = 0; v < VPT / 4; ++v) bias2[v] = *reinterpret_cast<const f4u*>(a.b2 + c0 + 4 * v);
  float b3[NOUT];
#pragma unroll
  for (int k = 0; k < NOUT; ++k) b3[k] = a.b3[k];
  // ---- inputs and W3 to LDS
#pragma unroll
  for (int u = 0; u < XB; ++u) {
    const int c = tid % 16 + 16 * u;
    if (c < px) Xs[row * px + c] = c < a.Din ? x[u] : 0.f;
  }
  for (int c1 = tid % 16 + 16 * XB; c1 < px; c1 += 16 * XB) {  // wide inputs
#pragma unroll
    for (int u = 0; u < XB; ++u) x[u] = xrow[min(c1 + 16 * u, a.Din - 1)];
#pragma unroll
    for (int u = 0; u < XB; ++u)
      if (c1 + 16 * u < px) Xs[row * px + c1 + 16 * u] = c1 + 16 * u < a.Din ? x[u] : 0.f;
  }
#pragma unroll
  for (int u = 0; u < W3T; ++u)
    if (tid + 256 * u < H * NOUT) W3s[tid + 256 * u] = w3[u];
  lds_barrier();
  floatx4 acc[4];  // register r of acc[e]: sample 4 q + r, column col + e
  auto clear = [&]() {
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = floatx4{0.f, 0.f, 0.f, 0.f};
  };
  auto group = [&](const float* A, const f4 (&w)[4]) {  // A: this lane's sample, + 4 q of the group
    const f4 v = *reinterpret_cast<const f4*>(A);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j], w[j][e], acc[e], 0, 0, 0);
  };
  auto put = [&]() {
#pragma unroll
    for (int r = 0; r < 4; ++r) *reinterpret_cast<f4*>(&Ps[(kw * BM + 4 * q + r) * PH + col]) = f4{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
    lds_barrier();
  };
  auto activation = [&](int v, const f4& bias) {  // units c0 + 4 v .. of this thread's sample
    f4 t = *reinterpret_cast<const f4*>(&Ps[row * PH + c0 + 4 * v]);
#pragma unroll
    for (int p = 1; p < KW; ++p) t += *reinterpret_cast<const f4*>(&Ps[(p * BM + row) * PH + c0 + 4 * v]);
    t += bias;
    return f4{tanh_f32(t[0]), tanh_f32(t[1]), tanh_f32(t[2]), tanh_f32(t[3])};
  };
  // ---- layer 1
  clear();
#pragma unroll 1
  for (int t0 = 0; kw + KW * t0 < ng1; t0 += R1) {
#pragma unroll
    for (int d = 0; d < R1; ++d) {
      const int g = kw + KW * (t0 + d);
      if (g < ng1) {  // uniform
        f4 w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) w[j][e] = 16 * g + 4 * q + j < a.Din ? w1[d][j][e] : 0.f;
        group(Xs + i * px + 16 * g + 4 * q, w);
        if (g + KW * R1 < ng1) load(a.W1, a.Din, g + KW * R1, w1[d]);
      }
    }
  }
  put();
#pragma unroll
  for (int v = 0; v < VPT / 4; ++v) *reinterpret_cast<f4*>(&Hs[row * PH + c0 + 4 * v]) = activation(v, bias1[v]);
  lds_barrier();
  // ---- layer 2
  clear();
#pragma unroll
  for (int t = 0; t < NG2 / KW; ++t) {
    const int g = kw + KW * t;
    group(Hs + i * PH + 16 * g + 4 * q, w2[t % R2]);
    if (t + R2 < NG2 / KW) load(a.W2, H, g + KW * R2, w2[t % R2]);
  }
  put();
  // ---- output layer: a thread's units, then the sixteen threads of a sample
  float out[NOUT];
#pragma unroll
  for (int k = 0; k < NOUT; ++k) out[k] = 0.f;
#pragma unroll
  for (int v = 0; v < VPT / 4; ++v) {
    const f4 h = activation(v, bias2[v]);
    float w[4 * NOUT];
#pragma unroll
    for (int u = 0; u < NOUT; ++u) {
      const f4 t = *reinterpret_cast<const f4*>(&W3s[(c0 + 4 * v) * NOUT + 4 * u]);
      w[4 * u] = t[0]; w[4 * u + 1] = t[1]; w[4 * u + 2] = t[2]; w[4 * u + 3] = t[3];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int k = 0; k < NOUT; ++k) out[k] = fmaf(h[e], w[e * NOUT + k], out[k]);
  }
#pragma unroll
  for (int o = 1; o < 16; o *= 2)
#pragma unroll
    for (int k = 0; k < NOUT; ++k) out[k] += __shfl_xor(out[k], o);
#pragma unroll
  for (int k = 0; k < NOUT; ++k) out[k] += b3[k];
  if (tid % 16 == 0 && s0 + row < a.S) fin(s0 + row, out, nullptr, nullptr);
}

// Both networks of a small call in one launch, with unstaged weights: workgroups 0 .. grid_a - 1 the first.
template <int HA, int HB, int NOUT_A, int NOUT_B, class FinishA, class FinishB>
__global__ void __launch_bounds__(256, 2) fused_forward_small_kernel(FusedFwdArgs a, FinishA fa, FusedFwdArgs b, FinishB fb, unsigned grid_a) {
  if (blockIdx.x < grid_a) fused_forward_body<HA, NOUT_A, FinishA>(a, fa, blockIdx.x);
  else fused_forward_body<HB, NOUT_B, FinishB>(b, fb, blockIdx.x - grid_a);
}

// Few enough rows that a call is a chain of latencies: one launch on the unstaged parameters against a staging kernel and a launch per network on split
// operands.  us, one launch / staged, 2048 samples, 4096, 8192, 16 384: 75 inputs, 64 / 64 units 5.1 / 17.6, 6.0 / 17.8, 8.2 / 17.7, 13.6 / 19.3; 128 / 128 units
// 7.0 / 19.6, 9.0 / 19.7, 15.9 / 20.2, 29.0 / 21.5; 147 inputs, 256 / 256 units 16.7 / 31.3, 23.7 / 31.3, 45.1 / 32.7, 85.4 / 56.7.  So the two cross at 6000 samples
// (256 units), 11 000 (128) and beyond 16 384 (64), and calls between the line and there take the slower route: the line is an earlier kernel's,
// which crossed at 4000.  The one launch runs on the fp32 instruction, so that wherever the line lies an output's last bits differ on its two sides.
constexpr int64_t kForwardSmall = 2048;

template <int HA, int HB, int NOUT_A, int NOUT_B, class FinishA, class FinishB>
inline int32_t launch_fused_forward_small_inst(const FusedFwdArgs& a, const FinishA& fa, const FusedFwdArgs& b, const FinishB& fb, hipStream_t s) {
  auto kern = fused_forward_small_kernel<HA, HB, NOUT_A, NOUT_B, FinishA, FinishB>;
  const size_t bytes = std::max(fused_forward_small_lds(HA, a.px, NOUT_A), fused_forward_small_lds(HB, b.px, NOUT_B));
  if (bytes > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
    return MARL_E_LAUNCH;
  const unsigned grid_a = (unsigned)((a.S + kSmallRows - 1) / kSmallRows), grid_b = (unsigned)((b.S + kSmallRows - 1) / kSmallRows);
  if (grid_a + grid_b == 0) return MARL_OK;
  hipLaunchKernelGGL(kern, dim3(grid_a + grid_b), dim3(256), bytes, s, a, fa, b, fb, grid_a);
  return launch_status();
}
// a network with S = 0 is left out
template <int NOUT_A, int NOUT_B, class FinishA, class FinishB>
inline int32_t launch_fused_forward_small(int HA, const FusedFwdArgs& a, const FinishA& fa, int HB, const FusedFwdArgs& b, const FinishB& fb, hipStream_t s) {
  TimedLaunch timed(KC_GEMM_NN, 2.0 * (double)a.S * ((double)a.Din * HA + (double)HA * HA) + 2.0 * (double)b.S * ((double)b.Din * HB + (double)HB * HB), s);
  switch (HA / 64 * 10 + HB / 64) {
    case 11: return launch_fused_forward_small_inst<64, 64, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    case 12: return launch_fused_forward_small_inst<64, 128, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    case 14: return launch_fused_forward_small_inst<64, 256, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    case 21: return launch_fused_forward_small_inst<128, 64, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    case 22: return launch_fused_forward_small_inst<128, 128, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    case 24: return launch_fused_forward_small_inst<128, 256, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    case 41: return launch_fused_forward_small_inst<256, 64, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    case 42: return launch_fused_forward_small_inst<256, 128, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    default: return launch_fused_forward_small_inst<256, 256, NOUT_A, NOUT_B>(a, fa, b, fb, s);
  }
}

}  // namespace marl
