// Forward pass of small calls: both hidden layers, the output layer and whatever consumes the outputs of both networks in one
// launch, on the caller's unstaged parameters and the fp32 instruction, with the first hidden activation kept in LDS.
//
// Workgroup = 4 wavefronts on a tile of BM samples x H hidden units: (BM/32) x (H/32) MFMA tiles of 32x32, one or two per
// wavefront.  The row tile of the input sits in LDS at its whole width; a tile's wavefronts read the weights once.
#pragma once
#include "gemm.h"
#include "heads.h"

namespace marl {

struct FusedFwdArgs {
  RowSrc X;   // S rows of Din floats (optionally gathered)
  int64_t S;
  int Din;
  int xvec;   // 1: rows are 16-byte aligned and Din % 4 == 0: 16-byte loads of X.  2: rows start at any 4-byte boundary of a
              // buffer whose two ends are 16-byte aligned: a row is fetched as the aligned 16-byte chunks that cover it
  const float *W1, *b1, *W2, *b2, *W3, *b3;  // W[in][H], at any 4-byte boundary
  int kpad1;               // Din rounded up to a multiple of 16
  int px;                  // pitch of the X tile in LDS: a multiple of 4 with px / 4 odd, >= kpad1
};

// The kernel's body: workgroup `bid` of `nblk` that share the tiles.
template <int H, int BM, int NOUT, class Finish>
__device__ __forceinline__ void fused_forward_body(const FusedFwdArgs& a, const Finish& fin, const unsigned bid, const unsigned nblk) {
  constexpr int PH = H + 4, GROUPS = 256 / BM;
  constexpr int NTN = H / 32, MT = BM / 32, TILES = MT * NTN, TPW = TILES / 4;
  static_assert(TILES % 4 == 0 && (TPW == 1 || TPW == 2), "4 wavefronts share the tile evenly");
  static_assert(TPW == 1 || NTN % 2 == 0, "two tiles of a wavefront share their rows");
  constexpr int NTH = 256;
  constexpr int TPR = NTH / BM;  // threads staging one row of X
  extern __shared__ __attribute__((aligned(16))) float lds[];
  struct {
    float *Xs, *Hs, *red, *W3s;
  } L;
  const int px = a.px;
  L.Xs = lds;                          // [BM][px]   input rows, k-contiguous; columns Din .. px stay zero
  L.Hs = L.Xs + BM * px;               // [BM][PH]   h1, then h2
  L.red = L.Hs + BM * PH;              // [GROUPS][BM][NOUT]
  L.W3s = L.red + GROUPS * BM * NOUT;  // [H][NOUT]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lo = lane & 31, hi = lane >> 5;
  const int mt = (wave * TPW) / NTN, nt0 = (wave * TPW) % NTN;  // this wavefront's tiles: (mt, nt0 .. nt0+TPW-1)

  for (int i = tid; i < H * NOUT; i += NTH) L.W3s[i] = a.W3[i];  // ordered before its first use by the barriers of layer 1
  for (int i = tid; i < BM * px; i += NTH) L.Xs[i] = 0.f;        // the padding columns stay zero for good
  __syncthreads();
  const int64_t ntiles = (a.S + BM - 1) / BM;
  for (int64_t tile = bid; tile < ntiles; tile += nblk) {
    const int64_t s0 = tile * BM;
    // ---- this tile's rows to LDS: thread -> row tid / TPR, every TPR-th 16-byte (or 4-byte) piece of it, four
    // (twelve) loads in flight at a time.  Rows past the end re-read the last row (their results are never stored).
    {
      const int xr_row = tid / TPR, c0 = tid % TPR;
      const float* xrow = a.X.ptr(min(s0 + xr_row, a.S - 1));
      float* xdst = L.Xs + xr_row * px;
      if (a.xvec == 2) {
        // element j of chunk q is column 4 q + j - xo of the row; the chunks never leave the buffer (its ends are aligned)
        // (pointer arithmetic, not an integer round trip, so that the loads stay global loads)
        const int xo = (int)((reinterpret_cast<uintptr_t>(xrow) >> 2) & 3), last = ((xo + a.Din + 3) >> 2) - 1;
        const float4* const chunk = reinterpret_cast<const float4*>(xrow - xo);
        constexpr int XC = 3;  // chunks in flight per thread: a 75-wide row is one batch
        for (int q = c0; q <= last; q += XC * TPR) {
          float4 v[XC];
#pragma unroll
          for (int u = 0; u < XC; ++u) v[u] = chunk[min(q + u * TPR, last)];
#pragma unroll
          for (int u = 0; u < XC; ++u) {
            const float e[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const int c = 4 * (q + u * TPR) + j - xo;
              if (c >= 0 && c < a.Din && q + u * TPR <= last) xdst[c] = e[j];
            }
          }
        }
      } else if (a.xvec) {
        const int nv = a.Din / 4;
        for (int c = c0; c < nv; c += 4 * TPR) {
          float4 v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int cu = min(c + u * TPR, nv - 1);
            v[u] = *reinterpret_cast<const float4*>(xrow + 4 * cu);
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (c + u * TPR < nv) *reinterpret_cast<float4*>(xdst + 4 * (c + u * TPR)) = v[u];
        }
      } else {
        constexpr int XB = 12;  // loads in flight per thread: a 75- or 27-wide row is one batch
        for (int c = c0; c < a.Din; c += XB * TPR) {
          float v[XB];
#pragma unroll
          for (int u = 0; u < XB; ++u) v[u] = xrow[min(c + u * TPR, a.Din - 1)];
#pragma unroll
          for (int u = 0; u < XB; ++u)
            if (c + u * TPR < a.Din) xdst[c + u * TPR] = v[u];
        }
      }
    }
    __syncthreads();
    floatx16 acc[TPW];
    auto zero_acc = [&]() {
#pragma unroll
      for (int q = 0; q < TPW; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[q][r] = 0.f;
    };
    // ---- layer 1: h1 = tanh(X W1 + b1) -> LDS
    zero_acc();
#pragma unroll
    for (int q = 0; q < TPW; ++q)
      gemm_phase_direct<H>(L.Xs + (mt * 32 + lo) * px + 4 * hi, a.W1 + (nt0 + q) * 32 + lo, a.Din, hi, a.kpad1 / 16, acc[q]);
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
      const int n = (nt0 + q) * 32 + lo;
      const float bias = a.b1[n];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = mt * 32 + 8 * (r / 4) + 4 * hi + (r % 4);
        float v = tanh_f32(acc[q][r] + bias);
        L.Hs[m * PH + n] = v;
        if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);  // four elements in flight at a time keeps registers bounded
      }
    }
    __syncthreads();  // the h1 tile is complete
    // ---- layer 2: h2 = tanh(h1 W2 + b2), kept in registers
    zero_acc();
#pragma unroll
    for (int q = 0; q < TPW; ++q)
      gemm_phase_direct<H>(L.Hs + (mt * 32 + lo) * PH + 4 * hi, a.W2 + (nt0 + q) * 32 + lo, H, hi, H / 16, acc[q]);
    __syncthreads();  // every wavefront is past its last read of h1
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
      const int n = (nt0 + q) * 32 + lo;
      const float bias = a.b2[n];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = mt * 32 + 8 * (r / 4) + 4 * hi + (r % 4);
        float v = tanh_f32(acc[q][r] + bias);
        L.Hs[m * PH + n] = v;
        if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
    // ---- output layer on the ALUs: thread -> (sample tid % BM, slice tid / BM of the hidden units)
    {
      const int s = tid % BM, grp = tid / BM;
      constexpr int PER = H / GROUPS;
      float part[NOUT];
#pragma unroll
      for (int k = 0; k < NOUT; ++k) part[k] = 0.f;
      static_assert(PER % 4 == 0, "hidden units are read four at a time");
#pragma unroll 2
      for (int i = grp * PER; i < (grp + 1) * PER; i += 4) {
        const float4 hv = *reinterpret_cast<const float4*>(&L.Hs[s * PH + i]);
        const float hh[4] = {hv.x, hv.y, hv.z, hv.w};
        float wv[4 * NOUT];  // W3 rows i..i+3: 4 * NOUT consecutive floats, the same for every lane of the wavefront
#pragma unroll
        for (int q = 0; q < NOUT; ++q) {
          const float4 t = *reinterpret_cast<const float4*>(&L.W3s[i * NOUT + 4 * q]);
          wv[4 * q] = t.x; wv[4 * q + 1] = t.y; wv[4 * q + 2] = t.z; wv[4 * q + 3] = t.w;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int k = 0; k < NOUT; ++k) part[k] = fmaf(hh[j], wv[j * NOUT + k], part[k]);
      }
#pragma unroll
      for (int k = 0; k < NOUT; ++k) L.red[(grp * BM + s) * NOUT + k] = part[k];
    }
    __syncthreads();
    if (tid < BM) {
      float out[NOUT];
#pragma unroll
      for (int k = 0; k < NOUT; ++k) {
        float v = a.b3[k];
#pragma unroll
        for (int gq = 0; gq < GROUPS; ++gq) v += L.red[(gq * BM + tid) * NOUT + k];
        out[k] = v;
      }
      if (s0 + tid < a.S) fin(s0 + tid, out, nullptr, nullptr);
    }
    __syncthreads();  // the tile buffers are reused by the next row tile
  }
}

// Both networks of a small call in one launch, with unstaged weights: workgroups 0 .. grid_a - 1 the first.
template <int HA, int HB, int NOUT_A, int NOUT_B, class FinishA, class FinishB>
__global__ void __launch_bounds__(256, 2) fused_forward_small_kernel(FusedFwdArgs a, FinishA fa, FusedFwdArgs b, FinishB fb, unsigned grid_a) {
  if (blockIdx.x < grid_a) fused_forward_body<HA, HA == 64 ? 64 : 32, NOUT_A, FinishA>(a, fa, blockIdx.x, grid_a);
  else fused_forward_body<HB, HB == 64 ? 64 : 32, NOUT_B, FinishB>(b, fb, blockIdx.x - grid_a, gridDim.x - grid_a);
}

// Few enough rows that a call is a chain of latencies: one launch on the unstaged parameters (a tile's wavefronts read
// them once, 4 bytes at a time) against a staging kernel and a launch per network on split operands.  Measured, us, one
// launch / staged:
//   75 inputs, 128 / 128 units:   3 000 samples 12 / 24   12 288 samples 23 / 27   49 152 samples 80 / 53
//   147 inputs, 256 / 256 units:  3 000 samples 39 / 44    5 000 samples 50 / 46   20 480 samples 147 / 83
//   147 and 882 inputs, 256 / 128 units:  3 600 samples 41 / 65   24 576 samples 159 / 90
// The line lies below the smallest size at which any of them crosses (about 4 000).  The one launch runs on the fp32
// instruction, so that an output's last bits differ on the two sides.
constexpr int64_t kForwardSmall = 2048;

template <int HA, int HB, int NOUT_A, int NOUT_B, class FinishA, class FinishB>
inline int32_t launch_fused_forward_small_inst(const FusedFwdArgs& a, const FinishA& fa, const FusedFwdArgs& b, const FinishB& fb, hipStream_t s) {
  auto kern = fused_forward_small_kernel<HA, HB, NOUT_A, NOUT_B, FinishA, FinishB>;
  const size_t bytes = std::max(fused_forward_lds_bytes(HA, a.Din, NOUT_A), fused_forward_lds_bytes(HB, b.Din, NOUT_B));
  if (bytes > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
    return MARL_E_LAUNCH;
  const unsigned grid_a = (unsigned)((a.S + (HA == 64 ? 64 : 32) - 1) / (HA == 64 ? 64 : 32));
  const unsigned grid_b = (unsigned)((b.S + (HB == 64 ? 64 : 32) - 1) / (HB == 64 ? 64 : 32));
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
