// fp32 networks on split bf16 operands (split_bf16.h): a tile of rows through a whole network in one kernel, as bf16_net.h does it
// for the bf16 configuration.  The tile's activations sit in LDS as three planes of bf16 (their split is made once, by the
// epilogue that produces them); the split weights stream from the L2 in one sequence of k steps that runs on from layer to layer
// and from tile to tile.  In training the kernel also takes the loss, the output layer's gradient and the gradients of both
// hidden layers' pre-activations; h1 and h2 stay in registers for them, h1, dz2 and dz1 go to memory for the weight gradients.
//
// Measured on an MI355X against a kernel per layer (fp32 instruction, weights in registers, or 32-row tiles with the forward pass and the
// loss in one kernel).  Everything of a minibatch but the weight gradients: 262 144 samples, 300 inputs, 256 units, one output: 347 + 331 +
// 297 -> 725 us (150 TFLOP/s of fp32 products); 50 000 samples, 147 inputs: 256 units, six outputs 143 + 64 -> 138 us, 192 units, one
// output 42 + 38 + 30 + 38 -> 102 us.  Training iterations: 1000 environments, 256 / 192 units 15.8 -> 12.4 ms; 16 384 environments,
// central critic of 256 units 96.7 -> 92.2 ms.
// Bound (first of these sizes): no unit is full.  Matrix cores are busy 43 % and vector instructions 24 % of the cycles, and the weights
// come from the L2 at 15 TB/s (1.28 MB per tile of 32 rows; 86 million reads of 128 bytes), which two workgroups per CU (one above 256
// units) keep going through each other's phases; their 128 registers a lane leave a ring of two k steps of weights and up to 15 spilled
// registers (11, 1 and 15 at the sizes above; 51 at 32 units; loss statistics and constants in LDS, 1-2 % of a training iteration).  64-row tiles halve the bytes, but leave room for one workgroup per CU, whose phases
// without products (tanh, loss, gradients: 37 of 81 thousand cycles) nothing covers: the same time at the first size, 7 % longer updates
// at 50 000 samples.  Forward passes of many samples hold less and take the 64-row tiles.  h1 stored at the end of a tile instead of
// before layer 2's product, so that no weight waits behind it: 720 -> 759 us.
#pragma once
#include <type_traits>
#include <utility>

#include "gemm.h"
#include "heads.h"

namespace marl {

struct SplitNetArgs {
  RowSrc X;  // S rows of Din floats; a gather's divisor has its magic number
  int64_t S;
  int Din, Kp;     // Kp: rows of the staged W1, a multiple of 32
  const float* W;  // split copies of W1, W2 (, W2 transposed: training), one directly behind the other (ParamMap)
  const float *b1, *b2, *W3, *b3;
  float *h1, *dz2, *dz1;  // training: [S][H]
  float* partial;         // training: per workgroup the W3 gradient, the b3 gradient and five loss statistics
};

// Wavefronts: H / 32 side by side, WM below one another, each MT row tiles of 32.
template <int H, int BM>
struct SplitNetShape {
  static_assert(H % 32 == 0 && H <= kSplitNetMaxH && (BM == 32 || BM == 64), "split_net_supported");
  static constexpr int WN = H / 32, WM = BM == 64 && H <= 128 ? 2 : 1, MT = BM / (32 * WM), NW = WN * WM;
  static constexpr int P = (H < 64 ? 64 : H) + 8;  // pitch of a plane: an odd number of 16-byte units
  static constexpr int PD = BM + 8;
  // wavefronts per SIMD that the registers leave room for: in training two workgroups per CU (of six wavefronts each they need four:
  // the wavefronts of a workgroup are dealt 2, 2, 1, 1)
  static constexpr int waves(bool train) { return train ? (NW > 8 ? 3 : 4) : NW > 8 ? 3 : H <= 128 ? 4 : 2; }
  static constexpr size_t lds(bool train, int nout) {
    return sizeof(bf16_t) * 3 * (BM + 8) * P + sizeof(float) * (2 * H + 4) +
           (train ? sizeof(bf16_t) * 24 * PD + sizeof(float) * (12 + BM * 8 + H * (nout > 1 ? 8 : 1)) + sizeof(double) * BM / 16 * (nout + 5) : 0);
  }
};
// Training workgroups of narrow networks that share a CU's LDS (loss statistics of 32 sample slots instead of two groups took one of
// them: 50 000 samples of 147 inputs, 128 units, 20 minibatches 4.81 -> 4.97 ms)
static_assert(4 * SplitNetShape<128, 32>::lds(true, 6) <= 160 * 1024 && 5 * SplitNetShape<96, 32>::lds(true, 6) <= 160 * 1024 &&
                  7 * SplitNetShape<64, 32>::lds(true, 6) <= 160 * 1024, "workgroups per CU");

template <bool TRAIN, class Fin>
struct SplitNetLossIn { typedef int type, Prep; };
template <class Fin>
struct SplitNetLossIn<true, Fin> {
  typedef typename Fin::In type;
  typedef decltype(std::declval<Fin>().prepare()) Prep;  // two floats
};

// Fin: TRAIN: a loss functor (ActorLoss, CriticLoss); else what becomes of a sample's outputs, fin(s, out, nullptr, nullptr).
template <int H, int BM, int NOUT, bool TRAIN, class Fin>
__global__ void __launch_bounds__((64 * SplitNetShape<H, BM>::NW), (SplitNetShape<H, BM>::waves(TRAIN))) split_net_kernel(SplitNetArgs a, Fin fin) {
  using Sh = SplitNetShape<H, BM>;
  constexpr int MT = Sh::MT, WN = Sh::WN, WM = Sh::WM, NW = Sh::NW, P = Sh::P, PD = Sh::PD, THREADS = 64 * NW, PLANE = BM * P, PLANE3 = 8 * P;
  constexpr int RING = 2;                                  // k steps of weights on their way
  constexpr int XJ = H < 128 ? 1 : H < 192 ? 2 : 3;        // 64-column pieces of the input that are staged at a time
  constexpr int XR = (BM / 2 + NW - 1) / NW;               // pairs of input rows a wavefront stages
  constexpr int GPW = (BM / 16 + NW - 1) / NW;             // groups of 16 samples whose outputs a wavefront takes
  constexpr int W3P = NOUT > 1 ? 8 : 1, AS = NOUT + 5;
  // Forward passes above 128 units: the next tile's first piece of input waits in registers, and exact inputs take half of layer 1's
  // products (2.1 million samples, 300 inputs, 256 units: 3.61 -> 2.99 ms).  In training and in narrow networks other workgroups of the
  // CU cover the input's latency, and the registers are wanted for them (16.9 million samples, 27 inputs, 64 units: 2.23 ms with the
  // second form of layer 1, 2.06 without).
  constexpr bool AHEAD = !TRAIN && H > 128 && NW <= 8, EXACT_X = !TRAIN && H > 128;
  extern __shared__ __attribute__((aligned(16))) bf16_t split_net_lds[];
  bf16_t* const tile = split_net_lds;                            // [3][BM][P] X, h1, h2, dz2
  bf16_t* const w3t = tile + 3 * PLANE;                          // [3][8][P]  W3 transposed, split, rows past NOUT zero
  float* const bias = reinterpret_cast<float*>(w3t + 3 * PLANE3);  // [2][H]
  int* const inexact = reinterpret_cast<int*>(bias + 2 * H);     // [4] is a value of the tile's input not exact in bf16?
  float* const b3s = bias + 2 * H + 4;                           // TRAIN: [8]
  auto* const prep = reinterpret_cast<typename SplitNetLossIn<TRAIN, Fin>::Prep*>(b3s + 8);  // TRAIN
  double* const accD = reinterpret_cast<double*>(bias + 2 * H + 16);  // TRAIN: [BM / 16][AS] per group of sixteen samples: b3 gradient, loss statistics
  float* const dls = reinterpret_cast<float*>(accD + BM / 16 * AS);  // TRAIN: [BM][8] dL/d(output), zeros past NOUT
  float* const w3s = dls + BM * 8;                               // TRAIN: [H][W3P]
  bf16_t* const dlt = reinterpret_cast<bf16_t*>(w3s + H * W3P);  // TRAIN: [3][8][PD] dL/d(output), split and transposed

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int lane = tid & 63, lo = lane & 31, hi = lane >> 5, l15 = lane & 15, l4 = lane >> 4;
  const int wn = wave % WN, wm = wave / WN;
  const int64_t ntiles = (a.S + BM - 1) / BM;

  GroupCopy<H * NOUT, THREADS> w3;
  GroupCopy<H, THREADS> b1, b2;
  w3.request(tid, a.W3);
  b1.request(tid, a.b1);
  b2.request(tid, a.b2);
  // the output layer's bias: in LDS in training, whose registers are full, else in registers
  float bias3[TRAIN ? 1 : NOUT];
  [[maybe_unused]] float b3 = 0.f;
  if constexpr (TRAIN) {
    b3 = a.b3[min(tid, NOUT - 1)];
  } else {
#pragma unroll
    for (int k = 0; k < NOUT; ++k) bias3[k] = a.b3[k];
  }

  // ---- weights: k step `nxt` of the sequence layer 1, layer 2 (, dz1), and again for the next tile
  const int steps1 = a.Kp / 16, total = steps1 + (TRAIN ? 2 : 1) * (H / 16);
  const WeightRsrc wsrc = weight_rsrc(a.W, total * 16 * H * 3 / 2);
  const int woff = (hi * H + 32 * wn + lo) * 16;
  bf16x8 w[RING][3];
  int nxt = 0;
  auto load_w = [&](int slot) {
#pragma unroll
    for (int p = 0; p < 3; ++p) w[slot][p] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wsrc, woff, (nxt * 3 + p) * 32 * H, 0));
    nxt = nxt + 1 == total ? 0 : nxt + 1;
  };
#pragma unroll
  for (int u = 0; u < RING; ++u) load_w(u);

  if (tid == 0) *inexact = 0;
  if constexpr (TRAIN) {
    if (tid == 0) *prep = fin.prepare();
    if constexpr (W3P > NOUT) {
      constexpr int PAD = W3P - NOUT;
      for (int e = tid; e < H * PAD; e += THREADS) w3s[e / PAD * W3P + NOUT + e % PAD] = 0.f;
    }
    for (int e = tid; e < 24 * PD; e += THREADS) dlt[e] = 0;
    for (int e = tid; e < BM * 8; e += THREADS) dls[e] = 0.f;
    for (int e = tid; e < BM / 16 * AS; e += THREADS) accD[e] = 0.0;
  }
  for (int e = tid; e < (8 - NOUT) * H; e += THREADS) w3t[(NOUT + e / H) * P + e % H] = w3t[PLANE3 + (NOUT + e / H) * P + e % H] = w3t[2 * PLANE3 + (NOUT + e / H) * P + e % H] = 0;
  w3.store(tid, [&](int e, float v) {
    const int u = e / NOUT, k = e % NOUT;
    const SplitPair s = split_pair_any(v, 0.f);
    w3t[k * P + u] = (bf16_t)s.h;
    w3t[PLANE3 + k * P + u] = (bf16_t)s.m;
    w3t[2 * PLANE3 + k * P + u] = (bf16_t)s.l;
    if (TRAIN) w3s[u * W3P + k] = v;
  });
  b1.store(tid, [&](int e, float v) { bias[e] = v; });
  b2.store(tid, [&](int e, float v) { bias[H + e] = v; });
  if constexpr (TRAIN) {
    if (tid < NOUT) b3s[tid] = b3;
  }

  floatx16 acc[MT];
  auto zero_acc = [&]() {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  };
  // acc += weights x tile over `steps` (even) k steps; acc[i][r] belongs to unit 32 wn + 8 (r / 4) + 4 hi + r % 4 of sample
  // 32 (wm MT + i) + lo.  The products of the two operands' parts in mfma_split's order (the tile's part first).  The scheduling
  // barriers keep the requests where they are written (the compiler moves them to the end of the loop body).
  // EXACT: the tile's values are exact in bf16 (the windows of the library's own worlds hold small integers and halves), so the
  // products with their lower parts are zeros.
  auto product = [&](int steps, auto exact) {
    constexpr bool EXACT = decltype(exact)::value;
    const bf16_t* ap = tile + (32 * wm * MT + lo) * P + 8 * hi;
    Split8 x[2][MT];
    auto read = [&](const bf16_t* p) {
      if (!EXACT) return frag_row(p, PLANE);
      Split8 f;
      f.h = *reinterpret_cast<const bf16x8*>(p);
      return f;
    };
#pragma unroll
    for (int i = 0; i < MT; ++i) x[0][i] = read(ap + 32 * i * P);
#pragma unroll 1
    for (int s0 = 0; s0 < steps; s0 += RING) {
#pragma unroll
      for (int u = 0; u < RING; ++u) {
#pragma unroll
        for (int i = 0; i < MT; ++i) x[(u + 1) & 1][i] = read(ap + 32 * i * P + 16 * (u + 1));  // (past the last step: read, not used)
        __builtin_amdgcn_sched_barrier(0);
#define MARL_SPLIT_PRODUCT(XP, WP) \
  _Pragma("unroll") for (int i = 0; i < MT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[u][WP], x[u & 1][i].XP, acc[i], 0, 0, 0);
        if constexpr (!EXACT) { MARL_SPLIT_PRODUCT(l, 0) }
        MARL_SPLIT_PRODUCT(h, 2)
        if constexpr (!EXACT) { MARL_SPLIT_PRODUCT(m, 1) }
        if constexpr (!EXACT) { MARL_SPLIT_PRODUCT(m, 0) }
        MARL_SPLIT_PRODUCT(h, 1)
        MARL_SPLIT_PRODUCT(h, 0)
#undef MARL_SPLIT_PRODUCT
        load_w(u);
        __builtin_amdgcn_sched_barrier(0);
      }
      ap += 16 * RING;
    }
  };

  // ---- input rows: half a wavefront a row, a lane two neighbouring columns: rows 2 (wave + NW i) + hi, columns 64 j + 2 lo, + 1.
  // Lane i + 32 h keeps the offset of row 2 (wave + NW i) + h.
  int64_t roff;
  auto row_offsets = [&](int64_t t) {
    const int64_t s = min(min(t, ntiles - 1) * BM + min(2 * (wave + NW * min(lo, XR - 1)) + hi, BM - 1), a.S - 1);
    if (a.X.gather == nullptr) roff = s * a.X.ld;
    else roff = a.X.ptr_with<true>(s, a.X.gather_entry<true>(s)) - a.X.base;
  };
  typedef float f2 __attribute__((ext_vector_type(2), aligned(4)));  // rows start at any 4-byte boundary
  f2 xr[XJ][XR];  // the next tile's first piece waits here
  auto load_x = [&](int k0) {  // columns k0 .. k0 + 64 XJ - 1 of the rows at roff
#pragma unroll
    for (int i = 0; i < XR; ++i) {
      const int64_t off = __shfl(roff, i + 32 * hi);
#pragma unroll
      for (int j = 0; j < XJ; ++j) xr[j][i] = *reinterpret_cast<const f2*>(a.X.base + off + min(k0 + 64 * j + 2 * lo, a.Din - 2));
    }
  };
  auto store_x = [&](int k0) {
    // finite values that are exact in bf16 (their lower 16 bits are zero) need no split, and that is what windows consist of
    uint32_t low_bits = 0;
    float top = 0.f;
#pragma unroll
    for (int j = 0; j < XJ; ++j) {
      const int c = k0 + 64 * j + 2 * lo;
#pragma unroll
      for (int i = 0; i < XR; ++i) {
        xr[j][i].x = c >= a.Din ? 0.f : c == a.Din - 1 ? xr[j][i].y : xr[j][i].x;
        xr[j][i].y = c + 1 < a.Din ? xr[j][i].y : 0.f;
        low_bits |= __float_as_uint(xr[j][i].x) | __float_as_uint(xr[j][i].y);
        top = fmaxf(fmaxf(top, fabsf(xr[j][i].x)), fabsf(xr[j][i].y));
      }
    }
    const bool exact = __builtin_amdgcn_ballot_w64((low_bits & 0xffffu) != 0 || __builtin_isinf(top)) == 0;  // uniform
    if (EXACT_X && !exact) *inexact = 1;
#pragma unroll
    for (int j = 0; j < XJ; ++j) {
#pragma unroll
      for (int i = 0; i < XR; ++i) {
        const int row = 2 * (wave + NW * i) + hi;
        uint32_t* const d = reinterpret_cast<uint32_t*>(&tile[row * P + 64 * j + 2 * lo]);
        SplitPair s{__float_as_uint(xr[j][i].x) >> 16 | (__float_as_uint(xr[j][i].y) & 0xffff0000u), 0u, 0u};
        if (!exact) s = split_pair_any(xr[j][i].x, xr[j][i].y);
        if (XR * NW * 2 == BM || row < BM) {
          d[0] = s.h;
          d[PLANE / 2] = s.m;
          d[PLANE] = s.l;
        }
      }
    }
  };
  auto unit_of = [&](int g4) { return 32 * wn + 8 * g4 + 4 * hi; };  // first of four consecutive units
  auto row_of = [&](int i) { return 32 * (wm * MT + i) + lo; };
  // acc -> tanh(acc + bias) -> the tile, and kept in `keep` (TRAIN)
  auto tanh_out = [&](const float* b, floatx16 (&keep)[TRAIN ? MT : 1]) {
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const float4 bq = *reinterpret_cast<const float4*>(&b[unit_of(g4)]);
      const float bb[4] = {bq.x, bq.y, bq.z, bq.w};
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          v[j] = tanh_f32(acc[i][4 * g4 + j] + bb[j]);
          if (TRAIN) keep[TRAIN ? i : 0][4 * g4 + j] = v[j];
        }
        store_split4<false>(&tile[row_of(i) * P + unit_of(g4)], PLANE, make_float4(v[0], v[1], v[2], v[3]));
      }
    }
  };
  auto store_rows = [&](float* dst, int rows, const floatx16 (&v)[MT]) {  // four units of a sample a lane
#pragma unroll
    for (int i = 0; i < MT; ++i)
      if (row_of(i) < rows) {
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4)
          *reinterpret_cast<float4*>(dst + row_of(i) * H + unit_of(g4)) = make_float4(v[i][4 * g4], v[i][4 * g4 + 1], v[i][4 * g4 + 2], v[i][4 * g4 + 3]);
      }
  };

  typedef float f4 __attribute__((ext_vector_type(4)));
  f4 gw[2];  // TRAIN: W3 gradient: units 32 wn + 16 u + 4 l4 + r, output l15, this wavefront's samples
  floatx16 h1[TRAIN ? MT : 1], h2[TRAIN ? MT : 1];
  gw[0] = gw[1] = f4{0.f, 0.f, 0.f, 0.f};
  if ((int64_t)blockIdx.x < ntiles) {
    row_offsets(blockIdx.x);
    if (AHEAD) load_x(0);
  }
  __syncthreads();  // what was set up above, *inexact first of all
  for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
    asm volatile("" : "+v"(lane));  // what depends on the lane is formed anew for every tile: kept, the many addresses were spilled
    lo = lane & 31; hi = lane >> 5; l15 = lane & 15; l4 = lane >> 4;
    const int64_t s0 = t * BM;
    const int rows = (int)min((int64_t)BM, a.S - s0);
    const bool more = t + gridDim.x < ntiles;  // uniform
    [[maybe_unused]] int32_t entry[GPW];
    if constexpr (TRAIN) {
#pragma unroll
      for (int g = 0; g < GPW; ++g)
        if (wave + NW * g < BM / 16) entry[g] = fin.template row_entry<true>(min(s0 + min(16 * (wave + NW * g), BM - 16) + l15, a.S - 1));
    }
    // ---- layer 1
    zero_acc();
    for (int k0 = 0; k0 < a.Kp; k0 += 64 * XJ) {
      if (!AHEAD || k0 > 0) load_x(k0);
      if (k0 > 0) __syncthreads();
      store_x(k0);
      __syncthreads();
      const int steps = min(steps1 - k0 / 16, 4 * XJ);
      if (EXACT_X && *inexact == 0) product(steps, std::integral_constant<bool, EXACT_X>{});  // uniform
      else product(steps, std::false_type{});
    }
    row_offsets(t + gridDim.x);
    __syncthreads();  // the input has been read
    if (EXACT_X && tid == 0) *inexact = 0;
    tanh_out(bias, h1);
    __syncthreads();
    if constexpr (TRAIN) store_rows(a.h1 + s0 * H, rows, h1);
    // ---- layer 2
    zero_acc();
    if (AHEAD && more) load_x(0);
    product(H / 16, std::false_type{});
    typename SplitNetLossIn<TRAIN, Fin>::type lin[GPW];
    if constexpr (TRAIN) {
#pragma unroll
      for (int g = 0; g < GPW; ++g)
        if (wave + NW * g < BM / 16) lin[g] = fin.template load_with<true>(min(s0 + min(16 * (wave + NW * g), BM - 16) + l15, a.S - 1), entry[g]);
    }
    __syncthreads();
    tanh_out(bias + H, h2);
    __syncthreads();
    // ---- output layer: W3^T x h2 for sixteen samples at a time; outputs 0 .. 3 land in lanes 0 .. 15, 4 .. 7 in the next sixteen
    float outs[GPW][NOUT];
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
      const int grp = wave + NW * g;
      if (GPW * NW == BM / 16 || grp < BM / 16) {  // uniform
        f4 o = {0.f, 0.f, 0.f, 0.f}, small = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
        for (int k = 0; k < H; k += 32) {
          const Split8 wv = frag_row(&w3t[(lane & 7) * P + k + 8 * l4], PLANE3), xv = frag_row(&tile[(16 * grp + l15) * P + k + 8 * l4], PLANE);
          small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv.h, xv.l, small, 0, 0, 0);
          small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv.l, xv.h, small, 0, 0, 0);
          small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv.m, xv.m, small, 0, 0, 0);
          small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv.h, xv.m, small, 0, 0, 0);
          small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv.m, xv.h, small, 0, 0, 0);
          o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv.h, xv.h, o, 0, 0, 0);
        }
        const f4 v = small + o;
#pragma unroll
        for (int k = 0; k < NOUT; ++k) outs[g][k] = (k < 4 ? v[k & 3] : __shfl(v[k & 3], (lane + 16) & 63)) + (TRAIN ? b3s[k] : bias3[TRAIN ? 0 : k]);
      }
    }
    if constexpr (!TRAIN) {
#pragma unroll
      for (int g = 0; g < GPW; ++g) {
        const int64_t s = s0 + 16 * (wave + NW * g) + l15;
        if ((GPW * NW == BM / 16 || wave + NW * g < BM / 16) && lane < 16 && s < a.S) fin(s, outs[g], nullptr, nullptr);
      }
      __syncthreads();  // the tile is free
    } else {
#pragma unroll
      for (int g = 0; g < GPW; ++g) {
        const int grp = wave + NW * g;
        const int64_t s = s0 + 16 * grp + l15;
        if ((GPW * NW == BM / 16 || grp < BM / 16) && lane < 16) {
          float dl[NOUT], st[5] = {0.f, 0.f, 0.f, 0.f, 0.f}, mine = 0.f;
#pragma unroll
          for (int k = 0; k < NOUT; ++k) dl[k] = 0.f;
          if (s < a.S) fin.compute(lin[g], *prep, outs[g], dl, st);
#pragma unroll
          for (int k = 0; k < NOUT; ++k) {
            dls[(16 * grp + l15) * 8 + k] = dl[k];
            const SplitPair sp = split_pair_any(dl[k], 0.f);
            dlt[k * PD + 16 * grp + l15] = (bf16_t)sp.h;
            dlt[(8 + k) * PD + 16 * grp + l15] = (bf16_t)sp.m;
            dlt[(16 + k) * PD + 16 * grp + l15] = (bf16_t)sp.l;
          }
#pragma unroll
          for (int k = 0; k < AS; ++k) {
            if (k >= NOUT && (Fin::kStats >> (k >= NOUT ? k - NOUT : 0) & 1) == 0) continue;
            const float v = row_sum16(k < NOUT ? dl[k < NOUT ? k : 0] : st[k < NOUT ? 0 : k - NOUT]);
            mine = l15 == k ? v : mine;
          }
          if (l15 < AS) accD[grp * AS + l15] += mine;
        }
      }
      __syncthreads();
      // From here to the next barrier a wavefront reads and writes nothing of the tile but its own rows and columns.
      // ---- W3 gradient: h2^T x dl
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int sb = 32 * (wm * MT + i);
        const Split8 d = frag_row(&dlt[(lane & 7) * PD + sb + 8 * l4], 8 * PD);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const bf16_t* const p = &tile[(sb + 8 * l4 + (l15 >> 2)) * P + 32 * wn + 16 * u + 4 * (lane & 3)];
          const Split8 h = Split8{read_col8(p, P), read_col8(p + PLANE, P), read_col8(p + 2 * PLANE, P)};
          gw[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h.l, d.h, gw[u], 0, 0, 0);
          gw[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h.h, d.l, gw[u], 0, 0, 0);
          gw[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h.m, d.m, gw[u], 0, 0, 0);
          gw[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h.m, d.h, gw[u], 0, 0, 0);
          gw[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h.h, d.m, gw[u], 0, 0, 0);
          gw[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h.h, d.h, gw[u], 0, 0, 0);
        }
      }
      // ---- dz2 = (dl W3^T) (1 - h2^2), into h2's registers and over h2 in the tile
      float dv[MT][8];
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const float4 d0 = *reinterpret_cast<const float4*>(&dls[row_of(i) * 8]);
        dv[i][0] = d0.x; dv[i][1] = d0.y; dv[i][2] = d0.z; dv[i][3] = d0.w;
        if (NOUT > 4) {
          const float4 d1 = *reinterpret_cast<const float4*>(&dls[row_of(i) * 8 + 4]);
          dv[i][4] = d1.x; dv[i][5] = d1.y; dv[i][6] = d1.z; dv[i][7] = d1.w;
        }
      }
      float top = 0.f;
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float wv[8];
          const float* const wp = &w3s[(unit_of(g4) + j) * W3P];
          if (NOUT > 1) {
            const float4 w0 = *reinterpret_cast<const float4*>(wp), w1 = *reinterpret_cast<const float4*>(wp + (NOUT > 1 ? 4 : 0));
            wv[0] = w0.x; wv[1] = w0.y; wv[2] = w0.z; wv[3] = w0.w; wv[4] = w1.x; wv[5] = w1.y;
          } else {
            wv[0] = *wp;
          }
#pragma unroll
          for (int i = 0; i < MT; ++i) {
            float d = 0.f;
#pragma unroll
            for (int k = 0; k < NOUT; ++k) d = fmaf(dv[i][k], wv[k], d);
            const float h = h2[i][4 * g4 + j];
            h2[i][4 * g4 + j] = d * (1.0f - h * h);
            top = fmaxf(top, fabsf(h2[i][4 * g4 + j]));
          }
        }
      const bool wild = split_out_of_range(top);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const float4 v = make_float4(h2[i][4 * g4], h2[i][4 * g4 + 1], h2[i][4 * g4 + 2], h2[i][4 * g4 + 3]);
          bf16_t* const d = &tile[row_of(i) * P + unit_of(g4)];
          if (wild) store_split4<true>(d, PLANE, v);
          else store_split4<false>(d, PLANE, v);
        }
      __syncthreads();
      store_rows(a.dz2 + s0 * H, rows, h2);
      // ---- dz1 = (W2 dz2^T) (1 - h1^2)
      zero_acc();
      product(H / 16, std::false_type{});
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] *= 1.0f - h1[i][r] * h1[i][r];
      store_rows(a.dz1 + s0 * H, rows, acc);
      __syncthreads();  // the tile is free
    }
  }
  if constexpr (TRAIN) {
    // this workgroup's sums: the WM wavefronts that share their columns meet in LDS
    constexpr int COUNT = H * NOUT + NOUT + 5;
    float* const G = reinterpret_cast<float*>(tile);  // [WM][H * NOUT]
    static_assert(WM * H * NOUT * 4 <= 3 * BM * P * 2, "room in the tile");
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (l15 < NOUT) G[wm * H * NOUT + (32 * wn + 16 * u + 4 * l4 + r) * NOUT + l15] = gw[u][r];
    __syncthreads();
    float* const own = a.partial + blockIdx.x * copy_pitch(COUNT);
    for (int e = tid; e < COUNT; e += THREADS) {
      float v = 0.f;
      if (e < H * NOUT) {
#pragma unroll
        for (int z = 0; z < WM; ++z) v += G[z * H * NOUT + e];
      } else {
        double sum = 0.0;
        for (int z = 0; z < BM / 16; ++z) sum += accD[z * AS + e - H * NOUT];
        v = (float)sum;
      }
      own[e] = v;
    }
  }
}

// Workgroups of a launch at most: twice as many as the chip holds at once, so that the last tiles find a free place (50 000 samples,
// 192 units: 132 us with as many as it holds, 104 with twice as many).  32-row tiles of 64 and 96 units: as many as it holds, seven and
// five per CU (20 minibatches of 400 000 samples of 147 inputs, both networks of 64 units: 15.4 ms, with twice as many 15.8, with 2048, of
// which the last 256 ran by themselves, 17.1; of 96 units 20.5, 20.7 and 21.7; of 50 000 samples and 96 units 4.08, 4.18 and 4.18).
constexpr unsigned split_net_grid(int H, int BM) {
  return BM == 32 && H == 64 ? 7 * 256 : BM == 32 && H == 96 ? 5 * 256 : H <= 128 ? 2048 : H <= 256 && BM == 32 ? 1024 : 512;
}
constexpr int kSplitTrainRows = 32;
inline int64_t split_net_partial_floats(int H, int nout) { return split_net_grid(H, kSplitTrainRows) * copy_pitch((int64_t)H * nout + nout + 5); }

template <int H, int BM, int NOUT, bool TRAIN, class Fin>
inline int32_t launch_split_net_inst(const SplitNetArgs& a, const Fin& fin, unsigned* grid_out, hipStream_t s) {
  auto kern = split_net_kernel<H, BM, NOUT, TRAIN, Fin>;
  const size_t bytes = SplitNetShape<H, BM>::lds(TRAIN, NOUT);
  if (bytes > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
    return MARL_E_LAUNCH;
  const int64_t tiles = (a.S + BM - 1) / BM;
  const unsigned grid = (unsigned)std::min<int64_t>(tiles, split_net_grid(H, BM));
  if (grid_out != nullptr) *grid_out = grid;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * SplitNetShape<H, BM>::NW), bytes, s, a, fin);
  return launch_status();
}
template <int BM, int NOUT, bool TRAIN, class Fin>
inline int32_t launch_split_net_rows(int H, const SplitNetArgs& a, const Fin& fin, unsigned* grid, hipStream_t s) {
  switch (H / 32) {
    case 1: return launch_split_net_inst<32, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 2: return launch_split_net_inst<64, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 3: return launch_split_net_inst<96, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 4: return launch_split_net_inst<128, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 5: return launch_split_net_inst<160, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 6: return launch_split_net_inst<192, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 7: return launch_split_net_inst<224, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 8: return launch_split_net_inst<256, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 9: return launch_split_net_inst<288, BM, NOUT, TRAIN>(a, fin, grid, s);
    default: return launch_split_net_inst<320, BM, NOUT, TRAIN>(a, fin, grid, s);
  }
}

// forward pass; what becomes of the outputs is fin's business
// Tiles of 32 rows below one 64-row tile per CU; the same bits in both.
constexpr int64_t kSplitSmallRows = 16384;
template <int NOUT, class Fin>
inline int32_t launch_split_forward(int H, const SplitNetArgs& a, const Fin& fin, hipStream_t s) {
  TimedLaunch timed(KC_GEMM_NN, 2.0 * (double)a.S * ((double)a.Din * H + (double)H * H), s);
  if (a.S < kSplitSmallRows) return launch_split_net_rows<32, NOUT, false>(H, a, fin, nullptr, s);
  return launch_split_net_rows<64, NOUT, false>(H, a, fin, nullptr, s);
}

}  // namespace marl
