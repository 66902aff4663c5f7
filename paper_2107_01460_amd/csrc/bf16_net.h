// Networks of the bf16 configuration: v_mfma_f32_32x32x16_bf16 with fp32 accumulation, activations rounded to bf16 where they
// feed a product, everything element-wise, the output layer's sums, the loss and all gradients in fp32.
//
// bf16_net_kernel takes a tile of rows through a whole network: both hidden layers, the output layer and, in training, the
// loss, the gradients of both hidden layers' pre-activations and the output layer's weight gradient.  A tile's activations
// sit in LDS ([rows][H], one buffer that every layer reads and then overwrites); the weights stream from the L2 straight into
// registers in the order the instruction takes them, one continuous sequence of k steps that runs on from layer to layer and
// from tile to tile.  bf16_wgrad_kernel takes the weight gradients, contracting over the samples of row-major activations
// with transposing LDS reads, so that no transposed copy of an activation ever exists.
//
// Measured on an MI355X against a kernel per layer with packed inputs and transposed copies, 147 inputs, 512 units: minibatch of
// 262 144 samples, actor: pack 72 + layers 146 + 205 + output layer and loss 278 + dz1 203 us -> one launch of 491 us (W3 gradient
// included; 671 TFLOP/s); weight gradients 237 + 104 -> 158 + 109 us; a training iteration of 4096 environments 164 -> 111 ms;
// forward pass of 32 768 samples through both networks and the sampling 159 -> 73 us, with both networks and both stagings in one launch each 64 us.
// Bound: two workgroups of four wavefronts share a CU (64 rows each, 128 of a lane's 256 registers accumulators), and a tile is
// a chain of products (39 of 107 thousand cycles for the pair), tanh (16), gradients on the output side (15), copies and barriers
// that the other workgroup's phases cover; the weights take 1.2 MB from the L2 per tile; at 512 units 36 (six outputs) and 38 (one)
// registers are spilled.  One workgroup of 128 rows per CU halves
// that and left every phase uncovered: 778 us; eight wavefronts of 128 registers per 64 rows: 750 us (spills).
#pragma once
#include <utility>

#include "gemm.h"
#include "heads.h"

namespace marl {

inline int64_t round_up64(int64_t x) { return (x + 63) / 64 * 64; }

// ---- weights ------------------------------------------------------------------------------------------------
// One network's matrices B [K][H] one after the other, each in fragment order: element (k, n) at bf16_frag_index(k, n, H), so
// that the 16 bytes a lane feeds to one instruction are one load and a wavefront's 32 columns x 16 k one contiguous KB.
//   W1 (zero-padded to Kp rows), W2, W2 transposed (for dz1 = dz2 W2^T).
struct Bf16NetWeights {
  bf16_t* w;
  int Kp;
};
__host__ __device__ inline int64_t bf16_frag_index(int64_t k, int64_t n, int64_t H) { return ((k / 16 * (H / 32) + n / 32) * 64 + n % 32 + 32 * (k % 16 / 8)) * 8 + k % 8; }
inline int64_t bf16_net_weight_elems(int Din, int H) { return (round_up64(Din) + 2 * (int64_t)H) * H; }

struct Bf16StageNet {
  const float *W1, *W2;
  bf16_t* w;
  int Din, Kp, H;
};
// A thread takes eight consecutive k of one column: one 16-byte store.
__device__ __forceinline__ void bf16_stage(const Bf16StageNet& a, const Bf16StageNet& b, int64_t i) {
  const int64_t na = (int64_t)(a.Kp + 2 * a.H) * a.H / 8;
  const bool second = i >= na;
  const Bf16StageNet n = second ? b : a;
  if (second) i -= na;
  if (i >= (int64_t)(n.Kp + 2 * n.H) * n.H / 8) return;
  const int k = (int)(i / n.H) * 8, c = (int)(i % n.H);
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (k < n.Kp) v[j] = k + j < n.Din ? n.W1[(int64_t)(k + j) * n.H + c] : 0.f;
    else if (k < n.Kp + n.H) v[j] = n.W2[(int64_t)(k - n.Kp + j) * n.H + c];
    else v[j] = n.W2[(int64_t)c * n.H + (k - n.Kp - n.H + j)];
  }
  *reinterpret_cast<uint4*>(n.w + bf16_frag_index(k, c, n.H)) =
      make_uint4(pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]), pack2_bf16(v[4], v[5]), pack2_bf16(v[6], v[7]));
}
static __global__ void __launch_bounds__(256) bf16_stage_kernel(Bf16StageNet a, Bf16StageNet b) { bf16_stage(a, b, (int64_t)blockIdx.x * 256 + threadIdx.x); }
inline unsigned bf16_stage_blocks(const Bf16StageNet& a, const Bf16StageNet& b) {
  return (unsigned)((((int64_t)(a.Kp + 2 * a.H) * a.H + (int64_t)(b.Kp + 2 * b.H) * b.H) / 8 + 255) / 256);
}
inline void launch_bf16_stage(const Bf16StageNet& a, const Bf16StageNet& b, hipStream_t s) {
  hipLaunchKernelGGL(bf16_stage_kernel, dim3(bf16_stage_blocks(a, b)), dim3(256), 0, s, a, b);
}

// ---- a row tile through a network -----------------------------------------------------------------------------
struct Bf16NetArgs {
  RowSrc X;  // S rows of Din floats; a gather's divisor has its magic number
  int64_t S;
  int Din;
  Bf16NetWeights w;
  const float *b1, *b2, *W3, *b3;  // rounded to bf16
  bf16_t *h1, *dz2, *dz1;          // training: [S][H]
  float* partial;                  // training: per workgroup the W3 gradient, the b3 gradient and five loss statistics
};

// Wavefronts: WN side by side, each NT column tiles of 32, and WM below one another, each MT row tiles of 32.
template <int H, int BM>
struct Bf16Shape {
  static_assert(H % 64 == 0 && H <= 512 && (BM == 32 || BM == 64), "widths the configuration allows");
  static constexpr int NT = H == 512 ? 4 : H > 256 ? 2 : 1, WN = H / (32 * NT);
  static constexpr int WM = BM == 32 || H > 128 ? 1 : 2, MT = BM / (32 * WM), NW = WM * WN;
  // wavefronts per SIMD the registers have to leave room for: two workgroups per CU, which cover each other's phases
  static constexpr int WAVES = NW == 8 ? 4 : NW > 4 ? 3 : 2;
  static constexpr int P = H + 8;    // pitch of the tile: an odd number of 16-byte units
  static constexpr int PD = BM + 8;  // pitch of the output gradients
  // (64 rows of 512 units in training: 80 KB, half of a CU's)
  static constexpr size_t lds(bool train) { return sizeof(bf16_t) * ((BM + 8) * P + (train ? 32 * PD : 0) + 2 * H) + (train ? sizeof(float) * (NW * 11 + 8) : 0); }
};

static_assert(2 * Bf16Shape<512, 64>::lds(true) <= 160 * 1024, "workgroups per CU");

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));  // 16 bytes between a load and an LDS store (HIP's uint4 arrays may stay in scratch memory)
__device__ __forceinline__ floatx16 mfma32_bf16(const bf16x8& a, const bf16x8& b, const floatx16& c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
typedef float bf16_floatx4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16_floatx4 mfma16_bf16(const bf16x8& a, const bf16x8& b, const bf16_floatx4& c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

template <bool TRAIN, class Fin>
struct LossIn { typedef int type, Prep; };
template <class Fin>
struct LossIn<true, Fin> {
  typedef typename Fin::In type;
  typedef decltype(std::declval<Fin>().prepare()) Prep;  // two floats
};

// The kernel's body: workgroup `bid` of `nblk` that share the tiles.
// Fin: TRAIN: a loss functor (ActorLoss, CriticLoss); else what becomes of a sample's outputs, fin(s, out, nullptr, nullptr).
template <int H, int BM, int NOUT, bool TRAIN, class Fin>
__device__ __forceinline__ void bf16_net_body(const Bf16NetArgs& a, const Fin& fin, const unsigned bid, const unsigned nblk) {
  using Sh = Bf16Shape<H, BM>;
  constexpr int NT = Sh::NT, MT = Sh::MT, WN = Sh::WN, NW = Sh::NW, P = Sh::P, PD = Sh::PD, THREADS = 64 * NW;
  constexpr int RING = NT == 1 ? 4 : 2;        // k steps of weights on their way
  constexpr int XJ = H < 192 ? H / 64 : 3;     // 64-column pieces of the input that are staged at a time
  constexpr int RPW = (BM + NW - 1) / NW;      // input rows a wavefront stages
  constexpr int GPW = (BM / 16 + NW - 1) / NW; // groups of 16 samples whose outputs a wavefront takes
  // 16-byte pieces of the tile: a thread has piece pc of the rows pr + PS q, q < QP
  constexpr int PS = THREADS / (H / 8), QP = (BM + PS - 1) / PS;
  static_assert(THREADS % (H / 8) == 0, "a thread's pieces are one column of the tile");
  extern __shared__ __attribute__((aligned(16))) bf16_t bf16_net_lds[];
  bf16_t* const tile = bf16_net_lds;                            // [BM][P] X, h1, h2, dz2, dz1
  bf16_t* const w3t = tile + BM * P;                            // [8][P]  W3 transposed, rows past NOUT zero
  bf16_t* const dlt = w3t + 8 * P;                              // TRAIN: [4][8][PD] dL/d(output), split: three parts and zeros
  bf16_t* const bias = dlt + (TRAIN ? 32 * PD : 0);             // [2][H] (rounded values, exact)
  constexpr int AS = NOUT + 5;
  float* const b3s = reinterpret_cast<float*>(bias + 2 * H);    // TRAIN: [6]
  auto* const prep = reinterpret_cast<typename LossIn<TRAIN, Fin>::Prep*>(b3s + 6);  // TRAIN
  float* const accS = b3s + 8;                                  // TRAIN: [NW][AS] every wavefront's b3 gradient and loss statistics

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
  const int steps1 = a.w.Kp / 16, total = steps1 + (TRAIN ? 2 : 1) * (H / 16);
  const WeightRsrc wsrc = __builtin_amdgcn_make_buffer_rsrc(a.w.w, (short)0, total * 32 * H, 0x00020000);
  const int woff = (wn * NT * 64 + lane) * 16;
  bf16x8 w[RING][NT];
  int nxt = 0;
  auto load_w = [&](int slot) {
#pragma unroll
    for (int q = 0; q < NT; ++q) w[slot][q] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wsrc, woff + 1024 * q, nxt * 32 * H, 0));
    nxt = nxt + 1 == total ? 0 : nxt + 1;
  };
#pragma unroll
  for (int u = 0; u < RING; ++u) load_w(u);

  if constexpr (TRAIN) {
    if (tid == 0) *prep = fin.prepare();
    for (int e = tid; e < NW * AS; e += THREADS) accS[e] = 0.f;
    for (int e = tid; e < 32 * PD; e += THREADS) dlt[e] = 0;
  }
  for (int e = tid; e < (8 - NOUT) * H; e += THREADS) w3t[(NOUT + e / H) * P + e % H] = 0;
  w3.store(tid, [&](int e, float v) { w3t[e % NOUT * P + e / NOUT] = to_bf16(v); });
  b1.store(tid, [&](int e, float v) { bias[e] = to_bf16(v); });
  b2.store(tid, [&](int e, float v) { bias[H + e] = to_bf16(v); });
  if constexpr (TRAIN) {
    if (tid < NOUT) b3s[tid] = b3;
  }

  floatx16 acc[MT][NT];
  auto zero_acc = [&]() {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int q = 0; q < NT; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][q][r] = 0.f;
  };
  // acc += weights x tile over `steps` (a multiple of four) k steps; acc[i][q][r] belongs to unit 32 (wn NT + q) + 8 (r / 4) +
  // 4 hi + r % 4 of sample 32 (wm MT + i) + lo
  // (The scheduling barriers keep the order written here: a step's weights are requested RING steps ahead and its rows of the
  // tile are read one step ahead.  Left alone, the compiler moves the requests to the end of the loop body, where the next
  // iteration waits for them, and reads every operand just in front of its use.)
  auto product = [&](int steps) {
    const bf16_t* ap = tile + (32 * wm * MT + lo) * P + 8 * hi;
    bf16x8 x[2][MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) x[0][i] = *reinterpret_cast<const bf16x8*>(ap + 32 * i * P);
#pragma unroll 1
    for (int s0 = 0; s0 < steps; s0 += RING) {
#pragma unroll
      for (int u = 0; u < RING; ++u) {
#pragma unroll
        for (int i = 0; i < MT; ++i) x[(u + 1) & 1][i] = *reinterpret_cast<const bf16x8*>(ap + 32 * i * P + 16 * (u + 1));  // (past the last step: read, not used)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int q = 0; q < NT; ++q) acc[i][q] = mfma32_bf16(w[u][q], x[u & 1][i], acc[i][q]);
        load_w(u);
        __builtin_amdgcn_sched_barrier(0);
      }
      ap += 16 * RING;
    }
  };

  // ---- input rows: wavefront -> rows wave + NW i, lane -> columns 64 j + lane.  The rows' offsets sit one per lane.
  int64_t roff;
  auto row_offsets = [&](int64_t t) {
    const int64_t s = min(min(t, ntiles - 1) * BM + min(wave + NW * min(lane, RPW - 1), BM - 1), a.S - 1);
    if (a.X.gather == nullptr) roff = s * a.X.ld;
    else roff = a.X.ptr_with<true>(s, a.X.gather_entry<true>(s)) - a.X.base;
  };
  auto stage_x = [&](int k0) {  // columns k0 .. k0 + 64 XJ - 1 of the tile's rows
    float xr[XJ][RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
      const uint32_t off_lo = __builtin_amdgcn_readlane((int)(uint32_t)roff, i), off_hi = __builtin_amdgcn_readlane((int)(roff >> 32), i);
      const float* const p = a.X.base + (int64_t)((uint64_t)off_hi << 32 | off_lo);
#pragma unroll
      for (int j = 0; j < XJ; ++j) xr[j][i] = p[min(k0 + 64 * j + lane, a.Din - 1)];
    }
#pragma unroll
    for (int j = 0; j < XJ; ++j) {
      const bool in = k0 + 64 * j + lane < a.Din;
#pragma unroll
      for (int i = 0; i < RPW; ++i)
        if (RPW * NW == BM || wave + NW * i < BM) tile[(wave + NW * i) * P + 64 * j + lane] = in ? to_bf16(xr[j][i]) : (bf16_t)0;
    }
  };
  // the whole tile to global memory (samples past the end stay away)
  auto copy_out = [&](bf16_t* dst, int rows) {
    int f = tid;
    asm volatile("" : "+v"(f));  // the offsets are formed here: kept across the tile loop they would be spilled
    const int pr = f / (H / 8), pc = 8 * (f % (H / 8));
    if (rows == BM && BM % PS == 0) {  // uniform
      constexpr int QB = QP % 8 == 0 ? 8 : QP % 4 == 0 ? 4 : 1;
#pragma unroll
      for (int q0 = 0; q0 < QP; q0 += QB) {
        u32x4_t v[QB];
#pragma unroll
        for (int q = 0; q < QB; ++q) v[q] = *reinterpret_cast<const u32x4_t*>(&tile[(pr + PS * (q0 + q)) * P + pc]);
#pragma unroll
        for (int q = 0; q < QB; ++q) *reinterpret_cast<u32x4_t*>(dst + (pr + PS * (q0 + q)) * H + pc) = v[q];
      }
    } else {
#pragma unroll 1
      for (int r = pr; r < rows; r += PS) *reinterpret_cast<u32x4_t*>(dst + r * H + pc) = *reinterpret_cast<const u32x4_t*>(&tile[r * P + pc]);
    }
  };
  // this lane's four consecutive units 8 g4 + 4 hi .. of column tile q, as an offset into a row of the tile
  auto unit_of = [&](int q, int g4) { return 32 * (wn * NT + q) + 8 * g4 + 4 * hi; };
  auto row_of = [&](int i) { return 32 * (wm * MT + i) + lo; };
  // acc -> tanh(acc + bias) in bf16 -> the tile
  auto tanh_out = [&](const bf16_t* b) {
#pragma unroll
    for (int q = 0; q < NT; ++q)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const uint2 bq = *reinterpret_cast<const uint2*>(&b[unit_of(q, g4)]);
        const float bb[4] = {__uint_as_float(bq.x << 16), __uint_as_float(bq.x & 0xffff0000u), __uint_as_float(bq.y << 16), __uint_as_float(bq.y & 0xffff0000u)};
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          float v[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = tanh_f32(acc[i][q][4 * g4 + j] + bb[j]);
          *reinterpret_cast<uint2*>(&tile[row_of(i) * P + unit_of(q, g4)]) = make_uint2(pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]));
        }
      }
  };

  // four values of the tile, times g, back in place: x -> g (1 - x^2)
  auto dtanh_in_place = [&](int i, int q, const floatx16& g) {
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      uint2* const p = reinterpret_cast<uint2*>(&tile[row_of(i) * P + unit_of(q, g4)]);
      const uint2 h = *p;
      const float hh[4] = {__uint_as_float(h.x << 16), __uint_as_float(h.x & 0xffff0000u), __uint_as_float(h.y << 16), __uint_as_float(h.y & 0xffff0000u)};
      float v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = g[4 * g4 + j] * (1.0f - hh[j] * hh[j]);
      *p = make_uint2(pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]));
    }
  };

  bf16_floatx4 gw[TRAIN ? 2 * NT : 1];  // W3 gradient: units 16 u + 4 l4 + r of this wavefront's columns, output l15, its own samples
#pragma unroll
  for (int u = 0; u < (TRAIN ? 2 * NT : 1); ++u) gw[u] = bf16_floatx4{0.f, 0.f, 0.f, 0.f};

  if ((int64_t)bid < ntiles) row_offsets(bid);
  for (int64_t t = bid; t < ntiles; t += nblk) {
    asm volatile("" : "+v"(lane));  // what depends on the lane is formed anew for every tile: kept, the many addresses were spilled
    lo = lane & 31; hi = lane >> 5; l15 = lane & 15; l4 = lane >> 4;
    const int64_t s0 = t * BM;
    const int rows = (int)min((int64_t)BM, a.S - s0);
    const bool more = t + nblk < ntiles;       // uniform
    [[maybe_unused]] int32_t entry[GPW];       // the loss's row order entries of this wavefront's samples, requested long before the rows
    if constexpr (TRAIN) {
#pragma unroll
      for (int g = 0; g < GPW; ++g)
        if (GPW * NW == BM / 16 || wave + NW * g < BM / 16) entry[g] = fin.template row_entry<true>(min(s0 + 16 * (wave + NW * g) + l15, a.S - 1));
    }
    // ---- layer 1
    stage_x(0);
    __syncthreads();
    zero_acc();
    product(min(steps1, 4 * XJ));
    for (int k0 = 64 * XJ; k0 < a.w.Kp; k0 += 64 * XJ) {
      __syncthreads();
      stage_x(k0);
      __syncthreads();
      product(min(steps1 - k0 / 16, 4 * XJ));
    }
    if (more) row_offsets(t + nblk);
    __syncthreads();  // the input has been read
    tanh_out(bias);
    __syncthreads();
    if (TRAIN) copy_out(a.h1 + s0 * H, rows);
    // ---- layer 2
    zero_acc();
    product(H / 16);
    __syncthreads();
    typename LossIn<TRAIN, Fin>::type lin[GPW];
    if constexpr (TRAIN) {
#pragma unroll
      for (int g = 0; g < GPW; ++g)
        if (GPW * NW == BM / 16 || wave + NW * g < BM / 16) lin[g] = fin.template load_with<true>(min(s0 + 16 * (wave + NW * g) + l15, a.S - 1), entry[g]);
    }
    tanh_out(bias + H);
    __syncthreads();
    // ---- output layer: W3^T x h2 for sixteen samples at a time; outputs 0 .. 3 land in lanes 0 .. 15, 4 .. 7 in the next sixteen
    float outs[GPW][NOUT];
#pragma unroll
    for (int g = 0; g < GPW; ++g) {
      const int grp = wave + NW * g;
      if (GPW * NW == BM / 16 || grp < BM / 16) {  // uniform
        bf16_floatx4 o[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll 2
        for (int k = 0; k < H; k += 64) {
#pragma unroll
          for (int z = 0; z < 2; ++z)
            o[z] = mfma16_bf16(*reinterpret_cast<const bf16x8*>(&w3t[(lane & 7) * P + k + 32 * z + 8 * l4]),
                               *reinterpret_cast<const bf16x8*>(&tile[(16 * grp + l15) * P + k + 32 * z + 8 * l4]), o[z]);
        }
        const bf16_floatx4 v = o[0] + o[1];
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
            const SplitPair sp = split_pair_any(dl[k], 0.f);
            dlt[k * PD + 16 * grp + l15] = (bf16_t)sp.h;
            dlt[(8 + k) * PD + 16 * grp + l15] = (bf16_t)sp.m;
            dlt[(16 + k) * PD + 16 * grp + l15] = (bf16_t)sp.l;
          }
#pragma unroll
          for (int k = 0; k < AS; ++k) {  // (sums over the sixteen samples: there is no room for one per sample)
            if (k >= NOUT && (Fin::kStats >> (k >= NOUT ? k - NOUT : 0) & 1) == 0) continue;
            const float v = row_sum16(k < NOUT ? dl[k < NOUT ? k : 0] : st[k < NOUT ? 0 : k - NOUT]);
            mine = l15 == k ? v : mine;
          }
          if (l15 < AS) accS[wave * AS + l15] += mine;
        }
      }
      __syncthreads();
      // From here to the next barrier a wavefront reads and writes nothing of the tile but its own rows and columns.
      // ---- W3 gradient: h2^T x dl (h2 is exact in bf16, dl split in three), small parts first
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int sb = 32 * (wm * MT + i);
        bf16x8 d[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) d[p] = *reinterpret_cast<const bf16x8*>(&dlt[(8 * p + (lane & 7)) * PD + sb + 8 * l4]);
#pragma unroll
        for (int u = 0; u < 2 * NT; ++u) {
          const bf16x8 h = read_col8(&tile[(sb + 8 * l4 + (l15 >> 2)) * P + 32 * wn * NT + 16 * u + 4 * (lane & 3)], P);
#pragma unroll
          for (int p = 2; p >= 0; --p) gw[u] = mfma16_bf16(h, d[p], gw[u]);
        }
      }
      // ---- dz2 = (W3 dl^T) (1 - h2^2): k = 0 .. 7 the outputs with one part of dl, k = 8 .. 15 with the next
#pragma unroll
      for (int q = 0; q < NT; ++q) {
        const bf16x8 w3 = read_col8(&w3t[(l15 >> 2) * P + 32 * (wn * NT + q) + 16 * (l4 & 1) + 4 * (lane & 3)], P);
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          const bf16_t* const d = &dlt[(8 * hi + (l15 >> 2)) * PD + 32 * (wm * MT + i) + 16 * (l4 & 1) + 4 * (lane & 3)];
          floatx16 g;
#pragma unroll
          for (int r = 0; r < 16; ++r) g[r] = 0.f;
          g = mfma32_bf16(w3, read_col8(d + 16 * PD, PD), g);
          g = mfma32_bf16(w3, read_col8(d, PD), g);
          dtanh_in_place(i, q, g);
        }
      }
      __syncthreads();
      copy_out(a.dz2 + s0 * H, rows);
      // ---- dz1 = (W2 dz2^T) (1 - h1^2)
      zero_acc();
      product(H / 16);
      // the tile's h1 comes back, every thread the pieces it stored (half of them at a time, for want of registers)
      {
        constexpr int QH = (QP + 1) / 2;
        int f = tid;
        asm volatile("" : "+v"(f));
        const int pr = f / (H / 8), pc = 8 * (f % (H / 8));
        const bf16_t* const src = a.h1 + s0 * H;
#pragma unroll
        for (int q0 = 0; q0 < QP; q0 += QH) {
          u32x4_t hv[QH];
#pragma unroll
          for (int q = 0; q < QH; ++q) hv[q] = *reinterpret_cast<const u32x4_t*>(src + min(pr + PS * (q0 + q), rows - 1) * H + pc);  // (rows past the end: the last one)
          if (q0 == 0) __syncthreads();  // dz2 has been read
#pragma unroll
          for (int q = 0; q < QH; ++q)
            if (pr + PS * (q0 + q) < BM) *reinterpret_cast<u32x4_t*>(&tile[(pr + PS * (q0 + q)) * P + pc]) = hv[q];
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < NT; ++q)
#pragma unroll
        for (int i = 0; i < MT; ++i) dtanh_in_place(i, q, acc[i][q]);
      __syncthreads();
      copy_out(a.dz1 + s0 * H, rows);
      __syncthreads();  // the tile is free
    }
  }
  if constexpr (TRAIN) {
    // this workgroup's sums: the WM wavefronts that share their columns meet in LDS
    constexpr int WM = Sh::WM, COUNT = H * NOUT + NOUT + 5;
    float* const G = reinterpret_cast<float*>(tile);  // [WM][H * NOUT]
    static_assert(WM * H * NOUT * 4 <= BM * P * 2, "room in the tile");
#pragma unroll
    for (int u = 0; u < 2 * NT; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (l15 < NOUT) G[wm * H * NOUT + (32 * wn * NT + 16 * u + 4 * l4 + r) * NOUT + l15] = gw[u][r];
    __syncthreads();
    float* const own = a.partial + bid * copy_pitch(COUNT);
    for (int e = tid; e < COUNT; e += THREADS) {
      float v = 0.f;
      if (e < H * NOUT) {
#pragma unroll
        for (int z = 0; z < WM; ++z) v += G[z * H * NOUT + e];
      } else {
#pragma unroll
        for (int z = 0; z < NW; ++z) v += accS[z * AS + e - H * NOUT];
      }
      own[e] = v;
    }
  }
}

template <int H, int BM, int NOUT, bool TRAIN, class Fin>
__global__ void __launch_bounds__((64 * Bf16Shape<H, BM>::NW), (Bf16Shape<H, BM>::WAVES)) bf16_net_kernel(Bf16NetArgs a, Fin fin) {
  bf16_net_body<H, BM, NOUT, TRAIN, Fin>(a, fin, blockIdx.x, gridDim.x);
}
// Forward pass of two networks of one width in one launch, workgroups 0 .. grid_a - 1 the first.
template <int H, int BM, int NOUT_A, int NOUT_B, class FinA, class FinB>
__global__ void __launch_bounds__((64 * Bf16Shape<H, BM>::NW), (Bf16Shape<H, BM>::WAVES)) bf16_net_pair_kernel(Bf16NetArgs a, FinA fa, Bf16NetArgs b, FinB fb, unsigned grid_a) {
  if (blockIdx.x < grid_a) bf16_net_body<H, BM, NOUT_A, false, FinA>(a, fa, blockIdx.x, grid_a);
  else bf16_net_body<H, BM, NOUT_B, false, FinB>(b, fb, blockIdx.x - grid_a, gridDim.x - grid_a);
}

// Forward passes of fewer samples take tiles of 32 rows instead of 64: below one taller tile per CU the lower ones occupy more of
// the chip.  us, 64 / 32 rows, one network: 512 units, 8192 samples 31.8 / 27.1, 16 384: 33.6 / 34.2, 32 768: 42.6 / 52.4;
// 256 units, 12 288: 16.1 / 15.4, 32 768: 20.7 / 24.8.  (Same bits: both take a sample's sums in the same order.)
constexpr int64_t kBf16SmallRows = 16384;
inline int64_t bf16_net_partial_floats(int H, int nout) { return (int64_t)H * nout + nout + 5; }
// Workgroups of a launch at most: what fits the chip at once above 256 units, up to twice as many below (a workgroup's prologue stages W3
// and asks for its first weights).
constexpr unsigned bf16_net_grid(int H) { return H > 256 ? 512 : 1024; }

inline unsigned bf16_net_blocks(int H, int BM, int64_t S) { return (unsigned)std::min<int64_t>((S + BM - 1) / BM, BM == 32 ? 2 * bf16_net_grid(H) : bf16_net_grid(H)); }

template <int H, int BM, int NOUT, bool TRAIN, class Fin>
inline int32_t launch_bf16_net_inst(const Bf16NetArgs& a, const Fin& fin, unsigned* grid_out, hipStream_t s) {
  auto kern = bf16_net_kernel<H, BM, NOUT, TRAIN, Fin>;
  const size_t bytes = Bf16Shape<H, BM>::lds(TRAIN);
  if (bytes > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
    return MARL_E_LAUNCH;
  const unsigned grid = bf16_net_blocks(H, BM, a.S);
  if (grid_out != nullptr) *grid_out = grid;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * Bf16Shape<H, BM>::NW), bytes, s, a, fin);
  return launch_status();
}
template <int BM, int NOUT, bool TRAIN, class Fin>
inline int32_t launch_bf16_net_rows(int H, const Bf16NetArgs& a, const Fin& fin, unsigned* grid, hipStream_t s) {
  switch (H) {
    case 64: return launch_bf16_net_inst<64, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 128: return launch_bf16_net_inst<128, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 192: return launch_bf16_net_inst<192, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 256: return launch_bf16_net_inst<256, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 320: return launch_bf16_net_inst<320, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 384: return launch_bf16_net_inst<384, BM, NOUT, TRAIN>(a, fin, grid, s);
    case 448: return launch_bf16_net_inst<448, BM, NOUT, TRAIN>(a, fin, grid, s);
    default: return launch_bf16_net_inst<512, BM, NOUT, TRAIN>(a, fin, grid, s);
  }
}
// forward pass; what becomes of the outputs is fin's business
template <int NOUT, class Fin>
inline int32_t launch_bf16_forward(int H, const Bf16NetArgs& a, const Fin& fin, hipStream_t s) {
  TimedLaunch timed(KC_GEMM_NN, 2.0 * (double)a.S * ((double)a.Din * H + (double)H * H), s);
  if (a.S < kBf16SmallRows) return launch_bf16_net_rows<32, NOUT, false>(H, a, fin, nullptr, s);
  return launch_bf16_net_rows<64, NOUT, false>(H, a, fin, nullptr, s);
}
// ... of two networks of one width whose tiles have the same height
inline bool bf16_pair_supported(int Ha, int64_t Sa, int Hb, int64_t Sb) { return Ha == Hb && (Sa < kBf16SmallRows) == (Sb < kBf16SmallRows); }
template <int H, int BM, int NOUT_A, int NOUT_B, class FinA, class FinB>
inline int32_t launch_bf16_pair_inst(const Bf16NetArgs& a, const FinA& fa, const Bf16NetArgs& b, const FinB& fb, hipStream_t s) {
  auto kern = bf16_net_pair_kernel<H, BM, NOUT_A, NOUT_B, FinA, FinB>;
  const size_t bytes = Bf16Shape<H, BM>::lds(false);
  if (bytes > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
    return MARL_E_LAUNCH;
  const unsigned ga = bf16_net_blocks(H, BM, a.S), gb = bf16_net_blocks(H, BM, b.S);
  hipLaunchKernelGGL(kern, dim3(ga + gb), dim3(64 * Bf16Shape<H, BM>::NW), bytes, s, a, fa, b, fb, ga);
  return launch_status();
}
template <int BM, int NOUT_A, int NOUT_B, class FinA, class FinB>
inline int32_t launch_bf16_pair_rows(int H, const Bf16NetArgs& a, const FinA& fa, const Bf16NetArgs& b, const FinB& fb, hipStream_t s) {
  switch (H) {
    case 64: return launch_bf16_pair_inst<64, BM, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    case 128: return launch_bf16_pair_inst<128, BM, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    case 192: return launch_bf16_pair_inst<192, BM, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    case 256: return launch_bf16_pair_inst<256, BM, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    case 320: return launch_bf16_pair_inst<320, BM, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    case 384: return launch_bf16_pair_inst<384, BM, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    case 448: return launch_bf16_pair_inst<448, BM, NOUT_A, NOUT_B>(a, fa, b, fb, s);
    default: return launch_bf16_pair_inst<512, BM, NOUT_A, NOUT_B>(a, fa, b, fb, s);
  }
}
template <int NOUT_A, int NOUT_B, class FinA, class FinB>
inline int32_t launch_bf16_forward_pair(int H, const Bf16NetArgs& a, const FinA& fa, const Bf16NetArgs& b, const FinB& fb, hipStream_t s) {
  TimedLaunch timed(KC_GEMM_NN, 2.0 * (double)a.S * ((double)a.Din * H + (double)H * H) + 2.0 * (double)b.S * ((double)b.Din * H + (double)H * H), s);
  if (a.S < kBf16SmallRows) return launch_bf16_pair_rows<32, NOUT_A, NOUT_B>(H, a, fa, b, fb, s);
  return launch_bf16_pair_rows<64, NOUT_A, NOUT_B>(H, a, fa, b, fb, s);
}


// ---- weight gradients -------------------------------------------------------------------------------------------
// Bound: 64-sample chunks of both operands through LDS, two chunks per CU on their way; at 512 x 512 outputs over 262 144 samples
// 158 us where the bytes take 113 and the products 67, at 147 x 512 109 us (89 and 19).
// slab z of `out`: C[m][n] = sum over the samples of k range z of A[s][m] B[s][n], the column sums of B behind it; the slabs are
// added in a fixed order by reduce_partials_kernel.
struct Bf16WgradArgs {
  RowSrc X;          // XROWS: fp32 rows, rounded on their way; otherwise unused
  const bf16_t* A;   // !XROWS: [S][lda]
  int64_t lda;
  const bf16_t* B;   // [S][N]
  int64_t S;
  int M, N;
  int64_t per;       // samples of a k range, a multiple of the chunk
  unsigned tiles_m, tiles_n;
  float* out;
};

constexpr int kWgradChunk = 64;  // samples staged at a time
// Pitch of an LDS tile that is read along its columns: four consecutive rows on different quarters of the banks.
constexpr int wgrad_pitch(int cols) { return cols % 64 == 0 ? cols + 32 : cols; }

template <bool XROWS, int MT, int NT, int WM, int WN>
__global__ void __launch_bounds__(64 * WM * WN, 2) bf16_wgrad_kernel(Bf16WgradArgs g) {
  constexpr int BM = 32 * MT * WM, BN = 32 * NT * WN, THREADS = 64 * WM * WN, NW = WM * WN, KC = kWgradChunk;
  constexpr int PA = wgrad_pitch(BM), PB = wgrad_pitch(BN), STAGE = KC * (PA + PB);
  constexpr int QA = KC * BM / 8 / THREADS, QB = KC * BN / 8 / THREADS;  // 16-byte pieces a thread stages
  constexpr int RA = THREADS / (BM / 8 > 0 ? BM / 8 : 1), RB = THREADS / (BN / 8);  // rows between a thread's pieces
  constexpr int XR = KC / NW, XJ = (BM + 63) / 64;  // XROWS: rows of a wavefront, 64-column pieces of a row
  static_assert(XROWS || (QA >= 1 && KC * BM / 8 % THREADS == 0 && THREADS % (BM / 8) == 0), "A pieces");
  static_assert(QB >= 1 && KC * BN / 8 % THREADS == 0 && THREADS % (BN / 8) == 0, "B pieces");
  extern __shared__ __attribute__((aligned(16))) bf16_t wgrad_lds[];  // two stages of [A: KC x PA | B: KC x PB]

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lo = lane & 31, hi = lane >> 5, wm = wave / WN, wn = wave % WN;
  // the output tiles of a k range are neighbours on one XCD and share its rows in the L2
  const unsigned lg = xcd_remap(blockIdx.x, gridDim.x);
  const unsigned tn = lg % g.tiles_n, tm = lg / g.tiles_n % g.tiles_m, z = lg / (g.tiles_n * g.tiles_m);
  const int m0 = tm * BM, n0 = tn * BN;
  const int64_t k_begin = (int64_t)z * g.per, k_end = min(g.S, k_begin + g.per);
  const int nchunks = (int)((k_end - k_begin + KC - 1) / KC);

  floatx16 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // A chunk travels in one of two named register sets, is written to LDS one iteration before it is multiplied and was
  // requested three iterations before.  Rows and columns past the end re-read the last ones; rows past it are staged as zeros.
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  const int ap = XROWS ? 0 : tid % (BM / 8), ar = XROWS ? 0 : tid / (BM / 8), bp = tid % (BN / 8), br = tid / (BN / 8);
  const bf16_t* const abase = XROWS ? nullptr : g.A + min(m0 + 8 * ap, g.M - 8);
  const bf16_t* const bbase = g.B + min(n0 + 8 * bp, g.N - 8);
  u4 a0[XROWS ? 1 : QA], a1[XROWS ? 1 : QA], b0[QB], b1[QB];
  float x0[XROWS ? XJ : 1][XR], x1[XROWS ? XJ : 1][XR];
  // XROWS: lane i < XR holds the row order entry of row i of this wavefront's rows of the next chunk, requested a chunk ahead
  int32_t xentry = 0;
  auto row_at = [&](int c, int r) { return min(k_begin + (int64_t)c * KC + r, k_end - 1); };
  auto request_entry = [&](int c) {
    if (XROWS && g.X.gather != nullptr) xentry = g.X.gather_entry<true>(row_at(min(c, nchunks - 1), wave * XR + min(lane, XR - 1)));
  };
  auto fetch = [&](int i, auto set) {
    const int c = min(i, nchunks - 1);  // past the end: the last chunk again, never multiplied
    constexpr bool FIRST = decltype(set)::value == 0;
    if constexpr (XROWS) {
      const int64_t s = row_at(c, wave * XR + min(lane, XR - 1));
      const int64_t off = g.X.ptr_with<true>(s, xentry) - g.X.base;
#pragma unroll
      for (int r = 0; r < XR; ++r) {
        const uint32_t off_lo = __builtin_amdgcn_readlane((int)(uint32_t)off, r), off_hi = __builtin_amdgcn_readlane((int)(off >> 32), r);
        const float* const p = g.X.base + (int64_t)((uint64_t)off_hi << 32 | off_lo);
#pragma unroll
        for (int j = 0; j < XJ; ++j) {
          const float v = p[min(m0 + 64 * j + lane, g.M - 1)];
          if constexpr (FIRST) x0[j][r] = v;
          else x1[j][r] = v;
        }
      }
      request_entry(i + 1);
    } else {
#pragma unroll
      for (int q = 0; q < QA; ++q) {
        const u4 v = *reinterpret_cast<const u4*>(abase + row_at(c, ar + RA * q) * g.lda);
        if constexpr (FIRST) a0[q] = v;
        else a1[q] = v;
      }
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const u4 v = *reinterpret_cast<const u4*>(bbase + row_at(c, br + RB * q) * g.N);
      if constexpr (FIRST) b0[q] = v;
      else b1[q] = v;
    }
  };
  float bsum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto stage = [&](int buf, int c, auto set) {
    constexpr bool FIRST = decltype(set)::value == 0;
    bf16_t* const As = wgrad_lds + buf * STAGE;
    bf16_t* const Bs = As + KC * PA;
    const int64_t left = c < nchunks ? k_end - (k_begin + (int64_t)c * KC) : 0;  // live rows of the chunk
    const u4 zero = {0u, 0u, 0u, 0u};
    if constexpr (XROWS) {
#pragma unroll
      for (int r = 0; r < XR; ++r) {
        const int row = wave * XR + r;
#pragma unroll
        for (int j = 0; j < XJ; ++j) {
          const float v = FIRST ? x0[j][r] : x1[j][r];
          if (64 * j + 64 <= BM || lane < BM - 64 * j) As[row * PA + 64 * j + lane] = row < left ? to_bf16(v) : (bf16_t)0;
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < QA; ++q) *reinterpret_cast<u4*>(&As[(ar + RA * q) * PA + 8 * ap]) = ar + RA * q < left ? (FIRST ? a0[q] : a1[q]) : zero;
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const u4 v = br + RB * q < left ? (FIRST ? b0[q] : b1[q]) : zero;
      *reinterpret_cast<u4*>(&Bs[(br + RB * q) * PB + 8 * bp]) = v;
      if (tm == 0) {  // uniform
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          bsum[2 * e] += __uint_as_float(v[e] << 16);
          bsum[2 * e + 1] += __uint_as_float(v[e] & 0xffff0000u);
        }
      }
    }
  };
  const bool idle = n0 + 32 * NT * wn >= g.N || m0 + 32 * MT * wm >= g.M;  // uniform: this wavefront's part of the tile is padding
  auto multiply = [&](int buf) {
    if (idle) return;
    const bf16_t* const As = wgrad_lds + buf * STAGE + frag_col_offset(lane, PA) + 32 * MT * wm;
    const bf16_t* const Bs = wgrad_lds + buf * STAGE + KC * PA + frag_col_offset(lane, PB) + 32 * NT * wn;
#pragma unroll
    for (int ks = 0; ks < KC / 16; ++ks) {
      bf16x8 a[MT], b[NT];
#pragma unroll
      for (int i = 0; i < MT; ++i) a[i] = read_col8(As + 16 * ks * PA + 32 * i, PA);
#pragma unroll
      for (int j = 0; j < NT; ++j) b[j] = read_col8(Bs + 16 * ks * PB + 32 * j, PB);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = mfma32_bf16(a[i], b[j], acc[i][j]);
    }
  };
  using Set0 = std::integral_constant<int, 0>;
  using Set1 = std::integral_constant<int, 1>;
  request_entry(0);
  fetch(0, Set0{});
  fetch(1, Set1{});
  stage(0, 0, Set0{});
  fetch(2, Set0{});
#pragma unroll 1
  for (int i = 0; i < nchunks; i += 2) {  // chunks in pairs; one past the end is zeros
    __syncthreads();
    stage(1, i + 1, Set1{});
    fetch(i + 3, Set1{});
    multiply(0);
    __syncthreads();
    stage(0, i + 2, Set0{});
    fetch(i + 4, Set0{});
    multiply(1);
  }
  float* const out = g.out + (int64_t)z * ((int64_t)g.M * g.N + g.N);
  if (!idle) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const int n = n0 + 32 * (NT * wn + j) + lo;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m0 + 32 * (MT * wm + i) + 8 * (r / 4) + 4 * hi + (r % 4);
          if (m < g.M && n < g.N) out[(int64_t)m * g.N + n] = acc[i][j][r];
        }
      }
  }
  if (tm == 0) {  // uniform: the column sums, added over the threads that staged the same columns
    __syncthreads();
    float* const red = reinterpret_cast<float*>(wgrad_lds);  // [RB][BN]
    static_assert(RB * BN * 4 <= 2 * STAGE * 2, "room for the partial column sums");
#pragma unroll
    for (int e = 0; e < 8; ++e) red[br * BN + 8 * bp + e] = bsum[e];
    __syncthreads();
    for (int e = tid; e < BN; e += THREADS)
      if (n0 + e < g.N) {
        float v = 0.f;
#pragma unroll
        for (int r = 0; r < RB; ++r) v += red[r * BN + e];
        out[(int64_t)g.M * g.N + n0 + e] = v;
      }
  }
}

// Output tile and number of k ranges of a product of M x N outputs over S samples: one workgroup per CU.
struct Bf16WgradPlan {
  int bm, bn;
  unsigned tiles_m, tiles_n;
  int64_t per, splits;
};
inline Bf16WgradPlan bf16_wgrad_plan(bool xrows, int M, int N, int64_t S) {
  Bf16WgradPlan p;
  p.bn = N > 128 ? 256 : 128;
  p.bm = xrows ? (M <= 32 ? 32 : M <= 96 ? 96 : 160) : p.bn;
  p.tiles_m = (unsigned)((M + p.bm - 1) / p.bm);
  p.tiles_n = (unsigned)((N + p.bn - 1) / p.bn);
  const int64_t want = std::max<int64_t>(1, 256 / ((int64_t)p.tiles_m * p.tiles_n));
  p.per = std::max<int64_t>(256, round_up64((S + want - 1) / want));
  p.splits = (S + p.per - 1) / p.per;
  return p;
}
inline int64_t bf16_wgrad_floats(bool xrows, int M, int N, int64_t S) { return bf16_wgrad_plan(xrows, M, N, S).splits * ((int64_t)M * N + N); }

template <bool XROWS, int MT, int NT, int WM, int WN>
inline int32_t launch_bf16_wgrad_inst(const Bf16WgradArgs& g, int64_t splits, hipStream_t s) {
  auto kern = bf16_wgrad_kernel<XROWS, MT, NT, WM, WN>;
  const size_t bytes = sizeof(bf16_t) * 2 * kWgradChunk * (wgrad_pitch(32 * MT * WM) + wgrad_pitch(32 * NT * WN));
  if (bytes > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
    return MARL_E_LAUNCH;
  hipLaunchKernelGGL(kern, dim3((unsigned)(g.tiles_m * g.tiles_n * splits)), dim3(64 * WM * WN), bytes, s, g);
  return launch_status();
}
// gW [M][N] += A^T B, the column sums of B behind it; A: the fp32 rows X (xrows) or bf16 [S][lda]
inline int32_t launch_bf16_wgrad(bool xrows, Bf16WgradArgs g, float* gW, hipStream_t s) {
  const Bf16WgradPlan p = bf16_wgrad_plan(xrows, g.M, g.N, g.S);
  g.tiles_m = p.tiles_m; g.tiles_n = p.tiles_n; g.per = p.per;
  int32_t rc;
  {
    TimedLaunch timed(KC_GEMM_TN, 2.0 * (double)g.S * g.M * g.N, s);
    if (xrows) {
      if (p.bn == 256) rc = p.bm == 32 ? launch_bf16_wgrad_inst<true, 1, 1, 1, 8>(g, p.splits, s)
                          : p.bm == 96 ? launch_bf16_wgrad_inst<true, 3, 1, 1, 8>(g, p.splits, s) : launch_bf16_wgrad_inst<true, 5, 1, 1, 8>(g, p.splits, s);
      else rc = p.bm == 32 ? launch_bf16_wgrad_inst<true, 1, 1, 1, 4>(g, p.splits, s)
              : p.bm == 96 ? launch_bf16_wgrad_inst<true, 3, 1, 1, 4>(g, p.splits, s) : launch_bf16_wgrad_inst<true, 5, 1, 1, 4>(g, p.splits, s);
    } else {
      rc = p.bn == 256 ? launch_bf16_wgrad_inst<false, 4, 2, 2, 4>(g, p.splits, s) : launch_bf16_wgrad_inst<false, 2, 1, 2, 4>(g, p.splits, s);
    }
  }
  if (rc == MARL_OK) launch_reduce_partials(g.out, (int)p.splits, (int64_t)g.M * g.N + g.N, gW, s);
  return rc;
}

}  // namespace marl
