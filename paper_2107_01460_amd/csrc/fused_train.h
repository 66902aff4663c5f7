// Whole-network training pass for the small networks (hidden width 64 or 128, input width <= 93):
// forward, PPO loss, and the complete backward pass of one network in ONE kernel.  Nothing but the
// observations and a few scalars per sample is read from HBM and nothing but the parameter gradient is
// written: h1, h2, dz2, dz1 live in LDS / registers for the lifetime of a row tile, and the weight
// gradients are accumulated in registers over all row tiles a workgroup owns.
//
// Workgroup = a wavefront per 32 units, persistent; row tile = 32 samples; two (128 units) or four (64) workgroups share a CU,
// whose phases cover one another: what one splits or waits for, another multiplies.  Products are taken transposed (units x
// samples), so that a lane holds runs of four units of one sample: an epilogue splits its values ONCE and stores them as 8-byte
// pieces of three bf16 planes in LDS (split_bf16.h), which every product afterwards reads as operands, by rows or, for the weight
// gradients, through the transposing read.  Weights stream from the L2 in one sequence of k steps that runs on from layer to layer
// and from tile to tile.  Per tile, a barrier where | stands:
//   layer 1 -> h1 (A) | layer 2 -> h2 (registers, B), output layer | loss -> dL/dout | W3 gradient, dz2 = (dL/dout W3^T)(1 - h2^2) -> B |
//   dW2 += h1^T dz2, dz1 = (dz2 W2^T)(1 - h1^2), the next tile's X to LDS | dz1 -> A, dW1 += X^T dz1
// A wavefront's share of dW1 needs no dz1 but its own.  The tiles' rows have no padding; a row's 16-byte units are permuted
// (tile_swizzle) so that both ways of reading a plane meet every bank once.  (The epilogues' 8-byte stores do not: rows sixteen apart share
// their places.  Bank conflicts are 7-8 % of the cycles at 128 units, 10-12 % at 64.)
// Exact inputs: windows hold small integers and halves, whose lower split parts are zero.  X is then one plane and its products three
// instead of six; the first tile with any other value, and all behind it, go through a second form of the loop, which splits X into three
// planes once per tile (16 minibatches of 98 304 samples of 75 inputs, both networks of 64 units: 1.97 ms, in the second form 2.18; of 128
// units 3.47 and 3.79.  With X staged twice a tile in blocks of 32 columns, each waited for: 2.87 and 4.18).
// At the end a workgroup stores its partial gradient into a copy of its own, every sum in a fixed
// order; reduce_partials_kernel adds the copies.
// Against one workgroup of eight wavefronts per CU that split activations where it read them (MI355X): 1 048 576 samples of 75 inputs,
// 128 units, 6 outputs 1200 -> 890 us (161 TFLOP/s of fp32 products); 98 304 samples 141 -> 100 us; 2 097 152 of 27 inputs, 64 units 765 ->
// 640 us.  Bound: the chain of a tile's phases.  Matrix cores are busy 41-46 % of the cycles at 128 units and 33 % at 64, vector
// instructions 42 and 54 %; a wavefront waits a third of its time for barriers, LDS and memory and as long for an issue slot.  All
// weights from the L1 instead of the L2 would save 5 % of a training iteration.  At 128 units and 96 inputs all 256 registers are in use;
// a form with 77 of them spilled in the tile loop took a fifth longer.  64-row tiles leave room for one workgroup per CU only.
#pragma once
#include "gemm.h"

namespace marl {

struct FusedTrainArgs {
  RowSrc X;  // S rows of Din floats (gathered)
  int64_t S;
  int Din, Kp;     // Kp: rows of the staged W1, Din rounded up to a multiple of 32
  const float* W;  // split operand-order copies of W1, W2 and W2 transposed, one directly behind the other (ParamMap)
  const float *b1, *b2, *W3, *b3;
  float* grad;     // the network's gradient: W1, b1, W2, b2, W3, b3, `gcount` floats
  float* stats;    // five loss statistics
  // Workgroup b writes its sums into its own copy of the gradient at partial + b * pstride and the statistics of `stats_mask` into
  // the five floats at partial + b * pstride + stats_at; reduce_partials_kernel adds the copies to `grad` and `stats`.
  // (Several hundred workgroups adding to the same few hundred cache lines at the same moment cost 60-180 us per launch.)
  float* partial;
  int64_t gcount, pstride, stats_at;
  unsigned stats_mask;
};

constexpr int kFusedTile = 32;  // samples of a tile

// bf16 elements of LDS for two tiles of exact inputs and the wavefronts' shares of the outputs, or for one tile of any inputs in three
// planes, the third of which begins where the outputs do.
constexpr size_t fused_train_x_region(int H, int DMAX) {
  const size_t exact = 2 * 32 * DMAX + 2 * (H / 32) * 32 * 8, planes = 3 * 32 * DMAX;
  return exact > planes ? exact : planes;
}
// Bytes of LDS (with DMAX columns of X).  Two workgroups of 128 units, four of 64 units and 32 inputs, three of 64 units and 96
// inputs fit a CU's 160 KB.
constexpr size_t fused_train_lds(int H, int NOUT, int DMAX) {
  return sizeof(bf16_t) * (2 * 3 * 32 * H + fused_train_x_region(H, DMAX) + 24 * (H + 8) + 24 * 40) +
         sizeof(float) * (2 * H + H * NOUT + 32 * (NOUT + 5) + 12);
}
static_assert(2 * fused_train_lds(128, 6, 96) <= 160 * 1024 && 4 * fused_train_lds(64, 6, 32) <= 160 * 1024 && 3 * fused_train_lds(64, 6, 96) <= 160 * 1024,
              "workgroups per CU");

// Where the 16-byte unit u of row r of a tile with H elements a row (H = 32: blocks of X) stands: at unit u ^ tile_swizzle(r).
// Sixteen rows of one unit (row reads) and four units of four rows (transposing reads) then lie in 64 different banks each.
template <int H>
__device__ __forceinline__ int tile_swizzle(int r) {
  const int low = (r >> 2) & 3;
  return H == 128 ? (r & 3) << 2 | low : H == 64 ? (r & 2) << 1 | low : low;
}

// c + the sum of eight values.  The dot instruction cuts its addends off below the last bit of the largest: first parts of a split are
// summed by themselves (8 bits each, so that nothing is lost unless they are 2^16 apart), and the other parts by themselves.  All
// three on one running sum over the tiles lost what a tile has to add where it is small against that sum.
__device__ __forceinline__ float sum8(bf16x8 v, float c) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
  c = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(v, v, 0, 1), one, c, false);
  c = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(v, v, 2, 3), one, c, false);
  c = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(v, v, 4, 5), one, c, false);
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(v, v, 6, 7), one, c, false);
}

// The kernel's body: workgroup `bid` of `nblk` that share the tiles of one network's minibatch.
template <int H, int NOUT, int DMAX, class LossFn>
__device__ __forceinline__ void fused_train_body(const FusedTrainArgs& a, const LossFn& fn, const unsigned bid, const unsigned nblk) {
  constexpr int BM = kFusedTile, NW = H / 32, THREADS = 64 * NW, PLANE = BM * H, Q1 = DMAX / 32, XBUF = BM * DMAX;
  constexpr int XR = 8 / NW;                            // rows of X a lane stages of each 32-column block
  constexpr int P3 = H + 8, PLANE3 = 8 * P3, PD = BM + 8, AS = NOUT + 5, RING = 2;
  // The next tile's rows are requested behind layer 2 or, where their registers would be spilled, behind dW2 (64 units, 27 inputs: 4 %
  // longer behind dW2; 128 units, 75 inputs: a fifth longer behind layer 2).
  constexpr bool X_EARLY = H == 64;
  constexpr int TI = NW == 4 ? 2 : 1, TJ = 2;           // dW2: a wavefront's block of 32 x 32 tiles
  static_assert((H == 64 || H == 128) && (DMAX == 32 || DMAX == 96), "tile shapes");
  extern __shared__ __attribute__((aligned(16))) bf16_t fused_lds[];
  bf16_t* const tA = fused_lds;                         // [3][BM][H] h1, later dz1
  bf16_t* const tB = tA + 3 * PLANE;                    // [3][BM][H] h2, later dz2
  bf16_t* const xs = tB + 3 * PLANE;                    // exact: [2][Q1][BM][32], one tile and the next; else [3][Q1][BM][32]
  float* const outp = reinterpret_cast<float*>(xs + 2 * XBUF);   // [NW][BM][8] every wavefront's share of the outputs; then the first as
  float* const dls = outp;                              // [BM][8] dL/d(output), zeros past NOUT
  bf16_t* const w3t = xs + fused_train_x_region(H, DMAX);        // [3][8][P3] W3 transposed, split, rows past NOUT zero
  bf16_t* const dlt = w3t + 3 * PLANE3;                 // [3][8][PD] dL/d(output), split and transposed
  float* const bias = reinterpret_cast<float*>(dlt + 24 * PD);  // [2][H]
  float* const w3s = bias + 2 * H;                      // [H][NOUT]
  float* const accS = w3s + H * NOUT;                   // [BM][AS] per sample slot: b3 gradient, loss statistics
  float* const b3s = accS + BM * AS;                    // [8]
  typedef decltype(fn.prepare()) Prep;                  // two floats
  Prep* const prep = reinterpret_cast<Prep*>(b3s + 8);
  int* const inexact = reinterpret_cast<int*>(b3s + 10);

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int lane = tid & 63;
  GroupCopy<H * NOUT, THREADS> w3;
  GroupCopy<H, THREADS> b1, b2;
  w3.request(tid, a.W3);
  b1.request(tid, a.b1);
  b2.request(tid, a.b2);
  const float b3 = a.b3[min(tid, NOUT - 1)];

  // ---- weights: k step `nxt` of the sequence layer 1, layer 2, dz1, and again for the next tile
  const int steps1 = a.Kp / 16, total = steps1 + 2 * (H / 16);
  const WeightRsrc wsrc = weight_rsrc(a.W, total * 16 * H * 3 / 2);
  const int woff = ((lane >> 5) * H + 32 * wave + (lane & 31)) * 16;
  bf16x8 w[RING][3];
  int nxt = 0;
  auto load_w = [&](int slot) {
#pragma unroll
    for (int p = 0; p < 3; ++p) w[slot][p] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wsrc, woff, (nxt * 3 + p) * 32 * H, 0));
    nxt = nxt + 1 == total ? 0 : nxt + 1;
  };
#pragma unroll
  for (int u = 0; u < RING; ++u) load_w(u);

  if (tid == 0) {
    *inexact = 0;
    *prep = fn.prepare();
  }
  for (int e = tid; e < 24 * PD; e += THREADS) dlt[e] = 0;
  for (int e = tid; e < BM * AS; e += THREADS) accS[e] = 0.f;
  for (int e = tid; e < (8 - NOUT) * H; e += THREADS) w3t[(NOUT + e / H) * P3 + e % H] = w3t[PLANE3 + (NOUT + e / H) * P3 + e % H] = w3t[2 * PLANE3 + (NOUT + e / H) * P3 + e % H] = 0;
  w3.store(tid, [&](int e, float v) {
    const int u = e / NOUT, k = e % NOUT;
    const SplitPair s = split_pair_any(v, 0.f);
    w3t[k * P3 + u] = (bf16_t)s.h;
    w3t[PLANE3 + k * P3 + u] = (bf16_t)s.m;
    w3t[2 * PLANE3 + k * P3 + u] = (bf16_t)s.l;
    w3s[e] = v;
  });
  b1.store(tid, [&](int e, float v) { bias[e] = v; });
  b2.store(tid, [&](int e, float v) { bias[H + e] = v; });
  if (tid < NOUT) b3s[tid] = b3;

  // dW2: this wavefront's block of tiles; of its two columns, the one whose sums (the b2 gradient) it takes
  const int it0 = NW == 4 ? 2 * (wave >> 1) : wave, jt0 = NW == 4 ? 2 * (wave & 1) : 0, gb2_j = NW == 4 ? wave >> 1 : wave;
  const int loss_wave = (bid >> 8) % NW;  // (workgroups 256 apart share a CU: another SIMD for each)
  floatx16 acc1[Q1], acc2[TI * TJ];  // dW1 / dW2 tiles of this wavefront, persistent
  floatx16 acc, h1, h2;              // a product; this wavefront's units of the samples (element r: unit 8 (r / 4) + 4 hi + r % 4, sample lo)
  typedef float f4 __attribute__((ext_vector_type(4)));
  f4 gw[2];                          // W3 gradient: units 32 wave + 16 u + 4 (lane / 16) + r, output lane % 16
  // b1 gradient of unit 32 wave + lo, b2 gradient of unit 32 (jt0 + gb2_j) + lo: samples 8 hi .. 8 hi + 7 of every sixteen (one register
  // each; a sum per sample slot takes sixteen), a tile's sum added at once
  float gb1 = 0.f, gb2 = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
#pragma unroll
    for (int q = 0; q < Q1; ++q) acc1[q][r] = 0.f;
#pragma unroll
    for (int q = 0; q < TI * TJ; ++q) acc2[q][r] = 0.f;
  }
  gw[0] = gw[1] = f4{0.f, 0.f, 0.f, 0.f};

  const int64_t ntiles = (a.S + BM - 1) / BM;
  int64_t t = bid;
  int lo, hi, l15, l4;
  auto lane_parts = [&]() {
    asm volatile("" : "+v"(lane));  // what depends on the lane is formed anew: kept, the many addresses were spilled
    lo = lane & 31; hi = lane >> 5; l15 = lane & 15; l4 = lane >> 4;
  };
  lane_parts();
  const auto zero_acc = [&]() {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  };
  // acc += weights x tile over `steps` (even) k steps.  X32: the tile is made of 32-column blocks; ONE: of one plane, whose values are
  // exact.  The products of the parts in mfma_split's order.  The scheduling barriers keep the requests where they are written.
  auto product = [&](const bf16_t* tile, int plane, int steps, auto x32, auto one) {
    constexpr bool X32 = decltype(x32)::value, ONE = decltype(one)::value;
    constexpr int PITCH = X32 ? 32 : H;
    // (a row's units stand within an aligned block of its size: the step is an exclusive or on the offset)
    const int off0 = (int)(tile - fused_lds) + lo * PITCH + ((hi ^ tile_swizzle<PITCH>(lo)) << 3);
    Split8 x[2];
    auto read = [&](int step) {
      const bf16_t* const p = fused_lds + (X32 ? (step >> 1) * (BM * 32) + (off0 ^ (step & 1) << 4) : off0 ^ step << 4);
      if (!ONE) return frag_row(p, plane);
      Split8 f;
      f.h = *reinterpret_cast<const bf16x8*>(p);
      return f;
    };
    x[0] = read(0);
#pragma unroll 1
    for (int s0 = 0; s0 < steps; s0 += RING) {
#pragma unroll
      for (int u = 0; u < RING; ++u) {
        x[(u + 1) & 1] = read(min(s0 + u + 1, steps - 1));
        __builtin_amdgcn_sched_barrier(0);
        const Split8 wv{w[u][0], w[u][1], w[u][2]};
        if constexpr (ONE) {
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv.l, x[u & 1].h, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv.m, x[u & 1].h, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv.h, x[u & 1].h, acc, 0, 0, 0);
        } else {
          acc = mfma_split(wv, x[u & 1], acc);
        }
        load_w(u);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // Operand of a weight gradient: 32 columns (block ct) of a tile over the samples kb .. kb + 15.
  auto col8 = [&](const bf16_t* tile, auto pitch, int ct, int kb) {
    constexpr int PITCH = decltype(pitch)::value;
    typedef __attribute__((address_space(3))) shortx4 lds_shortx4;
    const int r = 8 * hi + (l15 >> 2), sw = (2 * (l4 & 1) + ((lane >> 1) & 1)) ^ tile_swizzle<PITCH>(r);
    const bf16_t* const p = tile + (kb + r) * PITCH + 4 * (lane & 1);
    const shortx4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)(p + ((sw ^ (4 * ct)) << 3)));
    const shortx4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)(p + 4 * PITCH + ((sw ^ (4 * ct) ^ 1) << 3)));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  typedef std::integral_constant<int, H> TileP;
  typedef std::integral_constant<int, 32> BlockP;
  auto col_split = [&](const bf16_t* tile, int plane, auto pitch, int ct, int kb) {
    return Split8{col8(tile, pitch, ct, kb), col8(tile + plane, pitch, ct, kb), col8(tile + 2 * plane, pitch, ct, kb)};
  };
  // four units of this lane's sample into a tile's three planes
  auto store4 = [&](bf16_t* tile, int g4, float4 v, bool wild) {
    bf16_t* const d = tile + lo * H + (((4 * wave + g4) ^ tile_swizzle<H>(lo)) << 3) + 4 * hi;
    if (__builtin_expect(wild, 0)) store_split4<true>(d, PLANE, v);
    else store_split4<false>(d, PLANE, v);
  };
  auto tanh_out = [&](bf16_t* tile, const float* b, floatx16& keep) {
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const float4 bq = *reinterpret_cast<const float4*>(&b[32 * wave + 8 * g4 + 4 * hi]);
      const float bb[4] = {bq.x, bq.y, bq.z, bq.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) keep[4 * g4 + j] = tanh_f32(acc[4 * g4 + j] + bb[j]);
      store4(tile, g4, make_float4(keep[4 * g4], keep[4 * g4 + 1], keep[4 * g4 + 2], keep[4 * g4 + 3]), false);
    }
  };
  auto store_gradient = [&](bf16_t* tile, const floatx16& v) {
    float top = 0.f;  // (a NaN stays one: split with its neighbour it would reach that unit's weight gradient)
#pragma unroll
    for (int r = 0; r < 16; ++r) top = __builtin_elementwise_maximum(top, fabsf(v[r]));
    const bool wild = __builtin_amdgcn_ballot_w64(!(top < kSplitLimit)) != 0;
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) store4(tile, g4, make_float4(v[4 * g4], v[4 * g4 + 1], v[4 * g4 + 2], v[4 * g4 + 3]), wild);
  };

  // ---- input rows: a quarter of a wavefront a row, a lane two neighbouring columns of a 32-column block: rows 4 (wave + NW i) + l4,
  // columns 32 q + 2 l15, + 1.  Rows past the last sample: the last one again, with a zero gradient.
  typedef float f2 __attribute__((ext_vector_type(2), aligned(4)));  // rows start at any 4-byte boundary
  int32_t xentry[XR];
  f2 xr[Q1][XR];
  auto x_row = [&](int i) { return 4 * (wave + NW * i) + l4; };
  auto fetch_entries = [&](int64_t tile) {
#pragma unroll
    for (int i = 0; i < XR; ++i) xentry[i] = a.X.template gather_entry<true>(min(tile * BM + x_row(i), a.S - 1));
  };
  // (32-bit products: the general address of RowSrc was a tenth of the tile's vector instructions)
  const uint32_t row_floats = (uint32_t)a.X.ld, entry_floats = (uint32_t)(a.X.per * a.X.ld);
  auto x_ptr = [&](int64_t tile, int i) {
    const uint32_t smp = (uint32_t)min(tile * BM + x_row(i), a.S - 1);
    const uint32_t agent = smp - (uint32_t)a.X.pd.template div<true>(smp, a.X.per) * (uint32_t)a.X.per;
    return a.X.base + ((uint64_t)(uint32_t)xentry[i] * entry_floats + agent * row_floats);
  };
  auto x_col = [&](int q) { return min(32 * q + 2 * l15, a.Din - 2); };
  auto request_x = [&](int64_t tile) {
#pragma unroll
    for (int i = 0; i < XR; ++i) {
      const float* const row = x_ptr(min(tile, ntiles - 1), i);
#pragma unroll
      for (int q = 0; q < Q1; ++q) xr[q][i] = *reinterpret_cast<const f2*>(row + x_col(q));
    }
  };
  auto fix_x = [&](int i, int q) {
    const int c = 32 * q + 2 * l15;
    const f2 v = xr[q][i];
    xr[q][i].x = c >= a.Din ? 0.f : c == a.Din - 1 ? v.y : v.x;
    xr[q][i].y = c + 1 < a.Din ? v.y : 0.f;
  };
  auto x_slot = [&](int i) { return x_row(i) * 32 + (((l15 >> 2) ^ tile_swizzle<32>(x_row(i))) << 3) + 2 * (l15 & 3); };
  // the rows to one plane; are they all exact?
  auto store_x = [&](bf16_t* dst) {
    uint32_t low_bits = 0;
    float top = 0.f;
#pragma unroll
    for (int q = 0; q < Q1; ++q)
#pragma unroll
      for (int i = 0; i < XR; ++i) {
        fix_x(i, q);
        low_bits |= __float_as_uint(xr[q][i].x) | __float_as_uint(xr[q][i].y);
        top = fmaxf(fmaxf(top, fabsf(xr[q][i].x)), fabsf(xr[q][i].y));
        *reinterpret_cast<uint32_t*>(dst + q * (BM * 32) + x_slot(i)) = __float_as_uint(xr[q][i].x) >> 16 | (__float_as_uint(xr[q][i].y) & 0xffff0000u);
      }
    if (__builtin_amdgcn_ballot_w64((low_bits & 0xffffu) != 0 || __builtin_isinf(top)) != 0) *inexact = 1;
  };
  // The rows, split, to three planes (general form of the loop).  The outputs overwrite the third plane's first KEEP blocks, whose pieces
  // stay in registers.
  constexpr int KEEP = NW / 2 < Q1 ? NW / 2 : Q1;
  static_assert(NW * BM * 8 * 2 <= KEEP * BM * 32 || KEEP == Q1, "blocks under the outputs");
  uint32_t low[KEEP][XR];
  auto put_x = [&](auto any) {
#pragma unroll
    for (int q = 0; q < Q1; ++q)
#pragma unroll
      for (int i = 0; i < XR; ++i) {
        const SplitPair s = split_two<decltype(any)::value>(xr[q][i].x, xr[q][i].y);
        uint32_t* const d = reinterpret_cast<uint32_t*>(xs + q * (BM * 32) + x_slot(i));
        d[0] = s.h;
        d[XBUF / 2] = s.m;
        d[XBUF] = s.l;
        if (q < KEEP) low[q < KEEP ? q : 0][i] = s.l;
      }
  };
  auto split_x = [&]() {
    float top = 0.f;
#pragma unroll
    for (int q = 0; q < Q1; ++q)
#pragma unroll
      for (int i = 0; i < XR; ++i) {
        fix_x(i, q);
        top = __builtin_elementwise_maximum(top, __builtin_elementwise_maximum(fabsf(xr[q][i].x), fabsf(xr[q][i].y)));
      }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(top < kSplitLimit)) != 0, 0)) put_x(std::true_type{});
    else put_x(std::false_type{});
  };
  auto put_low = [&]() {
#pragma unroll
    for (int q = 0; q < KEEP; ++q)
#pragma unroll
      for (int i = 0; i < XR; ++i) reinterpret_cast<uint32_t*>(xs + 2 * XBUF + q * (BM * 32) + x_slot(i))[0] = low[q][i];
  };

  // All tiles from t on, or (EXACT) up to the first whose inputs are not exact.
  auto train_tiles = [&](auto exact) {
    constexpr bool EXACT = decltype(exact)::value;
    if (!EXACT) {  // (store_x has set what is past a row's end)
      fetch_entries(t);
      request_x(t);
    }
    for (int it = 0; t < ntiles; t += nblk, ++it) {
      if (EXACT && __builtin_amdgcn_readfirstlane(*inexact) != 0) break;
      lane_parts();
      const int64_t s0 = t * BM;
      const bool more = t + nblk < ntiles;  // uniform
      bf16_t* const X = EXACT ? xs + (it & 1) * XBUF : xs;
      const int64_t smp = s0 + lo;  // the sample whose loss a lane of the wavefront `loss_wave` takes
      int32_t lentry = 0;
      if (wave == loss_wave) lentry = fn.template row_entry<true>(min(smp, a.S - 1));
      fetch_entries(min(t + nblk, ntiles - 1));
      // ---- layer 1
      if constexpr (!EXACT) {
        __syncthreads();  // the last tile's X has been read
        split_x();
        __syncthreads();
      }
      zero_acc();
      if constexpr (EXACT) {
        product(X, 0, steps1, std::true_type{}, std::true_type{});
      } else {
        product(X, XBUF, steps1, std::true_type{}, std::false_type{});
      }
      tanh_out(tA, bias, h1);
      __syncthreads();
      // ---- layer 2
      zero_acc();
      product(tA, PLANE, H / 16, std::false_type{}, std::false_type{});
      typename LossFn::In lin;
      if (wave == loss_wave) lin = fn.template load_with<true>(min(smp, a.S - 1), lentry);
      if (X_EARLY) request_x(t + nblk);
      tanh_out(tB, bias + H, h2);
      // ---- output layer: W3^T x h2 over this wavefront's units for sixteen samples at a time; outputs 0 .. 3 land in lanes 0 .. 15,
      // 4 .. 7 in the next sixteen
      {
        const Split8 wv = frag_row(&w3t[(lane & 7) * P3 + 32 * wave + 8 * l4], PLANE3);
        Split8 xv[2];
        f4 o[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int g = 0; g < 2; ++g) xv[g] = frag_row(&tB[(16 * g + l15) * H + (((4 * wave + l4) ^ tile_swizzle<H>(l15)) << 3)], PLANE);
#define MARL_OUT(WP, XP) \
  _Pragma("unroll") for (int g = 0; g < 2; ++g) o[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv.WP, xv[g].XP, o[g], 0, 0, 0);
        MARL_OUT(h, l)
        MARL_OUT(l, h)
        MARL_OUT(m, m)
        MARL_OUT(h, m)
        MARL_OUT(m, h)
        MARL_OUT(h, h)
#undef MARL_OUT
        if (lane < (NOUT > 4 ? 32 : 16)) {
#pragma unroll
          for (int g = 0; g < 2; ++g) *reinterpret_cast<f4*>(&outp[(wave * BM + 16 * g + l15) * 8 + 4 * l4]) = o[g];
        }
      }
      __syncthreads();
      if (wave == loss_wave && lane < BM) {
        float out[NOUT], dl[NOUT], st[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < NOUT; ++k) {
          out[k] = b3s[k];
          dl[k] = 0.f;
        }
#pragma unroll
        for (int z = 0; z < NW; ++z)
#pragma unroll
          for (int k = 0; k < NOUT; ++k) out[k] += outp[(z * BM + lo) * 8 + k];
        if (smp < a.S) fn.compute(lin, *prep, out, dl, st);
#pragma unroll
        for (int k = 0; k < NOUT; ++k) {
          accS[lo * AS + k] += dl[k];
          const SplitPair sp = split_pair_any(dl[k], 0.f);
          dlt[k * PD + lo] = (bf16_t)sp.h;
          dlt[(8 + k) * PD + lo] = (bf16_t)sp.m;
          dlt[(16 + k) * PD + lo] = (bf16_t)sp.l;
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) accS[lo * AS + NOUT + k] += st[k];
#pragma unroll
        for (int k = 0; k < 8; k += 4)
          *reinterpret_cast<float4*>(&dls[lo * 8 + k]) = make_float4(k < NOUT ? dl[k < NOUT ? k : 0] : 0.f, k + 1 < NOUT ? dl[k + 1 < NOUT ? k + 1 : 0] : 0.f,
                                                                     k + 2 < NOUT ? dl[k + 2 < NOUT ? k + 2 : 0] : 0.f, k + 3 < NOUT ? dl[k + 3 < NOUT ? k + 3 : 0] : 0.f);
      }
      __syncthreads();
      // From here to the next barrier a wavefront reads and writes nothing of B but its own columns.
      // ---- W3 gradient: h2^T x dl, a tile's sum by itself and then one fp32 addition.  (A matrix instruction cuts its addends off below
      // the last bit of the largest, always downwards: with gw as the accumulator the error grew with the number of tiles, 2.0e-6 with
      // 128 and 3.6e-6 with 256 tiles per workgroup, against 8e-8 now; no difference in time.)
      {
        const Split8 d = frag_row(&dlt[(lane & 7) * PD + 8 * l4], 8 * PD);
        const int r = 8 * l4 + (l15 >> 2), sw = (4 * wave + ((lane >> 1) & 1)) ^ tile_swizzle<H>(r);
        typedef __attribute__((address_space(3))) shortx4 lds_shortx4;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          auto part = [&](const bf16_t* tile) {
            const bf16_t* const p = tile + r * H + 4 * (lane & 1);
            const shortx4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)(p + ((sw ^ (2 * u)) << 3)));
            const shortx4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)(p + 4 * H + ((sw ^ (2 * u) ^ 1) << 3)));
            return __builtin_bit_cast(bf16x8, __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7));
          };
          const Split8 h{part(tB), part(tB + PLANE), part(tB + 2 * PLANE)};
          f4 small = {0.f, 0.f, 0.f, 0.f}, top = small;
          small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h.l, d.h, small, 0, 0, 0);
          small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h.h, d.l, small, 0, 0, 0);
          small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h.m, d.m, small, 0, 0, 0);
          small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h.m, d.h, small, 0, 0, 0);
          small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h.h, d.m, small, 0, 0, 0);
          top = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h.h, d.h, top, 0, 0, 0);
          gw[u] += small + top;
          asm volatile("" : "+v"(gw[u]));  // (its addition stays here: moved, it cost 22 spilled registers at 128 units and 96 inputs)
        }
      }
      // ---- dz2 = (W3 dl) (1 - h2^2) over h2; the rank-NOUT product on the fp32 instruction, k = 4 hi + j
      {
        const float4 dv = *reinterpret_cast<const float4*>(&dls[lo * 8 + 4 * hi]);
        const float df[4] = {dv.x, dv.y, dv.z, dv.w};
        zero_acc();
#pragma unroll
        for (int j = 0; j < (NOUT < 4 ? NOUT : 4); ++j) {
          const float wf = 4 * hi + j < NOUT ? w3s[(32 * wave + lo) * NOUT + (4 * hi + j < NOUT ? 4 * hi + j : 0)] : 0.f;
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf, df[j], acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          acc[r] *= 1.0f - h2[r] * h2[r];
        }
        store_gradient(tB, acc);
      }
      __syncthreads();
      // ---- dW2 += h1^T dz2
      float b2h = 0.f, b2m = 0.f;
#pragma unroll
      for (int kb = 0; kb < BM; kb += 16) {
        Split8 x[TI];
#pragma unroll
        for (int i = 0; i < TI; ++i) x[i] = col_split(tA, PLANE, TileP{}, it0 + i, kb);
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
          const Split8 y = col_split(tB, PLANE, TileP{}, jt0 + j, kb);
          if (j == gb2_j) {  // uniform
            b2h = sum8(y.h, b2h);
            b2m = sum8(y.m, sum8(y.l, b2m));
          }
#pragma unroll
          for (int i = 0; i < TI; ++i) acc2[i * TJ + j] = mfma_split(x[i], y, acc2[i * TJ + j]);
        }
      }
      gb2 += b2h + b2m;
      if (!X_EARLY) request_x(t + nblk);
      // ---- dz1 = (W2 dz2^T) (1 - h1^2) over h1
      zero_acc();
      product(tB, PLANE, H / 16, std::false_type{}, std::false_type{});
      if (!EXACT) put_low();
      else if (more) store_x(xs + ((it & 1) ^ 1) * XBUF);  // the next tile's inputs
      __syncthreads();  // h1 has been read
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] *= 1.0f - h1[r] * h1[r];
      store_gradient(tA, acc);
      // ---- dW1 += X^T dz1: all blocks of X, this wavefront's columns of dz1
      float b1h = 0.f, b1m = 0.f;
#pragma unroll
      for (int kb = 0; kb < BM; kb += 16) {
        const Split8 y = col_split(tA, PLANE, TileP{}, wave, kb);
        b1h = sum8(y.h, b1h);
        b1m = sum8(y.m, sum8(y.l, b1m));
        if constexpr (EXACT) {
          bf16x8 x[Q1];
#pragma unroll
          for (int q = 0; q < Q1; ++q) x[q] = col8(X + q * (BM * 32), BlockP{}, 0, kb);
#pragma unroll
          for (int q = 0; q < Q1; ++q) acc1[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[q], y.l, acc1[q], 0, 0, 0);
#pragma unroll
          for (int q = 0; q < Q1; ++q) acc1[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[q], y.m, acc1[q], 0, 0, 0);
#pragma unroll
          for (int q = 0; q < Q1; ++q) acc1[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[q], y.h, acc1[q], 0, 0, 0);
        } else {
#pragma unroll
          for (int q = 0; q < Q1; ++q) acc1[q] = mfma_split(col_split(X + q * (BM * 32), XBUF, BlockP{}, 0, kb), y, acc1[q]);
        }
      }
      gb1 += b1h + b1m;
    }
  };
  if (t < ntiles) {
    fetch_entries(t);
    request_x(t);
  }
  __syncthreads();  // what was set up above, *inexact first of all
  if (t < ntiles) store_x(xs);
  __syncthreads();
  train_tiles(std::true_type{});
  if (__builtin_expect(t < ntiles, 0)) train_tiles(std::false_type{});

  // ---- this workgroup's sums to its copy of the gradient
  lane_parts();
  __syncthreads();  // accS
  float* const gW1 = a.partial + (int64_t)bid * a.pstride;
  float* const gb1o = gW1 + a.Din * H;
  float* const gW2 = gb1o + H;
  float* const gb2o = gW2 + H * H;
  float* const gW3 = gb2o + H;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = 8 * (r / 4) + 4 * hi + (r % 4);
#pragma unroll
    for (int q = 0; q < TI * TJ; ++q) gW2[(32 * (it0 + q / TJ) + row) * H + 32 * (jt0 + q % TJ) + lo] = acc2[q][r];
#pragma unroll
    for (int q = 0; q < Q1; ++q) {
      const int d = 32 * q + row;
      if (d < a.Din) gW1[d * H + 32 * wave + lo] = acc1[q][r];
    }
  }
  gb1 += __shfl_xor(gb1, 32);
  if (hi == 0) gb1o[32 * wave + lo] = gb1;
  gb2 += __shfl_xor(gb2, 32);
  if (hi == 0) gb2o[32 * (jt0 + gb2_j) + lo] = gb2;
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (l15 < NOUT) gW3[(32 * wave + 16 * u + 4 * l4 + r) * NOUT + l15] = gw[u][r];
  if (tid < AS) {
    double v = accS[tid];
    for (int s = 1; s < BM; ++s) v += accS[s * AS + tid];
    if (tid < NOUT) gW3[H * NOUT + tid] = v;
    else if (a.stats_mask >> (tid - NOUT) & 1) gW1[a.stats_at + tid - NOUT] = v;
  }
}

template <int H, int NOUT, int DMAX, class LossFn>
__global__ void __launch_bounds__(2 * H, 2) fused_train_kernel(FusedTrainArgs a, LossFn fn) {
  fused_train_body<H, NOUT, DMAX>(a, fn, blockIdx.x, gridDim.x);
}

// Two networks of the same shape on the same number of samples in ONE launch: workgroups 0 .. grid_a - 1 train the
// first, the others the second.  For minibatches so small that neither launch fills the compute units (a few tiles
// each) the update is a chain of dependent launches, and this takes two links (a kernel and its reduction) out of it.
template <int H, int NOUT_A, int NOUT_B, int DMAX, class LossA, class LossB>
__global__ void __launch_bounds__(2 * H, 2) fused_train_pair_kernel(FusedTrainArgs a, LossA fa, FusedTrainArgs b, LossB fb, unsigned grid_a) {
  if (blockIdx.x < grid_a) fused_train_body<H, NOUT_A, DMAX>(a, fa, blockIdx.x, grid_a);
  else fused_train_body<H, NOUT_B, DMAX>(b, fb, blockIdx.x - grid_a, gridDim.x - grid_a);
}

inline bool fused_train_supported(int H, int Din) { return (H == 64 || H == 128) && Din <= 93; }

inline int64_t fused_train_tiles(int64_t S) { return (S + kFusedTile - 1) / kFusedTile; }
// Workgroups of a launch at most: as many as the chip holds at once.  Each has a copy of the gradient in the workspace.
inline int64_t fused_train_grid(int H, int Din, int64_t S) {
  return std::min<int64_t>(fused_train_tiles(S), H == 128 ? 512 : Din < 32 ? 1024 : 768);
}
// Floats of the copies of a network's gradient and statistics.
inline int64_t fused_train_partial_floats(int H, int Din, int64_t S, int64_t gcount) { return fused_train_grid(H, Din, S) * copy_pitch(gcount + 5); }

template <class Kernel>
inline int32_t fused_train_configure(Kernel kern, size_t bytes) {
  if (bytes <= 64 * 1024) return MARL_OK;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) == hipSuccess ? MARL_OK : MARL_E_LAUNCH;
}

template <int H, int NOUT, int DMAX, class LossFn>
inline int32_t launch_fused_train_inst(FusedTrainArgs a, const LossFn& fn, hipStream_t s) {
  auto kern = fused_train_kernel<H, NOUT, DMAX, LossFn>;
  constexpr size_t bytes = fused_train_lds(H, NOUT, DMAX);
  const int32_t rc = fused_train_configure(kern, bytes);
  if (rc != MARL_OK) return rc;
  const unsigned grid = (unsigned)fused_train_grid(H, a.Din, a.S);
  a.stats_at = a.gcount;
  a.pstride = copy_pitch(a.gcount + 5);
  a.stats_mask = 31;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(2 * H), bytes, s, a, fn);
  launch_reduce_partials(a.partial, (int)grid, a.gcount + 5, a.grad, s, a.gcount, a.stats);
  return launch_status();
}

template <int H, int NOUT_A, int NOUT_B, int DMAX, class LossA, class LossB>
inline int32_t launch_fused_train_pair_inst(FusedTrainArgs a, const LossA& fa, FusedTrainArgs b, const LossB& fb, hipStream_t s) {
  auto kern = fused_train_pair_kernel<H, NOUT_A, NOUT_B, DMAX, LossA, LossB>;
  constexpr size_t bytes = std::max(fused_train_lds(H, NOUT_A, DMAX), fused_train_lds(H, NOUT_B, DMAX));
  const int32_t rc = fused_train_configure(kern, bytes);
  if (rc != MARL_OK) return rc;
  const unsigned grid_a = (unsigned)fused_train_tiles(a.S);  // == the second network's (the caller checks the sizes)
  // copy k of the first network's range is directly followed by copy k of the second's and by their statistics: one reduction
  b.partial = a.partial + a.gcount;
  a.pstride = b.pstride = copy_pitch(a.gcount + b.gcount + 5);
  a.stats_at = a.gcount + b.gcount;
  b.stats_at = b.gcount;
  a.stats_mask = LossA::kStats;
  b.stats_mask = LossB::kStats;
  static_assert((LossA::kStats & LossB::kStats) == 0 && (LossA::kStats | LossB::kStats) == 31, "every statistic from one network");
  hipLaunchKernelGGL(kern, dim3(2 * grid_a), dim3(2 * H), bytes, s, a, fa, b, fb, grid_a);
  launch_reduce_partials(a.partial, (int)grid_a, a.gcount + b.gcount + 5, a.grad, s, a.gcount + b.gcount, a.stats);
  return launch_status();
}

// The kernel finds a row through its row order entry (x_ptr) and divides sample indices by the rows' and the loss's agent counts with
// SmallDiv's product.
inline bool fused_train_rows_ok(const RowSrc& X, int64_t S, const SmallDiv& agents) {
  return X.gather != nullptr && small_div_ok(X.pd, S) && small_div_ok(agents, S);
}

template <int NOUT, class LossFn>
inline int32_t launch_fused_train(int H, const FusedTrainArgs& a, const LossFn& fn, hipStream_t s) {
  if (!fused_train_rows_ok(a.X, a.S, fn.lc.ad)) return MARL_E_SIZE;
  // algorithmic flops: forward 2S(DH + HH), backward 2S(HH + HH + DH)
  TimedLaunch timed(KC_FUSED_TRAIN, 2.0 * (double)a.S * (2.0 * a.Din * H + 3.0 * H * H), s);
  if (H == 128) {
    if (a.Din < 32) return launch_fused_train_inst<128, NOUT, 32, LossFn>(a, fn, s);
    return launch_fused_train_inst<128, NOUT, 96, LossFn>(a, fn, s);
  }
  if (a.Din < 32) return launch_fused_train_inst<64, NOUT, 32, LossFn>(a, fn, s);
  return launch_fused_train_inst<64, NOUT, 96, LossFn>(a, fn, s);
}

// Whether two networks can share a launch: the same shape on the same number of samples, so few tiles that the chip holds the
// workgroups of both launches together, and gradient ranges that follow one another (a's, then
// b's) so that the interleaved copies reduce in one pass.
inline bool fused_train_pair_supported(int Ha, int Da, int64_t Sa, int Hb, int Db, int64_t Sb) {
  if (Ha != Hb || Da != Db || Sa != Sb || !fused_train_supported(Ha, Da)) return false;
  return 2 * fused_train_tiles(Sa) <= (Ha == 128 ? 512 : Da < 32 ? 1024 : 768);
}
// Floats of the copies of both.
inline int64_t fused_train_pair_partial_floats(int64_t S, int64_t gcount_a, int64_t gcount_b) { return fused_train_tiles(S) * copy_pitch(gcount_a + gcount_b + 5); }

// b.grad == a.grad + a.gcount
template <int NOUT_A, int NOUT_B, class LossA, class LossB>
inline int32_t launch_fused_train_pair(int H, const FusedTrainArgs& a, const LossA& fa, const FusedTrainArgs& b, const LossB& fb, hipStream_t s) {
  if (!fused_train_rows_ok(a.X, a.S, fa.lc.ad) || !fused_train_rows_ok(b.X, b.S, fb.lc.ad)) return MARL_E_SIZE;
  if (b.grad != a.grad + a.gcount) return MARL_E_SIZE;
  TimedLaunch timed(KC_FUSED_TRAIN, 2.0 * (double)(a.S + b.S) * (2.0 * a.Din * H + 3.0 * H * H), s);
  if (H == 128) {
    if (a.Din < 32) return launch_fused_train_pair_inst<128, NOUT_A, NOUT_B, 32, LossA, LossB>(a, fa, b, fb, s);
    return launch_fused_train_pair_inst<128, NOUT_A, NOUT_B, 96, LossA, LossB>(a, fa, b, fb, s);
  }
  if (a.Din < 32) return launch_fused_train_pair_inst<64, NOUT_A, NOUT_B, 32, LossA, LossB>(a, fa, b, fb, s);
  return launch_fused_train_pair_inst<64, NOUT_A, NOUT_B, 96, LossA, LossB>(a, fa, b, fb, s);
}

}  // namespace marl
