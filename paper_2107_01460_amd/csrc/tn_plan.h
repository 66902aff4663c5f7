// Output tile and k ranges of a weight-gradient product (gemm_split_kernel<GEMM_TN>).  Plain C++: no device code.
#pragma once
#include <algorithm>
#include <cstdint>

namespace marl {

constexpr int kGemmBK = 32;  // samples staged at a time

struct TnPlan {
  int bm, bn;         // output tile
  int64_t per;        // samples of a k range, a multiple of kGemmBK
  int64_t splits;     // k ranges: each writes its own copy of the M x N outputs and the N column sums
  bool wide = false;  // tiles of 192 columns, two in place of three of bn = 128
};

// What a tile costs, in us (MI355X, product and reduction of its copies; 368 shapes of 27 .. 1176 x 32 .. 1536 outputs over 256 ..
// 262 144 samples, fitted per tile to about 5 %): the launches, a MB of copies, and a step of kGemmBK samples with one, two, three or
// four workgroups on each CU.  Index 1: the rows of A are 16-byte aligned (M a multiple of four).  Index 0, for loads of 16 bytes at any
// 4-byte boundary: 827 products of 27 .. 1029 x 32 .. 512 outputs over 1024 .. 262 144 samples, fitted to 3-4 %.
struct TnTileCost {
  int bm, bn;
  float launch[2], copies[2], step[2][4];
};
constexpr TnTileCost kTnTiles[] = {
    {160, 128, {7.7f, 7.6f}, {0.41f, 0.44f}, {{2.81f, 3.39f}, {2.87f, 3.33f}}},
    {128, 128, {9.2f, 7.4f}, {0.45f, 0.53f}, {{2.06f, 2.73f}, {2.30f, 2.70f}}},
    {128, 64, {7.6f, 5.0f}, {0.42f, 0.61f}, {{1.50f, 1.98f, 2.61f, 3.65f}, {1.79f, 2.06f, 2.54f, 3.55f}}},
    {96, 128, {6.9f, 6.9f}, {0.47f, 0.59f}, {{1.94f, 2.28f}, {1.92f, 2.23f}}},
    {32, 128, {7.1f, 6.2f}, {0.51f, 0.71f}, {{0.98f, 1.26f}, {1.03f, 1.29f}}},
};
constexpr int64_t kTnCus = 256, kTnMinRange = 256;

// The k ranges: two workgroups of 128 columns per CU, no range below 256 samples.
inline TnPlan tn_ranges(int bm, int bn, int64_t M, int64_t N, int64_t K) {
  const int64_t tiles = ((M + bm - 1) / bm) * ((N + 127) / 128), want = std::max<int64_t>(1, 2 * kTnCus / tiles);
  const int64_t per = std::max<int64_t>(kTnMinRange, ((K + want - 1) / want + kGemmBK - 1) / kGemmBK * kGemmBK);
  return TnPlan{bm, bn, per, (K + per - 1) / per};
}
inline double tn_cost(const TnTileCost& t, int64_t M, int64_t N, int64_t K) {
  const TnPlan p = tn_ranges(t.bm, t.bn, M, N, K);
  const int v = M % 4 == 0;
  const int levels = t.bn == 64 ? 4 : 2;
  const int64_t groups = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * p.splits, load = (groups + kTnCus - 1) / kTnCus;
  double step = t.step[v][std::min<int64_t>(load, levels) - 1];
  if (load > levels) step *= (double)groups / (double)(levels * kTnCus);
  return t.launch[v] + (double)(p.per / kGemmBK) * step + t.copies[v] * 4e-6 * (double)(p.splits * (M * N + N));
}

// The tile that costs least.  Neither the padding alone nor the work of a tile decides it: a range of samples is a serial chain of steps,
// so that few samples, which do not fill the chip, want the lowest tile (480 x 480, 1024 samples: 32 rows 17.5 us, 96 24.7, 128 x 64
// 21.8), while many want the one that splits each value for the most products (588 x 512, 65 536 samples: 128 and 160 rows 243 and
// 234 us, 32 rows 440 although they pad least); in between padding counts (147 x 256, 262 144 samples: 160 rows 143 us, 96 174, 128
// 201, 32 231).  64 columns only where 128 would leave a half-empty last tile.  Among the 1864 products measured the choice is 0.1 % behind
// the fastest tile on average (unaligned rows, 1667 products: 0.1 %, at most 10 %); where two tiles are within 3 % the one that needs no
// further instantiation is taken.
inline TnPlan tn_plan(int64_t M, int64_t N, int64_t K) {
  const bool halves = N % 128 != 0;
  const TnTileCost* best = nullptr;
  double least = 0.0;
  for (const TnTileCost& t : kTnTiles) {
    if (t.bn == 64 && !halves) continue;
    const bool usual = M <= 32 ? t.bm == 32 : t.bm == 128 && (t.bn == 64) == halves;
    const double cost = tn_cost(t, M, N, K) * (usual ? 0.97 : 1.0);
    if (best == nullptr || cost < least) {
      best = &t;
      least = cost;
    }
  }
  TnPlan p = tn_ranges(best->bm, best->bn, M, N, K);
  // Where 128 x 128 tiles are the choice, whole tiles of 192 columns fit and the ranges of 512 workgroups of them have at least 512
  // samples: us with the sums of the copies, 128 / 192 columns: 128 x 384 over 262 144 samples 175.3 / 164.6, 1 048 576 702.9 / 602.7; 256 x 768
  // over 49 152 138.1 / 118.6, 262 144 628.7 / 535.7; 512 x 1536 over 16 384 178.1 / 145.2.  Shorter ranges win alone from 256 samples on (128 x 384 over
  // 98 304 79.4 / 75.0) but lose beside another network's kernels, to which half as many copies again are in the way: a recurrent
  // iteration of 1024 environments, 128 units, 24.4 ms without them and 25.3 with.
  const int64_t tiles = ((M + 127) / 128) * (N / 192);
  if (p.bm == 128 && p.bn == 128 && N % 384 == 0 && (double)K * (double)tiles >= (double)(4 * kTnCus * kTnMinRange)) {
    const int64_t want = std::max<int64_t>(1, 2 * kTnCus / tiles);
    p.per = std::max<int64_t>(kTnMinRange, ((K + want - 1) / want + kGemmBK - 1) / kGemmBK * kGemmBK);
    p.splits = (K + p.per - 1) / p.per;
    p.wide = true;
  }
  return p;
}
// floats of the copies of a product
inline int64_t tn_copy_floats(int64_t M, int64_t N, int64_t K) { return tn_plan(M, N, K).splits * (M * N + N); }

}  // namespace marl
