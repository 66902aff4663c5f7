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
};

// What a tile costs, in us (MI355X, product and reduction of its copies; 368 shapes of 27 .. 1176 x 32 .. 1536 outputs over 256 ..
// 262 144 samples, fitted per tile to about 5 %): the launches, a MB of copies, and a step of kGemmBK samples with one, two, three or
// four workgroups on each CU.  Index 1: the rows of A can be read 16 bytes at a time (M a multiple of four).
struct TnTileCost {
  int bm, bn;
  float launch[2], copies[2], step[2][4];
};
constexpr TnTileCost kTnTiles[] = {
    {160, 128, {9.2f, 7.6f}, {0.43f, 0.44f}, {{2.77f, 3.58f}, {2.87f, 3.33f}}},
    {128, 128, {8.2f, 7.4f}, {0.52f, 0.53f}, {{2.28f, 3.00f}, {2.30f, 2.70f}}},
    {128, 64, {4.2f, 5.0f}, {0.69f, 0.61f}, {{2.00f, 2.44f, 3.27f, 4.33f}, {1.79f, 2.06f, 2.54f, 3.55f}}},
    {96, 128, {7.8f, 6.9f}, {0.52f, 0.59f}, {{1.89f, 2.44f}, {1.92f, 2.23f}}},
    {32, 128, {6.2f, 6.2f}, {0.65f, 0.71f}, {{1.02f, 1.36f}, {1.03f, 1.29f}}},
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
// 234 us, 32 rows 440 although they pad least); in between padding counts (147 x 256, 262 144 samples: 160 rows 150 us, 96 190, 128
// 222, 32 258).  64 columns only where 128 would leave a half-empty last tile.  Among the 1864 products measured the choice is 0.1 % behind
// the fastest tile on average; where two tiles are within 3 % the one that needs no further instantiation is taken.
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
  return tn_ranges(best->bm, best->bn, M, N, K);
}
// floats of the copies of a product
inline int64_t tn_copy_floats(int64_t M, int64_t N, int64_t K) { return tn_plan(M, N, K).splits * (M * N + N); }

}  // namespace marl
