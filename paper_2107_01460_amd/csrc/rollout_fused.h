// Host-side dispatch of the rollout (rollout_train.h) and evaluation (rollout_eval.h) kernels.
#pragma once
#include <algorithm>

#include "rollout_eval.h"
#include "rollout_train.h"

namespace marl {

// Networks the kernels are instantiated for: hidden width 64 (64-sample tiles) or 128 (32-sample tiles).
inline bool rollout_fused_supported(int H, int A) { return (H == 64 || H == 128) && A <= 8; }

// Workgroups of an evaluation block per CU, and as many as are resident at once.
constexpr int rollout_eval_occupancy(int capacity, int V) { return capacity <= 4 && V <= 5 ? 2 : 1; }
inline int rollout_eval_places(int H, int A, int F, int V) { return 256 * rollout_eval_occupancy(std::max(A, F), V) * ((H == 64 ? 64 : 32) / A); }
// Rows of an environment in a block of n episodes: all resident at once (beyond that they would only follow one another), one for each counted episode
// and, where those leave compute units without a workgroup, up to twice as many.  (Two workgroups share a unit's time: 512 environments of three agents,
// 128 units, episodes of 60 of 60 steps, two of them in 205 workgroups 350 us, eight in 410 393 us.)
// 0: in one chain.  Where no more than two rows have a place they go side by side only if every compute unit has one workgroup of theirs: else their
// chain (n / 2 + 1 1/3 caps) is hardly shorter than the block's where episodes end early, at longer steps (6000 environments, two agents, 64
// units, two episodes of 15 of 25 steps 309 us against 218 in one chain; 424 environments of eight agents, 128 units, a workgroup a unit, four
// of 54 of 54 steps 840 against 1590).
inline int rollout_eval_copies(int H, int A, int F, int V, int N, int n) {
  const int most = rollout_eval_places(H, A, F, V) / N, alone = 256 * ((H == 64 ? 64 : 32) / A) / N;
  return n >= 2 && (most >= 3 || alone >= 2) ? std::min(most, std::max(n, std::min(2 * n, alone))) : 0;
}

// Samples of a training rollout's tile: 16 while the chip holds all of those workgroups at once (one per CU at 128 units, two
// at 64), else 64 or 32.  A step is a chain of barriers, reads of weights and dependent sums, shorter in a tile of 16, and the
// CUs that it takes would stand idle; where they would not, every tile's read of the weights counts.  32 steps, us, tiles of 64
// or 32 / of 16: 64 units, two agents, view 3: 64 environments 149 / 104, 2048 172 / 126, 4096 194 / 167, 8192 233 / 244,
// 16384 373 / 463; 128 units, three agents, view 5: 16 environments 245 / 195, 1280 274 / 226, 2048 290 / 308, 4096 466 / 587.
inline int rollout_rows(int H, int A, int N) {
  const int64_t groups = ((int64_t)N + 16 / A - 1) / (16 / A);
  return groups <= (H == 64 ? 512 : 256) ? 16 : H == 64 ? 64 : 32;
}

template <int H, int BM, int V, int CA, int KIND, bool EVAL>
inline int32_t launch_rollout_fused_inst(const RolloutArgs& a, hipStream_t s) {
  const int epw = BM / a.p.A;
  const unsigned grid = (unsigned)(((int64_t)a.p.N * std::max(a.eps.copies, 1) + epw - 1) / epw);
  constexpr int D = 3 * V * V;
  void (*kern)(RolloutArgs);
  size_t bytes;
  if constexpr (EVAL) {
    kern = rollout_eval_kernel<H, BM, V, CA, KIND, rollout_eval_occupancy(CA, V)>;
    bytes = 2 * (size_t)BM * (2 * rollout_eval_px(D) + 3 * (H + 8)) + sizeof(float) * ((H / 32) * kActions * BM + H * kActions + 2 * H + 4);
  } else {
    kern = rollout_train_kernel<H, BM, V, CA, KIND, BM == 16 ? 2 : ((H == 64 && CA <= 2) || (CA <= 4 && V <= 5)) ? 3 : 1>;
    bytes = sizeof(float) * (2 * (size_t)BM * rollout_train_px(D) + (size_t)BM * (H + 4) + (H / 16) * (size_t)BM * kActions + H * kActions + 2 * BM * 8);
  }
  if (bytes > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
    return MARL_E_LAUNCH;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), bytes, s, a);
  return launch_status();
}

template <int H, int V, int CA, int KIND, bool EVAL>
inline int32_t launch_rollout_fused_rows(const RolloutArgs& a, hipStream_t s) {
  if constexpr (!EVAL)
    if (a.rows == 16) return launch_rollout_fused_inst<H, 16, V, CA, KIND, false>(a, s);
  return launch_rollout_fused_inst<H, H == 64 ? 64 : 32, V, CA, KIND, EVAL>(a, s);
}
template <int V, int KIND, bool EVAL>
inline int32_t launch_rollout_fused_view(int H, const RolloutArgs& a, hipStream_t s) {
  const int cap = a.p.A > a.p.F ? a.p.A : a.p.F;  // every loop over entities is unrolled to the capacity
  if constexpr (V == 3 && KIND == 0) {  // the small foraging shape (two agents, one food): half the unrolled entity loops
    if (cap <= 2 && H == 64) return launch_rollout_fused_rows<64, V, 2, KIND, EVAL>(a, s);
  }
  if (H == 64) {
    if (cap <= 4) return launch_rollout_fused_rows<64, V, 4, KIND, EVAL>(a, s);
    return launch_rollout_fused_rows<64, V, 8, KIND, EVAL>(a, s);
  }
  if (cap <= 4) return launch_rollout_fused_rows<128, V, 4, KIND, EVAL>(a, s);
  return launch_rollout_fused_rows<128, V, 8, KIND, EVAL>(a, s);
}

// Defined in rollout_v3.hip / rollout_v5.hip / rollout_v7.hip (one translation unit per view size).
int32_t launch_rollout_fused_v3(int H, bool eval, const RolloutArgs& a, hipStream_t s);
int32_t launch_rollout_fused_v5(int H, bool eval, const RolloutArgs& a, hipStream_t s);
int32_t launch_rollout_fused_v7(int H, bool eval, const RolloutArgs& a, hipStream_t s);

template <int V>
inline int32_t launch_rollout_fused_tu(int H, bool eval, const RolloutArgs& a, hipStream_t s) {
  if (a.p.kind == 0) {
    if (eval) return launch_rollout_fused_view<V, 0, true>(H, a, s);
    return launch_rollout_fused_view<V, 0, false>(H, a, s);
  }
  if (eval) return launch_rollout_fused_view<V, 1, true>(H, a, s);
  return launch_rollout_fused_view<V, 1, false>(H, a, s);
}

}  // namespace marl
