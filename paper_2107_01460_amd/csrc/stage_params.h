// The working copy of a feed-forward system's parameters (ParamMap), one element at a time: blocks moved to their aligned offsets,
// optionally rounded to bf16, plus the copies of W1, W2 and W2 transposed that the fused kernels read.
#pragma once
#include "common.h"
#include "split_bf16.h"

namespace marl {

__device__ __forceinline__ void store_split_weight(float* copy, float v, int64_t k, int64_t n, int H) {
  const SplitPair s = split_pair_any(v, 0.f);
  bf16_t* const d = reinterpret_cast<bf16_t*>(copy) + split_weight_index(k, n, H);
  d[0] = (bf16_t)s.h;
  d[split_weight_plane(H)] = (bf16_t)s.m;
  d[2 * split_weight_plane(H)] = (bf16_t)s.l;
}
// What a working copy's actor is in.
enum RolloutCopy { COPY_SPLIT, COPY_FP32, COPY_FP32_16 };  // split; fp32 for a training rollout in tiles of 32 or 64 samples, of 16
// Where row k of a weight matrix stands for tiles of 16 samples: of every sixteen, quarter q of a wavefront takes k = 4 (q % 2) + q / 2 + 2 h of
// either eight, its four values beside one another.
__host__ __device__ inline int64_t rollout_order16(int64_t k) {
  const int64_t q = (k & 1) << 1 | (k >> 2 & 1), e = (k >> 3 & 1) << 1 | (k >> 1 & 1);
  return (k & ~(int64_t)15) | q << 2 | e;
}
// element (k, n) of a copy of network `net`
__device__ __forceinline__ void stage_element(float* dst, const ParamMap& pm, int net, int64_t copy, float v, int64_t k, int64_t n, int for_rollout) {
  const int H = pm.hidden[net];
  if (for_rollout == COPY_FP32_16 && net == 0) k = rollout_order16(k);
  if (for_rollout != COPY_SPLIT && net == 0) dst[copy + ((k / 4) * H + n) * 4 + k % 4] = v;
  else store_split_weight(dst + copy, v, k, n, H);
}
// parameter i, of value v
__device__ __forceinline__ void stage_param(float* dst, const ParamMap& pm, int64_t i, float v, bool round, int for_rollout, bool for_update) {
  int b = 0;
#pragma unroll
  for (int k = 1; k < 12; ++k) b += (i >= pm.src[k]) ? 1 : 0;
  if (round) v = round_to_bf16(v);
  const int64_t e = i - pm.src[b];
  const int net = b >= 6, H = pm.hidden[net];
  const bool w1 = b == 0 || b == 6, w2 = b == 2 || b == 8;
  if (!pm.fused[net] || !(w1 || w2)) {
    dst[pm.dst[b] + e] = v;
    return;
  }
  const uint32_t r = (uint32_t)e / (uint32_t)H, c = (uint32_t)e - r * (uint32_t)H;  // (a block has fewer than 2^32 elements; a 64-bit division is 180 instructions)
  stage_element(dst, pm, net, w1 ? pm.sw_w1[net] : pm.sw_w2[net], v, r, c, for_rollout);
  if (w2 && for_update) store_split_weight(dst + pm.sw_w2t[net], v, c, r, H);
}

}  // namespace marl
