// LDS-tiled fp32 GEMM for gfx950 on split bf16 operands (split_bf16.h), shared by the rollout forward
// pass and the PPO backward pass.  Three operand arrangements:
//   NN  C[m][n] = sum_k A[m][k] * B[k][n]     activations x weights
//   NT  C[m][n] = sum_k A[m][k] * B[n][k]     gradient x weights^T
//   TN  C[m][n] = sum_k A[k][m] * B[k][n]     activations^T x gradient (split over k across workgroups)
// "A" is always given by rows (optionally gathered through an index list), so a minibatch is read
// in place from the trajectory.
#pragma once
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "split_bf16.h"
#include "tn_plan.h"

namespace marl {

// Division of a sample index by a small run-time divisor (agents per row) without the 64-bit division sequence,
// which is about 180 vector instructions and sat on the critical path of every row tile: for s < 2^31 and
// d <= 64, s / d = (s * magic) >> shift exactly, with magic = floor(2^shift / d) + 1 and
// shift = 31 + ceil(log2 d) (the error term s * (magic * d - 2^shift) stays below 2^shift; d = 1 gives
// magic 2^31 + 1, shift 31).  div<true> is that product and nothing else -- the caller has checked on the host that
// the divisor has a magic number and that every index is below 2^31 (small_div_ok); div<false> is the plain division.
// (One function that chooses at run time keeps the long sequence in the instruction stream and was slower.)
struct SmallDiv {
  uint32_t magic = 0;
  int shift = 0;
  template <bool FAST>
  __device__ __forceinline__ int64_t div(int64_t s, int d) const {
    if (FAST) return (int64_t)(__umulhi(2 * (uint32_t)s, magic) >> (shift - 31));  // s * magic >> shift, the upper half of one 32-bit product
    return s / d;
  }
};
inline SmallDiv make_small_div(int d) {
  SmallDiv v;
  if (d < 1 || d > 64) return v;
  int lg = 0;
  while ((1 << lg) < d) ++lg;
  v.shift = 31 + lg;
  v.magic = (uint32_t)(((uint64_t)1 << v.shift) / (uint64_t)d + 1);
  return v;
}

// Rows of a matrix: row r = base + (src(r/per) * per + r%per) * ld, src = gather ? gather[.] : identity.
struct RowSrc {
  const float* base;
  int64_t ld;
  const int32_t* gather;
  int per;
  int64_t nrows;
  SmallDiv pd{};  // make_small_div(per), or default
  __device__ __forceinline__ const float* ptr(int64_t r) const {
    if (r >= nrows) return nullptr;
    if (gather == nullptr) return base + r * ld;
    const int64_t g = per == 1 ? r : r / per;  // (a 64-bit division is about 180 instructions; one row per entry needs none)
    const int a = (int)(r - g * per);
    return base + ((int64_t)gather[g] * per + a) * ld;
  }
  // The same address in two steps, so that the gather entry can be fetched long before the row is.
  template <bool FAST = false>
  __device__ __forceinline__ int32_t gather_entry(int64_t r) const {
    return gather == nullptr ? 0 : gather[pd.div<FAST>(r, per)];
  }
  template <bool FAST = false>
  __device__ __forceinline__ const float* ptr_with(int64_t r, int32_t entry) const {
    if (gather == nullptr) return base + r * ld;
    const int a = (int)(r - pd.div<FAST>(r, per) * per);
    return base + ((int64_t)entry * per + a) * ld;
  }
};
// div<true> may be used for indices below `count` with this divisor
inline bool small_div_ok(const SmallDiv& v, int64_t count) { return v.magic != 0 && count < ((int64_t)1 << 31); }

enum GemmMode { GEMM_NN = 0, GEMM_NT = 1, GEMM_TN = 2 };
enum GemmEpi {
  EPI_BIAS_TANH = 0,  // C = tanh(acc + aux_vec[n])
  EPI_DTANH = 1,      // C = acc * (1 - aux_mat[m][n]^2)
  EPI_ATOMIC_ADD = 2, // C += acc (fp32 atomics; split-k partial results)
  EPI_STORE = 3       // C = acc + aux_vec[n] (aux_vec nullable)
};

struct GemmArgs {
  RowSrc A;          // NN/NT: M rows of K;  TN: K rows of M
  const float* B;    // NN/TN: [K][ldb];  NT: [N][ldb]
  int64_t ldb;
  float* C;          // [M][ldc]
  int64_t ldc;
  const float* aux_vec;  // EPI_BIAS_TANH: bias [N]; EPI_STORE: nullable bias [N]
  const float* aux_mat;  // EPI_DTANH: previous activation [M][ldaux]
  int64_t ldaux;
  float* colsum;         // TN: column sums of B are added here ([N], atomic), nullable
  int64_t M, N, K;
  int64_t k_per_split;   // TN: samples of a k range (launch_gemm fills it in, from tn_plan)
  int c_rot;             // TN, multiple of 32 below N: column n of the product goes to column (n + c_rot) mod N of C and colsum
  // TN with EPI_ATOMIC_ADD, nullable: k split z stores its products at split_out + z * split_count + m * ldc + n and its
  // column sums of B behind them (at + M * ldc + n) with plain stores instead of adding to C / colsum with atomics; the
  // caller then adds the splits in a fixed order (reduce_partials_kernel), which makes the result the same in every run.
  // launch_gemm says whether the launch did.
  float* split_out;
  int64_t split_count;
};

// The kernels that finish with one partial result per workgroup (the training kernels of whole networks, the output-layer loss
// kernel) store those with plain stores and add them up here: a few hundred workgroups adding to the same
// cache lines with atomics at the same moment queue up at the L2 (60-180 us per launch).  The weight-gradient products
// do the same with one slab per k split when the caller passes split_out; without it, they add with atomics.

// out[i] += sum_b partial[b * copy_pitch(count) + i], the copies added in a fixed order, so that the result does not depend on the
// run; elements from `head` on go to tail[i - head] instead.  The order: 32 sums of the copies b = g, g + 32, g + 64, ... (eight at a time, as
// a tree), then a tree over g.  A group of 8 W lanes with 16 bytes each takes W of the 32 sums one after the other, so that a workgroup has
// 32 W elements and a launch fewer workgroups; the results are the same for every W.
// Bound: the copies' way from memory, and for few of them a launch.
constexpr int64_t copy_pitch(int64_t count) { return (count + 3) & ~(int64_t)3; }
template <int W>
static __global__ void __launch_bounds__(256) reduce_partials_kernel(const float* __restrict__ partial, int nblocks, int64_t count,
                                                                     float* __restrict__ out, int64_t head, float* __restrict__ tail) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  constexpr int LANES = 8 * W;
  static_assert(W == 1 || W == 2, "groups of a wavefront meet in its lanes");
  __shared__ f4 part[4][LANES];
  const int l = threadIdx.x % LANES, g = threadIdx.x / LANES * W, wave = threadIdx.x >> 6;
  const int64_t i0 = (int64_t)blockIdx.x * (4 * LANES), pitch = copy_pitch(count);
  f4 s[W];
#pragma unroll
  for (int w = 0; w < W; ++w) s[w] = f4{0.f, 0.f, 0.f, 0.f};
  if (i0 + 4 * l < pitch) {
    const float* const src = partial + i0 + 4 * l;
    if (nblocks <= 32) {  // one copy each
#pragma unroll
      for (int w = 0; w < W; ++w)
        if (g + w < nblocks) s[w] += *reinterpret_cast<const f4*>(src + (g + w) * pitch);
    } else {
#pragma unroll
      for (int w = 0; w < W; ++w)
        for (int b = g + w; b < nblocks; b += 256) {
          f4 v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            v[u] = f4{0.f, 0.f, 0.f, 0.f};
            if (b + 32 * u < nblocks) v[u] = *reinterpret_cast<const f4*>(src + (b + 32 * u) * pitch);
          }
          s[w] += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        }
    }
  }
#pragma unroll
  for (int w = 1; w < W; w *= 2)
#pragma unroll
    for (int u = 0; u < W; u += 2 * w) s[u] += s[u + w];
#pragma unroll
  for (int o = LANES; o < 64; o *= 2)
#pragma unroll
    for (int k = 0; k < 4; ++k) s[0][k] += __shfl_xor(s[0][k], o);
  if ((threadIdx.x & 63) < LANES) part[wave][l] = s[0];
  __syncthreads();
  const int64_t i = i0 + threadIdx.x;
  if (threadIdx.x < 4 * LANES && i < count) {
    const int q = threadIdx.x >> 2, k = threadIdx.x & 3;
    float* const dst = i < head ? out + i : tail + (i - head);
    *dst += (part[0][q][k] + part[1][q][k]) + (part[2][q][k] + part[3][q][k]);
  }
}
// `partial`: 16-byte aligned.  Workgroups of 32 elements for small gradients, of 64 for large ones, whose many workgroups cost more than
// the longer way through the copies: MI355X, us, one launch between events (6.1 when empty), with 32, 64 and 128 elements, and with 8
// groups of 32 4-byte loads: 1024 copies of 6464 floats 8.6, 10.5, 19.4, 14.5; 512 of 9728 7.5, 7.9, 12.4, 9.7; 512 of 26 880 13.0, 12.1,
// 14.3, 11.7; 170 of 49 536 9.5, 9.7, 10.2, 9.4; 42 of 197 376 10.0, 9.7, 11.6, 10.2; 21 of 197 376 8.0, 7.0, 8.0, 8.6; 8 of 197 376 7.7,
// 6.2, 7.3, 6.2; 32 of 262 656 10.0, 9.3, 10.9, 9.0.
inline void launch_reduce_partials(const float* partial, int nblocks, int64_t count, float* out, hipStream_t s, int64_t head = INT64_MAX,
                                   float* tail = nullptr) {
  auto launch = [&](auto kern, int elements) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((count + elements - 1) / elements)), dim3(256), 0, s, partial, nblocks, count, out, head, tail);
  };
  if (count < 16384) launch(reduce_partials_kernel<1>, 32);
  else launch(reduce_partials_kernel<2>, 64);
}

// tanh(x) = 1 - 2 / (e^{2x} + 1) with the hardware exp2 and reciprocal: absolute error ~1e-7 (the values feed
// sums of O(1) activations, so an absolute bound is what the 1e-4 tolerance on the outputs needs); saturates
// cleanly to +-1 when e^{2x} overflows or underflows.
__device__ __forceinline__ float tanh_f32(float x) {
  const float e = __builtin_amdgcn_exp2f(x * 2.885390081777927f);  // e^{2x}
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(e + 1.0f);
}

// Products of a row tile against weights: the weights from a split operand-order copy (ParamMap) straight from the cache hierarchy into
// registers, so that a layer needs no staging buffer and no barrier of its own.  The first kPhaseRing groups of 16 along k
// are requested one phase AHEAD of the product -- during the element-wise epilogue or the LDS-only product in front of it
// -- and the others as their slots become free, so that the product does not wait for the L2.  The loads are buffer
// loads: a resource descriptor in scalar registers, ONE vector register with the lane's byte offset for all of them, the
// group's offset as a scalar (as global loads each of them got a 64-bit address register pair of its own).
constexpr int kPhaseRing = 4;
template <int KG, int MOST = kPhaseRing>
struct PhaseW {
  static constexpr int RING = KG < MOST ? KG : MOST;
  bf16x8 w[RING][3];
};
typedef __amdgpu_buffer_rsrc_t WeightRsrc;
// descriptor of `floats` floats at p (raw buffer, no swizzle; reads past the end return zero)
__device__ __forceinline__ WeightRsrc weight_rsrc(const float* p, int floats) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, floats * 4, 0x00020000);
}
// descriptor of a split [K][H] copy
__device__ __forceinline__ WeightRsrc split_weight_rsrc(const float* p, int K, int H) { return weight_rsrc(p, K * H * 3 / 2); }
// lane_off: (hi * H + n) * 4 for this lane's column n
template <int H, int KG, int MOST>
__device__ __forceinline__ void phase_w_load(PhaseW<KG, MOST>& pw, WeightRsrc B, int lane_off, int g, int kgroups) {
  const int at = g < kgroups ? g : kgroups - 1;  // past the end: the last group again (never used)
#pragma unroll
  for (int p = 0; p < 3; ++p)
    pw.w[g % PhaseW<KG, MOST>::RING][p] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(B, lane_off * 4, (at * 3 + p) * 32 * H, 0));
}
template <int H, int KG, int MOST>
__device__ __forceinline__ void phase_w_request(PhaseW<KG, MOST>& pw, WeightRsrc B, int lane_off, int kgroups) {
#pragma unroll
  for (int g = 0; g < PhaseW<KG, MOST>::RING; ++g) phase_w_load<H>(pw, B, lane_off, g, kgroups);
}
// The transposed product, weights x samples: acc += B^T A^T for this wavefront's 32 units x 32 samples, so that a lane holds
// four times four consecutive units of one sample.  A by rows of split planes in LDS (xs points at this lane's row, + 8 * hi;
// planes `plane` elements apart).  EXACT: one plane, the values are exact in bf16 and the lower parts' products are zero.
template <int H, int KG, bool EXACT, int MOST>
__device__ __forceinline__ void gemm_phase_t(const bf16_t* xs, int plane, WeightRsrc B, int lane_off, int kgroups, floatx16& acc, PhaseW<KG, MOST>& pw) {
  constexpr int RING = PhaseW<KG, MOST>::RING;
#pragma unroll
  for (int g = 0; g < KG; ++g) {
    if (g < kgroups) {  // uniform
      const Split8 w{pw.w[g % RING][0], pw.w[g % RING][1], pw.w[g % RING][2]};
      if (EXACT) {
        const bf16x8 x = *reinterpret_cast<const bf16x8*>(xs + 16 * g);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w.l, x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w.m, x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w.h, x, acc, 0, 0, 0);
      } else {
        acc = mfma_split(w, frag_row(xs + 16 * g, plane), acc);
      }
      if (g + RING < KG) phase_w_load<H>(pw, B, lane_off, g + RING, kgroups);
    }
  }
}

// BM x BN tile, four wavefronts (2 x 2 at BM = 128, side by side at the other heights of TN), k tiles of 32 in one LDS buffer of split
// operands; the next k tile travels global -> registers while the current one is multiplied, and two workgroups per CU
// cover each other's staging and barriers.  A tile is kept in LDS in its source orientation: k-contiguous tiles are read
// with 16-byte reads (pitch 40 elements: an odd number of 16-byte units), the others with the transposing read (the
// pitches put four consecutive rows on different quarters of the banks).
// Bound: per k tile and wavefront 48 matrix instructions at BN = 128 (1536 cycles) against about 700 cycles of vector
// instructions that split 32 staged values per thread, which the other workgroup's matrix instructions cover; at
// contraction lengths of 128 .. 256 the activations' HBM traffic is the other bound.  Measured against the kernel on the
// fp32 instruction that this one replaced: dW of 256 x 256 over 262 144 samples 295 -> 196 us; a training iteration whose
// networks run layer by layer (147-256-6 and 147-192-1, 250 000 samples) 27.1 -> 19.9 ms.  The check for NaNs at the end of a
// tile (values out of split_pair's range) costs 1 %.  Requesting a k tile two tiles ahead instead of one changed nothing at 128 columns
// and cost 40 % at 64: the loads are not what a k tile waits for.
// Tiles of 192 columns (NN, TN): a wavefront's 64 x 96 part reads 15 fragments for 36 matrix instructions' worth of sums where 64 x 64 reads
// 12 for 24, and every value of A is split for 192 products in place of 128: 256 x 768 over 262 144 samples with its copies' sums
// 629 -> 536 us, 128 x 384 over 1 048 576 703 -> 603, 262 144 x 768 x 256 forward 667 -> 604, 262 144 x 192 x 147 176 -> 141.
template <int MODE, int EPI, int BM, int BN, bool AVEC>
__global__ void __launch_bounds__(256, 2) gemm_split_kernel(GemmArgs g) {
  constexpr int BK = kGemmBK;
  constexpr int WM = BM == 128 ? 2 : 1, WN = 4 / WM, TM = BM / (32 * WM), TN = BN / (32 * WN);
  static_assert(TM >= 1 && TN >= 1 && (BM == 128 || MODE == GEMM_TN), "wavefront tiles");
  constexpr bool A_KCONT = (MODE != GEMM_TN);  // A tile stored [m][k] else [k][m]
  constexpr bool B_KCONT = (MODE == GEMM_NT);  // B tile stored [n][k] else [k][n]
  constexpr int PK = BK + 8;
  constexpr int PMA = BM % 64 == 32 ? BM : BM + 32, PNB = BN + 32;  // rows 16 or 48 banks apart
  constexpr int A_PLANE = A_KCONT ? BM * PK : BK * PMA, B_PLANE = B_KCONT ? BN * PK : BK * PNB;
  constexpr int A_VECS = BK * BM / 4 / 256, B_VECS = BK * BN / 4 / 256;  // 16-byte pieces a thread stages
  static_assert(A_VECS >= 1 && B_VECS >= 1, "every thread stages");
  constexpr int BCH = BN == 192 ? 3 : 1, BPC = BN / 4 / BCH;  // a thread's pieces of B (b_row, b_col) lie in BCH places of a row throughout
  __shared__ __attribute__((aligned(16))) bf16_t As[3 * A_PLANE];
  __shared__ __attribute__((aligned(16))) bf16_t Bs[3 * B_PLANE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int lo = lane & 31, hi = lane >> 5;
  // Tiles that share an operand are neighbours on one XCD and meet in its L2: the column tiles of a row tile (NN, NT:
  // the activations, read once per column tile otherwise), the output tiles of a k slab (TN: with the plain order 1074 MB
  // came from HBM per launch at 256 x 256 outputs where 537 are algorithmic).
  const unsigned lg = xcd_remap(blockIdx.x, gridDim.x);
  const unsigned nbn = (unsigned)((g.N + BN - 1) / BN), nbm = (unsigned)((g.M + BM - 1) / BM);
  const unsigned by = lg % nbn, bx = MODE == GEMM_TN ? (lg / nbn) % nbm : lg / nbn, bz = MODE == GEMM_TN ? lg / (nbn * nbm) : 0;
  const int64_t m0 = (int64_t)bx * BM, n0 = (int64_t)by * BN;
  int64_t k_begin = 0, k_end = g.K;
  if (MODE == GEMM_TN) {
    k_begin = (int64_t)bz * g.k_per_split;
    k_end = min(g.K, k_begin + g.k_per_split);
    if (k_begin >= k_end) return;  // uniform
  }

  // ---- global -> registers.  Indices past the end are clamped to the last element: rows and columns past the end feed
  // outputs that are never stored; of the k past the end both operands are set to zero (zero times the infinity that the
  // last element may be would be a NaN).
  float4 ra[A_VECS], rb[B_VECS];
  const float* arow[A_VECS];           // A_KCONT: this thread's rows
  int q[A_VECS], rem[A_VECS];          // TN: gather index and agent of this thread's next row of A, advanced by BK per stage
  int32_t entry[A_VECS];               // ... and its gather entry, fetched one stage ahead
  const int per = g.A.per, dq = BK / per, dr = BK - dq * per;
  const int q_last = (int)((uint32_t)(k_end - 1) / (uint32_t)per), rem_last = (int)(k_end - 1) - q_last * per;
  if (A_KCONT) {
#pragma unroll
    for (int p = 0; p < A_VECS; ++p) arow[p] = g.A.ptr(min(m0 + ((tid + 256 * p) >> 3), g.M - 1));
  }
  auto fetch_entries = [&]() {  // TN with gathered rows: entries of the stage that (q, rem) stands at
    if (MODE == GEMM_TN && g.A.gather != nullptr) {
#pragma unroll
      for (int p = 0; p < A_VECS; ++p) entry[p] = g.A.gather[min(q[p], q_last)];
    }
  };
  auto b_row = [&](int p) { return tid / BPC + p / BCH * (256 / BPC); };  // of a tile of B in rows of k
  auto b_col = [&](int p) { return 4 * (tid % BPC + p % BCH * BPC); };
  auto fetch = [&](int64_t k0) {
    if (A_KCONT) {
      const int64_t k = k0 + 4 * (tid & 7);
#pragma unroll
      for (int p = 0; p < A_VECS; ++p) {
        if (AVEC) {
          const float4 v = *reinterpret_cast<const float4*>(arow[p] + min(k, k_end - 4));
          ra[p] = k < k_end ? v : make_float4(0.f, 0.f, 0.f, 0.f);
        } else {
          float e[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float v = arow[p][min(k + j, k_end - 1)];
            e[j] = k + j < k_end ? v : 0.f;
          }
          ra[p] = make_float4(e[0], e[1], e[2], e[3]);
        }
      }
    } else {
#pragma unroll
      for (int p = 0; p < A_VECS; ++p) {
        const int64_t m = m0 + 4 * ((tid + 256 * p) % (BM / 4));
        const bool past = q[p] > q_last || (q[p] == q_last && rem[p] > rem_last);
        const int qc = past ? q_last : q[p], rc = past ? rem_last : rem[p];
        const int64_t row = (g.A.gather != nullptr ? (int64_t)entry[p] : (int64_t)qc) * per + rc;
        const float* src = g.A.base + row * g.A.ld;
        if (AVEC) {
          ra[p] = *reinterpret_cast<const float4*>(src + min(m, g.M - 4));
        } else {
          // 16 bytes at any 4-byte boundary, within the row (M is at least 27): stage() moves the last columns into place
          typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
          const f4u v = *reinterpret_cast<const f4u*>(src + min(m, g.M - 4));
          ra[p] = make_float4(v.x, v.y, v.z, v.w);
        }
        if (past) ra[p] = make_float4(0.f, 0.f, 0.f, 0.f);
        q[p] += dq;
        rem[p] += dr;
        if (rem[p] >= per) {
          rem[p] -= per;
          ++q[p];
        }
      }
      fetch_entries();
    }
#pragma unroll
    for (int p = 0; p < B_VECS; ++p) {
      const int f = tid + 256 * p;
      if (B_KCONT) {  // (K is a multiple of the k tile: a hidden width, or two or three of them)
        const int64_t k = k0 + 4 * (f & 7), n = n0 + (f >> 3);
        rb[p] = *reinterpret_cast<const float4*>(g.B + min(n, g.N - 1) * g.ldb + min(k, k_end - 4));
      } else {
        const int64_t k = k0 + b_row(p), n = n0 + b_col(p);
        const float4 v = *reinterpret_cast<const float4*>(g.B + min(k, k_end - 1) * g.ldb + min(n, g.N - 4));
        rb[p] = k < k_end ? v : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
  };
  auto stage = [&](auto any) {
    constexpr bool ANY = decltype(any)::value;
#pragma unroll
    for (int p = 0; p < A_VECS; ++p) {
      const int f = tid + 256 * p;
      if (!A_KCONT && !AVEC) {
        const int64_t m = m0 + 4 * (f % (BM / 4));
        const int move = (int)(m - min(m, g.M - 4));
        if (move & 1) ra[p] = make_float4(ra[p].y, ra[p].z, ra[p].w, ra[p].w);
        if (move & 2) ra[p] = make_float4(ra[p].z, ra[p].w, ra[p].w, ra[p].w);
      }
      store_split4<ANY>(A_KCONT ? &As[(f >> 3) * PK + 4 * (f & 7)] : &As[(f / (BM / 4)) * PMA + 4 * (f % (BM / 4))], A_PLANE, ra[p]);
    }
#pragma unroll
    for (int p = 0; p < B_VECS; ++p) {
      const int f = tid + 256 * p;
      store_split4<ANY>(B_KCONT ? &Bs[(f >> 3) * PK + 4 * (f & 7)] : &Bs[b_row(p) * PNB + b_col(p)], B_PLANE, rb[p]);
    }
  };

  // TN: column sums of B (the bias gradient) ride along: each thread adds up the values it stages
  float4 bsum[BCH];
  const bool want_bsum = MODE == GEMM_TN && g.colsum != nullptr && bx == 0;

  floatx16 acc[TM][TN];
  const bf16_t* const a_frag = A_KCONT ? As + (wm * (BM / WM) + lo) * PK + 8 * hi : As + wm * (BM / WM) + frag_col_offset(lane, PMA);
  const bf16_t* const b_frag = B_KCONT ? Bs + (wn * (BN / WN) + lo) * PK + 8 * hi : Bs + wn * (BN / WN) + frag_col_offset(lane, PNB);

  auto multiply = [&](auto any) {  // the whole k range; any: the operands may hold values out of split_pair's range
    int64_t kb = k_begin;
    if (decltype(any)::value) kb += opaque_zero();  // no address is kept in registers from one form to the other
    if (!A_KCONT) {
#pragma unroll
      for (int p = 0; p < A_VECS; ++p) {
        const uint32_t k = (uint32_t)kb + (tid + 256 * p) / (BM / 4);
        q[p] = (int)(k / (uint32_t)per);
        rem[p] = (int)(k - q[p] * per);
      }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma unroll
    for (int c = 0; c < BCH; ++c) bsum[c] = make_float4(0.f, 0.f, 0.f, 0.f);
    fetch_entries();
    fetch(kb);
    for (int64_t k0 = kb; k0 < k_end; k0 += BK) {
      stage(any);
      if (MODE == GEMM_TN && want_bsum) {
#pragma unroll
        for (int p = 0; p < B_VECS; ++p) {
          float4& t = bsum[p % BCH];
          t.x += rb[p].x; t.y += rb[p].y; t.z += rb[p].z; t.w += rb[p].w;
        }
      }
      __syncthreads();
      if (k0 + BK < k_end) fetch(k0 + BK);
#pragma unroll
      for (int ks = 0; ks < BK / 16; ++ks) {
        Split8 a[TM], b[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
          a[i] = A_KCONT ? frag_row(a_frag + 32 * i * PK + 16 * ks, A_PLANE) : frag_col(a_frag + 32 * i + 16 * ks * PMA, PMA, A_PLANE);
#pragma unroll
        for (int j = 0; j < TN; ++j)
          b[j] = B_KCONT ? frag_row(b_frag + 32 * j * PK + 16 * ks, B_PLANE) : frag_col(b_frag + 32 * j + 16 * ks * PNB, PNB, B_PLANE);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = mfma_split(a[i], b[j], acc[i][j]);
      }
      __syncthreads();
    }
  };
  multiply(std::false_type{});
  float all = 0.f;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) all = sum_of(all, acc[i][j]);
  if (__builtin_expect(any_in_workgroup(all != all), 0)) multiply(std::true_type{});

  if (MODE == GEMM_TN && want_bsum) {
    // threads with equal tid % BPC hold partial sums of the same columns: combine them through LDS
    float4* red = reinterpret_cast<float4*>(Bs);  // the tile is no longer needed (the loop ended with a barrier)
    static_assert(B_PLANE * 3 * 2 >= 256 * 16 * BCH, "room for the partial column sums");
#pragma unroll
    for (int c = 0; c < BCH; ++c) red[256 * c + tid] = bsum[c];
    __syncthreads();
    constexpr int GROUPS = 256 / BPC;
    if (tid < BN / 4 && n0 + 4 * tid < g.N) {
      const int64_t n = n0 + 4 * tid + g.c_rot, nd = n < g.N ? n : n - g.N;
      const float4* const mine = red + 256 * (tid / BPC) + tid % BPC;
      float4 t = mine[0];
#pragma unroll
      for (int u = 1; u < GROUPS; ++u) {
        const float4 o = mine[u * BPC];
        t.x += o.x; t.y += o.y; t.z += o.z; t.w += o.w;
      }
      if (g.split_out != nullptr) {  // this k split's column sums, directly behind its copy of C
        *reinterpret_cast<float4*>(g.split_out + (int64_t)bz * g.split_count + g.M * g.ldc + nd) = t;
      } else {
        float* dst = g.colsum + nd;
        atomicAdd(dst + 0, t.x); atomicAdd(dst + 1, t.y); atomicAdd(dst + 2, t.z); atomicAdd(dst + 3, t.w);
      }
    }
  }

  // Epilogue (accumulator register r of a lane holds C[8*(r/4) + 4*hi + r%4][lo] of its 32x32 tile).  The biases arrive before the first
  // store: a load that is waited for between the stores waits for all stores before it, and the compiler moves the loads and the
  // arithmetic to where a row is stored (98 304 samples, 128 x 384 with a bias: 98 -> 76 us; 75 x 128 with tanh: 53 -> 38 us).
  float bias[TN];
#pragma unroll
  for (int jn = 0; jn < TN; ++jn) {
    bias[jn] = 0.f;
    if (EPI == EPI_BIAS_TANH || (EPI == EPI_STORE && g.aux_vec != nullptr)) bias[jn] = g.aux_vec[min(n0 + wn * (BN / WN) + jn * 32 + lo, g.N - 1)];
  }
  if (EPI == EPI_BIAS_TANH || EPI == EPI_STORE) {
#pragma unroll
    for (int jn = 0; jn < TN; ++jn) asm volatile("" : "+v"(bias[jn]));
  }
#pragma unroll
  for (int jn = 0; jn < TN; ++jn) {
    const int64_t n = n0 + wn * (BN / WN) + jn * 32 + lo;
    if (n0 + wn * (BN / WN) + jn * 32 >= g.N) continue;  // uniform per wavefront: N is a multiple of 32
    const int64_t nd = MODE == GEMM_TN && n + g.c_rot >= g.N ? n + g.c_rot - g.N : (MODE == GEMM_TN ? n + g.c_rot : n);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int64_t mb = m0 + wm * (BM / WM) + i * 32 + 4 * hi;
      float h[16];  // EPI_DTANH: all of the tile's operands requested before the first is used (C may alias them)
      if (EPI == EPI_DTANH) {
#pragma unroll
        for (int r = 0; r < 16; ++r) h[r] = g.aux_mat[min(mb + 8 * (r / 4) + (r % 4), g.M - 1) * g.ldaux + n];
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t m = mb + 8 * (r / 4) + (r % 4);
        float v = acc[i][jn][r];
        if (EPI == EPI_BIAS_TANH) {
          v = tanh_f32(v + bias[jn]);
        } else if (EPI == EPI_DTANH) {
          v = v * (1.0f - h[r] * h[r]);
        } else if (EPI == EPI_STORE) {
          v += bias[jn];
        }
        if (m < g.M) {
          if (EPI != EPI_ATOMIC_ADD) g.C[m * g.ldc + n] = v;
          else if (g.split_out != nullptr) g.split_out[(int64_t)bz * g.split_count + m * g.ldc + nd] = v;
          else atomicAdd(&g.C[m * g.ldc + nd], v);
        }
      }
    }
  }
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Host-side dispatch.  Every caller's N is a hidden width or three of them (a multiple of 32), its B 16-byte aligned with
// a row pitch that keeps it so; A may start and step at any 4-byte boundary.
// Returns true when the launch wrote its k splits to g.split_out (false: it added to C / colsum directly).
template <int MODE, int EPI, int BM, int BN>
inline void launch_gemm_inst(const GemmArgs& g, bool avec, hipStream_t s) {
  unsigned blocks = (unsigned)(((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN));
  if (MODE == GEMM_TN) blocks *= (unsigned)((g.K + g.k_per_split - 1) / g.k_per_split);
  if (avec) hipLaunchKernelGGL((gemm_split_kernel<MODE, EPI, BM, BN, true>), dim3(blocks), dim3(256), 0, s, g);
  else hipLaunchKernelGGL((gemm_split_kernel<MODE, EPI, BM, BN, false>), dim3(blocks), dim3(256), 0, s, g);
}
// Tiles of 192 columns for an NN product, by the rounds of 512 workgroups that either width takes: a round of 192 columns costs 1.39 of 128 and
// a round of 64 columns 0.57; one of up to 256 workgroups, one per CU, three quarters of a full one.  135 products of 1024 .. 262 144
// rows x 192 .. 960 columns: those chosen take 0.75 .. 1.01 of the other width's time; of those left out 1.05 .. 2 times it up to
// 8192 rows (3072 x 384 x 128 13.2 us, 192 columns 17.3), 1.05 .. 0.96 above (50 000 x 384 x 128 42.0, 44.2).
inline bool nn_wide(int64_t M, int64_t N) {
  if (N % 192 != 0) return false;
  const int64_t rows = (M + 127) / 128;
  auto rounds = [](int64_t tiles) { return (double)(tiles / 512) + (tiles % 512 == 0 ? 0.0 : tiles % 512 <= 256 ? 0.75 : 1.0); };
  const double other = N % 128 == 0 ? rounds(rows * (N / 128)) : 0.57 * rounds(rows * (N / 64));
  return 1.39 * rounds(rows * (N / 192)) < other;
}
template <int MODE, int EPI>
inline bool launch_gemm(const GemmArgs& g_in, hipStream_t s) {
  GemmArgs g = g_in;
  const int64_t M = g.M, N = g.N;
  TimedLaunch timed(MODE == GEMM_NN ? KC_GEMM_NN : (MODE == GEMM_NT ? KC_GEMM_NT : KC_GEMM_TN),
                    2.0 * (double)g.M * (double)g.N * (double)g.K, s);
  const bool avec = aligned16(g.A.base) && g.A.ld % 4 == 0 && (MODE == GEMM_TN ? M % 4 == 0 : g.K % 4 == 0);
  if (!(MODE == GEMM_TN && EPI == EPI_ATOMIC_ADD && g.ldc == N && N % 4 == 0)) g.split_out = nullptr;
  if constexpr (MODE == GEMM_TN) {
    const TnPlan p = tn_plan(M, N, g.K);
    g.k_per_split = p.per;
    if (p.wide) launch_gemm_inst<MODE, EPI, 128, 192>(g, avec, s);
    else if (p.bm == 32) launch_gemm_inst<MODE, EPI, 32, 128>(g, avec, s);
    else if (p.bm == 96) launch_gemm_inst<MODE, EPI, 96, 128>(g, avec, s);
    else if (p.bm == 160) launch_gemm_inst<MODE, EPI, 160, 128>(g, avec, s);
    else if (p.bn == 128) launch_gemm_inst<MODE, EPI, 128, 128>(g, avec, s);
    else launch_gemm_inst<MODE, EPI, 128, 64>(g, avec, s);
    return g.split_out != nullptr;
  }
  // 64 columns where 128 would leave a half-empty last tile
  if constexpr (MODE == GEMM_NN) {
    if (nn_wide(M, N)) {
      launch_gemm_inst<MODE, EPI, 128, 192>(g, avec, s);
      return false;
    }
  }
  if (N % 128 == 0) launch_gemm_inst<MODE, EPI, 128, 128>(g, avec, s);
  else launch_gemm_inst<MODE, EPI, 128, 64>(g, avec, s);
  return g.split_out != nullptr;
}

}  // namespace marl
