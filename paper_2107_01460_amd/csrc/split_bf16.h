// fp32 products on the bf16 matrix cores, at fp32 precision.
//
// An fp32 value is the exact sum of three bf16 values: h = bf16(x), m = bf16(x - h), l = x - h - m (round to nearest:
// |m| <= 2^-8 |x|, |l| <= 2^-17 |x|, and the 24 significant bits of x are used up, so l is a bf16 value itself; below about
// 2^-100 the lower parts underflow, an absolute error below the smallest normal number).  A product of two such sums is nine
// bf16 products, each exact in fp32; the three smallest (m l, l m, l l) are together at most 2^-24 of the product, one of
// fp32's own rounding units, and 2^-27.5 in the root mean square (four million random pairs), and are left out.  The other
// six go to v_mfma_f32_32x32x16_bf16, which accumulates in fp32.  What says that nothing is lost by this are the errors:
//
// Rates measured on an MI355X: v_mfma_f32_32x32x2_f32 137 TFLOP/s, v_mfma_f32_32x32x16_bf16 2050 TFLOP/s, i.e. 342 TFLOP/s
// of fp32 products.  Error against fp64 (tanh activations x normal weights, norm of the error over norm of the result,
// 64 products of 32 x 32 outputs): contraction length 128: 1.63e-7 here, 2.02e-7 with the fp32 instruction; 304: 2.58e-7
// and 3.12e-7; 1024: 4.86e-7 and 5.74e-7 -- the sixteen terms an instruction adds at once round less often.  With all nine
// products the figures are the same in every digit shown.
#pragma once
#include "common.h"

namespace marl {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef short shortx8 __attribute__((ext_vector_type(8)));

// two values, each part packed as two bf16 (the first value in the low half)
struct SplitPair {
  uint32_t h, m, l;
};
// Magnitudes from here on round to infinity in bf16: the only values that split_pair does not represent (a NaN gives NaNs).
constexpr float kSplitLimit = 0x1.ffp127f;
// For values below the limit, such as results of tanh.  split_pair_any takes every value.
__device__ __forceinline__ SplitPair split_pair(float x, float y) {
  SplitPair s;
  s.h = pack2_bf16(x, y);
  x -= __uint_as_float(s.h << 16);
  y -= __uint_as_float(s.h & 0xffff0000u);
  s.m = pack2_bf16(x, y);
  x -= __uint_as_float(s.m << 16);
  y -= __uint_as_float(s.m & 0xffff0000u);
  s.l = pack2_bf16(x, y);
  return s;
}
// A finite value at the limit or above takes the largest bf16 as its first part.  An infinity is (+-1, 0, +-inf): of the six
// products that mfma_split adds, the one of the last part with the other factor's first is then the infinity (a NaN where
// that factor is zero), those of the first part are finite or, from a second infinity, the same infinity, and the middle
// part's are zero -- with the infinity as the first part, infinity times a zero lower part would make every sum a NaN.
// (What is left: a finite product of 2^136 or more, far past the largest fp32 value, may be a NaN instead of an infinity.)
__device__ __forceinline__ SplitPair split_pair_any(float x, float y) {
  auto first = [](float v, uint32_t h) -> uint32_t {
    const uint32_t sign = (__float_as_uint(v) >> 16) & 0x8000u;
    return __builtin_isinf(v) ? 0x3f80u | sign : fabsf(v) >= kSplitLimit ? 0x7f7fu | sign : h & 0xffffu;
  };
  SplitPair s;
  s.h = pack2_bf16(x, y);
  s.h = first(x, s.h) | first(y, s.h >> 16) << 16;
  const float rx = x - __uint_as_float(s.h << 16), ry = y - __uint_as_float(s.h & 0xffff0000u);  // +-inf for an infinity
  s.m = pack2_bf16(__builtin_isinf(x) ? 0.f : rx, __builtin_isinf(y) ? 0.f : ry);
  s.l = pack2_bf16(rx - __uint_as_float(s.m << 16), ry - __uint_as_float(s.m & 0xffff0000u));
  return s;
}
// A value that split_pair does not represent has a NaN among its parts and makes every sum it enters a NaN.  So the kernels
// split with split_pair, look for a NaN in the sums, and where there is one do the work again with split_pair_any.  (Looking
// at the operands took a comparison per value and, in the inner loops, registers: 5 % of a training iteration, this 1 %.)
__device__ __forceinline__ float sum_of(float s, const floatx16& v) {  // (a NaN also where infinities meet: done again for nothing)
#pragma unroll
  for (int r = 0; r < 16; ++r) s += v[r];
  return s;
}
__device__ __forceinline__ bool any_in_workgroup(bool b) { return __builtin_amdgcn_readfirstlane(__syncthreads_or(b)) != 0; }
// Barrier for data exchanged through LDS only: global loads and stores stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// Barrier of a loop's head after LDS writes at the loop's end.  The compiler leaves out the wait for writes that come in over
// the back edge where other lanes' paths end without one (seen in the listing of the rollouts: ds_write, s_branch, s_barrier),
// and the other wavefronts could then read an old value: the wait is written out.  A few cycles where nothing is pending.
__device__ __forceinline__ void loop_head_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __syncthreads();
}
// A zero that the compiler does not know
__device__ __forceinline__ int opaque_zero() {
  int z = 0;
  asm volatile("" : "+v"(z));
  return __builtin_amdgcn_readfirstlane(z);
}
// Does any lane hold one (m: a magnitude; fmaxf passes over NaNs)?
__device__ __forceinline__ bool split_out_of_range(float m) { return __builtin_expect(__builtin_amdgcn_ballot_w64(m >= kSplitLimit) != 0, 0); }
__device__ __forceinline__ float max_abs(float m, float4 v) { return fmaxf(fmaxf(m, fmaxf(fabsf(v.x), fabsf(v.y))), fmaxf(fabsf(v.z), fabsf(v.w))); }

// Eight values along the contraction of one row (A) or column (B): what a lane feeds to one matrix instruction -- of the
// sixteen k of a step, lanes 0 .. 31 hold k = 0 .. 7, lanes 32 .. 63 hold k = 8 .. 15.
struct Split8 {
  bf16x8 h, m, l;
};

template <bool ANY>
__device__ __forceinline__ SplitPair split_two(float x, float y) { return ANY ? split_pair_any(x, y) : split_pair(x, y); }
// acc += A B over sixteen k (the small products first)
__device__ __forceinline__ floatx16 mfma_split(const Split8& a, const Split8& b, floatx16 acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.l, b.h, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.l, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.m, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.h, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.m, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.h, acc, 0, 0, 0);
  return acc;
}

// ---- operands in LDS: three planes (h, m, l) of bf16, `plane` elements apart ------------------------------------------
// Four consecutive values to the three planes with 8-byte stores.
template <bool ANY>
__device__ __forceinline__ void store_split4(bf16_t* dst, int plane, float4 v) {
  const SplitPair a = split_two<ANY>(v.x, v.y), b = split_two<ANY>(v.z, v.w);
  *reinterpret_cast<uint2*>(dst) = make_uint2(a.h, b.h);
  *reinterpret_cast<uint2*>(dst + plane) = make_uint2(a.m, b.m);
  *reinterpret_cast<uint2*>(dst + 2 * plane) = make_uint2(a.l, b.l);
}
// Fragment of a tile stored with the contraction contiguous: p points at this lane's row, k = 16 step + 8 (lane / 32).
__device__ __forceinline__ Split8 frag_row(const bf16_t* p, int plane) {
  Split8 f;
  f.h = *reinterpret_cast<const bf16x8*>(p);
  f.m = *reinterpret_cast<const bf16x8*>(p + plane);
  f.l = *reinterpret_cast<const bf16x8*>(p + 2 * plane);
  return f;
}
// Fragment of a tile stored with the contraction along the rows ([k][column]): the transposing LDS read gives each of the
// sixteen lanes of a group one column of a 4 x 16 block whose rows the group's lanes address four elements at a time.
// p points at frag_col_offset(lane, pitch) past the element (first k of the step, first of the 32 columns).
__device__ __forceinline__ int frag_col_offset(int lane, int pitch) {
  return (8 * (lane >> 5) + ((lane & 15) >> 2)) * pitch + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
}
__device__ __forceinline__ bf16x8 read_col8(const bf16_t* p, int pitch) {
  typedef __attribute__((address_space(3))) shortx4 lds_shortx4;
  const shortx4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)p);
  const shortx4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)(p + 4 * pitch));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}
__device__ __forceinline__ Split8 frag_col(const bf16_t* p, int pitch, int plane) {
  Split8 f;
  f.h = read_col8(p, pitch);
  f.m = read_col8(p + plane, pitch);
  f.l = read_col8(p + 2 * plane, pitch);
  return f;
}

}  // namespace marl
