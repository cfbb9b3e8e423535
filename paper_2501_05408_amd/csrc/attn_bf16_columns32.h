// Softmax of 32 (step, head) columns on the accumulators of 32x32x16 products, shared by the prompt kernel
// (attn_prefill_bf16.hip) and the stream kernel (attn_stream_bf16.hip): a lane's logits, weights, sum and
// output all belong to one column, which it shares with lane ^ 32.
#pragma once

#include "attn_bf16_common.h"

namespace tempo {
namespace {

// Three-operand maximum that propagates NaN (v_maximum3_f32).  fmaxf() would first
// canonicalise each matrix-core result, and inline assembly would hide from the compiler that
// it must wait for one.
__device__ inline float max3(float a, float b, float c) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}

// Accumulator tile of a 32x32x16 product: lane (column & 31) + 32 h holds rows
// 8 (r / 4) + 4 h + (r mod 4), r = 0 .. 15.
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Maximum over the two lanes that share a column (l and l ^ 32), left in both.
__device__ inline float half_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return max3(__uint_as_float(r[0]), __uint_as_float(r[1]), __uint_as_float(r[1]));
}
__device__ inline float half_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Maximum of this lane's sixteen logits.  x holds the RAW dot products (masked ones are -inf).
__device__ inline float tile_max(const f32x16& x) {
  const float a = max3(x[0], x[1], x[2]), b = max3(x[3], x[4], x[5]), c = max3(x[6], x[7], x[8]);
  const float d = max3(x[9], x[10], x[11]), e = max3(x[12], x[13], x[14]);
  return max3(max3(a, b, c), max3(d, e, x[15]), x[15]);
}

// Online softmax of one group (lazy reference: kSlack), first half: move the reference if this
// group's maximum calls for it.  A lane's sixteen logits, its accumulators and its share of the sum all belong to ONE column,
// so the rescale factor needs no exchange.  Most groups move nothing, so that case is one
// comparison: of the lane's own raw maximum (the lanes of a column meet only behind the branch)
// with `limit`, the raw dot product from which on the reference has to move.
template <int D>
__device__ inline void softmax_reference(float lane_max, float scale, float& limit, float& ref, float& base, f32x16* acc,
                                         float& sum) {
  if (__any(lane_max > limit)) {
    const float mx = half_max(lane_max) * scale;  // `scale` > 0 is s * log2(e)
    // ref = -inf until the column sees its first key; -inf + kSlack = -inf, so any finite mx moves it
    const bool move = mx > ref + kSlack;
    const float alpha = move ? fast_exp2(ref - mx) : 1.0f;  // exp2(-inf) = 0 on the first key
    ref = move ? mx : ref;
    limit = (ref + kSlack) / scale;
    base = ref == -INFINITY ? 0.f : ref;  // a column that has seen no key yet: weights exp2(-inf - 0) = 0
    sum *= alpha;
#pragma unroll
    for (int ot = 0; ot < D / 32; ++ot) {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ot][r] *= alpha;
    }
  }
}

// Second half: the bf16 weights 2^(scale * x - ref), the scale applied inside one fused
// multiply-add, in the order of the two 16-key steps of the weights x values product:
// a value unit (column tile, c) holds slots 4c .. 4c+3 and 16+4c .. 16+4c+3, and step
// `chunk` gives lane half h the units c = 2 chunk + h, i.e. accumulator registers
// 4 chunk .. +3 and 8 + 4 chunk .. +3 of this lane.  The sum is taken over the rounded
// weights, so the output stays a convex combination of value rows.  One call does logit i
// of sixteen (the odd ones finish a pair), so that the caller can put matrix instructions between them.
__device__ inline void softmax_weight(const f32x16& x, float scale, float base, int i, float& even, u32x4* pa, float& sum) {
  const int chunk = i >> 3, e = i & 7;
  const float w = fast_exp2(fmaf(x[(e < 4 ? e : 4 + e) + 4 * chunk], scale, -base));
  if ((i & 1) == 0) {
    even = w;
    return;
  }
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  const bf16x2 both = {(__bf16)even, (__bf16)w};
  pa[chunk][e >> 1] = __builtin_bit_cast(uint32_t, both);
  sum = __builtin_amdgcn_fdot2_f32_bf16(both, ones, sum, false);
}

// Index mask of a group that some column's range cuts: -inf outside THIS lane's column
// range [lo_col, hi_col].
__device__ inline void mask_tile(int grp, int lo_col, int hi_col, int lane, f32x16& x) {
  const int j0 = (grp << 5) + 4 * (lane >> 5);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int j = j0 + 8 * (r >> 2) + (r & 3);
    x[r] = (j >= lo_col && j <= hi_col) ? x[r] : -INFINITY;
  }
}

}  // namespace
}  // namespace tempo
