// fp32 values as sums of three bf16 numbers for products on the bf16 matrix
// cores (device code only).
//
// x = hi + mid + lo: hi is x rounded to bf16 (nearest even), mid the remainder
// rounded, lo the remainder of that: 8 + 8 + 8 bits, all of x's from 2^-110 on.
// (Below, the last piece leaves bf16's range: relative error 2.4e-7 at 2^-112,
// 6e-5 at 2^-120, 2e-3 at 2^-125; an absolute error under 2^-133 everywhere.)
// A product a b is taken as its six partial products whose size reaches fp32's
// own rounding,
//   ah bh + (ah bm + am bh + am bm + ah bl + al bh).
// Where it passes fp32's range, the small ones may pass it with the other
// sign: the convolutions, which sum them apart, then drop them and give
// infinity as fp32 does; the weight gradients, with one sum for all, NaN.  An
// infinity times another is NaN in both.
#pragma once
#include "internal.h"

namespace lnm {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));

// pieces (hi 0, mid 1, lo 2) of the two operands: the small products, then
// the large one
constexpr int kSplitTerm[6][2] = {{0, 2}, {2, 0}, {1, 1}, {0, 1}, {1, 0}, {0, 0}};

__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{a, b}, bf16x2));
}
__device__ __forceinline__ float bf_lo(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float bf_hi(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }

struct Pieces {
  u2 hi, mid, lo;  // four bf16 each
};

// Values from kOver on round to infinity in bf16.  The general form (SAFE)
// takes them too: a finite one keeps its leading bits as hi (truncated, so
// the remainder is exact as well); an infinity goes to lo alone, which meets
// only the other operand's hi, so its products have the signs that fp32's
// have.  (A NaN makes NaN of every product either way.)
constexpr float kOver = 0x1.ffp127f;
// The plain form makes `over` NaN where a value was >= kOver, infinite or NaN
// (its last remainder is then inf - inf; two multiply-adds where comparing the
// four values takes ten instructions).  `over` can overflow without such a
// value, never miss one.
template <bool SAFE>
__device__ __forceinline__ Pieces split(f4 v, float& over) {
  Pieces p;
  f4 h = v, m;
  if constexpr (SAFE) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (fabsf(v[e]) >= kOver) h[e] = __uint_as_float(__float_as_uint(v[e]) & 0xffff0000u);
      if (fabsf(v[e]) == INFINITY) h[e] = 0.0f;
    }
  }
  p.hi = u2{pk_bf16(h.x, h.y), pk_bf16(h.z, h.w)};
  f4 r = f4{v.x - bf_lo(p.hi.x), v.y - bf_hi(p.hi.x), v.z - bf_lo(p.hi.y), v.w - bf_hi(p.hi.y)};
  m = r;
  if constexpr (SAFE) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (fabsf(v[e]) == INFINITY) m[e] = 0.0f;
  }
  p.mid = u2{pk_bf16(m.x, m.y), pk_bf16(m.z, m.w)};
  r = f4{r.x - bf_lo(p.mid.x), r.y - bf_hi(p.mid.x), r.z - bf_lo(p.mid.y), r.w - bf_hi(p.mid.y)};
  p.lo = u2{pk_bf16(r.x, r.y), pk_bf16(r.z, r.w)};
  if constexpr (!SAFE) over = __builtin_fmaf(r.x, r.y, __builtin_fmaf(r.z, r.w, over));
  return p;
}

}  // namespace lnm
