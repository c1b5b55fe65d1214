// fp32 products on the bf16 matrix cores.
//
// An fp32 value is the sum of three bf16 ones, x = h + m + l (h = bf16(x),
// m = bf16(x - h), l = x - h - m: 8 + 8 + 8 bits, the differences exact), and a
// product of two is h h' + h m' + m h' + m m' + h l' + l h' to within 2^-25 of
// it: six exact products accumulated in fp32 by v_mfma_f32_32x32x16_bf16, of
// which the card does sixteen in the time of one fp32 matrix product.  Inputs
// that are infinite, or that round to infinity in bf16, and sums that overflow
// leave infinities or NaN in the result: a kernel checks for those and forms
// such blocks with the fp32 instruction instead.
#pragma once

#include "jarq_internal.h"

namespace jarq {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16 mfma_bf16(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// x = h + m + l of two values (one per half of each word)
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t& h, uint32_t& m,
                                           uint32_t& l) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  auto cvt = [](float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
  };
  auto lo = [](uint32_t w) { return __uint_as_float(w << 16); };
  auto hi = [](uint32_t w) { return __uint_as_float(w & 0xffff0000u); };
  h = cvt(x0, x1);
  const float r0 = x0 - lo(h), r1 = x1 - hi(h);
  m = cvt(r0, r1);
  l = cvt(r0 - lo(m), r1 - hi(m));
}

// big[a] + small[a] += A_a B for the planes (h, m, l) of AB row blocks and one
// column block: the leading products in one sum, the five small ones in
// another, so that only one of six roundings is at the size of the result.
template <int AB>
__device__ __forceinline__ void mfma_bf16x3(const bf16x8 (&fa)[AB][3], const bf16x8 (&fb)[3],
                                            f32x16 (&big)[AB], f32x16 (&small)[AB]) {
  constexpr int pa[5] = {2, 0, 1, 1, 0}, pb[5] = {0, 2, 1, 0, 1};
#pragma unroll
  for (int t = 0; t < 5; ++t)
#pragma unroll
    for (int a = 0; a < AB; ++a) small[a] = mfma_bf16(fa[a][pa[t]], fb[pb[t]], small[a]);
#pragma unroll
  for (int a = 0; a < AB; ++a) big[a] = mfma_bf16(fa[a][0], fb[0], big[a]);
}

}  // namespace jarq
