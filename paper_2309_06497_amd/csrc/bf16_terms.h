// Float32 operands of the matrix cores as three bf16 terms, split in registers (the same terms as bf16_planes.h keeps in
// memory).  An operand of a 32 x 32 x 16 product is 8 values of k of one row or column per lane: lane = row % 32 + 32 (k / 8).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "lds_dma.h"

namespace shampoo {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx8 __attribute__((ext_vector_type(8)));
// x = h + l + m, eight elements: 8 + 8 + 8 bits
struct Bf16Terms { bf16x8 h, l, m; };
// two of them rounded, and what that leaves (written out: from vector conversions the compiler makes every one twice)
__device__ __forceinline__ uint32_t bf16_round2(float &x, float &y, bool left) {
  typedef float pair __attribute__((ext_vector_type(2)));
  typedef __bf16 bpair __attribute__((ext_vector_type(2)));
  const uint32_t u = __builtin_bit_cast(uint32_t, __builtin_convertvector(pair{x, y}, bpair));
  if (left) { x -= __uint_as_float(u << 16); y -= __uint_as_float(u & 0xffff0000u); }
  return u;
}
template <bool ONE>      // ONE: x holds bf16 values
__device__ __forceinline__ void bf16_split(floatx8 x, Bf16Terms &t) {
  u32x4 h, l, m;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float a = x[2 * e], b = x[2 * e + 1];
    h[e] = bf16_round2(a, b, !ONE);
    if constexpr (!ONE) { l[e] = bf16_round2(a, b, true); m[e] = bf16_round2(a, b, false); }
  }
  t.h = __builtin_bit_cast(bf16x8, h);
  if constexpr (!ONE) { t.l = __builtin_bit_cast(bf16x8, l); t.m = __builtin_bit_cast(bf16x8, m); }
}
__device__ __forceinline__ floatx16 bf16_mfma(const bf16x8 &a, const bf16x8 &b, const floatx16 &c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// The products of two splits, smallest first, but for h h': five, or fewer where one side has a single term.
template <bool AONE, bool BONE>
__device__ __forceinline__ floatx16 bf16_small_products(const Bf16Terms &a, const Bf16Terms &b, floatx16 c) {
  if constexpr (!BONE) c = bf16_mfma(a.h, b.m, c);
  if constexpr (!AONE) c = bf16_mfma(a.m, b.h, c);
  if constexpr (!AONE && !BONE) c = bf16_mfma(a.l, b.l, c);
  if constexpr (!BONE) c = bf16_mfma(a.h, b.l, c);
  if constexpr (!AONE) c = bf16_mfma(a.l, b.h, c);
  return c;
}
// The same sixteen values of k on the float32 matrix cores: a product is a sum over k in any order, as long as both
// operands have the same one.
__device__ __forceinline__ floatx16 fp32_products(const floatx8 &a, const floatx8 &b, floatx16 c) {
#pragma unroll
  for (int e = 0; e < 8; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], c, 0, 0, 0);
  return c;
}

// Element (i, k .. k + 7) of an operand in LDS, read along rows: two 16-byte reads (rows are 16-byte aligned and 4 banks
// apart: the 16 lanes that are served at a time cover the 64 banks).
template <int LD> __device__ __forceinline__ floatx8 lds_row8(const float *Gs, int i, int k) {
  const float4 x = *reinterpret_cast<const float4 *>(Gs + i * LD + k), y = *reinterpret_cast<const float4 *>(Gs + i * LD + k + 4);
  return floatx8{x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
}
// (k .. k + 7, j), read down a column: eight 4-byte reads, whose two half wavefronts are 32 banks apart
template <int LD> __device__ __forceinline__ floatx8 lds_col8(const float *Gs, int k, int j) {
  floatx8 x;
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = Gs[(k + e) * LD + j];
  return x;
}
// A power of two that brings a largest element outside 2^-40 ... 2^40 to 0.5 ... 1, so that neither the small terms nor their
// products underflow; otherwise 1.  For products with gradients, whose size is the caller's.  The others go without: elements below about
// 2^-110 of theirs lose the third term, which is 2^-16 of the element.  Newton's iterates are around 1, or around the
// root itself; F on the way back of a root is f of the spectrum; the second product of diagonal Shampoo takes D G, and where that is so
// small, the norm of the direction, a sum of squares in float32, is zero for any root below 1e10, and with it the step.
__device__ __forceinline__ float range_scale(float largest) {
  if (!(largest > 0.f) || !(largest < 3.4e38f) || (largest >= 0x1p-40f && largest <= 0x1p40f)) return 1.f;
  int e;
  (void)frexpf(largest, &e);
  return ldexpf(1.f, min(-e, 120));
}

}  // namespace shampoo
