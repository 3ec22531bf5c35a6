// The cut of fp32 operands into bf16 pieces for the matrix instructions, shared by the locate kernel (lutkan_kernels.hip),
// the base-branch product (lutkan_base_gemm.hip) and the B-spline layer (bspline_matrix.hip).
#pragma once

#include <hip/hip_runtime.h>

// a = h + m + l exactly for finite a: h is a rounded to bf16, m the rest rounded to bf16, l what is left of that (24
// significand bits = 8 + 8 + 8, each rest with a sign of its own).  |m| <= 2^-8 and |l| <= 2^-17 of a's binade, so of the nine
// piece products of two operands the three that are not computed (m l, l m, l l) are at most 2^-24 of the product together, with
// either sign.  (Pieces by truncation: up to 2^-21, always towards zero.)  Rounding costs what truncation did: the
// conversion packs two values.

typedef float lutkan_cut_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 lutkan_cut_bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned lutkan_round_bf16_pair(float a0, float a1) {
  union { lutkan_cut_bf16x2 h; unsigned u; } c;
  c.h = __builtin_convertvector(lutkan_cut_f32x2{a0, a1}, lutkan_cut_bf16x2);      // to nearest, ties to even
  return c.u;
}

constexpr float kLargestBf16 = 3.3895313892515355e38f;

// The pieces of two values, packed (a0 in the lower halves): p[0] = h, p[1] = m, p[2] = l.  A value beyond the largest bf16 value
// may round to an infinite h; it, an infinity and a NaN leave an infinity or a NaN among the pieces.
__device__ __forceinline__ void lutkan_cut3_pair(float a0, float a1, unsigned p[3]) {
  p[0] = lutkan_round_bf16_pair(a0, a1);
  const float r0 = a0 - __uint_as_float(p[0] << 16), r1 = a1 - __uint_as_float(p[0] & 0xffff0000u);
  p[1] = lutkan_round_bf16_pair(r0, r1);
  p[2] = lutkan_round_bf16_pair(r0 - __uint_as_float(p[1] << 16), r1 - __uint_as_float(p[1] & 0xffff0000u));
}

// One value's pieces as bit patterns.  Beyond the largest bf16 value h is that value and the rest is still exact; inf and NaN
// keep their class in the high piece, the other two are zero.
__device__ __forceinline__ void lutkan_cut3(float a, unsigned &h, unsigned &m, unsigned &l) {
  const unsigned ab = __float_as_uint(a);
  if ((ab & 0x7f800000u) == 0x7f800000u) {
    h = (ab >> 16) | ((ab & 0x007fffffu) ? 0x0040u : 0u);
    m = l = 0u;
    return;
  }
  h = lutkan_round_bf16_pair(__builtin_amdgcn_fmed3f(a, -kLargestBf16, kLargestBf16), 0.0f) & 0xffffu;
  const float r = a - __uint_as_float(h << 16);
  m = lutkan_round_bf16_pair(r, 0.0f) & 0xffffu;
  l = lutkan_round_bf16_pair(r - __uint_as_float(m << 16), 0.0f) & 0xffffu;
}
