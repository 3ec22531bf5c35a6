// What the kernels that locate inputs share: steps 1-4 of Sec. 4.5 with the domain test of Sec. 5.2 for one (row, input), and
// the interpolation of byte codes.  Included by files compiled with -ffp-contract=off.
#pragma once

#include "lutkan_device.h"

namespace {

__device__ __forceinline__ f16x2 bits_to_f16x2(unsigned v) {
  union { unsigned u; f16x2 h; } c;
  c.u = v;
  return c.h;
}

struct Located {
  int k, l0;
  float w;
  bool inside, is_nan;
};


// s_knots: the K+1 knots of this element's input in LDS.  With one vector per layer (PERIN false) the comparisons
// run against the copy in the kernel arguments (scalar registers) and LDS serves the two lookups by the lane's own
// segment index; with one vector per input every lane reads its own input's row.
template <bool PERIN, typename Args>
__device__ __forceinline__ Located locate_one(const Args &a, const float *s_knots, float x) {
  Located o;
  const float t0 = PERIN ? s_knots[0] : a.knots[0];
  const float tK = PERIN ? s_knots[a.K] : a.knots[a.K];
  const float tKs = PERIN ? (a.closed ? tK : next_float_below(tK)) : a.tKs;
  o.is_nan = (x != x);
  o.inside = a.closed ? (x >= t0 && x <= tK) : (x >= t0 && x < tK);
  float xc = o.is_nan ? t0 : x;
  xc = (xc < t0) ? t0 : xc;
  xc = (xc > tKs) ? tKs : xc;
  // k = #{kappa in 1..K-1 : T[kappa] <= x'}; T[0] <= x' always holds and T[K] is clipped away (Eq. 14).
  int k = 0;
  for (int kappa = 1; kappa < a.K; ++kappa) k += ((PERIN ? s_knots[kappa] : a.knots[kappa]) <= xc) ? 1 : 0;
  const float tk = s_knots[k], tk1 = s_knots[k + 1];
  const float num = __fsub_rn(xc, tk);
  const float den = __fsub_rn(tk1, tk);
  const float u = __fdiv_rn(num, den);                       // Eq. 15, correctly rounded
  const float z = __fmul_rn(u, (float)(a.L - 1));            // Eq. 16
  int l0 = (int)floorf(z);
  l0 = min(max(l0, 0), a.L - 1);
  o.k = k;
  o.l0 = l0;
  o.w = __fsub_rn(z, (float)l0);
  return o;
}

// Eq. 15 by a reciprocal that every segment keeps: num / den correctly rounded from y = RN(1/den) in five operations -- a
// quotient within two units, one correction that makes it faithful, one that rounds it correctly (Markstein's theorem: q + r y,
// rounded once, is the rounded a/b if r = a - b q is exact, q faithful and y = RN(1/b)) -- where the compiler's division takes
// eleven and a hardware reciprocal.  r is exact while num >= 2^-90 and den lies in [2^-30, 2^30]; other pairs are divided.
constexpr unsigned kPlainNumerator = 0x12800000u;      // 2^-90
__device__ __forceinline__ float quotient(float num, float den, float y) {
  const float q0 = __fmul_rn(num, y);
  const float q1 = fmaf(fmaf(-q0, den, num), y, q0);
  return fmaf(fmaf(-q1, den, num), y, q1);
}

// The rows that the second locate_side_by_side looks up, in LDS: of segment k its first knot, width (rounded as Eq. 15 rounds it) and the
// width's reciprocal.  fill_segments covers segments 0 .. K-1 with the threads of a work-group.
template <typename Args>
__device__ __forceinline__ void fill_segments(const Args &a, f32x4 *s_seg, int tid) {
  if (tid >= a.K) return;
  const float tk = a.knots[tid], den = __fsub_rn(a.knots[tid + 1], tk);
  s_seg[tid] = f32x4{tk, den, __fdiv_rn(1.0f, den), 0.0f};
}
// A numerator whose bits - 1 are at most this is divided instead: one below 2^-90 (0, whose bits - 1 wrap round, is not: its quotient
// by a plain width is 0), or every one, 0 included, if a width is not plain: its reciprocal may be 0 or infinite.
inline unsigned last_divided(const float *knots, int K) {
  for (int k = 0; k < K; ++k) {
    const float den = knots[k + 1] - knots[k];
    if (!(den >= 0x1p-30f && den <= 0x1p30f)) return 0xffffffffu;
  }
  return kPlainNumerator - 2;
}

// Steps 1-4 of Sec. 4.5 for VEC inputs side by side: the arithmetic of locate_one (same results to the bit) without its
// branches.  In(x) is t0 <= x <= tKs under either boundary mode.  The knots above x' are counted by the sign of x' - T
// (exact; +inf past the last knot), shifted into a word: two instructions a knot and no condition register.  Ten segments are
// searched without a loop, their knots in scalar registers; more in steps of eight.  FEW = 4: grids of up to five segments stop there.
template <int VEC, int FEW, typename Args>
__device__ __forceinline__ void clip_and_search(const Args &a, const float x[VEC], float xc[VEC], int k[VEC]) {
  constexpr int kFirst = 9;
  unsigned above[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) {
    xc[v] = __builtin_amdgcn_fmed3f(x[v], a.t0, a.tKs) + 0.0f;   // (a NaN comes out inside and is put back in w; -0 becomes
    above[v] = 0;                                                  // +0, whose difference from a knot at 0 has no sign bit)
#pragma unroll
    for (int q = 0; q < FEW; ++q) above[v] = __builtin_amdgcn_alignbit(above[v], __float_as_uint(xc[v] - a.inner[q]), 31);
    k[v] = FEW - __popc(above[v]);
  }
  if (FEW == kFirst || a.K > FEW + 1) {                  // uniform
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
#pragma unroll
      for (int q = FEW; q < kFirst; ++q) above[v] = __builtin_amdgcn_alignbit(above[v], __float_as_uint(xc[v] - a.inner[q]), 31);
      k[v] = kFirst - __popc(above[v]);
    }
#pragma unroll 1
    for (int g = kFirst; g < a.K - 1; g += 8) {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float knot = a.inner[min(g + q, LUTKAN_MAX_K - 1)];
#pragma unroll
        for (int v = 0; v < VEC; ++v) k[v] += (knot <= xc[v]) ? 1 : 0;
      }
    }
  }
}

template <int VEC, typename Args>
__device__ __forceinline__ void round_down(const Args &a, const float x[VEC], const float u[VEC], int l0[VEC], float w[VEC]) {
#pragma unroll
  for (int v = 0; v < VEC; ++v) {
    const float z = __fmul_rn(u[v], (float)(a.L - 1));                                 // Eq. 16; 0 <= u <= 1
    const float below = floorf(z);
    l0[v] = (int)below;
    w[v] = (x[v] != x[v]) ? __builtin_nanf("") : __fsub_rn(z, below);
  }
}

// Eq. 15 divided, from the knots in LDS: for threads that locate one or two elements.  The segments' rows below cost a work-group a
// division ahead of its first barrier, and FEW = 4 one more wait for the knots, which so few elements do not pay for: launches
// replayed, with them -> so, microseconds: 11 -> 880 at 422 rows 17.12 -> 16.92, 9 -> 66 -> 249 at 805 25.9 -> 25.5, 10 -> 93 at 1104
// 10.03 -> 9.88, 24 -> 243 at 2620 18.6 -> 18.4.
template <int VEC, typename Args>
__device__ __forceinline__ void locate_side_by_side(const Args &a, const float *s_knots, const float x[VEC], int k[VEC], int l0[VEC], float w[VEC]) {
  float xc[VEC], u[VEC];
  clip_and_search<VEC, 9>(a, x, xc, k);
#pragma unroll
  for (int v = 0; v < VEC; ++v) {
    const float tk = s_knots[k[v]], tk1 = s_knots[k[v] + 1];
    u[v] = __fdiv_rn(__fsub_rn(xc[v], tk), __fsub_rn(tk1, tk));                        // correctly rounded
  }
  round_down<VEC>(a, x, u, l0, w);
}

// Eq. 15 by the segments' reciprocals: for threads that locate eight elements, or input after input (78 -> 16 at 65536 rows 34.6 ->
// 31.1; a chain of three locate passes at 131072 rows 595 -> 592).
template <int VEC, typename Args>
__device__ __forceinline__ void locate_side_by_side(const Args &a, const f32x4 *s_seg, const float x[VEC], int k[VEC], int l0[VEC], float w[VEC]) {
  float xc[VEC], num[VEC], den[VEC], u[VEC];
  clip_and_search<VEC, 4>(a, x, xc, k);
  unsigned smallest = 0xffffffffu;
#pragma unroll
  for (int v = 0; v < VEC; ++v) {
    const f32x4 seg = s_seg[k[v]];
    num[v] = __fsub_rn(xc[v], seg.x);
    den[v] = seg.y;
    u[v] = quotient(num[v], den[v], seg.z);                                            // correctly rounded
    smallest = min(smallest, __float_as_uint(num[v]) - 1u);
  }
  if (smallest <= a.last_divided) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) u[v] = __fdiv_rn(num[v], den[v]);
  }
  round_down<VEC>(a, x, u, l0, w);
}

// Eq. 17 on the four codes of a lane (one dword of table row l0, one of row l0+1) as t = (q0 + w * (q1 - q0)) * 2^-24: a byte
// zero-extended to 16 bits is the binary16 denormal byte * 2^-24, so the difference and the removal of the excess-128 bias of
// symmetric codes are exact packed arithmetic and the interpolation has one fp32 rounding.
template <int SCHEME>
__device__ __forceinline__ void interpolate_codes(unsigned c0, unsigned c1, float w, float t[4]) {
  f16x2 q0lo = bits_to_f16x2(__builtin_amdgcn_perm(c0, c0, 0x0c010c00u)), q0hi = bits_to_f16x2(__builtin_amdgcn_perm(c0, c0, 0x0c030c02u));
  const f16x2 q1lo = bits_to_f16x2(__builtin_amdgcn_perm(c1, c1, 0x0c010c00u)), q1hi = bits_to_f16x2(__builtin_amdgcn_perm(c1, c1, 0x0c030c02u));
  const f16x2 dlo = q1lo - q0lo, dhi = q1hi - q0hi;
  if (SCHEME == LUTKAN_SYM_INT8) {
    const f16x2 bias = bits_to_f16x2(0x00800080u);
    q0lo = q0lo - bias;
    q0hi = q0hi - bias;
  }
  t[0] = fmaf(w, (float)dlo.x, (float)q0lo.x);
  t[1] = fmaf(w, (float)dlo.y, (float)q0lo.y);
  t[2] = fmaf(w, (float)dhi.x, (float)q0hi.x);
  t[3] = fmaf(w, (float)dhi.y, (float)q0hi.y);
}

}  // namespace
