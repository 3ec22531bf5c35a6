// The B-spline layer as a dense contraction on the matrix cores:
//     y[b][j] = sum_i sum_r N_r(x[b][i]) * c[i][r][j]
// with the R = G + 3 basis values of an input as contraction index (four of them are non-zero).  The tiled kernel
// (bspline_kernels.hip) spends four multiply-adds per edge and is bound by the 16 bytes of coefficients per edge that it
// reads from LDS at a row's own offset; here the coefficients are the second operand of a matrix instruction, read from
// LDS once per 32 rows, and the price is the zeros: R (padded to 8 or 16 slots) products per edge instead of 4.
// The basis is evaluated where it is consumed, so the pass that writes and reads 32 bytes per (row, input) falls away.
//
// fp32 accuracy from bf16 matrix instructions, as in lutkan_base_gemm.hip: every fp32 operand is cut exactly into three
// bf16 pieces and six of the nine piece products are accumulated in fp32; the other three are at most 2^-24 of the product
// together (lutkan_pieces.h).  The products
// of the two high pieces have an accumulator of their own, apart from the five small ones: with one accumulator for all
// six, every small product rounds the large sum once more and the layer came out 1.2 - 1.8 times further from a 64-bit
// evaluation than the tiled kernel; apart, it is nearer than that kernel (64 -> 128 at 131072 rows 1.5e-7 against 3.0e-7,
// 1024 -> 1024 at 4096 rows, G = 10, 4.8e-7 against 5.7e-7).
//
// Operand A without LDS: in v_mfma_f32_32x32x16_bf16 a lane holds 8 consecutive k of one row, and k may be numbered
// freely as long as both operands agree, so k is numbered such that a lane's 8 slots belong to ONE input of its row:
//   SLOTS = 8   (R <= 8)   a k step covers two inputs, the lower lanes' and the upper lanes' one; a lane's slots are the
//                          input's 8 coefficient rows
//   SLOTS = 16  (R <= 16)  a k step covers one input; the lower lanes hold its even coefficient rows, the upper lanes
//                          the odd ones (two of the four non-zero values each)
// A lane thus locates its (row, input), evaluates the four cubics and shifts their pieces into its slots in registers.
// Operand B (coefficients): a work-group stages 8 (SLOTS 16: 4) inputs at a time, cut into pieces on the way into LDS, as
// [unit][piece][column][8 slots]; unit = input (SLOTS 16: input and parity), k step s reads units s and s + 4.
//
// A work-group is 8 waves of 32*RT rows x 32*NT columns (one column tile of the coefficient table); two waves share a
// SIMD, so that one's vector work (basis, pieces) overlaps the other's matrix instructions.
//
// Bound: the matrix cores at the clock they leave the chip.  96 (SLOTS 16: 192) flop per edge; 1024 -> 1024 at 32768 rows,
// G = 5: 3.30 TFLOP in 2.70 ms = 1.22 PFLOP/s, what a bf16 library product of 8192^3 reaches on such a card, against 6.16 ms on
// the tiled kernel.  In one run under counters 2.88 ms at 1.83 GHz: matrix pipes 0.60 busy (1.15 PFLOP/s), vector issue 0.41, LDS
// 0.24.
// Whole layers, tiled -> matrix, microseconds (one run; boards and runs differ by 5 %): 128 -> 128 at 131072 rows, G = 5,
// 587 -> 182; 64 -> 8 162 -> 34; 256 -> 256 at 16384 rows 273 -> 104 (G = 5), 272 -> 183 (G = 8); 1024 -> 1024, G = 10, at 4096 rows
// 790 -> 684, at 32768 6290 -> 5250; 128 -> 128 at 64 rows 19 -> 13.  Exchanging lanes so that each half of a wave evaluates the
// basis of every other input only (SLOTS 16) gave nothing, nor did records from a locate pass of its own (1024 -> 1024 at 4096
// rows 634 against 635).
// The file is compiled with -ffp-contract=off; fused multiply-adds are written out as fmaf().
#include "bspline_matrix.h"
#include "lutkan_device.h"
#include "lutkan_pieces.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kMxWaves = 8;
constexpr int kMxMaxSegments = 13;       // R = G + 3 <= 16
constexpr int kMxSegFloats = 14;         // of a segment: 8 polynomial coefficients, its ends, middle and scale, the two outer factors
constexpr int kMxSegStride = 20;         // ... in LDS: 80-byte rows spread the banks
constexpr int kMxLdsTail = (kMxMaxSegments + 1) * (kMxSegStride * 4 + 2 * 16) + 16;      // behind the stages in LDS: segments, places, a flag

struct SplineMatrixArgs {
  const float *x;            // [B][d]
  const float *coef_table;   // [t][i][R][jt]
  float *y;
  int64_t B;
  int32_t d, m, R, segments, jt, n_tiles;
  int32_t x_vec4;            // rows of x are whole aligned 16-byte vectors
  int32_t chunk;             // inputs per work-group (blockIdx.y), a multiple of 8
  int64_t split_stride;
  float t0, tKs;             // the clip range
  float masked_below, masked_above;      // zero_spline: inputs outside contribute nothing; clip_x: -inf, +inf
  float knots[kMxMaxSegments - 1];       // the inner knots, +inf past the last
  float segment[kMxMaxSegments][kMxSegFloats];     // see segment_constants
};

// Where an input lies: the clipped x' (NaN for a NaN input) and its segment, a.segments for one that contributes nothing.
struct Position {
  float x;
  int segment;
};

// SLOTS - 4 inner knots at most.  `dead`: an input past the work-group's last, x finite.
template <int SLOTS>
__device__ __forceinline__ Position locate(const SplineMatrixArgs &a, float x, bool dead) {
  const float xc = __builtin_amdgcn_fmed3f(x, a.t0, a.tKs);
  int k = 0;
#pragma unroll
  for (int kappa = 0; kappa < SLOTS - 4; ++kappa) k += (a.knots[kappa] <= xc) ? 1 : 0;
  const bool masked = dead || x < a.masked_below || x > a.masked_above;
  k = masked ? a.segments : k;
  return Position{(x != x) ? __builtin_nanf("") : xc, k};
}

// The four non-zero cubics, each with a small error relative to itself.  The two outer ones have a triple zero at an end of
// the segment and are a factor times the cube of the distance from that end; a polynomial about the middle would cancel there
// (values below 1e-3 came out with a median relative error of 5e-6 and more, some negative).  The two middle ones stay
// away from zero (bspline_matrix_fits) and are polynomials about the middle, coefficients rounded once from 64 bits.
// Distances are scaled by a power of two, which rounds nothing.  Against the Cox-de Boor recursion in fp32 a third of the
// instructions; root of the summed squares of the four errors on uniform knots, G = 5 / 8 / 10: 2.4e-8 / 2.5e-8 / 2.4e-8
// (recursion 5.5e-8 / 2.8e-8 / 4.1e-8), largest relative error 3.6e-7 (3.8e-7).  The segment a.segments of s_seg is all zero.
__device__ __forceinline__ void basis_of(const float *s_seg, const Position &at, float n[4]) {
  const float *seg = s_seg + at.segment * kMxSegStride;
  const f32x4 p32 = *reinterpret_cast<const f32x4 *>(seg), p10 = *reinterpret_cast<const f32x4 *>(seg + 4);
  const f32x4 place = *reinterpret_cast<const f32x4 *>(seg + 8);                     // left end, right end, middle, scale
  const f32x2 outer = *reinterpret_cast<const f32x2 *>(seg + 12);
  const float from_right = __fmul_rn(__fsub_rn(place.y, at.x), place.w);
  const float from_left = __fmul_rn(__fsub_rn(at.x, place.x), place.w);
  const float v = __fmul_rn(__fsub_rn(at.x, place.z), place.w);
  n[0] = __fmul_rn(__fmul_rn(__fmul_rn(from_right, from_right), from_right), outer.x);
  n[1] = fmaf(fmaf(fmaf(p32.x, v, p32.z), v, p10.x), v, p10.z);
  n[2] = fmaf(fmaf(fmaf(p32.y, v, p32.w), v, p10.y), v, p10.w);
  n[3] = __fmul_rn(__fmul_rn(__fmul_rn(from_left, from_left), from_left), outer.y);
}

__device__ __forceinline__ void fill_segments(const SplineMatrixArgs &a, float *s_seg, int tid, int threads) {
  for (int q = tid; q < (a.segments + 1) * kMxSegFloats; q += threads) {
    const int s = q / kMxSegFloats, e = q - s * kMxSegFloats;
    s_seg[s * kMxSegStride + e] = (s < a.segments) ? a.segment[s][e] : 0.0f;
  }
}

union Slots { u32x4 u; bf16x8 h; };

// Where the four non-zero values of a segment go in a lane's 8 slots: for each of their four words the byte permute that takes
// it out of the packed values (SLOTS 8: {n0, n1} and {n2, n3}, moved up by `first` slots; SLOTS 16: the two of the lane's
// parity, moved to slot `at`).  One 16-byte LDS read and a permute per word and piece, in place of shifts and selects.
template <int SLOTS>
__device__ __forceinline__ void fill_places(u32x4 *s_place, int segments, int tid) {
  constexpr unsigned kNone = 0x0c0cu, kValue[4] = {0x0100u, 0x0302u, 0x0504u, 0x0706u};      // two bytes of zero; value 0 .. 3
  if (tid >= 2 * (segments + 1)) return;
  const int first = tid >> 1, half = tid & 1;
  const int at = (SLOTS == 8) ? first : (first + ((first ^ half) & 1) - half) >> 1, n = (SLOTS == 8) ? 4 : 2;
  unsigned w[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int lo = 2 * q - at, hi = lo + 1;                // which of the packed values lands in slots 2q and 2q + 1
    w[q] = ((lo >= 0 && lo < n) ? kValue[lo & 3] : kNone) | ((hi >= 0 && hi < n) ? kValue[hi & 3] : kNone) << 16;
  }
  s_place[tid] = u32x4{w[0], w[1], w[2], w[3]};
}

// a lane's 8 slots of one (row, input), three pieces
template <int SLOTS>
__device__ __forceinline__ void slots_of(const u32x4 *s_place, const float n[4], int first, int half, Slots out[3]) {
  const u32x4 place = s_place[2 * first + half];
  if constexpr (SLOTS == 8) {
    unsigned p01[3], p23[3];
    lutkan_cut3_pair(n[0], n[1], p01);
    lutkan_cut3_pair(n[2], n[3], p23);
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int w = 0; w < 4; ++w) out[q].u[w] = __builtin_amdgcn_perm(p23[q], p01[q], place[w]);
  } else {
    // rows first .. first+3; this lane holds those of parity `half`
    const bool same = ((first ^ half) & 1) == 0;
    unsigned p[3];
    lutkan_cut3_pair(same ? n[0] : n[1], same ? n[2] : n[3], p);
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int w = 0; w < 4; ++w) out[q].u[w] = __builtin_amdgcn_perm(p[q], p[q], place[w]);
  }
}

template <int SLOTS, int RT, int NT>
__global__ __launch_bounds__(kMxWaves * 64, 2) void bspline_matrix_kernel(const SplineMatrixArgs a) {
  constexpr int BN = 32 * NT;
  constexpr int IS = (SLOTS == 8) ? 8 : 4;                // inputs per stage: 8 units of 8 slots, 4 k steps
  constexpr int kThreads = kMxWaves * 64;
  constexpr int kUnits = 8 * BN;                          // (unit, column) pairs of a stage, one thread cuts 8 coefficients of each
  constexpr int UPT = (kUnits + kThreads - 1) / kThreads;
  constexpr int kStageBytes = 8 * 3 * BN * 16;
  extern __shared__ __align__(16) unsigned char lds[];
  float *const s_seg = reinterpret_cast<float *>(lds + 2 * kStageBytes);
  u32x4 *const s_place = reinterpret_cast<u32x4 *>(s_seg + (kMxMaxSegments + 1) * kMxSegStride);
  int *const s_uncut = reinterpret_cast<int *>(s_place + 2 * (kMxMaxSegments + 1));
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, col = lane & 31;
  const int t = blockIdx.x % a.n_tiles;
  const int64_t row0 = (int64_t)(blockIdx.x / a.n_tiles) * (kMxWaves * 32 * RT) + wave * (32 * RT);
  const bool wave_live = row0 < a.B;                      // wave-uniform; a wave without rows still stages and meets the barriers
  const int i_begin = blockIdx.y * a.chunk;
  const int i_end = min(a.d, i_begin + a.chunk);

  fill_segments(a, s_seg, tid, kThreads);
  fill_places<SLOTS>(s_place, a.segments, tid);
  if (tid == 0) *s_uncut = 0;

  // this thread's coefficient columns of a stage: unit u = (input u) resp. (input u & 3, parity u >> 2)
  const float *tile = a.coef_table + (size_t)t * a.d * a.R * a.jt;
  float cf[UPT][8];
  float largest = 0.0f;                                    // of the magnitudes this thread staged; NaN if one was
  auto load_coefs = [&](int i0) {
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
      const int id = tid + q * kThreads;
      const int c = (id % BN) & (a.jt - 1);                // a column past the tile: a valid address, not stored
      // the unit of a wave's 64 threads (two neighbouring ones with 32 columns, of one parity)
      const int u = (BN >= 64) ? __builtin_amdgcn_readfirstlane((id / BN) & 7) : (id / BN) & 7;
      const int parity = (SLOTS == 8) ? 0 : __builtin_amdgcn_readfirstlane(u >> 2);
      const int i = min(i0 + (SLOTS == 8 ? u : (u & 3)), a.d - 1);       // past the last input: its basis is zero
      const float *src = tile + (size_t)i * a.R * a.jt + c;
#pragma unroll
      for (int r = 0; r < 8; ++r)                          // slots past the last coefficient row: their basis is zero, any row will do
        cf[q][r] = src[min(SLOTS == 8 ? r : parity + 2 * r, a.R - 1) * a.jt];
    }
  };
  auto store_coefs = [&](unsigned char *buf) {
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
      const int id = tid + q * kThreads;
      if (kUnits < kThreads && id >= kUnits) break;
      const int u = id / BN, c = id % BN;
      unsigned p[4][3];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        lutkan_cut3_pair(cf[q][2 * r], cf[q][2 * r + 1], p[r]);
        largest = __builtin_elementwise_maximum(__builtin_elementwise_maximum(largest, fabsf(cf[q][2 * r])), fabsf(cf[q][2 * r + 1]));
      }
#pragma unroll
      for (int w = 0; w < 3; ++w) *reinterpret_cast<u32x4 *>(buf + ((u * 3 + w) * BN + c) * 16) = u32x4{p[0][w], p[1][w], p[2][w], p[3][w]};
    }
  };

  // this lane's inputs of a stage: four consecutive ones of its row (the upper lanes' follow the lower lanes' with SLOTS 8)
  const int lane_input = (SLOTS == 8) ? 4 * half : 0;
  int64_t row[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) row[rt] = min(row0 + rt * 32 + col, a.B - 1);
  float xv[RT][4];
  auto load_inputs = [&](int i0) {
    const int i = i0 + lane_input;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      if (a.x_vec4) {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(a.x + row[rt] * a.d + min(i, a.d - 4));
        xv[rt][0] = v.x; xv[rt][1] = v.y; xv[rt][2] = v.z; xv[rt][3] = v.w;
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) xv[rt][s] = a.x[row[rt] * a.d + min(i + s, a.d - 1)];
      }
    }
  };

  f32x16 acc[RT][NT], low[RT][NT];       // the products of the high pieces, and the five smaller ones
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
#pragma unroll
      for (int v = 0; v < 16; ++v) { acc[rt][ct][v] = 0.0f; low[rt][ct][v] = 0.0f; }

  load_coefs(i_begin);
  if (wave_live) load_inputs(i_begin);
  store_coefs(lds);
  __syncthreads();

  int cur = 0;
  for (int i0 = i_begin; i0 < i_end; i0 += IS) {
    const bool more = i0 + IS < i_end;
    // the inputs of this stage; one past the work-group's last takes the all-zero segment (and a finite x)
    float xc[RT][4];
    bool dead[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      dead[s] = i0 + lane_input + s >= i_end;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) xc[rt][s] = dead[s] ? a.t0 : xv[rt][s];
    }
    if (more) {                                            // the next stage travels while this one multiplies
      load_coefs(i0 + IS);
      if (wave_live) load_inputs(i0 + IS);
    }
    if (wave_live) {
      const unsigned char *buf = lds + cur * kStageBytes + half * (4 * 3 * BN * 16) + col * 16;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        Slots af[RT][3];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const Position at = locate<SLOTS>(a, xc[rt][s], dead[s]);
          float n[4];
          basis_of(s_seg, at, n);
          slots_of<SLOTS>(s_place, n, at.segment, half, af[rt]);
        }
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
          Slots wf[3];
#pragma unroll
          for (int q = 0; q < 3; ++q) wf[q].u = *reinterpret_cast<const u32x4 *>(buf + ((s * 3 + q) * BN + ct * 32) * 16);
          // the six piece products, the small ones first
          constexpr int kPieceOfA[5] = {2, 0, 1, 1, 0}, kPieceOfW[5] = {0, 2, 1, 0, 1};
#pragma unroll
          for (int p = 0; p < 5; ++p)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
              low[rt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[rt][kPieceOfA[p]].h, wf[kPieceOfW[p]].h, low[rt][ct], 0, 0, 0);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            acc[rt][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[rt][0].h, wf[0].h, acc[rt][ct], 0, 0, 0);
        }
      }
    }
    if (more) store_coefs(lds + (cur ^ 1) * kStageBytes);   // (everyone left that buffer before the last barrier)
    else if (!(largest <= kLargestBf16)) *s_uncut = 1;
    __syncthreads();
    cur ^= 1;
  }

  // accumulator of a 32 x 32 tile: element v of a lane is row 8*(v/4) + 4*(lane/32) + v%4, column lane%32
  float *yout = a.y + (int64_t)blockIdx.y * a.split_stride;
  const int width = min(a.jt, BN);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) {
      const int c = ct * 32 + col;
      const int j = t * a.jt + c;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t b = row0 + rt * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
        if (b < a.B && c < width && j < a.m) yout[b * a.m + j] = acc[rt][ct][v] + low[rt][ct][v];
      }
    }
  // A coefficient that is not finite (in a table that its owner wrote: the compiler refuses them), or has no bf16 value above it,
  // makes every row of the product NaN, by 0 * inf.  It belongs to the rows on its support: the work-group sums its outputs
  // again, term by term.
  if (*s_uncut == 0) return;
#pragma unroll 1
  for (int e = 0; e < RT * NT * 16; ++e) {
    const int rt = e / (NT * 16), c = (e / 16 % NT) * 32 + col, v = e % 16;
    const int j = t * a.jt + c;
    const int64_t b = row0 + rt * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
    if (b >= a.B || c >= width || j >= a.m) continue;
    float sum = 0.0f;
#pragma unroll 1
    for (int i = i_begin; i < i_end; ++i) {
      const Position at = locate<SLOTS>(a, a.x[b * a.d + i], false);
      if (at.segment == a.segments) continue;
      float n[4];
      basis_of(s_seg, at, n);
      const float *src = tile + ((size_t)i * a.R + at.segment) * a.jt + c;
#pragma unroll
      for (int q = 0; q < 4; ++q) sum = fmaf(n[q], src[q * a.jt], sum);
    }
    yout[b * a.m + j] = sum;
  }
}

// What the kernel knows of the span [tau[mu], tau[mu+1]): the two middle ones of its four cubics as polynomials in
// v = (x - middle) * scale (de Boor's triangle on polynomials, 64 bits) -- v^3 of both, v^2 of both, v, 1 --, its ends, middle
// and scale (the power of two that takes its width into [1, 2)), and the factors of the two outer ones' cubed distances.
void segment_constants(const float *tau, int mu, float out[kMxSegFloats]) {
  const double left = tau[mu], right = tau[mu + 1];
  int exponent;
  (void)std::frexp(right - left, &exponent);
  const double scale = std::ldexp(1.0, 1 - exponent), width = 1.0 / scale;
  const float middle = (float)(0.5 * (left + right));
  const double mid = middle;
  double n[4][4] = {{1.0, 0.0, 0.0, 0.0}};               // n[e][deg]
  for (int q = 1; q <= 3; ++q) {
    double saved[4] = {0.0, 0.0, 0.0, 0.0};
    for (int r = 0; r < q; ++r) {
      const double hi = (double)tau[mu + r + 1], lo = (double)tau[mu + 1 - q + r];
      double t[4];
      for (int g = 0; g < 4; ++g) t[g] = n[r][g] / (hi - lo);
      // n[r] = saved + (hi - x) * t;  saved = (x - lo) * t,   x = mid + width * v
      double next[4], carry[4];
      for (int g = 0; g < 4; ++g) {
        const double below = g ? t[g - 1] * width : 0.0;
        next[g] = saved[g] + (hi - mid) * t[g] - below;
        carry[g] = (mid - lo) * t[g] + below;
      }
      for (int g = 0; g < 4; ++g) { n[r][g] = next[g]; saved[g] = carry[g]; }
    }
    for (int g = 0; g < 4; ++g) n[q][g] = saved[g];
  }
  for (int g = 0; g < 4; ++g) {
    out[(3 - g) * 2] = (float)n[1][g];
    out[(3 - g) * 2 + 1] = (float)n[2][g];
  }
  out[8] = (float)left; out[9] = (float)right; out[10] = middle; out[11] = (float)scale;
  // N = (right - x)^3 / ((tau[mu+1] - tau[mu-2]) (tau[mu+1] - tau[mu-1]) (tau[mu+1] - tau[mu])), and its mirror image
  out[12] = (float)(width / (right - tau[mu - 2]) * (width / (right - tau[mu - 1])) * (width / (right - left)));
  out[13] = (float)(width / (tau[mu + 3] - left) * (width / (tau[mu + 2] - left)) * (width / (right - left)));
}

struct MatrixPlan {
  int rt, n_split, chunk;
  double cost;
};

// Launch shape: 32-row tiles per wave (rt) and chunks of inputs, by the same kind of cost model as the tiled kernels
// (microseconds): a stage costs a SIMD's two waves their matrix instructions (32 cycles each, 0.8 of the time) or their
// vector work, whichever is more, and 1000 cycles of barrier and latency, at the 1.7 GHz of a chip under matrix load
// (128 -> 128 at 131072 rows: 5.2 us per stage of 8 inputs); a work-group adds its fill; the launch runs in rounds of 256
// work-groups; chunks add the summing pass and are as many as the caller's workspace holds sums for.  Two accumulators
// of 64 rows x 128 columns would not fit the registers of two waves per SIMD: rt = 1 there.
MatrixPlan plan_matrix(int64_t B, int d, int m, int n_tiles, int nt, int slots, size_t partial_bytes) {
  const int is = (slots == 8) ? 8 : 4;
  MatrixPlan best{1, 1, d, 1e300};
  for (int rt = 1; rt <= (nt == 4 ? 1 : 2); ++rt) {
    const int64_t groups = (B + kMxWaves * 32 * rt - 1) / (kMxWaves * 32 * rt) * n_tiles;
    const double matrix = 2.0 * 4 * rt * nt * 6 * 32 * 1.25, vector = 2.0 * (4 * rt * 80 + 45 * nt) * 4.0;
    const double stage = (std::max(matrix, vector) + 1000.0) / 1700.0;
    for (int want = 1; want <= 64; ++want) {
      const int chunk = (int)round_up((d + want - 1) / want, 8);
      const int split = (d + chunk - 1) / chunk;
      if (split > 1 && (size_t)split * (size_t)B * (size_t)m * 4 > partial_bytes) break;
      const double rounds = (double)((groups * split + 255) / 256);
      double cost = rounds * (4.0 + (double)((chunk + is - 1) / is) * stage);
      if (split > 1) cost += 4.0 + (double)split * (double)B * m * 4.0 / 3e6;
      if (cost < best.cost) best = MatrixPlan{rt, split, chunk, cost};
      if (chunk <= 8) break;
    }
  }
  return best;
}

template <int SLOTS, int RT, int NT>
int launch_matrix(const SplineMatrixArgs &ma, int n_split, hipStream_t s) {
  constexpr int kRows = kMxWaves * 32 * RT;
  const int64_t groups = (ma.B + kRows - 1) / kRows * ma.n_tiles;
  if (groups > 0x7fffffffLL) return fail(LUTKAN_EUNSUPPORTED, "bspline_matrix_kernel: B * m too large for one launch");
  const size_t lds = 2 * (size_t)(8 * 3 * 32 * NT * 16) + kMxLdsTail;
  static LdsCap raised;
  if (int rc = raise_lds_cap(bspline_matrix_kernel<SLOTS, RT, NT>, &raised, "bspline_matrix_kernel")) return rc;
  hipLaunchKernelGGL((bspline_matrix_kernel<SLOTS, RT, NT>), dim3((unsigned)groups, (unsigned)n_split), dim3(kMxWaves * 64), lds, s, ma);
  return check_launch("bspline_matrix_kernel");
}

template <int SLOTS>
int launch_matrix_slots(const SplineMatrixArgs &ma, int rt, int nt, int n_split, hipStream_t s) {
  if (nt == 4) return launch_matrix<SLOTS, 1, 4>(ma, n_split, s);
  if (nt == 2) return rt == 2 ? launch_matrix<SLOTS, 2, 2>(ma, n_split, s) : launch_matrix<SLOTS, 1, 2>(ma, n_split, s);
  return rt == 2 ? launch_matrix<SLOTS, 2, 1>(ma, n_split, s) : launch_matrix<SLOTS, 1, 1>(ma, n_split, s);
}

}  // namespace

namespace lutkan {

int bspline_matrix_forward(const bspline_dev_layer *l, const float *x, int64_t B, float *y, void *workspace, size_t workspace_bytes,
                           void *hip_stream) {
  SplineMatrixArgs ma = {};
  ma.x = x; ma.coef_table = l->coef_table;
  ma.B = B; ma.d = l->d; ma.m = l->m; ma.R = l->G + 3; ma.segments = l->G; ma.jt = l->jt; ma.n_tiles = l->n_tiles;
  ma.x_vec4 = (l->d % 4 == 0) && (reinterpret_cast<uintptr_t>(x) & 15) == 0;
  const float *T = l->ext_knots + 3;
  // the safe clip value of Eq. 13; In(x) is t0 <= x <= tKs under either boundary mode
  ma.t0 = T[0];
  ma.tKs = (l->boundary == LUTKAN_CLOSED) ? T[l->G] : std::nextafterf(T[l->G], -INFINITY);
  ma.masked_below = (l->oob == LUTKAN_ZERO_SPLINE) ? ma.t0 : -INFINITY;
  ma.masked_above = (l->oob == LUTKAN_ZERO_SPLINE) ? ma.tKs : INFINITY;
  for (int k = 0; k < kMxMaxSegments - 1; ++k) ma.knots[k] = (k + 1 < l->G) ? T[k + 1] : INFINITY;
  for (int k = 0; k < l->G; ++k) segment_constants(l->ext_knots, 3 + k, ma.segment[k]);
  const int slots = (ma.R <= 8) ? 8 : 16;
  const int nt = ma.jt >= 128 ? 4 : ma.jt >= 64 ? 2 : 1;
  float *const partials = static_cast<float *>(workspace);
  const MatrixPlan mp = plan_matrix(B, l->d, l->m, l->n_tiles, nt, slots, workspace_bytes);
  ma.chunk = mp.chunk;
  ma.y = y;
  if (mp.n_split > 1) { ma.y = partials; ma.split_stride = B * l->m; }
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (int rc = slots == 8 ? launch_matrix_slots<8>(ma, mp.rt, nt, mp.n_split, s) : launch_matrix_slots<16>(ma, mp.rt, nt, mp.n_split, s)) return rc;
  plan_note("bspline_matrix np=%d split=%d slots=%d; ", mp.rt, mp.n_split, slots);
  if (mp.n_split == 1) return LUTKAN_OK;
  const int64_t n = B * l->m;
  hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, s, partials, y, n, mp.n_split, 0);
  plan_note("sum; ");
  return check_launch("sum_partials_kernel");
}

bool bspline_matrix_fits(const bspline_dev_layer *l) {
  if (l->value_repr != LUTKAN_REPR_PHI || l->knot_span != LUTKAN_SPAN_DOMAIN || l->knots_per_input) return false;
  if (l->G > kMxMaxSegments) return false;
  // segments far narrower or wider than any grid in use: their polynomial coefficients could leave fp32's range
  double gap[LUTKAN_MAX_K + 6];
  for (int r = 0; r < l->G + 6; ++r) {
    gap[r] = (double)l->ext_knots[r + 1] - (double)l->ext_knots[r];
    if (!(gap[r] > 1e-30 && gap[r] < 1e30)) return false;
  }
  // The two middle functions of a segment, as polynomials about its middle, have an error of some 3e-8; they are smallest at
  // the segment's ends, where they are an outer function of the neighbour at its inner end.  1/6 on uniform knots, 1/28 where
  // gaps differ by a factor of 3; on a grid that takes one below 1/32 it would be lost from the sixth digit on: the kernels with
  // the recursion serve that layer.
  for (int r = 3; r <= l->G + 2; ++r) {
    const double around = gap[r - 1] + gap[r] + gap[r + 1];
    if (32.0 * gap[r + 1] * gap[r + 1] < (gap[r] + gap[r + 1]) * around || 32.0 * gap[r - 1] * gap[r - 1] < (gap[r - 1] + gap[r]) * around) return false;
  }
  return true;
}

}  // namespace lutkan
