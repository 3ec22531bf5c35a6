// The B-spline layer as a dense contraction on the matrix cores:
//     y[b][j] = sum_i sum_r N_r(x[b][i]) * c[i][r][j]
// with the R = G + 3 basis values of an input as contraction index, four neighbouring ones of which are non-zero.  The tiled
// kernel (bspline_kernels.hip) spends four multiply-adds per edge and is bound by the 16 bytes of coefficients per edge that it
// reads from LDS at a row's own offset; here the coefficients are the second operand of a matrix instruction, read from
// LDS once per 32 rows.  The basis is evaluated where it is consumed, so the pass that writes and reads 32 bytes per (row, input)
// falls away.
//
// fp32 accuracy from bf16 matrix instructions, as in lutkan_base_gemm.hip: every fp32 operand is cut exactly into three
// bf16 pieces and six of the nine piece products are accumulated in fp32; the other three are at most 2^-24 of the product
// together (lutkan_pieces.h).  The products
// of the two high pieces have an accumulator of their own, apart from the five small ones: with one accumulator for all
// six, every small product rounds the large sum once more and the layer came out 1.2 - 1.8 times further from a 64-bit
// evaluation than the tiled kernel; apart, it is nearer than that kernel (64 -> 128 at 131072 rows 1.1e-7 against 3.0e-7,
// 1024 -> 1024 at 4096 rows, G = 10, 4.0e-7 against 5.7e-7).
//
// Operand A, sparse and without LDS: v_smfmac_f32_32x32x32_bf16 takes operand A with two stored values of every four
// consecutive k (a group) and two bits each for where they stand, and does twice the dense instruction's k in the same time (55.8
// cycles at 2.4 GHz against 54.1, both at the clock that random operands leave the chip).  A basis always fits: coefficient row r
// goes to group r % GRP of its input, so four neighbouring rows put at most two values into a group.  GRP groups per input:
//   GRP = 2   R <= 8: two values in each group, nothing stored is zero
//   GRP = 3   R <= 12: two, one and one
//   GRP = 4   R <= 16: one in each
// A lane holds 8 stored values of one row, four groups, and k may be numbered freely as long as both operands agree, so a lane's
// groups are those of its own inputs: the lower lanes take the first half of a stage's inputs, the upper lanes the second, and
// every basis value is evaluated once per wave.  A lane locates its (row, input), evaluates the four cubics, cuts them and moves
// the pieces into its groups by byte permutes.
// Operand B (coefficients): a work-group stages 8 (GRP 4: 4) inputs at a time, cut into pieces on the way into LDS, as
// [unit][piece][column][8 slots]; a unit is two groups of an input half.  What a lane stores at e = 0 .. 3 meets operand B of the
// lower lanes, at e = 4 .. 7 that of the upper lanes, in elements 0 .. 7 (a lower lane's) or 8 .. 15 (an upper lane's).
//
// A work-group is 8 waves of 32*RT rows x 32*NT columns (one column tile of the coefficient table); two waves share a
// SIMD, so that one's vector work (basis, pieces) overlaps the other's matrix instructions.
//
// Bound: matrix and vector issue, at the clock they leave the chip.  48 / 72 / 96 sparse flop per edge; 1024 -> 1024, G = 10, at 4096
// rows: matrix pipes 0.46 busy, vector issue 0.43, LDS 0.33, 1.9 GHz; 128 -> 128, G = 5, at 131072 rows 0.36, 0.46, 0.30.  One such instruction of each of two waves and the 7 vector
// instructions that go with it take 64 cycles at 2.4 GHz when nothing else does, here 83: vector instructions hide behind a matrix
// instruction only up to about four.  (Spreading them between the matrix instructions by hand, evaluating a step ahead: 4 %
// faster with 128 columns, 4 - 10 % slower with 64 and fewer, whose registers then spill; four waves of 64 rows x 128 columns:
// 13 % slower.)
// Whole layers, dense matrix instructions -> sparse, microseconds (one run each): 64 -> 128 at 131072 rows, G = 5, 111 -> 84;
// 128 -> 128 190 -> 142; 128 -> 128, G = 8, 338 -> 191; 256 -> 256 at 16384 rows, G = 8, 189 -> 110; 1024 -> 1024 at 4096 rows, G = 5 /
// 8 / 10, 348 / 658 / 658 -> 255 / 350 / 441; 64 -> 8 at 131072 rows 36 -> 31 (with scalar addresses, below, 128 -> 128 123, 1024 -> 1024 235 / 337 / 415).  The tiled kernel takes 587 for 128 -> 128 (G = 5), 790
// for 1024 -> 1024 (G = 10).
// The file is compiled with -ffp-contract=off; fused multiply-adds are written out as fmaf().
#include "bspline_matrix.h"
#include "lutkan_device.h"
#include "lutkan_pieces.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kMxWaves = 8;
constexpr int kMxMaxSegments = 13;       // R = G + 3 <= 16
constexpr int kMxSegFloats = 14;         // of a segment: 8 polynomial coefficients, its ends, middle and scale, the two outer factors
constexpr int kMxSegStride = 20;         // ... in LDS: 80-byte rows spread the banks
constexpr int kMxLdsTail = (kMxMaxSegments + 1) * (kMxSegStride * 4 + 16 + 4) + 16;      // behind the stages in LDS: segments, places, indices, a flag

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

// 4 GRP - 4 inner knots at most.  `dead`: an input past the work-group's last, x finite.
template <int GRP>
__device__ __forceinline__ Position locate(const SplineMatrixArgs &a, float x, bool dead) {
  const float xc = __builtin_amdgcn_fmed3f(x, a.t0, a.tKs);
  int k = 0;
#pragma unroll
  for (int kappa = 0; kappa < 4 * GRP - 4; ++kappa) k += (a.knots[kappa] <= xc) ? 1 : 0;
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

union Sparse { u32x4 u; bf16x8 h; };          // a lane's 8 values of operand A: two of each of its four groups of slots
union Dense { u32x4 u[2]; bf16x16 h; };       // a lane's 16 values of operand B

// Where the four non-zero values of a segment go.  Coefficient row r is slot r / GRP of group r % GRP, so the rows first ..
// first+3 lie in every group once (GRP 4), once or twice (3) or twice (2).  place[g]: the byte permute that takes group g's two
// values out of the packed {n0, n1} and {n2, n3}, in the order of their slots; bits 4g .. 4g+3 of the index: those two slots, the
// lower one first (a group with one value has a zero beside it).  The entry of a.segments places nothing.
template <int GRP>
__device__ __forceinline__ void fill_places(u32x4 *s_place, unsigned *s_index, int segments, int tid) {
  constexpr unsigned kNone = 0x0c0cu, kValue[4] = {0x0100u, 0x0302u, 0x0504u, 0x0706u};      // two bytes of zero; value 0 .. 3
  if (tid > segments) return;
  unsigned w[4] = {0u, 0u, 0u, 0u}, index = 0;
#pragma unroll
  for (int g = 0; g < GRP; ++g) {
    const int n = (g + 2 * GRP * 4 - tid) % GRP;          // the first of the window's values in this group, from row tid + n
    const int slot = (tid + n) / GRP;
    unsigned lo = kValue[n & 3], hi = (n + GRP < 4) ? kValue[(n + GRP) & 3] : kNone;
    int at = slot;
    if (slot == 3) { hi = lo; lo = kNone; at = 2; }        // (the last slot: a single value, after an empty one)
    if (tid == segments) { lo = hi = kNone; at = 0; }
    w[g] = lo | (hi << 16);
    index |= (unsigned)(at | ((at + 1) << 2)) << (4 * g);
  }
  s_place[tid] = u32x4{w[0], w[1], w[2], w[3]};
  s_index[tid] = index;
}

template <int GRP, int RT, int NT>
__global__ __launch_bounds__(kMxWaves * 64, 2) void bspline_matrix_kernel(const SplineMatrixArgs a) {
  constexpr int BN = 32 * NT;
  constexpr int IPL = (GRP == 4) ? 2 : 4;                 // inputs a lane evaluates per stage
  constexpr int IS = 2 * IPL;                             // inputs per stage
  constexpr int STEPS = IPL * GRP / 4;                    // matrix k steps per stage, four groups of a lane each
  constexpr int kThreads = kMxWaves * 64;
  constexpr int kUnits = 4 * STEPS;                       // of 8 slots of a column: what a lane reads of operand B per step and half of the inputs
  constexpr int kPairs = kUnits * BN;                     // (unit, column) pairs of a stage, one thread cuts 8 coefficients of each
  constexpr int UPT = (kPairs + kThreads - 1) / kThreads;
  constexpr int kStageBytes = kUnits * 3 * BN * 16;
  extern __shared__ __align__(16) unsigned char lds[];
  float *const s_seg = reinterpret_cast<float *>(lds + 2 * kStageBytes);
  u32x4 *const s_place = reinterpret_cast<u32x4 *>(s_seg + (kMxMaxSegments + 1) * kMxSegStride);
  unsigned *const s_index = reinterpret_cast<unsigned *>(s_place + (kMxMaxSegments + 1));
  int *const s_uncut = reinterpret_cast<int *>(s_index + (kMxMaxSegments + 1));
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
  fill_places<GRP>(s_place, s_index, a.segments, tid);
  if (tid == 0) *s_uncut = 0;

  // This thread's coefficient columns of a stage.  Unit u = (h * STEPS + step) * 2 + p: the groups 4 step + 2p and the next one
  // of the lanes of half h, whose groups are those of its inputs one after the other.
  // Where they lie from the stage's first slice on, in floats, is the same for every stage and (from 64 columns on) for a wave:
  // computed once, in scalar registers.  With the addresses computed at every load a wave spent 190 scalar instructions a stage on
  // them: 1024 -> 1024 at 4096 rows, G = 10, 432 -> 409 us, 128 -> 128 at 131072, G = 5 / 8, 126 -> 123 / 176 -> 170 (buffer
  // loads with the offsets as their scalar operands: 417, 124, 168).
  const float *tile = a.coef_table + (size_t)t * a.d * a.R * a.jt;
  float cf[UPT][8];
  float largest = 0.0f;                                    // of the magnitudes this thread staged; NaN if one was
  auto unit_of = [&](int q) {                              // (with 32 columns a wave has two; past the last one, where not stored)
    const int id = tid + q * kThreads;
    return min((BN >= 64) ? __builtin_amdgcn_readfirstlane(id / BN) : id / BN, kUnits - 1);
  };
  auto row_of = [&](int u, int e, int &of) {               // the first coefficient row of a unit's group e, and the input of the stage
    const int h = u / (2 * STEPS), group = 4 * ((u >> 1) - h * STEPS) + 2 * (u & 1) + e;
    of = h * IPL + group / GRP;
    return group % GRP;
  };
  int offset[UPT][8];
#pragma unroll
  for (int q = 0; q < UPT; ++q)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      int of;
      const int g = row_of(unit_of(q), e, of);
#pragma unroll
      for (int r = 0; r < 4; ++r)                          // slots past the last coefficient row: no value goes there, any row will do
        offset[q][4 * e + r] = (of * a.R + min(g + GRP * r, a.R - 1)) * a.jt;
    }
  auto load_coefs = [&](int i0) {
    if (BN >= 64 && i0 + IS <= a.d) {
      const float *stage = tile + (size_t)i0 * a.R * a.jt;
#pragma unroll
      for (int q = 0; q < UPT; ++q) {
        const unsigned c = (unsigned)((tid + q * kThreads) % BN) & (unsigned)(a.jt - 1);
#pragma unroll
        for (int r = 0; r < 8; ++r) cf[q][r] = (stage + offset[q][r])[c];
      }
      return;
    }
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
      const int c = ((tid + q * kThreads) % BN) & (a.jt - 1);      // a column past the tile: a valid address, not stored
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        int of;
        const int g = row_of(unit_of(q), e, of);
        const int i = min(i0 + of, a.d - 1);               // past the last input: its basis is zero
        const float *src = tile + (size_t)i * a.R * a.jt + c;
#pragma unroll
        for (int r = 0; r < 4; ++r) cf[q][4 * e + r] = src[min(g + GRP * r, a.R - 1) * a.jt];
      }
    }
  };
  auto store_coefs = [&](unsigned char *buf) {
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
      const int id = tid + q * kThreads;
      if (kPairs % kThreads != 0 && id >= kPairs) break;
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

  // this lane's inputs of a stage: consecutive ones of its row, the upper lanes' after the lower lanes'
  const int lane_input = IPL * half;
  int64_t row[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) row[rt] = min(row0 + rt * 32 + col, a.B - 1);
  float xv[RT][IPL];
  auto load_inputs = [&](int i0) {
    const int i = i0 + lane_input;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      if (a.x_vec4) {
        if constexpr (IPL == 4) {
          const f32x4 v = *reinterpret_cast<const f32x4 *>(a.x + row[rt] * a.d + min(i, a.d - 4));
          xv[rt][0] = v.x; xv[rt][1] = v.y; xv[rt][2] = v.z; xv[rt][3] = v.w;
        } else {
          const f32x2 v = *reinterpret_cast<const f32x2 *>(a.x + row[rt] * a.d + min(i, a.d - 2));
          xv[rt][0] = v.x; xv[rt][1] = v.y;
        }
      } else {
#pragma unroll
        for (int s = 0; s < IPL; ++s) xv[rt][s] = a.x[row[rt] * a.d + min(i + s, a.d - 1)];
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
    float xc[RT][IPL];
    bool dead[IPL];
#pragma unroll
    for (int s = 0; s < IPL; ++s) {
      dead[s] = i0 + lane_input + s >= i_end;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) xc[rt][s] = dead[s] ? a.t0 : xv[rt][s];
    }
    if (more) {                                            // the next stage travels while this one multiplies
      load_coefs(i0 + IS);
      if (wave_live) load_inputs(i0 + IS);
    }
    if (wave_live) {
      const unsigned char *buf = lds + cur * kStageBytes + half * (3 * BN * 16) + col * 16;
      unsigned value[RT][3][IPL * GRP], index[RT][IPL];    // per piece the lane's groups, two values each; where they belong
#pragma unroll
      for (int s = 0; s < STEPS; ++s) {
#pragma unroll
        for (int of = (s == 0) ? 0 : (4 * s + GRP - 1) / GRP; of < (4 * s + 4 + GRP - 1) / GRP; ++of)      // the inputs this step is the first to need
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            const Position at = locate<GRP>(a, xc[rt][of], dead[of]);
            float n[4];
            basis_of(s_seg, at, n);
            const u32x4 place = s_place[at.segment];
            index[rt][of] = s_index[at.segment];
            unsigned p01[3], p23[3];
            lutkan_cut3_pair(n[0], n[1], p01);
            lutkan_cut3_pair(n[2], n[3], p23);
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
              for (int g = 0; g < GRP; ++g) value[rt][q][of * GRP + g] = __builtin_amdgcn_perm(p23[q], p01[q], place[g]);
          }
        Sparse af[RT][3];
        int slots[RT];                                     // bits 4g .. 4g+3: the slots of the step's group g
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          if constexpr (GRP == 4) slots[rt] = (int)index[rt][s];
          else if constexpr (GRP == 2) slots[rt] = (int)(index[rt][2 * s] | (index[rt][2 * s + 1] << 8));
          else slots[rt] = (int)((index[rt][s] >> (4 * s)) | (index[rt][s + 1] << (12 - 4 * s)));
#pragma unroll
          for (int q = 0; q < 3; ++q) af[rt][q].u = u32x4{value[rt][q][4 * s], value[rt][q][4 * s + 1], value[rt][q][4 * s + 2], value[rt][q][4 * s + 3]};
        }
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
          Dense wf[3];
#pragma unroll
          for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h) wf[q].u[h] = *reinterpret_cast<const u32x4 *>(buf + (((h * STEPS + s) * 6 + q) * BN + ct * 32) * 16);
          // the six piece products, the small ones first
          constexpr int kPieceOfA[5] = {2, 0, 1, 1, 0}, kPieceOfW[5] = {0, 2, 1, 0, 1};
#pragma unroll
          for (int p = 0; p < 5; ++p)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
              low[rt][ct] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(af[rt][kPieceOfA[p]].h, wf[kPieceOfW[p]].h, low[rt][ct], slots[rt], 0, 0);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            acc[rt][ct] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(af[rt][0].h, wf[0].h, acc[rt][ct], slots[rt], 0, 0);
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
      const Position at = locate<GRP>(a, a.x[b * a.d + i], false);
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
// vector work, whichever is more, and 1000 cycles of barrier and latency, at 1.45 GHz (128 -> 128 at 131072 rows: 3.4 us per stage
// of 8 inputs with two groups each, 5.1 with three; 1024 -> 1024: 3.3 per stage of 4 with four groups); a work-group adds its fill; the launch runs in rounds of 256
// work-groups; chunks add the summing pass and are as many as the caller's workspace holds sums for.  Two accumulators
// of 64 rows x 128 columns would not fit the registers of two waves per SIMD: rt = 1 there.
MatrixPlan plan_matrix(int64_t B, int d, int m, int n_tiles, int nt, int grp, size_t partial_bytes) {
  const int is = (grp == 4) ? 4 : 8, steps = is * grp / 8;
  MatrixPlan best{1, 1, d, 1e300};
  for (int rt = 1; rt <= (nt == 4 ? 1 : 2); ++rt) {
    const int64_t groups = (B + kMxWaves * 32 * rt - 1) / (kMxWaves * 32 * rt) * n_tiles;
    const double matrix = 2.0 * steps * rt * nt * 6 * 32 * 1.25, vector = 2.0 * (is / 2 * rt * 80 + 45 * nt) * 4.0;
    const double stage = (std::max(matrix, vector) + 1000.0) / 1450.0;
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

template <int GRP, int RT, int NT>
int launch_matrix(const SplineMatrixArgs &ma, int n_split, hipStream_t s) {
  constexpr int kRows = kMxWaves * 32 * RT;
  const int64_t groups = (ma.B + kRows - 1) / kRows * ma.n_tiles;
  if (groups > 0x7fffffffLL) return fail(LUTKAN_EUNSUPPORTED, "bspline_matrix_kernel: B * m too large for one launch");
  const size_t lds = 2 * (size_t)((GRP == 3 ? 12 : 8) * 3 * 32 * NT * 16) + kMxLdsTail;
  static LdsCap raised;
  if (int rc = raise_lds_cap(bspline_matrix_kernel<GRP, RT, NT>, &raised, "bspline_matrix_kernel")) return rc;
  hipLaunchKernelGGL((bspline_matrix_kernel<GRP, RT, NT>), dim3((unsigned)groups, (unsigned)n_split), dim3(kMxWaves * 64), lds, s, ma);
  return check_launch("bspline_matrix_kernel");
}

template <int GRP>
int launch_matrix_groups(const SplineMatrixArgs &ma, int rt, int nt, int n_split, hipStream_t s) {
  if (nt == 4) return launch_matrix<GRP, 1, 4>(ma, n_split, s);
  if (nt == 2) return rt == 2 ? launch_matrix<GRP, 2, 2>(ma, n_split, s) : launch_matrix<GRP, 1, 2>(ma, n_split, s);
  return rt == 2 ? launch_matrix<GRP, 2, 1>(ma, n_split, s) : launch_matrix<GRP, 1, 1>(ma, n_split, s);
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
  const int grp = (ma.R <= 8) ? 2 : (ma.R <= 12) ? 3 : 4;
  const int nt = ma.jt >= 128 ? 4 : ma.jt >= 64 ? 2 : 1;
  float *const partials = static_cast<float *>(workspace);
  const MatrixPlan mp = plan_matrix(B, l->d, l->m, l->n_tiles, nt, grp, workspace_bytes);
  ma.chunk = mp.chunk;
  ma.y = y;
  if (mp.n_split > 1) { ma.y = partials; ma.split_stride = B * l->m; }
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int rc = grp == 2 ? launch_matrix_groups<2>(ma, mp.rt, nt, mp.n_split, s) : grp == 3 ? launch_matrix_groups<3>(ma, mp.rt, nt, mp.n_split, s)
                                                                                : launch_matrix_groups<4>(ma, mp.rt, nt, mp.n_split, s);
  if (rc) return rc;
  plan_note("bspline_matrix np=%d split=%d slots=%d; ", mp.rt, mp.n_split, 4 * grp);
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
