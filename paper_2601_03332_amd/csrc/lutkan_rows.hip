// The LUT layer forward of a few rows in one launch: locate, gather and sum in one work-group per (rows, column tile).
//
// A batch of a few rows on a layer of some hundred inputs and outputs is a chain of waits, not work: locate kernel, gather
// kernel with the inputs split over the GPU, summing pass, each 4 - 6 us for its launch, its dependent reads and its drain.
// Here a work-group of 16 waves carries one row (or four, four waves each) through one column tile:
//   locate   its threads run steps 1-4 of Sec. 4.5 on the row's inputs and leave the records in LDS (every column tile
//            repeats this: a few instructions per input against the 64 edges it serves)
//   gather   LPR lanes own 4 adjacent columns each, so a wave is 64/LPR groups and the row has WPR*64/LPR of them; group g
//            takes the inputs g, g + groups, ..., four or two at a time with all their table reads in flight (256 inputs on
//            64-column tiles: one round trip to L2), with the arithmetic of the gather kernel
//   sum      a fixed butterfly over the groups of a wave, then over the waves through LDS, in wave order
// No workspace, no partial sums in memory, bit-reproducible; nearer to a 64-bit evaluation than the passes (short sums).
//
// Bound: dependent reads up to about a hundred rows, then the table bytes the lanes request (12 - 15 TB/s through the L2s).
// Whole layers replayed from a HIP graph, passes -> this kernel, microseconds: 256 -> 256, L = 64, at 1 / 64 / 256 / 512 rows
// 11.4 / 20.4 / 26 / 29 -> 4.1 / 4.7 / 10.0 / 17.8 (at 1000 the passes run); 1024 -> 64 at 128 rows 30 -> 9.3; 512 -> 512, L = 32, at
// 32 rows 24.5 -> 6.2; 30 -> 1000 with spline_component at 128 rows 16.8 -> 7.9; 700 -> 130 at 128 rows 30 -> 17.8.  Called one by one
// the small ones take 6.5, the host's share.
// The file is compiled with -ffp-contract=off; every fused multiply-add is written out as fmaf().
#include "lutkan_device.h"
#include "lutkan_locate.h"
#include "lutkan_rows.h"

namespace {

constexpr int kRowsWaves = 16;
constexpr int kRowsMaxInputs = 2048;     // records of four rows in LDS
constexpr int64_t kRowsMaxBatch = 6144; // beyond, the passes win: 40 -> 60 -> 60 -> 10 at 5000 rows 44 us (48 by passes), at 7500 64 (62)

struct RowsArgs {
  const float *x;                        // [B][d]
  const unsigned char *table;
  float *y;
  const float *input_knots;              // nullable: [d][K+1], one knot vector per input
  int64_t B;
  int32_t d, m, K, L, n_tiles, blob_bytes;
  int32_t codes_off, params_off;
  int32_t closed, with_base, param_fp16;
  float t0, tKs;
  float masked_below, masked_above;      // zero_spline: inputs outside contribute nothing; clip_x: -inf, +inf
  int32_t zero_spline;
  float inner[LUTKAN_MAX_K];             // the inner knots T[1] .. T[K-1], +inf past the last
  float knots[LUTKAN_MAX_K + 1];
};

// DEPTH: inputs of every group in a round, four or two, a kernel of its own each: 71 - 91 vector registers and one work-group per compute
// unit, or at most 64 and two.  (Two also need at most 80 scalar registers, which the launch bounds ask for: with 82 100 -> 200 at 600
// rows took 14.5 us instead of 11.1.)  See launch_rows_depth.
template <int SCHEME, int LPR, int WPR, int DEPTH>
__global__ __launch_bounds__(kRowsWaves * 64, DEPTH == 2 ? 8 : 4) void lutkan_rows_kernel(const RowsArgs a) {
  constexpr int ROWS = kRowsWaves / WPR, JT = 4 * LPR, GROUPS = WPR * (64 / LPR);
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int rrow = wave / WPR, wr = wave % WPR;
  const int rtid = wr * 64 + lane;
  const int t = blockIdx.x % a.n_tiles;
  const int64_t row = (int64_t)(blockIdx.x / a.n_tiles) * ROWS + rrow;
  const float *xrow = a.x + min(row, a.B - 1) * a.d;                      // (a row past the last repeats it and is not stored)
  // LDS: sums of the waves [16][JT], records [ROWS][d], knots
  f32x4 (*const s_part)[LPR] = reinterpret_cast<f32x4 (*)[LPR]>(lds);
  u32x4 *const s_rec_all = reinterpret_cast<u32x4 *>(lds + kRowsWaves * JT * 4);
  u32x4 *const s_rec = s_rec_all + (size_t)rrow * a.d;
  float *const s_knots = reinterpret_cast<float *>(s_rec_all + (size_t)ROWS * a.d);
  const int plane = JT * (a.param_fp16 ? 2 : 4);
  const int param_row = plane * (SCHEME == LUTKAN_ASYM_UINT8 ? 2 : 1);

  float x0 = xrow[min(rtid, a.d - 1)];                                    // in flight while the knots are placed
  if (!a.input_knots && tid <= a.K) s_knots[tid] = a.knots[tid];
  __syncthreads();
  for (int i = rtid; i < a.d; i += WPR * 64) {
    const float x = (i == rtid) ? x0 : xrow[i];
    unsigned row_at, segment;
    float w;
    bool masked;
    if (a.input_knots) {
      const Located o = locate_one<true>(a, a.input_knots + (int64_t)i * (a.K + 1), x);
      masked = a.zero_spline && !o.inside && !o.is_nan;
      row_at = (unsigned)(o.k * a.L + o.l0);
      segment = (unsigned)o.k;
      w = o.is_nan ? __builtin_nanf("") : o.w;
    } else {
      int k[1], l0[1];
      const float xs[1] = {x};
      float ws[1];
      locate_side_by_side<1>(a, s_knots, xs, k, l0, ws);
      masked = (x < a.masked_below) | (x > a.masked_above);
      row_at = (unsigned)(k[0] * a.L + l0[0]);
      segment = (unsigned)k[0];
      w = ws[0];
    }
    // byte offsets in the slice; a masked input reads its all-zero rows
    const unsigned code_at = (unsigned)a.codes_off + (masked ? (unsigned)(a.K * a.L) : row_at) * JT;
    const unsigned param_at = (unsigned)a.params_off + (masked ? (unsigned)a.K : segment) * (unsigned)param_row;
    const float sx = a.with_base ? __fdiv_rn(x, 1.0f + expf(-x)) : 0.0f;      // at the raw input, never masked
    s_rec[i] = u32x4{code_at, param_at, masked ? 0u : __float_as_uint(w), __float_as_uint(sx)};
  }
  __syncthreads();

  const int sub = lane & (LPR - 1);
  const int g = wr * (64 / LPR) + lane / LPR;
  const unsigned char *tile = a.table + (size_t)t * a.d * a.blob_bytes;
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  auto round = [&](auto count, int i0) {
    constexpr int U = decltype(count)::value;
    u32x4 rec[U];
    unsigned c0[U], c1[U];
    f32x4 al[U], ym[U], bg[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + u * GROUPS, a.d - 1);
      rec[u] = s_rec[i];
      const unsigned char *slice = tile + (size_t)i * a.blob_bytes;
      const unsigned char *cp = slice + rec[u].x + sub * 4, *pp = slice + rec[u].y;
      c0[u] = *reinterpret_cast<const unsigned *>(cp);
      c1[u] = *reinterpret_cast<const unsigned *>(cp + JT);
      ym[u] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (a.param_fp16) {
        const u32x2 ha = *reinterpret_cast<const u32x2 *>(pp + sub * 8);
        const f16x2 a01 = bits_to_f16x2(ha.x), a23 = bits_to_f16x2(ha.y);
        al[u] = f32x4{(float)a01.x, (float)a01.y, (float)a23.x, (float)a23.y};
        if (SCHEME == LUTKAN_ASYM_UINT8) {
          const u32x2 hy = *reinterpret_cast<const u32x2 *>(pp + plane + sub * 8);
          const f16x2 y01 = bits_to_f16x2(hy.x), y23 = bits_to_f16x2(hy.y);
          ym[u] = f32x4{(float)y01.x, (float)y01.y, (float)y23.x, (float)y23.y};
        }
      } else {
        al[u] = *reinterpret_cast<const f32x4 *>(pp + sub * 16);
        if (SCHEME == LUTKAN_ASYM_UINT8) ym[u] = *reinterpret_cast<const f32x4 *>(pp + plane + sub * 16);
      }
      bg[u] = a.with_base ? *reinterpret_cast<const f32x4 *>(slice + sub * 16) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (i0 + u * GROUPS < a.d) {
        const float w = __uint_as_float(rec[u].z), sx = __uint_as_float(rec[u].w);
        float q[4];
        interpolate_codes<SCHEME>(c0[u], c1[u], w, q);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          acc[c] = fmaf(al[u][c], q[c] * kTwoTo24, acc[c]);                   // (exact: undo the 2^-24 of the codes)
          if (SCHEME == LUTKAN_ASYM_UINT8) acc[c] += ym[u][c];
          if (a.with_base) acc[c] = fmaf(bg[u][c], sx, acc[c]);
        }
      }
    }
  };
  if (DEPTH == 2 && a.d <= GROUPS) {
    round(std::integral_constant<int, 1>{}, g);
  } else {
    for (int i0 = g; i0 < a.d; i0 += DEPTH * GROUPS) round(std::integral_constant<int, DEPTH>{}, i0);
  }
#pragma unroll
  for (int off = LPR; off < 64; off <<= 1) {
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] += __shfl_xor(acc[c], off, kWave);
  }
  if (lane < LPR) s_part[wave][lane] = f32x4{acc[0], acc[1], acc[2], acc[3]};
  __syncthreads();
  if (rtid < JT && row < a.B) {
    const int j = t * JT + rtid;
    const float *part = reinterpret_cast<const float *>(s_part[rrow * WPR]) + rtid;
    float total = part[0];
#pragma unroll
    for (int v = 1; v < WPR; ++v) total += part[v * JT];                      // wave order
    if (j < a.m) a.y[row * a.m + j] = total;
  }
}

int64_t rows_groups(int64_t B, int wpr, int n_tiles) {
  const int rows = kRowsWaves / wpr;
  return (B + rows - 1) / rows * n_tiles;
}

size_t rows_lds(int jt, int wpr, int d) { return (size_t)kRowsWaves * jt * 4 + (size_t)(kRowsWaves / wpr) * d * 16 + (LUTKAN_MAX_K + 1) * 4; }

// Four rows per work-group, more work-groups than compute units, and LDS for two on each (up to 1211 inputs on 64-column tiles; LDS is
// handed out in pieces of 1280 bytes): two share a unit, if their registers let them.
bool two_on_a_unit(int64_t B, int n_tiles, int jt, int wpr, int d) {
  return wpr == 4 && rows_groups(B, wpr, n_tiles) > 256 && 2 * round_up((int64_t)rows_lds(jt, wpr, d), 1280) <= lutkan::kLdsPerWorkGroup;
}

// inputs of every group in a round; see launch_rows_depth
int rows_depth(int64_t B, int n_tiles, int jt, int wpr, int d) {
  return (d <= 2 * wpr * (64 / (jt / 4)) || two_on_a_unit(B, n_tiles, jt, wpr, d)) ? 2 : 4;
}

template <int SCHEME, int LPR, int WPR, int DEPTH>
int launch_rows_kernel(const RowsArgs &ra, hipStream_t s) {
  const int64_t groups = rows_groups(ra.B, WPR, ra.n_tiles);
  if (groups > 0x7fffffffLL) return fail(LUTKAN_EUNSUPPORTED, "lutkan_rows_kernel: B * m too large for one launch");
  const size_t lds = rows_lds(4 * LPR, WPR, ra.d);
  static LdsCap raised;
  if (int rc = raise_lds_cap(lutkan_rows_kernel<SCHEME, LPR, WPR, DEPTH>, &raised, "lutkan_rows_kernel")) return rc;
  hipLaunchKernelGGL((lutkan_rows_kernel<SCHEME, LPR, WPR, DEPTH>), dim3((unsigned)groups), dim3(kRowsWaves * 64), lds, s, ra);
  return check_launch("lutkan_rows_kernel");
}

// Two inputs a round where no group has more (a round reads the rows of the inputs that it lacks again), or where more work-groups of four
// rows than compute units wait for one another and the LDS holds two: two run on a unit then, which is worth more than the longer rounds
// (with one on a unit they cost: 1230 -> 64 at 1100 rows 63 -> 76, 1300 -> 64 66 -> 80).  Replayed,
// us, four -> two: 64 -> 1024 at 16 rows 3.75 -> 3.40, 30 -> 700 at 500 20.3 -> 12.2, 11 -> 880 at 422 16.7 -> 9.8; 100 -> 200 at 600 15.4 -> 11.1,
// 64 -> 1000 at 300 17.6 -> 13.0, 450 -> 200 at 300 33.5 -> 29.4, 256 -> 256 at 400 16.4 -> 14.6, 64 -> 64 at 1500 7.3 -> 6.0; but 256 -> 256 at 200 rows
// (200 work-groups) 8.8 -> 10.2, 450 -> 200 at 100 rows with 16 waves a row 11.6 -> 12.0.
template <int SCHEME, int LPR, int WPR>
int launch_rows_depth(const RowsArgs &ra, hipStream_t s) {
  return rows_depth(ra.B, ra.n_tiles, 4 * LPR, WPR, ra.d) == 2 ? launch_rows_kernel<SCHEME, LPR, WPR, 2>(ra, s) : launch_rows_kernel<SCHEME, LPR, WPR, 4>(ra, s);
}

template <int SCHEME, int LPR>
int launch_rows(const RowsArgs &ra, int wpr, hipStream_t s) {
  return wpr == 16 ? launch_rows_depth<SCHEME, LPR, 16>(ra, s) : launch_rows_depth<SCHEME, LPR, 4>(ra, s);
}

template <int SCHEME>
int launch_rows_width(const RowsArgs &ra, int jt, int wpr, hipStream_t s) {
  switch (jt) {
    case 64: return launch_rows<SCHEME, 16>(ra, wpr, s);
    case 32: return launch_rows<SCHEME, 8>(ra, wpr, s);
    case 16: return launch_rows<SCHEME, 4>(ra, wpr, s);
    case 8: return launch_rows<SCHEME, 2>(ra, wpr, s);
    default: return launch_rows<SCHEME, 1>(ra, wpr, s);
  }
}

}  // namespace

namespace lutkan {

// The launch shape by a cost model (microseconds; constants from 30 -> 1000 ... 1024 -> 64 layers at 1 to 4000 rows): 3.5 for
// launch, locate and sum; then 2.9 (3.2 with four rows, 1.6 where two work-groups share a unit) per round of 512 work-groups -- 3.5 more where every input has its own
// knots, read from memory -- and the table bytes a batch requests, in lines of 128, at 15 TB/s, or 1.3 per dependent round
// of a wave's walk over its inputs, whichever is longer.
// (1.6: the passes -> this kernel, replayed, 100 -> 200 at 1000 / 1500 rows 19.1 -> 14.1 / 20.3 -> 18.7, 150 -> 150 at 1000 25.3 -> 19.3, 32 -> 300 at 1500
// 18.0 -> 16.5; not with knots per input where a row's 256 lanes locate more than one input each from memory: 401 -> 64 at 1045 rows 23.7 -> 30.0,
// 793 -> 28 at 1863 35.7 -> 51.2; with 1.4 for all launches of rounds of two 60 -> 100 at 300 rows 4.3 -> 6.6, 8 -> 600 at 1000 10.1 -> 14.7.)
// Against the passes 1.6 is too low for up to 64 inputs that share their knots and several column tiles (one tile: the chain kernel
// leaves its layers to this kernel at this price, and none was slower), whose passes, also priced too high, are a few
// launches without partial sums: 1 -> 272 at 1104 rows 5.8 by the passes and 9.8 here, 2 -> 976 at 290 6.4 and 9.0, 34 -> 1000 at 870 22.0 and 32.5.
// Such a launch is taken if 3.2 a round is less than the passes, or if a price fitted to 240 launches (3.4, 1.8 and 0.6 per input of a group for every round,
// and a quarter of the bytes' time) is less by 5.5, and by 1 less for every 20 inputs: of 1890 drawn calls 1.6 alone moves 85 from the passes (geometric
// mean 0.90 of their time, the worst 1.53), with this 49 at 0.77, the worst 1.22.
RowsPlan rows_plan(const lutkan_dev_layer *l, int64_t B) {
  RowsPlan best{0, 1e300, 1e300};
  if (l->d > kRowsMaxInputs || B > kRowsMaxBatch) return best;
  const BlobLayout lay = blob_layout(l->K, l->L, l->jt, l->scheme, l->value_repr, l->param_dtype);
  const double bytes = (double)B * l->n_tiles * l->d * (std::max(128, 2 * l->jt) + std::max(128, lay.param_row_bytes) + (lay.params_off ? std::max(128, lay.params_off) : 0));
  for (int wpr = 16; wpr >= 4; wpr -= 12) {
    const int row_groups = wpr * (64 / (l->jt / 4)), inputs_per_round = 4 * row_groups;
    const double rounds = (double)rows_groups(B, wpr, l->n_tiles) / 512.0;
    const bool two = two_on_a_unit(B, l->n_tiles, l->jt, wpr, l->d);
    auto priced = [&](double per_round) {
      return 3.5 + std::max(std::max(1.0, rounds) * (per_round + (l->knots_per_input ? 3.5 : 0.0)) + bytes / 15e6, 1.3 * ((l->d + inputs_per_round - 1) / inputs_per_round));
    };
    const double cost = priced(wpr == 16 ? 2.9 : two && !(l->knots_per_input && l->d > 256) ? 1.6 : 3.2);
    if (cost >= best.cost) continue;
    best = RowsPlan{wpr, cost, cost};
    if (two && l->d <= 64 && l->n_tiles > 1 && !l->knots_per_input) {
      const double fitted = 3.4 + rounds * (1.8 + 0.6 * ((l->d + row_groups - 1) / row_groups)) + 0.25 * bytes / 15e6;
      best.against_passes = std::max(cost, std::min(priced(3.2), fitted + 5.5 - l->d / 20.0));
    }
  }
  return best;
}

int rows_forward(const lutkan_dev_layer *l, const RowsPlan &plan, const float *x, int64_t B, float *y, void *hip_stream) {
  const BlobLayout lay = blob_layout(l->K, l->L, l->jt, l->scheme, l->value_repr, l->param_dtype);
  RowsArgs ra = {};
  ra.x = x; ra.table = static_cast<const unsigned char *>(l->table); ra.y = y;
  ra.input_knots = l->knots_per_input ? l->input_knots : nullptr;
  ra.B = B; ra.d = l->d; ra.m = l->m; ra.K = l->K; ra.L = l->L; ra.n_tiles = l->n_tiles; ra.blob_bytes = l->blob_bytes;
  ra.codes_off = lay.codes_off; ra.params_off = lay.params_off;
  ra.closed = (l->boundary == LUTKAN_CLOSED);
  ra.with_base = (l->value_repr == LUTKAN_REPR_SPLINE_COMPONENT);
  ra.param_fp16 = device_params_are_half(l->value_repr, l->param_dtype, l->jt);
  ra.zero_spline = (l->oob == LUTKAN_ZERO_SPLINE);
  ra.t0 = l->knots[0];
  ra.tKs = ra.closed ? l->knots[l->K] : std::nextafterf(l->knots[l->K], -INFINITY);
  ra.masked_below = ra.zero_spline ? ra.t0 : -INFINITY;
  ra.masked_above = ra.zero_spline ? ra.tKs : INFINITY;
  for (int k = 0; k <= l->K; ++k) ra.knots[k] = l->knots[k];
  for (int k = 0; k < LUTKAN_MAX_K; ++k) ra.inner[k] = (k + 1 < l->K) ? l->knots[k + 1] : INFINITY;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int rc = (l->scheme == LUTKAN_SYM_INT8) ? launch_rows_width<LUTKAN_SYM_INT8>(ra, l->jt, plan.waves_per_row, s)
                                                : launch_rows_width<LUTKAN_ASYM_UINT8>(ra, l->jt, plan.waves_per_row, s);
  if (rc) return rc;
  plan_note("rows wpr=%d depth=%d; ", plan.waves_per_row, rows_depth(B, l->n_tiles, l->jt, plan.waves_per_row, l->d));
  return LUTKAN_OK;
}

}  // namespace lutkan
