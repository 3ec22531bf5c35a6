// The LUT layer forward of a narrow layer (one column tile of at most 32 columns) at large batches, in one launch.
//
// On such a layer the passes around the edge kernel cost as much as the edges: per (row, input) the locate kernel reads
// 4 bytes and writes 8, the tiled kernel copies those 8 back and spends only 5 lane-instructions per edge on 2 to 32
// edges, and with one short table slice per input it meets a barrier every few hundred cycles.  Here a wave locates its
// own inputs and hands the result to the lanes of the row in registers, a barrier covers up to 8 inputs, and nothing
// but x, y and the table touches memory.
//
// A wave carries 64/LPR rows, LPR lanes per row with 4 adjacent columns each (as in the tiled kernel).  Inputs are taken
// in blocks of 8: the LPR lanes of a row locate 8/LPR inputs each (steps 1-4 of Sec. 4.5, the arithmetic of the locate
// kernel), turn the segment and the table row into LDS byte offsets, and every lane of the row then receives input s of
// the block from the lane that located it by a DPP broadcast, which rides on the address additions.  Table slices of
// S inputs (8, or 4 for long slices) are contiguous (one column tile: slices are ordered by input) and stream global ->
// LDS into one of two buffers while the other is used.
//
// The arithmetic per edge is that of the tiled kernel on the byte table: codes as binary16 denormals, one mixed-precision
// multiply-add for the interpolation, one for the scale; the running sums carry 2^-24.  Sums run over the 8 inputs of a block,
// then over the blocks, which keeps them nearer to a 64-bit evaluation than the tiled kernel's chunks (78 -> 16 at 65536 rows
// 1.1e-7 against 1.4e-7; as one running sum it was 2.4e-7).
//
// Bound: vector issue and waits.  A block is about 150 instructions for its edges (132 with symmetric codes) and 45 for each input a
// lane locates (35 on grids of up to five segments; 66 before the segments' reciprocals, 78 -> 16 at 65536 rows 34.6 -> 31.1), at 6.2 cycles per instruction and SIMD with four waves (the 16-byte code rows of 16 rows collide in the
// LDS banks).  Whole layers, locate + tiled + sum -> this kernel, microseconds: 78 -> 16, uint8 codes, L = 64, at 65536 rows
// 49 -> 33; 16 -> 2 at 131072 rows 24 -> 11; 64 -> 8 at 131072 rows, L = 32, 51 -> 30, with spline_component 68 -> 42; 1000 -> 4 at
// 20000 rows 109 -> 73; 100 -> 30 at 65536 rows 81 -> 56; 300 -> 10 at 1000 rows 19 -> 14.
// The file is compiled with -ffp-contract=off; every fused multiply-add is written out as fmaf().
#include "lutkan_device.h"
#include "lutkan_locate.h"
#include "lutkan_narrow.h"

namespace {

constexpr int kBlock = 8;                // inputs located at a time

struct NarrowArgs {
  const float *x;                        // [B][d]
  const unsigned char *table;            // one column tile: slice of input i at i * blob_bytes
  float *y;
  int64_t B;
  int32_t d, m, K, L, jt, blob_bytes;
  int32_t codes_off, params_off;
  int32_t chunk;                         // inputs per work-group (blockIdx.y), a multiple of 8
  int64_t split_stride;
  float t0, tKs;
  float masked_below, masked_above;      // zero_spline: inputs outside contribute nothing; clip_x: -inf, +inf
  uint32_t last_divided;                 // see last_divided()
  float inner[LUTKAN_MAX_K];             // the inner knots T[1] .. T[K-1], +inf past the last
  float knots[LUTKAN_MAX_K + 1];
};

// lane `from` of every group of LPR lanes, to all lanes of the group (LPR = 1, 2, 4, 8)
template <int LPR, int from>
__device__ __forceinline__ unsigned from_lane(unsigned v) {
  static_assert(from < LPR, "a lane of the group");
  if constexpr (LPR == 1) return v;
  else if constexpr (LPR == 2) return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, from | (from << 2) | ((2 + from) << 4) | ((2 + from) << 6), 0xf, 0xf, true);
  else if constexpr (LPR == 4) return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, from * 0x55, 0xf, 0xf, true);   // quad_perm, the same lane four times
  else {
    // row_newbcast of a lane of the lower, then of the upper eight of every 16; the bank mask picks the lanes written
    const int lower = __builtin_amdgcn_update_dpp(0, (int)v, 0x150 + from, 0xf, 0x3, false);
    return (unsigned)__builtin_amdgcn_update_dpp(lower, (int)v, 0x150 + 8 + from, 0xf, 0xc, false);
  }
}

template <int SCHEME, int LPR, int S, int NW, bool BASE, bool PH>
__global__ __launch_bounds__(NW * 64) void lutkan_narrow_kernel(const NarrowArgs a) {
  static_assert(!(BASE && PH), "with the base branch the device table holds fp32 products, never binary16 parameters");
  static_assert(kBlock % LPR == 0 && kBlock % S == 0, "whole elements per lane, whole stages per block");
  constexpr int VEC = kBlock / LPR;      // inputs a lane locates per block
  constexpr int RPS = 64 / LPR;
  constexpr int PSZ = PH ? 8 : 16, PLANE = 4 * LPR * (PH ? 2 : 4), kParamRow = PLANE * (SCHEME == LUTKAN_ASYM_UINT8 ? 2 : 1);
  extern __shared__ __align__(16) unsigned char lds[];
  f32x4 *const s_seg = reinterpret_cast<f32x4 *>(lds + 2 * S * a.blob_bytes);
  typedef const __attribute__((address_space(3))) unsigned char *lds_bytes;
  typedef const __attribute__((address_space(3))) unsigned *lds_u32;
  typedef const __attribute__((address_space(3))) u32x2 *lds_u32x2;
  typedef const __attribute__((address_space(3))) f32x4 *lds_f32x4;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sub = lane & (LPR - 1);
  const int64_t b = ((int64_t)blockIdx.x * NW + wave) * RPS + lane / LPR;
  const float *xrow = a.x + min(b, a.B - 1) * a.d;
  const int i_begin = blockIdx.y * a.chunk;
  const int i_end = min(a.d, i_begin + a.chunk);
  const unsigned stage_bytes = S * a.blob_bytes;
  const unsigned lane_off = lane * 16;
  fill_segments(a, s_seg, tid);

  // the slices of the up to S inputs from i on, one contiguous run
  auto stage = [&](int i, int buf) {
    stage_slice<NW>(a.table + (size_t)i * a.blob_bytes, lds + buf * stage_bytes, (min(S, i_end - i) * a.blob_bytes) >> 4, wave, lane, lane_off);
  };
  float xv[VEC];
  auto load_x = [&](int i0) {            // this lane's inputs of the block that starts at i0: consecutive ones of its row
    const float *src = xrow + i0 + sub * VEC;
    if (i0 + kBlock <= a.d) {
      __builtin_memcpy(xv, src, sizeof(xv));             // (rows need not be aligned to more than 4 bytes)
    } else {
#pragma unroll
      for (int v = 0; v < VEC; ++v) xv[v] = src[min(v, a.d - 1 - (i0 + sub * VEC))];
    }
  };
  stage(i_begin, 0);
  load_x(i_begin);
  wait_all_vector_loads();
  __syncthreads();

  // the sum over a block's inputs, and over the blocks: short sums of short sums round less than one long one
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f}, total[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  const unsigned lds_base = (unsigned)(uintptr_t)(lds_bytes)lds;
  int cur = 0;
  for (int i0 = i_begin; i0 < i_end; i0 += kBlock) {
    // ---- locate this lane's inputs of the block: byte offsets of their code row and parameter row inside their stage
    unsigned code_at[VEC], param_at[VEC], weight[VEC], silu[VEC];
    int k[VEC], l0[VEC];
    float w[VEC];
    locate_side_by_side<VEC>(a, s_seg, xv, k, l0, w);
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      const int s = sub * VEC + v;
      const bool dead = i0 + s >= i_end;
      const bool masked = dead | (xv[v] < a.masked_below) | (xv[v] > a.masked_above);
      // a masked input reads its slice's all-zero rows, one past the last input those of its stage's first slice
      const int slice = dead ? 0 : (s % S) * a.blob_bytes;
      int located = (int)__umul24(k[v], a.L) + l0[v];
      asm("" : "+v"(located));             // (computed for every lane: a select, not a branch around three instructions)
      const int row = masked ? a.K * a.L : located, segment = masked ? a.K : k[v];
      code_at[v] = (unsigned)(slice + a.codes_off + row * (4 * LPR));
      param_at[v] = (unsigned)(slice + a.params_off + segment * kParamRow);
      weight[v] = masked ? 0u : __float_as_uint(w[v]);
      silu[v] = 0u;
      if constexpr (BASE) {
        const float sx = __fdiv_rn(xv[v], 1.0f + expf(-xv[v]));                     // at the raw input, never masked
        silu[v] = dead ? 0u : __float_as_uint(sx);
      }
    }
    load_x(min(i0 + kBlock, i_end - 1));                   // (past the end: something valid, unused)

    auto edges_of = [&](auto input, unsigned col_codes, unsigned col_params, unsigned base_at) {
      constexpr int s = decltype(input)::value, from = s / VEC, v = s % VEC;
      const unsigned code_addr = from_lane<LPR, from>(code_at[v]) + col_codes;
      const unsigned param_addr = from_lane<LPR, from>(param_at[v]) + col_params;
      const float w = __uint_as_float(from_lane<LPR, from>(weight[v]));
      const unsigned c0 = *(lds_u32)(lds_bytes)(uintptr_t)code_addr;
      const unsigned c1 = *(lds_u32)((lds_bytes)(uintptr_t)code_addr + 4 * LPR);
      lds_bytes pp = (lds_bytes)(uintptr_t)param_addr;
      float al[4], ym[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if constexpr (PH) {
        union { unsigned u; f16x2 h; } lo, hi;
        const u32x2 ha = *(lds_u32x2)pp;
        lo.u = ha.x; hi.u = ha.y;
        al[0] = (float)lo.h.x; al[1] = (float)lo.h.y; al[2] = (float)hi.h.x; al[3] = (float)hi.h.y;
        if (SCHEME == LUTKAN_ASYM_UINT8) {
          const u32x2 hy = *(lds_u32x2)(pp + PLANE);
          lo.u = hy.x; hi.u = hy.y;
          ym[0] = (float)lo.h.x; ym[1] = (float)lo.h.y; ym[2] = (float)hi.h.x; ym[3] = (float)hi.h.y;
        }
      } else {
        const f32x4 pa = *(lds_f32x4)pp;
        al[0] = pa.x; al[1] = pa.y; al[2] = pa.z; al[3] = pa.w;
        if (SCHEME == LUTKAN_ASYM_UINT8) {
          const f32x4 pb = *(lds_f32x4)(pp + PLANE);
          ym[0] = pb.x; ym[1] = pb.y; ym[2] = pb.z; ym[3] = pb.w;
        }
      }
      float t[4];
      interpolate_codes<SCHEME>(c0, c1, w, t);
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = fmaf(al[c], t[c], acc[c]);
      if (SCHEME == LUTKAN_ASYM_UINT8) {
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = fmaf(ym[c], kTwoToMinus24, acc[c]);
      }
      if constexpr (BASE) {
        const f32x4 gain = *(lds_f32x4)(lds_bytes)(uintptr_t)base_at * kTwoToMinus24;
        const float sx = __uint_as_float(from_lane<LPR, from>(silu[v]));
        acc[0] = fmaf(gain.x, sx, acc[0]); acc[1] = fmaf(gain.y, sx, acc[1]);
        acc[2] = fmaf(gain.z, sx, acc[2]); acc[3] = fmaf(gain.w, sx, acc[3]);
      }
    };

    // ---- the block's stages: the next one streams into the other buffer while this one is used
#pragma unroll
    for (int part = 0; part < kBlock / S; ++part) {
      const int i = i0 + part * S;
      if (part > 0 && i >= i_end) break;                 // uniform over the work-group
      if (i + S < i_end) stage(i + S, cur ^ 1);
      const unsigned buf = lds_base + cur * stage_bytes;
      const unsigned col_codes = buf + sub * 4, col_params = buf + sub * PSZ;
      auto slice_base = [&](int s) { return buf + (unsigned)(i + s < i_end ? s : 0) * (unsigned)a.blob_bytes + sub * 16; };
      auto unroll = [&](auto self, auto n) -> void {
        constexpr int s = decltype(n)::value;
        if constexpr (s < S) {
          if (part == 0) edges_of(std::integral_constant<int, s>{}, col_codes, col_params, slice_base(s));
          else edges_of(std::integral_constant<int, (kBlock / S > 1 ? S + s : s)>{}, col_codes, col_params, slice_base(s));
          self(self, std::integral_constant<int, s + 1>{});
        }
      };
      unroll(unroll, std::integral_constant<int, 0>{});
      if (i + S < i_end) {
        wait_all_vector_loads();                           // my share of the next stage has landed ...
        lds_barrier();                                     // ... everyone's has, and everyone is done with this one
        cur ^= 1;
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      total[c] += acc[c];
      acc[c] = 0.0f;
    }
  }

  if (b >= a.B) return;
  const int j = sub * 4;
  float *yout = a.y + (int64_t)blockIdx.y * a.split_stride + b * a.m + j;
#pragma unroll
  for (int c = 0; c < 4; ++c) total[c] *= kTwoTo24;          // exact: undo the 2^-24 of the codes
  if (j + 3 < a.m && (a.m & 3) == 0) {
    *reinterpret_cast<f32x4 *>(yout) = f32x4{total[0], total[1], total[2], total[3]};
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (j + c < a.m) yout[c] = total[c];
  }
}

inline size_t narrow_lds_bytes(int stage, int blob_bytes, int K) { return 2 * (size_t)stage * blob_bytes + (size_t)K * 16; }

// Inputs per stage: 8 or 4, as two stages fit the LDS; 0: this kernel does not serve the layer.  With the base branch 4: the
// reads of eight inputs and their base rows together do not fit the registers of 16 waves.
int narrow_stage(const lutkan_dev_layer *l, bool base) {
  if (l->n_tiles != 1 || l->jt > 32 || l->knots_per_input) return 0;
  if (!base && narrow_lds_bytes(8, l->blob_bytes, l->K) <= (size_t)kMaxTiledLds) return 8;
  if (!base && l->jt < 16) return 0;                       // (slices of 4 and 8 columns that long are not built for)
  return narrow_lds_bytes(4, l->blob_bytes, l->K) <= (size_t)kMaxTiledLds ? 4 : 0;
}

template <int SCHEME, int LPR, int S, int NW>
int launch_narrow(const NarrowArgs &na, bool base, bool half_params, int n_split, hipStream_t s) {
  constexpr int kRows = NW * (64 / LPR);
  const int64_t groups = (na.B + kRows - 1) / kRows;
  if (groups > 0x7fffffffLL) return fail(LUTKAN_EUNSUPPORTED, "lutkan_narrow_kernel: B too large for one launch");
  const dim3 grid((unsigned)groups, (unsigned)n_split);
  const size_t lds = narrow_lds_bytes(S, na.blob_bytes, na.K);
#define LUTKAN_LAUNCH_NARROW(BASE, PH)                                                                                            \
  do {                                                                                                                            \
    static LdsCap raised;                                                                                                         \
    if (int rc = raise_lds_cap(lutkan_narrow_kernel<SCHEME, LPR, S, NW, BASE, PH>, &raised, "lutkan_narrow_kernel")) return rc;    \
    hipLaunchKernelGGL((lutkan_narrow_kernel<SCHEME, LPR, S, NW, BASE, PH>), grid, dim3(NW * 64), lds, s, na);                     \
    return check_launch("lutkan_narrow_kernel");                                                                                  \
  } while (0)
  if constexpr (S == 4) { if (base) LUTKAN_LAUNCH_NARROW(true, false); }       // (narrow_stage: with the base branch always 4)
  if constexpr (S == 8 || LPR >= 4) {
    if (half_params) LUTKAN_LAUNCH_NARROW(false, true);
    LUTKAN_LAUNCH_NARROW(false, false);
  }
#undef LUTKAN_LAUNCH_NARROW
  return fail(LUTKAN_EUNSUPPORTED, "lutkan_narrow_kernel: no such variant");
}

template <int SCHEME, int LPR, int NW>
int launch_narrow_stage(const NarrowArgs &na, int stage, bool base, bool half_params, int n_split, hipStream_t s) {
  return stage == 4 ? launch_narrow<SCHEME, LPR, 4, NW>(na, base, half_params, n_split, s) : launch_narrow<SCHEME, LPR, 8, NW>(na, base, half_params, n_split, s);
}

template <int SCHEME, int NW>
int launch_narrow_width(const NarrowArgs &na, int stage, bool base, bool half_params, int n_split, hipStream_t s) {
  switch (na.jt) {
    case 4: return launch_narrow_stage<SCHEME, 1, NW>(na, stage, base, half_params, n_split, s);
    case 8: return launch_narrow_stage<SCHEME, 2, NW>(na, stage, base, half_params, n_split, s);
    case 16: return launch_narrow_stage<SCHEME, 4, NW>(na, stage, base, half_params, n_split, s);
    default: return launch_narrow_stage<SCHEME, 8, NW>(na, stage, base, half_params, n_split, s);
  }
}

}  // namespace

namespace lutkan {

// The launch shape by a cost model (microseconds, constants from 16 -> 2 ... 1000 -> 4 layers at 1000 to 131072 rows): a block
// of 8 inputs costs a SIMD 6.2 cycles for each of its waves' instructions (5.2 with the 32-byte code rows, which collide less
// in the LDS banks: 5.1 to 5.4 measured on 100 -> 30, 128 -> 32 and 200 -> 24; 4.7 if symmetric and eight waves share the
// SIMD), at least 13 for each of one wave's (alone on its SIMD a wave waits for its own results: 1000 -> 4 at 65536 rows) and
// 2000 a stage (the slices' way from L2); a work-group 3 us of fill; as many work-groups share a compute unit as the LDS
// holds; chunks of inputs add the summing pass.  Half the stage where that lets a second symmetric work-group of 32-byte rows
// share the unit: 100 -> 30, L = 32, at 131072 rows 99 us against 118, at 65536 54 against 60 (unsymmetric codes lose: 128 -> 32
// 83 against 75).
NarrowPlan narrow_plan(const lutkan_dev_layer *l, int64_t B, size_t workspace_bytes) {
  NarrowPlan best{0, 1, l->d, 0, 1e300};
  const bool base = (l->value_repr == LUTKAN_REPR_SPLINE_COMPONENT), symmetric = (l->scheme == LUTKAN_SYM_INT8);
  const int widest = narrow_stage(l, base);
  if (!widest) return best;
  const int lpr = l->jt / 4, vec = kBlock / lpr;
  const double instructions = (symmetric ? 132 : 150) + 45 * vec + (lpr == 8 ? 56 : 0) + (base ? 60 + 25 * vec : 0);
  for (int waves = 4; waves <= 16; waves += 12) {          // (fewer on a tie: their barriers hold up less; 64 -> 8 at 131072 rows 30 against 33)
    const int64_t groups = (B + (int64_t)waves * (64 / lpr) - 1) / ((int64_t)waves * (64 / lpr));
    for (int stage = widest; stage >= (symmetric && lpr == 8 && waves == 16 ? 4 : widest); stage -= 4) {
      const int resident = (int)std::min<size_t>(32 / waves, kMaxTiledLds / narrow_lds_bytes(stage, l->blob_bytes, l->K));
      for (int want = 1; want <= 64; ++want) {
        const int chunk = (int)round_up((l->d + want - 1) / want, kBlock);
        const int split = (l->d + chunk - 1) / chunk;
        if (split > 1 && (size_t)split * (size_t)B * (size_t)l->m * 4 > workspace_bytes) break;
        const double per_unit = (double)((groups * split + 255) / 256);              // work-groups per compute unit
        const double together = std::min((double)resident, per_unit);
        const double cycles = lpr < 8 ? 6.2 : symmetric && together * waves >= 32 ? 4.7 : stage == 4 ? 5.6 : 5.2;
        const double block = std::max(std::max(2000.0 * kBlock / stage, 13.0 * instructions), cycles * instructions * together * waves / 4.0) / 2400.0;
        double cost = std::ceil(per_unit / together) * (3.0 + chunk / kBlock * block);
        if (split > 1) cost += 4.0 + (double)split * (double)B * l->m * 4.0 / 3e6;
        if (cost < best.cost) best = NarrowPlan{waves, split, chunk, stage, cost};
        if (chunk <= kBlock) break;
      }
    }
  }
  return best;
}

int narrow_forward(const lutkan_dev_layer *l, const NarrowPlan &plan, const float *x, int64_t B, float *y, void *workspace, void *hip_stream) {
  const BlobLayout lay = blob_layout(l->K, l->L, l->jt, l->scheme, l->value_repr, l->param_dtype);
  NarrowArgs na = {};
  na.x = x; na.table = static_cast<const unsigned char *>(l->table); na.y = y;
  na.B = B; na.d = l->d; na.m = l->m; na.K = l->K; na.L = l->L; na.jt = l->jt; na.blob_bytes = l->blob_bytes;
  na.codes_off = lay.codes_off; na.params_off = lay.params_off;
  na.t0 = l->knots[0];
  na.tKs = (l->boundary == LUTKAN_CLOSED) ? l->knots[l->K] : std::nextafterf(l->knots[l->K], -INFINITY);
  na.masked_below = (l->oob == LUTKAN_ZERO_SPLINE) ? na.t0 : -INFINITY;
  na.masked_above = (l->oob == LUTKAN_ZERO_SPLINE) ? na.tKs : INFINITY;
  for (int k = 0; k <= l->K; ++k) na.knots[k] = l->knots[k];
  for (int k = 0; k < LUTKAN_MAX_K; ++k) na.inner[k] = (k + 1 < l->K) ? l->knots[k + 1] : INFINITY;
  na.last_divided = last_divided(l->knots, l->K);
  na.chunk = plan.chunk;
  float *const partials = static_cast<float *>(workspace);
  if (plan.n_split > 1) { na.y = partials; na.split_stride = B * l->m; }
  const bool base = (l->value_repr == LUTKAN_REPR_SPLINE_COMPONENT), half_params = device_params_are_half(l->value_repr, l->param_dtype, l->jt);
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  int rc;
  if (l->scheme == LUTKAN_SYM_INT8)
    rc = plan.waves == 16 ? launch_narrow_width<LUTKAN_SYM_INT8, 16>(na, plan.stage, base, half_params, plan.n_split, s)
                          : launch_narrow_width<LUTKAN_SYM_INT8, 4>(na, plan.stage, base, half_params, plan.n_split, s);
  else
    rc = plan.waves == 16 ? launch_narrow_width<LUTKAN_ASYM_UINT8, 16>(na, plan.stage, base, half_params, plan.n_split, s)
                          : launch_narrow_width<LUTKAN_ASYM_UINT8, 4>(na, plan.stage, base, half_params, plan.n_split, s);
  if (rc) return rc;
  plan_note("narrow split=%d waves=%d; ", plan.n_split, plan.waves);
  if (plan.n_split == 1) return LUTKAN_OK;
  const int64_t n = B * l->m;
  hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, s, partials, y, n, plan.n_split, 0);
  plan_note("sum; ");
  return check_launch("sum_partials_kernel");
}

}  // namespace lutkan
