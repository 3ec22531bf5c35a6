// The base branch of value_repr = spline_component (Eq. 2) for a whole layer as one dense contraction on the matrix
// cores:  Y0[b][j] = sum_i SiLU(x[b][i]) * (s_out * s_base)[i][j].  It is the one piece of the layer forward without
// a gather: a [B, d] x [d, m] product.  The LUT edge kernel then adds the spline branch on top of Y0.
//
// fp32 accuracy from bf16 matrix instructions: every fp32 operand is cut, exactly, into three bf16 pieces of eight
// significand bits each (a = a_h + a_m + a_l, nothing is lost), and the product is accumulated in fp32 from the six piece
// products h*h, h*m, m*h, m*m, h*l, l*h; the other three are at most 2^-24 of it together (lutkan_pieces.h).  bf16 has the
// exponent range of fp32, so no scaling is needed.  A non-finite SiLU(x) keeps its class in the high piece; its row comes out
// non-finite (NaN where an edge-by-edge evaluation may give +-inf).
//
// Both operands arrive already cut: SiLU(x) by the locate kernel (lutkan_cut3 below, three planes [piece][row][input]),
// s_out*s_base by lutkan_base_pieces_kernel from the base rows of the LUT device table (three planes
// [piece][column][input]); in both the inputs are contiguous, which is the operand order of the matrix instruction
// (a lane holds 8 consecutive k of one row resp. column).  One work-group of 512 threads computes a 128 x 128 tile of
// Y0, its eight waves 64 x 32 each as two tiles of v_mfma_f32_32x32x16_bf16; the inputs are walked 32 at a time: 48 KiB
// of pieces go global -> registers -> one of two LDS buffers (the loads of the next step are in flight while this step
// multiplies, one barrier a step), each wave then reads its operands with 16-byte LDS reads.
//
// Bound: LDS and matrix issue, about 12 us each of 512 -> 512 at 8192 rows, and the barriers between: 32 us, 0.8 PFLOP/s.  With four
// waves of 64 x 64 (one per SIMD where a launch has 256 tiles), one buffer and the column tiles of a row tile spread over the XCDs
// 39; loads two steps ahead 32.  The layer 321 -> 316 us, 1024 -> 1024, G = 10, 1356 -> 1346, 512 -> 300 at 5000 rows 195 -> 190.
#include "lutkan_device.h"
#include "lutkan_pieces.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kBM = 128, kBN = 128, kBK = 32, kGemmWaves = 8;
constexpr int kLdk = kBK + 8;            // bf16 elements per LDS row: 80 bytes, so that the 16 rows of a 16-byte read group fall into different banks
constexpr int kVecPerStep = 3 * kBM * kBK * 2 / 16;      // 16-byte vectors of one operand per k step: 1536, three per thread

struct BasePiecesArgs {
  const unsigned char *table;        // LUT device table: slice (t, i) starts with the jt floats s_out*s_base of its columns
  uint16_t *w_pieces;                // [3][m_pad][d] bf16 bit patterns, rows m .. m_pad-1 zero
  int32_t d, m, m_pad, jt_log2, blob_bytes;
};

// One thread per (column, group of 8 inputs): adjacent threads take adjacent columns, so the eight 4-byte reads of a
// wave are contiguous runs of the base rows; each thread writes three 16-byte vectors.
__global__ __launch_bounds__(256) void lutkan_base_pieces_kernel(const BasePiecesArgs a) {
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int j = (int)(g % a.m_pad);
  const int k = (int)(g / a.m_pad) * 8;
  if (k >= a.d) return;
  unsigned h[8], m[8], l[8];
  const unsigned char *w = a.table + ((size_t)(j >> a.jt_log2) * a.d + k) * a.blob_bytes + (size_t)(j & ((1 << a.jt_log2) - 1)) * 4;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float v = (j < a.m) ? *reinterpret_cast<const float *>(w + (size_t)e * a.blob_bytes) : 0.0f;   // d is a multiple of 32
    lutkan_cut3(v, h[e], m[e], l[e]);
  }
  const size_t plane = (size_t)a.m_pad * a.d;
  uint16_t *dst = a.w_pieces + (size_t)j * a.d + k;
  *reinterpret_cast<u32x4 *>(dst) = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
  *reinterpret_cast<u32x4 *>(dst + plane) = u32x4{m[0] | (m[1] << 16), m[2] | (m[3] << 16), m[4] | (m[5] << 16), m[6] | (m[7] << 16)};
  *reinterpret_cast<u32x4 *>(dst + 2 * plane) = u32x4{l[0] | (l[1] << 16), l[2] | (l[3] << 16), l[4] | (l[5] << 16), l[6] | (l[7] << 16)};
}

struct BaseGemmArgs {
  const uint16_t *a_pieces;          // [3][Bp][d]: SiLU(x) cut into pieces, rows B .. Bp-1 zero (Bp a multiple of 128)
  const uint16_t *w_pieces;          // [3][m_pad][d]
  float *y;                          // [B][m]
  int64_t B, Bp;
  int32_t d, m, m_pad;
};

__global__ __launch_bounds__(kGemmWaves * 64) void lutkan_base_gemm_kernel(const BaseGemmArgs a) {
  static_assert(kBM == kBN, "both operand tiles share one LDS shape");
  extern __shared__ __align__(16) uint16_t lds[];       // two buffers of [operand][piece][row or column][kLdk]
  constexpr int kTile = 3 * kBM * kLdk, kBuffer = 2 * kTile, kThreads = kGemmWaves * 64, kPer = kVecPerStep / kThreads;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wr = wave >> 2, wc = wave & 3;               // this wave's 64 x 32 eighth of the tile
  // The column tiles of a row tile run on one XCD (work-groups go to the eight in turn) and find its SiLU pieces in that L2: row
  // tiles in groups of eight, the row tile the fastest of a group's indices.
  const unsigned col_tiles = a.m_pad / kBN, row_tiles = (unsigned)((a.B + kBM - 1) / kBM);
  const unsigned in_groups = row_tiles / 8 * 8 * col_tiles, rest = row_tiles % 8;
  unsigned row_tile, col_tile;
  if (blockIdx.x < in_groups) {
    const unsigned in = blockIdx.x % (8 * col_tiles);
    row_tile = blockIdx.x / (8 * col_tiles) * 8 + in % 8;
    col_tile = in / 8;
  } else {
    row_tile = row_tiles - rest + (blockIdx.x - in_groups) % rest;
    col_tile = (blockIdx.x - in_groups) / rest;
  }
  const int64_t row0 = (int64_t)row_tile * kBM;
  const int col0 = (int)col_tile * kBN;

  f32x16 acc[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[rt][v] = 0.0f;

  // this thread's vectors of each operand tile: vector v = tid + threads * q is piece v / 512, row (v % 512) / 4,
  // inputs 8 * (v % 4) .. + 7 of the step (four adjacent threads read the 64 contiguous bytes of one row)
  static_assert(kVecPerStep % kThreads == 0, "whole vectors per thread and operand");
  const uint16_t *ga[kPer], *gw[kPer];
  int at[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int v = tid + kThreads * q;
    const int piece = v >> 9, r = (v & 511) >> 2, k8 = (v & 3) * 8;
    ga[q] = a.a_pieces + ((size_t)piece * a.Bp + row0 + r) * a.d + k8;
    gw[q] = a.w_pieces + ((size_t)piece * a.m_pad + col0 + r) * a.d + k8;
    at[q] = (piece * kBM + r) * kLdk + k8;
  }
  u32x4 ra[kPer], rw[kPer];
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < kPer; ++q) { ra[q] = *reinterpret_cast<const u32x4 *>(ga[q] + k0); rw[q] = *reinterpret_cast<const u32x4 *>(gw[q] + k0); }
  };
  auto store = [&](uint16_t *buf) {
#pragma unroll
    for (int q = 0; q < kPer; ++q) { *reinterpret_cast<u32x4 *>(buf + at[q]) = ra[q]; *reinterpret_cast<u32x4 *>(buf + kTile + at[q]) = rw[q]; }
  };
  load(0);
  store(lds);
  if (kBK < a.d) load(kBK);
  __syncthreads();

  int cur = 0;
  for (int k0 = 0; k0 < a.d; k0 += kBK) {
    const uint16_t *sA = lds + cur * kBuffer + (wr * 64 + (lane & 31)) * kLdk, *sW = lds + cur * kBuffer + kTile + (wc * 32 + (lane & 31)) * kLdk;
    // ---- 2 k sub-steps of 16: a lane holds 8 consecutive k of row resp. column lane % 32, k offset 8 * (lane / 32)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int kk = ks * 16 + (lane >> 5) * 8;
      bf16x8 af[2][3], wf[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        wf[p] = *reinterpret_cast<const bf16x8 *>(sW + p * kBN * kLdk + kk);
#pragma unroll
        for (int t = 0; t < 2; ++t) af[t][p] = *reinterpret_cast<const bf16x8 *>(sA + (p * kBM + t * 32) * kLdk + kk);
      }
      // the six piece products, the small ones first; the two accumulators take turns
      constexpr int kPieceOfA[6] = {2, 0, 1, 1, 0, 0}, kPieceOfW[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int p = 0; p < 6; ++p)
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
          acc[rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[rt][kPieceOfA[p]], wf[kPieceOfW[p]], acc[rt], 0, 0, 0);
    }
    if (k0 + kBK < a.d) {
      store(lds + (cur ^ 1) * kBuffer);                  // (everyone left that buffer before the last barrier)
      if (k0 + 2 * kBK < a.d) load(k0 + 2 * kBK);        // travels while the next step multiplies
    }
    // orders LDS traffic only: the loads stay in flight
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    cur ^= 1;
  }

  // ---- the accumulator of a 32 x 32 tile: element v of a lane is row 8*(v/4) + 4*(lane/32) + v%4, column lane%32
  const int j = col0 + wc * 32 + (lane & 31);
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t b = row0 + wr * 64 + rt * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
      if (b < a.B && j < a.m) a.y[b * a.m + j] = acc[rt][v];
    }
}

inline int32_t padded_columns(int32_t m) { return (m + kBN - 1) / kBN * kBN; }

}  // namespace

namespace lutkan {

// A launch holds fewer than 2^32 threads.  Batches beyond 65535 row tiles leave the base branch in the edge kernel: it serves them as fast
// or faster (32 -> 64 at 8388865 rows 4.09 ms against 5.02 by the product, 64 -> 128 12.07 against 12.08).
bool base_product_fits(int32_t d, int32_t m, int64_t B) {
  const int64_t row_tiles = (B + kBM - 1) / kBM;
  return d % kBK == 0 && m >= 64 && row_tiles <= 65535 && row_tiles * (padded_columns(m) / kBN) * (kGemmWaves * 64) <= 0xffffffffLL;
}

size_t base_product_workspace_bytes(int32_t d, int32_t m) {
  return base_product_fits(d, m, 1) ? ((size_t)6 * padded_columns(m) * d + 255) / 256 * 256 : 0;
}

int launch_base_product(const uint16_t *silu_pieces, int64_t Bp, const void *table, uint16_t *w_pieces, int32_t d, int32_t m, int32_t jt,
                        int32_t blob_bytes, int64_t B, float *y, void *hip_stream, const char *who) {
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  BasePiecesArgs p;
  p.table = static_cast<const unsigned char *>(table);
  p.w_pieces = w_pieces;
  p.d = d; p.m = m; p.m_pad = padded_columns(m); p.blob_bytes = blob_bytes;
  p.jt_log2 = 0;
  while ((1 << p.jt_log2) < jt) ++p.jt_log2;
  const int64_t groups = ((int64_t)p.m_pad * (d / 8) + 255) / 256;
  hipLaunchKernelGGL(lutkan_base_pieces_kernel, dim3((unsigned)groups), dim3(256), 0, s, p);
  BaseGemmArgs a;
  a.a_pieces = silu_pieces; a.w_pieces = w_pieces; a.y = y;
  a.B = B; a.Bp = Bp; a.d = d; a.m = m; a.m_pad = p.m_pad;
  constexpr size_t lds = 2 * 2 * 3 * kBM * kLdk * sizeof(uint16_t);
  static LdsCap raised;
  if (int rc = raise_lds_cap(lutkan_base_gemm_kernel, &raised, who)) return rc;
  hipLaunchKernelGGL(lutkan_base_gemm_kernel, dim3((unsigned)(p.m_pad / kBN * ((B + kBM - 1) / kBM))), dim3(kGemmWaves * 64), lds, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(LUTKAN_EHIP, "%s: base-branch product: %s", who, hipGetErrorString(e));
  return LUTKAN_OK;
}

}  // namespace lutkan
