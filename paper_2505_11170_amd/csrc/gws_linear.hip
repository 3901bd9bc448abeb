// The choice of the GEMM's kernel, and the one for every shape that the others (gws_gemm_stream.hip, gws_gemm128.hip,
// gws_gemm256.hip) do not take or are not faster for: a BF16 MFMA GEMM for gfx950 with an optional GaussWS sampling stage in
// the weight-operand path: Y = X * w_hat (fused; paper Eq. 3 + cast applied to each
// 32x32 block of W on its way from global memory to LDS) or Y = X * W (plain
// twin, same tiling, used as the reference point for the fused overhead).
//
// Tiling.  Workgroup = 256 threads = 2x2 wavefronts, block tile 128 x 128 x 32;
// a wavefront owns 64 x 64 of the output as 2x2 v_mfma_f32_32x32x16_bf16 tiles.
// Both operands sit in LDS K-contiguous ([row][k], 80-byte row pitch), so every
// MFMA operand is one 16-byte LDS read per lane.  BK = 32 = b_l, hence one
// K-step of the weight tile holds whole 32x32 blocks: a wavefront loads exactly
// one block (two 16-byte groups per lane), reduces max|w| across its 64 lanes,
// samples in registers and writes w_hat to LDS.  Global loads for step k+1 are
// issued before the MFMAs of step k.
#include <math.h>

#include "gws_launch.h"

namespace gws {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int BM = 128, BN = 128, BK = 32;
constexpr int LDSP = BK + 8;  // LDS row pitch in elements (80 bytes)

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o));
  return v;
}

union Frag {
  uint4 u;
  bf16x8 v;
};

// W_NK: weight stored [N x K] (K contiguous) instead of [K x N].
template <bool FUSED, int FMT, bool W_NK>
__global__ __launch_bounds__(256) void gemm_kernel(const GemmArgs g) {
  __shared__ __attribute__((aligned(16))) uint16_t As[BM * LDSP];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[BN * LDSP];

  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const uint32_t n_tiles_n = (g.N + BN - 1) / BN;
  const uint32_t tile_m = blockIdx.x / n_tiles_n, tile_n = blockIdx.x % n_tiles_n;
  const uint32_t m0 = tile_m * BM, n0 = tile_n * BN;
  const uint32_t wm = wave >> 1, wn = wave & 1;

  // ---- global -> register staging -------------------------------------------
  // X tile: 128 rows x 32 k = 512 groups of 8; thread: row = tid/4 + 64 i, kgroup = tid%4
  const uint32_t a_kg = tid & 3;
  uint32_t a_row[2];
  const uint16_t* a_ptr[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    a_row[i] = (tid >> 2) + 64 * i;
    uint32_t r = m0 + a_row[i];
    r = r < g.M ? r : g.M - 1;  // clamp: rows past M are computed and discarded
    a_ptr[i] = g.x + (size_t)r * g.ldx + a_kg * 8;
  }
  // W tile: wavefront `wave` owns the 32x32 block at n-offset 32*wave of the tile.
  //   [N x K]: lane -> n = 32 wave + lane/4 + 16 i, k-group = lane%4
  //   [K x N]: lane -> k = lane/4 + 16 i,           n-group = 4 wave + lane%4
  const uint32_t b_q = lane & 3, b_r = lane >> 2;
  const uint32_t blk_n = n0 + 32 * wave;  // first n of this wave's block
  const bool blk_ok = blk_n < g.N;        // N is a multiple of 32: a block is whole or absent
  const uint16_t* b_ptr[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if (W_NK) b_ptr[i] = g.w + (size_t)(blk_ok ? blk_n + b_r + 16 * i : 0) * g.ldw + b_q * 8;
    else b_ptr[i] = g.w + (size_t)(b_r + 16 * i) * g.ldw + (blk_ok ? blk_n + b_q * 8 : 0);
  }
  const uint32_t nbc = W_NK ? (g.K >> 5) : (g.N >> 5);  // blocks per storage row of b_t / scale

  u32x4 ra[2], rb[2];
  auto load_tiles = [&](uint32_t kt) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      ra[i] = *(const u32x4*)(a_ptr[i] + (size_t)kt * BK);
      if (W_NK) rb[i] = *(const u32x4*)(b_ptr[i] + (size_t)kt * BK);
      else rb[i] = *(const u32x4*)(b_ptr[i] + (size_t)kt * BK * g.ldw);
      if (!blk_ok) rb[i] = u32x4{0, 0, 0, 0};
    }
  };

  // Eq. 3 + cast on this wavefront's 32x32 block held in rb[0..1].
  auto sample_block = [&](uint32_t kt) {
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) m = absmax_pk(rb[i], m);
    m = max(m & 0xFFFFu, m >> 16);
    const uint32_t a16 = wave_max_u32(m);
    // storage coordinates of the block: (block row, block col) in the stored matrix
    const uint32_t brow = W_NK ? (blk_n >> 5) : kt;
    const uint32_t bcol = W_NK ? kt : (blk_n >> 5);
    const float btv = blk_ok ? g.bt[(size_t)brow * nbc + bcol] : 0.0f;
    BlockScale b = block_scale(a16, btv);
    if (FMT == 1) cast_constants<8, -6>(a16, b);
    if (FMT == 2) cast_constants<4, -2>(a16, b);
    const bool writer = blk_ok && tile_m == 0 && g.w_hat != nullptr;
    if (writer && lane == 0) g.scale[(size_t)brow * nbc + bcol] = b.s32;
    const bool hw = (FMT == 1) && b.hw_safe;  // uniform: the whole wavefront holds one block
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t srow = (W_NK ? blk_n : kt * 32) + b_r + 16 * i;        // storage row
      const uint32_t scol = (W_NK ? kt * 32 : blk_n) + b_q * 8;             // storage column
      const Noise n = group_noise(g.cg0 + (scol >> 3), g.row0 + srow, g.step_lo, g.step_hi,
                                  g.seed_lo, g.seed_hi);
      rb[i] = hw ? sample_group<FMT>(rb[i], n, b, true) : sample_group<FMT>(rb[i], n, b, false);
      if (writer) *(u32x4*)(g.w_hat + (size_t)srow * g.ldw + scol) = rb[i];
    }
  };

  auto store_lds = [&]() {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      *(u32x4*)(As + a_row[i] * LDSP + a_kg * 8) = ra[i];
      if (W_NK) {
        *(u32x4*)(Bs + (32 * wave + b_r + 16 * i) * LDSP + b_q * 8) = rb[i];
      } else {
        // transpose while storing: the lane holds 8 consecutive n at one k
        const uint32_t e[4] = {rb[i][0], rb[i][1], rb[i][2], rb[i][3]};
        const uint32_t k = b_r + 16 * i, nb = 32 * wave + b_q * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j)
          Bs[(nb + j) * LDSP + k] = (uint16_t)(e[j >> 1] >> ((j & 1) * 16));
      }
    }
  };

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  const uint32_t nk = g.K / BK;
  load_tiles(0);
  for (uint32_t kt = 0; kt < nk; ++kt) {
    if (FUSED) sample_block(kt);
    store_lds();
    __syncthreads();
    if (kt + 1 < nk) load_tiles(kt + 1);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      Frag fa[2], fb[2];
      const uint32_t koff = ks * 16 + (lane >> 5) * 8;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[i].u = *(const uint4*)(As + (64 * wm + 32 * i + (lane & 31)) * LDSP + koff);
        fb[i].u = *(const uint4*)(Bs + (64 * wn + 32 * i + (lane & 31)) * LDSP + koff);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i].v, fb[j].v, acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }

  // ---- epilogue: fp32 -> BF16 (RNE), 32x32 accumulator layout:
  //      acc[e] is row 8*(e/4) + 4*(lane/32) + e%4, column lane%32 of the MFMA tile
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t col = n0 + 64 * wn + 32 * j + (lane & 31);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const uint32_t row = m0 + 64 * wm + 32 * i + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (row < g.M && col < g.N) g.y[(size_t)row * g.ldy + col] = (uint16_t)bf16_rne_bits(acc[i][j][e]);
      }
    }
}

template <bool FUSED, int FMT>
static int launch_layout(const GemmArgs& g, int w_is_nk, dim3 grid, hipStream_t s) {
  if (w_is_nk) hipLaunchKernelGGL((gemm_kernel<FUSED, FMT, true>), grid, dim3(256), 0, s, g);
  else hipLaunchKernelGGL((gemm_kernel<FUSED, FMT, false>), grid, dim3(256), 0, s, g);
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

// Which kernel multiplies.  Chosen by the sizes alone, the same for the plain and the sampling form and whether or not a
// weight rides along, so that the sums over K run in the same order in all of them (the middle, large and narrow tiles and
// the sampling kernel above walk K from end to end; the stream kernels split it).  Estimates in us, fitted to MI355X timings
// of all of them at some thirty sizes.  Rounds are rounds of workgroups, one per compute unit; a K-step is 64 deep.
//   middle: tiles of 128 x 128 or 128 x 96 (34 sizes in both layouts, the choice 0.03 % from the fastest in the mean).  A K-step of a
//     128 x 96 tile takes four fifths of the larger one's: they win where they need no more rounds, or three for two.  W [K x N],
//     128 x 96 and 128 x 128: 4096 x 3072 -> 768 23.7 and 27.7 (256 tiles and 192); 1000 x 768 -> 2304 7.9 and 8.7; 8192 x 2304 -> 768
//     32.8 and 35.9 (two rounds of either; narrow 37); 2048 x 2048 -> 2048 27 and 18.8 (two rounds and one)
//     A middle tile takes a product from the larger ones where a 128 x 128 tile at 0.42 a K-step ([K x N] 0.45) would, or where the
//     estimate is below theirs by more than it errs: 4096 x 2048 -> 1056 28.1 (narrow 33.3), 7000 x 1536 -> 640 23.2 (27.6)
//   stream or one of the others: against that 128 x 128 tile too: the products that the 128 x 96 tile would take from the stream kernel
//     (2500 x 2048 -> 512: 14.8, stream 17.3; 512 x 2304 -> 3072: 15.2 and 15.8) would have fp32 sums four times as long
//   large: 1.05 to 1.25 a K-step, the card's power limit with all compute units at work.  5000 x 2048 -> 2560: 43 (middle 66);
//     8192 x 2048 -> 2048: 50 (69); 8000 x 768 -> 2304: 41 (39); 6000 x 512 -> 1536: 17 (19)
//   narrow (256 x 192): four fifths of the large tile's K-step for three quarters of its columns, where that takes fewer or
//     fuller rounds.  4100 x 4096 -> 4096: 129 (large 161); 8192 x 2048 -> 2560: 77 (94); 8000 x 768 -> 2304: 36 (43);
//     4096 x 768 -> 3072: 22 (25); 8192 x 2048 -> 2048: 71 (54)
GemmRoute gemm_route(const GemmArgs& g, int w_is_nk, RoutePlan& plan) {
  const double cus = compute_units() > 0 ? compute_units() : 256;
  const double nk = ceil(g.K / 64.0);
  auto tiles = [&](double t) { return ceil(g.M / t) * ceil(g.N / t); };
  plan = RoutePlan{{0, 0, 0, 0, 0, 0, 0, 1e30}, 1e30, 1e30, 1e30, 4, 1e30};
  if (gemm256_edge_applicable(g) || gemm256_applicable(g)) {
    const double n = tiles(256.0);
    plan.large_us = 6.0 + ceil(n / cus) * (3.0 + nk * (1.05 + 0.2 * fmin(1.0, n / cus)));
  }
  if (gemm256_edge_applicable(g)) {
    const double n = ceil(g.M / 256.0) * ceil(g.N / 192.0);
    plan.narrow_us = 6.0 + ceil(n / cus) * (3.0 + nk * 0.8 * (1.05 + 0.2 * fmin(1.0, n / cus)));
  }
  if (gemm128_applicable(g)) {
    const double n = tiles(128.0), busy = n > cus ? 1.0 : 0.0;
    plan.middle_line = 3.3 + ceil(n / cus) * (2.0 + nk * (w_is_nk ? 0.42 + 0.05 * busy : 0.45 + 0.07 * busy));
    for (int nj = 3; nj <= 4; ++nj) {
      const double t = ceil(g.M / 128.0) * ceil(g.N / (32.0 * nj));
      const double us = 2.4 + ceil(t / cus) * (2.0 + nk * ((nj == 3 ? 0.26 : 0.33) + 0.08 * fmin(1.0, t / cus) + (w_is_nk ? 0.0 : 0.02)));
      if (us < plan.middle_us) {
        plan.middle_us = us;
        plan.middle_nj = nj;
      }
    }
  }
  if (stream_applicable(g)) plan.stream = stream_plan(g.M, g.N, g.K, w_is_nk != 0);
  const double larger = fmin(plan.large_us, plan.narrow_us);
  if (plan.stream.p > 0 && plan.stream.us < fmin(larger, plan.middle_line)) return GemmRoute::kStream;
  if (fmin(larger, plan.middle_line) > 1e29) return GemmRoute::kSmall;
  if (plan.middle_line < larger || 1.07 * plan.middle_us < larger) return GemmRoute::kMiddle;
  return plan.large_us <= plan.narrow_us ? GemmRoute::kLarge : GemmRoute::kNarrow;
}

// Whether sampling in the operand load beats the sampling kernel and the GEMM behind it: one tile of rows of X (every block
// is then sampled once in either form), where the vector ALU work on the N / 32 workgroups' compute units is shorter than a
// kernel over all of them plus a launch.  Estimates in us from MI355X timings (M = 16 / 64, in-operand and two kernels):
// 512 x 512 7.0 / 6.5 and 9.5; 1024 x 3072 8.3 / 10.0 and 10.6 / 11.1; 2304 x 800 14.8 / 17.0 and 11.3 / 12.5; 2048 x 5632
// 14.7 / 20.1 and 19.0 / 19.7.  A wavefront takes 1.2 a block, with more than 16 rows 1.6; the sampling kernel 3.4 and 0.65
// a million elements, the gap to the next launch 1.5.
bool sample_in_operand(const GemmArgs& g, int w_is_nk) {
  RoutePlan plan;
  if (g.M > 64 || gemm_route(g, w_is_nk, plan) != GemmRoute::kStream) return false;
  const double cus = compute_units() > 0 ? compute_units() : 256;
  const double fused = 3.3 + (g.M <= 16 ? 1.2 : 1.6) * ceil(g.K / 32.0 / plan.stream.p) * ceil(g.N / 32.0 / cus);
  return fused < 0.95 * (3.4 + 0.65e-6 * g.K * g.N + 1.5 + plan.stream.us);
}

// Y on top of an operand.  Where one workgroup makes all of Y it has read the operands before it writes, so a product of one
// tile may be computed in place; the kernels below of smaller tiles would give it to several.
static bool in_place(const GemmArgs& g, int w_is_nk, int fused) {
  const uintptr_t y0 = (uintptr_t)g.y, y1 = y0 + ((size_t)(g.M - 1) * g.ldy + g.N) * 2;
  auto on_y = [&](const void* p, size_t bytes) { return (uintptr_t)p < y1 && y0 < (uintptr_t)p + bytes; };
  const uint32_t rows = w_is_nk ? g.N : g.K, cols = w_is_nk ? g.K : g.N;
  return on_y(g.x, ((size_t)(g.M - 1) * g.ldx + g.K) * 2) || on_y(g.w, ((size_t)(rows - 1) * g.ldw + cols) * 2) ||
         (fused && on_y(g.bt, (size_t)(rows >> 5) * (cols >> 5) * sizeof(float)));
}

GemmForm gemm_form(const GemmArgs& g, int w_is_nk, int fused, RoutePlan& plan) {
  const GemmRoute route = gemm_route(g, w_is_nk, plan);
  if (route == GemmRoute::kStream) return fused ? GemmForm::kStreamSample : GemmForm::kStream;
  if (fused) return rows_sample_applicable(g, w_is_nk) ? GemmForm::kRowsSample : GemmForm::kAnyShapeSample;
  switch (route) {
    case GemmRoute::kMiddle: return GemmForm::kMiddle;
    case GemmRoute::kNarrow: return GemmForm::kNarrow;
    case GemmRoute::kLarge: return gemm256_applicable(g) ? GemmForm::kLarge : GemmForm::kLargeEdge;
    default: return GemmForm::kAnyShape;
  }
}

void gemm_tile(const GemmArgs& g, GemmForm form, const RoutePlan& plan, uint32_t& rows, uint32_t& cols) {
  rows = cols = 256;
  switch (form) {
    case GemmForm::kStream: rows = 16u * plan.stream.mt; cols = 16u * plan.stream.nt; break;
    case GemmForm::kMiddle: rows = 128; cols = 32u * plan.middle_nj; break;
    case GemmForm::kLarge:
    case GemmForm::kLargeEdge: break;
    case GemmForm::kNarrow: cols = 192; break;
    case GemmForm::kStreamSample: rows = stream_sample_rows(g, plan.stream.p); cols = 32; break;
    case GemmForm::kRowsSample: rows = cols = rows_sample_tile(g); break;
    case GemmForm::kAnyShape:
    case GemmForm::kAnyShapeSample: rows = BM; cols = BN; break;
  }
}

int launch_gemm(const GemmArgs& g, int w_is_nk, int fused, int fmt, hipStream_t stream) {
  const uint64_t tiles = (uint64_t)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  if (tiles == 0) return GWS_OK;
  if (tiles >= 0x7FFFFFFFull) return GWS_ERR_SHAPE;
  const dim3 grid((uint32_t)tiles);
  const bool just_sampled = fused == kJustSampled;
  if (just_sampled) fused = 0;
  RoutePlan plan;
  GemmForm form = gemm_form(g, w_is_nk, fused, plan);
  const bool large_tile = !fused && g.M == 256 && g.N == 256 && gemm256_applicable(g);
  if ((tiles == 1 || large_tile) && in_place(g, w_is_nk, fused))
    form = large_tile ? GemmForm::kLarge : fused ? GemmForm::kAnyShapeSample : GemmForm::kAnyShape;
  switch (form) {
    case GemmForm::kStream:
      if (just_sampled) stream_after_sampling(g, w_is_nk, plan.stream);
      return launch_gemm_stream(g, w_is_nk, plan.stream, stream);
    case GemmForm::kMiddle: return launch_gemm128(g, w_is_nk, plan.middle_nj, stream);
    case GemmForm::kLarge: return launch_gemm256(g, w_is_nk, stream);
    case GemmForm::kLargeEdge: return launch_gemm256_edge(g, w_is_nk, stream);
    case GemmForm::kNarrow: return launch_gemm256_narrow(g, w_is_nk, stream);
    case GemmForm::kAnyShape: return launch_layout<false, 0>(g, w_is_nk, grid, stream);
    case GemmForm::kStreamSample: return launch_gemm_stream_sample(g, w_is_nk, fmt, plan.stream.p, stream);
    case GemmForm::kRowsSample: return launch_gemm_rows_sample(g, w_is_nk, fmt, stream);
    case GemmForm::kAnyShapeSample: break;
  }
  switch (fmt) {
    case GWS_FMT_BF16: return launch_layout<true, 0>(g, w_is_nk, grid, stream);
    case GWS_FMT_FP8_E4M3: return launch_layout<true, 1>(g, w_is_nk, grid, stream);
    case GWS_FMT_FP6_E3M2: return launch_layout<true, 2>(g, w_is_nk, grid, stream);
    default: return GWS_ERR_FORMAT;
  }
}

}  // namespace gws
