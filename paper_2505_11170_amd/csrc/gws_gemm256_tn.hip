// Weight-gradient GEMM of the sampled-weight linear for gfx950, with the reduction of
// the paper's Eq. 4 in its epilogue:
//   C[P x Q] = A^T * B,  A [Mc x P], B [Mc x Q] row-major BF16 (contraction over the rows),
// i.e. dW = X^T dY for a weight stored [K x N] (A = X, B = dY) and dW = dY^T X for one
// stored [N x K] (A = dY, B = X); fp32 accumulation, one round-to-nearest-even to BF16.
// P, Q multiples of 256, Mc of 64.
//
// Same 256 x 256 x 64 tile as the forward GEMM (gws_gemm256_core.h).  Both operands arrive with
// the output index contiguous, so both tiles stay as loaded and both MFMA operands are read
// with the transposing LDS load (ds_read_b64_tr_b16).
//
// Epilogue: the BF16 tile is staged in LDS and written 16 bytes per lane; a 16-byte group is
// 8 consecutive elements of a row of dW, exactly what one Philox call covers, and the 32x32
// blocks of the weight coincide with 32-row x 32-column pieces of the wavefront's 128 x 128
// tile.  On the way out each lane regenerates R for its groups (same seed, step and
// coordinates as the forward pass), accumulates dW .* 2R with v_dot2c_f32_bf16 over the 8
// groups it owns of a block, the 16 lanes of the block reduce, and one lane writes
//   dL/db_t = -ln2 * s32 * sum(dW .* R)
// computed on the rounded BF16 dW, as gws_sample_bwd would from the same bytes.
#include "gws_gemm256_core.h"
#include "gws_launch.h"

namespace gws {

// The way out of a wavefront's 128 x 128 part of dW (origin (p0, q0) in the weight): BF16 through the staging
// area, and with DBT the reduction of Eq. 4 over the groups as they pass.
template <bool DBT>
__device__ __forceinline__ void tn_write_half(const GemmArgs& g, const f32x4 (&a4)[4][8], int h, uint16_t* cs, uint32_t p0,
                                              uint32_t q0, uint32_t lane, float& part) {
  uint16_t* yw = g.y + (size_t)p0 * g.ldy + q0;
  if (!DBT) {
    epilogue_bf16_half(a4, h, cs, yw, g.ldy, lane, NoHook{});
    return;
  }
  const uint32_t nbc = g.N >> 5;
  // step `it` covers rows 4 it .. 4 it + 3 of the wavefront's part; lane = (row % 4, 16-byte column group)
  epilogue_bf16_half(a4, h, cs, yw, g.ldy, lane, [&](int it, uint32_t row, uint32_t c, const u32x4& v) {
    const Noise n = group_noise(g.cg0 + ((q0 + c) >> 3), g.row0 + p0 + row, g.step_lo, g.step_hi, g.seed_lo, g.seed_hi);
    part = dot_group_2r(v, n, part);
    if ((it & 7) == 7) {
      // rows 32 b .. 32 b + 31 are done: the block's 16 lanes (4 column groups x 4 row lanes) reduce
      float s = part;
      s += __uint_as_float(dpp_u32<0xB1>(__float_as_uint(s)));   // lane ^ 1
      s += __uint_as_float(dpp_u32<0x4E>(__float_as_uint(s)));   // lane ^ 2
      s += __uint_as_float((uint32_t)__builtin_amdgcn_ds_swizzle((int)__float_as_uint(s), 0x401F));  // lane ^ 16
      s += __shfl_xor(s, 32);
      if ((lane & 3) == 0 && (lane >> 4) == 0) {
        const size_t blk = (size_t)((p0 >> 5) + (it >> 3)) * nbc + (q0 >> 5) + ((lane & 15) >> 2);
        const float neg_ln2 = __uint_as_float(0xBF317218u);  // -ln 2
        g.dbt[blk] = (neg_ln2 * g.scale[blk]) * (s * 0.5f);
      }
      part = 0.0f;
    }
  });
}

template <bool DBT>
__device__ __forceinline__ void gemm256_tn_tile(const GemmArgs& g, uint32_t L) {
  using namespace g256;
  uint32_t tile_m, tile_n;
  tile_of(TileGrid{g.M / TM, g.N / TN, g.inv_band, g.inv_last}, L, tile_m, tile_n);
  const uint32_t m0 = tile_m * TM, n0 = tile_n * TN;
  gemm256_accumulate<true, true>(g.x, g.ldx, g.w, g.ldw, g.K / TK, m0, n0,
                                 [&](f32x4 (&acc)[8][8], uint16_t* cs, uint32_t wave, uint32_t lane) {
    const uint32_t p0 = m0 + 128 * (wave >> 1), q0 = n0 + 128 * (wave & 1);   // origin of the wavefront's part in dW
    float part = 0.0f;
    tn_write_half<DBT>(g, *reinterpret_cast<const f32x4 (*)[4][8]>(&acc[0]), 0, cs, p0, q0, lane, part);
    tn_write_half<DBT>(g, *reinterpret_cast<const f32x4 (*)[4][8]>(&acc[4]), 1, cs, p0, q0, lane, part);
  });
}

template <bool DBT>
__global__ __launch_bounds__(256, 1) void gemm256_tn_kernel(GWS_GEMM_PARAMS, const GemmSampling sampling) {
  const GemmArgs g = GWS_GEMM_GATHER(sampling);
  gemm256_tn_tile<DBT>(g, blockIdx.x);
}

// The same with tiles of 256 x 192: more of them, each three quarters of the work.  For weights whose 256 x 256 tiles leave
// compute units idle in a round that as many narrow ones fill: 2048 x 5632 over 8192 tokens has 176 of the one (188 us) and
// 240 of the other (163), on 256 compute units.
template <bool DBT>
__global__ __launch_bounds__(256, 1) void gemm256_tn_narrow_kernel(GWS_GEMM_PARAMS, const GemmSampling sampling) {
  using namespace g256;
  const GemmArgs g = GWS_GEMM_GATHER(sampling);
  uint32_t tile_m, tile_n;
  tile_of(TileGrid{g.M / TM, (g.N + kNarrow - 1) / kNarrow, g.inv_band, g.inv_last}, blockIdx.x, tile_m, tile_n);
  const uint32_t m0 = tile_m * TM, n0 = tile_n * kNarrow, cols = g.N - n0 < kNarrow ? g.N - n0 : kNarrow;
  gemm256_accumulate<true, true, true, 6>(g.x, g.ldx, g.w, g.ldw, g.K / TK, m0, n0,
                                          [&](f32x4 (&acc)[8][6], uint16_t* cs, uint32_t wave, uint32_t lane) {
    const uint32_t p0 = m0 + 128 * (wave >> 1), q0 = n0 + 96 * (wave & 1);
    uint16_t* yw = g.y + (size_t)p0 * g.ldy + q0;
    float part = 0.0f;
    auto hook = [&](uint32_t row, uint32_t c, const u32x4& v) {
      if (DBT) part = dot_group_2r(v, group_noise(g.cg0 + ((q0 + c) >> 3), g.row0 + p0 + row, g.step_lo, g.step_hi, g.seed_lo, g.seed_hi), part);
    };
    auto done = [&](int rb, int cb) {
      if (!DBT) return;
      part = block_sum_f32(part);
      part += __shfl_xor(part, 4);   // the block is the whole wavefront's here
      if (lane == 0) {
        const size_t blk = (size_t)((p0 >> 5) + rb) * (g.N >> 5) + (q0 >> 5) + cb;
        const float neg_ln2 = __uint_as_float(0xBF317218u);  // -ln 2
        g.dbt[blk] = (neg_ln2 * g.scale[blk]) * (part * 0.5f);
      }
      part = 0.0f;
    };
    const int wc = (int)cols - 96 * (int)(wave & 1);
    epilogue_narrow_half(*reinterpret_cast<const f32x4 (*)[4][6]>(&acc[0]), 0, cs, yw, g.ldy, lane, 128, wc, hook, done);
    epilogue_narrow_half(*reinterpret_cast<const f32x4 (*)[4][6]>(&acc[4]), 1, cs, yw, g.ldy, lane, 128, wc, hook, done);
  }, TM, cols, g.K);
}

// ---- the contraction split over several workgroups per tile ----
// A weight of few tiles (2048 x 2048: 64) leaves most compute units without work while each tile walks all tokens.
// Workgroup (tile L, part s) accumulates the tokens [kb, ke) of its part and leaves its accumulators in the
// workspace, as fp32 in register order (slab (s, L): 4 wavefronts x 64 accumulators x 64 lanes x 16 bytes, each
// store 1 KiB of consecutive memory); a second kernel adds a tile's parts in the order of s, rounds once to BF16 and
// goes out the same way as the one-kernel form (with the Eq. 4 reduction if asked for).  The result does not depend
// on timing: no atomics, no arrival order.
constexpr uint32_t kSlabFloats = 256 * 256;

__global__ __launch_bounds__(256, 1) void gemm256_tn_part_kernel(GWS_GEMM_PARAMS, const uint32_t parts, float* __restrict__ ws) {
  using namespace g256;
  const GemmArgs g = GWS_GEMM_GATHER({});
  const uint32_t tiles = (g.M / TM) * (g.N / TN);
  const uint32_t L = blockIdx.x % tiles, s = blockIdx.x / tiles;
  uint32_t tile_m, tile_n;
  tile_of(TileGrid{g.M / TM, g.N / TN, g.inv_band, g.inv_last}, L, tile_m, tile_n);
  const uint32_t nk = g.K / TK;
  const uint32_t kb = (uint32_t)((uint64_t)nk * s / parts), ke = (uint32_t)((uint64_t)nk * (s + 1) / parts);
  float* slab = ws + ((size_t)s * tiles + L) * kSlabFloats;
  gemm256_accumulate<true, true>(g.x + (size_t)kb * TK * g.ldx, g.ldx, g.w + (size_t)kb * TK * g.ldw, g.ldw, ke - kb,
                                 tile_m * TM, tile_n * TN, [&](f32x4 (&acc)[8][8], uint16_t*, uint32_t wave, uint32_t lane) {
    f32x4* out = reinterpret_cast<f32x4*>(slab) + (size_t)wave * 64 * 64 + lane;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j) out[(i * 8 + j) * 64] = acc[i][j];
  });
}

// One wavefront per 32 x 32 block of the weight: it takes the block's four registers of every part's slab (all of them
// requested before the first is added), so that a few dozen tiles still make thousands of wavefronts.  Bound by the slabs'
// bytes out of the last-level cache; with one wavefront per 64 x 128 (288 for 36 tiles) the loads' latency was: 768 x 3072,
// seven parts, 66 MB: 19.0 us, 12.3 like this.
constexpr uint32_t kMaxParts = 8;

template <bool DBT>
__global__ __launch_bounds__(256) void gemm256_tn_sum_kernel(GWS_GEMM_PARAMS, const uint32_t parts, const float* __restrict__ ws, const GemmSampling sampling) {
  using namespace g256;
  const GemmArgs g = GWS_GEMM_GATHER(sampling);
  constexpr uint32_t PB = 32 + 8;   // pitch of a block's staged rows (elements)
  __shared__ __attribute__((aligned(16))) uint16_t stage[4 * 32 * PB];
  const uint32_t tiles = (g.M / TM) * (g.N / TN), lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // workgroup: 32 rows (br) of one 128-column half (wn) of a tile; wavefront: 32 columns of it
  const uint32_t L = blockIdx.x >> 4, br = (blockIdx.x >> 1) & 7, wn = blockIdx.x & 1;
  uint32_t tile_m, tile_n;
  tile_of(TileGrid{g.M / TM, g.N / TN, g.inv_band, g.inv_last}, L, tile_m, tile_n);
  const uint32_t p0 = tile_m * TM + 32 * br, q0 = tile_n * TN + 128 * wn + 32 * wave;
  // register (i, j) of the accumulating wavefront 2 (br / 4) + wn: i = 2 (br % 4) + ii, j = 2 wave + jj
  const f32x4* in = reinterpret_cast<const f32x4*>(ws) + ((size_t)L * 4 + 2 * (br >> 2) + wn) * 4096 + (2 * (br & 3) * 8 + 2 * wave) * 64 + lane;
  const size_t step = (size_t)tiles * (kSlabFloats / 4);
  f32x4 v[kMaxParts][4];
#pragma unroll
  for (uint32_t s = 0; s < kMaxParts; ++s)
    if (s < parts) {
#pragma unroll
      for (int r = 0; r < 4; ++r) v[s][r] = in[s * step + ((r >> 1) * 8 + (r & 1)) * 64];
    }
  uint16_t* cs = stage + wave * 32 * PB;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    f32x4 a = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (uint32_t s = 0; s < kMaxParts; ++s)
      if (s < parts) {
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = __fadd_rn(a[e], v[s][r][e]);
      }
    *(u32x2*)(cs + (16 * (r >> 1) + (lane & 15)) * PB + 16 * (r & 1) + 4 * (lane >> 4)) = u32x2{pack_bf16_rne(a[0], a[1]), pack_bf16_rne(a[2], a[3])};
  }
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wavefront's LDS writes have landed
  __builtin_amdgcn_wave_barrier();
  // out: lane = (row % 16, 16-byte column group); dL/db_t as in tn_write_half
  const uint32_t row = lane >> 2, c = (lane & 3) * 8;
  float part = 0.0f;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const u32x4 o = *(const u32x4*)(cs + (row + 16 * t) * PB + c);
    *(u32x4*)(g.y + (size_t)(p0 + row + 16 * t) * g.ldy + q0 + c) = o;
    if (DBT) part = dot_group_2r(o, group_noise(g.cg0 + ((q0 + c) >> 3), g.row0 + p0 + row + 16 * t, g.step_lo, g.step_hi, g.seed_lo, g.seed_hi), part);
  }
  if (DBT) {
    part = block_sum_f32(part);
    part += __shfl_xor(part, 4);   // the block is the whole wavefront's here
    if (lane == 0) {
      const size_t blk = (size_t)(p0 >> 5) * (g.N >> 5) + (q0 >> 5);
      const float neg_ln2 = __uint_as_float(0xBF317218u);  // -ln 2
      g.dbt[blk] = (neg_ln2 * g.scale[blk]) * (part * 0.5f);
    }
  }
}

bool gemm256_tn_applicable(const GemmArgs& g) {
  return g.M > 0 && g.N > 0 && g.K > 0 && g.M % g256::TM == 0 && g.N % g256::TN == 0 && g.K % g256::TK == 0 &&
         g.ldx < g256::kMaxLd && g.ldw < g256::kMaxLd;
}

int launch_gemm256_tn(const GemmArgs& args, bool with_dbt, hipStream_t stream) {
  GemmArgs g = args;
  const uint64_t tiles = (uint64_t)(g.M / g256::TM) * (g.N / g256::TN);
  if (tiles >= 0x7FFFFFFFull) return GWS_ERR_SHAPE;
  set_tile_grid(g, g.M / g256::TM, g.N / g256::TN, patch_band(g.M / g256::TM, g.N / g256::TN, g256::TM, g256::TN));
  if (with_dbt) hipLaunchKernelGGL(gemm256_tn_kernel<true>, dim3((uint32_t)tiles), dim3(256), 0, stream, GWS_GEMM_PASS(g), (const GemmSampling&)g);
  else hipLaunchKernelGGL(gemm256_tn_kernel<false>, dim3((uint32_t)tiles), dim3(256), 0, stream, GWS_GEMM_PASS(g), (const GemmSampling&)g);
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

int launch_gemm256_tn_narrow(const GemmArgs& args, bool with_dbt, hipStream_t stream) {
  GemmArgs g = args;
  const uint32_t mt = g.M / g256::TM, nt = (g.N + g256::kNarrow - 1) / g256::kNarrow;
  if ((uint64_t)mt * nt >= 0x7FFFFFFFull) return GWS_ERR_SHAPE;
  set_tile_grid(g, mt, nt, patch_band(mt, nt, g256::TM, g256::kNarrow));
  if (with_dbt) hipLaunchKernelGGL(gemm256_tn_narrow_kernel<true>, dim3(mt * nt), dim3(256), 0, stream, GWS_GEMM_PASS(g), (const GemmSampling&)g);
  else hipLaunchKernelGGL(gemm256_tn_narrow_kernel<false>, dim3(mt * nt), dim3(256), 0, stream, GWS_GEMM_PASS(g), (const GemmSampling&)g);
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

size_t gemm256_tn_split_bytes(const GemmArgs& g, uint32_t parts) {
  return (size_t)parts * (g.M / g256::TM) * (g.N / g256::TN) * kSlabFloats * sizeof(float);
}

int launch_gemm256_tn_split(const GemmArgs& args, bool with_dbt, float* ws, uint32_t parts, hipStream_t stream) {
  GemmArgs g = args;
  const uint64_t tiles = (uint64_t)(g.M / g256::TM) * (g.N / g256::TN);
  if (parts < 2 || parts > kMaxParts || parts > g.K / g256::TK || tiles * 16 >= 0x7FFFFFFFull) return GWS_ERR_SHAPE;
  set_tile_grid(g, g.M / g256::TM, g.N / g256::TN, patch_band(g.M / g256::TM, g.N / g256::TN, g256::TM, g256::TN));
  hipLaunchKernelGGL(gemm256_tn_part_kernel, dim3((uint32_t)(tiles * parts)), dim3(256), 0, stream, GWS_GEMM_PASS(g), parts, ws);
  if (hipGetLastError() != hipSuccess) return GWS_ERR_LAUNCH;
  if (with_dbt) hipLaunchKernelGGL(gemm256_tn_sum_kernel<true>, dim3((uint32_t)(tiles * 16)), dim3(256), 0, stream, GWS_GEMM_PASS(g), parts, (const float*)ws, (const GemmSampling&)g);
  else hipLaunchKernelGGL(gemm256_tn_sum_kernel<false>, dim3((uint32_t)(tiles * 16)), dim3(256), 0, stream, GWS_GEMM_PASS(g), parts, (const float*)ws, (const GemmSampling&)g);
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

}  // namespace gws
