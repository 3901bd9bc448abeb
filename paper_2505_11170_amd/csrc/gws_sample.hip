// GaussWS elementwise kernels: forward (paper Eq. 3 + the cast of Sec. 3.3),
// backward (Eq. 4) and the packed-noise dump (Sec. 3.4), for gfx950.
//
// Work decomposition.  A wavefront owns a 32-row x 64-column tile (two 32x32
// blocks side by side); lane = 8 * r + c loads the 16-byte group of 8 BF16 at
// rows {r, r+8, r+16, r+24}, column group c.  Each load instruction of a wave
// therefore covers 8 rows x 128 contiguous bytes, the four waves of a workgroup
// sit side by side (512 contiguous bytes per row), and the per-block reductions
// (absmax, sum of g.*R) stay inside one wavefront: no LDS and no barrier, except
// where microscaling codes are gathered into rows of the workgroup (store_mx_rows).
// A workgroup covers one such 32 x 256 tile in the forward pass and up to four
// neighbouring column tiles in the lighter backward pass, where the per-wavefront
// set-up would otherwise show.  Four wavefronts a SIMD hide the latency of memory,
// and more are slower where it is memory that bounds a pass (GWS_FOUR_WAVES).
// One Philox4x32-10 call yields the 16 bits x 8 elements of one 16-byte group,
// so the noise lives only in registers (2 bytes per parameter of HBM traffic per
// operand, Sec. 3.5; the 0.5 byte per parameter temporary of the paper is gone).
//
// Many tensors per launch: the descriptors travel in the kernel-argument
// segment (no device table, no allocation); a workgroup finds its tensor by a
// scalar scan over the tile prefix.
#include "gws_launch.h"
#include "gws_sample_tile.h"

namespace gws {

// Which tensor, which block-row group and which column strip this workgroup owns, and that
// tensor's descriptor.  Pure scalar work: tile_begin[] ascends, unused entries are
// 0x7FFFFFFF, so (wg - tile_begin[i]) has its top bit clear exactly for the tensors that
// start at or before wg.
// A wavefront lives for one tile, so what it waits for before its first global load counts:
// the prefix table is fetched with four wide scalar loads issued together, the descriptor
// with three, i.e. two scalar-cache round trips in all.  (Left to itself the compiler
// fetches the table in three dependent steps and the descriptor field by field, as each is
// first used: six to nine round trips.)  The empty asm statements pin the loaded values in
// scalar registers at that point, which makes the loads of a batch issue back to back.
typedef uint32_t u32x16s __attribute__((ext_vector_type(16)));
typedef uint32_t u32x8s __attribute__((ext_vector_type(8)));
static_assert(kMaxTensorsPerLaunch == 56 && sizeof(TileDesc) == 96, "locate() is laid out for this table");

// local / tiles_x by the host's reciprocal: the estimate is at most one too small
__device__ __forceinline__ void tile_position(const TileDesc& d, uint32_t local, uint32_t& byg, uint32_t& bx) {
  uint32_t q = __umulhi(local, d.tiles_x_inv);
  uint32_t r = local - q * d.tiles_x;
  if (r >= d.tiles_x) {
    ++q;
    r -= d.tiles_x;
  }
  byg = q;
  bx = r;
}

// Workgroups are dealt round-robin to the 8 XCDs: sixteen neighbouring tiles go to one XCD, so that a cache line shared by
// two of them (rows that do not start on lines) meets in its L2.  Rows of 2000 bytes, w and w_hat of 75 M parameters: with
// ordinary stores 62 us forward, like this 59 (streaming stores 93 and 83); whole lines too: the 1B model's forward pass
// 667 -> 624 us (8 tiles 644, 32 tiles 630).
__device__ __forceinline__ uint32_t dealt_out(uint32_t wg) { return (wg & ~127u) + (wg & 7) * 16 + ((wg >> 3) & 15); }

// One tensor: its descriptor is the kernel's argument.
__device__ __forceinline__ TileDesc locate(const OneArgs& a, uint32_t& byg, uint32_t& bx) {
  tile_position(a.t, blockIdx.x < a.dealt ? dealt_out(blockIdx.x) : blockIdx.x, byg, bx);
  return a.t;
}

__device__ __forceinline__ TileDesc locate(const LaunchArgs& a, uint32_t& byg, uint32_t& bx) {
  const uint32_t wg = blockIdx.x < gridDim.x / 128 * 128 ? dealt_out(blockIdx.x) : blockIdx.x;
  const uint32_t* tb = a.tile_begin;
  u32x16s t0 = *(const u32x16s*)(tb), t1 = *(const u32x16s*)(tb + 16), t2 = *(const u32x16s*)(tb + 32);
  u32x8s t3 = *(const u32x8s*)(tb + 48);
  asm volatile("" : "+s"(t0), "+s"(t1), "+s"(t2), "+s"(t3));
  uint32_t after = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) after += ((wg - t0[i]) >> 31) + ((wg - t1[i]) >> 31) + ((wg - t2[i]) >> 31);
#pragma unroll
  for (int i = 0; i < 8; ++i) after += (wg - t3[i]) >> 31;
  const uint32_t ti = kMaxTensorsPerLaunch - 1 - after;

  const uint32_t* dp = (const uint32_t*)&a.t[ti];
  u32x16s d0 = *(const u32x16s*)(dp);
  u32x8s d1 = *(const u32x8s*)(dp + 16);
  asm volatile("" : "+s"(d0), "+s"(d1));
  uint32_t w[24];
#pragma unroll
  for (int i = 0; i < 16; ++i) w[i] = d0[i];
#pragma unroll
  for (int i = 0; i < 8; ++i) w[16 + i] = d1[i];
  TileDesc d;
  __builtin_memcpy(&d, w, sizeof d);

  tile_position(d, wg - d.first_wg, byg, bx);
  return d;
}

// The tiles of one workgroup: `tiles_per_wg_x` neighbouring column tiles by `tiles_per_wg`
// block rows, column tiles first, so that the workgroups running at any moment cover a
// contiguous stretch of the tensor.  Each wavefront handles its 64-column strip of every
// tile; `body(by, col_base, tile)` is called for strips that exist.  The first tile is
// loaded ahead of the loop, so the common one-tile case stays straight-line code.
template <int STREAM, class ARGS, class F>
__device__ __forceinline__ void walk_tiles(const ARGS& a, const TileDesc& d, uint32_t byg, uint32_t bxg,
                                           F&& body) {
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const GWS_GLOBAL uint16_t* __restrict__ src = global_ptr<uint16_t>(d.p0);
  const uint32_t nbr = (d.rows + 31) >> 5, ntx = (d.cols + kTileCols - 1) / kTileCols;
  const uint32_t by0 = byg * a.tiles_per_wg, by_end = min(by0 + a.tiles_per_wg, nbr);
  const uint32_t bx0 = bxg * a.tiles_per_wg_x, bx_end = min(bx0 + a.tiles_per_wg_x, ntx);
  uint32_t by = by0, bx = bx0;
  uint32_t col_base = bx * kTileCols + wave * 64;
  Tile t = load_tile<STREAM>(src, d, by, col_base, lane);
  for (;;) {
    if (col_base < d.cols) body(by, col_base, t);
    if (++bx >= bx_end) {
      bx = bx0;
      if (++by >= by_end) break;
    }
    col_base = bx * kTileCols + wave * 64;
    t = load_tile<STREAM>(src, d, by, col_base, lane);
  }
}

// Exactly four wavefronts a SIMD, whatever the registers would allow.  64 KiB of loads in flight on a compute unit cover the
// latency of memory, and more tiles under way spread the accesses over more DRAM pages: forward and backward of the 1B model
// with 8, 7, 6, 5, 4 and 2 wavefronts a SIMD 927, 923, 891, 891, 876 and 1004 us, of the 124M model 87, 87, 85, 85, 83, 95.
// The registers that this leaves (128) let the compiler interleave a tile's groups: MX-FP6 of 352 M parameters 195 -> 182 us.
#define GWS_FOUR_WAVES __attribute__((amdgpu_waves_per_eu(4, 4)))
// Weights of any shape: up to eight (EIGHT) while what the pass reads and writes fits in the last-level cache, wherever it only reads
// and where much of the tiles lies outside the weights (run_batched).  Backward pass of the comparison bases on whole tiles: up to
// eight too, as they have more left to do when the tile has come (uniform, 34.7 M parameters 11.3 us, 12.0 with four; Box-Muller, 33.5 M
// 16.5, 16.9).
#define GWS_WAVES(eight) __attribute__((amdgpu_waves_per_eu(4, (eight) ? 8 : 4)))

// MX: write element codes and E8M0 block scales instead of the BF16 container.
// STREAM: see load16.
// BASIS: the method's bit-built noise, or one of the two comparison bases.
template <int FMT, bool MX, int STREAM, int BASIS, bool EIGHT, class ARGS>
__global__ __launch_bounds__(kThreads) GWS_WAVES(EIGHT) void sample_fwd_kernel(const ARGS a) {
  uint32_t byg, bxg;
  const TileDesc d = locate(a, byg, bxg);
  const uint32_t lane = threadIdx.x & 63;
  walk_tiles<STREAM>(a, d, byg, bxg, [&](uint32_t by, uint32_t col_base, Tile& t) {
    TileNoise<BASIS> n[1];
    if (t.full) {   // the block's parameter with the tile: behind the noise, its latency would be paid in full
      const float bt = *at_byte(global_ptr<float>(d.p2) + ((size_t)by * ((d.cols + 31) >> 5) + (col_base >> 5)), lane & 4);
      draw_noise(a.step_lo, a.step_hi, d, tile_rows(d, by, lane, a.step_lo), col_base, lane, n);
      fwd_tile<FMT, true, STREAM, MX, BASIS>(d, t, n[0], by, col_base, lane, bt);
    } else {
      const float bt = lane_bt(d, by, col_base, lane);
      draw_noise_edge(a.step_lo, a.step_hi, d, by, col_base, lane, n[0]);
      fwd_tile<FMT, false, STREAM, MX, BASIS>(d, t, n[0], by, col_base, lane, bt);
    }
  });
}

template <bool FULL, bool COPY, int STREAM, int BASIS>
__device__ __forceinline__ void bwd_tile(const TileDesc& d, const Tile& t, const TileNoise<BASIS>& noise, uint32_t by,
                                         uint32_t col_base, uint32_t lane) {
  const uint32_t row_base = by * 32;
  const uint32_t gc = lane & 7, r0 = lane >> 3;
  const uint32_t col = col_base + gc * 8;
  GWS_GLOBAL uint16_t* __restrict__ dw = global_ptr<uint16_t>(d.p1);
  GWS_GLOBAL float* __restrict__ dbt = global_ptr<float>(d.p2);
  const GWS_GLOBAL float* __restrict__ scale = global_ptr<float>(d.p3);
  const uint32_t off = lane_offset(d.ld, lane);   // full tiles

  // the block's lane that writes the gradient fetches what it needs first
  const uint32_t nbc = (d.cols + 31) >> 5;
  const uint32_t bcol = (col_base >> 5) + (gc >> 2);
  const bool writer = (FULL || bcol < nbc) && (gc & 3) == 0 && r0 == 0;
  const size_t blk = (size_t)by * nbc + bcol;
  float s32 = 0.0f, bi = 0.0f;
  if (writer) {
    s32 = scale[blk];
    if (d.p4 != nullptr) bi = global_ptr<float>(d.p4)[blk];
  }

  // sum_{b_l}(g .* R), accumulated as sum(g .* 2R) / 2: every product is exact
  // in fp32, the order of the additions is fixed (per lane group by group, two
  // elements per step, then the lane tree), so the result is reproducible.
  float acc = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (!FULL && t.nv[i] == 0) continue;
    const uint32_t row = row_base + r0 + 8 * i;
    if (COPY) {  // dL/dw = dL/dw_hat, bit for bit
      if (FULL) store16<STREAM>(at_byte(dw + ((size_t)(row_base + 8 * i) * d.ld + col_base), off), t.v[i]);
      else if (t.nv[i] == 8) store16<STREAM>(dw + (size_t)row * d.ld + col, t.v[i]);
      else store_partial(dw + (size_t)row * d.ld + col, t.v[i], t.nv[i]);
    }
    const u32x4 gv = (FULL || t.nv[i] == 8) ? t.v[i] : mask_group(t.v[i], t.nv[i]);
    if constexpr (BASIS == kBasisBits) acc = dot_group_2r(gv, noise.x[i], acc);
    else acc = dot_group_basis<BASIS>(gv, noise.x[i], acc);
  }
  acc = block_sum_f32(acc) * (BASIS == kBasisBits ? 0.5f : 1.0f);

  if (writer) {
    const float neg_ln2 = __uint_as_float(0xBF317218u);  // -ln 2
    float grad = (neg_ln2 * s32) * acc;                  // dL/db_t, Eq. 4
    if (d.p4 != nullptr) {
      // dL'/db_i, Eq. 11 and Eq. 12: b_t is recomputed exactly as the forward pass formed it,
      // the subgradient of |b_t - b_target| at 0 is taken as 0
      const float btv = __fadd_rn(d.b_target, __fmul_rn(bi, d.b_delta));
      const float sgn = btv > d.b_target ? 1.0f : (btv < d.b_target ? -1.0f : 0.0f);
      grad = d.b_delta * (grad + d.lambda_m * sgn);
    }
    dbt[blk] = grad;
  }
}

template <int STREAM, int BASIS, bool EIGHT, class ARGS>
__global__ __launch_bounds__(kThreads) GWS_WAVES(EIGHT) void sample_bwd_kernel(const ARGS a) {
  uint32_t byg, bxg;
  const TileDesc d = locate(a, byg, bxg);
  const uint32_t lane = threadIdx.x & 63;
  const bool copy = d.p1 != nullptr;  // NULL: the pass-through is an alias
  walk_tiles<STREAM>(a, d, byg, bxg, [&](uint32_t by, uint32_t col_base, Tile& t) {
    TileNoise<BASIS> n[1];
    if (t.full) {
      draw_noise(a.step_lo, a.step_hi, d, tile_rows(d, by, lane, a.step_lo), col_base, lane, n);
      if (copy) bwd_tile<true, true, STREAM, BASIS>(d, t, n[0], by, col_base, lane);
      else bwd_tile<true, false, STREAM, BASIS>(d, t, n[0], by, col_base, lane);
    } else {
      draw_noise_edge(a.step_lo, a.step_hi, d, by, col_base, lane, n[0]);
      if (copy) bwd_tile<false, true, STREAM, BASIS>(d, t, n[0], by, col_base, lane);
      else bwd_tile<false, false, STREAM, BASIS>(d, t, n[0], by, col_base, lane);
    }
  });
}

// The forward pass on a workgroup's 32 x 256 tile with MX output: the codes are staged in LDS and go to memory by rows, 16 bytes
// a thread, so that an instruction covers whole rows of the tile (192 bytes of FP6, 256 of FP8) and not each wavefront's quarter
// of many.  FP6 from the wavefronts' own 48 bytes a row made 3.7 times as many write requests as lines: 352 M parameters 183 us,
// 159 like this, 6.3 TB/s with no idle cycle of the vector ALU (FP8 173, 170); 809 M in rows of 4096 and 11008 elements 407 us,
// 351 (FP8 392, 369).  Rows of FP6 codes are 2-byte aligned, rows of FP8 codes 8-byte aligned.
template <int FMT, int STREAM>
__device__ __forceinline__ void store_mx_rows(const TileDesc& d, Tile& t, const TileNoise<kBasisBits>& n, uint32_t by, uint32_t bx, float bt) {
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, gc = lane & 7, r0 = lane >> 3;
  constexpr uint32_t kRow = FMT == 1 ? kTileCols : kTileCols / 8 * 6, kPitch = kRow + 16, kChunks = kRow / 16;
  __shared__ __attribute__((aligned(16))) char staged[32 * kPitch];
  const BlockScale b = tile_scale<FMT, true, true, true>(d, t, by, bx * kTileCols + wave * 64, lane, bt);
  tile_sum<true>(t, b, n);
  if constexpr (FMT == 1) {
    const bool hw = __builtin_amdgcn_ballot_w64(!b.hw_safe) == 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t pk[4] = {t.v[i][0], t.v[i][1], t.v[i][2], t.v[i][3]};
      const MxCodes c = mx_fp8_codes(pk, b, hw);
      *(uint64_t*)(staged + (r0 + 8 * i) * kPitch + wave * 64 + gc * 8) = ((uint64_t)c.hi << 32) | c.lo;
    }
  } else {
    const u32x6 c = tile_codes_fp6<true>(t, b);
    const uint32_t cw[6] = {c[0], c[1], c[2], c[3], c[4], c[5]};
    const Codes24 q = codes_fp6_quad(lane, cw);
    uint64_t* to = (uint64_t*)(staged + (r0 + 8 * (lane & 3)) * kPitch + wave * 48 + (lane & 4) * 6);
#pragma unroll
    for (int k = 0; k < 3; ++k) to[k] = ((uint64_t)q.w[2 * k + 1] << 32) | q.w[2 * k];
  }
  __syncthreads();
  typedef uint32_t u32x4a2 __attribute__((ext_vector_type(4), aligned(2)));
  GWS_GLOBAL uint8_t* codes = global_ptr<uint8_t>(d.p1) + ((size_t)(by * 32) * d.ldc + bx * kRow);
#pragma unroll
  for (uint32_t c = threadIdx.x; c < 32 * kChunks; c += kThreads) {
    const uint32_t row = c / kChunks, k = 16 * (c % kChunks);
    const u32x4 v = *(const u32x4*)(staged + row * kPitch + k);
    GWS_GLOBAL u32x4a2* to = (GWS_GLOBAL u32x4a2*)(codes + ((size_t)row * d.ldc + k));
    // FP6 calls read past the caches only where they are large; what they write then goes the same way (352 M parameters
    // 177 us with ordinary stores, 159)
    if (STREAM == kStreamAll || (FMT == 2 && STREAM == kStreamReads)) __builtin_nontemporal_store(v, to);
    else *to = v;
  }
}

// The forward pass for tensors of whole tiles only (rows a multiple of 32, columns of 256), one tile a workgroup, straight
// through: the loads are issued, the noise is drawn while they are in flight (it depends on none of them) and kept as a
// register a group, the rest follows.
template <int FMT, bool MX, int STREAM, int BASIS, class ARGS>
__global__ __launch_bounds__(kThreads) GWS_FOUR_WAVES void sample_fwd_full_kernel(const ARGS a) {
  uint32_t byg, bxg;
  const TileDesc d = locate(a, byg, bxg);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const GWS_GLOBAL uint16_t* __restrict__ src = global_ptr<uint16_t>(d.p0);
  const uint32_t col_base = bxg * kTileCols + wave * 64;
  Tile t = load_full_tile<STREAM>(src, d, byg, col_base, lane);
  const float bt = *at_byte(global_ptr<float>(d.p2) + ((size_t)byg * (d.cols >> 5) + (col_base >> 5)), lane & 4);
  TileNoise<BASIS> n[1];
  draw_noise(a.step_lo, a.step_hi, d, tile_rows(d, byg, lane, a.step_lo), col_base, lane, n);
  __builtin_amdgcn_sched_barrier(0);   // the noise is drawn while the loads are in flight
  if constexpr (MX) store_mx_rows<FMT, STREAM>(d, t, n[0], byg, bxg, bt);
  else fwd_tile<FMT, true, STREAM, MX, BASIS>(d, t, n[0], byg, col_base, lane, bt);
}

// The backward pass for the shape the method meets in a model: every tensor of the launch has whole tiles only
// (rows a multiple of 32, columns of 256) and dL/dw is an alias (nothing to copy).  Straight-line per tile, and
// the vector ALU work is cut where it can be: the Philox rounds that depend on the row alone are computed once
// per wavefront and reused for every column tile it walks, those that depend on the column group alone once per
// tile.  The next tile's loads are issued after the current tile's arithmetic and complete under the next tile's
// Philox rounds.
template <int STREAM, int BASIS, class ARGS>
__global__ __launch_bounds__(kThreads) GWS_WAVES(BASIS != kBasisBits) void sample_bwd_full_kernel(const ARGS a) {
  uint32_t byg, bxg;
  const TileDesc d = locate(a, byg, bxg);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t gc = lane & 7, r0 = lane >> 3;
  const GWS_GLOBAL uint16_t* __restrict__ src = global_ptr<uint16_t>(d.p0);
  const uint32_t ntx = d.cols / kTileCols, nbc = d.cols >> 5;
  const uint32_t by = byg;                                                  // one block row per workgroup
  const uint32_t bx0 = bxg * a.tiles_per_wg_x, bx_end = min(bx0 + a.tiles_per_wg_x, ntx);
  const bool writer = (gc & 3) == 0 && r0 == 0;
  const PhiloxRows rp = tile_rows(d, by, lane, a.step_lo);

  Tile t;
  float s32 = 0.0f, bi = 0.0f;
  auto block0 = [&](uint32_t bx) { return (size_t)by * nbc + ((bx * kTileCols + wave * 64) >> 5); };   // of the tile's left block
  auto load = [&](uint32_t bx) {
    t = load_full_tile<STREAM>(src, d, by, bx * kTileCols + wave * 64, lane);
    if (writer) {   // the block's writer lane fetches what it needs with the tile
      s32 = *at_byte(global_ptr<float>(d.p3) + block0(bx), gc);   // gc is 0 or 4 here
      if (d.p4 != nullptr) bi = *at_byte(global_ptr<float>(d.p4) + block0(bx), gc);
    }
  };
  load(bx0);
  for (uint32_t bx = bx0; bx < bx_end; ++bx) {
    TileNoise<BASIS> n[1];
    draw_noise(a.step_lo, a.step_hi, d, rp, bx * kTileCols + wave * 64, lane, n);
    // sum_{b_l}(g .* R) as sum(g .* 2R) / 2: exact products, fixed order (see bwd_tile)
    float acc = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (BASIS == kBasisBits) acc = dot_group_2r(t.v[i], n[0].x[i], acc);
      else acc = dot_group_basis<BASIS>(t.v[i], n[0].x[i], acc);
    }
    acc = block_sum_f32(acc) * (BASIS == kBasisBits ? 0.5f : 1.0f);
    if (writer) {
      const float neg_ln2 = __uint_as_float(0xBF317218u);   // -ln 2
      float grad = (neg_ln2 * s32) * acc;                   // dL/db_t, Eq. 4
      if (d.p4 != nullptr) {                                // dL'/db_i, Eq. 11 and Eq. 12 (as in bwd_tile)
        const float btv = __fadd_rn(d.b_target, __fmul_rn(bi, d.b_delta));
        const float sgn = btv > d.b_target ? 1.0f : (btv < d.b_target ? -1.0f : 0.0f);
        grad = d.b_delta * (grad + d.lambda_m * sgn);
      }
      *at_byte(global_ptr<float>(d.p2) + block0(bx), gc) = grad;
    }
    if (bx + 1 < bx_end) load(bx + 1);
  }
}

// The forward kernel's memory traffic without its arithmetic: every tile is loaded and
// stored back unchanged, same workgroup shape, same loads and stores.  What this kernel
// reaches is the ceiling the memory system sets for the access pattern.
__global__ __launch_bounds__(kThreads) GWS_FOUR_WAVES void copy_tiles_kernel(const LaunchArgs a) {
  uint32_t byg, bxg;
  const TileDesc d = locate(a, byg, bxg);
  const uint32_t lane = threadIdx.x & 63;
  GWS_GLOBAL uint16_t* __restrict__ dst = global_ptr<uint16_t>(d.p1);
  walk_tiles<kStreamAll>(a, d, byg, bxg, [&](uint32_t by, uint32_t col_base, Tile& t) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (t.nv[i] == 0) continue;
      GWS_GLOBAL uint16_t* p = dst + (size_t)(by * 32 + (lane >> 3) + 8 * i) * d.ld + col_base + (lane & 7) * 8;
      if (t.nv[i] == 8) store16(p, t.v[i]);
      else store_partial(p, t.v[i], t.nv[i]);
    }
  });
}

// Step one of the forward pass alone: a = max|w| per 32x32 block (exact), written as fp32.
// Reads every element once and writes 4 bytes per block, the traffic profile of the backward
// pass: its rate is the ceiling the memory system sets for a read-only pass of this shape.
__global__ __launch_bounds__(kThreads) GWS_FOUR_WAVES void block_absmax_kernel(const LaunchArgs a) {
  uint32_t byg, bxg;
  const TileDesc d = locate(a, byg, bxg);
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t gc = lane & 7, r0 = lane >> 3;
  GWS_GLOBAL float* __restrict__ out = global_ptr<float>(d.p3);
  const uint32_t nbc = (d.cols + 31) >> 5;
  walk_tiles<kStreamAll>(a, d, byg, bxg, [&](uint32_t by, uint32_t col_base, Tile& t) {
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) m = absmax_pk(t.nv[i] < 8 ? mask_group(t.v[i], t.nv[i]) : t.v[i], m);
    m = max(m & 0xFFFFu, m >> 16);
    const uint32_t a16 = block_max_u32(m);
    const uint32_t bcol = (col_base >> 5) + (gc >> 2);
    if (bcol < nbc && (gc & 3) == 0 && r0 == 0) out[(size_t)by * nbc + bcol] = __uint_as_float(a16 << 16);
  });
}

__global__ __launch_bounds__(256) void noise_packed_kernel(uint32_t* __restrict__ out, uint32_t rows,
                                                           uint32_t ngrp, uint32_t row0, uint32_t cg0,
                                                           uint32_t seed_lo, uint32_t seed_hi,
                                                           uint32_t step_lo, uint32_t step_hi) {
  const uint64_t idx = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (uint64_t)rows * ngrp) return;
  const uint32_t row = (uint32_t)(idx / ngrp), cgl = (uint32_t)(idx % ngrp);
  out[idx] = packed_codes(group_noise(cg0 + cgl, row0 + row, step_lo, step_hi, seed_lo, seed_hi));
}

// R of every element under a comparison basis, as BF16 values [rows x 8 ngrp]: one thread per group of 8.
template <int BASIS>
__global__ __launch_bounds__(256) void noise_basis_kernel(u32x4* __restrict__ out, uint32_t rows, uint32_t ngrp,
                                                          uint32_t row0, uint32_t cg0, uint32_t seed_lo, uint32_t seed_hi,
                                                          uint32_t step_lo, uint32_t step_hi) {
  const uint64_t idx = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (uint64_t)rows * ngrp) return;
  const uint32_t row = (uint32_t)(idx / ngrp), cgl = (uint32_t)(idx % ngrp);
  out[idx] = basis_group_bf16<BASIS>(philox4x32_10(cg0 + cgl, row0 + row, step_lo, step_hi, seed_lo, seed_hi));
}

// Both ways to R of the Box-Muller basis over the words first .. first + n - 1 (gws_box_muller_check of gws_bench.h).
__global__ __launch_bounds__(256) void box_muller_check_kernel(uint64_t first, uint64_t n, unsigned long long* __restrict__ out) {
  uint32_t differ = 0, exact = 0, worst = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256) {
    const uint32_t word = (uint32_t)(first + i);
    float r[2], e[2];
    uint32_t near = 0;
    box_muller_pair_fast(word, r[0], r[1], near);
    box_muller_pair(word, e[0], e[1]);
    if ((near & kBoxMullerNear) == 0) {
      differ += __float_as_uint(r[0]) != __float_as_uint(e[0]) || __float_as_uint(r[1]) != __float_as_uint(e[1]) ? 1 : 0;
      continue;
    }
    ++exact;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const float m = __builtin_fabsf(r[k]), f = m - __builtin_floorf(m);   // 0.5: on the threshold
      if (f != 0.0f && __builtin_floorf(m) + (f >= 0.5f ? 1.0f : 0.0f) != __builtin_fabsf(e[k]))
        worst = max(worst, (uint32_t)(__builtin_fabsf(f - 0.5f) * 0x1p24f));
    }
  }
  if (differ) atomicAdd(&out[0], (unsigned long long)differ);
  if (exact) atomicAdd(&out[1], (unsigned long long)exact);
  if (worst) atomicMax(&out[2], (unsigned long long)worst);
}

// ---------------------------------------------------------------------------
// Host-side launchers
// ---------------------------------------------------------------------------
template <int FMT, bool MX, int STREAM, int BASIS, class ARGS>
static void launch_fwd(const ARGS& a, uint32_t n_wg, int variant, hipStream_t stream) {
  if (variant == 1) hipLaunchKernelGGL((sample_fwd_full_kernel<FMT, MX, STREAM, BASIS, ARGS>), dim3(n_wg), dim3(kThreads), 0, stream, a);
  else if (variant == 2) hipLaunchKernelGGL((sample_fwd_kernel<FMT, MX, STREAM, BASIS, true, ARGS>), dim3(n_wg), dim3(kThreads), 0, stream, a);
  else hipLaunchKernelGGL((sample_fwd_kernel<FMT, MX, STREAM, BASIS, false, ARGS>), dim3(n_wg), dim3(kThreads), 0, stream, a);
}

// One weight (the call inside every sampled linear) takes the small argument block: five kilobytes of arguments and two dependent reads of
// them are a fifth of a small kernel's time, 768 x 768 4.5 -> 3.6 us, and show in larger ones: backward of 2048 x 8192 7.4 -> 6.6, Box-Muller
// 16.5 -> 15.7 and 10.8 -> 10.2, FP6 codes of 2048 x 5632 8.8 -> 7.7.
template <int FMT, bool MX, int BASIS>
static void launch_fwd_stream(const LaunchArgs& a, uint32_t n_wg, int mode, int variant, hipStream_t stream) {
  if (mode == kKeep && a.n == 1) launch_fwd<FMT, MX, kKeep, BASIS>(one_of(a, n_wg), n_wg, variant, stream);
  else if (mode == kStreamReads && a.n == 1) launch_fwd<FMT, MX, kStreamReads, BASIS>(one_of(a, n_wg), n_wg, variant, stream);
  else if (mode == kKeep) launch_fwd<FMT, MX, kKeep, BASIS>(a, n_wg, variant, stream);
  else if (mode == kStreamReads) launch_fwd<FMT, MX, kStreamReads, BASIS>(a, n_wg, variant, stream);
  else launch_fwd<FMT, MX, kStreamAll, BASIS>(a, n_wg, variant, stream);
}

template <int BASIS>
static int launch_fwd_fmt(const LaunchArgs& a, uint32_t n_wg, int fmt, int mode, int variant, hipStream_t stream) {
  switch (fmt) {
    case GWS_FMT_BF16: launch_fwd_stream<0, false, BASIS>(a, n_wg, mode, variant, stream); return GWS_OK;
    case GWS_FMT_FP8_E4M3: launch_fwd_stream<1, false, BASIS>(a, n_wg, mode, variant, stream); return GWS_OK;
    case GWS_FMT_FP6_E3M2: launch_fwd_stream<2, false, BASIS>(a, n_wg, mode, variant, stream); return GWS_OK;
    default: return GWS_ERR_FORMAT;
  }
}

int launch_sample_fwd(const LaunchArgs& a, uint32_t n_wg, int fmt, bool mx, int basis, int mode, int variant, hipStream_t stream) {
  if (n_wg == 0) return GWS_OK;
  int rc = GWS_OK;
  if (mx && fmt == GWS_FMT_FP8_E4M3 && basis == kBasisBits) launch_fwd_stream<1, true, kBasisBits>(a, n_wg, mode, variant, stream);
  else if (mx && fmt == GWS_FMT_FP6_E3M2 && basis == kBasisBits) launch_fwd_stream<2, true, kBasisBits>(a, n_wg, mode, variant, stream);
  else if (mx) rc = GWS_ERR_FORMAT;
  else if (basis == kBasisBits) rc = launch_fwd_fmt<kBasisBits>(a, n_wg, fmt, mode, variant, stream);
  else if (basis == kBasisUniform) rc = launch_fwd_fmt<kBasisUniform>(a, n_wg, fmt, mode, variant, stream);
  else if (basis == kBasisBoxMuller) rc = launch_fwd_fmt<kBasisBoxMuller>(a, n_wg, fmt, mode, variant, stream);
  else rc = GWS_ERR_FORMAT;
  if (rc != GWS_OK) return rc;
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

template <int STREAM, int BASIS, class ARGS>
static void launch_bwd(const ARGS& a, uint32_t n_wg, int variant, hipStream_t stream) {
  if (variant == 1) hipLaunchKernelGGL((sample_bwd_full_kernel<STREAM, BASIS, ARGS>), dim3(n_wg), dim3(kThreads), 0, stream, a);
  else if (variant == 2) hipLaunchKernelGGL((sample_bwd_kernel<STREAM, BASIS, true, ARGS>), dim3(n_wg), dim3(kThreads), 0, stream, a);
  else hipLaunchKernelGGL((sample_bwd_kernel<STREAM, BASIS, false, ARGS>), dim3(n_wg), dim3(kThreads), 0, stream, a);
}

template <int BASIS>
static void launch_bwd_stream(const LaunchArgs& a, uint32_t n_wg, int mode, int variant, hipStream_t stream) {
  if (mode == kKeep && a.n == 1) launch_bwd<kKeep, BASIS>(one_of(a, n_wg), n_wg, variant, stream);
  else if (mode == kStreamReads && a.n == 1) launch_bwd<kStreamReads, BASIS>(one_of(a, n_wg), n_wg, variant, stream);
  else if (mode == kKeep) launch_bwd<kKeep, BASIS>(a, n_wg, variant, stream);
  else if (mode == kStreamReads) launch_bwd<kStreamReads, BASIS>(a, n_wg, variant, stream);
  else launch_bwd<kStreamAll, BASIS>(a, n_wg, variant, stream);
}

int launch_sample_bwd(const LaunchArgs& a, uint32_t n_wg, int basis, int mode, int variant, hipStream_t stream) {
  if (n_wg == 0) return GWS_OK;
  switch (basis) {
    case kBasisBits: launch_bwd_stream<kBasisBits>(a, n_wg, mode, variant, stream); break;
    case kBasisUniform: launch_bwd_stream<kBasisUniform>(a, n_wg, mode, variant, stream); break;
    case kBasisBoxMuller: launch_bwd_stream<kBasisBoxMuller>(a, n_wg, mode, variant, stream); break;
    default: return GWS_ERR_FORMAT;
  }
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

int launch_noise_basis(void* out, uint32_t rows, uint32_t ngrp, uint32_t row0, uint32_t cg0, uint64_t seed, uint64_t step,
                       int basis, hipStream_t stream) {
  const uint64_t total = (uint64_t)rows * ngrp;
  if (total == 0) return GWS_OK;
  const uint32_t grid = (uint32_t)((total + 255) / 256);
  const uint32_t slo = (uint32_t)seed, shi = (uint32_t)(seed >> 32), tlo = (uint32_t)step, thi = (uint32_t)(step >> 32);
  if (basis == kBasisUniform)
    hipLaunchKernelGGL(noise_basis_kernel<kBasisUniform>, dim3(grid), dim3(256), 0, stream, (u32x4*)out, rows, ngrp, row0, cg0, slo, shi, tlo, thi);
  else if (basis == kBasisBoxMuller)
    hipLaunchKernelGGL(noise_basis_kernel<kBasisBoxMuller>, dim3(grid), dim3(256), 0, stream, (u32x4*)out, rows, ngrp, row0, cg0, slo, shi, tlo, thi);
  else return GWS_ERR_FORMAT;
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

int launch_box_muller_check(uint64_t first, uint64_t n, uint64_t* out, hipStream_t stream) {
  if (n == 0) return GWS_OK;
  hipLaunchKernelGGL(box_muller_check_kernel, dim3((uint32_t)(n < 4096 * 256 ? (n + 255) / 256 : 4096)), dim3(256), 0, stream, first, n,
                     (unsigned long long*)out);
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

int launch_copy_tiles(const LaunchArgs& a, uint32_t n_wg, hipStream_t stream) {
  if (n_wg == 0) return GWS_OK;
  hipLaunchKernelGGL(copy_tiles_kernel, dim3(n_wg), dim3(kThreads), 0, stream, a);
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

int launch_block_absmax(const LaunchArgs& a, uint32_t n_wg, hipStream_t stream) {
  if (n_wg == 0) return GWS_OK;
  hipLaunchKernelGGL(block_absmax_kernel, dim3(n_wg), dim3(kThreads), 0, stream, a);
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

int launch_noise_packed(uint32_t* out, uint32_t rows, uint32_t ngrp, uint32_t row0, uint32_t cg0,
                        uint64_t seed, uint64_t step, hipStream_t stream) {
  const uint64_t total = (uint64_t)rows * ngrp;
  if (total == 0) return GWS_OK;
  const uint32_t grid = (uint32_t)((total + 255) / 256);
  hipLaunchKernelGGL(noise_packed_kernel, dim3(grid), dim3(256), 0, stream, out, rows, ngrp, row0, cg0,
                     (uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)step, (uint32_t)(step >> 32));
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

}  // namespace gws
