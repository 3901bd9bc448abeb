// BF16 GEMM for few rows of X on gfx950: Y[M x N] = X[M x K] * W (W stored [K x N] or [N x K]), plain or with the
// GaussWS sampling of W on its way in (paper Eq. 3 + cast).
//
// What bounds it: the weight's bytes.  A tile of the output that walks all of K alone waits for memory K / 64 times, and
// a few rows of X make a few tiles.  So a workgroup owns a small piece of Y (16 MT rows x 16 NT columns) and its
// wavefronts split K: wavefront w takes a contiguous range of 64-deep units of K, keeps several units of loads on their way
// into its own ring of LDS stages, and meets the others at a barrier only for the partial sums, which are added in LDS in
// the order of the wavefronts (one defined order; the plain and the sampling kernel split K alike, so their Y is the same
// bits).  How many wavefronts split K goes by M, N, K and the number of compute units (stream_plan), so a row of Y is not
// the same bits for every number of rows beside it.
#include "gws_gemm_stream_core.h"

namespace gws {

// A wavefront's share of a tile's columns of the weight, fetched into the XCD's L2 and dropped: one load instruction touches 64 pieces
// of lines, every part-th unit of 64 k.  A compute unit gets about 60 B/ns from beyond its L2, a line every 2 ns whether 64 bytes of it are
// wanted or 128, so few tiles on few compute units wait for the weight while the others idle; what an idle one has fetched comes at 150.
// A wavefront has one load on its way: the empty statement uses its register, so the next one waits for it.  How many workgroups a tile
// fetch (stream_plan) is fitted to that.
template <int BN, bool W_NK>
__device__ __forceinline__ void warm_l2(const GemmArgs& g, uint32_t n0, uint32_t u0, uint32_t u1, uint32_t part, uint32_t parts) {
  const uint32_t lane = threadIdx.x & 63;
  constexpr uint32_t UNITS = W_NK ? 64 / BN : 1;   // of an instruction
  for (uint32_t u = u0 + part * UNITS; u < u1; u += parts * UNITS) {
    const uint32_t k = stream::umin(64 * (u + (W_NK ? lane / BN : 0)), g.K - 64);
    const uint32_t v = *(const uint32_t*)(W_NK ? g.w + (size_t)stream::umin(n0 + lane % BN, g.N - 1) * g.ldw + k : g.w + (size_t)(k + lane) * g.ldw + n0);
    asm volatile("" ::"v"(v));
  }
}

// A wavefront keeps D units of 64 k on their way into its own ring of LDS stages (global_load_lds_dwordx4, 8 rows x 128
// contiguous bytes per instruction).  Loaded straight into the MFMA's register layout instead (16 rows x 64 bytes: a
// quarter-wavefront touches 16 cache lines for 16 bytes each) a compute unit takes 39 B/ns whatever is in flight; in this
// form 130-180 B/ns (L2-resident operands, one workgroup per compute unit).  Layouts as in gws_gemm256_core.h: rows of 128
// bytes with chunk c of row r in slot c ^ ((r / 2) % 8); a [K x N] weight as 64 k-rows of 32 NT bytes, read with the
// transposing LDS load, chunk c of row k in slot c ^ swizzle(k).
// WARM: the grid has more workgroups a tile (blockIdx.y > 0) that only warm_l2; they share nothing with the others.
// BM x BN is the workgroup's tile: 16 MT x 16 NT, or eight rows, eight columns where one MFMA tile has that many of use (the others
// are computed on repeated ones and not stored).
template <int MT, int NT, int P, int D, bool W_NK, int BM = 16 * MT, int BN = 16 * NT, bool WARM = false>
__global__ __launch_bounds__(64 * P) void gemm_stream_kernel(GWS_GEMM_PARAMS) {
  using namespace stream;
  const GemmArgs g = GWS_GEMM_GATHER({});
  static_assert((BM == 16 * MT || (BM == 8 && MT == 1)) && (BN == 16 * NT || (BN == 8 && NT == 1 && W_NK)), "whole MFMA tiles or half a one");
  constexpr int XS = BM * 64, WS = BN * 64, STG = XS + WS;          // elements of a stage
  constexpr int QX = BM / 8, QW = BN / 8, LOADS = QX + QW;          // load instructions of a unit
  static_assert(LOADS * (D - 1) <= 63, "the wait for a unit counts the loads behind it");
  static_assert(W_NK || NT == 2 || NT == 4 || NT == 8, "swizzle of the [K x N] stage");
  constexpr int MC = MT > 4 ? 4 : MT;                               // row tiles of a pass of the reduction
  constexpr int kRing = P * D * STG * 2, kRed = red_bytes(MC, NT, P);
  __shared__ __attribute__((aligned(1024))) char lds[kRing > kRed ? kRing : kRed];
  const uint32_t lane = threadIdx.x & 63, li = lane & 15, grp = lane >> 4;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint16_t* ring = (uint16_t*)lds + wave * (D * STG);
  const TileGrid t = {(g.M + BM - 1) / BM, (g.N + BN - 1) / BN, g.inv_band, g.inv_last};
  uint32_t m0, n0;
  if (t.joined()) tile_of_joined(t, blockIdx.x, m0, n0);   // StreamPlan::parts
  else tile_of_groups(t, !W_NK && NT == 2, blockIdx.x, m0, n0);
  m0 *= BM;
  n0 *= BN;
  uint32_t u0, u1;
  unit_range(g.K, wave, P, u0, u1);
  if (WARM && (blockIdx.y > 0 || blockIdx.x >= t.mt * t.nt)) {   // uniform; a row of the grid is whole rounds of the XCDs
    if (blockIdx.x < t.mt * t.nt) warm_l2<BN, W_NK>(g, n0, u0, u1, blockIdx.y - 1, gridDim.y - 1);
    return;
  }

  // lane offsets in bytes; rows and columns past the edge are read from the last ones and not stored
  uint32_t xo[QX], wo[W_NK ? QW : 1];
#pragma unroll
  for (int q = 0; q < QX; ++q)
    xo[q] = (umin(8u * q + (lane >> 3), g.M - 1 - m0) * g.ldx + ((lane & 7) ^ (4 * (q & 1) + (lane >> 4))) * 8) * 2;
  if (W_NK) {
#pragma unroll
    for (int q = 0; q < QW; ++q)
      wo[q] = (umin(8u * q + (lane >> 3), g.N - 1 - n0) * g.ldw + ((lane & 7) ^ (4 * (q & 1) + (lane >> 4))) * 8) * 2;
  }
  // [K x N]: an instruction covers RPI k-rows of 2 NT chunks
  constexpr uint32_t CPR = 2 * NT, RPI = 64 / CPR;
  const uint32_t wk = lane / CPR, ws = lane % CPR;
  const GWS_GLOBAL char* xb = (const GWS_GLOBAL char*)(g.x + (size_t)m0 * g.ldx);
  const GWS_GLOBAL char* wb = (const GWS_GLOBAL char*)(W_NK ? g.w + (size_t)n0 * g.ldw : g.w + n0);
  const uint32_t last_chunk = (g.N - n0) / 8 - 1;
  constexpr int NV = W_NK ? 1 : 16 / RPI;   // the swizzle depends on k % 16
  uint32_t wv[NV];
  if (!W_NK) {
#pragma unroll
    for (int v = 0; v < NV; ++v) wv[v] = (wk * g.ldw + umin(ws ^ oc_swizzle<W_NK ? 2 : NT>(wk + RPI * v), last_chunk) * 8) * 2;
  }
  auto load = [&](uint32_t u, uint32_t slot) {
    uint16_t* st = ring + slot * STG;
    const uint32_t k0 = umin(64 * u, g.K - 64);   // the half unit at the end of K is fetched as the second half of a whole one
#pragma unroll
    for (int q = 0; q < QW; ++q) {
      if (W_NK) direct(wb + (size_t)k0 * 2, wo[q], st + XS + q * 512);
      else direct(wb + (size_t)(k0 + RPI * q) * g.ldw * 2, wv[q % NV], st + XS + q * 512);
    }
#pragma unroll
    for (int q = 0; q < QX; ++q) direct(xb + (size_t)k0 * 2, xo[q], st + q * 512);
  };

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const uint32_t n = u1 - u0;
#pragma unroll
  for (int d = 0; d < D; ++d)
    if ((uint32_t)d < n) load(u0 + d, d);
  uint32_t slot = 0;
  const uint32_t lx = BM == 8 ? li & 7 : li, lw = BN == 8 ? li & 7 : li;
  for (uint32_t i = 0; i < n; ++i) {
    if (i + D <= n) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS * (D - 1)) : "memory");   // the unit has landed
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const uint16_t* xs = ring + slot * STG;
    const uint16_t* wsg = xs + XS;
    Frag8 fx[2][MT], fw[2][NT];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int r = 0; r < MT; ++r) fx[h][r].u = *(const u32x4*)(xs + (16 * r + lx) * 64 + (((4 * h + grp) ^ ((lx >> 1) & 7)) * 8));
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        if (W_NK) {
          fw[h][j].u = *(const u32x4*)(wsg + (16 * j + lw) * 64 + (((4 * h + grp) ^ ((lw >> 1) & 7)) * 8));
        } else {
          fw[h][j] = read_oc<W_NK ? 2 : NT>(wsg, h, j, li, grp);
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read: the stage can be filled again
    __builtin_amdgcn_sched_barrier(0);
    if (i + D < n) load(u0 + i + D, slot);
    slot = slot + 1 == D ? 0 : slot + 1;
    const bool half = 64 * (u0 + i) + 64 > g.K;   // only the second half of the stage belongs to this unit
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h == 0 && half) continue;
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < MT; ++r) acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[h][j].v, fx[h][r].v, acc[r][j], 0, 0, 0);
    }
  }
  reduce_store<MT, NT, P, MC, BM, BN>(acc, lds, g, m0, n0);
}

// Eq. 3 + cast on the weight's blocks on their way into the MFMA, B (1 or 2) at a time: the wavefront's 32 columns of Y and the
// 32 B k of step s.  Group i of block h of a lane: storage row lane / 4 + 16 i, columns 8 (lane % 4) .. + 7 of the block.  Two
// blocks together are two independent chains (maximum over the wavefront, scale, sums, cast), which one or two wavefronts a
// SIMD need; one at a time takes half the registers.  The noise depends on none of the loads and comes first, its Philox
// calls round by round with what they share drawn once (a column group of a [K x N] weight, two rows of an [N x K] one).
constexpr int LP = 40;   // row pitch of a staged block (elements)
template <int FMT, bool W_NK, int B>
struct Blocks {
  uint32_t n0, nbc;          // the wavefront's columns of Y; blocks per storage row
  uint32_t q, r;             // lane % 4, lane / 4
  PhiloxCols cols;           // [K x N]
  PhiloxRows rows;           // [N x K], two of them
  const GWS_GLOBAL char* base;
  uint32_t off;

  __device__ __forceinline__ Blocks(const GemmArgs& g, uint32_t n) : n0(n), nbc((W_NK ? g.K : g.N) >> 5) {
    const uint32_t lane = threadIdx.x & 63;
    q = lane & 3;
    r = lane >> 2;
    if (W_NK) {
      const uint32_t row[4] = {g.row0 + n0 + r, g.row0 + n0 + r + 16, 0, 0};
      rows = philox_rows(row, g.step_lo, g.seed_lo);
    } else {
      cols = philox_cols(g.cg0 + (n0 >> 3) + q, g.step_lo, g.step_hi, g.seed_lo, g.seed_hi);
    }
    base = (const GWS_GLOBAL char*)(W_NK ? g.w + (size_t)n0 * g.ldw : g.w + n0);
    off = (r * g.ldw + 8 * q) * 2;
  }
  // block b along K: its first storage row and column, its number
  __device__ __forceinline__ uint32_t row_of(uint32_t b) const { return W_NK ? n0 : 32 * b; }
  __device__ __forceinline__ uint32_t col_of(uint32_t b) const { return W_NK ? 32 * b : n0; }
  __device__ __forceinline__ size_t number(uint32_t b) const { return W_NK ? (size_t)(n0 >> 5) * nbc + b : (size_t)b * nbc + (n0 >> 5); }

  struct Raw {
    u32x4 w[B][2];
    float bt[B];
  };
  // blocks B s ..; of half a step at the end of K the first one twice
  __device__ __forceinline__ void load(const GemmArgs& g, uint32_t s, Raw& x) const {
#pragma unroll
    for (int h = 0; h < B; ++h) {
      const uint32_t b = stream::umin(B * s + h, (g.K >> 5) - 1);
      const GWS_GLOBAL char* p = base + (W_NK ? (size_t)b * 64 : (size_t)b * 64 * g.ldw);
#pragma unroll
      for (int i = 0; i < 2; ++i) x.w[h][i] = *(const GWS_GLOBAL u32x4*)(p + (size_t)(16 * i) * g.ldw * 2 + off);
      x.bt[h] = global_ptr<float>(g.bt)[number(b)];
    }
  }

  // The sampled blocks to `blk`, B x 32 x LP elements of LDS; writer: this wavefront stores w_hat and scale (if wanted).
  __device__ __forceinline__ void stage(const GemmArgs& g, uint32_t step, const Raw& x, bool writer, uint16_t* blk) const {
    const uint32_t lane = threadIdx.x & 63;
    Noise n[B][2];   // [block][group]
    if (W_NK) {
      PhiloxCols pc[B];
#pragma unroll
      for (int h = 0; h < B; ++h) pc[h] = philox_cols(g.cg0 + 4 * (B * step + h) + q, g.step_lo, g.step_hi, g.seed_lo, g.seed_hi);
      Philox4 p[B][2];
      philox_tiles(pc, rows, g.seed_lo, g.seed_hi, p);
#pragma unroll
      for (int k = 0; k < 2 * B; ++k) n[k >> 1][k & 1] = noise_codes(p[k >> 1][k & 1]);
    } else {
      const uint32_t k0 = g.row0 + 32 * B * step + r, row[4] = {k0, k0 + 16, k0 + 32, k0 + 48};
      const PhiloxCols pc[1] = {cols};
      Philox4 p[1][2 * B];
      philox_tiles(pc, philox_rows(row, g.step_lo, g.seed_lo), g.seed_lo, g.seed_hi, p);
#pragma unroll
      for (int k = 0; k < 2 * B; ++k) n[k >> 1][k & 1] = noise_codes(p[0][k]);
    }
#pragma unroll
    for (int k = 0; k < 2 * B; ++k) asm volatile("" : "+v"(n[k >> 1][k & 1].c));   // here, while the weight is on its way
    BlockScale s[B];
#pragma unroll
    for (int h = 0; h < B; ++h) {
      uint32_t m = absmax_pk(x.w[h][1], absmax_pk(x.w[h][0], 0));
      m = max(m & 0xFFFFu, m >> 16);
      m = block_max_u32(m);
      const uint32_t a16 = max(m, (uint32_t)__shfl_xor((int)m, 4));   // the block is the whole wavefront's here
      s[h] = block_scale(a16, x.bt[h]);
      if (FMT == 1) cast_constants<8, -6>(a16, s[h]);
      if (FMT == 2) cast_constants<4, -2>(a16, s[h]);
    }
    u32x4 v[B][2];
    if (FMT == 1 && s[0].hw_safe && s[B - 1].hw_safe) {   // uniform: the wavefront holds the blocks
#pragma unroll
      for (int k = 0; k < 2 * B; ++k) v[k >> 1][k & 1] = sample_group<FMT>(x.w[k >> 1][k & 1], n[k >> 1][k & 1], s[k >> 1], true);
    } else {
#pragma unroll
      for (int k = 0; k < 2 * B; ++k) v[k >> 1][k & 1] = sample_group<FMT>(x.w[k >> 1][k & 1], n[k >> 1][k & 1], s[k >> 1], false);
    }
    if (writer && g.w_hat != nullptr) {
#pragma unroll
      for (int h = 0; h < B; ++h) {
        const uint32_t b = B * step + h;
        if (b >= g.K >> 5) break;
        if (lane == 0) g.scale[number(b)] = s[h].s32;
#pragma unroll
        for (int i = 0; i < 2; ++i) *(u32x4*)(g.w_hat + (size_t)(row_of(b) + r + 16 * i) * g.ldw + col_of(b) + 8 * q) = v[h][i];
      }
    }
#pragma unroll
    for (int k = 0; k < 2 * B; ++k) *(u32x4*)(blk + ((k >> 1) * 32 + r + 16 * (k & 1)) * LP + 8 * q) = v[k >> 1][k & 1];
  }
  // column half j of a staged block
  static __device__ __forceinline__ Frag8 fragment(const uint16_t* p, int j) {
    const uint32_t lane = threadIdx.x & 63, li = lane & 15, grp = lane >> 4;
    Frag8 f;
    if (W_NK) {
      f.u = *(const u32x4*)(p + (16 * j + li) * LP + 8 * grp);
    } else {   // transposing read: lanes 4 t .. 4 t + 3 of 16 point at 16 outputs of row k0 + t
#pragma unroll
      for (int t = 0; t < 2; ++t)
        f.h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GWS_LDS i16x4*)(p + (8 * grp + 4 * t + (li >> 2)) * LP + 16 * j + 4 * (li & 3)));
    }
    return f;
  }
  // the sampled blocks as fragments f[block][column half] (16 outputs, 32 k)
  __device__ __forceinline__ void sample(const GemmArgs& g, uint32_t step, const Raw& x, bool writer, uint16_t* blk, Frag8 (&f)[B][2]) const {
    stage(g, step, x, writer, blk);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the wavefront's own writes have landed
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int h = 0; h < B; ++h)
#pragma unroll
      for (int j = 0; j < 2; ++j) f[h][j] = fragment(blk + h * 32 * LP, j);
  }
};

// The sampling form: a wavefront keeps a step's blocks on their way into registers while it samples those of the step before,
// turns them through its own 2.5 KiB of LDS a block and multiplies.  Bound by the sampling, which every 16 MT rows of X repeat: with
// 16 rows, two wavefronts a SIMD, the vector ALU issues in 66 % of a workgroup's cycles, and the rest is the chain from a block's
// maximum to its MFMA.  Two blocks a step where a compute unit has only one such workgroup's wavefronts (16 rows: 16 x 2048
// -> 5632 11.6 -> 11.4 us, 16 x 768 -> 3072 8.0 -> 7.6), one where it may have several (300 x 2048 -> 5632 41 us, two blocks 46).
// TAIL: K ends with half a step of two blocks.  W: wavefronts a SIMD that the registers have to leave room for.
template <int MT, int P, int FMT, bool W_NK, int B, bool TAIL, int W>
__global__ __launch_bounds__(64 * P) __attribute__((amdgpu_waves_per_eu(W)))
void gemm_stream_sample_kernel(GWS_GEMM_PARAMS, const GemmSampling sampling) {
  using namespace stream;
  const GemmArgs g = GWS_GEMM_GATHER(sampling);
  static_assert(B == 2 || !TAIL, "half a step is one of two blocks");
  constexpr int kRed = red_bytes(MT, 2, P), kBlk = P * B * 32 * LP * 2;
  __shared__ __attribute__((aligned(16))) char lds[kRed > kBlk ? kRed : kBlk];
  const uint32_t lane = threadIdx.x & 63, li = lane & 15, grp = lane >> 4;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint16_t* blk = (uint16_t*)lds + wave * B * 32 * LP;
  uint32_t m0, n0, s0, s1;
  tile_origin(g, 16 * MT, 32, !W_NK, m0, n0);
  unit_range(g.K, wave, P, s0, s1);
  if (B == 1) {
    s0 *= 2;
    s1 = umin(2 * s1, g.K >> 5);
  }

  uint32_t xo[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) xo[i] = (umin(16u * i + li, g.M - 1 - m0) * g.ldx + 8 * grp) * 2;
  const GWS_GLOBAL char* xb = (const GWS_GLOBAL char*)(g.x + (size_t)m0 * g.ldx);
  const Blocks<FMT, W_NK, B> w(g, n0);

  f32x4 acc[MT][2];
#pragma unroll
  for (int i = 0; i < MT; ++i) acc[i][0] = acc[i][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  typename Blocks<FMT, W_NK, B>::Raw nxt;
  if (s0 < s1) w.load(g, s0, nxt);
  const uint32_t whole = TAIL ? umin(s1, g.K >> 6) : s1;
  for (uint32_t s = s0; s < whole; ++s) {
    const typename Blocks<FMT, W_NK, B>::Raw cur = nxt;
    w.load(g, umin(s + 1, s1 - 1), nxt);
    Frag8 x[B][MT], f[B][2];
#pragma unroll
    for (int h = 0; h < B; ++h)
#pragma unroll
      for (int i = 0; i < MT; ++i) x[h][i].u = *(const GWS_GLOBAL u32x4*)(xb + (size_t)umin(B * s + h, (g.K >> 5) - 1) * 64 + xo[i]);
    w.sample(g, s, cur, m0 == 0, blk, f);
#pragma unroll
    for (int h = 0; h < B; ++h)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[h][j].v, x[h][i].v, acc[i][j], 0, 0, 0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the reads are done before the blocks are overwritten
    __builtin_amdgcn_wave_barrier();
  }
  if (TAIL && whole < s1) {
    // half a step at the end of K: one block, as the wavefront beside this one on the SIMD has work of its own
    const Blocks<FMT, W_NK, 1> last(g, n0);
    const typename Blocks<FMT, W_NK, 1>::Raw one = {{{nxt.w[0][0], nxt.w[0][1]}}, {nxt.bt[0]}};
    Frag8 x[MT], f[1][2];
#pragma unroll
    for (int i = 0; i < MT; ++i) x[i].u = *(const GWS_GLOBAL u32x4*)(xb + (size_t)(2 * whole) * 64 + xo[i]);
    last.sample(g, 2 * whole, one, m0 == 0, blk, f);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[0][j].v, x[i].v, acc[i][j], 0, 0, 0);
  }
  reduce_store<MT, 2, P, MT>(acc, lds, g, m0, n0);
}

// Many rows of X, the weight sampled on its way in, K from end to end (the order of the middle and large tiles' sums, so Y is
// their Y): a workgroup owns 256 rows x 256 columns, a wavefront 32 of the columns.  X comes through LDS in units of 64 k, a
// ring of stages that the wavefronts share, one barrier a unit; the weight's blocks go from a wavefront's registers through its
// own LDS as above, two a unit.  Bound by the sampling, which every tile of rows repeats (128 rows a tile: twice of it): the
// vector ALU issues in 64 % of the cycles, the matrix cores work in 29 %.  Two of the eight wavefronts share a SIMD, and the
// barrier keeps them abreast: the later four multiply a unit after the next barrier (hence a third stage), before they sample,
// so that one's MFMAs run under the other's sampling.  FP8, [K x N] and [N x K], us, tiles of 128 x 128 by four wavefronts and
// this: 8192 x 2048 -> 5632 462, 424 -> 290, 304 (FP6 548, 508 -> 359, 368; BF16 385, 373 -> 288, 285); 8192 x 2048 -> 2048 160,
// 161 -> 99, 106.
template <int FMT, bool W_NK>
__global__ __launch_bounds__(512, 2) void gemm_rows_sample_kernel(GWS_GEMM_PARAMS, const GemmSampling sampling) {
  using namespace stream;
  const GemmArgs g = GWS_GEMM_GATHER(sampling);
  constexpr int MT = 16, NW = 8, BM = 16 * MT, D = 3, XS = BM * 64, LX = BM / (8 * NW);   // LX: load instructions of a wavefront and unit
  __shared__ __attribute__((aligned(1024))) uint16_t ring[D * XS];
  __shared__ __attribute__((aligned(16))) uint16_t blocks[NW * 2 * 32 * LP];
  const uint32_t lane = threadIdx.x & 63, li = lane & 15, grp = lane >> 4;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint16_t* blk = blocks + wave * 2 * 32 * LP;
  uint32_t m0, n0;
  tile_origin(g, BM, 32 * NW, false, m0, n0);
  n0 += 32 * wave;
  const bool live = n0 < g.N;   // N is a multiple of 32: a wavefront's columns exist or do not
  const uint32_t nu = (g.K + 63) >> 6;

  uint32_t xo[LX];
#pragma unroll
  for (int i = 0; i < LX; ++i) {   // rows 8 LX wave + 8 i + lane / 8
    const uint32_t row = 8 * LX * wave + 8 * i + (lane >> 3);
    xo[i] = (umin(row, g.M - 1 - m0) * g.ldx + ((lane & 7) ^ ((row >> 1) & 7)) * 8) * 2;
  }
  const GWS_GLOBAL char* xb = (const GWS_GLOBAL char*)(g.x + (size_t)m0 * g.ldx);
  auto load_x = [&](uint32_t u, uint32_t slot) {
    const uint32_t k0 = umin(64 * u, g.K - 64);   // the half unit at the end of K is fetched as the second half of a whole one
#pragma unroll
    for (int i = 0; i < LX; ++i) direct(xb + (size_t)k0 * 2, xo[i], ring + slot * XS + (wave * LX + i) * 512);
  };
  const Blocks<FMT, W_NK, 2> w(g, live ? n0 : 0);   // a wavefront past the edge reads the first columns and multiplies nothing
  typename Blocks<FMT, W_NK, 2>::Raw nxt;

  f32x4 acc[MT][2];
#pragma unroll
  for (int i = 0; i < MT; ++i) acc[i][0] = acc[i][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  w.load(g, 0, nxt);
  load_x(0, 0);
  uint32_t slot = 0, next = 1, last = D - 1;   // of this unit, the next one and the one before
  Frag8 f[2][2];
  auto multiply = [&](uint32_t u, uint32_t at) __attribute__((always_inline)) {
    // MFMAs and LDS reads are 8 bytes each: four bytes off, every eighth one lies on two lines of the instruction cache (BF16 8192 x 2048 ->
    // 5632 [K x N] 293 -> 281 us; where the loop falls otherwise, [N x K] 296 -> 281)
    asm volatile(".p2align 3");
    const uint16_t* xs = ring + at * XS;
    const bool half = 64 * u + 64 > g.K;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h == 1 && half) break;   // one block, whose k are the second half of the stage
      const int hx = half ? 1 : h;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        Frag8 x;
        x.u = *(const u32x4*)(xs + (16 * i + li) * 64 + (((4 * hx + grp) ^ ((li >> 1) & 7)) * 8));
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[h][j].v, x.v, acc[i][j], 0, 0, 0);
      }
    }
  };
  const bool late = wave >= 4;   // uniform
  // A shift of the code that measured faster, not an alignment of the loop: its header comes about 140 instructions later, 44 or 48 bytes
  // past a line of the instruction cache.  FP8 [K x N] 8192 x 2048 -> 5632 with and without 287, 294 us, FP6 358, 360; [N x K] 305, 303 and 369, 367.
  asm volatile(".p2align 6");
  for (uint32_t u = 0; u < nu; ++u) {
    // this unit, requested a unit's sampling ago, has landed, and every wavefront is past its reads of the stage filled next
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (u + 1 < nu) load_x(u + 1, next);
    if (live) {
      if (late && u > 0) multiply(u - 1, last);
      const typename Blocks<FMT, W_NK, 2>::Raw cur = nxt;
      w.load(g, umin(u + 1, nu - 1), nxt);
      w.sample(g, u, cur, m0 == 0, blk, f);
      if (!late) multiply(u, slot);
    }
    last = slot;
    slot = next;
    next = next + 1 == D ? 0 : next + 1;
  }
  if (!live) return;
  if (late) multiply(nu - 1, last);
#pragma unroll
  for (int i = 0; i < MT; ++i) {   // row 16 i + lane % 16, columns 16 j + 4 (lane / 16) .. + 3
    const uint32_t row = m0 + 16 * i + li;
    if (row < g.M) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
        *(u32x2*)(g.y + (size_t)row * g.ldy + n0 + 16 * j + 4 * grp) =
            u32x2{pack_bf16_rne(acc[i][j][0], acc[i][j][1]), pack_bf16_rne(acc[i][j][2], acc[i][j][3])};
    }
  }
}

// The same with tiles of 128 x 128, for fewer of them.  Of the eight wavefronts two share the columns: each samples one block of a
// unit and multiplies half of the rows by both blocks, a unit later, past the barrier that makes both visible.  Of the two
// wavefronts of a SIMD one multiplies first, one samples first.  Four wavefronts that sampled and multiplied for themselves waited
// for their own serial chains.  us, four wavefronts and this, one workgroup on a compute unit: 4000 x 2304 -> 800 68 -> 53 (FP6 84 ->
// 66, BF16 63 -> 47; [N x K] 69 -> 54), 4000 x 3072 -> 1024 91 -> 72, 8192 x 512 -> 512 19.5 -> 16.8; two: 4096 x 1024 -> 2048 47 -> 44,
// 2862 x 1184 -> 1920 53 -> 50; several rounds of two: 8192 x 2048 -> 2048 160 -> 147.
// HALF: K ends with half a unit, of which one wavefront samples its block and the other nothing (4000 x 160 -> 1664 in FP6 17.1 ->
// 16.3).  The first unit's X comes with the weight: 1678 x 64 -> 3104 in FP6 10.9 -> 10.2.
template <int FMT, bool W_NK, bool HALF>
__global__ __launch_bounds__(512, 2) void gemm_rows_pair_sample_kernel(GWS_GEMM_PARAMS, const GemmSampling sampling) {
  using namespace stream;
  const GemmArgs g = GWS_GEMM_GATHER(sampling);
  constexpr int MT = 4, BM = 128, XS = BM * 64, LX = 2;   // row tiles of a wavefront; elements of a stage; load instructions of a wavefront
  __shared__ __attribute__((aligned(1024))) uint16_t ring[2 * XS];
  __shared__ __attribute__((aligned(16))) uint16_t blocks[2][4][2][32 * LP];   // [unit][32 columns][block]
  const uint32_t lane = threadIdx.x & 63, li = lane & 15, grp = lane >> 4;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), rm = wave >> 2, cn = wave & 3;
  uint32_t m0, n0;
  tile_origin(g, BM, 128, false, m0, n0);
  n0 += 32 * cn;
  const bool live = n0 < g.N;   // N is a multiple of 32: a wavefront's columns exist or do not
  const uint32_t nu = (g.K + 63) >> 6;

  uint32_t xo[LX];
#pragma unroll
  for (int i = 0; i < LX; ++i) {   // rows 16 wave + 8 i + lane / 8
    const uint32_t row = 16 * wave + 8 * i + (lane >> 3);
    xo[i] = (umin(row, g.M - 1 - m0) * g.ldx + ((lane & 7) ^ ((row >> 1) & 7)) * 8) * 2;
  }
  const GWS_GLOBAL char* xb = (const GWS_GLOBAL char*)(g.x + (size_t)m0 * g.ldx);
  const Blocks<FMT, W_NK, 1> w(g, live ? n0 : 0);   // a wavefront past the edge reads the first columns and multiplies nothing
  typename Blocks<FMT, W_NK, 1>::Raw nxt;
  f32x4 acc[MT][2];
#pragma unroll
  for (int i = 0; i < MT; ++i) acc[i][0] = acc[i][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  auto multiply = [&](uint32_t u) __attribute__((always_inline)) {
    const uint16_t* xs = ring + (u & 1) * XS;
    const bool half = HALF && 64 * u + 64 > g.K;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h == 1 && half) break;   // one block, whose k are the second half of the stage
      const int hx = half ? 1 : h;
      Frag8 f[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) f[j] = Blocks<FMT, W_NK, 1>::fragment(blocks[u & 1][cn][h], j);
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        Frag8 x;
        x.u = *(const u32x4*)(xs + (64 * rm + 16 * i + li) * 64 + (((4 * hx + grp) ^ ((li >> 1) & 7)) * 8));
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[j].v, x.v, acc[i][j], 0, 0, 0);
      }
    }
  };
  w.load(g, rm, nxt);
  for (uint32_t u = 0; u < nu; ++u) {
    // the unit before has landed and is sampled, and every wavefront is past its reads of the stages filled next (the first unit
    // waits for nothing: X comes with the weight)
    if (u > 0) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const uint32_t k0 = umin(64 * u, g.K - 64);   // the half unit at the end of K is fetched as the second half of a whole one
#pragma unroll
    for (int i = 0; i < LX; ++i) direct(xb + (size_t)k0 * 2, xo[i], ring + (u & 1) * XS + (wave * LX + i) * 512);
    if (!live) continue;
    if (rm == 1 && u > 0) multiply(u - 1);
    const typename Blocks<FMT, W_NK, 1>::Raw cur = nxt;
    w.load(g, 2 * umin(u + 1, nu - 1) + rm, nxt);
    if (!HALF || 2 * u + rm < g.K >> 5) w.stage(g, 2 * u + rm, cur, m0 == 0, blocks[u & 1][cn][rm]);   // of half a unit one block
    if (rm == 0 && u > 0) multiply(u - 1);
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  if (!live) return;
  multiply(nu - 1);
#pragma unroll
  for (int i = 0; i < MT; ++i) {   // row 16 i + lane % 16, columns 16 j + 4 (lane / 16) .. + 3
    const uint32_t row = m0 + 64 * rm + 16 * i + li;
    if (row < g.M) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
        *(u32x2*)(g.y + (size_t)row * g.ldy + n0 + 16 * j + 4 * grp) =
            u32x2{pack_bf16_rne(acc[i][j][0], acc[i][j][1]), pack_bf16_rne(acc[i][j][2], acc[i][j][3])};
    }
  }
}

// ---------------------------------------------------------------------------
// Which tile and how many parts of K.  The estimate (us) is a launch plus, per round of workgroups (one per compute unit:
// the rings fill its LDS), a fixed part (the last round's ends before the next one's loads arrive) and the bytes of the
// tile's operands at the rate a compute unit takes them.  Measured on MI355X (weights taken in turn from four copies), us by
// tile (rows x columns, parts of K), and the 128-tile kernel that these products took before:
//   M x K -> N            16x16,8 16x32,8 32x32,8 32x64,4 64x64,4 128x64,4  before
//   4 x 5632 -> 2048 NK     6.0     7.2                                      103
//   16 x 2048 -> 5632 KN    -       7.6                                       60
//   64 x 5632 -> 2048 NK                    9.8    13.8    18.3              105
//   64 x 2048 -> 5632 KN                   12.0     8.9    11.1               60
//   256 x 2048 -> 5632 KN                  29.4    20.0    18.2               40
//   1000 x 2304 -> 768 KN                  21.6    15.1    11.0    16.1       66
//   1000 x 5632 -> 2048 NK                                 36.6    29.9      107
// (in the order of the tiles then; as they are dealt now the first 5.6, 1000 x 2304 -> 768 in 64x64 10.6).
// ---------------------------------------------------------------------------
StreamPlan stream_plan(uint64_t M, uint64_t N, uint64_t K, bool w_is_nk) {
  StreamPlan best = {0, 0, 0, 0, 0, 0, 0, 1e30};
  if (K < 64) return best;
  const int cus = compute_units() > 0 ? compute_units() : 256;
  // bytes per ns: eight wavefronts keep twice the loads in flight that four do
  static const struct { int mt, nt, p; double rate; } tiles[] = {{1, 1, 8, 130.0}, {1, 2, 8, 130.0}, {2, 2, 8, 130.0},
                                                                 {2, 4, 4, 100.0}, {4, 4, 4, 100.0}, {8, 4, 4, 72.0}};
  for (const auto& t : tiles) {
    if (t.mt == 1 && M > 16) continue;
    if (t.nt == 1 && !w_is_nk) continue;   // 32 bytes of a row of a [K x N] weight: a quarter of a cache line
    const uint64_t wgs = ((M + 16 * t.mt - 1) / (16 * t.mt)) * ((N + 16 * t.nt - 1) / (16 * t.nt));
    const double rounds = (double)((wgs + cus - 1) / cus);
    const double us = 1.8 + 2.7 * rounds + rounds * (double)K * 2 * 16 * (t.mt + t.nt) / t.rate * 1e-3;
    if (wgs < 0x7FFFFFFFull && us < best.us) best = {t.mt, t.nt, t.p, 16 * t.mt, 16 * t.nt, 0, 0, us};
  }
  if (best.p == 0) return best;
  // Of one MFMA tile's rows and columns those that are wanted.  Up to eight rows of X are one load instruction a unit instead of
  // two (4 x 5632 -> 2048 6.09 -> 5.64 us).  Eight columns of an [N x K] weight make twice the workgroups: faster where they still
  // fit one a compute unit and K is long enough for the bytes to count (16 x 5632 -> 2048 6.48 -> 5.95, 4 x 4096 -> 512 3.95 -> 3.89,
  // 16 x 3072 -> 768 4.32 -> 3.91; short: 16 x 768 -> 768 2.67 -> 2.79, 4 x 768 -> 3072 3.06 -> 3.30).
  if (best.mt == 1 && M <= 8) best.bm = 8;
  if (best.nt == 1 && N / 8 <= (uint64_t)cus && K >= 2048) best.bn = 8;
  // Idle compute units fetch the weight into the L2s (warm_l2), two or three workgroups a tile that all find one, of an [N x K] weight
  // one.  [K x N], where a tile takes half of each line: 4 x 5632 -> 2048 13.5 -> 8.0 us, 8 x 4096 -> 512 8.3 -> 5.2, 16 x 5632 -> 2048 14.3 ->
  // 9.3, 64 x 4096 -> 1024 11.0 -> 7.2; one alone gets no further ahead than the tile's own loads (7 x 2464 -> 3328 7.5 -> 6.6, but 6 x 4896
  // -> 3936 11.4 -> 13.0).  [N x K], 32 columns a tile: 32 x 5632 -> 2048 9.9 -> 9.1 (with three 10.8), 64 x 4096 -> 1024 7.1 -> 6.5.  More
  // than the chip holds cost: 4 x 2048 -> 5632 (176 tiles) 7.1 -> 7.7.  Not where the weight is small (1 x 768 -> 768 2.93, 2.97) or X is not
  // (2000 x 5632 -> 64 12.0, 12.4).  These are of weights in the last-level cache; from HBM 4 x 5632 -> 2048 22.1 -> 10.4, 8 x 4096 -> 512 16.2 -> 7.3;
  // one weight multiplied again and again out of the L2s pays for it, 6.8 -> 7.1, 16 x 5632 -> 2048 6.9 -> 7.7.
  if (best.nt == 2 && (!w_is_nk || best.mt == 2) && 4 * M <= N && K >= 512 && K * N >= (uint64_t)1 << 20) {
    const uint64_t row = ((M + best.bm - 1) / best.bm * ((N + best.bn - 1) / best.bn) + 7) / 8 * 8, spare = (uint64_t)cus / row;
    best.warm = w_is_nk ? (spare >= 2 ? 1 : 0) : spare >= 4 ? 3 : spare == 3 ? 2 : 0;
  }
  // A contiguous part of the tiles per XCD, eight tile rows high, reads least into its L2, and what the L2s read comes in at 8 TB/s in
  // all: 1000 x 2304 -> 768 with groups of one tile column dealt round-robin 40 MB, 11.0 us, like this 25 MB, 10.0 ([K x N] 11.6,
  // 10.6); 2800 x 5184 -> 608 42.6, 30.7; 300 x 768 -> 768 4.9, 4.4; 68 sizes 0.97.  Few tiles or columns of them stay dealt out
  // ([K x N] 822 x 2816 -> 64 7.2, as a part 7.8, 372 x 4320 -> 128 11.3, 12.1; [N x K] 601 x 5568 -> 128 10.6, 10.3), and one row of them on
  // a [K x N] weight (16 x 2048 -> 5632 7.4, 7.7).
  // [K x N] weights of a multiple of 512 columns: the groups are whole rounds of the XCDs there, and beyond 2048 columns in one round of
  // workgroups they stay too.  The orders differ only for a weight that is multiplied again and again out of the L2s; in turn out of the L2s
  // and from HBM, groups and parts: 48 x 4096 -> 3072 7.7, 10.9 and 17.4, 17.3, 132 x 4096 -> 2560 10.5, 12.3 and 19.7, 19.7; up to 2048 columns
  // 48 x 4096 -> 2048 7.1, 7.3 and 16.5, 16.2, 250 x 1440 -> 1024 5.4, 5.4 and 7.9, 7.7; of more than a round 132 x 4096 -> 5632 24.1, 21.8 and 36.1,
  // 31.4.  Other widths: 48 x 4096 -> 2336 10.0, 7.9 and 13.3, 13.0, 132 x 4096 -> 2336 14.1, 12.4 and 17.4, 17.1; 18 of them beyond 2304 columns
  // 0.98 out of the L2s, 0.97 from the last-level cache, 0.98 from HBM.
  const uint64_t rows = (M + best.bm - 1) / best.bm, columns = (N + best.bn - 1) / best.bn, all = rows * columns;
  best.parts = columns >= (w_is_nk ? 4 : 6) && all >= 32 && (w_is_nk || (rows > 1 && (N % 512 != 0 || N <= 2048 || all > (uint64_t)cus)));
  return best;
}

// An [N x K] weight of 8 MB or more that the launch before wrote, and up to four tile rows: the order by groups.  What was written last
// comes in slower, and by parts that is all one XCD's.  us by parts and by groups, sampling in FP8 (8.1 of 2048 x 5632) and product: 1 x
// 2048 -> 5632 21.8, 17.3; 1 x 5632 -> 2048 20.3, 18.1; 64 x 2048 -> 5632 23.8, 19.9; 30 x 4096 -> 4096 26.2, 24.0; 203 x 2048 -> 3424 20.5,
// 18.4; 1 x 2048 -> 2048 10.7, 10.2.  Parts where the weight is smaller (469 x 1440 -> 2272 18.5, 19.2; 1 x 2272 -> 736 8.3, 8.5) or shared by
// more rows (261 x 2336 -> 5952 32.7, 33.5; 457 x 5792 -> 1792 33.0, 36.3); [K x N] 59 x 4128 -> 1888 18.8, 21.6.
void stream_after_sampling(const GemmArgs& g, int w_is_nk, StreamPlan& p) {
  if (p.p > 0 && w_is_nk && ((uint64_t)g.M + p.bm - 1) / p.bm <= 4 && (uint64_t)g.K * g.N >= (uint64_t)1 << 22) p.parts = 0;
}

bool stream_applicable(const GemmArgs& g) {
  return g.K >= 64 && g.K % 32 == 0 && g.N % 32 == 0 && g.M > 0 && g.N > 0 && g.ldx < stream::kMaxLd && g.ldw < stream::kMaxLd;
}

// WARM_KN, WARM_NK: the forms that stream_plan lets warm the L2
template <int MT, int NT, int P, int D, int BM = 16 * MT, int BN = 16 * NT, bool WARM_KN = false, bool WARM_NK = false>
static void launch_plain(GemmArgs g, int w_is_nk, const StreamPlan& p, hipStream_t s) {
  const int warm = WARM_KN || WARM_NK ? p.warm : 0;
  const dim3 tiles(stream::tile_grid(g, BM, BN, p.parts != 0)), grid(warm ? (tiles.x + 7) / 8 * 8 : tiles.x, 1 + warm), block(64 * P);
  if constexpr (WARM_NK) {
    if (w_is_nk && warm) {
      hipLaunchKernelGGL((gemm_stream_kernel<MT, NT, P, D, true, BM, BN, true>), grid, block, 0, s, GWS_GEMM_PASS(g));
      return;
    }
  }
  if constexpr (WARM_KN) {
    if (!w_is_nk && warm) {
      hipLaunchKernelGGL((gemm_stream_kernel<MT, NT, P, D, false, BM, BN, true>), grid, block, 0, s, GWS_GEMM_PASS(g));
      return;
    }
  }
  if (w_is_nk) {
    hipLaunchKernelGGL((gemm_stream_kernel<MT, NT, P, D, true, BM, BN>), tiles, block, 0, s, GWS_GEMM_PASS(g));
  } else if constexpr (NT >= 2) {
    hipLaunchKernelGGL((gemm_stream_kernel<MT, NT, P, D, false, BM, BN>), tiles, block, 0, s, GWS_GEMM_PASS(g));
  }
}

int launch_gemm_stream(const GemmArgs& g, int w_is_nk, const StreamPlan& p, hipStream_t s) {
  // Up to 16 rows of X on [N x K] weights: two units on their way a wavefront; more are in the way where the weight is in a cache.  us with two,
  // three and four, 4 x 5632 -> 2048 (8 x 8) in the last-level cache 5.7, 5.8, 5.9, from HBM 6.8, 6.2, 6.2; 16 x 5632 -> 2048 (16 x 8) 5.9, 6.1, 6.2 and
  // 7.8, 7.9, 8.0; 16 x 768 -> 768 (16 x 16) 2.6, 2.6, 2.6 and 3.0, 3.1, 3.1.
  if (p.bn == 8) p.bm == 8 ? launch_plain<1, 1, 8, 2, 8, 8>(g, w_is_nk, p, s) : launch_plain<1, 1, 8, 2, 16, 8>(g, w_is_nk, p, s);
  else if (p.bn == 16) p.bm == 8 ? launch_plain<1, 1, 8, 2, 8, 16>(g, w_is_nk, p, s) : launch_plain<1, 1, 8, 2>(g, w_is_nk, p, s);
  else if (p.bm == 8) launch_plain<1, 2, 8, 2, 8, 32, true>(g, w_is_nk, p, s);
  else if (p.mt == 1) launch_plain<1, 2, 8, 2, 16, 32, true>(g, w_is_nk, p, s);
  else if (p.mt == 2 && p.nt == 2) launch_plain<2, 2, 8, 2, 32, 32, true, true>(g, w_is_nk, p, s);
  else if (p.mt == 2) launch_plain<2, 4, 4, 3>(g, w_is_nk, p, s);
  else if (p.mt == 4) launch_plain<4, 4, 4, 2>(g, w_is_nk, p, s);
  else launch_plain<8, 4, 4, 1>(g, w_is_nk, p, s);
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

template <int MT, int P, int FMT, int B, bool TAIL>
static void launch_sampled(GemmArgs g, int w_is_nk, hipStream_t s) {
  const dim3 grid(stream::tile_grid(g, 16 * MT, 32));
  const uint32_t cus = compute_units() > 0 ? compute_units() : 256;
  // [N x K] in FP8 at 64 rows is 131 registers, three wavefronts a SIMD; with more workgroups than those hold, four and two registers
  // in scratch: 755 x 96 -> 2592 8.0 -> 6.8 us (with one workgroup a compute unit 61 x 160 -> 672 4.8 -> 5.0)
  constexpr bool kTight = MT == 4 && FMT == 1;
  if (w_is_nk && kTight && grid.x > (P == 4 ? 3 : 1) * cus)
    hipLaunchKernelGGL((gemm_stream_sample_kernel<MT, P, FMT, true, B, TAIL, kTight ? 4 : P / 4>), grid, dim3(64 * P), 0, s, GWS_GEMM_PASS(g), (const GemmSampling&)g);
  else if (w_is_nk) hipLaunchKernelGGL((gemm_stream_sample_kernel<MT, P, FMT, true, B, TAIL, P / 4>), grid, dim3(64 * P), 0, s, GWS_GEMM_PASS(g), (const GemmSampling&)g);
  else hipLaunchKernelGGL((gemm_stream_sample_kernel<MT, P, FMT, false, B, TAIL, P / 4>), grid, dim3(64 * P), 0, s, GWS_GEMM_PASS(g), (const GemmSampling&)g);
}

uint32_t stream_sample_rows(const GemmArgs& g, int p) { return p == 4 ? 64 : g.M <= 16 ? 16 : g.M <= 32 ? 32 : 64; }

// Up to 16 rows: two blocks a step where a compute unit has one workgroup, one where it has several, which then fit (16 x 96 -> 3232
// in FP6 5.6 us with a half step as a whole one, 4.9 as half; 1 x 2176 -> 20736 in FP8 36.5 us by two blocks, 28.1 by one).
template <int FMT>
static void launch_sampled_fmt(const GemmArgs& g, int w_is_nk, int p, hipStream_t s) {
  const uint32_t cus = compute_units() > 0 ? compute_units() : 256;
  const uint32_t rows = stream_sample_rows(g, p);
  if (p == 4) launch_sampled<4, 4, FMT, 1, false>(g, w_is_nk, s);
  else if (rows == 16 && g.N / 32 > cus) launch_sampled<1, 8, FMT, 1, false>(g, w_is_nk, s);
  else if (rows == 16 && (g.K & 32)) launch_sampled<1, 8, FMT, 2, true>(g, w_is_nk, s);
  else if (rows == 16) launch_sampled<1, 8, FMT, 2, false>(g, w_is_nk, s);
  else if (rows == 32) launch_sampled<2, 8, FMT, 1, false>(g, w_is_nk, s);
  else launch_sampled<4, 8, FMT, 1, false>(g, w_is_nk, s);
}

// 256 x 256 tiles (one on a compute unit) or 128 x 128 (two share it, or one has it).  us a unit of 64 k and round, FP8: 3.1; 2.25 with
// two and 1.45 with one.  FP6 and BF16 stand in the same proportion.  8192 x 2048 -> 2048 (1 round, 2 of two) 99 and 147 us; 5113 x
// 2592 -> 1664 (1, 1 and one of one) 132 and 146; 5497 x 1248 -> 4096 (2, 3 of two) 136 and 140; 6000 x 1536 -> 3072 (2, 2 and one of one)
// 159 and 141; 4096 x 1024 -> 2048 (1, 1) 56 and 44; 4000 x 2304 -> 800 (1, one of one) 102 and 53.
uint32_t rows_sample_tile(const GemmArgs& g) {
  const uint64_t cus = compute_units() > 0 ? compute_units() : 256;
  const uint64_t n = (uint64_t)((g.M + 127) / 128) * ((g.N + 127) / 128), rest = n % (2 * cus);
  const uint64_t n256 = (uint64_t)((g.M + 255) / 256) * ((g.N + 255) / 256);
  const double small = 2.25 * (double)(n / (2 * cus)) + (rest == 0 ? 0.0 : rest <= cus ? 1.45 : 2.25);
  return g.K > 64 && 3.1 * (double)((n256 + cus - 1) / cus) < small ? 256 : 128;   // one unit: 14.3 and 14.1 us for 4224 x 64 -> 2048
}
template <int FMT>
static void launch_rows(GemmArgs g, int w_is_nk, hipStream_t s) {
  const uint32_t t = rows_sample_tile(g);
  const dim3 grid(stream::tile_grid(g, t, t));
  if (t == 256 && w_is_nk) hipLaunchKernelGGL((gemm_rows_sample_kernel<FMT, true>), grid, dim3(512), 0, s, GWS_GEMM_PASS(g), (const GemmSampling&)g);
  else if (t == 256) hipLaunchKernelGGL((gemm_rows_sample_kernel<FMT, false>), grid, dim3(512), 0, s, GWS_GEMM_PASS(g), (const GemmSampling&)g);
  else if (w_is_nk && (g.K & 32)) hipLaunchKernelGGL((gemm_rows_pair_sample_kernel<FMT, true, true>), grid, dim3(512), 0, s, GWS_GEMM_PASS(g), (const GemmSampling&)g);
  else if (w_is_nk) hipLaunchKernelGGL((gemm_rows_pair_sample_kernel<FMT, true, false>), grid, dim3(512), 0, s, GWS_GEMM_PASS(g), (const GemmSampling&)g);
  else if (g.K & 32) hipLaunchKernelGGL((gemm_rows_pair_sample_kernel<FMT, false, true>), grid, dim3(512), 0, s, GWS_GEMM_PASS(g), (const GemmSampling&)g);
  else hipLaunchKernelGGL((gemm_rows_pair_sample_kernel<FMT, false, false>), grid, dim3(512), 0, s, GWS_GEMM_PASS(g), (const GemmSampling&)g);
}

// Two workgroups of 128 rows run on a compute unit: between one and one and a half rounds of them the 128 x 128 x 32 kernel, which
// packs them closer, is faster for [N x K] weights, which it need not transpose, where K is short.  4001 x K -> 2144, that kernel and
// 256 x 256 here: K = 160 17.5 and 17.9 us, 320 27.6 and 24.0, 544 43 and 36, 768 57 and 44, 2048 139 and 100.  The line is not at
// the crossing but where the difference is worth more than a launch.
bool rows_sample_applicable(const GemmArgs& g, int w_is_nk) {
  const uint64_t cus = compute_units() > 0 ? compute_units() : 256, n = (uint64_t)((g.M + 127) / 128) * ((g.N + 127) / 128);
  return stream_applicable(g) && !(w_is_nk && n > 2 * cus && n <= 3 * cus && g.K < 576);
}

int launch_gemm_rows_sample(const GemmArgs& g, int w_is_nk, int fmt, hipStream_t s) {
  switch (fmt) {
    case GWS_FMT_BF16: launch_rows<0>(g, w_is_nk, s); break;
    case GWS_FMT_FP8_E4M3: launch_rows<1>(g, w_is_nk, s); break;
    case GWS_FMT_FP6_E3M2: launch_rows<2>(g, w_is_nk, s); break;
    default: return GWS_ERR_FORMAT;
  }
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

// The same parts of K as the plain kernel (p), whatever the tile: the sums are the same bits.
int launch_gemm_stream_sample(const GemmArgs& g, int w_is_nk, int fmt, int p, hipStream_t s) {
  if ((uint64_t)((g.M + 15) / 16) * (g.N / 32) >= 0x7FFFFFFFull) return GWS_ERR_SHAPE;
  switch (fmt) {
    case GWS_FMT_BF16: launch_sampled_fmt<0>(g, w_is_nk, p, s); break;
    case GWS_FMT_FP8_E4M3: launch_sampled_fmt<1>(g, w_is_nk, p, s); break;
    case GWS_FMT_FP6_E3M2: launch_sampled_fmt<2>(g, w_is_nk, p, s); break;
    default: return GWS_ERR_FORMAT;
  }
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

}  // namespace gws
