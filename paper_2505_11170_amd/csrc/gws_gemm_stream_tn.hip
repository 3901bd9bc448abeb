// Weight gradient C[P x Q] = A^T B (A [tokens x P], B [tokens x Q], as in gws_gemm256_tn.hip) for weights of few tiles: a
// workgroup owns a piece of C, 64 x 32 to 128 x 128.  Two kernels:
//  - gemm_stream_tn_kernel: its four wavefronts split the tokens, as in gws_gemm_stream.hip.  No barrier, but every wavefront holds the
//    whole piece's sums, which are added through LDS at the end (up to 144 KiB through it, 2 to 4 us).
//  - gemm_tile_tn_kernel: 2 x 2 wavefronts walk the tokens together, each with a quarter of the piece.  No sum to add up and a way
//    out of bf16 only, but a barrier every 64 tokens, at which all wait for the last line: the faster one for few tokens, and for longer the
//    nearer the operands lie.  us, first and second, from the last-level cache (tokens x P x Q):
//      64 x 768 x 768 in 64 x 64 4.9, 4.3, 128 4.9, 4.6, 256 5.1, 5.2, 1024 7.5, 8.1
//      64 x 768 x 2304 in 128 x 64 6.9, 5.4, 512 9.1, 8.7, 1024 11.7, 11.5, 1536 13.8, 13.8, 4032 x 2304 x 512 25.2, 25.7
//      64 x 768 x 3072 in 96 x 96 7.7, 6.3, 512 10.2, 10.2, 832 x 1536 x 1536 12.7, 11.9, 1536 x 768 x 3072 15.5, 15.8
//      2048 x 2048 x 2048 in 128 x 128 25.1, 24.2, 3072 32.0, 31.4, 4096 38.0, 38.3, 6144 52.5, 52.8
//    and from HBM: 2048 x 2048 x 2048 25.0, 26.2, 3072 32.0, 34.8, 4096 39.5, 46.7, 6144 52.3, 62.1; means of four to ten weights by tokens, second to
//    first, last-level cache, HBM, X from HBM and dY from the cache: 128 x 128 1024 0.95, 1.0, 1.0, 2048 0.97, 1.06, 1.06, 2560 0.98, 1.08, 1.08, 4096 0.99, 1.15,
//    1.14; 96 x 96 768 0.99, 1.02, 1.01, 1024 1.0, 1.04, 1.07, 1408 0.97, 1.05, 1.08; 128 x 64 896 0.92, 0.96, 0.92, 1216 0.96, 1.0, 0.99.
// What bounds them: the operands' bytes, which every piece reads for itself.  All wavefronts of an XCD walk the tokens abreast, so
// most loads wait for a line that is on its way into the L2 (1.4 us), and the 110 to 160 KiB that the rings keep in flight give
// 72 to 92 B/ns a compute unit; the same loads from the L2 give 150 (96 x 96 pieces of 768 x 3072 over 4096 tokens: 84 % of the requests
// hit, the matrix cores work in 30 % of the cycles, the vector ALU in 20 %).  Against the 256-tile kernel with the tokens split over
// workgroups, no fp32 slabs go through memory and there is no second kernel.  Which piece: a whole number of rounds of workgroups,
// and few bytes.  Measured on MI355X with dL/db_t, us (tokens x P x Q; 64 x 32, 64 x 64, 128 x 64, 96 x 96, 128 x 128, and the
// 256-tile form that the sizes would take otherwise):
//   512 x 512 x 512 5.4, 6.2, 8.7, 9.7, 12, 19;       2048 x 1024 x 1024 18, 11.1, 16.9, 19.3, 23, 25;   4096 x 768 x 768 31, 16.2, 26, 30, -, 24
//   4096 x 768 x 3072 71, 49, 52, 30, -, 41;          2048 x 2048 x 2048 62, 41, 33, 37, 24, 40;         4096 x 768 x 2304 60, 36, 26, 29, -, 35
//   8192 x 2048 x 2048 272, 127, 97, 119, 68, 76;     1024 x 2048 x 4096 80, 52, 44, 47, 30, 40;         8192 x 512 x 512 29, 36, 48, 54, -, 29
// Both operands lie output-contiguous, so both stages are rows of 2 bytes an output a token and both fragments come from the
// transposing LDS load.  The tokens are summed in four fp32 sums, so that none is longer than in that form with four parts: a wavefront's
// share of the tokens each, and the tile kernel adds its accumulators to a second set after every quarter of them.  Where the workspace at
// hand would hold more than four parts (from 2560 tokens on) the wavefronts sum their shares in two halves, eight sums; the tile kernel
// has no such form: below 2560 tokens nothing asks for it, and pieces of 128 x 128 are not taken then (stream_tn_plan).  On the way out each
// wavefront takes 32 x 32 blocks of the weight: 16 bytes a lane, one Philox group each, and the reduction of Eq. 4 over the wavefront.
#include <math.h>

#include "gws_gemm_stream_core.h"

namespace gws {

constexpr uint32_t kTnMaxLd = 1u << 26;   // leading dimensions the 32-bit lane offsets reach (31 rows x 2 bytes)
constexpr uint32_t kTileMaxLd = 1u << 25;   // (63 rows x 2 bytes)

// A 32 x 32 block as four 16 x 16 tiles in the MFMA's layout, rounded (pk[row half][column half]: lane l has row l % 16, columns
// 4 (l / 16) .. + 3), turned into 16-byte groups of rows: o[t] is row l % 16 + 16 t, columns 8 c .. + 7 with c = 0, 2, 1, 3 for
// l / 16 = 0 .. 3.  v_permlane16_swap exchanges the odd 16-lane rows of one register with the even ones of another.
__device__ __forceinline__ void swap_rows(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void rows_of_block(u32x2 (&pk)[2][2], u32x4 (&o)[2]) {
  u32x4 c[2];   // column half j: lanes of even rows have tile (0, j), of odd rows tile (1, j), 8 columns each
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    uint32_t a[2] = {pk[0][j][0], pk[0][j][1]}, b[2] = {pk[1][j][0], pk[1][j][1]};
    swap_rows(a[0], b[0]);
    swap_rows(a[1], b[1]);
    c[j] = u32x4{a[0], a[1], b[0], b[1]};
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t a = c[0][e], b = c[1][e];
    swap_rows(a, b);
    o[0][e] = a;
    o[1][e] = b;
  }
}

// The numbering runs along the longer side of C.  64 x 32 pieces of which an XCD gets at most eight: eight of one row, which read whole
// lines of dY, rather than four of two columns, which share one.  Over 64 to 8192 tokens 32 and 64 pieces 0.81 to 0.99 of along the rows
// (2688 x 256 x 512 12.0 -> 10.0 us, 4096 x 256 x 256 16.0 -> 14.4, 256 x 256 x 256 4.6 -> 4.5), 96 to 256 of them 0.98 to 1.11 (4096 x 256 x 768
// 14.4 -> 15.3, 8192 x 256 x 1280 25.0 -> 27.7, 8192 x 512 x 512 26.2, 26.2).
template <int NT>
__host__ __device__ __forceinline__ bool along_columns(const GemmArgs& g, uint32_t mt, uint32_t nt) {
  return g.M > g.N || (NT == 2 && mt * nt <= 64);
}

// A wavefront keeps D units of 32 tokens on their way into its own ring: both operands are rows of the outputs, so a unit may be
// as shallow as the MFMA is deep.
// HALVES: every wavefront sums its tokens in two halves, eight fp32 sums an element instead of four.
template <int MT, int NT, int D, bool DBT, bool HALVES>
__global__ __launch_bounds__(256, 1) void gemm_stream_tn_kernel(GWS_GEMM_PARAMS, const GemmSampling sampling) {
  using namespace stream;
  const GemmArgs g = GWS_GEMM_GATHER(sampling);
  constexpr int P = 4, U = 32, BM = 16 * MT, BN = 16 * NT;
  constexpr int XS = BM * U, STG = (BM + BN) * U, LOADS = MT + NT;   // elements of a stage; load instructions of a unit
  constexpr int BC = NT / 2, BLOCKS = MT / 2 * BC;                   // 32 x 32 blocks of the weight in the piece
  constexpr int PASS = BLOCKS <= 9 ? BLOCKS : 8, PASSES = BLOCKS / PASS, OWN = (PASS + P - 1) / P;   // blocks of a pass of the way out
  static_assert(MT % 2 == 0 && NT % 2 == 0 && PASS * PASSES == BLOCKS, "whole blocks");
  static_assert(LOADS * (D - 1) <= 63, "the wait for a unit counts the loads behind it");
  constexpr int kRing = P * D * STG * 2, kRed = P * PASS * 4 * 64 * 16;
  static_assert(kRing <= 160 * 1024 && kRed <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) char lds[kRing > kRed ? kRing : kRed];
  const uint32_t tid = threadIdx.x, lane = tid & 63, li = lane & 15, grp = lane >> 4;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint16_t* ring = (uint16_t*)lds + wave * (D * STG);
  uint32_t m0, n0, u0, u1;
  // Each XCD takes a contiguous part of the pieces, in bands along the shorter side of C: neighbouring pieces share lines and an
  // operand.  Along the rows whatever the shape, every XCD read all of the longer operand of a weight of few columns (1856 tokens
  // x 1792 x 256 in pieces of 64 x 32 11.9 us, like this 10.1; 7680 x 4096 x 256 in 64 x 64 47.2, 30.0); with groups of eight dealt
  // round-robin 2048 x 1024 x 1024 12.9, like this 11.0, 3072 x 768 x 256 13.8, 11.9, 8192 x 2048 x 2048 67.7, 66.0; 50 sizes 0.97.
  const uint32_t mt = (g.M + BM - 1) / BM, nt = (g.N + BN - 1) / BN;
  if (along_columns<NT>(g, mt, nt)) tile_of(TileGrid{nt, mt, g.inv_band, g.inv_last}, blockIdx.x, n0, m0);
  else tile_of(TileGrid{mt, nt, g.inv_band, g.inv_last}, blockIdx.x, m0, n0);
  m0 *= BM;
  n0 *= BN;
  unit_range(g.K, wave, P, u0, u1);
  u0 *= 2;   // in units of 32 (the tokens are whole 64s)
  u1 *= 2;

  // instruction q fetches the 64 chunks from 64 q of a stage of 32 rows of 2 T chunks; columns past the edge are read from the
  // first ones and not stored
  uint32_t xo[MT], wo[NT];
#pragma unroll
  for (uint32_t q = 0; q < MT; ++q) {
    const uint32_t id = 64 * q + lane, k = id / (2 * MT), c = (id % (2 * MT)) ^ oc_swizzle<MT>(k);
    xo[q] = (k * g.ldx + (8 * c < g.M - m0 ? 8 * c : 0)) * 2;
  }
#pragma unroll
  for (uint32_t q = 0; q < NT; ++q) {
    const uint32_t id = 64 * q + lane, k = id / (2 * NT), c = (id % (2 * NT)) ^ oc_swizzle<NT>(k);
    wo[q] = (k * g.ldw + (8 * c < g.N - n0 ? 8 * c : 0)) * 2;
  }
  const GWS_GLOBAL char* xb = (const GWS_GLOBAL char*)(g.x + m0);
  const GWS_GLOBAL char* wb = (const GWS_GLOBAL char*)(g.w + n0);
  auto load = [&](uint32_t u, uint32_t slot) __attribute__((always_inline)) {
    uint16_t* st = ring + slot * STG;
    const GWS_GLOBAL char* xu = xb + (size_t)(U * u) * g.ldx * 2;
    const GWS_GLOBAL char* wu = wb + (size_t)(U * u) * g.ldw * 2;
#pragma unroll
    for (uint32_t q = 0; q < MT; ++q) direct(xu, xo[q], st + q * 512);
#pragma unroll
    for (uint32_t q = 0; q < NT; ++q) direct(wu, wo[q], st + XS + q * 512);
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
  // Block b = PASS pass + P k + wave leaves through this wavefront.  Its noise is drawn while the first loads are on their way:
  // of each of its rows a lane writes 16 bytes, row lane % 16 + 16 t, column group 0, 2, 1 or 3 for lane / 16 = 0 .. 3.
  const uint32_t cgl = (grp >> 1) | ((grp & 1) << 1);
  auto block_of = [&](int pass, int k) { return (uint32_t)(PASS * pass + P * k) + wave; };
  auto exists = [&](int k, uint32_t b) { return P * k + wave < (uint32_t)PASS && m0 + b / BC * 32 < g.M && n0 + b % BC * 32 < g.N; };   // uniform
  Noise noise[PASSES][OWN][2];
  float scale[PASSES][OWN];
  if (DBT) {
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass)
#pragma unroll
      for (int k = 0; k < OWN; ++k) {
        const uint32_t b = block_of(pass, k), p0 = m0 + b / BC * 32, q0 = n0 + b % BC * 32;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          noise[pass][k][t] = group_noise(g.cg0 + (q0 >> 3) + cgl, g.row0 + p0 + li + 16 * t, g.step_lo, g.step_hi, g.seed_lo, g.seed_hi);
          asm volatile("" : "+v"(noise[pass][k][t].c));   // here and now
        }
        scale[pass][k] = exists(k, b) ? g.scale[(size_t)(p0 >> 5) * (g.N >> 5) + (q0 >> 5)] : 0.0f;
      }
  }
  uint32_t slot = 0;
  auto units = [&](uint32_t i, uint32_t end) __attribute__((always_inline)) {
    for (; i < end; ++i) {
      if (i + D <= n) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS * (D - 1)) : "memory");   // the unit has landed
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const uint16_t* xs = ring + slot * STG;
      Frag8 fx[MT], fw[NT];
#pragma unroll
      for (int r = 0; r < MT; ++r) fx[r] = read_oc<MT>(xs, 0, r, li, grp);
#pragma unroll
      for (int j = 0; j < NT; ++j) fw[j] = read_oc<NT>(xs + XS, 0, j, li, grp);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read: the stage can be filled again
      __builtin_amdgcn_sched_barrier(0);
      if (i + D < n) load(u0 + i + D, slot);
      slot = slot + 1 == D ? 0 : slot + 1;
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < MT; ++r) acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[j].v, fx[r].v, acc[r][j], 0, 0, 0);
    }
  };
  if (!HALVES) {
    units(0, n);
  } else {
    const uint32_t half = 2 * ((n / 2 + 1) >> 1);
    units(0, half);
    f32x4 first[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        first[i][j] = acc[i][j];
        acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      }
    units(half, n);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j][e] = __fadd_rn(first[i][j][e], acc[i][j][e]);
  }

  // The way out: all partial sums to LDS in register order (a block of 4 x 64 x 16 bytes per wavefront: every access 1 KiB of
  // consecutive memory), one barrier, and each wavefront adds its blocks' in the order of the wavefronts, rounds, and turns
  // the MFMA's layout into rows by swapping half rows between lanes (v_permlane16_swap): no second trip through LDS.
  f32x4* red = (f32x4*)lds;
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    __syncthreads();   // what was in this memory is read
#pragma unroll
    for (int b = 0; b < PASS; ++b) {
      const int i = (PASS * pass + b) / BC * 2, j = (PASS * pass + b) % BC * 2;
#pragma unroll
      for (int r = 0; r < 4; ++r) red[((b * P + wave) * 4 + r) * 64 + lane] = acc[i + (r >> 1)][j + (r & 1)];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < OWN; ++k) {
      const uint32_t b = block_of(pass, k), p0 = m0 + b / BC * 32, q0 = n0 + b % BC * 32;
      if (!exists(k, b)) continue;
      const f32x4* in = red + (P * k + wave) * (P * 4 * 64) + lane;
      f32x4 v[P][4];
#pragma unroll
      for (int w = 0; w < P; ++w)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[w][r] = in[(w * 4 + r) * 64];
      u32x2 pk[2][2];   // [row half][column half]: row lane % 16, columns 4 (lane / 16) .. + 3 of the 16 x 16 tile
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        f32x4 s = v[0][r];
#pragma unroll
        for (int w = 1; w < P; ++w)
#pragma unroll
          for (int e = 0; e < 4; ++e) s[e] = __fadd_rn(s[e], v[w][r][e]);
        pk[r >> 1][r & 1] = u32x2{pack_bf16_rne(s[0], s[1]), pack_bf16_rne(s[2], s[3])};
      }
      u32x4 o[2];
      rows_of_block(pk, o);
      float part = 0.0f;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        *(u32x4*)(g.y + (size_t)(p0 + li + 16 * t) * g.ldy + q0 + 8 * cgl) = o[t];
        if (DBT) part = dot_group_2r(o[t], noise[pass][k][t], part);
      }
      if (DBT) {
        part = block_sum_f32(part);
        part += __shfl_xor(part, 4);   // the block is the whole wavefront's here
        const float neg_ln2 = __uint_as_float(0xBF317218u);  // -ln 2
        if (lane == 0) g.dbt[(size_t)(p0 >> 5) * (g.N >> 5) + (q0 >> 5)] = (neg_ln2 * scale[pass][k]) * (part * 0.5f);
      }
    }
  }
}

uint32_t patch_band(uint32_t mt, uint32_t nt, uint32_t rows, uint32_t cols) {
  const int cus = compute_units();
  const double per = fmax(1.0, fmin((double)mt * nt, cus > 0 ? cus : 256) / 8);
  auto patch = [&](double r) {   // what the bands of r rows read, by their tile columns
    const double c = fmin(fmax(1.0, per / r), nt);
    return r * fmax(r, per / c) * rows + r * c * cols;
  };
  auto reads = [&](uint32_t b) { return mt / b * patch(b) + (mt % b ? patch(mt % b) : 0); };
  return !leaves_few(mt) && reads(4) < reads(8) * (1 - 1e-9) ? 4 : 8;
}

template <int MT, int NT, int D, bool HALVES>
static void launch_tn(GemmArgs g, bool with_dbt, hipStream_t s) {
  const uint32_t mt = (g.M + 16 * MT - 1) / (16 * MT), nt = (g.N + 16 * NT - 1) / (16 * NT);
  if (along_columns<NT>(g, mt, nt)) set_tile_grid(g, nt, mt, patch_band(nt, mt, 16 * NT, 16 * MT));
  else set_tile_grid(g, mt, nt, patch_band(mt, nt, 16 * MT, 16 * NT));
  const dim3 grid(mt * nt);
  if (with_dbt) hipLaunchKernelGGL((gemm_stream_tn_kernel<MT, NT, D, true, HALVES>), grid, dim3(256), 0, s, GWS_GEMM_PASS(g), (const GemmSampling&)g);
  else hipLaunchKernelGGL((gemm_stream_tn_kernel<MT, NT, D, false, HALVES>), grid, dim3(256), 0, s, GWS_GEMM_PASS(g), (const GemmSampling&)g);
}

// A piece of 32 WM x 32 WN by 2 x 2 wavefronts: all four load a stage of 64 tokens, D of them on their way, and each reads the
// fragments of its own quarter, half a stage ahead of the MFMAs that use them; one barrier a stage, between its halves, behind
// which the stage is filled again.  fold: the stages of an fp32 sum.
template <int WM, int WN, int D, bool DBT>
__global__ __launch_bounds__(256, 1) void gemm_tile_tn_kernel(GWS_GEMM_PARAMS, uint32_t fold, const GemmSampling sampling) {
  using namespace stream;
  const GemmArgs g = GWS_GEMM_GATHER(sampling);
  constexpr int BM = 32 * WM, BN = 32 * WN, TM = BM / 16, TN = BN / 16, U = 64;
  constexpr int XB = BM * U * 2, STG = (BM + BN) * U * 2, LOADS = WM + WN;   // bytes of the X stage, of a stage
  constexpr int BC = BN / 32, BLOCKS = BM / 32 * BC, OWN = (BLOCKS + 3) / 4, PITCH = BN + 8;
  constexpr int kRing = D * STG, kOut = BM * PITCH * 2;
  static_assert(kRing <= 160 * 1024 && LOADS * (D - 1) <= 63, "LDS; the wait for a stage counts the loads behind it");
  __shared__ __attribute__((aligned(1024))) char lds[kRing > kOut ? kRing : kOut];
  const uint32_t lane = threadIdx.x & 63, li = lane & 15, grp = lane >> 4;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave >> 1, wn = wave & 1;
  uint32_t m0, n0;
  const uint32_t mt = (g.M + BM - 1) / BM, nt = (g.N + BN - 1) / BN;
  if (g.M > g.N) tile_of(TileGrid{nt, mt, g.inv_band, g.inv_last}, blockIdx.x, n0, m0);
  else tile_of(TileGrid{mt, nt, g.inv_band, g.inv_last}, blockIdx.x, m0, n0);
  m0 *= BM;
  n0 *= BN;
  uint32_t xo[WM], wo[WN];
#pragma unroll
  for (uint32_t q = 0; q < WM; ++q) {
    const uint32_t id = 64 * (WM * wave + q) + lane, k = id / (2 * TM), c = (id % (2 * TM)) ^ oc_swizzle<TM>(k);
    xo[q] = (k * g.ldx + (8 * c < g.M - m0 ? 8 * c : 0)) * 2;
  }
#pragma unroll
  for (uint32_t q = 0; q < WN; ++q) {
    const uint32_t id = 64 * (WN * wave + q) + lane, k = id / (2 * TN), c = (id % (2 * TN)) ^ oc_swizzle<TN>(k);
    wo[q] = (k * g.ldw + (8 * c < g.N - n0 ? 8 * c : 0)) * 2;
  }
  const GWS_GLOBAL char* xb = (const GWS_GLOBAL char*)(g.x + m0);
  const GWS_GLOBAL char* wb = (const GWS_GLOBAL char*)(g.w + n0);
  const uint64_t xs = (uint64_t)g.ldx * (U * 2), ws = (uint64_t)g.ldw * (U * 2);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(GWS_LDS void*)lds, lds_x = lds0 + wave * (WM * 1024), lds_w = lds0 + XB + wave * (WN * 1024);
  auto load_n = [&](uint32_t stage, int n) __attribute__((always_inline)) {
    const uint32_t dst = (n < WM ? lds_x + n * 1024 : lds_w + (n - WM) * 1024) + stage;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(n < WM ? xo[n % WM] : wo[(n - WM) % WN]), "s"(n < WM ? xb : wb), "s"(dst) : "m0", "memory");
#pragma clang diagnostic pop
  };
  auto advance = [&]() __attribute__((always_inline)) {
    xb += xs;
    wb += ws;
  };
  Frag8 fx[2][WM], fw[2][WN];
  constexpr int NR = 2 * (WM + WN), NM = WM * WN;
  uint32_t xr[WM], wr[WN];
#pragma unroll
  for (int r = 0; r < WM; ++r) {
    const uint32_t k = 8 * grp + (li >> 2), c = 2 * (WM * wm + r) + ((li >> 1) & 1);
    xr[r] = k * (32 * TM) + (c ^ oc_swizzle<TM>(k)) * 16 + (li & 1) * 8;
  }
#pragma unroll
  for (int j = 0; j < WN; ++j) {
    const uint32_t k = 8 * grp + (li >> 2), c = 2 * (WN * wn + j) + ((li >> 1) & 1);
    wr[j] = XB + k * (32 * TN) + (c ^ oc_swizzle<TN>(k)) * 16 + (li & 1) * 8;
  }
  auto read_n = [&](int h, uint32_t stage, int n) __attribute__((always_inline)) {   // X 0, W 0 .. , X 1 ..
    const char* st = (const char*)lds + stage;
    const int t = n & 1, f = n >> 1;
    if (f == 0 || f > WN) {
      const int r = f == 0 ? 0 : f - WN;
      fx[h][r].h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GWS_LDS i16x4*)(st + xr[r] + 32 * TM * (32 * h + 4 * t)));
    } else {
      fw[h][f - 1].h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GWS_LDS i16x4*)(st + wr[f - 1] + 32 * TN * (32 * h + 4 * t)));
    }
  };
  f32x4 acc[WM][WN], sum[WM][WN];
#pragma unroll
  for (int r = 0; r < WM; ++r)
#pragma unroll
    for (int j = 0; j < WN; ++j) acc[r][j] = sum[r][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const uint32_t nk = g.K / U;
#pragma unroll
  for (int s = 0; s < D; ++s)
    if ((uint32_t)s < nk) {
#pragma unroll
      for (int n = 0; n < LOADS; ++n) load_n(s * STG, n);
      advance();
    }
  // noise of this wavefront's blocks while the first loads are on their way
  Noise noise[OWN][2];
  float scale[OWN];
  auto exists = [&](uint32_t b) { return b < (uint32_t)BLOCKS && m0 + b / BC * 32 < g.M && n0 + b % BC * 32 < g.N; };   // uniform
  if (DBT) {
#pragma unroll
    for (int k = 0; k < OWN; ++k) {
      const uint32_t b = 4 * k + wave, p0 = m0 + b / BC * 32, q0 = n0 + b % BC * 32;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        noise[k][t] = group_noise(g.cg0 + (q0 >> 3) + (lane & 3), g.row0 + p0 + (lane >> 2) + 16 * t, g.step_lo, g.step_hi, g.seed_lo, g.seed_hi);
        asm volatile("" : "+v"(noise[k][t].c));
      }
      scale[k] = exists(b) ? g.scale[(size_t)(p0 >> 5) * (g.N >> 5) + (q0 >> 5)] : 0.0f;
    }
  }
  if (nk >= D) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LOADS * (D - 1)) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
  for (int n = 0; n < NR; ++n) read_n(0, 0, n);
  auto mfma_n = [&](int h, int n) __attribute__((always_inline)) {
    const int r = n / WN, j = (r & 1) ? WN - 1 - n % WN : n % WN;
    acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[h][j].v, fx[h][r].v, acc[r][j], 0, 0, 0);
  };
  // half h's MFMAs, the next half's reads spread over them; in the second half the stage's refill too
  auto half = [&](int h, uint32_t stage, uint32_t next, bool more) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < NM; ++n) {
      mfma_n(h, n);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = n * NR / NM; k < (n + 1) * NR / NM; ++k) read_n(h ^ 1, h ? next : stage, k);
      if (h == 1 && more) {
#pragma unroll
        for (int k = n * LOADS / NM; k < (n + 1) * LOADS / NM; ++k) load_n(stage, k);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  uint32_t kt = 0, stage = 0, left = fold;
  auto after = [](uint32_t s) { return s == (D - 1) * STG ? 0u : s + STG; };
  auto folded = [&]() __attribute__((always_inline)) {
    if (--left == 0) {
      left = fold;
#pragma unroll
      for (int r = 0; r < WM; ++r)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            sum[r][j][e] = __fadd_rn(sum[r][j][e], acc[r][j][e]);
            acc[r][j][e] = 0.0f;
          }
    }
  };
  for (; kt + D < nk; ++kt) {
    half(0, stage, stage, false);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LOADS * (D - 2)) : "memory");
    half(1, stage, after(stage), true);
    advance();
    stage = after(stage);
    folded();
  }
  for (; kt < nk; ++kt) {
    half(0, stage, stage, false);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    half(1, stage, after(stage), false);
    stage = after(stage);
    folded();
  }
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the ring is read
  uint16_t* cs = (uint16_t*)lds;   // the piece as rows, rounded
#pragma unroll
  for (int r = 0; r < WM; ++r)
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = __fadd_rn(sum[r][j][e], acc[r][j][e]);
      *(u32x2*)(cs + (16 * (WM * wm + r) + li) * PITCH + 16 * (WN * wn + j) + 4 * grp) = u32x2{pack_bf16_rne(v[0], v[1]), pack_bf16_rne(v[2], v[3])};
    }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < OWN; ++k) {
    const uint32_t b = 4 * k + wave, p0 = m0 + b / BC * 32, q0 = n0 + b % BC * 32;
    if (!exists(b)) continue;
    float part = 0.0f;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const uint32_t row = (lane >> 2) + 16 * t, c = 8 * (lane & 3);
      const u32x4 o = *(const u32x4*)(cs + (b / BC * 32 + row) * PITCH + b % BC * 32 + c);
      *(u32x4*)(g.y + (size_t)(p0 + row) * g.ldy + q0 + c) = o;
      if (DBT) part = dot_group_2r(o, noise[k][t], part);
    }
    if (DBT) {
      part = block_sum_f32(part);
      part += __shfl_xor(part, 4);
      const float neg_ln2 = __uint_as_float(0xBF317218u);  // -ln 2
      if (lane == 0) g.dbt[(size_t)(p0 >> 5) * (g.N >> 5) + (q0 >> 5)] = (neg_ln2 * scale[k]) * (part * 0.5f);
    }
  }
}

template <int WM, int WN, int D>
static void launch_tile(GemmArgs g, bool with_dbt, hipStream_t s) {
  const uint32_t mt = (g.M + 32 * WM - 1) / (32 * WM), nt = (g.N + 32 * WN - 1) / (32 * WN);
  if (g.M > g.N) set_tile_grid(g, nt, mt, patch_band(nt, mt, 32 * WN, 32 * WM));
  else set_tile_grid(g, mt, nt, patch_band(mt, nt, 32 * WM, 32 * WN));
  const dim3 grid(mt * nt);
  const uint32_t fold = (g.K / 64 + 3) / 4;
  if (with_dbt) hipLaunchKernelGGL((gemm_tile_tn_kernel<WM, WN, D, true>), grid, dim3(256), 0, s, GWS_GEMM_PASS(g), fold, (const GemmSampling&)g);
  else hipLaunchKernelGGL((gemm_tile_tn_kernel<WM, WN, D, false>), grid, dim3(256), 0, s, GWS_GEMM_PASS(g), fold, (const GemmSampling&)g);
}

// The piece with the smallest estimate in us: a launch, and per round of workgroups (one per compute unit: the rings fill its
// LDS) a fixed part that grows with the rounds (a round's way out meets the next one's loads), and the bytes of the piece's
// operands at the rate a compute unit takes them, which falls with the share of them at work.
// lines: every row of X, dY and dW starts on a cache line (as they do in a model's own buffers).  Others touch one line more a row of
// a piece: the same fixed parts, lower rates, the lowest for the narrowest pieces (4096 x 768 x 3072, rows on lines and off: 64 x 64
// 48.5 and 67.5 us, 128 x 64 52 and 61, 96 x 96 30 and 33; 8192 x 2048 x 2048 in 128 x 128 72 and 76).
// Fitted to MI355X timings of every piece at 330 sizes either way, operands in turn from copies beyond the L2 (4 to 6 % off at one
// size), the choice between them, the 256-tile forms and the parts 0.05 % from the fastest in the mean, 0.2 % for rows off the lines.
TnPlan stream_tn_plan(const GemmArgs& g, bool lines, bool halves) {
  const double cus = compute_units() > 0 ? compute_units() : 256;
  TnPlan best = {0, 0, 1e30};
  if (g.ldx >= kTnMaxLd || g.ldw >= kTnMaxLd) return best;
  // fixed part of a round, what it grows by, bytes per ns with few and with all compute units at work (on lines, off), what the
  // halves cost
  static const struct { int mt, nt; double round, more, rate[2][2], halves; } tiles[] = {
      {4, 2, 0.9, 0.52, {{67.0, 65.0}, {52.5, 49.5}}, 0.1}, {4, 4, 1.45, 0.58, {{81.0, 70.0}, {57.5, 52.5}}, 0.5},
      {8, 4, 3.3, 0.64, {{85.0, 73.0}, {67.0, 60.0}}, 1.0}, {6, 6, 4.0, 0.61, {{80.0, 66.0}, {68.0, 60.5}}, 0.8},
      {8, 8, 6.3, 0.68, {{83.5, 68.0}, {73.0, 59.5}}, 0.0}};   // (by 2 x 2 wavefronts a little less: no choice among 75 sizes changes)
  for (const auto& t : tiles) {
    // 128 x 128: where eight sums are asked for the parts stay the form that gws_linear_bwd_w_form names (4544 x 1024 x 3072 45.1 us; in
    // pieces 40.0)
    if (t.mt * t.nt == 64 && (halves || g.ldx >= kTileMaxLd || g.ldw >= kTileMaxLd)) continue;
    const double n = ceil(g.M / (16.0 * t.mt)) * ceil(g.N / (16.0 * t.nt)), rounds = ceil(n / cus);
    const double* r = t.rate[lines ? 0 : 1];
    const double a_round = t.round + t.more * fmin(rounds - 1.0, 2.0) + (double)g.K * 2 * 16 * (t.mt + t.nt) / (r[0] + (r[1] - r[0]) * fmin(1.0, n / cus)) * 1e-3;
    const double us = 2.8 + rounds * a_round + (halves ? t.halves : 0.0);
    if (us < best.us) best = {t.mt, t.nt, us};
  }
  return best;
}

// halves: eight fp32 sums an element (768 x 768 over 4096 tokens 18.4 -> 18.9 us, 768 x 2304 26.4 -> 27.5).
// The bounds on the tokens lie where what the second kernel loses on operands from HBM passes what it gains on cached ones (head of this
// file; an activation that the forward pass kept comes from HBM).  The smaller the piece, the less there is to add up at the end, and the
// more a barrier costs.  The first kernel's wavefronts take whole units of 64 tokens, so off multiples of 256 the longest of the four
// shares is up to a tenth more than a quarter, and the bound lies further on (first to second, last-level cache and HBM, 128 x 128: 2112 tokens 1.09,
// 0.99, 2496 1.05, 0.95, 3136 1.06, 0.95; 2304 1.03, 0.94).
int launch_gemm_stream_tn(const GemmArgs& g, bool with_dbt, const TnPlan& p, bool halves, hipStream_t stream) {
  if ((uint64_t)((g.M + 31) / 32) * ((g.N + 31) / 32) >= 0x7FFFFFFFull) return GWS_ERR_SHAPE;
  const bool tile = g.ldx < kTileMaxLd && g.ldw < kTileMaxLd;   // 2 x 2 wavefronts
  const bool uneven = g.K % 256 != 0;
  if (p.mt == 8 && p.nt == 8) {
    if (g.K <= 2048 || (uneven && g.K < 4096)) launch_tile<4, 4, 5>(g, with_dbt, stream);
    else launch_tn<8, 8, 2, false>(g, with_dbt, stream);
  } else if (p.mt == 6) {
    if (tile && (g.K <= 960 || (uneven && g.K <= 1408))) launch_tile<3, 3, 6>(g, with_dbt, stream);
    else halves ? launch_tn<6, 6, 3, true>(g, with_dbt, stream) : launch_tn<6, 6, 3, false>(g, with_dbt, stream);
  } else if (p.mt == 8) {
    if (tile && g.K <= 1216) launch_tile<4, 2, 6>(g, with_dbt, stream);
    else halves ? launch_tn<8, 4, 3, true>(g, with_dbt, stream) : launch_tn<8, 4, 3, false>(g, with_dbt, stream);
  } else if (p.nt == 4) {
    if (tile && g.K <= 128) launch_tile<2, 2, 8>(g, with_dbt, stream);
    else halves ? launch_tn<4, 4, 4, true>(g, with_dbt, stream) : launch_tn<4, 4, 4, false>(g, with_dbt, stream);
  } else {
    if (tile && g.K <= 128) launch_tile<2, 1, 12>(g, with_dbt, stream);
    else halves ? launch_tn<4, 2, 4, true>(g, with_dbt, stream) : launch_tn<4, 2, 4, false>(g, with_dbt, stream);
  }
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

}  // namespace gws
