// Weight gradient C[P x Q] = A^T B (A [tokens x P], B [tokens x Q], as in gws_gemm256_tn.hip) for weights of few tiles: a
// workgroup owns a piece of C, 64 x 32 to 128 x 128, and its four wavefronts split the tokens, as in gws_gemm_stream.hip.
// What bounds it: the operands' bytes, which every piece reads for itself.  All wavefronts of an XCD walk the tokens abreast, so
// most loads wait for a line that is on its way into the L2 (1.4 us), and the 110 to 140 KiB that the rings keep in flight give
// 72 to 92 B/ns a compute unit; the same loads from the L2 give 150 (96 x 96 pieces of 768 x 3072 over 4096 tokens: 84 % of the requests
// hit, the matrix cores work in 30 % of the cycles, the vector ALU in 20 %).  Against the 256-tile kernel with the tokens split over
// workgroups, no fp32 slabs go through memory and there is no second kernel.  Which piece: a whole number of rounds of workgroups,
// and few bytes.  Measured on MI355X with dL/db_t, us (tokens x P x Q; 64 x 32, 64 x 64, 128 x 64, 96 x 96, 128 x 128, and the
// 256-tile form that the sizes would take otherwise):
//   512 x 512 x 512 5.4, 6.2, 8.7, 9.7, 12, 19;       2048 x 1024 x 1024 18, 13.1, 16.9, 19.3, 23, 25;   4096 x 768 x 768 31, 19, 26, 30, -, 24
//   4096 x 768 x 3072 71, 49, 52, 30, -, 41;          2048 x 2048 x 2048 62, 41, 33, 37, 26, 40;         4096 x 768 x 2304 60, 36, 27, 29, -, 35
//   8192 x 2048 x 2048 272, 127, 97, 119, 72, 76;     1024 x 2048 x 4096 80, 52, 44, 47, 35, 40;         8192 x 512 x 512 29, 36, 48, 54, -, 29
// Both operands lie output-contiguous, so both stages are rows of 32 MT and 32 NT bytes a token and both fragments come from the
// transposing LDS load.  Where the workspace at hand would hold more than four parts, a wavefront sums its tokens in two
// halves, so that no fp32 sum is longer than in that form (not in 128 x 128 pieces, whose sums fill the registers).  On the way
// out each wavefront takes 32 x 32 blocks of the weight: 16 bytes a lane, one Philox group each, and the reduction of Eq. 4 over
// the wavefront.
#include <math.h>

#include "gws_gemm_stream_core.h"

namespace gws {

constexpr uint32_t kTnMaxLd = 1u << 26;   // leading dimensions the 32-bit lane offsets reach (31 rows x 2 bytes)

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
  if (g.M > g.N) tile_of(TileGrid{nt, mt, g.inv_band, g.inv_last}, blockIdx.x, n0, m0);
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
  return reads(4) < reads(8) * (1 - 1e-9) ? 4 : 8;
}

template <int MT, int NT, int D, bool HALVES>
static void launch_tn(GemmArgs g, bool with_dbt, hipStream_t s) {
  const uint32_t mt = (g.M + 16 * MT - 1) / (16 * MT), nt = (g.N + 16 * NT - 1) / (16 * NT);
  if (g.M > g.N) set_tile_grid(g, nt, mt, patch_band(nt, mt, 16 * NT, 16 * MT));   // the numbering runs along the longer side
  else set_tile_grid(g, mt, nt, patch_band(mt, nt, 16 * MT, 16 * NT));
  const dim3 grid(mt * nt);
  if (with_dbt) hipLaunchKernelGGL((gemm_stream_tn_kernel<MT, NT, D, true, HALVES>), grid, dim3(256), 0, s, GWS_GEMM_PASS(g), (const GemmSampling&)g);
  else hipLaunchKernelGGL((gemm_stream_tn_kernel<MT, NT, D, false, HALVES>), grid, dim3(256), 0, s, GWS_GEMM_PASS(g), (const GemmSampling&)g);
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
      {8, 8, 6.3, 0.68, {{83.5, 68.0}, {73.0, 59.5}}, 0.0}};
  for (const auto& t : tiles) {
    if (halves && t.mt * t.nt == 64) continue;
    const double n = ceil(g.M / (16.0 * t.mt)) * ceil(g.N / (16.0 * t.nt)), rounds = ceil(n / cus);
    const double* r = t.rate[lines ? 0 : 1];
    const double a_round = t.round + t.more * fmin(rounds - 1.0, 2.0) + (double)g.K * 2 * 16 * (t.mt + t.nt) / (r[0] + (r[1] - r[0]) * fmin(1.0, n / cus)) * 1e-3;
    const double us = 2.8 + rounds * a_round + (halves ? t.halves : 0.0);
    if (us < best.us) best = {t.mt, t.nt, us};
  }
  return best;
}

// halves: eight fp32 sums an element (768 x 768 over 4096 tokens 18.4 -> 18.9 us, 768 x 2304 26.4 -> 27.5).
int launch_gemm_stream_tn(const GemmArgs& g, bool with_dbt, const TnPlan& p, bool halves, hipStream_t stream) {
  if ((uint64_t)((g.M + 31) / 32) * ((g.N + 31) / 32) >= 0x7FFFFFFFull) return GWS_ERR_SHAPE;
  if (p.mt == 4 && p.nt == 2) halves ? launch_tn<4, 2, 4, true>(g, with_dbt, stream) : launch_tn<4, 2, 4, false>(g, with_dbt, stream);
  else if (p.mt == 4) halves ? launch_tn<4, 4, 4, true>(g, with_dbt, stream) : launch_tn<4, 4, 4, false>(g, with_dbt, stream);
  else if (p.mt == 6) halves ? launch_tn<6, 6, 3, true>(g, with_dbt, stream) : launch_tn<6, 6, 3, false>(g, with_dbt, stream);
  else if (p.nt == 4) halves ? launch_tn<8, 4, 3, true>(g, with_dbt, stream) : launch_tn<8, 4, 3, false>(g, with_dbt, stream);
  else launch_tn<8, 8, 2, false>(g, with_dbt, stream);
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

}  // namespace gws
