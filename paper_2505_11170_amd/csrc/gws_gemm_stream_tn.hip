// Weight gradient C[P x Q] = A^T B (A [tokens x P], B [tokens x Q], as in gws_gemm256_tn.hip) for weights of few tiles: a
// workgroup owns a 64 x 64 or 128 x 64 piece of C and its four wavefronts split the tokens, as in gws_gemm_stream.hip.
// What bounds it: the operands' bytes, which every tile reads for itself.  Against the 256-tile kernel with the tokens split
// over workgroups, no fp32 slabs go through memory and there is no second kernel.  Measured on MI355X with dL/db_t, us (tokens x
// P x Q; 64 x 64, 128 x 64 and the 256-tile form that the sizes took before): 512 x 512 x 512 5.8, 9.8, 19.1; 2048 x 1024 x
// 1024 12.1, 16.7, 25.6; 1536 x 1536 x 1024 17.6, 15.3, 25.9; 4096 x 768 x 768 17.1, 26.6, 23.9; 8192 x 1024 x 1024 34, 45,
// 37; 4096 x 768 x 3072 48, 49, 40.
// Both operands lie output-contiguous, so both stages are k-rows of 32 MT and 32 NT bytes and both fragments come from the
// transposing LDS load.  Where the workspace at hand would hold more than four parts, a wavefront sums its tokens in two
// halves, so that no fp32 sum is longer than in that form.  On the way out the sums are rounded to BF16 in LDS and each wavefront takes one 32 x 32 block of the
// weight: 16 bytes a lane, one Philox group each, and the reduction of Eq. 4 over the wavefront.
#include <math.h>

#include "gws_gemm_stream_core.h"

namespace gws {

// HALVES: every wavefront sums its tokens in two halves, eight fp32 sums an element instead of four.
template <int MT, int NT, int D, bool DBT, bool HALVES>
__global__ __launch_bounds__(256) void gemm_stream_tn_kernel(const GemmArgs g) {
  using namespace stream;
  constexpr int P = 4, BM = 16 * MT, BN = 16 * NT, PB = 64 + 8;
  constexpr int XS = BM * 64, STG = (BM + BN) * 64, QX = BM / 8, QW = BN / 8, LOADS = QX + QW;
  static_assert(NT == 4 && (MT == 4 || MT == 8), "a pass of the way out is 64 x 64: a block for each wavefront");
  static_assert(LOADS * (D - 1) <= 63, "the wait for a unit counts the loads behind it");
  constexpr int kRing = P * D * STG * 2, kRed = red_bytes(4, NT, P), kOut = 64 * PB * 2;
  __shared__ __attribute__((aligned(1024))) char lds[kRing > kRed + kOut ? kRing : kRed + kOut];
  const uint32_t tid = threadIdx.x, lane = tid & 63, li = lane & 15, grp = lane >> 4;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint16_t* ring = (uint16_t*)lds + wave * (D * STG);
  uint32_t m0, n0, u0, u1;
  tile_origin(g, BM, BN, false, m0, n0);
  unit_range(g.K, wave, P, u0, u1);

  // an instruction covers 512 / (16 T) k-rows of an operand 16 T outputs wide
  constexpr uint32_t RX = 32 / MT, RW = 32 / NT, NX = 16 / RX, NW = 16 / RW;
  uint32_t xo[NX], wo[NW];
#pragma unroll
  for (uint32_t v = 0; v < NX; ++v) {
    const uint32_t k = lane / (2 * MT), s = lane % (2 * MT);
    xo[v] = (k * g.ldx + (s ^ oc_swizzle<MT>(k + RX * v)) * 8) * 2;
  }
#pragma unroll
  for (uint32_t v = 0; v < NW; ++v) {
    const uint32_t k = lane / (2 * NT), s = lane % (2 * NT);
    wo[v] = (k * g.ldw + (s ^ oc_swizzle<NT>(k + RW * v)) * 8) * 2;
  }
  const GWS_GLOBAL char* xb = (const GWS_GLOBAL char*)(g.x + m0);
  const GWS_GLOBAL char* wb = (const GWS_GLOBAL char*)(g.w + n0);
  auto load = [&](uint32_t u, uint32_t slot) {
    uint16_t* st = ring + slot * STG;
#pragma unroll
    for (uint32_t q = 0; q < QX; ++q) direct(xb + (size_t)(64 * u + RX * q) * g.ldx * 2, xo[q % NX], st + q * 512);
#pragma unroll
    for (uint32_t q = 0; q < QW; ++q) direct(wb + (size_t)(64 * u + RW * q) * g.ldw * 2, wo[q % NW], st + XS + q * 512);
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
  auto units = [&](uint32_t i, uint32_t end) {
    for (; i < end; ++i) {
      if (i + D <= n) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS * (D - 1)) : "memory");   // the unit has landed
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const uint16_t* xs = ring + slot * STG;
      Frag8 fx[2][MT], fw[2][NT];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int r = 0; r < MT; ++r) fx[h][r] = read_oc<MT>(xs, h, r, li, grp);
#pragma unroll
        for (int j = 0; j < NT; ++j) fw[h][j] = read_oc<NT>(xs + XS, h, j, li, grp);
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read: the stage can be filled again
      __builtin_amdgcn_sched_barrier(0);
      if (i + D < n) load(u0 + i + D, slot);
      slot = slot + 1 == D ? 0 : slot + 1;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int r = 0; r < MT; ++r) acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[h][j].v, fx[h][r].v, acc[r][j], 0, 0, 0);
    }
  };
  if (!HALVES) {
    units(0, n);
  } else {
    const uint32_t half = (n + 1) >> 1;
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

  uint16_t* cs = (uint16_t*)(lds + kRed);
#pragma unroll
  for (int i0 = 0; i0 < MT; i0 += 4) {
    sum_parts<MT, NT, P, 4>(acc, lds, i0, [&](uint32_t r, uint32_t c, const f32x4& s) {
      *(u32x2*)(cs + r * PB + 4 * c) = u32x2{pack_bf16_rne(s[0], s[1]), pack_bf16_rne(s[2], s[3])};
    });
    __syncthreads();
    const uint32_t p0 = m0 + 16 * i0 + 32 * (wave >> 1), q0 = n0 + 32 * (wave & 1), row = lane >> 2, c = (lane & 3) * 8;
    float part = 0.0f;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const u32x4 o = *(const u32x4*)(cs + (32 * (wave >> 1) + row + 16 * t) * PB + 32 * (wave & 1) + c);
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
}

template <int MT, int D, bool HALVES>
static void launch_tn(const GemmArgs& g, bool with_dbt, hipStream_t s) {
  const dim3 grid((g.M / (16 * MT)) * (g.N / 64));
  if (with_dbt) hipLaunchKernelGGL((gemm_stream_tn_kernel<MT, 4, D, true, HALVES>), grid, dim3(256), 0, s, g);
  else hipLaunchKernelGGL((gemm_stream_tn_kernel<MT, 4, D, false, HALVES>), grid, dim3(256), 0, s, g);
}

// mt: row tiles of 16 of the piece (4 or 8); us: the estimate as in stream_plan.  The larger piece's fixed part of a round
// grows with the rounds (a round's reductions and stores meet the next one's loads): 1024 tokens in one, three and four rounds
// 10, 36 and 44 us.
TnPlan stream_tn_plan(const GemmArgs& g, bool halves) {
  const double cus = compute_units() > 0 ? compute_units() : 256;
  TnPlan best = {0, 1e30};
  // fixed part of a round, what it grows by, bytes per ns that a compute unit takes, what the halves cost
  static const struct { int mt; double round, more, rate, halves; } tiles[] = {{4, 2.7, 0.0, 82.0, 0.6}, {8, 3.5, 0.7, 75.0, 1.8}};
  for (const auto& t : tiles) {
    const double rounds = ceil((double)(g.M / (16 * t.mt)) * (double)(g.N / 64) / cus);
    const double a_round = t.round + t.more * fmin(rounds - 1.0, 2.0) + (double)g.K * 2 * 16 * (t.mt + 4) / t.rate * 1e-3;
    const double us = 2.8 + rounds * a_round + (halves ? t.halves : 0.0);
    if (us < best.us) best = {t.mt, us};
  }
  return best;
}

// halves: eight fp32 sums an element (512 x 512 over 1024 tokens 6.7 -> 7.9 us, 768 x 2304 over 4096 27.6 -> 29.0).
int launch_gemm_stream_tn(const GemmArgs& g, bool with_dbt, const TnPlan& p, bool halves, hipStream_t stream) {
  if ((uint64_t)(g.M / 64) * (g.N / 64) >= 0x7FFFFFFFull) return GWS_ERR_SHAPE;
  if (p.mt == 4) halves ? launch_tn<4, 2, true>(g, with_dbt, stream) : launch_tn<4, 2, false>(g, with_dbt, stream);
  else halves ? launch_tn<8, 1, true>(g, with_dbt, stream) : launch_tn<8, 1, false>(g, with_dbt, stream);
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

}  // namespace gws
