// Middle-tile BF16 MFMA GEMM for gfx950: Y[M x N] = X[M x K] * W (W stored [K x N] or [N x K]), any M, N and K of whole
// 32s.  For products with too few 256 x 256 tiles to fill the chip, or with edges that the large tile would pad.
//
// Workgroup = 2 x 2 wavefronts, tile 128 x 32 NJ (NJ 4 or 3), K-steps of 64; a wavefront owns 64 x 16 NJ of the output as 4 x NJ
// v_mfma_f32_16x16x32_bf16 tiles.  Both operand tiles (16 KiB, and 16 or 12) go global -> LDS directly into a ring of four stages,
// in the layouts of gws_gemm256_core.h (96 columns of a [K x N] weight as in gws_gemm_stream_core.h), three K-steps ahead; one
// barrier a K-step, between its two 32-deep halves: the second half's fragments are read under the first half's MFMAs, the next
// step's first ones under the second half's.
// What bounds it: a K-step of 128 x 128 takes 0.41 us (W [N x K]; 0.43 for [K x N]), of which the operands' 32 KiB from L2 alone 0.34, the
// MFMAs alone 0.25 and the LDS reads alone 0.17; misses in L2 are not it (0.39 without any).  A launch starts and
// ends in 5.7 us (6.0 with divisions in the tile numbering and the arguments in memory).
// 128 x 96 is for the sizes whose 128 x 128 tiles leave compute units idle in their rounds: 4096 x 3072 -> 768 is 256 tiles instead of
// 192, one round of either, 27.7 -> 23.7 us (816 TFLOP/s); 1000 x 768 -> 2304 8.7 -> 7.9; 3500 x 3008 -> 800 24.6 -> 21.2; 8192 x 2304
// -> 768, two rounds, 35.9 -> 32.8.  All of W [K x N]; [N x K] alike.  Each element's sum runs in the same order in both.
#include "gws_gemm_stream_core.h"

namespace gws {

namespace g128 {
constexpr int T = 128, TK = 64, D = 4;   // rows of a tile, depth of a K-step, stages
constexpr uint32_t kMaxLd = 1u << 24;    // 32-bit lane offsets: 127 rows x 2 bytes
__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }
}  // namespace g128

template <bool W_NK, int NJ>
__global__ __launch_bounds__(256) void gemm128_kernel(GWS_GEMM_PARAMS) {
  using namespace g128;
  const GemmArgs g = GWS_GEMM_GATHER({});
  constexpr int TN = 32 * NJ, OP = T * TK, STG = OP + TN * TK;   // columns of a tile; elements of the X tile, of a stage
  constexpr int PC = 16 * NJ + 8;                                // pitch of a wavefront's staged rows (elements)
  constexpr int LOADS = 4 + NJ;                                  // load instructions of a wavefront and K-step
  __shared__ __attribute__((aligned(1024))) uint16_t lds[D * STG];
  const uint32_t lane = threadIdx.x & 63, li = lane & 15, grp = lane >> 4;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave >> 1, wn = wave & 1;
  uint32_t tile_m, tile_n;
  tile_of(TileGrid{(g.M + T - 1) / T, (g.N + TN - 1) / TN, g.inv_band, g.inv_last}, blockIdx.x, tile_m, tile_n);
  const uint32_t m0 = tile_m * T, n0 = tile_n * TN;

  // a wavefront's load instructions of an operand tile, four and NJ; rows and columns past the edge are read from the last ones
  uint32_t xo[4], wo[NJ];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t row = 32 * wave + 8 * q + (lane >> 3), chunk = (lane & 7) ^ (4 * (q & 1) + (lane >> 4));
    // an instruction's offset counts on both sides: 1 KiB a load in LDS, taken back here
    xo[q] = (umin(row, g.M - 1 - m0) * g.ldx + chunk * 8) * 2 + 1024 * (3 - q);
  }
#pragma unroll
  for (int q = 0; q < NJ; ++q) {
    if (W_NK) {
      const uint32_t row = 8 * (NJ * wave + q) + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
      wo[q] = (umin(row, g.N - 1 - n0) * g.ldw + chunk * 8) * 2;
    } else {
      const uint32_t id = 64 * (NJ * wave + q) + lane, k = id / (4 * NJ), chunk = (id % (4 * NJ)) ^ stream::oc_swizzle<2 * NJ>(k);
      wo[q] = (k * g.ldw + umin(chunk, (g.N - n0) / 8 - 1) * 8) * 2;
    }
    wo[q] += 1024 * (3 - q);
  }
  const GWS_GLOBAL char* xb = (const GWS_GLOBAL char*)(g.x + (size_t)m0 * g.ldx) - 3072;
  const GWS_GLOBAL char* wb = (const GWS_GLOBAL char*)(W_NK ? g.w + (size_t)n0 * g.ldw : g.w + n0) - 3072;
  uint32_t k_next = 0;                   // first k of the step that is fetched next
  const uint32_t lds_x = (uint32_t)(uintptr_t)(GWS_LDS void*)lds + wave * 4096;
  const uint32_t lds_w = (uint32_t)(uintptr_t)(GWS_LDS void*)lds + OP * 2 + wave * (NJ * 1024);
  // two of a step's loads (n = 0 .. 3): X, W, X, W (of three of W the last one comes alone).  One wavefront a SIMD issues an
  // instruction in about five cycles, an MFMA takes sixteen: the loop has room for two instructions beside each MFMA, so addresses
  // are kept as running scalars and two loads share one setting of M0.
  auto load_n = [&](uint32_t stage, int n) {
    const uint32_t dst = (n & 1 ? lds_w : lds_x) + stage;
    const bool alone = NJ == 3 && n == 3;
    const uint32_t v0 = n & 1 ? wo[n & 2] : xo[n & 2], v1 = alone ? 0 : n & 1 ? wo[((n & 2) + 1) % NJ] : xo[(n & 2) + 1];
    const GWS_GLOBAL char* base = n & 1 ? wb : xb;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    if (n < 2)
      asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024"
                   ::"v"(v0), "v"(v1), "s"(base), "s"(dst) : "m0", "memory");
    else if (alone)
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:2048" ::"v"(v0), "s"(base), "s"(dst) : "m0", "memory");
    else
      asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2 offset:2048\n\tglobal_load_lds_dwordx4 %1, %2 offset:3072"
                   ::"v"(v0), "v"(v1), "s"(base), "s"(dst) : "m0", "memory");
#pragma clang diagnostic pop
  };
  auto load_advance = [&]() {   // the half step at the end of K is fetched as the second half of a whole one
    const uint32_t k = umin(k_next + TK, g.K - TK), d = __builtin_amdgcn_readfirstlane(k - k_next);
    xb += d * 2;
    wb += W_NK ? d * 2 : d * (g.ldw * 2);
    k_next = k;
  };
  Frag8 fx[2][4], fw[2][NJ];
  // read fragments of half h, step n of NR, in the order the MFMAs need them: X 0, W 0 .. NJ - 1, X 1 .. 3
  constexpr int RW = W_NK ? 1 : 2, NR = 4 + NJ * RW;
  uint32_t xr[2], wr[W_NK ? 2 : NJ];   // byte offsets in a stage
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t sl = ((4 * h + grp) ^ ((li >> 1) & 7)) * 16;
    xr[h] = (64 * wm + li) * 128 + sl;
    if (W_NK) wr[h] = OP * 2 + (16 * NJ * wn + li) * 128 + sl;
  }
  if (!W_NK)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const uint32_t k = 8 * grp + (li >> 2), c = 2 * (NJ * wn + j) + ((li >> 1) & 1);
      wr[j] = OP * 2 + k * (64 * NJ) + (c ^ stream::oc_swizzle<2 * NJ>(k)) * 16 + (li & 1) * 8;
    }
  auto read_n = [&](int h, uint32_t stage, int n) {
    const char* st = (const char*)lds + stage;
    if (n == 0 || n > NJ * RW) {
      const int i = n == 0 ? 0 : n - NJ * RW;
      fx[h][i].u = *(const u32x4*)(st + xr[h] + 2048 * i);
    } else if (W_NK) {
      fw[h][n - 1].u = *(const u32x4*)(st + wr[h] + 2048 * (n - 1));
    } else {
      const int j = (n - 1) >> 1, t = (n - 1) & 1;
      fw[h][j].h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GWS_LDS i16x4*)(st + wr[j] + 64 * NJ * (32 * h + 4 * t)));
    }
  };
  f32x4 acc[4][NJ];   // row 16 i + lane % 16, columns 16 j + 4 (lane / 16) .. + 3 of the wavefront's part
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  auto mfma_n = [&](int h, int n) {
    const int i = n / NJ, j = n % NJ;
    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[h][j].v, fx[h][i].v, acc[i][j], 0, 0, 0);
  };
  const uint32_t nk = (g.K + TK - 1) / TK;
#pragma unroll
  for (int s = 0; s < D; ++s)
    if ((uint32_t)s < nk) {
#pragma unroll
      for (int n = 0; n < 4; ++n) load_n(s * STG * 2, n);
      load_advance();
    }
  if (nk >= D) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LOADS * (D - 1)) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
  for (int n = 0; n < NR; ++n) read_n(0, 0, n);
  // The order is written out and pinned: a read behind each of the first MFMAs of a half, two loads of the step four ahead
  // behind every fourth MFMA of the second half (into the stage that the barrier has just released).
  auto first_half = [&](uint32_t stage) {
#pragma unroll
    for (int n = 0; n < 4 * NJ; ++n) {
      mfma_n(0, n);
      __builtin_amdgcn_sched_barrier(0);
      if (n < NR) read_n(1, stage, n);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto second_half = [&](uint32_t stage, uint32_t next, bool more) {
#pragma unroll
    for (int n = 0; n < 4 * NJ; ++n) {
      mfma_n(1, n);
      __builtin_amdgcn_sched_barrier(0);
      if (n < NR) read_n(0, next, n);
      if (more && n % NJ == NJ - 1) load_n(stage, n / NJ);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (more) load_advance();
  };
  uint32_t kt = 0, stage = 0;   // of the ring, in bytes
  auto after = [](uint32_t s) { return NJ == 4 ? (s + STG * 2) & (D * STG * 2 - 1) : s == (D - 1) * STG * 2 ? 0u : s + STG * 2; };
  for (; kt + D < nk; ++kt) {
    first_half(stage);
    // this stage is read; the next step has landed when all but the two steps behind it have
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LOADS * (D - 2)) : "memory");
    second_half(stage, after(stage), true);
    stage = after(stage);
  }
  // without this the register allocator passes the last accumulators on from register to register in the loop above (20 moves a
  // K-step and the waits for the MFMAs before them)
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) asm("" : "+a"(acc[i][j]));
  for (; kt < nk; ++kt) {   // everything is on its way: the reads past the last step fetch a stage that nobody multiplies
    if (TK * kt + TK > g.K) {
      // half a step at the end of K: the stage's first half belongs to the step before
#pragma unroll
      for (int i = 0; i < 4; ++i) fx[0][i].u = u32x4{0, 0, 0, 0};
#pragma unroll
      for (int j = 0; j < NJ; ++j) fw[0][j].u = u32x4{0, 0, 0, 0};
    }
    first_half(stage);
    if (kt + D == nk) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LOADS * (D - 2)) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    second_half(stage, after(stage), false);
    stage = after(stage);
  }
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the ring is read

  // out through LDS, 16 bytes a lane
  uint16_t* cs = lds + wave * (64 * PC);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      *(u32x2*)(cs + (16 * i + li) * PC + 16 * j + 4 * grp) =
          u32x2{pack_bf16_rne(acc[i][j][0], acc[i][j][1]), pack_bf16_rne(acc[i][j][2], acc[i][j][3])};
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wavefront's LDS writes have landed
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int it = 0; it < 2 * NJ; ++it) {
    const uint32_t id = 64 * it + lane, r = id / (2 * NJ), c = id % (2 * NJ), row = m0 + 64 * wm + r, col = n0 + 16 * NJ * wn + 8 * c;
    if (row < g.M && col < g.N) *(u32x4*)(g.y + (size_t)row * g.ldy + col) = *(const u32x4*)(cs + r * PC + 8 * c);
  }
}

bool gemm128_applicable(const GemmArgs& g) {
  return g.M > 0 && g.N > 0 && g.N % 32 == 0 && g.K % 32 == 0 && g.K >= 64 && g.ldx < g128::kMaxLd && g.ldw < g128::kMaxLd;
}

template <int NJ>
static int launch_tiles(GemmArgs g, int w_is_nk, hipStream_t stream) {
  const uint32_t mt = (uint32_t)(((uint64_t)g.M + g128::T - 1) / g128::T), nt = (uint32_t)(((uint64_t)g.N + 32 * NJ - 1) / (32 * NJ));
  if ((uint64_t)mt * nt >= 0x7FFFFFFFull) return GWS_ERR_SHAPE;
  set_tile_grid(g, mt, nt);
  if (w_is_nk) hipLaunchKernelGGL((gemm128_kernel<true, NJ>), dim3(mt * nt), dim3(256), 0, stream, GWS_GEMM_PASS(g));
  else hipLaunchKernelGGL((gemm128_kernel<false, NJ>), dim3(mt * nt), dim3(256), 0, stream, GWS_GEMM_PASS(g));
  return hipGetLastError() == hipSuccess ? GWS_OK : GWS_ERR_LAUNCH;
}

int launch_gemm128(const GemmArgs& g, int w_is_nk, int nj, hipStream_t stream) {
  return nj == 3 ? launch_tiles<3>(g, w_is_nk, stream) : launch_tiles<4>(g, w_is_nk, stream);
}

}  // namespace gws
