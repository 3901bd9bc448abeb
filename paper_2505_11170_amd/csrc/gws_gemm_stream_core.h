// Pieces of the GEMMs whose wavefronts split the contraction (gws_gemm_stream.hip, gws_gemm_stream_tn.hip); internal to
// csrc/.  What these kernels are and why is said there.
#pragma once

#include "gws_gemm256_core.h"
#include "gws_launch.h"

namespace gws {

namespace stream {
constexpr uint32_t kMaxLd = 1u << 23;   // leading dimensions the 32-bit lane offsets reach (255 rows x 2 bytes)

__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }

// 64 lanes x 16 bytes from base + voff to 1 KiB of LDS at dst; the waits for such loads are the caller's.
__device__ __forceinline__ void direct(const GWS_GLOBAL char* base, uint32_t voff, uint16_t* dst) {
  const uint32_t a = (uint32_t)(uintptr_t)(GWS_LDS void*)dst;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(a) : "m0", "memory");
#pragma clang diagnostic pop
}

// Slot of a 16-byte chunk of k-row k in a stage stored output-contiguous, 16 T outputs wide: chunk ^ swizzle.  The 32 lanes
// that a transposing read serves together take four rows k % 4 of two row groups k / 8; with 256, 192, 128 and 64 bytes a row
// this puts them on different banks.
template <int T>
__device__ __forceinline__ uint32_t oc_swizzle(uint32_t k) {
  static_assert(T == 2 || T == 4 || T == 6 || T == 8, "");
  return T == 6 ? 2 * ((k >> 3) & 1) : T == 8 ? 4 * (k & 3) + 2 * ((k >> 3) & 1) : T == 4 ? 4 * ((k >> 1) & 1) + 2 * ((k >> 3) & 1) : 2 * ((k >> 3) & 1);
}

// Fragment (16 outputs from 16 j, 32 k from 32 h) of such a stage for lane (li = lane % 16, grp = lane / 16).
template <int T>
__device__ __forceinline__ Frag8 read_oc(const uint16_t* st, int h, int j, uint32_t li, uint32_t grp) {
  Frag8 f;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const uint32_t k = 32 * h + 8 * grp + 4 * t + (li >> 2), c = 2 * j + ((li >> 1) & 1);
    f.h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GWS_LDS i16x4*)(st + k * 16 * T + (c ^ oc_swizzle<T>(k)) * 8 + (li & 1) * 4));
  }
  return f;
}

// The units of 64 k that wavefront w of P takes, as even as they go (the last unit of K may be half a one).
__device__ __forceinline__ void unit_range(uint32_t K, uint32_t w, uint32_t P, uint32_t& u0, uint32_t& u1) {
  const uint32_t nu = (K + 63) >> 6;
  u0 = nu * w / P;
  u1 = nu * (w + 1) / P;
}

// First row and column of the workgroup's tile of bm x bn (tile_of_groups).
__device__ __forceinline__ void tile_origin(const GemmArgs& g, uint32_t bm, uint32_t bn, bool pairs, uint32_t& m0, uint32_t& n0) {
  uint32_t tm, tn;
  tile_of_groups(TileGrid{(g.M + bm - 1) / bm, (g.N + bn - 1) / bn, g.inv_band, g.inv_last}, pairs, blockIdx.x, tm, tn);
  m0 = tm * bm;
  n0 = tn * bn;
}
// The grid of such tiles, its reciprocals put into g; 0 if it is too large.  parts: for tile_of_joined.
inline uint32_t tile_grid(GemmArgs& g, uint32_t bm, uint32_t bn, bool parts = false) {
  const uint32_t mt = (uint32_t)(((uint64_t)g.M + bm - 1) / bm), nt = (uint32_t)(((uint64_t)g.N + bn - 1) / bn);
  if ((uint64_t)mt * nt >= 0x7FFFFFFFull) return 0;
  set_tile_grid(g, mt, nt, 8, parts);
  return mt * nt;
}

// The partial sums of the P wavefronts added in the order of the wavefronts, MC row tiles at a time.
// acc[i][j][e] is row 16 i + lane % 16, column 16 j + 4 (lane / 16) + e.  In LDS a row of partial sums is 16 NT floats and
// 16 bytes of padding: written by 16 lanes of as many rows, read along the row.
constexpr int red_bytes(int mc, int nt, int p) { return p * mc * 16 * (4 * nt + 1) * 16; }

// MC row tiles from i0: out(row, column / 4, sum) for every four columns of the 16 MC x 16 NT piece, spread over the threads.
template <int MT, int NT, int P, int MC, class Out>
__device__ __forceinline__ void sum_parts(const f32x4 (&acc)[MT][NT], char* lds, int i0, Out&& out) {
  constexpr uint32_t PITCH = 4 * NT + 1;
  f32x4* red = (f32x4*)lds;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __syncthreads();   // what was in this memory is read
#pragma unroll
  for (int i = 0; i < MC; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) red[((wave * MC + i) * 16 + (lane & 15)) * PITCH + 4 * j + (lane >> 4)] = acc[i0 + i][j];
  __syncthreads();
  for (uint32_t it = tid; it < MC * 16 * 4 * NT; it += P * 64) {
    const uint32_t r = it / (4 * NT), c = it % (4 * NT);
    f32x4 s = red[r * PITCH + c];
#pragma unroll
    for (int w = 1; w < P; ++w) {
      const f32x4 v = red[(w * MC * 16 + r) * PITCH + c];
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] = __fadd_rn(s[e], v[e]);
    }
    out(r, c, s);
  }
}

// BM x BN: the part of the 16 MT x 16 NT that is stored.
template <int MT, int NT, int P, int MC, int BM = 16 * MT, int BN = 16 * NT>
__device__ __forceinline__ void reduce_store(const f32x4 (&acc)[MT][NT], char* lds, const GemmArgs& g, uint32_t m0,
                                             uint32_t n0) {
#pragma unroll
  for (int i0 = 0; i0 < MT; i0 += MC)
    sum_parts<MT, NT, P, MC>(acc, lds, i0, [&](uint32_t r, uint32_t c, const f32x4& s) {
      const uint32_t row = m0 + 16 * i0 + r, col = n0 + 4 * c;
      if (row < g.M && col < g.N && (BM == 16 * MT || r < BM) && (BN == 16 * NT || 4 * c < BN))
        *(u32x2*)(g.y + (size_t)row * g.ldy + col) = u32x2{pack_bf16_rne(s[0], s[1]), pack_bf16_rne(s[2], s[3])};
    });
}
}  // namespace stream

}  // namespace gws
