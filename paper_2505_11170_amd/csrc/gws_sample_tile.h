// Wavefront-tile building blocks of the forward pass (paper Eq. 3 + cast), shared by
// the elementwise kernel and the sampling prologue of the fused linear.
// Internal to csrc/.
#pragma once

#include "gws_launch.h"

namespace gws {

// Valid elements of the 16-byte group at (row, col): 8, fewer at a ragged right
// edge, 0 outside.
__device__ __forceinline__ int valid_count(uint32_t row, uint32_t col, uint32_t rows, uint32_t cols) {
  if (row >= rows || col >= cols) return 0;
  const uint32_t left = cols - col;
  return left >= 8 ? 8 : (int)left;
}

// Streaming (non-temporal) or ordinary accesses.  STREAM = kKeep: everything stays in the caches, right for a call whose output
// is read at once and for rows that do not start on cache lines (a line written in two halves is put together in L2; written
// past it, each half costs a partial write); kStreamReads: what is read streams past the caches; kStreamAll: writes too.
template <int STREAM = kStreamAll>
__device__ __forceinline__ u32x4 load16(const GWS_GLOBAL uint16_t* p) {
  if (STREAM != kKeep) return __builtin_nontemporal_load((const GWS_GLOBAL u32x4*)p);
  return *(const GWS_GLOBAL u32x4*)p;
}
template <int STREAM = kStreamAll>
__device__ __forceinline__ void store16(GWS_GLOBAL uint16_t* p, const u32x4 v) {
  if (STREAM == kStreamAll) __builtin_nontemporal_store(v, (GWS_GLOBAL u32x4*)p);
  else *(GWS_GLOBAL u32x4*)p = v;
}

// Zero the elements of a group that lie past the right edge (nv valid of 8).
__device__ __forceinline__ u32x4 mask_group(u32x4 v, int nv) {
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if (k >= nv) v[k >> 1] &= (k & 1) ? 0x0000FFFFu : 0xFFFF0000u;
  return v;
}

__device__ __forceinline__ void store_partial(GWS_GLOBAL uint16_t* dst, const u32x4 v, int nv) {
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if (k < nv) dst[k] = (uint16_t)(v[k >> 1] >> ((k & 1) * 16));
}

// The four 16-byte groups a lane holds of one wavefront tile.
struct Tile {
  u32x4 v[4];
  int nv[4];   // valid elements per group (8 everywhere on a full tile)
  uint32_t rows;   // of the tile that exist (unset on a full tile)
  bool full;   // the 32x64 tile lies inside the tensor: no validity tests needed
};

// A full tile is addressed by a scalar base per group of eight rows and one 32-bit byte offset of the lane for all of them
// (15 of 454 vector instructions of a BF16 tile were 64-bit address additions); tensors with longer rows go tile by tile as
// edges do, with 64-bit addresses (kMaxLaneLd).
__device__ __forceinline__ uint32_t lane_offset(uint32_t ld, uint32_t lane) { return ((lane >> 3) * ld + (lane & 7) * 8) * 2; }

// A uniform pointer plus the lane's bytes.  The empty asm statement keeps the compiler from adding the lane's share first and
// the scalar one to each row's address in vector registers, and from widening the lane's share ahead of time.
template <class T>
__device__ __forceinline__ GWS_GLOBAL T* at_byte(GWS_GLOBAL T* p, uint32_t byte) {
  uint64_t base = (uint64_t)(uintptr_t)p;
  asm("" : "+s"(base), "+v"(byte));
  return (GWS_GLOBAL T*)((GWS_GLOBAL char*)(uintptr_t)base + byte);
}

template <int STREAM = kStreamAll>
__device__ __forceinline__ Tile load_full_tile(const GWS_GLOBAL uint16_t* __restrict__ src, const TileDesc& d, uint32_t by,
                                               uint32_t col_base, uint32_t lane) {
  Tile t;
  t.full = true;
  const uint32_t off = lane_offset(d.ld, lane);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    t.nv[i] = 8;
    t.v[i] = load16<STREAM>(at_byte(src + ((size_t)(by * 32 + 8 * i) * d.ld + col_base), off));
  }
  return t;
}

// A 16-byte load never leaves its row: ld % 8 == 0 and ld >= cols.
template <int STREAM = kStreamAll>
__device__ __forceinline__ Tile load_tile(const GWS_GLOBAL uint16_t* __restrict__ src, const TileDesc& d, uint32_t by,
                                          uint32_t col_base, uint32_t lane) {
  const uint32_t row_base = by * 32, col = col_base + (lane & 7) * 8;
  if (row_base + 32 <= d.rows && col_base + 64 <= d.cols && d.ld < kMaxLaneLd && d.ldc < kMaxLaneLd)
    return load_full_tile<STREAM>(src, d, by, col_base, lane);
  Tile t;
  t.full = false;
  t.rows = d.rows - row_base;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t row = row_base + (lane >> 3) + 8 * i;
    t.nv[i] = valid_count(row, col, d.rows, d.cols);
    t.v[i] = u32x4{0, 0, 0, 0};
    if (t.nv[i] > 0) t.v[i] = load16<STREAM>(src + (size_t)row * d.ld + col);
  }
  return t;
}

// What the noise of a lane's four groups is kept as until it is applied: the bit basis as codes (a register a group), the
// comparison bases as the random words.  It depends on no load, so it is drawn while the tile is on its way.
template <int BASIS>
struct TileNoise {
  Philox4 x[4];
};
template <>
struct TileNoise<kBasisBits> {
  Noise x[4];
};

// The lane's block parameter, 0 for a block past the right edge.
__device__ __forceinline__ float lane_bt(const TileDesc& d, uint32_t by, uint32_t col_base, uint32_t lane) {
  const uint32_t nbc = (d.cols + 31) >> 5, bcol = (col_base >> 5) + ((lane >> 2) & 1);
  return bcol < nbc ? global_ptr<float>(d.p2)[(size_t)by * nbc + bcol] : 0.0f;
}

// Pins the noise where it is drawn; of the random words those that the basis uses (the uniform basis two of four: the others are
// then not computed).
__device__ __forceinline__ void pin_noise(Noise& n) { asm volatile("" : "+v"(n.c)); }
template <int BASIS>
__device__ __forceinline__ void pin_noise(Philox4& x) {
  asm volatile("" : "+v"(x.x0), "+v"(x.x1));
  if (BASIS != kBasisUniform) asm volatile("" : "+v"(x.x2), "+v"(x.x3));
}

__device__ __forceinline__ PhiloxRows tile_rows(const TileDesc& d, uint32_t by, uint32_t lane, uint32_t step_lo) {
  uint32_t rows[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) rows[i] = d.row0 + by * 32 + (lane >> 3) + 8 * i;
  return philox_rows(rows, step_lo, d.seed_lo);
}

// T tiles of one block row, 64 columns apart from col_base on
template <int BASIS, int T>
__device__ __forceinline__ void draw_noise(uint32_t step_lo, uint32_t step_hi, const TileDesc& d, const PhiloxRows& rp,
                                           uint32_t col_base, uint32_t lane, TileNoise<BASIS> (&n)[T]) {
  PhiloxCols pc[T];
#pragma unroll
  for (int t = 0; t < T; ++t) pc[t] = philox_cols(d.cg0 + ((col_base + 64 * t) >> 3) + (lane & 7), step_lo, step_hi, d.seed_lo, d.seed_hi);
  Philox4 x[T][4];
  philox_tiles(pc, rp, d.seed_lo, d.seed_hi, x);
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (BASIS == kBasisBits) n[t].x[i] = noise_codes(x[t][i]);
      else n[t].x[i] = x[t][i];
    }
  // here and now: the compiler would sink the noise to its use, behind the wait for the tile
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (BASIS == kBasisBits) pin_noise(n[t].x[i]);
      else pin_noise<BASIS>(n[t].x[i]);
    }
}

// The noise of a tile at an edge: two groups of eight rows together, one alone, none for rows past the tensor's (eight weights of 16
// rows of 312128, backward: 33 us with all four groups, 24 like this).
template <int BASIS>
__device__ __forceinline__ void draw_noise_edge(uint32_t step_lo, uint32_t step_hi, const TileDesc& d, uint32_t by, uint32_t col_base,
                                                uint32_t lane, TileNoise<BASIS>& n) {
  const PhiloxCols pc[1] = {philox_cols(d.cg0 + (col_base >> 3) + (lane & 7), step_lo, step_hi, d.seed_lo, d.seed_hi)};
  const uint32_t rows = d.rows - by * 32;
  auto groups = [&](auto& x, int i) __attribute__((always_inline)) {   // as many as x holds from group i on
    constexpr int R = sizeof(x[0]) / sizeof(Philox4);
    const uint32_t r = d.row0 + by * 32 + (lane >> 3) + 8 * i, row[4] = {r, r + 8, 0, 0};
    philox_tiles(pc, philox_rows(row, step_lo, d.seed_lo), d.seed_lo, d.seed_hi, x);
#pragma unroll
    for (int k = 0; k < R; ++k) {
      if constexpr (BASIS == kBasisBits) n.x[i + k] = noise_codes(x[0][k]);
      else n.x[i + k] = x[0][k];
    }
  };
#pragma unroll
  for (int i = 0; i < 4; i += 2) {   // uniform branches
    n.x[i] = n.x[i + 1] = {};
    if (rows > 8u * i + 8) {
      Philox4 x[1][2];
      groups(x, i);
    } else if (rows > 8u * i) {
      Philox4 x[1][1];
      groups(x, i);
    }
  }
}

// Element codes of one group to memory.  FP8: 8 bytes at column col.  FP6: 6 bytes at
// (col / 8) * 6, written as three 2-byte stores (a row of codes is only 2-byte aligned).
// nv < 8: only the bytes that hold existing elements (unused bits of the last one are 0).
template <int FMT, int STREAM>
__device__ __forceinline__ void store_codes(GWS_GLOBAL uint8_t* row, uint32_t col, const MxCodes c, int nv) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  if (FMT == 1) {
    GWS_GLOBAL uint8_t* dst = row + col;
    if (nv == 8) {
      if (STREAM == kStreamAll) __builtin_nontemporal_store(u32x2{c.lo, c.hi}, (GWS_GLOBAL u32x2*)dst);
      else *(GWS_GLOBAL u32x2*)dst = u32x2{c.lo, c.hi};
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k < nv) dst[k] = (uint8_t)((k < 4 ? c.lo : c.hi) >> (8 * (k & 3)));
    }
  } else {
    GWS_GLOBAL uint8_t* dst = row + (col >> 3) * 6;
    if (nv == 8) {
      GWS_GLOBAL uint16_t* d16 = (GWS_GLOBAL uint16_t*)dst;
      d16[0] = (uint16_t)c.lo;
      d16[1] = (uint16_t)(c.lo >> 16);
      d16[2] = (uint16_t)c.hi;
    } else {
      // the fields of elements past the edge hold noise: clear them
      const uint64_t bits = (((uint64_t)c.hi << 32) | c.lo) & (((uint64_t)1 << (6 * nv)) - 1);
      const int nbytes = (nv * 6 + 7) >> 3;
#pragma unroll
      for (int k = 0; k < 6; ++k)
        if (k < nbytes) dst[k] = (uint8_t)(bits >> (8 * k));
    }
  }
}

// The FP6 codes of a whole tile.  A lane holds 48 bits of each of its four rows r0 + 8 i; within each quad of lanes (four
// column groups side by side) the 4 x 4 pieces are exchanged, so that a lane ends up with the 24 consecutive bytes of one
// row: row r0 + 8 (lane % 4), byte (lane & 4) * 6 of the tile's 48.
struct Codes24 {
  uint32_t w[6];
};
__device__ __forceinline__ Codes24 codes_fp6_quad(uint32_t lane, const uint32_t (&c)[6]) {
  // piece i = 32 low bits lo[i] and 16 high bits: of pieces 0, 1 in h01, of pieces 2, 3 in h23
  uint32_t lo[4] = {c[0], __builtin_amdgcn_alignbit(c[2], c[1], 16), c[3], __builtin_amdgcn_alignbit(c[5], c[4], 16)};
  const uint32_t h01 = __builtin_amdgcn_perm(c[2], c[1], 0x07060100u), h23 = __builtin_amdgcn_perm(c[5], c[4], 0x07060100u);
  const bool odd = lane & 1, upper = lane & 2;
  // lane q of a quad collects piece q of every lane: exchange with lane ^ 1, then with lane ^ 2
#pragma unroll
  for (int i = 0; i < 4; i += 2) {
    const uint32_t a = lo[i], b = lo[i + 1], pa = dpp_u32<0xB1>(a), pb = dpp_u32<0xB1>(b);
    lo[i] = odd ? pb : a;       // from the even lane of the pair
    lo[i + 1] = odd ? b : pa;   // from the odd one
  }
  // now lo[i + j] is piece i + lane % 2 of lane (pair base) + j, i = 0, 2
  uint32_t l[4];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const uint32_t a = lo[j], b = lo[2 + j], pa = dpp_u32<0x4E>(a), pb = dpp_u32<0x4E>(b);
    l[j] = upper ? pb : a;       // lane j of the quad
    l[2 + j] = upper ? b : pa;   // lane 2 + j
  }
  const uint32_t p01 = dpp_u32<0x4E>(h01), p23 = dpp_u32<0x4E>(h23);
  const uint32_t first = upper ? p23 : h01, second = upper ? h23 : p01;   // pieces of the lower and the upper lane of {q, q ^ 2}
  const uint32_t pf = dpp_u32<0xB1>(first), ps = dpp_u32<0xB1>(second);
  // halves of this lane's and its neighbour's word, the even lane's first: bytes 0-3 of v_perm are the second operand's
  const uint32_t sel = odd ? 0x07060302u : 0x05040100u;
  const uint32_t g01 = odd ? __builtin_amdgcn_perm(first, pf, sel) : __builtin_amdgcn_perm(pf, first, sel);
  const uint32_t g23 = odd ? __builtin_amdgcn_perm(second, ps, sel) : __builtin_amdgcn_perm(ps, second, sel);
  return Codes24{{l[0], __builtin_amdgcn_perm(l[1], g01, 0x05040100u), __builtin_amdgcn_perm(g01, l[1], 0x07060302u), l[2],
                  __builtin_amdgcn_perm(l[3], g23, 0x05040100u), __builtin_amdgcn_perm(g23, l[3], 0x07060302u)}};
}

typedef __bf16 bf16x32 __attribute__((ext_vector_type(32)));
typedef uint32_t u32x6 __attribute__((ext_vector_type(6)));

// FP6-E3M2: the 32-wide hardware converters (v_cvt_scalef32_pk32_bf6_bf16 and back) take
// a lane's whole tile at once, round to nearest even with gradual underflow and saturate
// at 28 * X (checked against the cast's definition on every finite BF16 input at several
// scales).
template <bool FULL>
__device__ __forceinline__ u32x6 tile_codes_fp6(const Tile& t, const BlockScale& b) {
  uint32_t pk[16];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int k = 0; k < 4; ++k) pk[4 * i + k] = !FULL && t.nv[i] == 0 ? 0 : t.v[i][k];
  bf16x32 v;
  __builtin_memcpy(&v, pk, 64);
  return __builtin_amdgcn_cvt_scalef32_pk32_bf6_bf16(v, b.x_scale);
}

// The forward pass on one wavefront tile, in three phases.
//
// tile_scale: a = max|w| of the lane's block (exact), the block's scale and cast constants.
//   bt: this lane's block parameter, which the caller fetches with the tile.
//   STORE: the block's writer lane stores scale (and, MX, the E8M0 block scale) here; off, the caller does.
// tile_sum: noise times scale added, rounded to BF16 (the tile's registers are overwritten with the sums).
//   n: the noise of the tile (draw_noise).
// tile_store: cast, store.
//   STREAM: see load16.
//   MX: the output is element codes (p1, row stride ldc) and E8M0 block scales (p4) instead of the BF16 container.
//   BASIS: kBasisBits is the method's noise (Sec. 3.4); the other two are the comparison bases (no MX form).
//   USE_HW: FP8-E4M3 through the hardware converters (the caller has shown that no block of the wavefront can
//   overflow); off, the arithmetic cast.  Same bits either way where both apply.
// No phase branches when FULL and !STORE, so a caller that works on several tiles at once gets straight-line
// code it can interleave.
template <int FMT, bool FULL, bool MX, bool STORE>
__device__ __forceinline__ BlockScale tile_scale(const TileDesc& d, Tile& t, uint32_t by, uint32_t col_base, uint32_t lane,
                                                 float bt) {
  const uint32_t gc = lane & 7, r0 = lane >> 3;
  const uint32_t nbc = (d.cols + 31) >> 5;
  const size_t blk0 = (size_t)by * nbc + (col_base >> 5);   // of the left block
  if (!FULL) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (t.nv[i] < 8) t.v[i] = mask_group(t.v[i], t.nv[i]);  // elements past cols do not exist
  }
  // ---- a = max_{b_l}|w| on the magnitude bits (exact) ----
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) m = absmax_pk(t.v[i], m);
  m = max(m & 0xFFFFu, m >> 16);
  const uint32_t a16 = block_max_u32(m);
  // ---- per-block scale ----
  const bool block_exists = FULL || (col_base >> 5) + (gc >> 2) < nbc;
  // Eq. 11 (the product and the sum rounded separately); identity for a plain b_t
  const float btv = __fadd_rn(d.b_target, __fmul_rn(bt, d.b_delta));
  BlockScale b = block_scale(a16, btv);
  if (FMT == 1) cast_constants<8, -6>(a16, b);
  if (FMT == 2) cast_constants<4, -2>(a16, b);
  if (STORE && block_exists && (gc & 3) == 0 && r0 == 0) {
    *at_byte(global_ptr<float>(d.p3) + blk0, gc) = b.s32;   // gc is 0 or 4 here
    // shared exponent of the block: biased exponent of X; X = 1 for an all-zero block
    if (MX) *at_byte(global_ptr<uint8_t>(d.p4) + blk0, gc >> 2) = a16 ? (uint8_t)(__float_as_uint(b.x_scale) >> 23) : (uint8_t)127;
  }
  return b;
}

template <bool FULL, int BASIS>
__device__ __forceinline__ void tile_sum(Tile& t, const BlockScale& b, const TileNoise<BASIS>& n) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (!FULL && t.rows <= 8 * i) continue;   // uniform
    const u32x4 w = t.v[i];
    uint32_t pk[4];
    if constexpr (BASIS == kBasisBits) {
      const GroupR g = group_r(n.x[i]);
      pk[0] = sampled_pair<0>(w[0], g, b);
      pk[1] = sampled_pair<1>(w[1], g, b);
      pk[2] = sampled_pair<2>(w[2], g, b);
      pk[3] = sampled_pair<3>(w[3], g, b);
    } else {
      sampled_group_basis<BASIS>(w, n.x[i], b, pk);
    }
    t.v[i] = u32x4{pk[0], pk[1], pk[2], pk[3]};
  }
}

template <int FMT, bool FULL, int STREAM, bool MX, bool USE_HW>
__device__ __forceinline__ void tile_store(const TileDesc& d, const Tile& t, const BlockScale& b, uint32_t by, uint32_t col_base,
                                           uint32_t lane) {
  static_assert(!USE_HW || FMT == 1, "hardware converters by choice exist for FP8-E4M3 only");
  const uint32_t row_base = by * 32;
  const uint32_t gc = lane & 7, r0 = lane >> 3;
  const uint32_t col = col_base + gc * 8;
  GWS_GLOBAL uint16_t* __restrict__ w_hat = global_ptr<uint16_t>(d.p1);
  const uint32_t off = lane_offset(d.ld, lane);   // full tiles
  auto store_group = [&](int i, const u32x4& o) {
    if (FULL) store16<STREAM>(at_byte(w_hat + ((size_t)(row_base + 8 * i) * d.ld + col_base), off), o);
    else if (t.nv[i] == 8) store16<STREAM>(w_hat + (size_t)(row_base + r0 + 8 * i) * d.ld + col, o);
    else store_partial(w_hat + (size_t)(row_base + r0 + 8 * i) * d.ld + col, o, t.nv[i]);
  };
  if constexpr (FMT != 2) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (!FULL && t.nv[i] == 0) continue;
      const uint32_t pk[4] = {t.v[i][0], t.v[i][1], t.v[i][2], t.v[i][3]};
      if constexpr (MX) {
        const MxCodes c = mx_fp8_codes(pk, b, USE_HW);
        if (FULL) store_codes<FMT, STREAM>(at_byte(global_ptr<uint8_t>(d.p1) + ((size_t)(row_base + 8 * i) * d.ldc + col_base), r0 * d.ldc + gc * 8), 0, c, 8);
        else store_codes<FMT, STREAM>(global_ptr<uint8_t>(d.p1) + (size_t)(row_base + r0 + 8 * i) * d.ldc, col, c, t.nv[i]);
      } else {
        i16x2 chain = {0, 0};
        store_group(i, u32x4{cast_pair<FMT>(pk[0], b, USE_HW, chain), cast_pair<FMT>(pk[1], b, USE_HW, chain),
                             cast_pair<FMT>(pk[2], b, USE_HW, chain), cast_pair<FMT>(pk[3], b, USE_HW, chain)});
      }
      }
  } else {
    const u32x6 c = tile_codes_fp6<FULL>(t, b);
    if (MX && FULL && (((uint32_t)(uintptr_t)d.p1 | d.ldc) & 3) == 0) {   // uniform
      const uint32_t cw[6] = {c[0], c[1], c[2], c[3], c[4], c[5]};
      const Codes24 q = codes_fp6_quad(lane, cw);
      GWS_GLOBAL uint8_t* dst = at_byte(global_ptr<uint8_t>(d.p1) + (size_t)row_base * d.ldc + (col_base >> 3) * 6, (r0 + 8 * (lane & 3)) * d.ldc + (lane & 4) * 6);
      typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));
      typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
      typedef uint32_t u32x2a4 __attribute__((ext_vector_type(2), aligned(4)));
      *(GWS_GLOBAL u32x4a4*)dst = u32x4{q.w[0], q.w[1], q.w[2], q.w[3]};
      *(GWS_GLOBAL u32x2a4*)(dst + 16) = u32x2{q.w[4], q.w[5]};
    } else if constexpr (MX) {
      // element k of the lane's 32 sits in bits [6k, 6k + 6): 48 bits per group
      const MxCodes gc4[4] = {{c[0], c[1] & 0xFFFFu},
                              {(c[1] >> 16) | (c[2] << 16), c[2] >> 16},
                              {c[3], c[4] & 0xFFFFu},
                              {(c[4] >> 16) | (c[5] << 16), c[5] >> 16}};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (!FULL && t.nv[i] == 0) continue;
        const uint32_t row = row_base + r0 + 8 * i;
        store_codes<FMT, STREAM>(global_ptr<uint8_t>(d.p1) + (size_t)row * d.ldc, col, gc4[i], FULL ? 8 : t.nv[i]);
      }
    } else {
      const bf16x32 q = __builtin_amdgcn_cvt_scalef32_pk32_bf16_bf6(c, b.x_scale);
      uint32_t o[16];
      __builtin_memcpy(o, &q, 64);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (!FULL && t.nv[i] == 0) continue;
        store_group(i, u32x4{o[4 * i], o[4 * i + 1], o[4 * i + 2], o[4 * i + 3]});
      }
    }
  }
}

// The phases for one tile; FP8-E4M3 takes the hardware converters only if neither block of this wavefront can
// overflow (they give NaN where the cast saturates).
template <int FMT, bool FULL, int STREAM = kStreamAll, bool MX = false, int BASIS = kBasisBits>
__device__ __forceinline__ void fwd_tile(const TileDesc& d, Tile& t, const TileNoise<BASIS>& n, uint32_t by, uint32_t col_base,
                                         uint32_t lane, float bt) {
  static_assert(BASIS == kBasisBits || !MX, "the comparison bases have no MX output");
  const BlockScale b = tile_scale<FMT, FULL, MX, true>(d, t, by, col_base, lane, bt);
  tile_sum<FULL, BASIS>(t, b, n);
  if constexpr (FMT == 1) {
    if (__builtin_amdgcn_ballot_w64(!b.hw_safe) == 0) tile_store<FMT, FULL, STREAM, MX, true>(d, t, b, by, col_base, lane);
    else tile_store<FMT, FULL, STREAM, MX, false>(d, t, b, by, col_base, lane);
  } else {
    tile_store<FMT, FULL, STREAM, MX, false>(d, t, b, by, col_base, lane);
  }
}

}  // namespace gws
