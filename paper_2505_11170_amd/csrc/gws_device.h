// Device-side building blocks of the GaussWS kernels (gfx950 only).
// Internal to csrc/: not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gws {

// Pointers into global memory, typed as such: the accesses through them are global (not
// flat) instructions whatever the pointer's provenance.
#define GWS_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ GWS_GLOBAL T* global_ptr(const void* p) {
  return (GWS_GLOBAL T*)(uintptr_t)p;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): the counter-based bit source named in
// the paper's Sec. 3.4.  One call yields the 128 bits of a group of 8
// row-contiguous elements (16 bits per element).  Counter = (column group,
// row, step lo, step hi), key = per-tensor seed.  Calls of one lane that differ
// only in the row share the multiplies of the first rounds (the compiler folds
// them once the calls are inlined side by side).
// ---------------------------------------------------------------------------
struct Philox4 {
  uint32_t x0, x1, x2, x3;
};

__device__ __forceinline__ Philox4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                 uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
    const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return Philox4{c0, c1, c2, c3};
}

// The four Philox calls of a lane (rows row[0..3], one column group) with the work of the first three rounds
// that does not depend on all of the counter done once.  With counter (cg, row, step_lo, step_hi):
//   round 0: M1 * step_lo is uniform; M0 * cg depends on the column group only; the new c0 on the row only;
//   round 1: M0 * c0 depends on the row only (PhiloxRows: kept across the column tiles a wavefront walks),
//            M1 * c2 on the column group only;
//   round 2: M0 * c0 depends on the column group only; from M1 * c2 on everything depends on both.
// 63 multiplies per four calls instead of 80 (67 with the row part), same bits as philox4x32_10:
// philox_rows once per wavefront, philox_cols once per tile, philox_tiles for the calls.
struct PhiloxRows {
  uint32_t hi[4], lo[4];   // M0 * (c0 after round 0) for the four rows
};

__device__ __forceinline__ PhiloxRows philox_rows(const uint32_t (&row)[4], uint32_t step_lo, uint32_t k0) {
  const uint32_t base = (uint32_t)(((uint64_t)0xCD9E8D57u * step_lo) >> 32) ^ k0;   // uniform
  PhiloxRows r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint64_t d = (uint64_t)0xD2511F53u * (base ^ row[i]);
    r.hi[i] = (uint32_t)(d >> 32);
    r.lo[i] = (uint32_t)d;
  }
  return r;
}

// The column-group share of the first three rounds (four registers), then one call per row.
struct PhiloxCols {
  uint32_t c3_1, c1_2, hi_f, c3_3;
};

__device__ __forceinline__ PhiloxCols philox_cols(uint32_t cg, uint32_t step_lo, uint32_t step_hi, uint32_t k0, uint32_t k1) {
  constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u;
  const uint32_t c1_1 = (uint32_t)((uint64_t)M1 * step_lo);                      // round 0, uniform
  const uint64_t b = (uint64_t)M0 * cg;                                          // round 0, column group
  const uint32_t c2_1 = xor3((uint32_t)(b >> 32), step_hi, k1);
  const uint64_t c = (uint64_t)M1 * c2_1;                                        // round 1, column group
  const uint32_t c0_2 = xor3((uint32_t)(c >> 32), c1_1, k0 + W0);
  const uint64_t f = (uint64_t)M0 * c0_2;                                        // round 2, column group
  return PhiloxCols{(uint32_t)b, (uint32_t)c, (uint32_t)(f >> 32), (uint32_t)f};
}

// A value that is the same in all lanes, in a vector register.  On gfx950 the 32-bit adds, right shifts, bitwise operations
// and fp32 multiply-adds issue in two cycles with operands in vector registers (or constants of the instruction) and in four
// as soon as one of them is a scalar register.
__device__ __forceinline__ uint32_t in_vgpr(uint32_t v) {
  asm("" : "+v"(v));
  return v;
}

// The R T calls of T tiles (column groups pc[0 .. T-1]; the same R rows, four or the first two) advanced round by round
// together: independent multiplies keep the vector ALU fed where few wavefronts share it, and the round keys, in vector
// registers, are stepped once for all calls.
template <int T, int R>
__device__ __forceinline__ void philox_tiles(const PhiloxCols (&pc)[T], const PhiloxRows& rp, uint32_t k0, uint32_t k1,
                                             Philox4 (&out)[T][R]) {
  constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
  constexpr int N = R * T;
  uint32_t c0[N], c1[N], c2[N], c3[N];
  uint32_t ka = in_vgpr(k0 + 2 * W0), kb = in_vgpr(k1 + W1);
  uint64_t e[N];
#pragma unroll
  for (int k = 0; k < N; ++k) e[k] = (uint64_t)M1 * xor3(rp.hi[k % R], pc[k / R].c3_1, kb);   // rounds 1 and 2
  kb += W1;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    c0[k] = xor3((uint32_t)(e[k] >> 32), pc[k / R].c1_2, ka);
    c1[k] = (uint32_t)e[k];
    c2[k] = xor3(pc[k / R].hi_f, rp.lo[k % R], kb);
    c3[k] = pc[k / R].c3_3;
  }
#pragma unroll
  for (int r = 3; r < 10; ++r) {
    ka += W0;
    kb += W1;
    uint64_t p0[N], p1[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      p0[k] = (uint64_t)M0 * c0[k];
      p1[k] = (uint64_t)M1 * c2[k];
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
      c0[k] = xor3((uint32_t)(p1[k] >> 32), c1[k], ka);
      c2[k] = xor3((uint32_t)(p0[k] >> 32), c3[k], kb);
      c1[k] = (uint32_t)p1[k];
      c3[k] = (uint32_t)p0[k];
    }
  }
#pragma unroll
  for (int k = 0; k < N; ++k) out[k / R][k % R] = Philox4{c0[k], c1[k], c2[k], c3[k]};
}

// ---------------------------------------------------------------------------
// 128 random bits -> the noise of eight elements (paper Sec. 3.4, Eq. 9 and
// Eq. 10), evaluated for all eight at once on nibble planes.  Each element owns
// one nibble position in each of the four words (16 independent bits):
//   |R| = 2 : (b|b) & (8 bits all set)              -> 3/4 * 2^-8
//   |R| = 1 : (b|b) & (b|b) & b, unless |R| = 2     -> (3/4)^2 * 2^-1 * (1 - P(|R|=2))
//   sign    : 1 bit (bit 3 of the x3 nibble; x3 is kept as is)
// Element k of a group owns nibble (k>>1) + 4*(k&1): the two BF16 values of a
// 32-bit register take their bits from the low and the high half of each word.
// ---------------------------------------------------------------------------
//
// The result is 2R of the eight elements as FP4-E2M1 numbers, one per nibble: 0, +-2 (code 4), +-4 (code 6), the sign bit of a
// zero kept; the hardware converters make fp32 or BF16 of them.  Written with what issues in two cycles (see in_vgpr; left
// shifts, three-operand shifts and byte permutes take four): 15 instructions, about 38 cycles a wavefront, where separate
// planes and their way into FP8 bytes took 21 and 63.
struct Noise {
  uint32_t c;  // nibble element_nibble(k): E2M1 code of 2R of element k
};

__device__ __forceinline__ Noise noise_codes(const Philox4& x) {
  const uint32_t k4 = in_vgpr(0x44444444u), kc = in_vgpr(0xCCCCCCCCu);
  // (v & 7) + 1 carries into bit 3 where the low three bits are set, (v & 3) + 3 into bit 2 where one of the low two is
  const uint32_t a = x.x0 & x.x1;
  const uint32_t all8 = (((a & 0x77777777u) + 0x11111111u) & a) >> 1;                    // bit 2: all 8 bits set
  const uint32_t b01 = (x.x2 & 0x33333333u) + 0x33333333u;                               // bit 2: b|b (A)
  const uint32_t d = (x.x3 & 0x33333333u) + 0x33333333u;                                 // bit 2: b|b (D)
  const uint32_t cd = __builtin_amdgcn_bitop3_b32(x.x2, x.x2 >> 1, d, 0xA8);             // bit 2: (b|b) & (b|b)  (C & D)
  const uint32_t m2 = __builtin_amdgcn_bitop3_b32(all8, b01, k4, 0x80);                  // bit 2: |R| = 2, the others clear
  const uint32_t nz = __builtin_amdgcn_bitop3_b32(cd, x.x3, m2, 0xEA);                   // bit 2: R != 0
  const uint32_t snz = __builtin_amdgcn_bitop3_b32(nz, k4, x.x3, 0xE2);                  // bit 2 from nz, the others from x3
  return Noise{(uint32_t)__builtin_amdgcn_bitop3_b32(snz, kc, m2 >> 1, 0xEA)};                     // sign, nz, m2, 0
}

__device__ __forceinline__ Noise group_noise(uint32_t cg, uint32_t row, uint32_t step_lo, uint32_t step_hi,
                                             uint32_t seed_lo, uint32_t seed_hi) {
  return noise_codes(philox4x32_10(cg, row, step_lo, step_hi, seed_lo, seed_hi));
}

// Nibble position of element k of a group.
__host__ __device__ constexpr int element_nibble(int k) { return (k >> 1) + 4 * (k & 1); }

// The packed output format of Sec. 3.4: 4-bit sign-magnitude codes, element k
// in bits 4k..4k+3 (only the noise dump needs it).
__device__ __forceinline__ uint32_t packed_codes(const Noise& n) {
  const uint32_t c = (n.c & 0x88888888u) | (((n.c >> 2) & 0x11111111u) + ((n.c >> 1) & 0x11111111u));  // per nibble: sign<<3 | |R|
  uint32_t out = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) out |= ((c >> (4 * element_nibble(k))) & 0xFu) << (4 * k);
  return out;
}

// ---------------------------------------------------------------------------
// 2^t as one fixed fp32 function (for the block scale 2^(1-b_t) of Eq. 3 with a
// real-valued b_t): n = rint(t), f = t - n, degree-6 Horner polynomial in f with
// fused multiply-adds, scaled by 2^n.  Exact for integer t.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float exp2_fixed(float t) {
  const float n = rintf(t);
  const float f = t - n;
  float p = __uint_as_float(0x39222002u);
  p = __fmaf_rn(p, f, __uint_as_float(0x3AAF844Bu));
  p = __fmaf_rn(p, f, __uint_as_float(0x3C1D950Eu));
  p = __fmaf_rn(p, f, __uint_as_float(0x3D6357B6u));
  p = __fmaf_rn(p, f, __uint_as_float(0x3E75FDF0u));
  p = __fmaf_rn(p, f, __uint_as_float(0x3F317218u));
  p = __fmaf_rn(p, f, 1.0f);
  return ldexpf(p, (int)n);
}

// fp32 -> BF16 bits, round to nearest even (finite values).
__device__ __forceinline__ uint32_t bf16_rne_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}

// Two fp32 -> packed BF16 pair (lo in bits 0..15), round to nearest even, in
// hardware (v_cvt_pk_bf16_f32; identical to the integer rounding above for
// every finite input).
__device__ __forceinline__ uint32_t pack_bf16_rne(float lo, float hi) {
  bf16x2 p = {(__bf16)lo, (__bf16)hi};
  uint32_t u;
  __builtin_memcpy(&u, &p, 4);
  return u;
}

// ---------------------------------------------------------------------------
// Per-block constants of the forward pass.
// ---------------------------------------------------------------------------
struct BlockScale {
  float s32;        // max|w| * 2^(1-b_t), unrounded fp32 (stored; Eq. 4 reuses it)
  uint32_t s_bits;  // bf16_rne(s32) as fp32 bits (sign clear): the step of the PQN
  float x_scale;    // cast: X = 2^(Ea + 1 - EMAX) as fp32
  uint32_t emin_b;  // cast: fp32 exponent field (<<23) of the lowest normal binade of X*format
  uint32_t max_b;   // cast: fp32 bits of max*X (saturation bound)
  bool hw_safe;     // cast: no element of the block can exceed max*X (a + 2s <= max*X)
};

template <int EMAX, int EMIN>
__device__ __forceinline__ void cast_constants(uint32_t a16, BlockScale& b) {
  // Ea = floor(log2 max|w|) from the BF16 exponent field; clamped so that every
  // constant below is a normal fp32 (blocks with max|w| < 2^-100 are outside the
  // supported domain and only have to stay in bounds).
  int ef = (int)(a16 >> 7);
  ef = ef < 27 ? 27 : ef;
  b.x_scale = __uint_as_float((uint32_t)(ef + 1 - EMAX) << 23);
  b.emin_b = (uint32_t)(ef + 1 - EMAX + EMIN) << 23;  // lowest normal = X * 2^EMIN
  b.max_b = ((uint32_t)(ef + 1) << 23) | 0x00600000u; // 1.75 * 2^EMAX * X = 1.75 * 2^(Ea+1)
  const float a = __uint_as_float(a16 << 16);
  b.hw_safe = a + 2.0f * __uint_as_float(b.s_bits) <= __uint_as_float(b.max_b);
}

__device__ __forceinline__ BlockScale block_scale(uint32_t a16, float bt) {
  BlockScale b;
  const float a = __uint_as_float(a16 << 16);
  const float p = exp2_fixed(1.0f - bt);
  b.s32 = a * p;
  b.s_bits = bf16_rne_bits(b.s32) << 16;
  b.x_scale = 1.0f;
  b.emin_b = 0;
  b.max_b = 0;
  b.hw_safe = true;
  return b;
}

// ---------------------------------------------------------------------------
// Block-scaled fp_{e,m} cast (paper Sec. 3.3) of a BF16 value held in fp32, in
// plain arithmetic: round to nearest even onto the grid of spacing
// 2^(max(e_v, emin) - M) by adding and subtracting 2^(23 - M) times that binade
// (the fp32 adder performs the rounding), then saturate and restore the sign.
// ---------------------------------------------------------------------------
template <int M>
__device__ __forceinline__ uint32_t cast_scaled_bits(uint32_t h16, const BlockScale& b) {
  const uint32_t u = h16 << 16;
  const uint32_t au = u & 0x7FFFFFFFu;
  uint32_t eb = au & 0x7F800000u;
  eb = eb > b.emin_b ? eb : b.emin_b;
  const float c = __uint_as_float(eb + ((uint32_t)(23 - M) << 23));
  float r = (__uint_as_float(au) + c) - c;
  r = fminf(r, __uint_as_float(b.max_b));
  return (__float_as_uint(r) | (u & 0x80000000u)) >> 16;
}

// Cast of a packed BF16 pair.  FP8-E4M3 goes through the hardware converters
// (v_cvt_scalef32_pk_fp8_bf16 and back: round to nearest even, gradual
// underflow, division by the power-of-two scale), which produce NaN instead of
// saturating, so they are used only where the block cannot overflow.  FP6-E3M2 is
// cast in arithmetic here; this per-pair form serves the GEMM kernel's operand
// path, while the tile code converts FP6 with the 32-wide hardware converters.
template <int FMT>
__device__ __forceinline__ uint32_t cast_pair(uint32_t pk, const BlockScale& b, bool hw, i16x2& chain) {
  if (FMT == 0) return pk;
  if (FMT == 1 && hw) {
    bf16x2 v;
    __builtin_memcpy(&v, &pk, 4);
    // the converter writes one 16-bit half of its destination and keeps the other:
    // chaining the previous result as "old" avoids a register clear per call
    chain = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(chain, v, b.x_scale, false);
    uint32_t cu;
    __builtin_memcpy(&cu, &chain, 4);
    const bf16x2 r = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(cu, b.x_scale, false);
    uint32_t ru;
    __builtin_memcpy(&ru, &r, 4);
    return ru;
  }
  constexpr int M = (FMT == 1) ? 3 : 2;
  return cast_scaled_bits<M>(pk & 0xFFFFu, b) | (cast_scaled_bits<M>(pk >> 16, b) << 16);
}

// Byte i of x as fp32 (v_cvt_f32_ubyte<i>).
template <int I>
__device__ __forceinline__ float byte_to_f32(uint32_t x) {
  return (float)((x >> (8 * I)) & 0xFFu);
}

// ---------------------------------------------------------------------------
// Eq. 3 + cast on one 16-byte group (8 BF16 in 4 registers).  R is sign-magnitude: |R| * s is
// exact and the sign is kept on a zero (R = -0 gives -0.0); the fp32 fused multiply-add
// followed by one RNE to BF16 equals the exact BF16 sum.
// ---------------------------------------------------------------------------
struct GroupR {
  float r[8];  // R of element k as fp32
};

// Byte d of the codes holds the elements of nibbles 2 d and 2 d + 1: 0 and 2, 4 and 6, 1 and 3, 5 and 7.
__device__ __forceinline__ GroupR group_r(const Noise& n) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  const f32x2 n02 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(n.c, 0.5f, 0), n46 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(n.c, 0.5f, 1);
  const f32x2 n13 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(n.c, 0.5f, 2), n57 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(n.c, 0.5f, 3);
  return GroupR{{n02[0], n13[0], n02[1], n13[1], n46[0], n57[0], n46[1], n57[1]}};
}

// bf16_rne(w + R * s) for elements 2d and 2d+1 of a group (register d), packed.
template <int D>
__device__ __forceinline__ uint32_t sampled_pair(uint32_t wd, const GroupR& g, const BlockScale& b) {
  const float s = __uint_as_float(b.s_bits);
  const float w_lo = __uint_as_float(wd << 16), w_hi = __uint_as_float(wd & 0xFFFF0000u);
  return pack_bf16_rne(__fmaf_rn(g.r[2 * D], s, w_lo), __fmaf_rn(g.r[2 * D + 1], s, w_hi));
}

template <int FMT>
__device__ __forceinline__ u32x4 sample_group(const u32x4 w, const Noise& n, const BlockScale& b, bool hw) {
  const GroupR g = group_r(n);
  i16x2 chain = {0, 0};
  u32x4 out;
  out[0] = cast_pair<FMT>(sampled_pair<0>(w[0], g, b), b, hw, chain);
  out[1] = cast_pair<FMT>(sampled_pair<1>(w[1], g, b), b, hw, chain);
  out[2] = cast_pair<FMT>(sampled_pair<2>(w[2], g, b), b, hw, chain);
  out[3] = cast_pair<FMT>(sampled_pair<3>(w[3], g, b), b, hw, chain);
  return out;
}

// ---------------------------------------------------------------------------
// The same group as microscaling element codes (OCP MX: FP8 E4M3 with bias 7,
// FP6 E3M2 with bias 3) of q / X, X the block's power-of-two scale.
// ---------------------------------------------------------------------------
struct MxCodes {
  uint32_t lo, hi;  // FP8: 8 code bytes.  FP6: 8 codes of 6 bits, element k in bits [6k, 6k+6) of hi:lo
};

// Code of a BF16 value under the block scale, in plain arithmetic.  Adding
// 2^(23 - M) times the binade (the binade of the value, or the lowest normal one
// of X * format below it) makes the fp32 adder round the value to nearest even
// onto the format's grid and leaves the count of grid steps, k, in the low
// mantissa bits; the code is that count on top of the binade's first code.
template <int M, int EBITS, uint32_t MAXCODE>
__device__ __forceinline__ uint32_t encode_scaled(uint32_t h16, const BlockScale& b) {
  const uint32_t u = h16 << 16;
  const uint32_t au = u & 0x7FFFFFFFu;
  uint32_t eb = au & 0x7F800000u;
  eb = eb > b.emin_b ? eb : b.emin_b;
  const uint32_t cb = eb + ((uint32_t)(23 - M) << 23);
  const float t = __uint_as_float(au) + __uint_as_float(cb);
  const uint32_t k = __float_as_uint(t) - cb;            // 0 .. 2^(M+1)
  uint32_t code = ((eb - b.emin_b) >> (23 - M)) + k;     // (E - 1) << M, plus k
  code = code < MAXCODE ? code : MAXCODE;                // saturate at the largest finite code
  return code | ((u >> 31) << (M + EBITS));
}

// FP8-E4M3 codes of one group's four packed BF16 sums.  (FP6-E3M2 codes come from the 32-wide converter, a lane's
// whole tile at a time: see tile_store.)
__device__ __forceinline__ MxCodes mx_fp8_codes(const uint32_t (&pk)[4], const BlockScale& b, bool hw) {
  MxCodes c;
  if (hw) {
    // hardware converter: rounds to nearest even under the scale; each call fills one
    // 16-bit half of its destination register
    bf16x2 v[4];
    __builtin_memcpy(v, pk, 16);
    i16x2 a = {0, 0}, h = {0, 0};
    a = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(a, v[0], b.x_scale, false);
    a = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(a, v[1], b.x_scale, true);
    h = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(h, v[2], b.x_scale, false);
    h = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(h, v[3], b.x_scale, true);
    __builtin_memcpy(&c.lo, &a, 4);
    __builtin_memcpy(&c.hi, &h, 4);
    return c;
  }
  // the block can exceed 448 X, where the converter would give NaN: saturating arithmetic form
  uint32_t e[8];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    e[2 * d] = encode_scaled<3, 4, 0x7Eu>(pk[d] & 0xFFFFu, b);
    e[2 * d + 1] = encode_scaled<3, 4, 0x7Eu>(pk[d] >> 16, b);
  }
  c.lo = e[0] | (e[1] << 8) | (e[2] << 16) | (e[3] << 24);
  c.hi = e[4] | (e[5] << 8) | (e[6] << 16) | (e[7] << 24);
  return c;
}

// ---------------------------------------------------------------------------
// Comparison noise bases (paper Sec. 4): the same pipeline with R drawn as a BF16
// U(-0.5, 0.5) value (the paper's "DiffQ" extension) or as the exact rounded normal
// round(N(0,1) / 2) from a Box-Muller transform (the "bm" baseline of its forward
// unit benchmark).  Both take the group's Philox call as it is; only the map from
// the 128 bits to the eight R differs.
//   uniform:    element k owns byte k % 4 of word k / 4; R = (2 byte - 255) / 512, one of the
//               256 midpoints of a 1/256 grid on (-0.5, 0.5), each a BF16 value.  R * s is not
//               exact here and is rounded to BF16 before the add (the BF16 operator of Sec. 3.3).
//   Box-Muller: the pair of elements (2d, 2d + 1) owns word d; u1 = (low half + 0.5) / 2^16,
//               u2 = (high half + 0.5) / 2^16, z = sqrt(-2 ln u1) (cos, sin)(2 pi u2),
//               R = rint(z / 2).  Floating point decides an integer here, so the fp32 operations
//               and their order are fixed (no contraction, correctly rounded square root).
// ---------------------------------------------------------------------------
constexpr int kBasisBits = 0, kBasisUniform = 1, kBasisBoxMuller = 2;

// R of elements 2d and 2d + 1 of a group as fp32 (exact), uniform basis.
template <int D>
__device__ __forceinline__ void uniform_pair(const Philox4& x, float& r_lo, float& r_hi) {
  const uint32_t word = (D >> 1) ? x.x1 : x.x0;   // elements 0..3 in x0, 4..7 in x1
  const float step = __uint_as_float(0x3B800000u), off = __uint_as_float(0xBEFF0000u);   // 2^-8, -255/512
  r_lo = __fmaf_rn(byte_to_f32<2 * (D & 1)>(word), step, off);
  r_hi = __fmaf_rn(byte_to_f32<2 * (D & 1) + 1>(word), step, off);
}

// ln(u) for u = (k + 0.5) / 2^16: u = m 2^e with m in [1/sqrt2, sqrt2), ln u = e ln2 + f P(f), f = m - 1,
// P of degree 8 evaluated by Horner's rule with fused multiply-adds.
__device__ __forceinline__ float bm_log(float u) {
  const uint32_t ub = __float_as_uint(u);
  int e = (int)(ub >> 23) - 127;
  float m = __uint_as_float((ub & 0x007FFFFFu) | 0x3F800000u);
  if (m > __uint_as_float(0x3FB504F3u)) {
    m = __fmul_rn(m, 0.5f);
    e += 1;
  }
  const float f = __fsub_rn(m, 1.0f);
  float p = __uint_as_float(0x3DB31375u);
  p = __fmaf_rn(p, f, __uint_as_float(0xBE13394Fu));
  p = __fmaf_rn(p, f, __uint_as_float(0x3E191428u));
  p = __fmaf_rn(p, f, __uint_as_float(0xBE2994DFu));
  p = __fmaf_rn(p, f, __uint_as_float(0x3E4C5C05u));
  p = __fmaf_rn(p, f, __uint_as_float(0xBE8002D3u));
  p = __fmaf_rn(p, f, __uint_as_float(0x3EAAABC8u));
  p = __fmaf_rn(p, f, __uint_as_float(0xBEFFFFFCu));
  p = __fmaf_rn(p, f, 1.0f);
  return __fmaf_rn((float)e, __uint_as_float(0x3F317218u), __fmul_rn(p, f));
}

// R of the two elements that own `word`, as fp32 in {-2, -1, -0, 0, 1, 2}.
__device__ __forceinline__ void box_muller_pair(uint32_t word, float& r_lo, float& r_hi) {
  const float u1 = __fmul_rn(__fadd_rn((float)(word & 0xFFFFu), 0.5f), __uint_as_float(0x37800000u));
  const float L = __fmul_rn(-2.0f, bm_log(u1));
  const float r = __builtin_sqrtf(L);   // correctly rounded
  const uint32_t hi = word >> 16, q = hi >> 14, j = hi & 0x3FFFu;
  // angle = q pi/2 + pi/4 + t, t = (2 j + 1 - 16384) fl(pi / 65536) in (-pi/4, pi/4)
  const float t = __fmul_rn((float)(2 * (int)j + 1 - 16384), __uint_as_float(0x38490FDBu));
  const float t2 = __fmul_rn(t, t);
  float sp = __uint_as_float(0xB94D6501u);
  sp = __fmaf_rn(sp, t2, __uint_as_float(0x3C088615u));
  sp = __fmaf_rn(sp, t2, __uint_as_float(0xBE2AAAA9u));
  const float st = __fmaf_rn(__fmul_rn(t, t2), sp, t);
  float cp = __uint_as_float(0x37CD3809u);
  cp = __fmaf_rn(cp, t2, __uint_as_float(0xBAB60706u));
  cp = __fmaf_rn(cp, t2, __uint_as_float(0x3D2AAAA6u));
  cp = __fmaf_rn(cp, t2, __uint_as_float(0xBF000000u));
  const float ct = __fmaf_rn(t2, cp, 1.0f);
  const float h = __uint_as_float(0x3F3504F3u);
  const float c = __fmul_rn(__fsub_rn(ct, st), h), sn = __fmul_rn(__fadd_rn(ct, st), h);
  // q quarter turns: (c, s) -> (-s, c) -> (-c, -s) -> (s, -c); negation is a sign-bit flip
  const uint32_t cb = __float_as_uint(c), sb = __float_as_uint(sn);
  const uint32_t cq = ((q & 1) ? sb : cb) ^ (((q + 1) & 2) << 30);
  const uint32_t sq = ((q & 1) ? cb : sb) ^ ((q & 2) << 30);
  r_lo = __builtin_rintf(__fmul_rn(0.5f, __fmul_rn(r, __uint_as_float(cq))));
  r_hi = __builtin_rintf(__fmul_rn(0.5f, __fmul_rn(r, __uint_as_float(sq))));
}

// The same R for the four pairs of a group, by thresholds instead of by value.  R = rint(z / 2) asks only whether |z|
// exceeds 1 and whether it reaches 3, z^2 = -2 ln u1 cos^2 (sin^2 = 1 - cos^2): one hardware logarithm (base 2) and one
// hardware cosine (of revolutions) a pair say so for all but the words near a threshold.  Each comparison is a multiply-add
// clamped to [0, 1] that is fractional within 2^-15 of the threshold (in units of z^2 / (2 ln 2)); a group with such an
// element in any lane (about one group in a hundred) takes the exact sequence above for all of its pairs.  The hardware
// functions need 2.5 % of that half window, 4.1e-5 of the words lie within it, and over all 2^32 words both ways give the
// same bits (gws_box_muller_check counts all three).  The sign is the quadrant's: the cosine's own, and a bit of the word.
// Bound by the vector ALU: 18 instructions a pair where the exact sequence takes 90, of what issues in two cycles (constants in
// vector registers, no permutes, no left shift, fractions collected as bits): backward of 2048 x 8192 10.3 -> 9.6 us, of 4096 x
// 8192 17.6 -> 16.5 (forward, which its bytes bound, 15.7 -> 15.5 and 24.9 -> 24.3).
// near: its low 21 bits are not all clear if an element lies within a window.
__device__ __forceinline__ void box_muller_pair_fast(uint32_t word, float& r_lo, float& r_hi, uint32_t& near) {
  constexpr float W = 16384.0f, T1 = 0.72134752f, T9 = 6.49212768f;   // 1 / window, 1 / (2 ln 2), 9 / (2 ln 2)
  constexpr uint32_t kMinusW = 0xC6800000u;
  // u1: 2^23 + low half, made (low half + 0.5) / 2^16 by an exact multiply-add.  u2: the high half and the half step as mantissa bits
  // of a number in [1, 2), one revolution more.
  const float u1 = __fmaf_rn(__uint_as_float(__builtin_amdgcn_bitop3_b32(word, in_vgpr(0xFFFFu), in_vgpr(0x4B000000u), 0xEA)), 0x1p-16f, -128.0f + 0x1p-17f);
  const float u2 = __uint_as_float(__builtin_amdgcn_bitop3_b32(word >> 9, in_vgpr(0x007FFF80u), in_vgpr(0x3F800040u), 0xEA));
  const float l2 = __builtin_amdgcn_logf(u1), c = __builtin_amdgcn_cosf(u2);
  const float qc = __fmul_rn(l2, __fmul_rn(c, c)), qs = __fsub_rn(l2, qc);   // -z^2 / (2 ln 2) of the two elements
  const float w = __uint_as_float(in_vgpr(kMinusW));
  auto magnitude = [&](float q) {
    const float m1 = __builtin_amdgcn_fmed3f(__fmaf_rn(q, w, 0.5f - T1 * W), 0.0f, 1.0f);
    const float m9 = __builtin_amdgcn_fmed3f(__fmaf_rn(q, w, 0.5f - T9 * W), 0.0f, 1.0f);
    return __fadd_rn(m1, m9);
  };
  const float mc = magnitude(qc), ms = magnitude(qs);
  // 4, 5 and 6 have no mantissa bits below bit 21
  near = __builtin_amdgcn_bitop3_b32(near, __float_as_uint(__fadd_rn(mc, 4.0f)), __float_as_uint(__fadd_rn(ms, 4.0f)), 0xFE);
  const uint32_t sign = in_vgpr(0x80000000u);
  r_lo = __uint_as_float(__builtin_amdgcn_bitop3_b32(__float_as_uint(c), sign, __float_as_uint(mc), 0xEA));
  r_hi = __uint_as_float(__builtin_amdgcn_bitop3_b32(word, sign, __float_as_uint(ms), 0xEA));
}
constexpr uint32_t kBoxMullerNear = 0x001FFFFFu;

__device__ __forceinline__ void box_muller_group(const Philox4& x, float (&r)[8]) {
  uint32_t near = 0;
  box_muller_pair_fast(x.x0, r[0], r[1], near);
  box_muller_pair_fast(x.x1, r[2], r[3], near);
  box_muller_pair_fast(x.x2, r[4], r[5], near);
  box_muller_pair_fast(x.x3, r[6], r[7], near);
  if (__builtin_amdgcn_ballot_w64((near & kBoxMullerNear) != 0) != 0) {
    box_muller_pair(x.x0, r[0], r[1]);
    box_muller_pair(x.x1, r[2], r[3]);
    box_muller_pair(x.x2, r[4], r[5]);
    box_muller_pair(x.x3, r[6], r[7]);
  }
}

// The eight R of a group under a comparison basis as fp32 (exact).
template <int BASIS>
__device__ __forceinline__ void basis_group(const Philox4& x, float (&r)[8]) {
  if constexpr (BASIS == kBasisUniform) {
    uniform_pair<0>(x, r[0], r[1]);
    uniform_pair<1>(x, r[2], r[3]);
    uniform_pair<2>(x, r[4], r[5]);
    uniform_pair<3>(x, r[6], r[7]);
  } else {
    box_muller_group(x, r);
  }
}

// bf16_rne(w + PQN) for the eight elements of a group under a comparison basis: PQN = bf16_rne(R * s) (exact for the
// integer R of the Box-Muller basis, where the fused multiply-add gives the same bits in one step).
template <int BASIS>
__device__ __forceinline__ void sampled_group_basis(const u32x4 w, const Philox4& x, const BlockScale& b, uint32_t (&pk)[4]) {
  float r[8];
  basis_group<BASIS>(x, r);
  const float s = __uint_as_float(b.s_bits);
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const uint32_t wd = w[d];
    const float w_lo = __uint_as_float(wd << 16), w_hi = __uint_as_float(wd & 0xFFFF0000u);
    if (BASIS == kBasisUniform) {
      const uint32_t pq = pack_bf16_rne(__fmul_rn(r[2 * d], s), __fmul_rn(r[2 * d + 1], s));
      pk[d] = pack_bf16_rne(__fadd_rn(w_lo, __uint_as_float(pq << 16)), __fadd_rn(w_hi, __uint_as_float(pq & 0xFFFF0000u)));
    } else {
      pk[d] = pack_bf16_rne(__fmaf_rn(r[2 * d], s, w_lo), __fmaf_rn(r[2 * d + 1], s, w_hi));
    }
  }
}

// The eight R of a group under a comparison basis as four packed BF16 pairs (every R is a BF16 value: the upper halves).
template <int BASIS>
__device__ __forceinline__ u32x4 basis_group_bf16(const Philox4& x) {
  float r[8];
  basis_group<BASIS>(x, r);
  u32x4 out;
#pragma unroll
  for (int d = 0; d < 4; ++d) out[d] = __builtin_amdgcn_perm(__float_as_uint(r[2 * d + 1]), __float_as_uint(r[2 * d]), 0x07060302u);
  return out;
}

// sum over one group of g .* R under a comparison basis (products exact, fp32 accumulation, fixed order).
template <int BASIS>
__device__ __forceinline__ float dot_group_basis(const u32x4 g, const Philox4& x, float acc) {
  const u32x4 r = basis_group_bf16<BASIS>(x);
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const uint32_t gd = g[d], rd = r[d];
    bf16x2 gv, rv;
    __builtin_memcpy(&gv, &gd, 4);
    __builtin_memcpy(&rv, &rd, 4);
    acc = __builtin_amdgcn_fdot2_f32_bf16(gv, rv, acc, false);
  }
  return acc;
}

// sum over one group of g .* (2R), two elements per v_dot2 (products exact, fp32
// accumulation).  The converter gives 2R in BF16 by pairs of nibbles; byte permutes pair them as the registers of g do.
__device__ __forceinline__ float dot_group_2r(const u32x4 g, const Noise& n, float acc) {
  const bf16x2 b[4] = {__builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(n.c, 1.0f, 0), __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(n.c, 1.0f, 1),
                       __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(n.c, 1.0f, 2), __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(n.c, 1.0f, 3)};
  uint32_t r[4];   // elements 0 and 2, 4 and 6, 1 and 3, 5 and 7
  __builtin_memcpy(r, b, 16);
  const uint32_t pat[4] = {__builtin_amdgcn_perm(r[2], r[0], 0x05040100u), __builtin_amdgcn_perm(r[2], r[0], 0x07060302u),
                           __builtin_amdgcn_perm(r[3], r[1], 0x05040100u), __builtin_amdgcn_perm(r[3], r[1], 0x07060302u)};
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const uint32_t gd = g[d];
    bf16x2 gv, rv;
    __builtin_memcpy(&gv, &gd, 4);
    __builtin_memcpy(&rv, &pat[d], 4);
    acc = __builtin_amdgcn_fdot2_f32_bf16(gv, rv, acc, false);
  }
  return acc;
}

// ---------------------------------------------------------------------------
// Cross-lane reductions over the 32 lanes of a wavefront that share a 32x32
// block.  Lane = 8 * row_in_8 + column_group; a block owns column groups
// {0..3} or {4..7}, so its lanes differ in lane bits 0, 1, 3, 4, 5.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

__device__ __forceinline__ uint32_t block_max_u32(uint32_t v) {
  v = max(v, dpp_u32<0xB1>(v));   // quad_perm [1,0,3,2]: lane ^ 1
  v = max(v, dpp_u32<0x4E>(v));   // quad_perm [2,3,0,1]: lane ^ 2
  v = max(v, dpp_u32<0x128>(v));  // row_ror 8: lane ^ 8 within a row of 16
  v = max(v, (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x401F));  // lane ^ 16
  v = max(v, (uint32_t)__shfl_xor((int)v, 32));
  return v;
}

__device__ __forceinline__ float block_sum_f32(float v) {
  v += __uint_as_float(dpp_u32<0xB1>(__float_as_uint(v)));
  v += __uint_as_float(dpp_u32<0x4E>(__float_as_uint(v)));
  v += __uint_as_float(dpp_u32<0x128>(__float_as_uint(v)));
  v += __uint_as_float((uint32_t)__builtin_amdgcn_ds_swizzle((int)__float_as_uint(v), 0x401F));
  v += __shfl_xor(v, 32);
  return v;
}

// max|w| of a 16-byte group, as BF16 magnitude bits in both halves of a register.
__device__ __forceinline__ uint32_t absmax_pk(const u32x4 w, uint32_t m) {
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const uint32_t a = w[d] & 0x7FFF7FFFu;
    u16x2 x, y;
    __builtin_memcpy(&x, &a, 4);
    __builtin_memcpy(&y, &m, 4);
    const u16x2 z = __builtin_elementwise_max(x, y);
    __builtin_memcpy(&m, &z, 4);
  }
  return m;
}

}  // namespace gws
