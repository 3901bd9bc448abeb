// Launch descriptors shared by the host API and the kernels (internal to csrc/).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gws.h"
#include "gws_device.h"

namespace gws {

constexpr int kThreads = 256;       // 4 wavefronts per workgroup
constexpr int kTileCols = 256;      // a workgroup covers 32 rows x 256 columns
constexpr int kMaxTensorsPerLaunch = 56;

// One tensor as a kernel sees it.  p0..p3 are, for the forward pass,
// (w, w_hat, bt-or-b_i, scale) and, for the backward pass, (g, dw-or-NULL,
// dbt-or-db_i, scale); p4 is the backward pass's b_i (NULL: the gradient asked
// for is dL/db_t itself).  The forward pass with MX output carries the element
// codes in p1 (row stride ldc bytes) and the E8M0 block scales in p4.
// The bitwidth a block uses is b_t = b_target + v * b_delta (paper Eq. 11) with v
// the value read through p2; a plain b_t input is the case b_target = 0,
// b_delta = 1, which leaves every finite value as it is.
struct TileDesc {
  const void* p0;
  void* p1;
  void* p2;
  void* p3;
  void* p4;
  uint32_t rows, cols, ld;
  uint32_t row0, cg0;          // shard origin: row offset, column-group (col0 / 8) offset
  uint32_t seed_lo, seed_hi;
  uint32_t tiles_x;            // workgroups per row of workgroups = ceil(ceil(cols / 256) / tiles_per_wg_x)
  float b_target, b_delta;     // Eq. 11: b_delta = b_init - b_target
  float lambda_m;              // Eq. 12: lambda / (blocks of the layer); backward only
  uint32_t ldc;                // MX output: bytes per row of element codes
  uint32_t first_wg;           // this tensor's first workgroup within the launch (= its tile_begin entry)
  uint32_t tiles_x_inv;        // min(floor(2^32 / tiles_x), 2^32 - 1): division by multiplication in locate()
};
static_assert(sizeof(TileDesc) == 96, "descriptor layout");

// Rows (ld in elements, ldc in bytes) whose full tiles the sampling code addresses with 32-bit lane offsets: 7 rows of elements
// and 31 rows of codes below 2^32 bytes.
constexpr uint32_t kMaxLaneLd = 1u << 27;

// Streaming (non-temporal) or ordinary accesses of the sampling passes (gws_sample_tile.h, load16).
constexpr int kKeep = 0, kStreamReads = 1, kStreamAll = 2;

// Passed by value: lives in the kernel-argument segment (about 5.5 KiB; the segment
// of a gfx950 code object is not limited to 4 KiB).
struct LaunchArgs {
  // First workgroup of every tensor within the launch; entries past n hold 0x7FFFFFFF.
  // Kept apart from the descriptors so a wavefront reads the whole prefix with a few
  // wide scalar loads instead of one dependent load per tensor.
  uint32_t tile_begin[kMaxTensorsPerLaunch];
  TileDesc t[kMaxTensorsPerLaunch];
  uint32_t n;
  uint32_t step_lo, step_hi;
  uint32_t tiles_per_wg;       // consecutive block rows one workgroup covers (>= 1)
  uint32_t tiles_per_wg_x;     // neighbouring 256-column tiles one workgroup covers (>= 1)
};
// The same for one tensor: a hundred bytes instead of five thousand, read in one go.  dealt: the first workgroups, whole rounds of 128,
// of which sixteen neighbouring ones go to one XCD (locate, gws_sample.hip).
struct OneArgs {
  TileDesc t;
  uint32_t step_lo, step_hi;
  uint32_t tiles_per_wg, tiles_per_wg_x;
  uint32_t dealt;
};
// Weights of more than 32 MB (2048 tiles) are dealt out as several are.  Without that rows off the cache lines, and codes, of one such
// weight took up to half as long again: 264 M parameters in rows of 408 FP8 343 us, like this 230, uniform basis 203 M 235, 196, MX-FP8 65 M
// 41.8, 34.9, copying backward with a parametrised bitwidth 270 M 312, 253; MX-FP6 of whole tiles 164 M 73, 70.  Up to 32 MB it goes either way:
// 9.5 M FP8 10.0, 10.4, 8.4 M copying backward 9.5, 10.0, 6.0 M MX-FP8 7.6, 7.2.
inline OneArgs one_of(const LaunchArgs& a, uint32_t n_wg) {
  const uint64_t tiles = (uint64_t)n_wg * a.tiles_per_wg * a.tiles_per_wg_x;
  return OneArgs{a.t[0], a.step_lo, a.step_hi, a.tiles_per_wg, a.tiles_per_wg_x, tiles > 2048 ? n_wg / 128 * 128 : 0};
}
static_assert(sizeof(LaunchArgs) <= 6144, "kernel arguments: keep within the size verified on the device");

// basis: kBasisBits, or a comparison basis (no MX output then); mode: kKeep, kStreamReads or kStreamAll
// variant: any shape (sample_fwd_kernel) with 0 = four, 2 = up to eight wavefronts a SIMD; 1 = whole tiles only, one a workgroup
// (sample_fwd_full_kernel)
int launch_sample_fwd(const LaunchArgs& a, uint32_t n_wg, int fmt, bool mx, int basis, int mode, int variant, hipStream_t stream);
// variant: any shape (sample_bwd_kernel) as above; 1 = whole tiles and aliased dL/dw only (sample_bwd_full_kernel)
int launch_sample_bwd(const LaunchArgs& a, uint32_t n_wg, int basis, int mode, int variant, hipStream_t stream);
int launch_noise_basis(void* out, uint32_t rows, uint32_t ngrp, uint32_t row0, uint32_t cg0, uint64_t seed, uint64_t step,
                       int basis, hipStream_t stream);
int launch_box_muller_check(uint64_t first, uint64_t n, uint64_t* out, hipStream_t stream);
int launch_copy_tiles(const LaunchArgs& a, uint32_t n_wg, hipStream_t stream);
int launch_block_absmax(const LaunchArgs& a, uint32_t n_wg, hipStream_t stream);
int launch_noise_packed(uint32_t* out, uint32_t rows, uint32_t ngrp, uint32_t row0, uint32_t cg0,
                        uint64_t seed, uint64_t step, hipStream_t stream);

// GEMM launchers (gws_linear.hip)
// What only the kernels that sample or reduce Eq. 4 need.
struct GemmSampling {
  const float* bt;
  float* scale;        // may be NULL
  uint16_t* w_hat;     // may be NULL
  uint32_t row0, cg0, seed_lo, seed_hi, step_lo, step_hi;
  float* dbt;          // weight-gradient GEMM only: dL/db_t per block (with scale as input)
};
struct GemmArgs : GemmSampling {
  const uint16_t* x;   // [M x K], ldx
  const uint16_t* w;   // [K x N] or [N x K], ldw
  uint16_t* y;         // [M x N], ldy
  uint32_t M, N, K;
  uint32_t ldx, ldw, ldy;
  uint32_t inv_band, inv_last;   // of the kernel's tile grid (TileGrid), for its numbering of the tiles
};
// The kernels take these one by one: the first sixteen scalar registers' worth of plain arguments is in registers when a
// wavefront starts (the build asks for it), where a structure is fetched from memory first.  With the reciprocals of TileGrid
// in the place of four divisions: 1 x 768 -> 768 2.85 -> 2.44 us, 4 x 5632 -> 2048 (both [N x K]) 6.35 -> 5.9.
#define GWS_GEMM_PARAMS                                                                                                        \
  const uint16_t *px, const uint16_t *pw, uint16_t *py, const uint32_t pM, const uint32_t pN, const uint32_t pK, const uint32_t pldx, \
      const uint32_t pldw, const uint32_t pldy, const uint32_t pinv_band, const uint32_t pinv_last
#define GWS_GEMM_GATHER(sampling) \
  GemmArgs { sampling, px, pw, py, pM, pN, pK, pldx, pldw, pldy, pinv_band, pinv_last }
#define GWS_GEMM_PASS(g) (g).x, (g).w, (g).y, (g).M, (g).N, (g).K, (g).ldx, (g).ldw, (g).ldy, (g).inv_band, (g).inv_last

// n / d by the host's reciprocal min(floor(2^32 / d), 2^32 - 1): the estimate is at most one too small for any 32-bit n (and, for n
// below 2^31, with the reciprocal's lowest bit cleared).
inline uint32_t reciprocal(uint32_t d) {
  const uint64_t inv = ((uint64_t)1 << 32) / d;
  return inv > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)inv;
}
__host__ __device__ __forceinline__ uint32_t divide(uint32_t n, uint32_t d, uint32_t inv) {
  const uint32_t q = (uint32_t)(((uint64_t)n * inv) >> 32);
  return q + (n - q * d >= d ? 1u : 0u);
}
// A grid of mt x nt tiles of Y in bands of B = 4 or 8 tile rows, the last band of mt % B where that is not 0: what its numbering
// divides by is B nt, the tiles of a band, and the last band's rows.  Two bits that the numbers divided here (below 2^31) do not need
// of the reciprocals: inv_band's lowest says that B is 4, inv_last's that the bands (of 8) are joined (tile_of_joined).
struct TileGrid {
  uint32_t mt, nt, inv_band, inv_last;
  __host__ __device__ __forceinline__ uint32_t log_band() const { return 3 - (inv_band & 1); }
  __host__ __device__ __forceinline__ bool joined() const { return (inv_last & 1) != 0; }
};
inline void set_tile_grid(GemmArgs& g, uint32_t mt, uint32_t nt, uint32_t band = 8, bool joined = false) {
  const uint32_t over = mt % band, last = over == 0 ? band : over <= 2 && joined && mt > band ? band + over : over;
  g.inv_band = (reciprocal(band * nt) & ~1u) | (band == 4 ? 1 : 0);
  g.inv_last = (reciprocal(last) & ~1u) | (joined ? 1 : 0);
}
// Tile L of the order that walks a band's rows down before it moves one tile right.
__host__ __device__ __forceinline__ void tile_in_bands(const TileGrid& t, uint32_t L, uint32_t& tile_m, uint32_t& tile_n) {
  const uint32_t s = t.log_band(), b = 1u << s, band = divide(L, t.nt << s, t.inv_band & ~1u), r = L - band * (t.nt << s);
  if (band * b + b <= t.mt) {
    tile_n = r >> s;
    tile_m = band * b + (r & (b - 1));
  } else {
    const uint32_t last = t.mt & (b - 1);
    tile_n = divide(r, last, t.inv_last);
    tile_m = band * b + r - tile_n * last;
  }
}
// Workgroups are dealt round-robin to the 8 XCDs, each with its own L2: number L of a launch of `total` as the place in an order of
// which XCD x gets a contiguous range (total / 8, one more for the first total % 8).
__host__ __device__ __forceinline__ uint32_t xcd_part(uint32_t total, uint32_t L) {
  const uint32_t per = total / 8, rem = total % 8, x = L % 8, j = L / 8;
  return x * per + (x < rem ? x : rem) + j;
}
// XCD-aware tile numbering: launch-order number L -> (tile_m, tile_n), the 32 workgroups running together on an XCD a
// 4 x 8 or 8 x 4 patch sharing 12 panels.
__host__ __device__ __forceinline__ void tile_of(const TileGrid& t, uint32_t L, uint32_t& tile_m, uint32_t& tile_n) {
  tile_in_bands(t, xcd_part(t.mt * t.nt, L), tile_m, tile_n);
}
// The same for small tiles, in joined bands: a remainder of one or two rows belongs to the band of eight before it.  As a band
// of its own it is the part of one XCD alone, which then reads every column of the weight: us with nine tile rows, joined and not, the operands
// in the last-level cache: [N x K] 258 x 2816 -> 1536 8.7, 10.9, 530 x 2816 -> 3584 21.4, 23.6; [K x N] 288 x 1440 -> 1536 7.0, 8.1.  Three
// rows stay alone (24 sizes of eleven tile rows 0.98 of joined).
__host__ __device__ __forceinline__ void tile_of_joined(const TileGrid& t, uint32_t L, uint32_t& tile_m, uint32_t& tile_n) {
  const uint32_t l = xcd_part(t.mt * t.nt, L);
  uint32_t band = divide(l, 8 * t.nt, t.inv_band), left = t.mt - 8 * band;   // tile rows from here on
  if (left <= 2 && band > 0) {
    --band;
    left += 8;
  }
  const uint32_t r = l - band * 8 * t.nt;
  if (left > 10) {
    tile_n = r >> 3;
    tile_m = 8 * band + (r & 7);
  } else {
    tile_n = divide(r, left, t.inv_last & ~1u);
    tile_m = 8 * band + r - tile_n * left;
  }
}
// The same for small tiles, dealt out: tiles that share a piece of the weight (the rows of a band of eight), and with narrow [K x N]
// tiles the two that share its cache lines, go to one XCD as a group, and the groups round-robin over the XCDs.
__host__ __device__ __forceinline__ void tile_of_groups(const TileGrid& t, bool pairs, uint32_t b, uint32_t& tile_m, uint32_t& tile_n) {
  const uint32_t p = pairs ? 1 : 0;   // groups of G = min(mt, 8) << p tiles
  const uint32_t whole = t.mt < 8 ? (t.nt >> (3 + p) << (3 + p)) * t.mt : t.mt * t.nt >> (6 + p) << (6 + p);   // of rounds of 8 G
  uint32_t L = b;
  if (b < whole) {
    const uint32_t j = b >> 3, q = t.mt < 8 ? divide(j >> p, t.mt, t.inv_last) : j >> (3 + p), G = (t.mt < 8 ? t.mt : 8) << p;
    L = (q * 8 + (b & 7)) * G + j - q * G;
  }
  tile_in_bands(t, L, tile_m, tile_n);
}
// fused: 0 = plain GEMM on g.w; kJustSampled = the same, the launch before writes g.w; kFusedInOperand = sampling in the weight operand
// load of every tile
constexpr int kJustSampled = 1, kFusedInOperand = 2;
int launch_gemm(const GemmArgs& g, int w_is_nk, int fused, int fmt, hipStream_t stream);
// few rows of X or few tiles (gws_gemm_stream.hip): the tile in units of 16 rows and 16 columns, the parts of K, the rows and
// columns of it that a workgroup owns, the workgroups a tile that warm the L2, whether each XCD takes a contiguous part of the tiles,
// and the estimated time; p == 0: the shape is not one for it
struct StreamPlan {
  int mt, nt, p, bm, bn, warm, parts;
  double us;
};
StreamPlan stream_plan(uint64_t M, uint64_t N, uint64_t K, bool w_is_nk);
void stream_after_sampling(const GemmArgs& g, int w_is_nk, StreamPlan& p);   // the plan where the launch before writes the weight
bool stream_applicable(const GemmArgs& g);
int launch_gemm_stream(const GemmArgs& g, int w_is_nk, const StreamPlan& p, hipStream_t stream);
int launch_gemm_stream_sample(const GemmArgs& g, int w_is_nk, int fmt, int p, hipStream_t stream);
uint32_t stream_sample_rows(const GemmArgs& g, int p);   // of its tile, which is 32 columns wide
// many rows, the weight sampled on its way in, K from end to end
bool rows_sample_applicable(const GemmArgs& g, int w_is_nk);
int launch_gemm_rows_sample(const GemmArgs& g, int w_is_nk, int fmt, hipStream_t stream);
uint32_t rows_sample_tile(const GemmArgs& g);   // rows and columns of its tile, 256 or 128
enum class GemmRoute { kStream, kMiddle, kLarge, kNarrow, kSmall };
struct RoutePlan {   // estimates in us; 1e30: not a shape for that kernel
  StreamPlan stream;
  double middle_us, large_us, narrow_us;
  int middle_nj;      // the middle tile is 128 x 32 middle_nj
  double middle_line; // what the stream kernel has to beat of the middle tile
};
GemmRoute gemm_route(const GemmArgs& g, int w_is_nk, RoutePlan& plan);
// the kernel that launch_gemm takes (Y apart from the operands); the values are GWS_GEMM_* of gws_bench.h
enum class GemmForm { kStream = 1, kMiddle, kLarge, kLargeEdge, kNarrow, kAnyShape, kStreamSample, kRowsSample, kAnyShapeSample };
GemmForm gemm_form(const GemmArgs& g, int w_is_nk, int fused, RoutePlan& plan);
void gemm_tile(const GemmArgs& g, GemmForm form, const RoutePlan& plan, uint32_t& rows, uint32_t& cols);   // of a workgroup of it
bool sample_in_operand(const GemmArgs& g, int w_is_nk);   // the faster way to a sampled product (same bits either way)
bool gemm256_edge_applicable(const GemmArgs& g);
int launch_gemm256_edge(const GemmArgs& g, int w_is_nk, hipStream_t stream);
int launch_gemm256_narrow(const GemmArgs& g, int w_is_nk, hipStream_t stream);   // shapes as gemm256_edge_applicable
bool gemm128_applicable(const GemmArgs& g);
int launch_gemm128(const GemmArgs& g, int w_is_nk, int nj, hipStream_t stream);   // tiles of 128 x 32 nj, nj 3 or 4
bool gemm256_applicable(const GemmArgs& g);
int launch_gemm256(const GemmArgs& g, int w_is_nk, hipStream_t stream);
// Weights whose forward sampling rides in a GEMM's launch: descriptors as the forward pass fills them, with
// first_wg = the weight's first 32 x 256 tile in the riders' numbering (rider 1); begin[j] = that number again for
// j < n and the total for every j >= n (so that a search over begin[1..] needs no n).
constexpr int kMaxRide = 4;
struct RideList {
  TileDesc d[kMaxRide];
  uint32_t begin[kMaxRide + 1];
  uint32_t n;
};
// the 256-tile GEMM (none if g.M == 0) followed, in the same grid, by `extra` workgroups that sample the weights of
// `r` as the forward pass does; rider: 0 = sample_tiles on r.d[0] alone (rows a multiple of 32, columns of 64),
// 1 = ride_tiles (every weight: rows a multiple of 32, columns of 256)
int launch_gemm256_ride(const GemmArgs& g, int w_is_nk, const RideList& r, int fmt, uint64_t step, uint32_t extra,
                        int rider, hipStream_t stream);
int compute_units();   // of the current device; 0 if the query fails
// Bands of four that leave one or two tile rows to a band of their own, which is the part of one or two XCDs and reads all of the other
// operand there.
inline bool leaves_few(uint32_t mt) { return mt % 4 == 1 || mt % 4 == 2; }
// The band for mt x nt tiles of the weight gradient: an XCD's workgroups at work form a patch of so many tile rows by the columns that
// follow, and what it reads into its L2 is the patch's rows of one operand and its columns of the other, over all bands fewer lines with
// 4 or with 8 (rows, cols: of a tile).  us with 8 and with 4: 4096 x 768 x 768 in 64 x 64 17.9, 16.2, 8192 x 2048 x 2560 81.8, 80.1; on a
// tie 8: 4096 x 3072 x 768 29.4, 30.0, 4096 x 768 x 3072 30.7, 30.9.  8 too where bands of four leave one or two rows over (leaves_few):
// 7040 x 768 x 2560 in 128 x 64, six tile rows, 39.8, 42.5.
uint32_t patch_band(uint32_t mt, uint32_t nt, uint32_t rows, uint32_t cols);
// Weight-gradient GEMM (gws_gemm256_tn.hip): y[M x N] = x^T * w with x [K x M], w [K x N]
// row-major (K = the contraction length); with_dbt adds Eq. 4's block reduction on y.
bool gemm256_tn_applicable(const GemmArgs& g);
int launch_gemm256_tn(const GemmArgs& g, bool with_dbt, hipStream_t stream);
int launch_gemm256_tn_narrow(const GemmArgs& g, bool with_dbt, hipStream_t stream);   // the same with tiles of 256 x 192
// weights of few tiles (gws_gemm_stream_tn.hip): a 16 mt x 16 nt piece a workgroup, the tokens in four fp32 sums (halves: in
// eight); us 1e30: no piece takes the leading dimensions
struct TnPlan {
  int mt, nt;
  double us;
};
TnPlan stream_tn_plan(const GemmArgs& g, bool lines, bool halves);
int launch_gemm_stream_tn(const GemmArgs& g, bool with_dbt, const TnPlan& p, bool halves, hipStream_t stream);
// the same result with the contraction of every tile split over `parts` (2 .. 8, at most K / 64) workgroups: fp32 partial tiles in
// `ws` (gemm256_tn_split_bytes, 16-byte aligned), added in a fixed order by a second kernel
size_t gemm256_tn_split_bytes(const GemmArgs& g, uint32_t parts);
int launch_gemm256_tn_split(const GemmArgs& g, bool with_dbt, float* ws, uint32_t parts, hipStream_t stream);

}  // namespace gws
