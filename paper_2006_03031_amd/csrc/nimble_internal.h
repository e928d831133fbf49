// Internal declarations shared by the host dispatcher and the kernel launchers.
#ifndef NIMBLE_INTERNAL_H_
#define NIMBLE_INTERNAL_H_

#include <cstdint>

#include "nimble.h"

namespace nimble {

struct VariantInfo {
  const char* name;
  int bm, bn, bk, threads;
};
extern const VariantInfo kVariants[NIMBLE_VAR_COUNT];

// The chip this library is written for: MI355X, 256 compute units in 8 XCDs.
constexpr int kComputeUnits = 256;
// Workgroups of a tiled variant that share a compute unit (LDS and registers permitting).
constexpr int kTilesPerCU[NIMBLE_VAR_COUNT] = {1, 1, 2, 2, 2, 1, 1};

// Record a message for nimble_last_error() and return `code`.
int fail(int code, const char* fmt, ...);
void clear_error();

bool tiled_variant_ok(int variant, int64_t M, int64_t N, int64_t K);
// bm = 0 or the variant's own height: always; else the heights the variant is also built at.
bool tile_rows_ok(int variant, int bm, int64_t N, int64_t K);

// Weights above this size are taken to come from HBM on every call (the L2s hold 32 MB, the
// memory-side cache 256 MB shared with everything else in flight); smaller layers are priced
// as cache-resident, which is what a layer loop or a token loop sees.
constexpr double kCachedWeightBytes = 64e6;

// What the memory-side cache holds.
constexpr double kMemorySideCacheBytes = 256.0 * 1024 * 1024;

// Whether a launch of up to 64 rows that reads the weights of an [N, K] layer once loads them non-temporally.  Where each call finds
// them in memory that is faster, since memory is then read at the rate of a plain read; but such loads leave nothing in the memory-side
// cache either, and a layer that this would have held (a wide layer among small ones) is slower with them.  Microseconds
// per layer, several layers in turn (1 GB of them) / one over and over, through the caches -> past them:
//   Streaming kernel,   1 row                       8 rows                      16 rows
//   8192 x 4096         13.3 / 12.2 -> 11.8 / 9.7   13.4 / 11.2 -> 12.0 / 10.5  15.7 / 12.2 -> 14.6 / 13.2
//   6144 x 6144         16.0 / 12.1 -> 14.6 / 12.7  18.0 / 12.6 -> 16.2 / 14.4  21.0 / 14.4 -> 19.8 / 18.2
//   7168 x 7168         19.0 / 15.7 -> 17.1 / 15.6  20.3 / 16.1 -> 18.6 / 17.2  25.2 / 17.6 -> 22.5 / 21.2
//   8192 x 8192         23.9 / 21.1 -> 21.7 / 19.7  24.2 / 20.0 -> 22.1 / 20.3  26.7 / 21.1 -> 25.6 / 24.2
//   5120 x 13824        30.6 / 24.0 -> 28.2 / 25.9  33.6 / 24.2 -> 31.6 / 29.8  39.3 / 27.4 -> 38.1 / 36.5
//   32000 x 4096        44.3 / 40.5 -> 39.8 / 37.0  45.7 / 37.5 -> 39.9 / 38.2  56.7 / 41.7 -> 53.0 / 51.1
//   8192 x 28672        78.5 / 77.5 -> 69.7 / 67.1  79.6 / 78.2 -> 72.2 / 70.1  90.0 / 88.9 -> 84.3 / 82.8
// Up to 8 rows what is gained in turn is what is lost over and over at most (but for layers that leave the cache to little else), beyond
// that it is less; what the cache cannot hold gains either way.
//   32-row tiles with K cut, 20 and 32 rows: 4096 x 8192 19.2 / 17.1 -> 18.9 / 16.8, 19.4 / 17.2 -> 19.7 / 18.2; 8192 x 4096 18.0 / 15.8 -> 15.6 /
// 14.1, 18.5 / 16.1 -> 15.9 / 14.3; 6144 x 6144 20.8 / 17.5 -> 20.2 / 18.5, 21.0 / 17.9 -> 21.1 / 19.7; 8192 x 8192 30.5 / 24.3 -> 28.1 / 26.8,
// 30.7 / 24.5 -> 28.6 / 27.4; 5120 x 13824 31.7 / 26.5 -> 29.7 / 28.0, 31.9 / 26.8 -> 30.3 / 29.2; 8192 x 14336 46.0 / 38.1 -> 40.2 / 38.7, 46.4 /
// 38.3 -> 40.6 / 39.3; with K in two, or more than a workgroup per compute unit, 13824 x 5120 32.3 / 25.1 -> 29.8 / 28.7, 14336 x 4096 28.4 /
// 22.8 -> 27.1 / 25.6, 32000 x 4096 61.7 / 46.1 -> 58.5 / 59.0.
//   64-row tiles with K cut, 64 rows: 6144 x 6144 23.1 / 19.5 -> 25.1 / 24.1, 7168 x 7168 26.4 / 22.7 -> 27.6 / 26.7, 8192 x 8192 32.4 /
// 26.1 -> 30.7 / 30.1, 8192 x 28672 90.1 / 89.0 -> 81.2 / 79.8.
inline bool weights_pass_by(int64_t rows, int64_t N, int64_t K, int64_t slices) {
  const double bytes = (double)N * (double)K * 2.0;
  if (bytes <= kCachedWeightBytes) return false;
  if (rows <= 8 || bytes > kMemorySideCacheBytes) return true;
  return rows > 16 && rows <= 32 && slices >= 3 && (N + 127) / 128 * slices <= kComputeUnits;
}

// Whether every one of `slices` K slices gets whole 64-wide stages (the 64-wide ring).  NIMBLE_RING32 (a
// measurement knob, read once) turns that ring off.
bool wide_stages_ok(int64_t K, int64_t slices);
// Whether a launch of the 64- or 128-row tile (128 wide) runs with eight waves per tile and a compute unit
// to itself: at most one tile per compute unit (all slices and batches counted), K in 64-wide stages.  A lone
// tile is a serial chain of stages, and eight waves walk it in less time than four: microseconds with four / eight
// waves, 64 rows: 509 x 2304 x 768 8.3 / 7.8, 509 x 3072 x 768 (GELU) 9.0 / 8.4; 128 rows: 800 x 4096 x 1024 (GELU)
// 15.3 / 13.6, 4000 x 1024 x 4096 45.7 / 36.8.  With more tiles two workgroups of four waves share a
// compute unit, which is the better use of it (600 x 4096 x 1024, 320 tiles of 64 rows: 14.4 / 16.9); 64 rows also
// stay with four waves where the chip is nearly full of long tiles, which all pull on the L2s (2600 x 768 x 3072,
// 246 tiles: 19.6 / 20.4; with 204 tiles 19.4 / 19.0), and with K cut (509 x 1024 x 4096 in four: 14.5 / 15.8).
inline bool eight_waves(int variant, uint64_t tiles, int64_t K, int64_t slices) {
  if (tiles > (uint64_t)kComputeUnits || !wide_stages_ok(K, slices)) return false;
  if (variant == NIMBLE_VAR_T64x128) return slices == 1 && (K <= 2048 || tiles <= (uint64_t)kComputeUnits * 7 / 8);
  return variant == NIMBLE_VAR_T128x128;
}

// Slots of gemm_quarter_kernel's ring, 0: not built for these tiles.
constexpr int quarter_slots(int bm, int bn) {
  if (bn == 256) return bm <= 256 ? 2 : 0;
  return bn != 128 ? 0 : bm == 256 ? 3 : bm == 128 ? 4 : 0;
}

// Whether a launch of `tiles` whole tiles (over all batches) runs four waves in place of eight, one per SIMD
// (gemm_quarter_kernel).  They walk a K stage 4 to 7 % faster, but have no second wave under the epilogue, the fill and the
// first loads: a workgroup has to walk enough stages, over all its tiles.  Microseconds, eight waves / four: 256-wide
// tiles, stages walked: 4 (2113 x 4096 x 256) 9.2 / 10.4, 12 (3500 x 4096 x 768) 23.4 / 23.9, 16 (3500 x 4096 x 1024 with GELU)
// 29.8 / 31.0, 24 (8192 x 4096 x 768 with GELU) 53.4 / 54.9, 24 (4096 x 4096 x 1536) 43.1 / 42.3, 32 (16129 x 4096 x 512 with
// GELU) 98.0 / 93.4, (5000 x 4096 x 1024) 40.5 / 39.7, (4096 x 4096 x 2048) 53.7 / 52.6, 64 (9000, 10240 and 16384 x 1024 x 4096)
// 62.6 / 58.5, 66.4 / 62.8, 95.7 / 91.3; 256 x 128: 24 (8192 x 1024 x 1536 with GELU) 27.2 / 27.6, 32 (x 2048) 32.2 / 31.8, 64
// 56.7 / 54.3; 128 x 128, alone on their compute units: 32 (2113 x 1024 x 2048) 17.0 / 17.2, 48 23.7 / 23.3, 64 29.9 / 29.1.
// (Tiles of 64 rows are slower throughout, two workgroups of 128 x 128 to a compute unit too: 6000 x 768 x 768 11.0 / 11.3.)
inline bool quarter_kernel_wins(int bm, int bn, int64_t tiles, int64_t K, int64_t slices, int64_t batch) {
  const int slots = quarter_slots(bm, bn);
  if (slots == 0 || !wide_stages_ok(K, slices)) return false;
  const int64_t stages = K >> 6, per = (stages + slices - 1) / slices;
  if (stages - (slices - 1) * per < slots) return false;  // (the first stages are loaded unconditionally)
  if (bm == 128 && bn == 128) return slices == 1 && tiles <= kComputeUnits && per >= 48;
  const int64_t walked = slices == 1 && batch == 1 ? (tiles + kComputeUnits - 1) / kComputeUnits : 1;
  return per * walked >= 32;
}

// Whether the ring kernels can run an [M, N] output over K: whole 32-wide stages, output rows of whole 16-byte pieces.
inline bool ring_shape_ok(int64_t N, int64_t K) { return K % 32 == 0 && N % 8 == 0; }

// Where they cannot (K is a multiple of 8): whether gemm_tile_kernel in the variant's own tiles, `tiles` of them over
// all batches, beats any_kernel in tiles of 64 x 64.  It does where its tiles fill the chip; with fewer, small
// tiles with K shared by groups of waves are the better use of it.  Microseconds, tile kernel / any_kernel, to f32:
// 64- and 128-row tiles: 392 (3130 x 1024 x 904) 18 / 24, 306 (1117 x 4240 x 2648) 53 / 70, 225 (606 x 5760 x 1608) 36 / 39,
// 190 (2332 x 432 x 712) 11.2 / 9.8; 256-wide tiles: 234 (6421 x 2304 x 2808) 124 / 210, 165 (2771 x 3656 x 4560) 168 / 219,
// 144 (6000 x 1502 x 6000) 226 / 241, 136 (951 x 8632 x 2256) 85 / 84, 126 (1484 x 2688 x 3416) 79 / 70.  Its lanes write
// the columns they own, four at a time, where any_kernel writes whole rows: K has to be long enough to make up for
// that.  6000 x 4096 to f32 25 / 29 at K = 40 and 84 / 113 at 1000, to bf16 42 / 34 at 136, 54 / 54 at 328, 79 / 83 at 648;
// 6000 x 4100 (rows of whole 8-byte pieces) to f32 39 / 38 at 136, 43 / 45 at 200, to bf16 71 / 68 at 456, 106 / 114 at
// 1000; 4442 x 6852 x 184 to f32 49 / 55; with N not a multiple of 4 the columns are written one by one: 4434 x 2078 x
// 2016 104 / 83, 2771 x 3471 x 4560 with GELU 181 / 199.
inline bool tile_kernel_wins(int variant, int64_t tiles, int64_t N, int64_t K, bool out_f32) {
  if (variant < NIMBLE_VAR_T64x128) return false;
  if (tiles < (variant <= NIMBLE_VAR_T128x128 ? 256 : K >= 4096 ? 140 : 160)) return false;
  if (N % 4 != 0) return K >= 4096;
  if (out_f32) return N % 8 == 0 || K >= 160;
  return K >= (N % 8 == 0 ? 448 : 896);
}

// Whether a launch of any_kernel shares each tile's K among four groups of waves: a workgroup per compute unit is all
// there is, and K is long enough to pay for handing the sums over: with b [N, K] two stages.  Microseconds, one group / four: 515 x 1001 to
// f32, K = 40 4.5 / 4.3, 64 4.3 / 4.3, 127 5.4 / 4.7, 256 5.4 / 4.7, 511 8.6 / 6.6; 1000 x 1000 to bf16, K = 40 4.3 / 4.5, 64
// 4.2 / 4.5, 128 4.6 / 4.5, 257 7.0 / 5.8; 70 x 130, K = 64 3.9 / 4.1, 128 4.3 / 4.1, 640 7.2 / 5.8.  With b [K, N] from K = 512 on, as
// measured before the groups shared the end of a tile too.  With 512 tiles at K = 1000 two groups already took 14.0 -> 15.1.
inline bool any_four_groups(int64_t tiles, int64_t K, bool b_is_kn) { return K >= (b_is_kn ? 512 : 65) && tiles <= kComputeUnits; }

// Whether a tiled plan the dispatch function made is launched in the 64 x 64 tiles of any_kernel instead (`tiles`: of
// the variant's own, over all batches; `small`: of 64 x 64).  Where the ring kernels can run, a partly empty last
// tile column costs them no more than its loads (ring / any_kernel, microseconds: 423 x 2928 x 3648 20 / 37,
// 12456 x 200 x 1024 12.5 / 19.6, 1240 x 1112 x 512 6.2 / 8.0), but a handful of tiles leaves the chip to few
// workgroups, and the smaller ones with K shared by four groups of waves are done earlier (953 x 64 x 512, 15 of them,
// 5.1 / 2.9, 662 x 184 x 2048, 33, 10.9 / 9.1, 1315 x 112 x 1024, 42, 6.8 / 7.5, 1637 x 112 x 512, 52, 5.2 / 6.0; where one
// group ran 238 x 264 x 96, 20, 3.9 / 4.4).
inline bool small_tiles_win(int variant, int64_t tiles, int64_t small, int bn, int64_t N, int64_t K, bool out_f32) {
  if (!ring_shape_ok(N, K)) return !tile_kernel_wins(variant, tiles, N, K, out_f32);
  return N % bn != 0 && small <= 40 && K >= 512;
}

// Whether a launch of any_kernel in `tiles` tiles, over all batches, leaves its output in the L2s.  Its rows start anywhere,
// so that nearly all of the 128-byte runs which a wave writes fall into two lines.  Where every workgroup stores at about the
// same time, the launch's end, f32 outputs gain by being written through all the same, since the next launch waits for it: one
// round of workgroups, or two of a short K.  Otherwise the pieces that go to memory are what counts.  Microseconds, left /
// written through: 144 tiles (515 x 1001 x 1003) 10.7 / 10.45, 230 (1433 x 635 x 322) 7.2 / 6.8, 256 (1000 x 1000 x 500) 8.0 / 7.5,
// 292 (4610 x 212 x 52) 5.8 / 5.4, 504 (1287 x 1517 x 111) 7.0 / 6.4; 285 (1187 x 941 x 473, GELU) 11.6 / 12.1, 384 (3038 x 470 x
// 339, GELU) 10.7 / 11.0, 573 (12205 x 147 x 138) 8.3 / 8.7, 752 (3000 x 1001 x 129) 9.7 / 10.0, 5250 (11134 x 1861 x 277)
// 52 / 79, 5922 (6000 x 4001 x 33) 32 / 61.  bf16 is no faster in one round either.
inline bool any_output_stays(int64_t tiles, int64_t K, bool out_f32) {
  return !out_f32 || tiles > (K <= 128 ? 2 : 1) * kComputeUnits;
}

// Query rows per workgroup of attention_chain_kernel with `waves` waves: 16 where these workgroups all find a place at once (16 KB
// of LDS per wave, 160 KB and 32 waves per compute unit), else 32.  Microseconds, 32 rows / 16: eight waves, 252 workgroups of 16 rows (12 heads of
// 333) 8.4 / 6.7, 264 (352) 8.2 / 10.3; four, 512 (32 of 250) 7.8 / 7.3, 624 (48 of 200) 8.9 / 10.0; two, 672 (96 of 100) 7.1 / 5.9,
// 1600 (200 of 128) 9.5 / 10.8; one, 1800 (600 of 33) 7.7 / 6.1.
inline int attention_chain_rows(int64_t heads, int64_t L, int waves) {
  return heads * ((L + 15) / 16) <= 8 * kComputeUnits / waves ? 16 : 32;
}

// Tiles of one launch of any_kernel (a launch holds less than 2^32 threads); larger outputs take several, each of at most
// `tm` x `tn` tiles.  (With the rest in the second grid dimension every launch paid 0.1 to 0.2 us for finding its tile.)
inline void any_launch_tiles(int64_t tiles_m, int64_t tiles_n, int64_t* tm, int64_t* tn) {
  constexpr int64_t most = 1 << 22;
  *tn = tiles_n < most ? tiles_n : most;
  *tm = tiles_m * *tn <= most ? tiles_m : most / *tn;
}

// Row groups (of 8) in one launch of the LSTM token loop: of H / 16 workgroups each on one XCD (two above H = 512), as many
// as give each of its compute units one workgroup at most.
inline int lstm_groups_per_launch(int64_t H) {
  const int n_wg = (int)(H / 16), span = n_wg > 32 ? 2 : 1, per_xcd = n_wg / span;
  return 8 / span * (per_xcd < kComputeUnits / 8 ? kComputeUnits / 8 / per_xcd : 1);
}

// Whether a weight-streaming launch of 16-row blocks over an [N, K] weight can run the LDS-staged
// streaming kernel (the LSTM cell needs Ix % 64 == 0 besides).
bool stream_kernel_shape_ok(int64_t N, int64_t K);

struct PlanOptions {
  uint64_t max_workspace = 0;   // bytes of caller scratch available (split-K partial sums)
  bool allow_row_split = true;  // may dispatch x = bm*k + r as two launches
  int force_split_k = 0;        // > 0 with a forced variant: cut K into exactly this many slices
  bool generic_rows = true;     // the generic variant may run in 16-row blocks (b is [N, K])
  bool out_f32 = false;         // the output is f32 (which kernel is better for a shape the ring kernels cannot run)
  bool use_table = true;        // consult the tuned dispatch table before the cost model
};

// Dispatch table shared by dense (batch = 1) and batch_matmul.
int plan_dense(int64_t batch, int64_t M, int64_t N, int64_t K, int epilogue, int force_variant,
               const PlanOptions& opt, nimble_plan* p);

// Whether the batch_matmul plan `p` with b [K, N], a tiled one, is launched on b transposed.
bool nn_transposes(const nimble_plan& p, int64_t batch, int64_t M, int64_t N, int64_t K);

// One C = epi(alpha * A.B^T + bias) problem as the kernels see it.  A is
// [M,K] with row stride lda, B is [N,K] with row stride ldb (or, when
// b_is_kn, [K,N] with row stride ldb), C is [M,N] with row stride ldc; strides
// in elements; batch strides sa/sb/sc in elements.
struct GemmArgs {
  const void* a;
  const void* b;
  const void* bias;
  void* c;
  int M, N, K;
  int lda, ldb, ldc;
  long long sa, sb, sc;
  float alpha;
  int epilogue;
  int out_f32;
  int b_is_kn;
  int batch;
  int weights_read;  // another launch of the same call has just read b (host only: weights_pass_by is not asked)
};

// Whether the tiled kernels leave their output in the L2s (plain stores) instead of writing it through them as it is made
// (store_through in device_common.h).  What goes to memory by itself has to be whole 64-byte pieces: rows that do not start on
// one cost about twice the writes.  Microseconds, left / written through.
//   Rows of whole pieces: bf16 leaves as whole lines and is written through whatever its size, 4096 x 4096 x 64 12.1 / 10.1,
//   20000 x 10240 x 128 130 / 123 (82 shapes: 4 % less in the mean, none lost more than 1.4 %).  f32 leaves as half lines, which is
//   as good while the output stays in the caches: 4736 x 2048 x 512 18.8 / 16.0, 4096 x 4096 x 256 21.6 / 18.7, 385 x 5760 x 1280
//   15.5 / 13.2; but 24 x 1024 x 1024 x 64 22.9 / 23.5, 12 x 2048 x 2048 x 64 39.3 / 41.7, and beside more weights from 32 MB on:
//   2000 x 12000 x 1536 85.7 / 92.2, 700 x 12288 x 1536 44.6 / 46.7, 466 x 19520 x 320 (50 layers in turn) 25.4 / 30.1 (512 x 32000 x
//   1024 would gain, 43.6 / 42.1).
//   Other rows: f32 loses mostly, 3000 x 4104 x 256 20.1 / 21.4, 10201 x 3864 x 64 48 / 86 (1605 x 840 x 192 with GELU would gain,
//   5.8 / 5.5).  bf16 gains where the output is large enough for its write-back at the kernel's end to show, 8658 x 696 x 128
//   9.6 / 8.0, 835 x 8336 x 480 16.1 / 14.6, 4096 x 4104 x 64 14.4 / 12.8 (4 of some 90 shapes lose 2 to 4 %, 5022 x 792 x 224
//   8.2 / 8.5), and loses below 1 MB, 706 x 328 x 288 4.56 / 4.65, and when there is too much of it, 3767 x 4616 x 1024 (60 layers
//   in turn) 50 / 53, 12869 x 2488 x 960 64 / 73, 10201 x 7736 x 64 54 / 90.
inline bool output_stays(const GemmArgs& g, int64_t slices) {
  constexpr int64_t MB = 1 << 20;
  if (slices > 1) return false;  // (partial_sums_stay)
  const int64_t width = g.out_f32 ? 4 : 2, out = (int64_t)g.batch * g.M * g.N * width;
  const bool few_weights = (int64_t)g.batch * g.N * g.K * 2 <= 8 * MB;
  const uint64_t starts = (uint64_t)reinterpret_cast<uintptr_t>(g.c) | (uint64_t)(g.ldc * width) | (g.batch > 1 ? (uint64_t)(g.sc * width) : 0);
  const bool whole = starts % 64 == 0;
  if (g.out_f32) return !whole || out > (few_weights ? 64 : 32) * MB;
  return !whole && (out < MB || out > (few_weights ? 36 : 24) * MB);
}

}  // namespace nimble
#endif
