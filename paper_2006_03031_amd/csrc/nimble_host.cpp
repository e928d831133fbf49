// Host side of the dynamic-shape path: shape functions (Section 3.2), storage
// sizes (Section 3.3), the residue split and the dispatch function's table
// (Section 3.5).  Integer arithmetic only; no HIP call in this file.
#include "nimble_internal.h"

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <map>
#include <tuple>
#include <vector>

namespace nimble {

static thread_local char g_err[256] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

void clear_error() { g_err[0] = '\0'; }

const VariantInfo kVariants[NIMBLE_VAR_COUNT] = {
    // name       bm   bn   bk  threads
    {"generic", 64, 64, 64, 256},
    {"skinny16", 16, 16, 32, 256},
    {"t32x128", 32, 128, 32, 256},
    {"t64x128", 64, 128, 32, 256},
    {"t128x128", 128, 128, 32, 256},
    {"t256x128", 256, 128, 32, 512},
    {"t256x256", 256, 256, 32, 512},
};

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Number of compute units of one MI355X.
static const int64_t kCUs = kComputeUnits;

// Estimated time of one macro tile, in arbitrary units: the tile's area times
// (K plus a fixed per-tile overhead expressed in units of K: pipeline fill and
// the epilogue, which is larger with GELU), divided by how well the variant
// keeps the matrix cores busy in steady state (measured per variant at
// M = 8192 on the BERT-large FFN shapes).
static double tile_cost(int variant, int64_t K, int epilogue, int bm = 0) {
  double eff;
  switch (variant) {
    case NIMBLE_VAR_T32x128: eff = 0.202; break;
    case NIMBLE_VAR_T64x128: eff = 0.450; break;
    case NIMBLE_VAR_T128x128: eff = 0.560; break;
    case NIMBLE_VAR_T256x128: eff = 1.031; break;
    case NIMBLE_VAR_T256x256: eff = 1.10; break;
    default: return 1e30;
  }
  const double k0 = (epilogue == NIMBLE_EPI_BIAS_GELU_ERF) ? 256.0 : 128.0;
  // a tile of another height loads the same weight panel for fewer or more rows: measured
  // time(bm) / time(256) = 0.09 + 0.91 bm/256 for the 256-wide tile (bm = 128..320)
  const double height = (bm > 0 && bm != kVariants[variant].bm)
                            ? 0.0925 + 0.9075 * (double)bm / (double)kVariants[variant].bm : 1.0;
  return (double)kVariants[variant].bm * kVariants[variant].bn * ((double)K + k0) * height / eff;
}

// Heights the 256-wide tile is built at: 2 wave rows of 4..10 MFMA tiles of 16 rows.
static const int kTileRows256[] = {320, 288, 256, 224, 192, 160, 128};

// The height of the 256-wide tile that may be shared by two workgroups, 128 columns each.
static const int kHalvedRows = 192;

bool tile_rows_ok(int variant, int bm, int64_t N, int64_t K) {
  if (bm == 0 || bm == kVariants[variant].bm) return true;
  if (variant != NIMBLE_VAR_T256x256) return false;
  if (N % 256 != 0 || K % 32 != 0) return false;  // the reduced heights have no ragged N/K body
  for (int h : kTileRows256)
    if (h == bm) return true;
  return false;
}

bool tiled_variant_ok(int variant, int64_t M, int64_t N, int64_t K) {
  (void)M;
  (void)N;
  if (variant < NIMBLE_VAR_T32x128 || variant > NIMBLE_VAR_T256x256) return false;
  // rows must stay 16-byte aligned; per-lane byte offsets inside a tile are 32-bit
  return K > 0 && K % 8 == 0 && K <= (1ll << 22);
}

// One unit of tile_cost in microseconds (a 256x256 tile at K = 1024 with GELU takes about 37 us
// when the whole chip is busy).
static const double kUsPerUnit = 4.4e-7;
// Gap between two dependent launches on one stream, microseconds.
static const double kLaunchGapUs = 3.5;
// The same gap as it shows between a K-split kernel and its reduction, whose launch the
// hardware queue has already decoded while the first kernel runs.
static const double kSplitGapUs = 1.80;

bool wide_stages_ok(int64_t K, int64_t slices) {
  static const bool off = std::getenv("NIMBLE_RING32") != nullptr;
  const int64_t stages = K >> 6, per = slices > 0 ? ceil_div(stages, slices) : 0;
  return !off && K > 0 && (K & 63) == 0 && per * (slices - 1) < stages;
}

// The 128-wide tiles up to 128 rows on the 64-wide ring, at most two tiles per compute unit, microseconds: a
// lone tile's fixed time plus its walk over the K stages (32 k each), slower the more tiles there are; from
// one tile per compute unit on, two workgroups share one.  Fitted to graph-timed launches over K = 768 .. 4096
// and 24 .. 450 tiles; GELU adds half a microsecond.  At K below 320 only up to one 64-row tile per compute unit:
// against the taller tiles, priced without a fixed time, 12 x 512 x 512 x 64 was run in 96 tiles of 256 rows, 6.3 us instead
// of 5.3 in 384 of 64, and 4956 x 1664 x 128 in 11.1 instead of 8.8.
// Nor from K = 12288 on, too far from the fit (1960 x 1792 x 16384 121 -> 131 us, 450 x 896 x 12288 with K in three
// 24 -> 32): there the older estimate decides alone, over cuts of K by powers of two.
static const int64_t kLongestFitted = 12288;
static double few_tiles_us(int v, int64_t tiles, int64_t stages, bool gelu) {
  const double t = (double)(tiles < kCUs ? tiles : kCUs);
  double fixed, per_stage, shared = 1.65, more = 0.25;
  switch (v) {
    case NIMBLE_VAR_T32x128:
      fixed = 0.85, per_stage = 0.108 + 0.0002 * t < 0.142 ? 0.108 + 0.0002 * t : 0.142, shared = 1.38, more = 0.2;
      break;
    case NIMBLE_VAR_T64x128: fixed = 1.1, per_stage = 0.105 + 0.0003 * t < 0.148 ? 0.105 + 0.0003 * t : 0.148; break;
    default: fixed = 2.2, per_stage = 0.183 + 0.00036 * (t > 100 ? t - 100 : 0); break;
  }
  const double us = fixed + (gelu ? 0.5 : 0.0) + per_stage * (double)stages;
  return tiles <= kCUs ? us : us * (shared + more * (double)(tiles - kCUs) / (double)kCUs);
}

// 192-row tiles of the 256-wide variant in two halves, a compute unit each: between what 128 rows hold in one round and what 256 do, which then
// leave a quarter to half of the chip idle.  Fixed time plus the walk over stages of 32 k, fitted (to 3 %) over
// K = 768 .. 4096 and 96 .. 256 halves.  Measured, microseconds, halves / the choice without them: 1100 x 4096 x 1024
// (GELU) 16.4 / 19.3, 1530 18.1 / 20.1; 4600 x 1024 x 4096 40.0 / 47.4, 6100 45.6 / 50.7; 2500 x 2304 x 768 13.9 / 15.6;
// 6000 x 768 x 3072 31.4 / 40.5.  Where 128-row tiles are one round they stay: 3500 x 1024 x 4096 38.3 / 34.5; so do two
// workgroups of 64-row tiles on short K: 1300 x 3072 x 768 (GELU) 13.9 / 13.5.
static double halved_us(int64_t halves, int64_t stages, bool gelu) {
  const double crowded = halves > 128 ? 0.00043 * (double)(halves - 128) : 0.0;
  return 3.0 + (gelu ? 2.0 : 0.0) + (0.244 + crowded) * (double)stages;
}

// Estimated time of one launch of tiled variant v over `rows` rows with K cut into `sk`
// slices, microseconds.  The tiles run in rounds of one per compute unit.  A full round runs
// at the chip's power-limited rate; the last, partial round runs faster per tile the fewer
// units it occupies.  So a dynamic M just past a tile boundary costs most of an extra round
// with big tiles, while smaller tiles quantise more finely but run the matrix cores less
// efficiently.  Cutting K multiplies the tiles and shortens each; the partial sums then cross
// HBM once more and a second small kernel adds them up.  The constants are a fit to graph-timed
// launches of every variant and K split over the BERT-base/large and LSTM layer shapes at
// 17 .. 2048 rows; over that set the choices made here cost 0.6 % more than the best ones.
static double tiled_cost_us(int v, int64_t batch, int64_t rows, int64_t N, int64_t K, int epilogue,
                            int sk = 1, int bm = 0) {
  const VariantInfo& vi = kVariants[v];
  const int64_t tiles = batch * ceil_div(rows, bm > 0 ? bm : vi.bm) * ceil_div(N, vi.bn) * sk;
  const int64_t k_slice = ceil_div(ceil_div(K, 32), sk) * 32;
  // a workgroup cannot go faster than its loads arrive through the direct global->LDS path:
  // a 32-wide stage of (bm + bn) rows costs a lone workgroup 0.13 .. 0.3 us.  A GELU epilogue
  // adds about a microsecond to such a latency-bound tile.
  static const double kStageFloorUs[NIMBLE_VAR_COUNT] = {0, 0, 0.1665, 0.161, 0.382, 0.237, 0.345};
  // time of a tile in a nearly empty last round relative to a full one
  static const double kLoneTile[NIMBLE_VAR_COUNT] = {0, 0, 0.185, 0.388, 0.678, 0.598, 0.659};
  const int64_t stages = ceil_div(k_slice, 32);
  const bool gelu = sk == 1 && epilogue == NIMBLE_EPI_BIAS_GELU_ERF;
  double us;
  // (with K this short the fixed time in the first estimate, which the second leaves out, would decide between them:
  // it is used only where all three tiles are priced by it; and only for shapes that the 64-wide ring runs)
  const bool few = v <= NIMBLE_VAR_T128x128 && tiles <= 2 * kCUs && K < kLongestFitted && (K >= 320 || batch * ceil_div(rows, 64) * ceil_div(N, 128) <= kCUs);
  if (few && N % 8 == 0 && wide_stages_ok(K, sk) && (double)N * (double)K * 2.0 <= kCachedWeightBytes) {
    us = few_tiles_us(v, tiles, stages, gelu);
  } else if (v == NIMBLE_VAR_T256x128 && bm == kHalvedRows) {  // (how the halves are priced)
    us = halved_us(tiles, stages, gelu);
  } else {
    const double latency_floor = (double)stages * kStageFloorUs[v] + (gelu ? 0.05 : 0.0);
    const double t_full = tile_cost(v, k_slice, sk > 1 ? NIMBLE_EPI_NONE : epilogue, bm) * kUsPerUnit;
    // a round is one tile per compute unit for the 8-wave tiles, two for the smaller ones
    const int64_t slots = kCUs * kTilesPerCU[v];
    const int64_t full_rounds = tiles / slots, rem = tiles % slots;
    us = (double)full_rounds * (t_full > latency_floor ? t_full : latency_floor);
    if (rem > 0) {
      const double occ = (double)rem / (double)slots;
      const double t_part = t_full * (kLoneTile[v] + (1.0 - kLoneTile[v]) * occ);
      us += t_part > latency_floor ? t_part : latency_floor;
    }
    // all workgroups together pull about 14 TB/s from the L2s into LDS with real operand data:
    // many small tiles re-fetch the operand panels often enough to hit that before anything else
    const double dma_us = (double)tiles * (double)stages * (double)((bm > 0 ? bm : vi.bm) + vi.bn) * 64.0 / 13.9e6;
    if (us < dma_us) us = dma_us;
  }
  // a layer too large to stay in the caches streams its weights from HBM: about 4.2 TB/s with
  // one workgroup per compute unit, 6.4 TB/s from two up
  if ((double)N * (double)K * 2.0 > kCachedWeightBytes) {
    double fill = (double)tiles / (double)kCUs - 1.0;
    fill = fill < 0.0 ? 0.0 : (fill > 1.0 ? 1.0 : fill);
    const double hbm_us = (double)N * (double)K * 2.0 / (4.19e6 + 2.21e6 * fill);
    if (us < hbm_us) us = hbm_us;
  }
  // the reduction: a dependent launch, a fixed cost per slice, and the partial sums' traffic
  if (sk > 1) us += kSplitGapUs + 0.259 * (double)sk + (double)(sk + 1) * (double)rows * (double)N * 4.0 / 3.97e6;
  return us;
}

// Launch-to-first-result time of one kernel, which the tiled estimates above leave out (it is
// the same for every single-launch choice) and the weight-streaming estimate includes.
static const double kLaunchUs = 3.5;

// Whether a weight-streaming launch of 16-row blocks runs the LDS-staged streaming kernel (the
// launcher applies the same test): K in whole 64-wide stages, 32-bit byte offsets into the weights.
// NIMBLE_NO_STREAM (a measurement knob) turns that kernel off in both places.
bool stream_kernel_shape_ok(int64_t N, int64_t K) {
  static const bool off = std::getenv("NIMBLE_NO_STREAM") != nullptr;
  return !off && K >= 64 && K % 64 == 0 && (uint64_t)N * (uint64_t)K * 2u < (1ull << 32);
}

// Row blocks of a weight-streaming launch: a workgroup takes 16 weight rows and 16..64
// activation rows.  Where the streaming kernel runs and the layer stays in the caches, every
// workgroup takes 16 activation rows (each block re-reads the weights, which then come from L2:
// the BERT-base and LSTM layers at 17..64 rows run 5-25 % faster that way than in blocks of 32..64
// rows on the register-layout kernel).  Otherwise: a narrow layer (few weight rows) fills the chip
// only when the activation rows are spread over several workgroups, each re-reading its weight
// rows (they meet in L2); a wide layer already has a workgroup per compute unit and keeps one block
// per 64 rows so that the weights cross HBM once.
static int64_t skinny_row_blocks(int64_t rows, int64_t N, int64_t K, bool stream_ok) {
  if (stream_ok && (double)N * (double)K * 2.0 <= kCachedWeightBytes) return rows > 16 ? ceil_div(rows, 16) : 1;
  int64_t blocks = kCUs / ceil_div(N, 16);
  const int64_t most = ceil_div(rows, 16), fewest = ceil_div(rows, 64);
  if (blocks > most) blocks = most;
  if (blocks < fewest) blocks = fewest;
  return blocks < 1 ? 1 : blocks;
}

// The weight-streaming kernels, launch latency included.
// Streaming kernel (blocks of 16 rows): whichever is longer of the weight stream and the waves'
// walk over their K stages, round of workgroups after round.  Measured: a 134 MB layer from HBM, through the caches,
// 24.0 us at 1..8 rows and 27.9 at 16 (past them 22 up to 8 rows, where nothing else is compared);
// cache-resident layers 2.5-2.8 us at K = 768..1024, 3.3-4.1 at K = 3072..4096 (0.14-0.20 us per stage of a wave's eight-way share of K); 17..64 rows on the 8 MB
// layers 3.6-4.9 us; 128 rows on 768 -> 768, 3072 -> 768 and 4096 -> 1024: 3.3, 5.7 and 6.7 us, where the
// best tile with K cut takes 6.9, 10.5 and 11.3; 256 rows on 768 -> 2304: 7.8 us (the 64-row tile 7.1).
// Register-layout kernel (any K): the activations are re-read once per 16 weight rows, which shows
// from 32 rows on; N / 16 workgroups only, so a short, wide layer leaves most of the chip idle.
// Fitted to 8 MB .. 134 MB layers at M = 1 .. 64.
static double skinny_cost_us(int64_t rows, int64_t N, int64_t K) {
  const double bytes = (double)N * (double)K * 2.0;
  const bool cached = bytes <= kCachedWeightBytes;
  if (stream_kernel_shape_ok(N, K) && (rows <= 16 || cached)) {
    // every 16-row block re-reads the weights: from L2 at about 15 TB/s when the layer is cache-resident
    const int64_t blocks16 = ceil_div(rows, 16);
    const int64_t wgs = ceil_div(N, 16) * blocks16;
    const double rate = cached ? 15e6 : (rows <= 8 ? 6.2e6 : 5.26e6);  // bytes per microsecond
    const double stream = bytes * (double)blocks16 / rate;
    double walk;
    if (wgs <= kCUs || !cached) {
      // one round of eight-wave workgroups: 0.45 us plus a wave's walk over its eighth of the K stages
      const int64_t rounds = ceil_div(wgs, kCUs);
      walk = (double)rounds * (0.45 + (double)ceil_div(ceil_div(K, 64), 8) * (rows <= 8 ? 0.14 : 0.20));
    } else {
      // four-wave workgroups, four to a compute unit: each holds its place for about 2 us plus 0.11 us per
      // stage of a wave's quarter of K
      walk = (double)wgs * (2.0 + 0.11 * (double)ceil_div(ceil_div(K, 64), 4)) / (4.0 * (double)kCUs);
      if (walk < 0.8) walk = 0.8;
    }
    const double us = kLaunchUs + (stream > walk ? stream : walk);
    // (more than the four to a compute unit that are resident: a last, partly empty round, which shows with long walks:
    // 378 x 768 x 4032 15.0 us against 12.9 in tiles with K in four, but 198 x 1536 x 576 4.6 against 5.5)
    return cached && wgs > 4 * kCUs && K >= 1024 ? 1.05 * us : us;
  }
  const int64_t nblocks = skinny_row_blocks(rows, N, K, false);
  const double mt = (double)ceil_div(rows, 16 * nblocks);
  const double blocks = (double)ceil_div(rows, 64);
  const double rate = !cached ? 5.94e6 : 6.79e6;  // bytes per microsecond
  const double stream = bytes / rate * (1.0 + 0.553 * (double)rows / (double)nblocks / 16.0);
  const double walk = (double)ceil_div(K, 128) * mt * 0.126;
  return kLaunchUs + blocks * (stream > walk ? stream : walk);
}

static bool split_k_ok(int v, int64_t batch, int64_t N, int64_t K, int sk) {
  if (sk == 1) return true;
  if (v < NIMBLE_VAR_T32x128 || batch != 1) return false;         // tiled kernels, dense only
  if (N % kVariants[v].bn != 0 || K % 32 != 0) return false;       // no ragged N/K tiles
  const int64_t stages = K / 32, per = ceil_div(stages, sk);
  return per >= 4 && per * (sk - 1) < stages;                      // every slice gets work
}

// Tuned overrides, keyed by (N, K, epilogue).
static std::map<std::tuple<int64_t, int64_t, int>, std::vector<nimble_table_entry>> g_tables;

static const nimble_table_entry* table_lookup(int64_t M, int64_t N, int64_t K, int epilogue) {
  auto it = g_tables.find(std::make_tuple(N, K, epilogue));
  if (it == g_tables.end()) return nullptr;
  for (const nimble_table_entry& e : it->second)
    if (M >= e.m_lo && M <= e.m_hi) return &e;
  return nullptr;
}

// Slice counts considered for a K split (three: 600 x 1024 x 4096 15.8 us on 64-row tiles, two 17.2, four 19.5).
static const int kSplits[] = {1, 2, 3, 4, 8, 16};

struct Launch {
  int variant = -1;
  int split_k = 1;
  int bm = 0;  // tile height when it differs from the variant's own
  bool halved = false;  // each tile is shared by two workgroups
  double us = 0;
};

// K slices for 17 to 64 rows of a layer of more than kCachedWeightBytes, in tiles of 128 columns and all rows, or 0 where the
// estimates decide: the most slices that give each compute unit one workgroup at most, from 160 workgroups on, so that each weight is
// read once and by all of the chip.  Slices of whole 4 KB are left out: then all workgroups read the same few memory
// channels (8192 x 8192 at 64 rows with K in four 36.8 us, in three 31.1).  Microseconds, several layers in turn (1 GB of them) / one over
// and over, by the estimates -> so, both through the caches, at 20, 32 and 64 rows:
//   4096 x 8192   22.4 / 19.6 -> 19.2 / 17.1   26.2 / 18.0 -> 19.4 / 17.2   23.4 / 19.4 -> 20.7 / 18.9
//   8192 x 4096   20.0 / 17.2 -> 18.0 / 15.8   20.8 / 18.0 -> 18.5 / 16.1   25.0 / 18.6 -> 19.6 / 17.7
//   6144 x 6144   23.7 / 19.0 -> 20.8 / 17.5   29.5 / 19.8 -> 21.0 / 17.9   30.5 / 21.4 -> 23.1 / 19.5
//   7168 x 7168   26.7 / 22.1 -> 24.3 / 20.9   27.3 / 22.8 -> 24.4 / 20.9   34.0 / 24.2 -> 26.4 / 22.7
//   4096 x 14336  30.6 / 26.1 -> 27.6 / 23.9   31.2 / 26.8 -> 27.6 / 24.1   36.5 / 26.9 -> 28.9 / 26.1
//   8192 x 8192   31.4 / 26.0 -> 30.5 / 24.3   32.2 / 26.5 -> 30.7 / 24.5   42.9 / 28.7 -> 32.4 / 26.1
//   5120 x 13824  37.6 / 30.7 -> 31.7 / 26.5   38.6 / 31.1 -> 31.9 / 26.8   46.8 / 33.6 -> 33.5 / 28.8
//   13824 x 5120  34.5 / 26.4 -> 32.3 / 25.1   35.3 / 27.3 -> 33.0 / 25.6   45.5 / 30.8 -> 36.1 / 27.3
//   8192 x 28672  86.1 / 85.0 -> 83.6 / 82.6   88.7 / 87.6 -> 85.4 / 84.2   95.2 / 93.4 -> 90.1 / 89.0
// (14336 x 4096, which would be cut in two of 4 KB, in turn 29.5 -> 31.3 at 20 rows.)  Which of them then load the weights past the caches
// is weights_pass_by's.
// Not to f32: fewer, longer sums are further from the exact ones there (20 x 6144 x 6144 in five slices 2.0e-7, in eight 1.6e-7),
// which a bf16 result does not show.
static int streamed_slices(int variant, int64_t rows, int64_t N, int64_t K) {
  if (rows <= 16 || rows > 64 || (double)N * (double)K * 2.0 <= kCachedWeightBytes || K % 64 != 0 || N % 128 != 0) return 0;
  const int64_t stages = K / 64;
  for (int sk = 16; sk >= 2; --sk) {
    if (N / 128 * sk > kCUs || !split_k_ok(variant, 1, N, K, sk) || !wide_stages_ok(K, sk) || ceil_div(stages, sk) % 32 == 0) continue;
    return N / 128 * sk >= 160 ? sk : 0;
  }
  return 0;
}

// Best single launch for `rows` rows: the least estimated time among weight streaming (up to
// 64 rows) and every tiled variant and K split that fits the workspace.
static Launch best_launch(int64_t batch, int64_t rows, int64_t N, int64_t K, int epilogue,
                          uint64_t max_workspace, bool allow_skinny, bool out_f32, bool allow_streamed, bool allow_halved = true) {
  Launch best, roomy;  // within the workspace, and with as much of it as anyone could bring
  double skinny_us = -1.0, least_tiled_us = 1e30;
  // weight streaming: up to 64 rows, and beyond that in 16-row blocks of the streaming kernel while
  // the layer is small enough for the blocks' re-reads to come from L2
  if (allow_skinny && batch == 1 &&
      (rows <= 64 || (rows <= 512 && stream_kernel_shape_ok(N, K) && (double)N * (double)K * 2.0 <= kCachedWeightBytes))) {
    skinny_us = skinny_cost_us(rows, N, K);
  }
  for (int v = NIMBLE_VAR_T32x128; v <= NIMBLE_VAR_T256x256; ++v) {
    if (!tiled_variant_ok(v, rows, N, K)) continue;
    if (v > NIMBLE_VAR_T32x128 && rows <= kVariants[v - 1].bm) break;  // tile taller than needed
    for (int sk : kSplits) {
      if (!split_k_ok(v, batch, N, K, sk)) continue;
      // (three slices only within the built-in scratch, so that the entry point that lives on it keeps taking
      // the calls it took when K was cut by powers of two)
      if (sk == 3 && K >= kLongestFitted) continue;
      if (sk == 3 && (uint64_t)sk * (uint64_t)rows * (uint64_t)N * 4u > (uint64_t)NIMBLE_NOALLOC_SCRATCH_BYTES) continue;
      const double us = tiled_cost_us(v, batch, rows, N, K, epilogue, sk);
      // (a finer cut takes more workspace and more of the memory's time: of the same tile, or of one of up to 128 rows
      // against a smaller tile, it has to win by more than the estimates are good for: 879 x 1024 x 6528 in 128-row
      // tiles with K in four 29.9 us, in 64-row tiles with K in two 23.1; 149 x 3712 x 6272 the same, 26.5 and 21.1)
      auto consider = [&](Launch* l) {
        const bool finer = l->split_k > 1 && K < kLongestFitted &&
                           (l->variant == v || (sk > l->split_k && v <= NIMBLE_VAR_T128x128));
        const double bar = finer ? 0.95 * l->us : l->us;
        if (l->variant < 0 || us < bar) {
          l->variant = v;
          l->split_k = sk;
          l->bm = 0;
          l->halved = false;
          l->us = us;
        }
      };
      consider(&roomy);
      if (sk > 1 && (uint64_t)sk * (uint64_t)rows * (uint64_t)N * 4u > max_workspace) continue;
      if (us < least_tiled_us) least_tiled_us = us;
      consider(&best);
    }
    // the same tile at a reduced height: with the run-time M known, pick the height at which
    // the tile rows fill whole rounds of the chip instead of leaving a mostly empty last round
    static const bool heights_on = !(std::getenv("NIMBLE_TILE_ROWS") && std::atoi(std::getenv("NIMBLE_TILE_ROWS")) == 0);
    if (v == NIMBLE_VAR_T256x128 && allow_halved && batch == 1 && heights_on && K >= 320 && K < kLongestFitted &&
        ceil_div(rows, kHalvedRows) * (N / 128) <= kCUs && tile_rows_ok(NIMBLE_VAR_T256x256, kHalvedRows, N, K) &&
        wide_stages_ok(K, 1)) {
      const double us = tiled_cost_us(v, batch, rows, N, K, epilogue, 1, kHalvedRows);
      // (not in place of K in two or three, however the estimates compare: 360 x 9216 x 11072 91.7 us, 82.3 in 128-row
      // tiles with K in two; 386 x 7424 x 4416 43.4 / 41.4.  Nor in place of 64-row tiles whose weights come from HBM, which
      // are priced too high: 234 x 12288 x 2688 28.2 / 25.8; nor of one round of 128-row tiles there: 378 x 10240 x 4288 51.6 /
      // 46.8, 336 x 9984 x 3456 with GELU 43.6 / 37.1 (8 to 17 % on 50 such shapes; of two rounds they are done in three
      // quarters of the time); nor of fewer tile rows of 256 there: 429 x 9984 x 11328 115.5 / 111.4.  In place of K in four they are faster than that and than any whole tile: 268 x 11008 x 8832 with GELU 92.7 us,
      // 113.5 in four, 115.2 in 64-row tiles; 414 x 8448 x 12096 126.7, 142.9, 136.3 in 256-row tiles; 584 x 6656 x 11072
      // 117.0, 143.7, 118.1: the least of 25 such shapes gained 1 % on whole tiles)
      const bool from_hbm = (double)N * (double)K * 2.0 > kCachedWeightBytes;
      auto kept = [&](const Launch& l) {
        return l.split_k == 2 || l.split_k == 3 || (from_hbm && l.variant == NIMBLE_VAR_T64x128) ||
               (from_hbm && l.variant == NIMBLE_VAR_T128x128 && l.split_k == 1 && ceil_div(rows, 128) * ceil_div(N, 128) <= kCUs) ||
               (from_hbm && l.variant == v && l.split_k == 1 && ceil_div(rows, kHalvedRows) > ceil_div(rows, kVariants[v].bm));
      };
      // Halves need no workspace, so they are taken or not whatever there is of it, by what they stand in place of where it
      // is plenty: the plan that is reported runs then in any workspace.  (Where that is a cut of K, they may still
      // serve callers who lack the workspace for it.)
      const Launch& instead = kept(roomy) ? best : roomy;
      if (us < instead.us && !kept(instead)) {
        best.variant = NIMBLE_VAR_T256x256;
        best.split_k = 1;
        best.bm = kHalvedRows;
        best.halved = true;
        best.us = us;
      }
    }
    if (v == NIMBLE_VAR_T256x256 && batch == 1 && heights_on)
      for (int bm : kTileRows256) {
        if (bm == kVariants[v].bm || rows <= bm || !tile_rows_ok(v, bm, N, K)) continue;
        const double us = tiled_cost_us(v, batch, rows, N, K, epilogue, 1, bm);
        if (us < best.us) {
          best.variant = v;
          best.split_k = 1;
          best.bm = bm;
          best.halved = false;
          best.us = us;
        }
      }
  }
  // up to 64 rows the small tiles (with K cut) compete with weight streaming (compared launch included, and at
  // the least of their estimates: 59 x 6656 x 2624 13.1 us with K in four, 15.5 streamed);
  // up to 16 rows the streaming kernel was the fastest choice on every layer measured
  if (skinny_us >= 0.0 && (best.variant < 0 || skinny_us <= least_tiled_us + kLaunchUs ||
                           (rows <= 16 && stream_kernel_shape_ok(N, K)))) {
    best = Launch();
    best.variant = NIMBLE_VAR_SKINNY16;
    best.us = skinny_us;
  }
  // (in place of another cut of K only: what ran without scratch still does)
  const int tile = rows <= 32 ? NIMBLE_VAR_T32x128 : NIMBLE_VAR_T64x128;
  const int slices = batch == 1 && best.split_k > 1 && allow_streamed && !out_f32 ? streamed_slices(tile, rows, N, K) : 0;
  if (slices > 1 && tiled_variant_ok(tile, rows, N, K) && (uint64_t)slices * (uint64_t)rows * (uint64_t)N * 4u <= max_workspace) {
    best.variant = tile;  // (its estimate stays: nothing is compared with it, 64 rows are never split)
    best.split_k = slices;
    best.bm = 0;
    best.halved = false;
  }
  return best;
}

static void fill_tiled(nimble_plan* p, int variant, int split_k, int64_t batch, int64_t M, int64_t N,
                       int64_t K, int bm = 0) {
  VariantInfo v = kVariants[variant];
  if (bm > 0) v.bm = bm;
  p->variant = variant;
  p->bm = v.bm;
  p->bn = v.bn;
  p->bk = v.bk;
  p->k = M / v.bm;
  p->r = (int32_t)(M % v.bm);
  p->residue_copy = (p->r != 0 || N % v.bn != 0 || K % v.bk != 0) ? 1 : 0;
  p->split_k = split_k;
  p->grid[0] = (uint32_t)(ceil_div(M, v.bm) * ceil_div(N, v.bn));
  p->grid[1] = (uint32_t)split_k;
  p->grid[2] = (uint32_t)batch;
  const int64_t tiles = (int64_t)p->grid[0] * batch;
  if (ring_shape_ok(N, K) && quarter_kernel_wins(v.bm, v.bn, tiles, K, split_k, batch))
    p->block = 256;
  else
    p->block = eight_waves(variant, (uint64_t)tiles * p->grid[1], K, split_k) ? 512u : (uint32_t)v.threads;
  p->workspace_bytes = split_k > 1 ? (uint64_t)split_k * (uint64_t)M * (uint64_t)N * 4u : 0;
}

// Makes `p` a launch of any_kernel: 64 x 64 tiles.
static void fill_any(nimble_plan* p, int64_t batch, int64_t M, int64_t N, int64_t K, bool b_is_kn) {
  const int64_t tiles_m = ceil_div(M, 64), tiles_n = ceil_div(N, 64), tiles = tiles_m * tiles_n;
  p->bm = p->bn = p->bk = 64;
  p->k = M / 64;
  p->r = (int32_t)(M % 64);
  p->residue_copy = 1;
  p->split_k = 1;
  p->grid[0] = (uint32_t)tiles;
  p->grid[1] = 1;
  if (tiles > 0) {
    int64_t tm, tn;
    any_launch_tiles(tiles_m, tiles_n, &tm, &tn);
    p->grid[0] = (uint32_t)(tm * tn);
    p->grid[1] = (uint32_t)(ceil_div(tiles_m, tm) * ceil_div(tiles_n, tn));  // launches, 1 but for outputs of over 17 G elements
  }
  p->grid[2] = (uint32_t)batch;
  p->block = any_four_groups(tiles * batch, K, b_is_kn) ? 1024u : 256u;
}

int plan_dense(int64_t batch, int64_t M, int64_t N, int64_t K, int epilogue, int force_variant,
               const PlanOptions& opt, nimble_plan* p) {
  std::memset(p, 0, sizeof(*p));
  p->residue_variant = NIMBLE_VAR_AUTO;
  if (M < 0 || N < 0 || K < 0 || batch < 0) return fail(NIMBLE_ERR_ARG, "negative extent");
  if (M > (1ll << 30) || N > (1ll << 30) || K > (1ll << 30) || batch > 65535)
    return fail(NIMBLE_ERR_ARG, "extent too large");
  if (M * N > (1ll << 40)) return fail(NIMBLE_ERR_ARG, "output too large");
  int variant = force_variant;
  if (variant == NIMBLE_VAR_AUTO) {
    // measurement knob, read once: a force_variant value applied to every automatic plan
    static const int env_variant = [] {
      const char* env = std::getenv("NIMBLE_FORCE_VARIANT");
      return (env && *env) ? std::atoi(env) : (int)NIMBLE_VAR_AUTO;
    }();
    variant = env_variant;
  }
  const bool forced = variant != NIMBLE_VAR_AUTO;
  // a forced variant may carry a forced K split in bits 8..15 (NIMBLE_FORCE_SPLIT_K) and a
  // forced tile height in bits 16..23 (NIMBLE_FORCE_TILE_ROWS)
  int forced_sk = opt.force_split_k;
  int tile_rows = 0;
  if (variant >= 0) {
    if ((variant >> 8) & 0xff) forced_sk = (variant >> 8) & 0xff;
    tile_rows = ((variant >> 16) & 0xff) * 16;
    variant &= 0xff;
  }
  if (variant < NIMBLE_VAR_AUTO || variant >= NIMBLE_VAR_COUNT)
    return fail(NIMBLE_ERR_ARG, "unknown variant %d", variant);

  const bool aligned_k = (K > 0 && K % 8 == 0);
  int64_t split_rows = 0;
  int residue_variant = NIMBLE_VAR_AUTO;
  int split_k = 1;
  bool halved = false;
  bool chosen = forced;  // by the caller or a tuned entry: launched as named
  if (variant == NIMBLE_VAR_AUTO) {
    if (!aligned_k || M == 0 || N == 0) {
      variant = NIMBLE_VAR_GENERIC;
    } else if (const nimble_table_entry* e = (batch == 1 && opt.use_table) ? table_lookup(M, N, K, epilogue) : nullptr;
               e && (e->variant == NIMBLE_VAR_SKINNY16 ||
                     (tiled_variant_ok(e->variant, M, N, K) && split_k_ok(e->variant, 1, N, K, e->split_k) &&
                      (e->split_k <= 1 ||
                       (uint64_t)e->split_k * (uint64_t)M * (uint64_t)N * 4u <= opt.max_workspace)))) {
      variant = e->variant;  // tuned: one launch of this configuration
      chosen = true;
      split_k = e->split_k > 1 ? e->split_k : 1;
    } else {
      // (streamed_slices was measured on calls of their own: the rest of a row split, whose weights the first launch has just read, goes
      // by the estimates with which the split is decided)
      const Launch single = best_launch(batch, M, N, K, epilogue, opt.max_workspace, true, opt.out_f32, opt.allow_row_split);
      variant = single.variant < 0 ? NIMBLE_VAR_GENERIC : single.variant;
      split_k = single.split_k;
      tile_rows = single.bm;
      halved = single.halved;
      // Alternative: two launches.  Whole tile rows (all k of them, or as many as fill whole
      // rounds of the chip) run the r = 0 copy of a big-tile variant: no bounds code, no
      // partial round.  The remaining rows, residue included, run whatever suits their
      // number.  Taken when the estimate beats the best single launch.
      if (opt.allow_row_split && variant >= NIMBLE_VAR_T32x128 && batch == 1) {
        double best_us = single.us;
        for (int v = NIMBLE_VAR_T128x128; v <= NIMBLE_VAR_T256x256; ++v) {
          const VariantInfo& vi = kVariants[v];
          if (N % vi.bn != 0 || K % vi.bk != 0) continue;
          const int64_t tiles_n = N / vi.bn;
          int64_t cuts[2] = {(M / vi.bm) * vi.bm, 0};
          const int64_t slots = kCUs * kTilesPerCU[v];
          if (slots % tiles_n == 0) {
            const int64_t rows_per_round = (slots / tiles_n) * vi.bm;
            cuts[1] = (M / rows_per_round) * rows_per_round;
          }
          for (int c = 0; c < 2; ++c) {
            const int64_t head = cuts[c], rest = M - head;
            if (head <= 0 || rest <= 0 || (c == 1 && head == cuts[0])) continue;
            const double head_us = tiled_cost_us(v, 1, head, N, K, epilogue) + kLaunchGapUs;
            if (head_us >= best_us) continue;  // (the tail's search is most of what a plan costs)
            // (priced without halved tiles: two launches picked for their sake took 1 to 2 % longer than one:
            // 4751 x 8192 x 7552 426.9 us, 417.7 in 320-row tiles)
            const Launch tail = best_launch(1, rest, N, K, epilogue, opt.max_workspace, true, opt.out_f32, false, false);
            if (tail.variant < 0) continue;
            // (a streamed tail's estimate and the gap both count its launch, which decides against halved tiles at
            // K > 2048: 4154 x 1024 x 3648 with GELU 36.6 us in two launches, 38.8 in halves)
            const bool twice = halved && tail.variant == NIMBLE_VAR_SKINNY16 && K > 2048;
            const double us = head_us + tail.us - (twice ? kLaunchUs + 1.0 : 0.0);
            if (us < best_us) {
              best_us = us;
              variant = v;
              split_k = 1;
              tile_rows = 0;
              halved = false;
              split_rows = head;
              residue_variant = tail.variant;
            }
          }
        }
      }
    }
  }

  if (variant == NIMBLE_VAR_GENERIC) {
    // Any shape and alignment.  A grid of at most two workgroups per compute unit, or a single block of
    // rows, streams both operands in 16 x 16 blocks whose waves share K; everything else runs in 64 x 64
    // tiles (any_kernel).  With K odd the blocks' loads of rows that start at odd elements take three times as long, and from some
    // length on the second workgroup of a compute unit is not worth it: on 120 shapes of 257 to 512 blocks tiles took, over blocks, 1.22
    // at K = 257 ... 320, 1.11 to 384, 1.05 to 512, 1.11 to 570, 0.92 from 571 to 704, 0.85 to 896, 0.75 to 1150.  Microseconds, blocks /
    // tiles: 52 x 1397 x 261 3.9 / 5.1, 28 x 2593 x 335 4.5 / 5.4, 226 x 413 x 499 5.7 / 6.5, 50 x 1079 x 523 5.1 / 6.4, 760 x 112 x 583
    // 6.4 / 6.2, 82 x 1265 x 635 7.1 / 6.5, 114 x 1024 x 979 10.0 / 8.0, 80 and 128 x 1001 x 1003 10.0 / 8.3 and 10.2 / 8.4, 154 x 487 x
    // 1121 11.5 / 8.5.  One block per compute unit: 64 x 1001 x 1003 (252) 6.3 / 8.3, 192 x 333 x 1399 8.4 / 9.8; K even: 64 and 128 x 1001 x
    // 1002 3.7 / 7.3 and 4.5 / 7.4.
    const int64_t cols16 = ceil_div(N, 16), rows16 = ceil_div(M, 16);
    const bool rows = opt.generic_rows && batch == 1 && K > 0 && rows16 <= 65535 &&
                      (rows16 <= 1 || cols16 * rows16 <= (K % 2 != 0 && K > 576 ? 1 : 2) * kCUs);
    p->variant = variant;
    fill_any(p, batch, M, N, K, !opt.generic_rows);
    if (rows) {
      p->bm = p->bn = 16;
      p->bk = 32;
      p->k = M / 16;
      p->r = (int32_t)(M % 16);
      p->grid[0] = (uint32_t)cols16;
      p->grid[1] = (uint32_t)rows16;
      p->block = 256;
    }
    return NIMBLE_OK;
  }
  if (variant == NIMBLE_VAR_SKINNY16) {
    if (!aligned_k) return fail(NIMBLE_ERR_ARG, "skinny16 needs K %% 8 == 0");
    if (batch != 1) return fail(NIMBLE_ERR_ARG, "skinny16 is not batched");
    const VariantInfo& v = kVariants[variant];
    p->variant = variant;
    p->bm = v.bm;
    p->bn = v.bn;
    p->bk = v.bk;
    p->k = M / v.bm;
    p->r = (int32_t)(M % v.bm);
    p->residue_copy = (p->r != 0 || N % v.bn != 0 || K % v.bk != 0) ? 1 : 0;
    p->grid[0] = (uint32_t)ceil_div(N, v.bn);
    p->grid[1] = (uint32_t)skinny_row_blocks(M, N, K, stream_kernel_shape_ok(N, K));  // up to four 16-row tiles per workgroup
    p->grid[2] = 1;
    // the waves of a workgroup split K among them: eight in the streaming kernel (16-row blocks,
    // 64-wide stages; four when a cache-resident layer gives more workgroups than compute units),
    // four in the register-layout kernel
    const bool streaming = stream_kernel_shape_ok(N, K) && ceil_div(M, (int64_t)p->grid[1]) <= 16;
    const bool many = (uint64_t)p->grid[0] * p->grid[1] > (uint64_t)kCUs && (double)N * (double)K * 2.0 <= kCachedWeightBytes;
    p->split_k = streaming && !many ? 8 : 4;
    p->bk = streaming ? 64 : v.bk;
    p->block = streaming && !many ? 512 : 256;
    return NIMBLE_OK;
  }
  if (!tiled_variant_ok(variant, M, N, K))
    return fail(NIMBLE_ERR_ARG, "variant %s cannot run K=%lld", kVariants[variant].name, (long long)K);
  if (!tile_rows_ok(variant, tile_rows, N, K))
    return fail(NIMBLE_ERR_ARG, "variant %s is not built with tiles of %d rows for N=%lld K=%lld",
                kVariants[variant].name, tile_rows, (long long)N, (long long)K);
  if (tile_rows > 0 && tile_rows != kVariants[variant].bm && forced_sk > 1)
    return fail(NIMBLE_ERR_ARG, "a reduced tile height cannot be combined with a K split");
  if (forced && forced_sk > 0) {
    if (!split_k_ok(variant, batch, N, K, forced_sk))
      return fail(NIMBLE_ERR_ARG, "variant %s cannot cut K=%lld into %d slices", kVariants[variant].name,
                  (long long)K, forced_sk);
    if (forced_sk > 1 && (uint64_t)forced_sk * (uint64_t)M * (uint64_t)N * 4u > opt.max_workspace)
      return fail(NIMBLE_ERR_WORKSPACE, "cutting K into %d slices needs %llu bytes of workspace", forced_sk,
                  (unsigned long long)((uint64_t)forced_sk * (uint64_t)M * (uint64_t)N * 4u));
    split_k = forced_sk;
  }
  fill_tiled(p, variant, split_k, batch, split_rows > 0 ? split_rows : M, N, K, tile_rows);
  if (halved) p->grid[1] = 2, p->block = 512;
  if (!chosen && split_rows == 0 &&
      small_tiles_win(variant, (int64_t)p->grid[0] * batch, batch * ceil_div(M, 64) * ceil_div(N, 64), p->bn, N, K, opt.out_f32))
    fill_any(p, batch, M, N, K, !opt.generic_rows);
  if (split_rows > 0) {
    // k and r describe the whole call; grid and residue_copy describe the first launch; the second
    // launch is planned here exactly as the entry point plans it, so that what is reported (its
    // variant, its K split, the scratch the call needs) is what runs
    PlanOptions tail_opt = opt;
    tail_opt.allow_row_split = false;
    nimble_plan tail;
    const int rc = plan_dense(1, M - split_rows, N, K, epilogue, NIMBLE_VAR_AUTO, tail_opt, &tail);
    if (rc != NIMBLE_OK) return rc;
    p->k = M / p->bm;
    p->r = (int32_t)(M % p->bm);
    p->split_rows = split_rows;
    p->residue_variant = tail.variant;
    p->residue_split_k = tail.split_k;
    if (tail.workspace_bytes > p->workspace_bytes) p->workspace_bytes = tail.workspace_bytes;
    (void)residue_variant;
  }
  return NIMBLE_OK;
}

// One launch of any_kernel, microseconds: a lone tile's walk over its stages of 64 k (a quarter of them where four
// groups of waves share it), or what a compute unit's tiles take one behind the other; b [K, N] takes longer than [N, K].
static double any_cost_us(int64_t batch, int64_t M, int64_t N, int64_t K, bool b_is_kn) {
  const int64_t tiles = batch * ceil_div(M, 64) * ceil_div(N, 64), stages = ceil_div(K, 64);
  const bool four = K >= 512 && tiles <= kCUs;  // (the [N, K] form too: with fewer stages one group's price still holds as an upper bound)
  const double deep = (double)(four ? ceil_div(stages, 4) : stages);
  double per_cu = (double)tiles / (double)kCUs;
  if (per_cu > 1.0 && per_cu < 2.0) per_cu = 2.0;
  double lone, many;
  if (b_is_kn) {
    lone = four ? 3.5 + 1.14 * deep : 3.0 + 0.67 * deep;
    many = 3.0 + per_cu * (0.6 + 0.42 * (double)stages);
  } else {
    lone = four ? 3.2 + 1.28 * deep : 4.0 + 0.56 * deep;
    many = 4.0 + per_cu * (0.69 + 0.27 * (double)stages);
  }
  return lone > many ? lone : many;
}

// Whether the product A.B with b [K, N] is done sooner by the launch `p` on b transposed (a graph node more, and 0.3
// microseconds per megabyte of b written and read back) than by any_kernel on b as it is.  The tiled estimates leave
// out the launch and what the operands take to memory and back, which counts for short K; the tile kernel for
// shapes that the ring kernels cannot run takes twice their time.  Checked on 290 products of 30 M to 40 G
// multiply-adds, 1 .. 96 batches: the choice costs 0.6 % over the better one of each.  any_kernel / transposed, microseconds:
// 12 x 512 x 64 x 512 6.1 / 13.2, 1 x 1000^3 9.9 / 20.4, 96 x 512 x 64 x 512 20 / 27, 24 x 1151 x 320 x 256 19 / 23;
// 1 x 4096 x 1024 x 512 15.5 / 13.0, 8 x 1000^3 56 / 48, 1 x 2048 x 2048 x 2040 62 / 51, 4 x 1905 x 2048 x 1408 123 / 62; in
// halved tiles 1 x 480 x 8448 x 1344 41 / 33, 1 x 661 x 6400 x 768 26 / 22, 1 x 370 x 10240 x 6400 205 / 178.
bool nn_transposes(const nimble_plan& p, int64_t batch, int64_t M, int64_t N, int64_t K) {
  double us = 8.0 + 0.3e-6 * (double)(batch * N * K * 2);
  if (p.bn == 64) {
    us += any_cost_us(batch, M, N, K, false) - 2.5;
  } else {
    // (tiles that two workgroups share have a price of their own, which is under the variant of half the width)
    const bool halved = p.variant == NIMBLE_VAR_T256x256 && p.bm == kHalvedRows && p.split_k == 1 && p.grid[1] == 2;
    const double tiled = tiled_cost_us(halved ? (int)NIMBLE_VAR_T256x128 : p.variant, batch, M, N, K, NIMBLE_EPI_NONE, 1, p.bm);
    us += (ring_shape_ok(N, K) ? tiled : 2.0 * tiled) + 0.12e-6 * (double)(batch * (M * K + N * K + M * N) * 2);
  }
  return us < any_cost_us(batch, M, N, K, true);
}

static size_t dtype_size(int dtype) {
  switch (dtype) {
    case NIMBLE_BF16: return 2;
    case NIMBLE_F32: return 4;
    default: return 0;
  }
}

}  // namespace nimble

using namespace nimble;

extern "C" {

int nimble_dense_shape(const int64_t* x_shape, int x_rank, const int64_t* w_shape, int w_rank,
                       int64_t* out_shape) {
  clear_error();
  if (!x_shape || !w_shape || !out_shape) return fail(NIMBLE_ERR_NULL, "null shape pointer");
  if (x_rank != 2 || w_rank != 2)
    return fail(NIMBLE_ERR_RANK, "dense expects ranks (2,2), got (%d,%d)", x_rank, w_rank);
  if (x_shape[0] < 0 || x_shape[1] < 0 || w_shape[0] < 0 || w_shape[1] < 0)
    return fail(NIMBLE_ERR_ARG, "negative extent");
  if (x_shape[1] != w_shape[1])
    return fail(NIMBLE_ERR_SHAPE, "dense: K of x (%lld) != K of w (%lld)", (long long)x_shape[1],
                (long long)w_shape[1]);
  out_shape[0] = x_shape[0];
  out_shape[1] = w_shape[0];
  return NIMBLE_OK;
}

int nimble_batch_matmul_shape(const int64_t* a_shape, int a_rank, const int64_t* b_shape,
                              int b_rank, int trans_b, int64_t* out_shape) {
  clear_error();
  if (!a_shape || !b_shape || !out_shape) return fail(NIMBLE_ERR_NULL, "null shape pointer");
  if (a_rank != 3 || b_rank != 3)
    return fail(NIMBLE_ERR_RANK, "batch_matmul expects ranks (3,3), got (%d,%d)", a_rank, b_rank);
  for (int i = 0; i < 3; ++i)
    if (a_shape[i] < 0 || b_shape[i] < 0) return fail(NIMBLE_ERR_ARG, "negative extent");
  const int64_t kb = trans_b ? b_shape[2] : b_shape[1];
  const int64_t nb = trans_b ? b_shape[1] : b_shape[2];
  if (a_shape[0] != b_shape[0])
    return fail(NIMBLE_ERR_SHAPE, "batch_matmul: batch %lld != %lld", (long long)a_shape[0],
                (long long)b_shape[0]);
  if (a_shape[2] != kb)
    return fail(NIMBLE_ERR_SHAPE, "batch_matmul: K %lld != %lld", (long long)a_shape[2], (long long)kb);
  out_shape[0] = a_shape[0];
  out_shape[1] = a_shape[1];
  out_shape[2] = nb;
  return NIMBLE_OK;
}

int nimble_lstm_shape(const int64_t* x_shape, const int64_t* h_shape, const int64_t* c_shape,
                      const int64_t* w_shape, int64_t* h_out_shape, int64_t* c_out_shape) {
  clear_error();
  if (!x_shape || !h_shape || !c_shape || !w_shape || !h_out_shape || !c_out_shape)
    return fail(NIMBLE_ERR_NULL, "null shape pointer");
  for (int i = 0; i < 2; ++i)
    if (x_shape[i] < 0 || h_shape[i] < 0 || c_shape[i] < 0 || w_shape[i] < 0)
      return fail(NIMBLE_ERR_ARG, "negative extent");
  const int64_t B = x_shape[0], Ix = x_shape[1], H = h_shape[1];
  if (h_shape[0] != B || c_shape[0] != B) return fail(NIMBLE_ERR_SHAPE, "lstm: batch extents differ");
  if (c_shape[1] != H) return fail(NIMBLE_ERR_SHAPE, "lstm: c is not (B,H)");
  if (w_shape[0] != 4 * H || w_shape[1] != Ix + H)
    return fail(NIMBLE_ERR_SHAPE, "lstm: w is not (4H, Ix+H)");
  h_out_shape[0] = c_out_shape[0] = B;
  h_out_shape[1] = c_out_shape[1] = H;
  return NIMBLE_OK;
}

int nimble_lstm_pre_shape(const int64_t* pre_shape, const int64_t* h_shape, const int64_t* c_shape,
                          const int64_t* wh_shape, int64_t* h_out_shape, int64_t* c_out_shape) {
  clear_error();
  if (!pre_shape || !h_shape || !c_shape || !wh_shape || !h_out_shape || !c_out_shape)
    return fail(NIMBLE_ERR_NULL, "null shape pointer");
  for (int i = 0; i < 2; ++i)
    if (pre_shape[i] < 0 || h_shape[i] < 0 || c_shape[i] < 0 || wh_shape[i] < 0)
      return fail(NIMBLE_ERR_ARG, "negative extent");
  const int64_t B = h_shape[0], H = h_shape[1];
  if (pre_shape[0] != B || c_shape[0] != B) return fail(NIMBLE_ERR_SHAPE, "lstm: batch extents differ");
  if (pre_shape[1] != 4 * H) return fail(NIMBLE_ERR_SHAPE, "lstm: pre is not (B,4H)");
  if (c_shape[1] != H) return fail(NIMBLE_ERR_SHAPE, "lstm: c is not (B,H)");
  if (wh_shape[0] != 4 * H || wh_shape[1] != H) return fail(NIMBLE_ERR_SHAPE, "lstm: w_h is not (4H,H)");
  h_out_shape[0] = c_out_shape[0] = B;
  h_out_shape[1] = c_out_shape[1] = H;
  return NIMBLE_OK;
}

int nimble_lstm_seq_shape(const int64_t* pre_shape, const int64_t* h0_shape, const int64_t* c0_shape,
                          const int64_t* wh_shape, int64_t* h_seq_shape, int64_t* c_out_shape) {
  clear_error();
  if (!pre_shape || !h0_shape || !c0_shape || !wh_shape || !h_seq_shape || !c_out_shape)
    return fail(NIMBLE_ERR_NULL, "null shape pointer");
  for (int i = 0; i < 3; ++i)
    if (pre_shape[i] < 0) return fail(NIMBLE_ERR_ARG, "negative extent");
  for (int i = 0; i < 2; ++i)
    if (h0_shape[i] < 0 || c0_shape[i] < 0 || wh_shape[i] < 0) return fail(NIMBLE_ERR_ARG, "negative extent");
  const int64_t T = pre_shape[0], B = h0_shape[0], H = h0_shape[1];
  if (pre_shape[1] != B || c0_shape[0] != B) return fail(NIMBLE_ERR_SHAPE, "lstm sequence: batch extents differ");
  if (pre_shape[2] != 4 * H) return fail(NIMBLE_ERR_SHAPE, "lstm sequence: pre is not (T,B,4H)");
  if (c0_shape[1] != H) return fail(NIMBLE_ERR_SHAPE, "lstm sequence: c0 is not (B,H)");
  if (wh_shape[0] != 4 * H || wh_shape[1] != H) return fail(NIMBLE_ERR_SHAPE, "lstm sequence: w_h is not (4H,H)");
  h_seq_shape[0] = T;
  h_seq_shape[1] = c_out_shape[0] = B;
  h_seq_shape[2] = c_out_shape[1] = H;
  return NIMBLE_OK;
}

int nimble_lstm_seq_supported(int64_t B, int64_t H) {
  return B >= 1 && B <= 4 && H >= 64 && H <= 1024 && (H % 64) == 0;
}

// A fixed rule, kept as callers know it: drawn when the loop took 2.4 microseconds per step at H = 512 with 4 rows and 2.7 / 4.0
// at H = 1024 with 1 / 4, against 2.65-2.95 for a captured graph of per-step launches.  It takes 1.0 and 1.5 / 1.5 now.
int nimble_lstm_seq_preferred(int64_t B, int64_t H) {
  return nimble_lstm_seq_supported(B, H) && (H <= 512 || B == 1);
}

size_t nimble_lstm_seq_workspace_bytes(int64_t B, int64_t H) {
  if (!nimble_lstm_seq_supported(B, H)) return 0;
  return 256 + 2 * (size_t)B * (size_t)H * 4;
}

// Weights in registers: at most two 64-wide K stages per wave, each wholly of x or of h.  Groups of 8 rows, each on the H / 16
// workgroups of one XCD (two above H = 512), one workgroup per compute unit at a time and four rounds of them
// (microseconds for 64 steps, loop / captured launches: H = Ix = 512 at 64, 128, 256 rows 119 / 241, 196 / 338, 369 / 556;
// H = 1024 with the inputs' product ahead at 40, 128 rows 262 / 355, 533 / 701; 32 steps of 512 rows at 256 175 / 218).
int nimble_lstm_loop_supported(int64_t B, int64_t Ix, int64_t H) {
  if (B < 1 || B > 65536 || H < 64 || H > 1024 || H % 64 != 0 || Ix < 0 || Ix > 1024 || Ix % 64 != 0) return 0;
  const int64_t stages = (Ix + H) / 64, per_wave = ceil_div(stages, 8);
  if (per_wave > 2 || Ix / 64 % per_wave != 0) return 0;
  // (where the per-step launch runs four waves the loop takes the sums over four ranges, of two or four whole stages)
  nimble_plan p;
  if (nimble_lstm_plan(B, Ix, H, &p) != NIMBLE_OK || (p.split_k == 4 && stages != 8 && stages != 16)) return 0;
  const int64_t n_wg = H / 16, span = n_wg > 32 ? 2 : 1;
  return ceil_div(ceil_div(B, 8) * span, 8) * (n_wg / span) <= 4 * (kCUs / 8);
}

// What the loop costs before its first step, some 15 us and 8 for each further launch, has to be earned.  Microseconds for 4, 6,
// 8, 12, 16 steps, loop / captured launches: H = Ix = 512, 1 row 22.7 / 18.2, 24.8 / 23.9, 27.4 / 29.3, 30.8 / 40.4, -; 64 rows
// 25.0 / 21.0, 27.1 / 28.4, 29.8 / 35.8, 34.5 / 50.9, -; two launches: 65 rows -, 40.8 / 31.9, 45.8 / 40.4, 55.2 / 57.9, 65.9 / 75.5,
// H = 1024 33 rows -, 51.9 / 43.5, 58.1 / 54.0, 72.7 / 73.1, 89.7 / 96.5; four: 256 rows -, -, 84.9 / 73.9, 104 / 108, 124 / 143,
// 512 of 256 -, -, 71.2 / 59.4, 88.0 / 84.6, 106 / 111.
int nimble_lstm_loop_preferred(int64_t T, int64_t B, int64_t Ix, int64_t H) {
  if (!nimble_lstm_loop_supported(B, Ix, H) || T > (int64_t)1 << 24) return 0;  // (nimble_lstm_loop_dyn takes no more steps)
  const int64_t launches = ceil_div(ceil_div(B, 8), lstm_groups_per_launch(H));
  return T >= (launches == 1 ? 7 : 8 + 2 * launches);
}

size_t nimble_lstm_loop_workspace_bytes(int64_t B, int64_t Ix, int64_t H) {
  if (!nimble_lstm_loop_supported(B, Ix, H)) return 0;
  return 256 + (size_t)(ceil_div(B, 8) * 8 + B) * (size_t)H * 4;
}

int64_t nimble_storage_bytes(const int64_t* shape, int rank, int dtype) {
  clear_error();
  if (rank < 0 || (rank > 0 && !shape)) return fail(NIMBLE_ERR_NULL, "null shape pointer");
  const size_t es = dtype_size(dtype);
  if (es == 0) return fail(NIMBLE_ERR_DTYPE, "unknown dtype %d", dtype);
  int64_t n = 1;
  for (int i = 0; i < rank; ++i) {
    if (shape[i] < 0) return fail(NIMBLE_ERR_ARG, "negative extent");
    if (shape[i] != 0 && n > std::numeric_limits<int64_t>::max() / (8 * shape[i]))
      return fail(NIMBLE_ERR_ARG, "size overflows int64");
    n *= shape[i];
  }
  return n * (int64_t)es;
}

int64_t nimble_storage_alignment(void) { return 64; }

int nimble_residue_split(int64_t x, int64_t tile, int64_t* k, int64_t* r) {
  clear_error();
  if (!k || !r) return fail(NIMBLE_ERR_NULL, "null output pointer");
  if (x < 0 || tile <= 0) return fail(NIMBLE_ERR_ARG, "need x >= 0 and tile > 0");
  *k = x / tile;
  *r = x % tile;
  return NIMBLE_OK;
}

int nimble_dense_plan(int64_t M, int64_t N, int64_t K, int epilogue, int out_dtype,
                      int force_variant, nimble_plan* plan) {
  clear_error();
  if (!plan) return fail(NIMBLE_ERR_NULL, "null plan");
  if (epilogue < NIMBLE_EPI_NONE || epilogue > NIMBLE_EPI_BIAS_GELU_ERF)
    return fail(NIMBLE_ERR_ARG, "unknown epilogue %d", epilogue);
  if (dtype_size(out_dtype) == 0) return fail(NIMBLE_ERR_DTYPE, "unknown dtype %d", out_dtype);
  PlanOptions opt;
  opt.max_workspace = ~0ull;  // report the plan for a caller that provides what it asks for
  opt.out_f32 = out_dtype == NIMBLE_F32;
  return plan_dense(1, M, N, K, epilogue, force_variant, opt, plan);
}

int nimble_dense_table_set(int64_t N, int64_t K, int epilogue, const nimble_table_entry* entries,
                           int count) {
  clear_error();
  if (N < 0 || K < 0 || count < 0) return fail(NIMBLE_ERR_ARG, "negative argument");
  if (epilogue < NIMBLE_EPI_NONE || epilogue > NIMBLE_EPI_BIAS_GELU_ERF)
    return fail(NIMBLE_ERR_ARG, "unknown epilogue %d", epilogue);
  const auto key = std::make_tuple(N, K, epilogue);
  if (count == 0) {
    g_tables.erase(key);
    return NIMBLE_OK;
  }
  if (!entries) return fail(NIMBLE_ERR_NULL, "null table");
  std::vector<nimble_table_entry> t;
  for (int i = 0; i < count; ++i) {
    const nimble_table_entry& e = entries[i];
    if (e.m_lo < 0 || e.m_hi < e.m_lo) return fail(NIMBLE_ERR_ARG, "entry %d: bad M range", i);
    if (e.variant < NIMBLE_VAR_SKINNY16 || e.variant >= NIMBLE_VAR_COUNT)
      return fail(NIMBLE_ERR_ARG, "entry %d: variant %d cannot be tabled", i, e.variant);
    if (e.split_k < 0 || e.split_k > 64) return fail(NIMBLE_ERR_ARG, "entry %d: bad split_k", i);
    if (e.variant == NIMBLE_VAR_SKINNY16 && e.m_hi > 64 && !stream_kernel_shape_ok(N, K))
      return fail(NIMBLE_ERR_ARG, "entry %d: skinny16 serves M <= 64 unless K is whole 64-wide stages", i);
    t.push_back(e);
  }
  g_tables[key] = t;
  return NIMBLE_OK;
}

int nimble_batch_matmul_plan(int64_t batch, int64_t M, int64_t N, int64_t K, int trans_b,
                             int out_dtype, nimble_plan* plan) {
  clear_error();
  if (!plan) return fail(NIMBLE_ERR_NULL, "null plan");
  if (dtype_size(out_dtype) == 0) return fail(NIMBLE_ERR_DTYPE, "unknown dtype %d", out_dtype);
  // batch_matmul is always one launch over all rows: no row split (its entry point launches the
  // plan as it stands), no K split (no reduction pass for batches), no tuned dense table
  PlanOptions bmm;
  bmm.allow_row_split = false;
  bmm.use_table = false;
  bmm.generic_rows = trans_b != 0;
  bmm.out_f32 = out_dtype == NIMBLE_F32;
  if (!trans_b) {
    // b is (T,K,N): its rows are not K-contiguous.  Where the tiled kernels could run the product
    // on b transposed (K a multiple of 8 and whole 16-byte batch strides) from about 32 M multiply-adds on,
    // the plan is that NT launch and its workspace is the transposed copy of b, unless any_kernel, which reads b
    // as it is, is done sooner: then the plan is in its 64 x 64 tiles.  The entry point runs any_kernel on b as it
    // is too when the caller brings less workspace.
    if (K > 0 && K % 8 == 0 && ((M * K) & 7) == 0 && ((N * K) & 7) == 0 && batch > 0 && M > 0 && N > 0 &&
        (double)batch * (double)M * (double)N * (double)K >= 32e6) {
      int rc = plan_dense(batch, M, N, K, NIMBLE_EPI_NONE, NIMBLE_VAR_AUTO, bmm, plan);
      if (rc != NIMBLE_OK) return rc;
      if (plan->variant >= NIMBLE_VAR_T32x128) {
        plan->workspace_bytes = (uint64_t)batch * (uint64_t)N * (uint64_t)K * 2u;
        if (!nn_transposes(*plan, batch, M, N, K)) fill_any(plan, batch, M, N, K, true);
        return NIMBLE_OK;
      }
    }
    return plan_dense(batch, M, N, K, NIMBLE_EPI_NONE, NIMBLE_VAR_GENERIC, bmm, plan);
  }
  return plan_dense(batch, M, N, K, NIMBLE_EPI_NONE, NIMBLE_VAR_AUTO, bmm, plan);
}

int nimble_lstm_plan(int64_t B, int64_t Ix, int64_t H, nimble_plan* plan) {
  clear_error();
  if (!plan) return fail(NIMBLE_ERR_NULL, "null plan");
  std::memset(plan, 0, sizeof(*plan));
  if (B < 0 || Ix < 0 || H < 0) return fail(NIMBLE_ERR_ARG, "negative extent");
  if (Ix % 8 != 0 || H % 8 != 0 || H == 0)
    return fail(NIMBLE_ERR_ARG, "lstm needs Ix and H to be multiples of 8 (H > 0)");
  if (B > (1ll << 24) || Ix > (1ll << 24) || H > (1ll << 24)) return fail(NIMBLE_ERR_ARG, "extent too large");
  plan->variant = NIMBLE_VAR_SKINNY16;
  plan->bm = 16;
  plan->bn = 16;  // four hidden units times four gates
  plan->bk = 32;
  plan->k = B / 16;
  plan->r = (int32_t)(B % 16);
  plan->residue_copy = plan->r != 0;
  plan->split_k = 4;
  plan->grid[0] = (uint32_t)ceil_div(H, 4);
  // row blocks as for the weight-streaming dense (4H weight rows; measured at H = 512: 2 blocks
  // of 32 rows at B = 64 take 5.6 us against 7.9 us for one block of 64)
  const bool stream_ok = stream_kernel_shape_ok(4 * H, Ix + H) && Ix % 64 == 0;
  plan->grid[1] = (uint32_t)skinny_row_blocks(B, 4 * H, Ix + H, stream_ok);
  plan->grid[2] = 1;
  plan->block = 256;
  if (stream_ok && ceil_div(B, (int64_t)plan->grid[1]) <= 16) {  // the streaming kernel: 64-wide stages
    const bool many = (uint64_t)plan->grid[0] * plan->grid[1] > (uint64_t)kCUs &&
                      (double)(4 * H) * (double)(Ix + H) * 2.0 <= kCachedWeightBytes;
    plan->split_k = many ? 4 : 8;
    plan->bk = 64;
    plan->block = many ? 256 : 512;
  }
  return NIMBLE_OK;
}

const char* nimble_variant_name(int variant) {
  if (variant < 0 || variant >= NIMBLE_VAR_COUNT) return nullptr;
  return kVariants[variant].name;
}

const char* nimble_last_error(void) { return g_err; }

}  // extern "C"
