// Token loop of a batch of LSTM sequences in a single launch: weights resident in registers, the hidden
// state handed from step to step through self-describing words in memory, every wait bounded.
#ifndef NIMBLE_LSTM_SEQ_KERNEL_H_
#define NIMBLE_LSTM_SEQ_KERNEL_H_
#include "device_common.h"

namespace nimble {

// ---------------------------------------------------------------------------
// The evaluation section's LSTM remark: a cell step is too small to fill the chip, so a sequence is
// bound by what separates the steps.  As one launch per step that is the 2-4 us between dependent
// kernels; here the steps of a sequence run inside one launch.
//   Inputs: w_h [4H, H] with pre [T, B, 4H] f32, the inputs' share of the gates with the bias added (one
//   dense call over all T*B tokens ahead of the loop), or the fused weight w [4H, Ix + H] with x [T, B, Ix] and
//   the bias; h_0 [B, H] bf16, c_0 [B, H] f32.
//   Grid: the rows of the batch are cut into groups of R = 8 (one of R = 4 up to 4 rows), which have nothing to do
//   with each other; per group H / 16 workgroups of 8 waves.  A workgroup owns U = 16 hidden units = 64 gate rows (G
//   = 4 groups of the i, f, g, o rows of 4 units) and keeps those rows of the weight in registers for the whole
//   sequence (wave w: the 64-wide K stages w * per_wave ...: 8 registers per group and stage; at most 128 in all, so that two
//   workgroups fit a compute unit).  A launch has as many row groups as give a compute unit one workgroup at most, more rows
//   take several launches one after the other: a loop then has at most half of the chip's places, and two loops on two
//   streams never wait for each other's.  (With all groups in one launch, two to an XCD at a time, 64 steps of 128 / 256 rows, H = Ix = 512, took 165 /
//   302 us instead of 196 / 369; but two such loops could each hold places that the other's next group lacked, and 4 in
//   70 gave up.  Captured launches per step 338 / 556.)  Per step a
//   wave multiplies its stages of x_t, loaded ahead, or its K range of h_{t-1}, and leaves its partial sums
//   in LDS; after one barrier the first R U lanes, one per (row, unit), add them up and update the cell.  c_t
//   stays in that lane's register.
//   Hand-over of h_t: 64-bit words of four neighbouring units of a row, stored into buffer t & 1 of two, in an order in
//   which a wave stores 128 contiguous bytes (8 workgroups' words in one line: 2.4 us per step) and loads
//   512 (8 rows of 32 k or 4 rows of 64 k).  |h| <= 1 leaves bit 14 of a bf16, the top bit of its exponent, zero: in the first value of a word it carries the phase, which changes with every use of a
//   buffer, in the second a mark that values of the word are NaN (then written as 0x3fff, which no h is).  A
//   consumer wave loads the words of its K range, device scope, until all of them are in this step's phase: data
//   and arrival are one word, no counter, no fence, one store and one load on the critical path (a counter
//   barrier over 16 workgroups was measured at 0.85 us per step bare).  Two buffers suffice: h_t overwrites
//   h_{t-2}, which every workgroup has finished reading before it publishes h_{t-1}, without which nobody can
//   compute h_t; and a wave polls the same words in every step, so it has seen a word's value of two steps ago when it
//   looks for this step's, and loads of one address never go back: the word it finds is one of these two, and one bit
//   tells them apart.  The words are
//   cleared by lstm_seq_init_kernel ahead of the launch on the same stream (the first phase is 1).
//   Scope of the stores.  A store of device scope goes through to the memory side (695 clocks until it is done, where a
//   plain one takes 273), and a load of device scope finds a plain store of the same XCD in that XCD's L2: one way
//   between two workgroups of an XCD 957 clocks with stores of device scope, 519 with plain ones (1370 between XCDs).
//   So each workgroup leaves its XCD's number in the first of its words of buffer 0, which nobody writes before every
//   workgroup has read them (that takes h_2), without the phase bit; a workgroup that finds all numbers
//   of its row group equal to its own stores plainly from then on, any other with device scope.  Nobody relies on the
//   others' choice: all are right, the plain stores are seen by all who can look for them.  128 steps, by kernel
//   trace, device-scope stores throughout / so: pre form of H = 512, 1, 4 and 16 rows 154 / 130, 154 / 133, 175 / 145 us, of H = 256, 1 row
//   137 / 122; x form of H = Ix = 512, 4, 37 and 64 rows 171 / 144, 182 / 159, 180 / 155.
//   x_t comes from memory, and what a compute unit's waves load returns in order, so that polls queue behind x.  The waves
//   that multiply x load it straight into LDS, three steps ahead and right behind the barrier, when this step's
//   polls are over and the next ones are some 900 clocks away (loaded into registers behind the products a step
//   ahead 4 / 37 rows, H = Ix = 512, took 153 / 175 us, into LDS but behind the products 152 / 162, by the polling waves as their words
//   had arrived 155 / 179, so 139 / 151; before the plain stores 163 / 169).  Those of them that update cells too wait for a step
//   more than they need, see there.  Over two XCDs, and in ORDER 2, whose waves hold units of x beside units of h, x is loaded into registers
//   a step ahead.
//   Every wait is bounded: a wave polls at most max_polls times per step, looking at the give-up word with every
//   eighth; a wave that runs out sets it, and every workgroup leaves at its next check.  So the
//   grid drains whatever happens (fewer workgroups resident than launched, a stalled neighbour).  Then either
//   the host reads the word and runs the sequence step by step, or lstm_seq_recover_kernel, enqueued behind, does.
//   max_polls = 0 gives up at the first wait: the host-side way to exercise that path.
//   Arithmetic: identical, bit for bit, to the per-step kernel on the same shapes (stream_kernel: the same
//   eight or four ranges of K stages, the same two accumulators per range, the same order of adding the ranges' sums,
//   the same cell function).
//   What bounds it: a chain of, in clocks by time stamps, products and partial sums to LDS 400, barrier 150, sums 250, cell 600,
//   and the way through the L2 to the slowest workgroup 700.  Microseconds per step, by kernel trace, pre form at
//   1 / 4 rows: H = 512 1.02 / 1.04, H = 1024 1.50 / 1.52, H = 256 0.96 / - (32-bit words with a step tag each, four lanes
//   per cell, workgroups over all XCDs: 1.60 / 1.64, 1.76 / 1.96); x form at 4 / 37 / 64 rows, H = Ix = 512: 1.12 / 1.24 /
//   1.21 (a captured graph of per-step launches: 2.9 / 3.65 / 3.7).  On the way there, 37 rows, x form: four lanes
//   per cell, 32-byte stores 2.31; one lane per cell, 128-byte stores 1.95; a row group's workgroups on one XCD
//   and a late first poll 1.56; operands polled straight into their registers, no address arithmetic in the loop 1.37.
//   Tried and not kept: system scope, exchanges instead of stores, raised priority for the cells (no change); a
//   first poll whose delay adapts, a step later for each failure and a quarter earlier for each success (1.7-1.9:
//   of 128 waves some one always fails); every wave multiplying its own 16 gate rows over the whole of K (4.1: the
//   waves' reads of all of h cost more LDS time than the sums saved); workgroup-scope loads within one XCD (they
//   hit the compute unit's own cache, and the words never become visible); with plain stores, four lanes per cell, one per gate
//   (1 / 4 / 37 rows 122 / 127 / 151 -> 120 / 131 / 149), and the products of all four groups ahead of their sums
//   (122 / 126 -> 125 / 128).
// ---------------------------------------------------------------------------
struct LstmSeqArgs {
  const u16* x;       // [T, B, Ix], or null
  const float* pre;   // [T, B, 4H], in place of x and bias
  const u16* w;       // [4H, Ix + H]
  const u16* bias;    // [4H], with x
  const u16* h0;      // [B, H]
  const float* c0;    // [B, H]
  u16* h_seq;         // [T, B, H]
  float* c_out;       // [B, H]
  uint32_t* ctl;      // 64 words: [0] give-up word, [1] workgroups that ran all T steps
  unsigned long long* exch;  // [row group][2][words of 4 units]: B * H / 2 words
  float* c_keep;      // [B, H] or null: c_0 for the recovery kernel (c_out may be c_0)
  int T, B, Ix, H;
  int ranges;         // of K stages with a sum of their own: 8, or 4 where the per-step launch runs four waves
  uint32_t max_polls;
  uint32_t apart;     // 0; tests: bit 0 (1) set, workgroups of even (odd) number store as if the row group did not share an XCD
};

// Clears the control words and the hand-over words, keeps c_0 for the recovery kernel.
__global__ void __launch_bounds__(256) lstm_seq_init_kernel(LstmSeqArgs a, int words) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int n = a.B * a.H;
  if (i < 64) a.ctl[i] = 0u;
  for (int j = i; j < words; j += gridDim.x * 256) a.exch[j] = 0ull;
  if (i < n && a.c_keep) a.c_keep[i] = a.c0[i];
}

// lane i of 16 takes the value of lane i + N
template <int N>
__device__ __forceinline__ uint32_t lane_up(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x100 + N, 0xf, 0xf, true);
}
// every lane of 4 takes the value of lane Q of them
template <int Q>
__device__ __forceinline__ uint32_t quad_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, Q * 0x55, 0xf, 0xf, true);
}

// the XCD that the wave runs on
__device__ __forceinline__ uint32_t xcc_id() { return __builtin_amdgcn_s_getreg(20 | (3 << 11)); }

constexpr uint32_t kHandOverPhase = 0x4000u, kHandOverNan = 0x40000000u;

// The address at a wave-uniform base plus a 32-bit byte offset of the lane's own.  (The offset is made opaque: left to
// itself the compiler adds the two ahead of the loop and keeps 64-bit addresses in vector registers.)
template <typename V>
__device__ __forceinline__ V* at(V* base, uint32_t bytes) {
  asm volatile("" : "+v"(bytes));
  return (V*)((const char*)base + bytes);
}

// phase of the words of step t = 1, 2, ... in their buffer t & 1: 1 at the first use, then in turn
__device__ __forceinline__ uint32_t lstm_seq_phase(int t) { return ((t - 1) & 2) ? 0u : kHandOverPhase; }

// 0x3fff in either half of a word marked so: NaN
__device__ __forceinline__ uint32_t lstm_seq_nans(uint32_t v) {
  const uint32_t lo = (v & 0x3fffu) == 0x3fffu ? 0x7fc0u : (v & 0xffffu);
  const uint32_t hi = (v & 0x3fff0000u) == 0x3fff0000u ? 0x7fc00000u : (v & 0xffff0000u);
  return lo | hi;
}

// PRE: the inputs' share comes precomputed, else from x; PW: K stages of 64 per wave, ceil((Ix + H) / 64 / 8); G: groups
// of 16 gate rows (4 units) per workgroup; R: rows per group of workgroups, 4 or 8.  rs_few: words per four units in the
// hand-over buffers for R = 4 (at least the group's rows).  group0: first of this launch's row groups.
// A wave's share of K is 2 PW units of 32 k.  ORDER 0, eight ranges: wave w has the units of range w one after the other,
// in two chains, as the per-step launch on eight waves.  ORDER 1, four ranges of 2 PW whole stages: that launch has four
// waves, each with the first halves of its stages in one chain and the second halves in the other; here waves 2 w and
// 2 w + 1 have one of these chains each, which gives the same sums without a wave doing more.  ORDER 2: as 1 where a
// range holds stages of x and of h (in place of 1 it takes 128 steps of 37 rows, H = Ix = 512, from 188 us to 204).
// ONE: a row group's workgroups go to one XCD, else to two (above H = 512).  Only there do the words meet in an L2, and only there is x
// loaded into LDS: with the words on their way for longer, x in registers a step ahead costs nothing, and the ring's waits and reads 3 to 4 %
// (128 steps of 5 rows, Ix = 128, H = 640, 200 us, with the ring 208; 4 rows, 256, 768, 194 and 202).
template <bool PRE, int PW, int G, int R, int ORDER, bool ONE>
__global__ void __launch_bounds__(512, 4) lstm_seq_kernel(LstmSeqArgs a, int group0, int row_groups, int rs_few, int xcd0) {
  static_assert(R == 4 || R == 8, "a load brings 8 rows of 32 k or 4 rows of 64");
  static_assert(ORDER == 0 || R == 8, "up to 4 rows the per-step launch runs eight waves");
  constexpr bool MIX = ORDER == 2;
  // Waves that hold two stages of x and of h wait for x from memory in front of their polls, whatever the stores' scope: 128 steps of 37
  // rows, Ix = 640, H = 384, 194 us, with plain stores 200.  (With one stage per wave 97 rows, 192, 320 347 and 285.)
  constexpr bool NEAR = ONE && !(MIX && PW == 2);
  constexpr int NU = 2 * PW;               // units of 32 k per wave
  constexpr int STEP = ORDER == 0 ? 32 : 64;  // k from one of them to the next
  const int rs = R == 8 ? 8 : rs_few;
  constexpr int SCOPE = __HIP_MEMORY_SCOPE_AGENT;
  constexpr int U = 4 * G;    // units per workgroup
  constexpr int LPS = R / 4;  // loads of 64 words per stage
  constexpr int CELLS = R * U;  // one lane each, in the first waves
  // partial sums [buffer][wave][cell]: the four gates of a cell are one 16-byte word
  __shared__ f32x4 red[2][8][CELLS];
  // operands of the waves that multiply x: three steps' [chunk of 8 k][row] (MIX and two XCDs: in registers)
  constexpr bool XR = !PRE && !MIX && ONE;
  constexpr int XLOADS = NU * 4 * R > 64 ? NU * 4 * R / 64 : 1;  // of 64 chunks, per step
  __shared__ uint4 x_ring[XR ? 7 : 1][3][XR ? XLOADS * 64 : 1];
  __shared__ int s_abort[2];  // by step parity: a wave already polling for step t+1 never writes the word step t reads

  // Workgroups go to the 8 XCDs in turn: a row group's workgroups are those of one XCD (of two, above 32 of them), so that
  // the hand-over words meet in that XCD's L2.  (Where they go elsewhere the loop is slower and as right.)
  const int H = a.H, Ix = PRE ? 0 : a.Ix, B = a.B, T = a.T;
  constexpr int span = ONE ? 1 : 2;
  const int n_wg = H / U, per_xcd = n_wg / span;
  const int xcd = ((int)blockIdx.x + xcd0) & 7, nth = (int)blockIdx.x >> 3;
  const int group = group0 + nth / per_xcd * (8 / span) + xcd / span;
  if (group >= row_groups) return;
  const int wg = (xcd & (span - 1)) * per_xcd + nth % per_xcd;
  const int row0 = group * R;
  // hand-over words of this row group: [buffer][unit / 4][row]
  const int plane = rs * (H >> 2);
  unsigned long long* exch = a.exch + (long long)row0 * (H >> 1);  // (groups but the last are R rows of rs = R)
  const unsigned long long here = xcc_id() + 1;  // (1 ... 8: neither phase nor mark)
  if (NEAR && threadIdx.x == 0) __hip_atomic_store(exch + wg * G * rs, here, __ATOMIC_RELAXED, SCOPE);
  const int rows = B - row0 < R ? B - row0 : R;  // of this group
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, gq = lane >> 4;

  // this wave's units: of the per-step kernel's ranges (ORDER < 2: all of x or all of h, Ix is whole ranges)
  const int x_stages = Ix >> 6, stages = (Ix + H) >> 6;
  int st_begin, n_st, k_begin;  // first stage, stages (ORDER > 0: pairs of units) <= PW, first k
  if (ORDER == 0) {
    const int per_wave = (stages + 7) / 8;  // <= PW (the launcher picks PW >= per_wave)
    st_begin = wave * per_wave;
    const int st_end = (st_begin + per_wave) < stages ? (st_begin + per_wave) : stages;
    n_st = st_end > st_begin ? st_end - st_begin : 0;
    k_begin = st_begin * 64;
  } else {
    st_begin = (wave >> 1) * NU;  // (the launcher: stages = 4 NU)
    n_st = PW;
    k_begin = st_begin * 64 + (wave & 1) * 32;
  }
  const bool of_x = !PRE && st_begin < x_stages;  // (MIX: its first units)
  const int x_units = !of_x ? 0 : x_stages - st_begin < NU ? x_stages - st_begin : NU;  // (MIX)

  // weights of this workgroup's 16 G gate rows over this wave's units, in the MFMA operand
  // layout: lane (r, gq) holds 8 k of tile row r = gate r & 3 of unit 4 g + (r >> 2)
  uint4 wt[G][NU];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const u16* wrow = a.w + ((long long)(r & 3) * H + wg * U + g * 4 + (r >> 2)) * (Ix + H);
#pragma unroll
    for (int s = 0; s < PW; ++s) {
      if (ORDER != 0 || s < n_st) {
        const int k = k_begin + 2 * s * STEP + gq * 8;
        wt[g][2 * s] = *(const uint4*)(wrow + k);
        wt[g][2 * s + 1] = *(const uint4*)(wrow + k + STEP);
      } else {
        wt[g][2 * s] = wt[g][2 * s + 1] = make_uint4(0, 0, 0, 0);
      }
      // (left to itself the compiler loads the weights anew in every step instead of keeping them)
      keep_in_registers(wt[g][2 * s]);
      keep_in_registers(wt[g][2 * s + 1]);
    }
  }

  // cell update: lane -> (group cg of 4 units, row mm, unit uu of the group); four neighbouring lanes hold the units
  // of a hand-over word, which the first of them stores, so that a wave stores 128 contiguous bytes
  const int uu = tid & 3, mm = (tid >> 2) & (R - 1), cg = tid / (4 * R);
  const bool cells = wave * 64 < CELLS;  // (wave-uniform)
  const bool owner = tid < CELLS && mm < rows;
  const uint32_t cell = owner ? (uint32_t)((row0 + mm) * H + wg * U + cg * 4 + uu) : 0u;
  const uint32_t put = (uint32_t)((wg * G + cg) * rs + mm) * 8u;  // the word of the lane's four units, in bytes
  float c = owner ? *at(a.c0, cell * 4u) : 0.f;

  if (tid < 2) s_abort[tid] = 0;
  __syncthreads();
  // word of this lane in a load: R = 8: 32 k, rows by lane & 7, pieces of 4 k by gq and bit 3; R = 4: 64 k
  uint32_t ask;   // (bytes, as is the next)
  uint32_t from;  // this lane's operand row in x_t or h_0 (lanes past the group's rows: columns never used)
  // first k of this wave within h (MIX: can be below 0, its first units are of x)
  const int h_begin = k_begin - x_stages * 64;
  {
    const int lrow = (r & (R - 1)) < rows ? r & (R - 1) : rows - 1;
    ask = (uint32_t)((R == 8 ? gq * 2 + (r >> 3) : (r >> 3) * 8 + gq * 2 + ((r >> 2) & 1)) * rs + lrow +
                     (MIX || of_x ? 0 : (h_begin >> 2) * rs)) * 8u;
    const int orow = row0 + (r < rows ? r : rows - 1);
    from = (uint32_t)(of_x ? orow * Ix + k_begin + gq * 8 : orow * H + h_begin + gq * 8) * 2u;
  }

  // operands of this wave's units for the step to come: x_t (from its ring; MIX: loaded a step ahead) or h_{t-1}
  uint4 f[NU];
#pragma unroll
  for (int j = 0; j < NU; ++j) f[j] = make_uint4(0, 0, 0, 0);  // (units that this wave does not have: zeros)
  auto load_rows = [&](const u16* src) {
#pragma unroll
    for (int s = 0; s < PW; ++s) {
      if (MIX ? 2 * s < x_units : ORDER != 0 || s < n_st) f[2 * s] = *(const uint4*)at(src + 2 * s * STEP, from);
      if (MIX ? 2 * s + 1 < x_units : ORDER != 0 || s < n_st) f[2 * s + 1] = *(const uint4*)at(src + (2 * s + 1) * STEP, from);
    }
  };
  uint32_t x_at = 0;  // (bytes) of the lane's chunk in x_t
  if (XR && of_x) {
    const int row = lane & (R - 1), chunk = lane / R & (NU * 4 - 1);
    x_at = (uint32_t)((row0 + (row < rows ? row : rows - 1)) * Ix + k_begin + (chunk >> 2) * STEP + (chunk & 3) * 8) * 2u;
  }
  const uint32_t x_lds = lds_addr_of(&x_ring[XR && of_x ? wave : 0][0][0]);
  auto load_x = [&](int t) {  // x of step t = 1, 2, ... into its slot (past the last step that one's again: the waits count)
    const u16* src = a.x + (long long)((t < T ? t : T) - 1) * B * Ix;
#pragma unroll
    for (int l = 0; l < XLOADS; ++l) dma16_so(x_at, src + l * 2 * STEP, x_lds + (uint32_t)(t % 3 * XLOADS + l) * 1024u);
  };
  if (XR && of_x) {
    load_x(1);
    load_x(2);
    load_x(3);
  }
  if (MIX) {
    const int orow = row0 + (r < rows ? r : rows - 1);
#pragma unroll
    for (int j = 0; j < NU; ++j)
      f[j] = *(const uint4*)((j < x_units ? a.x + orow * Ix + k_begin : a.h0 + orow * H + h_begin) + j * STEP + gq * 8);
  } else if (!XR || !of_x) {
    load_rows(of_x ? a.x : a.h0);
  }
  const bool waits = MIX ? x_units < NU : !of_x && n_st > 0;  // for h_t
  if (waits && a.max_polls == 0) s_abort[1] = 1;

  // The bias, or the inputs' share of the gates, which streams from memory, a fresh line per step: it is fetched
  // one step ahead, and behind the wave's poll loads (loads return in order: in front of them it would hold
  // every poll back by a trip to HBM).
  float pr[4] = {0.f, 0.f, 0.f, 0.f}, pr_next[4] = {0.f, 0.f, 0.f, 0.f};
  const uint32_t pre_at = owner ? (cell + (uint32_t)((row0 + mm) * 3 * H)) * 4u : 0u;  // [row, gate, unit], in bytes
  if (owner) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      pr[q] = PRE ? *at(a.pre + q * H, pre_at) : bf2f(a.bias[q * H + wg * U + cg * 4 + uu]);
  }
  // whether the row group's workgroups share an XCD, that is an L2 (behind the first loads, which take as long)
  bool near = false;
  if (NEAR) {
    const unsigned long long* ids = exch + (lane < n_wg ? lane : 0) * G * rs;
    const uint32_t most = a.max_polls < 256u ? a.max_polls : 256u;
    unsigned long long v = 0;
    for (uint32_t polls = 0; polls < most; ++polls) {
      v = __hip_atomic_load(ids, __ATOMIC_RELAXED, SCOPE);
      if (__all(v != 0ull)) break;
    }
    near = __all(v == here) && (a.apart >> (wg & 1) & 1u) == 0u;
  }
  if (XR && of_x) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  for (int t = 1;; ++t) {
    if (XR && of_x) {
      // this step's loads were issued three steps ago: behind them are those of two more steps and, from the cells' waves, two
      // stores per step (each such wave has a lane in row 0 that stores).  Half of these are counted: with a load per step
      // those waves wait for the next step's load too, i.e. run two steps ahead.
      if (cells)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * XLOADS + 3) : "memory");
      else
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * XLOADS) : "memory");
      const uint4* slot = &x_ring[wave][t % 3][0];
#pragma unroll
      for (int j = 0; j < NU; ++j) f[j] = slot[(j * 4 + gq) * R + (r & (R - 1))];
    }
    // (two groups at a time: four independent chains, and no more accumulators than that)
#pragma unroll
    for (int g0 = 0; g0 < G; g0 += 2) {
      f32x4 acc[2][2];
#pragma unroll
      for (int g = 0; g < 2; ++g) acc[g][0] = acc[g][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      auto product = [&](int j, int g) {
        const int chain = ORDER == 0 ? j & 1 : 0;
        acc[g][chain] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wt[g0 + g][j]), as_bf16x8(f[j]), acc[g][chain], 0, 0, 0);
      };
#pragma unroll
      for (int j = 0; j < NU; j += 2)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (ORDER == 0) product(j + (i & 1), i >> 1); else product(j + (i >> 1), i & 1);  // (ORDER > 0: one chain per group)
      // accumulator of lane (r, gq), register v: gate v of unit gq of the group, activation row r
#pragma unroll
      for (int g = 0; g < 2; ++g)
        if (r < R) red[t & 1][wave][((g0 + g) * R + r) * 4 + gq] = ORDER == 0 ? acc[g][0] + acc[g][1] : acc[g][0];  // rows past the group's are never used
    }
    if (!XR && of_x && t < T) load_rows(a.x + (long long)t * B * Ix);
    if (PRE && owner && t < T) {
      const float* src = a.pre + (long long)t * B * 4 * H;
#pragma unroll
      for (int q = 0; q < 4; ++q) pr_next[q] = *at(src + q * H, pre_at);
    }
    __syncthreads();
    if (XR && of_x) load_x(t + 3);  // (into this step's slot, which the wave has read)
    const int aborted = __builtin_amdgcn_readfirstlane(s_abort[t & 1]);  // written before the barrier (after an abort the cells are garbage, and not used)

    if (cells) {
      // the waves' partial sums in the per-step kernel's order (ORDER > 0: neighbours are its waves' two chains), the
      // inputs' share, the cell
      const f32x4* e = &red[t & 1][0][tid & (CELLS - 1)];
      f32x4 sum = (e[0] + e[CELLS]) + (e[2 * CELLS] + e[3 * CELLS]);
      if (PRE && PW > 1) __builtin_amdgcn_sched_barrier(0);  // (all eight at once do not fit beside the weights)
      sum += (e[4 * CELLS] + e[5 * CELLS]) + (e[6 * CELLS] + e[7 * CELLS]);
      const float gate[4] = {sum[0] + pr[0], sum[1] + pr[1], sum[2] + pr[2], sum[3] + pr[3]};
      float cn;
      const uint32_t hb = f2bf(lstm_cell(gate, c, cn));
      c = cn;
      // (the next step's share of the inputs has had this whole step to arrive; taking it over here, ahead of
      // the stores, keeps any wait for it off the path from the store below to the next step's first poll)
      if (PRE) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          pr[q] = pr_next[q];
          asm volatile("" : "+v"(pr[q]));
        }
      }
      const uint32_t lo = hb | (quad_lane<1>(hb) << 16), hi = quad_lane<2>(hb) | (quad_lane<3>(hb) << 16);
      if (owner && uu == 0) {
        uint32_t slo = lo, shi = hi;
        if ((lo | hi) & 0x40004000u) {  // a NaN among the four
          slo = (lo & 0x4000u ? 0x3fffu : lo & 0xffffu) | (lo & 0x40000000u ? 0x3fff0000u : lo & 0xffff0000u) | kHandOverNan;
          shi = (hi & 0x4000u ? 0x3fffu : hi & 0xffffu) | (hi & 0x40000000u ? 0x3fff0000u : hi & 0xffff0000u);
        }
        slo |= lstm_seq_phase(t);
        unsigned long long* word = at(exch + (long long)(t & 1) * plane, put);
        const unsigned long long v = ((unsigned long long)shi << 32) | slo;
        if (near)
          __hip_atomic_store(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else
          __hip_atomic_store(word, v, __ATOMIC_RELAXED, SCOPE);
        *(uint2*)at(a.h_seq + (long long)(t - 1) * B * H, cell * 2u) = make_uint2(lo, hi);
      }
    }
    // (the partial sums alternate between two buffers: a wave can write step t+1's only after this
    // step's barrier, and step t+2's only after the barrier of t+1, which every thread reaches after
    // it has read step t's)
    if (aborted || t == T) break;

    if (waits) {
      // h_t: this wave's k range of every row, polled until every word is in the phase of step t
      const uint32_t want = lstm_seq_phase(t);
      const unsigned long long* src = exch + (long long)(t & 1) * plane;
      uint32_t polls = 0, nan;
      // A poll that finds the words not there yet costs another round trip, and more polls on their way delay the
      // stores they wait for: the first goes out when the words can be expected, in units of 64 clocks.  Microseconds for
      // 128 steps with 12, 14, 16, 18, 20 units, x form of H = 512, 37 rows: 235, 205, 178, 183, 190 (on another card 14 was
      // the best: the edge moves by two units, so a little later); pre form, H = 512, 16 rows 207, 188, 185, 187, 192; 24 rows
      // of 256 198, 183, 179, 176, 181, of 1024 271, 257, 252, 255, 247.  Up to 4 rows, pre form, with 12, 13, 14, 15, 16 units,
      // means over the XCD it starts on: H = 512, 1 row 175, 163, 159, 165, 167, H = 256 175, 163, 148, 153, 157; two stages
      // per wave, H = 1024, with 14 to 18: 221, 215, 213, 213, 213.  Within an XCD, with plain stores, polls cost little and the
      // arrival is earlier: pre form of H = 512, 1 row, with 0, 3, 5, 7, 9, 11, 13 units 125, 127, 131, 126, 130, 134, 140 (the period is a
      // poll's), 16 rows 137, 141, 142, 137, 139, 140, 144; x form, 37 rows 162, 160, 160, 160, 154, 153, 156.
      if (near) {
        if (!cells) __builtin_amdgcn_s_sleep(PRE ? 7 : 9);
      } else if (!cells) {
        __builtin_amdgcn_s_sleep(R == 8 || PW > 1 ? 16 : 14);
      } else if (R == 8) {
        __builtin_amdgcn_s_sleep(4);
      }
      for (;;) {
        unsigned long long v[PW][LPS];  // R = 8: a unit per load; R = 4: two, the lanes of the upper 8 rows hold the second
#pragma unroll
        for (int s = 0; s < PW; ++s)
#pragma unroll
          for (int l = 0; l < LPS; ++l) {
            const int j = 2 * s + l;
            if (ORDER == 0)  // (a stage that this wave does not have: the words of its last one again)
              v[s][l] = __hip_atomic_load(at(src + (s < n_st ? s : n_st - 1) * 16 * rs, ask) + l * 8 * rs, __ATOMIC_RELAXED, SCOPE);
            else if (!MIX)
              v[s][l] = __hip_atomic_load(at(src + j * 16 * rs, ask), __ATOMIC_RELAXED, SCOPE);
            else  // (units of x: the words of its first unit of h)
              v[s][l] = __hip_atomic_load(at(src + (long long)((h_begin >> 2) + (j < x_units ? x_units : j) * 16) * rs, ask),
                                          __ATOMIC_RELAXED, SCOPE);
          }
        uint32_t bad = 0;
#pragma unroll
        for (int s = 0; s < PW; ++s)
#pragma unroll
          for (int l = 0; l < LPS; ++l) {
            const int j = 2 * s + l;
            const uint32_t lo = (uint32_t)v[s][l] ^ want;
            f[j].x = MIX && j < x_units ? f[j].x : lo;
            f[j].y = MIX && j < x_units ? f[j].y : (uint32_t)(v[s][l] >> 32);
            bad |= lo;
          }
        nan = bad & kHandOverNan;
        if (__all((bad & kHandOverPhase) == 0u)) break;
        // (wave-uniform: every lane counts alike and reads the same give-up word)
        ++polls;
        if (polls >= a.max_polls || ((polls & 7u) == 0u && __builtin_amdgcn_readfirstlane((int)__hip_atomic_load(a.ctl, __ATOMIC_RELAXED, SCOPE)) != 0)) {
          if (lane == 0) __hip_atomic_store(a.ctl, 1u, __ATOMIC_RELAXED, SCOPE);
          s_abort[(t + 1) & 1] = 1;
          break;
        }
      }
      if (__any(nan != 0u)) {
#pragma unroll
        for (int s = 0; s < PW; ++s)
#pragma unroll
          for (int j = 2 * s; j < 2 * s + LPS; ++j)
            if (f[j].x & (MIX && j < x_units ? 0u : kHandOverNan)) {
              f[j].x = lstm_seq_nans(f[j].x & ~kHandOverNan);
              f[j].y = lstm_seq_nans(f[j].y);
            }
      }
      // to the operand layout: the lanes of the first R rows collect the other pieces of their 8 k
#pragma unroll
      for (int s = 0; s < PW; ++s) {
        if (R == 4) f[2 * s + 1] = make_uint4(lane_up<8>(f[2 * s].x), lane_up<8>(f[2 * s].y), lane_up<12>(f[2 * s].x), lane_up<12>(f[2 * s].y));
#pragma unroll
        for (int j = 2 * s; j < 2 * s + LPS; ++j) {
          f[j].z = MIX && j < x_units ? f[j].z : lane_up<R == 8 ? 8 : 4>(f[j].x);
          f[j].w = MIX && j < x_units ? f[j].w : lane_up<R == 8 ? 8 : 4>(f[j].y);
        }
        if (ORDER == 0 && s > 0 && n_st <= s) f[2 * s] = make_uint4(0, 0, 0, 0), f[2 * s + 1] = make_uint4(0, 0, 0, 0);
      }
    }
  }

  if (XR && of_x) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing may arrive in LDS after the workgroup's end
  if (!(s_abort[0] | s_abort[1])) {
    if (owner) *at(a.c_out, cell * 4u) = c;
    if (tid == 0) __hip_atomic_fetch_add(a.ctl + 1, 1u, __ATOMIC_RELAXED, SCOPE);
  } else if (tid == 0) {
    __hip_atomic_store(a.ctl, 1u, __ATOMIC_RELAXED, SCOPE);
  }
}

// The same sequence by workgroups that wait for nobody, enqueued behind the loop and gone at once unless that
// gave up: a workgroup takes 16 rows through all steps, its waves walk the units in fours, each over the whole of K, with
// the same ranges and the same order of the sums.  h_{t-1} is read back from h_seq, c_t lives in c_keep.
// Bound by one compute unit's reading of the weights, some 50 us per step; runs only where the loop could not.
__global__ void __launch_bounds__(1024) lstm_seq_recover_kernel(LstmSeqArgs a) {
  if (__hip_atomic_load(a.ctl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, gq = lane >> 4;
  const int T = a.T, B = a.B, H = a.H, Ix = a.Ix;
  const int row = blockIdx.x * 16 + r;
  const int orow = row < B ? row : B - 1;
  const int x_stages = Ix >> 6, stages = (Ix + H) >> 6;
  const int per_range = (stages + a.ranges - 1) / a.ranges;
  for (int t = 0; t < T; ++t) {
    const u16* h_prev = t == 0 ? a.h0 : a.h_seq + (long long)(t - 1) * B * H;
    const u16* xr = a.x ? a.x + ((long long)t * B + orow) * Ix : nullptr;
    const u16* hr = h_prev + (long long)orow * H;
    for (int g = wave; g < H / 4; g += 16) {
      const u16* wrow = a.w + ((long long)(r >> 2) * H + g * 4 + (r & 3)) * (Ix + H) + gq * 8;
      f32x4 sum = {0.f, 0.f, 0.f, 0.f};
      for (int four = 0; four < a.ranges; four += 4) {
        f32x4 part[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
          const int begin = (four + v) * per_range;
          const int end = begin + per_range < stages ? begin + per_range : stages;
          for (int s = begin; s < end; ++s) {
            const u16* src = (s < x_stages ? xr + s * 64 : hr + (s - x_stages) * 64) + gq * 8;
            acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(*(const uint4*)(wrow + s * 64)),
                                                           as_bf16x8(*(const uint4*)src), acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(*(const uint4*)(wrow + s * 64 + 32)),
                                                           as_bf16x8(*(const uint4*)(src + 32)), acc1, 0, 0, 0);
          }
          part[v] = acc0 + acc1;
        }
        sum += (part[0] + part[1]) + (part[2] + part[3]);
      }
      // lane (r, gq), register v: gate gq of unit 4 g + v, row r; the lane then takes unit 4 g + gq
      float gate[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int col = gq * H + g * 4 + v;
        const float z = sum[v] + (a.pre ? a.pre[((long long)t * B + orow) * 4 * H + col] : bf2f(a.bias[col]));
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const float from = __shfl(z, r + 16 * p, 64);
          if (gq == v) gate[p] = from;
        }
      }
      if (row < B) {
        const long long cell = (long long)row * H + g * 4 + gq;
        float cn;
        const float hn = lstm_cell(gate, a.c_keep[cell], cn);
        a.c_keep[cell] = cn;
        a.h_seq[(long long)t * B * H + cell] = f2bf(hn);
        if (t == T - 1) a.c_out[cell] = cn;
      }
    }
    __syncthreads();  // (h_t is read by the workgroup's other waves)
  }
}

}  // namespace nimble
#endif
