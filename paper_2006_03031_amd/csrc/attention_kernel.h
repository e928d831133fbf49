// Fused attention for head dimension 64, without and with its intermediate results.
#ifndef NIMBLE_ATTENTION_KERNEL_H_
#define NIMBLE_ATTENTION_KERNEL_H_
#include <type_traits>

#include "device_common.h"

namespace nimble {

// ---------------------------------------------------------------------------
// O = softmax(alpha Q.K^T) V per head, in one launch, the scores never leave the chip.
//   Workgroup: RW waves of 32 query rows each, times KG key groups.  Key group g walks the blocks of 64
//   keys g, g + KG, ... with a running score reference and row sum; with KG > 1 the groups' results meet
//   in LDS at the end.
//   scores:  MFMA 32x32x16 with 32 key rows on the A side and the wave's 32 query rows on the B side: a
//            lane holds, for its query row lane & 31, the keys 32 t + 8 b + 4 (lane >> 5) + e of key
//            tile t (b, e = 0..3).
//   P.V:     k runs over keys, in an order that is free: the 8 k slots of half h = lane >> 5 in MFMA u are
//            DEFINED as the 8 keys the half already holds, 16 u + 4 h + (0..3) and 16 u + 8 + 4 h + (0..3), so P
//            goes from the score accumulators to the MFMA operand without leaving the lane.  The matching
//            values of V come out of the row-major tile with the transposing LDS read.
//   K and V blocks: direct global->LDS loads of whole 128-byte rows, S slots each per key group; chunk c of
//   K row r sits at c ^ ((r >> 1) & 7), of V row r at c ^ (4 ((r >> 1) & 1)) (conflict-free for the 16-byte
//   reads and for the transposing reads).
//   Pipeline: the scores of block i + 1 are multiplied while the probabilities of block i are formed; K of
//   block i + 2 and V of block i + 1 load meanwhile.
//   Softmax in base 2 on the raw scores (alpha > 0, checked by the entry point): p = 2^(a2 s - a2 max) with
//   a2 = alpha log2 e is one fused multiply-add and one exp2 per score; the running output is rescaled only when
//   some row's maximum moved.  (Rescaling only once a maximum has grown by 2^8 saves a tenth of the time, but then the
//   largest probabilities are no longer exactly 1 and the error against 64 bits grows from 2.19e-3 to 2.3e-3.)
//   What bounds it: per block of 64 keys and 32 rows about 1050 clocks of vector instructions, half of them the
//   exponentials, under which 512 clocks of MFMA run; 96 heads of 2048 keys: 115-120 us (860-900 TFLOP/s), the vector
//   instructions alone 84-96 at 2.1-2.4 GHz.  The kernel before it (16 rows per wave, V transposed through
//   registers with 2-byte LDS writes): 216 us; 12 heads of 512 keys 9.8 -> 5.8.  Without the overlap of
//   two blocks 140; eight row waves per workgroup 123, two 152.
//   The workgroups of a compute unit share its vector units: a wave that has its maxima runs at higher priority until
//   its last product is issued, so the matrix core is fed while the others look for theirs.  Raised from the rescaling
//   or the first score product on, over the maxima, or lowered a quarter earlier it gives less or nothing.  With it, with
//   the maximum starting from the reference and the loads' offsets kept, before -> now on one card: 96 x 2048 123.0 -> 119.6 us,
//   96 x 1000 36.5 -> 34.9, 24 x 2048 41.1 -> 38.0, 48 x 777 19.6 -> 18.1; 12 x 2048 (two key groups, the maximum
//   alone) 22.3 -> 22.1.
// ---------------------------------------------------------------------------
template <int RW, int KG, int S>
__global__ void __launch_bounds__(RW* KG * 64) __attribute__((amdgpu_waves_per_eu(2, 4)))
    attention_kernel(const u16* __restrict__ q, const u16* __restrict__ k, const u16* __restrict__ v,
                     u16* __restrict__ o, int L, float alpha) {
  constexpr int D = 64, BJ = 64;
  constexpr int TILE = BJ * 8;         // uint4 per tile of K or V
  constexpr int LD = 8 / RW;           // direct loads per wave and tile
  static_assert(8 % RW == 0 && (S == 1 || S == 2), "tiles are filled in 8 loads");
  // per key group: S tiles of K, then S tiles of V
  __shared__ __attribute__((aligned(256))) uint4 ring[KG][2][S][TILE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rw = wave % RW, kg = wave / RW;
  const int r32 = lane & 31, h = lane >> 5;
  // contiguous runs of (head, query block) per XCD: the query blocks of a head meet in one L2
  int qb, head_i;
  {
    const unsigned nb = gridDim.x * gridDim.y, id = blockIdx.y * gridDim.x + blockIdx.x;
    const unsigned per = nb >> 3, rem = nb & 7, xcd = id & 7;
    const unsigned pid = xcd * per + (xcd < rem ? xcd : rem) + (id >> 3);
    head_i = (int)(pid / gridDim.x);
    qb = (int)(pid % gridDim.x);
  }
  const long long head = (long long)head_i * L * D;
  const int m_row = (qb * RW + rw) * 32 + r32;
  const int m_ld = m_row < L ? m_row : L - 1;

  const int nblk = (L + BJ - 1) / BJ;            // key blocks of the head
  const int steps = (nblk + KG - 1) / KG;        // walked by every group (the barriers are the workgroup's)
  const int mine = (nblk - kg + KG - 1) / KG;    // of this group

  // direct loads: instruction j of a tile brings rows 8 j .. 8 j + 7, lane -> row 8 j + (lane >> 3), physical
  // chunk lane & 7
  const int rr = lane >> 3;
  const uint32_t ring_lds = __builtin_amdgcn_readfirstlane(lds_addr_of(&ring[kg][0][0][0]));
  // offsets of this lane's pieces of a K and of a V tile whose rows all exist.  Kept, like the priority below, only
  // without key groups: they save 8 instructions per block, but with groups 12 x 2048 took 22.2 -> 23.0 us.
  constexpr bool WHOLE = KG == 1;
  uint32_t off[2][LD];
#pragma unroll
  for (int n = 0; n < LD; ++n) {
    const int row = (rw * LD + n) * 8 + rr;
    off[0][n] = (uint32_t)(row * D + ((lane & 7) ^ ((row >> 1) & 7)) * 8) * 2u;
    off[1][n] = (uint32_t)(row * D + ((lane & 7) ^ (4 * ((row >> 1) & 1))) * 8) * 2u;
  }
  auto issue = [&](auto is_v, int i) {  // K or V tile of block i of this group
    constexpr bool V = decltype(is_v)::value;
    const int j0 = (i * KG + kg) * BJ;
    const u16* base = (V ? v : k) + head + (long long)j0 * D;
    const uint32_t dst = ring_lds + ((V ? S : 0) + (S == 1 ? 0 : (i & 1))) * (TILE * 16);
    const int last = L - 1 - j0;                 // rows past the head's last one repeat it
    if (WHOLE && last >= BJ - 1) {  // uniform
#pragma unroll
      for (int n = 0; n < LD; ++n) dma16_so(off[V][n], base, dst + (rw * LD + n) * 1024);
      return;
    }
#pragma unroll
    for (int n = 0; n < LD; ++n) {
      const int j = rw * LD + n;
      int row = j * 8 + rr;
      const int c = (lane & 7) ^ (V ? 4 * ((row >> 1) & 1) : ((row >> 1) & 7));
      row = row < last ? row : last;
      dma16_so((uint32_t)(row * D + c * 8) * 2u, base, dst + j * 1024);
    }
  };
  using K_TILE = std::false_type;
  using V_TILE = std::true_type;
  if (mine > 0) issue(K_TILE{}, 0), issue(V_TILE{}, 0);
  if (S > 1 && mine > 1) issue(K_TILE{}, 1);

  // the wave's query fragments: row m, d = 16 dd + 8 h .. + 7
  bf16x8 qf[4];
#pragma unroll
  for (int dd = 0; dd < 4; ++dd)
    qf[dd] = as_bf16x8(*(const uint4*)(q + head + (long long)m_ld * D + dd * 16 + h * 8));

  f32x16 oacc[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[t][e] = 0.f;
  float ref = -3.0e38f;                          // in raw-score units; finite: a block of infinitely low scores adds zeros
                                                 // (while 3e38 a2 is finite: up to alpha = 0.78)
  float sum0 = 0.f, sum1 = 0.f;                  // this lane's share of the row sum
  const float a2 = alpha * 1.4426950408889634f;

  // fragment addresses within a tile: K chunk 2 dd + h of row r32, and the transposing reads of V
  const int ksw = (r32 >> 1) & 7;
  const int i16 = lane & 15, dh = (lane >> 4) & 1;
  const uint32_t v_off = (uint32_t)((4 * h + (i16 >> 2)) * 128 +
                                    (((2 * dh + ((i16 & 3) >> 1)) ^ (4 * ((i16 >> 3) & 1))) * 16) + (i16 & 1) * 8);
  auto qk = [&](f32x16& s, int ks_slot, int t, int dd) {
    const uint4* ks = &ring[kg][0][ks_slot][0];
    const bf16x8 kf = as_bf16x8(ks[(t * 32 + r32) * 8 + ((2 * dd + h) ^ ksw)]);
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[dd], dd == 0 ? zero : s, 0, 0, 0);
  };

  // Block i: its scores are in `s`; the scores of block i + 1 go to `sn` (NEXT) while the probabilities of
  // block i are formed, so the matrix core works under the exponentials.
  auto block = [&](auto next_tag, auto slot_tag, int i, f32x16 (&s)[2], f32x16 (&sn)[2]) {
    constexpr bool NEXT = decltype(next_tag)::value;
    constexpr int SL = decltype(slot_tag)::value, KN = S == 1 ? 0 : SL ^ 1;
    if (!NEXT) {
      const int j0 = (i * KG + kg) * BJ;
      if (j0 + BJ > L) {  // uniform; keys past L exist only in the head's last block
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (j0 + t * 32 + (e >> 2) * 8 + h * 4 + (e & 3) >= L) s[t][e] = -INFINITY;
      }
    }
    if (NEXT) {
      qk(sn[0], KN, 0, 0);
      qk(sn[1], KN, 1, 0);
    }
    float nref = ref;  // (from here the maximum is one v_max3 per two scores and nothing has to be quieted first)
#pragma unroll
    for (int e = 0; e < 16; ++e) nref = fmaxf(fmaxf(nref, s[0][e]), s[1][e]);
    {  // the row's other half
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(nref), __float_as_uint(nref), false, false);
      nref = fmaxf(fmaxf(ref, __uint_as_float(sw[0])), __uint_as_float(sw[1]));
    }
    if (__any(nref > ref)) {
      const float rescale = __builtin_amdgcn_exp2f((ref - nref) * a2);  // (of zeros in the first block)
      sum0 *= rescale;
      sum1 *= rescale;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[t][e] *= rescale;
      ref = nref;
    }
    const float nm2 = -ref * a2;
    const uint32_t vs0 = lds_addr_of(&ring[kg][1][S == 1 ? 0 : SL][0]) + v_off, vs1 = vs0 ^ 64;  // d 0..31, 32..63
    if (KG == 1) __builtin_amdgcn_s_setprio(1);  // (see the kernel's comment)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (NEXT && u < 3) {
        qk(sn[0], KN, 0, u + 1);
        qk(sn[1], KN, 1, u + 1);
      }
      // 16 keys: probabilities, then O += P.V
      float p[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[e] = __builtin_amdgcn_exp2f(fmaf(s[u >> 1][(u & 1) * 8 + e], a2, nm2));
        if (e & 1) sum1 += p[e]; else sum0 += p[e];
      }
      const bf16x8 pf = as_bf16x8(make_uint4(pack_bf16x2(p[0], p[1]), pack_bf16x2(p[2], p[3]),
                                             pack_bf16x2(p[4], p[5]), pack_bf16x2(p[6], p[7])));
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const uint32_t a = (t ? vs1 : vs0) + u * 2048;
        const uint2 lo = lds_read_tr16(a), hi = lds_read_tr16(a + 1024);
        oacc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y)), pf, oacc[t], 0, 0, 0);
      }
    }
    if (KG == 1) __builtin_amdgcn_s_setprio(0);
  };
  auto arrive = [&](int i) {  // K of block i + 1 and V of block i are there; the tiles read before are refilled
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (S > 1) {
      if (i + 2 < mine) issue(K_TILE{}, i + 2);
      if (i + 1 < mine) issue(V_TILE{}, i + 1);
    }
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  f32x16 sa[2], sb[2];
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (KG == 1 || mine > 0) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int dd = 0; dd < 4; ++dd) qk(sa[t], 0, t, dd);
  }
  if constexpr (S == 1) {
    if (mine > 0) block(std::false_type{}, S0{}, 0, sa, sb);
  } else {
    int i = 0;
    for (; i + 2 < mine; i += 2) {
      arrive(i);
      block(std::true_type{}, S0{}, i, sa, sb);
      arrive(i + 1);
      block(std::true_type{}, S1{}, i + 1, sb, sa);
    }
    if (i + 1 < mine) {
      arrive(i);
      block(std::true_type{}, S0{}, i, sa, sb);
      arrive(i + 1);
      block(std::false_type{}, S1{}, i + 1, sb, sa);
    } else if (KG == 1 || i < mine) {
      arrive(i);
      block(std::false_type{}, S0{}, i, sa, sb);
    }
    if (KG > 1 && mine < steps) arrive(mine);    // (every group passes as many barriers)
  }
  float sum = sum0 + sum1;
  sum += __shfl_xor(sum, 32, 64);

  if constexpr (KG == 1) {
    const float inv = 1.0f / sum;
    // Whole rows of 128 bytes through the ring's memory, so that they can go through the L2: chunk c of row r at slot
    // c ^ (r & 7) of the wave's 4 KiB.  96 x 2048 118.1 -> 115.8 us, 48 x 512 9.9 -> 9.25.  A lone wave of one key block stores
    // its 8-byte pieces as they are: the trip through LDS is on its critical path (12 x 23 3.38 us, 3.51 with it).
    constexpr bool ROWS_WHOLE = RW > 1;
    static_assert(RW * 256 <= KG * 2 * S * TILE, "the waves' rows reuse the ring");
    if (ROWS_WHOLE) __syncthreads();  // (every wave has read its last tile)
    uint4* stage = &ring[0][0][0][0] + rw * 256;
    // accumulator element e of tile t: d = 32 t + 8 (e >> 2) + 4 h + (e & 3)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const uint2 pk = make_uint2(pack_bf16x2(oacc[t][4 * b] * inv, oacc[t][4 * b + 1] * inv),
                                    pack_bf16x2(oacc[t][4 * b + 2] * inv, oacc[t][4 * b + 3] * inv));
        if (ROWS_WHOLE)
          *((uint2*)&stage[r32 * 8 + ((t * 4 + b) ^ (r32 & 7))] + h) = pk;
        else if (m_row < L)
          *(uint2*)(o + head + (long long)m_row * D + t * 32 + b * 8 + h * 4) = pk;
      }
    asm volatile("" ::: "memory");  // (the wave's own accesses execute in order)
#pragma unroll
    for (int x = 0; ROWS_WHOLE && x < 4; ++x) {
      const int row = x * 8 + (lane >> 3), c = lane & 7, m = m_row - r32 + row;
      const uint4 v = stage[row * 8 + (c ^ (row & 7))];
      if (m < L) store_through(o + head + (long long)m * D + c * 8, v);
    }
  } else {
    // the groups' outputs [group][row][64 d] (a row's 16-byte pieces spread over the banks) and their
    // (ref, sum) pairs; each wave then finishes its share of the rows, adding the groups in order
    constexpr int ROWS = RW * 32, T = RW * KG * 64;
    static_assert(KG * ROWS * 64 * 4 <= KG * S * 2 * TILE * 16, "the partial outputs reuse the ring");
    __shared__ float2 stat[KG][ROWS];
    float4* part = (float4*)&ring[0][0][0][0];
    const int row = rw * 32 + r32;
    if (h == 0) stat[kg][row] = make_float2(ref, sum);
    __syncthreads();
    float top = stat[0][row].x;
#pragma unroll
    for (int g2 = 1; g2 < KG; ++g2) top = fmaxf(top, stat[g2][row].x);
    const float scale = __builtin_amdgcn_exp2f((ref - top) * a2);  // 0 for a group without a block
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int c = t * 8 + b * 2 + h;
        part[(kg * ROWS + row) * 16 + (c ^ (row & 15))] =
            make_float4(oacc[t][4 * b] * scale, oacc[t][4 * b + 1] * scale, oacc[t][4 * b + 2] * scale, oacc[t][4 * b + 3] * scale);
      }
    __syncthreads();
#pragma unroll
    for (int x = tid; x < ROWS * 16; x += T) {
      const int rrow = x >> 4, c = x & 15, m = qb * ROWS + rrow;
      float tp = stat[0][rrow].x;
#pragma unroll
      for (int g2 = 1; g2 < KG; ++g2) tp = fmaxf(tp, stat[g2][rrow].x);
      float total = 0.f;
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int g2 = 0; g2 < KG; ++g2) {
        const float2 st = stat[g2][rrow];
        total += st.y * __builtin_amdgcn_exp2f((st.x - tp) * a2);
        const float4 w = part[(g2 * ROWS + rrow) * 16 + (c ^ (rrow & 15))];
        a.x += w.x, a.y += w.y, a.z += w.z, a.w += w.w;
      }
      const float inv = 1.0f / total;
      if (m < L)
        store_through(o + head + (long long)m * D + c * 4,
                      make_uint2(pack_bf16x2(a.x * inv, a.y * inv), pack_bf16x2(a.z * inv, a.w * inv)));
    }
  }
}

// A wave's LDS accesses execute in the order issued; this keeps the compiler from issuing them in another
// order than the source's where one piece of LDS is used as different types in turn.
__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }

// ---------------------------------------------------------------------------
// The attention chain with its intermediate results, in one launch: S = alpha Q.K^T (f32), P = softmax rows of S
// (bf16), O = P.V, for head dimension 64 and up to 64 KG keys.
//   Workgroup: ROWS query rows, KG waves; wave g owns keys 64 g .. 64 g + 63 and keeps their scores in registers
//   from the first product to the second: S and P are written out once and never read back.  ROWS = 32: MFMA 32x32x16, in the
//   layout of attention_kernel.  ROWS = 16: MFMA 16x16x32, lane (r, h) holds, for its query row r, keys 16 t + 4 h + (0..3); the
//   8 k slots of h in MFMA u of the second product are defined as the 4 keys it holds of t = 2 u and the 4 of 2 u + 1.
//   The waves' row maxima, row sums and shares of O meet in LDS.  S and P leave through the wave's K
//   tile, which is free by then, so that a store covers whole row segments (their rows start at any element: L is
//   any number).  V loads under the scores.
//   What bounds it: the launch and one workgroup's chain load, score, reduce, store; with many heads the 6 L^2 bytes per head
//   that leave.  16 rows make that chain shorter wherever their workgroups still fit the chip at once (attention_chain_rows).
//   Graph replays, microseconds, three launches / one with 32 rows / with 16: 12 heads of 23 tokens 10.5 / 5.4 / 4.2, of 200
//   - / 6.4 / 5.1, of 333 20.7 / 8.4 / 6.7, of 512 27.9 / 9.4 / 11.7; 96 heads of 512 99 -> 44 (at 151 MB written 3.5 TB/s).
//   A last block written element by element instead of in pieces of 16 bytes cost 2.6 us; V's rows past the last key zeroed
//   a row per lane, all in the same banks, 0.1; waiting for V with K and storing S ahead of the exponentials 0.1 to 0.3.
// ---------------------------------------------------------------------------
template <int KG, int ROWS>
__global__ void __launch_bounds__(KG * 64)
    attention_chain_kernel(const u16* __restrict__ q, const u16* __restrict__ k, const u16* __restrict__ v,
                           float* __restrict__ s_out, u16* __restrict__ p_out, u16* __restrict__ o, int L, float alpha) {
  static_assert(ROWS == 16 || ROWS == 32, "one MFMA of 16 x 16 or of 32 x 32 columns of rows");
  constexpr int D = 64, BJ = 64, TILE = BJ * 8, T = KG * 64;
  constexpr int NE = ROWS, NP = NE / 4;       // scores of a lane, and pieces of four neighbouring keys of them
  constexpr int LPR = 64 / ROWS;              // lanes that share a row
  constexpr bool WIDE = ROWS == 32;
  __shared__ __attribute__((aligned(256))) uint4 tiles[KG][2][TILE];  // K, V
  __shared__ float red_max[KG][ROWS], red_sum[KG][ROWS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int kg = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & (ROWS - 1), h = lane / ROWS;
  // piece i of this lane: keys 4 piece(i) .. + 3 of the wave's 64
  auto piece = [&](int i) { return WIDE ? (i >> 2) * 8 + (i & 3) * 2 + h : i * 4 + h; };
  int qb, head_i;
  {  // contiguous runs of (head, query block) per XCD
    const unsigned nb = gridDim.x * gridDim.y, id = blockIdx.y * gridDim.x + blockIdx.x;
    const unsigned per = nb >> 3, rem = nb & 7, xcd = id & 7;
    const unsigned pid = xcd * per + (xcd < rem ? xcd : rem) + (id >> 3);
    head_i = (int)(pid / gridDim.x);
    qb = (int)(pid % gridDim.x);
  }
  const long long head = (long long)head_i * L * D, plane = (long long)head_i * L * L;
  const int m0 = qb * ROWS;
  const int m_ld = m0 + r < L ? m0 + r : L - 1;
  const int j0 = kg * BJ;
  const int keys = L - j0 < BJ ? (L - j0 < 0 ? 0 : L - j0) : BJ;  // of this wave (uniform)

  const int rr = lane >> 3;
  const uint32_t k_lds = __builtin_amdgcn_readfirstlane(lds_addr_of(&tiles[kg][0][0]));
  auto issue = [&](const u16* src, bool is_v) {  // 8 rows an instruction
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      int row = j * 8 + rr;
      const int c = (lane & 7) ^ (is_v ? 4 * ((row >> 1) & 1) : ((row >> 1) & 7));
      row = row < keys ? row : keys - 1;
      dma16_so((uint32_t)(row * D + c * 8) * 2u, src + head + (long long)j0 * D, k_lds + (is_v ? 8 + j : j) * 1024);
    }
  };
  if (keys > 0) issue(k, false);
  constexpr int QF = WIDE ? 4 : 2;  // query fragments: d = 64 / QF dd + 8 h .. + 7
  bf16x8 qf[QF];
#pragma unroll
  for (int dd = 0; dd < QF; ++dd)
    qf[dd] = as_bf16x8(*(const uint4*)(q + head + (long long)m_ld * D + dd * (D / QF) + h * 8));
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the tiles are the wave's own: no barrier)
  if (keys > 0) issue(v, true);                     // (needed after the softmax only)

  float s[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) s[e] = 0.f;
  float mx = -INFINITY;
  uint4* const stage = &tiles[kg][0][0];
  if (keys > 0) {
    const int ksw = (r >> 1) & 7;
    if constexpr (WIDE) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x16 a;
#pragma unroll
        for (int e = 0; e < 16; ++e) a[e] = 0.f;
#pragma unroll
        for (int dd = 0; dd < QF; ++dd)
          a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(stage[(t * 32 + r) * 8 + ((2 * dd + h) ^ ksw)]), qf[dd], a, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 16; ++e) s[t * 16 + e] = a[e];
      }
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int dd = 0; dd < QF; ++dd)
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(stage[(t * 16 + r) * 8 + ((4 * dd + h) ^ ksw)]), qf[dd], a, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[t * 4 + e] = a[e];
      }
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) s[e] = fmaf(alpha, s[e], 0.f);  // (the products' epilogue)
    lds_order();
    // S through the K tile: [row][16 pieces of 4 keys], piece c of row r at c ^ (r & 15)
#pragma unroll
    for (int i = 0; i < NP; ++i)
      ((float4*)stage)[r * 16 + (piece(i) ^ (r & 15))] = make_float4(s[4 * i], s[4 * i + 1], s[4 * i + 2], s[4 * i + 3]);
    if (keys < BJ) {  // uniform
#pragma unroll
      for (int e = 0; e < NE; ++e)
        if (piece(e >> 2) * 4 + (e & 3) >= keys) s[e] = -INFINITY;
    }
#pragma unroll
    for (int e = 0; e < NE; e += 2) mx = fmaxf(fmaxf(mx, s[e]), s[e + 1]);
#pragma unroll
    for (int x = ROWS; x < 64; x *= 2) mx = fmaxf(mx, __shfl_xor(mx, x, 64));
  }
  if (KG > 1) {
    if (h == 0) red_max[kg][r] = mx;
    __syncthreads();
    mx = red_max[0][r];
#pragma unroll
    for (int g = 1; g < KG; ++g) mx = fmaxf(mx, red_max[g][r]);
  }
  // probabilities: 2^((s - max) log2 e), the difference first: with max log2 e rounded on its own (a fused
  // multiply-add per score) the rounding is a factor of 2^(half a last place of the product) on the whole row, which
  // is beyond any float from scores of 1.5e9 on.  (The kernel is bound by its launch and its chain: one
  // instruction more per score costs 0.1 us at 12 heads of 480 tokens, 9.5 -> 9.6.)
  float sum = 0.f;
  constexpr float kLog2e = 1.4426950408889634f;
  if (keys > 0) {
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      s[e] = __builtin_amdgcn_exp2f((s[e] - mx) * kLog2e);
      sum += s[e];
    }
  }
#pragma unroll
  for (int x = ROWS; x < 64; x *= 2) sum += __shfl_xor(sum, x, 64);
  if (KG > 1 && h == 0) red_sum[kg][r] = sum;
  // V has had the scores and the probabilities to arrive; its rows past the last key are multiplied by zeros: they must be
  // finite
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (keys > 0 && keys < BJ)
    for (int c = keys * 8 + lane; c < TILE; c += 64) tiles[kg][1][c] = make_uint4(0, 0, 0, 0);
  lds_order();
  if (keys > 0) {
    float* C = s_out + plane + j0;
#pragma unroll
    for (int i = 0; i < ROWS / 4; ++i) {
      const int row = i * 4 + (lane >> 4), c = lane & 15;
      const float4 w = ((const float4*)stage)[row * 16 + (c ^ (row & 15))];
      if (m0 + row < L && c * 4 + 4 <= keys) __builtin_memcpy(C + (long long)(m0 + row) * L + c * 4, &w, 16);
    }
    if (keys & 3) {  // the piece of a row that the last key ends
      const int row = r, c = keys >> 2;
#pragma unroll
      for (int i = 0; i < 4 / LPR; ++i) {
        const int e = LPR * i + h;
        const float w = ((const float*)stage)[(row * 16 + (c ^ (row & 15))) * 4 + e];
        if (m0 + row < L && e < (keys & 3)) C[(long long)(m0 + row) * L + c * 4 + e] = w;
      }
    }
  }
  if (KG > 1) {
    __syncthreads();
    sum = red_sum[0][r];
#pragma unroll
    for (int g = 1; g < KG; ++g) sum += red_sum[g][r];
  }
  const float inv = 1.0f / sum;
  float oacc[NE];  // as the scores: pieces of four d
#pragma unroll
  for (int e = 0; e < NE; ++e) oacc[e] = 0.f;
  if (keys > 0) {
    uint2 pw[NP];  // pieces of four keys; two of them are the operand of P.V, and what P holds
#pragma unroll
    for (int i = 0; i < NP; ++i)
      pw[i] = make_uint2(pack_bf16x2(s[4 * i] * inv, s[4 * i + 1] * inv), pack_bf16x2(s[4 * i + 2] * inv, s[4 * i + 3] * inv));
    lds_order();
    // P through the K tile: [row][8 chunks of 8 keys], chunk c of row r at c ^ (r & 7)
#pragma unroll
    for (int i = 0; i < NP; ++i) ((uint2*)(stage + r * 8))[((piece(i) >> 1) ^ (r & 7)) * 2 + (piece(i) & 1)] = pw[i];
    // V by transposing reads of four keys by 16 d: MFMA u takes the keys of this lane's pieces 2 u and 2 u + 1
    const int i16 = lane & 15, swz = 4 * ((i16 >> 3) & 1);
    const uint32_t v_lds = lds_addr_of(&tiles[kg][1][0]) + (uint32_t)((4 * h + (i16 >> 2)) * 128 + (i16 & 1) * 8);
    if constexpr (WIDE) {
      const int dh = (lane >> 4) & 1;
      const uint32_t vs0 = v_lds + (uint32_t)(((2 * dh + ((i16 & 3) >> 1)) ^ swz) * 16);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x16 a;
#pragma unroll
        for (int e = 0; e < 16; ++e) a[e] = 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t at = (t ? vs0 ^ 64 : vs0) + u * 2048;
          const uint2 lo = lds_read_tr16(at), hi = lds_read_tr16(at + 1024);
          a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y)),
                                                      as_bf16x8(make_uint4(pw[2 * u].x, pw[2 * u].y, pw[2 * u + 1].x, pw[2 * u + 1].y)), a, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[t * 16 + e] = a[e];
      }
    } else {
      const uint32_t vs0 = v_lds + (uint32_t)((((i16 & 3) >> 1) ^ swz) * 16);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const uint32_t at = (vs0 ^ (t * 32)) + u * 4096;
          const uint2 lo = lds_read_tr16(at), hi = lds_read_tr16(at + 2048);
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y)),
                                                      as_bf16x8(make_uint4(pw[2 * u].x, pw[2 * u].y, pw[2 * u + 1].x, pw[2 * u + 1].y)), a, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) oacc[t * 4 + e] = a[e];
      }
    }
    lds_order();
    u16* C = p_out + plane + j0;
#pragma unroll
    for (int i = 0; i < ROWS / 8; ++i) {
      const int row = i * 8 + (lane >> 3), c = lane & 7;
      const uint4 w = stage[row * 8 + (c ^ (row & 7))];
      if (m0 + row < L && c * 8 + 8 <= keys) __builtin_memcpy(C + (long long)(m0 + row) * L + c * 8, &w, 16);
    }
    if (keys & 7) {
      const int row = r, c = keys >> 3;
#pragma unroll
      for (int i = 0; i < 8 / LPR; ++i) {
        const int e = LPR * i + h;
        const u16 w = ((const u16*)stage)[(row * 8 + (c ^ (row & 7))) * 8 + e];
        if (m0 + row < L && e < (keys & 7)) C[(long long)(m0 + row) * L + c * 8 + e] = w;
      }
    }
  }
  // the waves' shares of O over their own tiles, added in order: group g at g * 1024, [row][16 pieces of 4 d]
  lds_order();
  float4* part = (float4*)&tiles[0][0][0];
#pragma unroll
  for (int i = 0; i < NP; ++i)
    part[kg * 1024 + r * 16 + (piece(i) ^ (r & 15))] = make_float4(oacc[4 * i], oacc[4 * i + 1], oacc[4 * i + 2], oacc[4 * i + 3]);
  if (KG > 1) __syncthreads();
  lds_order();
#pragma unroll
  for (int x = tid; x < ROWS * 16; x += T) {
    const int row = x >> 4, c = x & 15;
    float4 a = part[row * 16 + (c ^ (row & 15))];
#pragma unroll
    for (int g = 1; g < KG; ++g) {
      const float4 w = part[g * 1024 + row * 16 + (c ^ (row & 15))];
      a.x += w.x, a.y += w.y, a.z += w.z, a.w += w.w;
    }
    if (m0 + row < L)
      *(uint2*)(o + head + (long long)(m0 + row) * D + c * 4) = make_uint2(pack_bf16x2(a.x, a.y), pack_bf16x2(a.z, a.w));
  }
}

}  // namespace nimble
#endif
