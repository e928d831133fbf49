// Tiles of up to 256 x 256 by four waves, one per SIMD, the halves of a ring stage read and refilled on their own.
#ifndef NIMBLE_GEMM_QUARTER_KERNEL_H_
#define NIMBLE_GEMM_QUARTER_KERNEL_H_
#include "gemm_ring_kernel.h"

namespace nimble {

// ---------------------------------------------------------------------------
// Tiles of BM x BN by four waves in two rows and two columns, one wave per SIMD with the whole register file: BM / 2 x
// BN / 2 outputs per wave (128 x 128: 256 accumulators).  Bound: MFMA, and for long K the power that MFMAs, fragment reads and
// loads take together: a wave twice as wide reads a third less from LDS per product than the eight waves of the ring kernels
// (128 KB per 64 k of a 256 x 256 tile, 192 there), which the chip turns into a higher clock.
//   LDS: S slots of 64-wide K stages, rows of 128 bytes swizzled as in the ring kernels.  With one wave per SIMD any wait
//   idles its matrix core, so a stage is multiplied in four quarters (a half of the wave's rows by a half of its columns,
//   over the stage's 64 k), and the halves of A and B are read, freed and refilled on their own: while a quarter is
//   multiplied the half that the next one needs is read into registers that the one before has left, and the loads of stage
//   s + S go where halves of stage s were read:
//     quarter      0: A0 B0     1: A0 B1     2: A1 B0     3: A1 B1
//     reads           B1 (s)       A1 (s)       A0 (s + 1)   B0 (s + 1)
//     loads, s + S    A0           B0           B1           A1
//   with a barrier ahead of quarters 0 and 2: what the next two quarters read has landed (S - 1 whole stages may be in
//   flight), and what they refill has been read by every wave.  Memory instructions stand one at a time between the MFMAs;
//   a load's M0 is written ahead of the MFMA that it follows.  Consecutive MFMAs share an operand, at the turn of a row too
//   (1 %: less toggling).
//   The loads past a tile's last stage are the next tile's first ones, so a walk over several tiles never drains its ring.
//   Arithmetic: the sums of the ring kernels in the same order, bit for bit.
//   Measured, eight waves / four: 8192^3 737 / 690 us, 8192 x 4096 x 4096 190 / 179, 16384 x 1024 x 4096 102.6 / 96.0,
//   10240 x 1024 x 4096 in 160-row tiles 69.6 / 65.6; one 64-wide stage of a 256 x 256 tile 1.39 / 1.31 us.  Without its
//   barriers and waits it is no faster; on a card where 8192^3 took 708 us as it is (1.90 GHz), 617 without the loads (2.12 GHz),
//   637 without the fragment reads, 525 without both (2.40 GHz).  Eight waves on the same ring, and in two groups that multiply and
//   read in turn, were no faster than the ring kernels and 7 % slower.  Where it does not pay: see quarter_kernel_wins.
// ---------------------------------------------------------------------------
// What one tile of a workgroup's walk hands to the next.
struct QuarterLink {
  bool next = false;    // a tile follows
  int next_m0 = 0, next_n0 = 0;
  bool filled = false;  // this tile's first two stages and its bias were asked for during the tile before
  int stores = 0;       // 1: that tile's epilogue issued exactly NST stores behind them
  int slot = 0;         // ring slot of this tile's first stage
  int parity = 0;       // its bias slot
};

template <int BM, int BN, int S, bool STAYS>
__device__ __forceinline__ int gemm_quarter_body(const GemmArgs& g, const int m0, const int n0, uint4* smem,
                                                 const QuarterLink& lk) {
  constexpr int WM = BM / 2, WN = BN / 2;
  constexpr int TM = WM / 16, TN = WN / 16;
  constexpr int H0 = (TM + 1) / 2, H1 = TM - H0;  // 16-row tiles in the two halves of a wave's rows
  constexpr int G = TN / 2;                       // 16-column tiles in either half of its columns
  static_assert(BM % 32 == 0 && H1 >= 1 && BN % 128 == 0, "whole 16 x 16 tiles in either half of a wave's rows and columns");
  constexpr int CH = 8;                       // 16-byte chunks per row and stage
  constexpr int SLOT = (BM + BN) * CH * 16;   // bytes
  constexpr int LDT = TM + TN;                // loads per wave and stage: H0, G, G, H1 of 32 rows each
  constexpr int FLIGHT = (S - 1) * LDT;       // loads that may be in flight at a barrier
  constexpr int NH = WN / 64;
  constexpr int NST = NH * (WM / 8);          // stores of the bf16 epilogue per wave
  static_assert(NST + FLIGHT <= 63 && FLIGHT + G + H1 <= 63, "the wait counter holds 63");

  const int z = blockIdx.z;
  const int stages_all = g.K >> 6;
  const int stages_per = (stages_all + (int)gridDim.y - 1) / (int)gridDim.y;
  const int stage0 = (int)blockIdx.y * stages_per;
  const int KS = (stages_all - stage0) < stages_per ? (stages_all - stage0) : stages_per;
  const u16* __restrict__ A = (const u16*)g.a + (long long)z * g.sa + (stage0 << 6);
  const u16* __restrict__ B = (const u16*)g.b + (long long)z * g.sb + (stage0 << 6);
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // (per-lane addresses are not kept alive from tile to tile)
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // row of the tile behind row q of half h of A (the halves of both rows of waves), the same for B
  auto a_row = [](int h, int q) {
    const int n = 16 * (h ? H1 : H0);
    return h * 16 * H0 + (q >= n ? WM - n : 0) + q;
  };
  auto b_row = [](int h, int q) { return h * 16 * G + (q >= 16 * G ? WN - 16 * G : 0) + q; };
  const int ld_row = tid >> 3;
  const int ld_c = (tid & 7) ^ ((ld_row >> 1) & 7);
  // loads of a stage in the order in which they are needed: H0 of A, G of B, G of B, H1 of A.  Offset of the lane, and
  // where in a slot the wave's 8 rows go.
  uint32_t off[LDT], lds_off[LDT];
  auto set_off = [&](const int tile_m0, const int tile_n0) {
#pragma unroll
    for (int u = 0; u < LDT; ++u) {
      const bool of_a = u < H0 || u >= H0 + TN;
      const int h = of_a ? u >= H0 : u >= H0 + G, q = of_a ? (h ? u - TN - H0 : u) * 32 : (u - H0 - G * h) * 32;
      int row = (of_a ? a_row(h, q + ld_row) : b_row(h, q + ld_row));
      const int last = of_a ? g.M - 1 - tile_m0 : g.N - 1 - tile_n0;
      row = row < last ? row : last;
      off[u] = (uint32_t)(row * (of_a ? g.lda : g.ldb) + ld_c * 8) * 2u;
    }
  };
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr_of(smem));
#pragma unroll
  for (int u = 0; u < LDT; ++u) {
    const bool of_a = u < H0 || u >= H0 + TN;
    const int h = of_a ? u >= H0 : u >= H0 + G, q = of_a ? (h ? u - TN - H0 : u) * 32 : (u - H0 - G * h) * 32;
    lds_off[u] = of_a ? a_row(h, q + wave * 8) * 128 : BM * 128 + b_row(h, q + wave * 8) * 128;
  }
  set_off(m0, n0);
  const u16* a_src = A + (long long)m0 * g.lda;
  const u16* b_src = B + (long long)n0 * g.ldb;
  auto src = [&](int u) { return u < H0 || u >= H0 + TN ? a_src : b_src; };

  const int fr_row = lane & 15, fr_q = lane >> 4;
  const int fr_phys = fr_q ^ ((fr_row >> 1) & 7);
  const int half = ((fr_phys ^ 4) - fr_phys);
  const uint4* a_rd = smem + (wm * WM + fr_row) * CH + fr_phys;
  const uint4* b_rd = smem + (BM + wn * WN + fr_row) * CH + fr_phys;

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  u16* const bias_slots = reinterpret_cast<u16*>(smem + S * SLOT / 16);
  u16* bias_lds = bias_slots + lk.parity * BN;
  const bool park_bias = g.epilogue != NIMBLE_EPI_NONE && !g.out_f32;
  auto fetch_bias = [&](const int tile_n0, const u16* dst) {
    if (park_bias && wave < BN / 128) {
      int n = tile_n0 + wave * 128;
      const uint32_t voff = n + 2 * lane >= g.N ? 0u : (uint32_t)lane * 4u;  // (values past N are not used)
      n = n < g.N - 2 ? n : g.N - 2;
      dma4_so(voff, (const u16*)g.bias + n, __builtin_amdgcn_readfirstlane(lds_addr_of(dst)) + wave * 256);
    }
  };
  int slot = lk.slot;
  int lax = __builtin_amdgcn_readfirstlane(lk.filled ? lk.stores : 0);
  if (!lk.filled) {
    fetch_bias(n0, bias_lds);
#pragma unroll
    for (int s = 0; s < S; ++s) {
#pragma unroll
      for (int u = 0; u < LDT; ++u) dma16_so(off[u], src(u), lds0 + s * SLOT + lds_off[u]);  // (the first tile: slot 0)
      a_src += 64;
      b_src += 64;
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(FLIGHT + G + H1) : "memory");
    __syncthreads();
  } else {
    a_src += 64 * S;
    b_src += 64 * S;
  }

  bf16x8 xa0[H0][2], xa1[H1][2], wb0[G][2], wb1[G][2];  // [tile][k half]
  auto rd_a0 = [&](int s, int x) { xa0[x % H0][x / H0] = as_bf16x8(a_rd[s * (SLOT / 16) + (x % H0) * 16 * CH + (x / H0) * half]); };
  auto rd_a1 = [&](int s, int x) { xa1[x % H1][x / H1] = as_bf16x8(a_rd[s * (SLOT / 16) + (H0 + x % H1) * 16 * CH + (x / H1) * half]); };
  auto rd_b0 = [&](int s, int x) { wb0[x % G][x / G] = as_bf16x8(b_rd[s * (SLOT / 16) + (x % G) * 16 * CH + (x / G) * half]); };
  auto rd_b1 = [&](int s, int x) { wb1[x % G][x / G] = as_bf16x8(b_rd[s * (SLOT / 16) + (G + x % G) * 16 * CH + (x / G) * half]); };
#pragma unroll
  for (int x = 0; x < 2 * H0; ++x) rd_a0(slot, x);
#pragma unroll
  for (int x = 0; x < TN; ++x) rd_b0(slot, x);

  // S - 1 whole stages may be in flight; with `lax` the previous epilogue's stores too
  auto sync = [&](int with_stores) {
    asm volatile(
        "s_waitcnt lgkmcnt(0)\n\t"
        "s_cmp_eq_u32 %0, 0\n\t"
        "s_cbranch_scc0 .Lnimble_ring_lax_%=\n\t"
        "s_waitcnt vmcnt(%2)\n"
        ".Lnimble_ring_lax_%=:\n\t"
        "s_waitcnt vmcnt(%1)\n" ::"s"(__builtin_amdgcn_readfirstlane(with_stores)),
        "n"(NST + FLIGHT), "n"(FLIGHT)
        : "memory", "scc");
    __syncthreads();
  };
  // TH x G tiles over the stage's 64 k; in between `nrd` fragment reads, then the loads u0 ... u0 + nld - 1 of a stage
  auto quarter = [&](auto& x, auto& w, auto th_tag, int j0, int i0, auto rd, int nrd, int u0, int nld, uint32_t dst, int last) {
    constexpr int TH = decltype(th_tag)::value, N = 2 * G * TH;
    const int nops = nrd + nld;
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int kh = n / (G * TH), i = n / TH % G, j = i & 1 ? TH - 1 - n % TH : n % TH;
      int u = -1;
#pragma unroll
      for (int m = (n * nops + N - 1) / N; m < ((n + 1) * nops + N - 1) / N; ++m) {
        if (m < nrd) {
          rd(m);
          asm volatile("" ::: "memory");
        } else {
          u = u0 + m - nrd;
        }
      }
      if (u >= 0)
        mfma_acc_load(acc[i0 + i][j0 + j], w[i][kh], x[j][kh], off[u], src(u), dst, lds_off[u]);
      else if (n == N - 1 && last >= 0)
        mfma_acc_last(acc[i0 + i][j0 + j], w[i][kh], x[j][kh], last);
      else
        mfma_acc(acc[i0 + i][j0 + j], w[i][kh], x[j][kh]);
    }
  };
  using T0 = std::integral_constant<int, H0>;
  using T1 = std::integral_constant<int, H1>;
  int step = 64;
  for (int ks = 0, end = KS - S;; end = KS) {
    for (; ks < end; ++ks) {
      const uint32_t dst = lds0 + slot * SLOT;
      const int next = S == 2 ? slot ^ 1 : slot + 1 == S ? 0 : slot + 1;
      sync(ks < S ? lax : 0);
      quarter(xa0, wb0, T0{}, 0, 0, [&](int m) { rd_b1(slot, m); }, TN, 0, H0, dst, -1);
      quarter(xa0, wb1, T0{}, 0, G, [&](int m) { rd_a1(slot, m); }, 2 * H1, H0, G, dst, -1);
      sync(ks < S - 1 ? lax : 0);
      quarter(xa1, wb0, T1{}, H0, 0, [&](int m) { rd_a0(next, m); }, 2 * H0, H0 + G, G, dst, -1);
      quarter(xa1, wb1, T1{}, H0, G, [&](int m) { rd_b0(next, m); }, TN, H0 + TN, H1, dst, ks + 1 >= KS);
      slot = next;
      a_src += step;
      b_src += step;
    }
    if (end == KS) break;
    // the last S stages load the next tile's first; if there is none, the last stage again, never read
    if (lk.next) {
      set_off(lk.next_m0, lk.next_n0);
      a_src = A + (long long)lk.next_m0 * g.lda;
      b_src = B + (long long)lk.next_n0 * g.ldb;
    } else {
      a_src -= 64;
      b_src -= 64;
      step = 0;
    }
  }
  // (not before this tile's barriers: its slot was the last one's of the tile before)
  if (lk.next) fetch_bias(lk.next_n0, bias_slots + (lk.parity ^ 1) * BN);
  const bool edge = m0 + BM > g.M || n0 + BN > g.N;

  // epilogue.  acc[i][j][v] is row m = wm*WM + 16 j + fr_row, column n = wn*WN + 16 i + 4 fr_q + v.
  const float alpha = g.alpha;
  const int epi = g.epilogue;
  float bias4[TN][4];
#pragma unroll
  for (int i = 0; i < TN; ++i) {
#pragma unroll
    for (int v = 0; v < 4; ++v) bias4[i][v] = 0.f;
    if (epi != NIMBLE_EPI_NONE && (!edge || park_bias || n0 + wn * WN + i * 16 + fr_q * 4 < g.N)) {
      const uint2 bb = park_bias ? *(const uint2*)(bias_lds + wn * WN + i * 16 + fr_q * 4)
                                 : *(const uint2*)((const u16*)g.bias + n0 + wn * WN + i * 16 + fr_q * 4);
      bias4[i][0] = bf2f((u16)(bb.x & 0xffff));
      bias4[i][1] = bf2f((u16)(bb.x >> 16));
      bias4[i][2] = bf2f((u16)(bb.y & 0xffff));
      bias4[i][3] = bf2f((u16)(bb.y >> 16));
    }
  }
  auto finish = [&](auto gelu_tag, auto edge_tag) -> int {
    constexpr bool GELU = decltype(gelu_tag)::value;
    const bool edge = decltype(edge_tag)::value;
    if (g.out_f32) {
      float* C = (float*)g.c + (long long)z * g.sc + (long long)blockIdx.y * g.M * g.ldc;
      const bool keep = STAYS || partial_sums_stay(g, gridDim.y);
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        const int m = m0 + wm * WM + j * 16 + fr_row;
        if (edge && m >= g.M) continue;
#pragma unroll
        for (int i = 0; i < TN; ++i) {
          const int n = n0 + wn * WN + i * 16 + fr_q * 4;
          if (edge && n >= g.N) continue;
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = fmaf(alpha, acc[i][j][e], bias4[i][e]);
          epilogue_of<GELU>(v);
          const float4 o = make_float4(v[0], v[1], v[2], v[3]);
          if (keep)
            *(float4*)(C + (long long)m * g.ldc + n) = o;
          else
            store_through(C + (long long)m * g.ldc + n, __builtin_bit_cast(uint4, o));
        }
      }
      return 0;
    }
    u16* C = (u16*)g.c + (long long)z * g.sc;
    // bf16 through the wave's own staging area, 16 rows at a time: [NH][16 rows][128 bytes], chunk c of row r at slot
    // c ^ ((r >> 1) & 7), written back out as full 128-byte lines, while the next 16 rows are computed.
    unsigned char* region = (unsigned char*)smem + S * SLOT + 2 * BN * 2 + wave * (16 * WN * 2);
    uint4 line[2 * NH];
    auto put = [&](int j) {
#pragma unroll
      for (int x = 0; x < 2 * NH; ++x) {
        const int row = (x & 1) * 8 + (lane >> 3), c = lane & 7;
        const int m = m0 + wm * WM + j * 16 + row, n = n0 + wn * WN + (x >> 1) * 64 + c * 8;
        if (edge && (m >= g.M || n >= g.N)) continue;
        store_out<STAYS>(C + (long long)m * g.ldc + n, line[x]);
      }
    };
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      uint2 pk[TN];
#pragma unroll
      for (int i = 0; i < TN; i += 2) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = fmaf(alpha, acc[i + (e >> 2)][j][e & 3], bias4[i + (e >> 2)][e & 3]);
        epilogue_of<GELU>(v);
        pk[i] = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
        pk[i + 1] = make_uint2(pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
      }
#pragma unroll
      for (int i = 0; i < TN; ++i) asm volatile("" : "+v"(pk[i].x), "+v"(pk[i].y));  // (computed ahead of the stores)
      if (j > 0) put(j - 1);
#pragma unroll
      for (int i = 0; i < TN; ++i) {
        const int col = (i & 3) * 16 + fr_q * 4;
        const int chunk = (col >> 3) ^ ((fr_row >> 1) & 7);
        *(uint2*)(region + (i >> 2) * (16 * 128) + fr_row * 128 + chunk * 16 + (col & 4) * 2) = pk[i];
      }
#pragma unroll
      for (int x = 0; x < 2 * NH; ++x) {
        const int row = (x & 1) * 8 + (lane >> 3), c = lane & 7;
        line[x] = *(const uint4*)(region + (x >> 1) * (16 * 128) + row * 128 + ((c ^ ((row >> 1) & 7)) * 16));
      }
    }
    put(TM - 1);
    return edge ? 0 : 1;
  };
  if (edge) return epi == NIMBLE_EPI_BIAS_GELU_ERF ? finish(std::true_type{}, std::true_type{}) : finish(std::false_type{}, std::true_type{});
  return epi == NIMBLE_EPI_BIAS_GELU_ERF ? finish(std::true_type{}, std::false_type{}) : finish(std::false_type{}, std::false_type{});
}

template <int BM, int BN, int S, bool STAYS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
    gemm_quarter_kernel(GemmArgs g, int tiles_m, int tiles_n, int group_m) {
  constexpr int kUint4 = S * (BM + BN) * 8 + 2 * (BN / 8) + 4 * 16 * (BN / 2) * 2 / 16;
  static_assert(kUint4 * 16 <= 160 * 1024, "ring, bias and staging areas in LDS");
  __shared__ __attribute__((aligned(16))) uint4 smem[kUint4];
  const int tiles_total = tiles_m * tiles_n;
  const int turn = (g.K >> 6) % S;  // (several tiles: one slice only)
  QuarterLink lk;
  int tile_m, tile_n;
  tile_of_block(blockIdx.x, tiles_total, tiles_m, tiles_n, group_m, tile_m, tile_n);
  lk.next_m0 = tile_m * BM;
  lk.next_n0 = tile_n * BN;
  for (int t = blockIdx.x; t < tiles_total; t += gridDim.x) {
    const int m0 = lk.next_m0, n0 = lk.next_n0;
    lk.next = t + (int)gridDim.x < tiles_total;
    if (lk.next) {
      tile_of_block(t + (int)gridDim.x, tiles_total, tiles_m, tiles_n, group_m, tile_m, tile_n);
      lk.next_m0 = tile_m * BM;
      lk.next_n0 = tile_n * BN;
    }
    lk.stores = gemm_quarter_body<BM, BN, S, STAYS>(g, m0, n0, smem, lk);
    lk.filled = true;
    lk.slot = (lk.slot + turn) % S;
    lk.parity ^= 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the loads past the last tile)
}

}  // namespace nimble
#endif
