// Matrix-core GEMM for any M, N, K, row stride and B layout: operands of any alignment.
#ifndef NIMBLE_ANY_KERNEL_H_
#define NIMBLE_ANY_KERNEL_H_
#include <type_traits>

#include "device_common.h"

namespace nimble {

// ---------------------------------------------------------------------------
// C = epi(alpha A.B + bias) with no condition on the shape.  A row of an operand with K % 8 != 0
// starts at any even address, so neither the direct global->LDS loads nor aligned vector loads can
// fetch it; here every lane brings 16-byte chunks through registers with unaligned loads.
//   Tile 64 x 64, 4 waves (2 x 2), stages of 64 k, two LDS buffers, one barrier per stage; the
//   chunks of the next P stages are on their way while a stage is multiplied (P register sets, 2 or 4).  K past
//   the end is zero-filled in the chunk that holds it, rows past M (N) repeat the last one and are
//   never stored.
//   KN: B is [K, N]; its tile keeps its rows (64 k of 64 n) in LDS and the fragments come out of
//   the transposing LDS read.
//   KG = 4: four groups of four waves take the stages in turn and add their sums at the end, each a quarter of the tile.
//   ODD: K is odd, every other row of either operand starts at an odd element.  16 waves of one compute unit load rows of 128 bytes
//   from the L2 at 114 KB per us where each lane's address is a whole 32-bit word, at 35 where it is not, at 54 where every other
//   row is not.  So such rows are loaded from the element before and moved down on the way to LDS; the word behind a stage's
//   last chunk is loaded by one lane per row (by all lanes, or all rows, it cost as much as it saved).  With four groups
//   only: in one group these words take the kernel from four workgroups per compute unit to three, 836 tiles (4819 x 665 x 641) 20.6 ->
//   23.6 us, 912 (1002 x 3587 x 453) 18.6 -> 20.6, without them 20.4 and 17.7; below 768 tiles they would gain 1 %.
//   What bounds it: a few hundred tiles of some ten stages are the whole launch, so that it is the chain load ->
//   LDS -> MFMA of one tile's stages.  By time stamps, 515 x 1001 x 1003 to f32: first stages 1.7 us, the other three rounds of
//   four 3.6, the end of the tile 1.7, launch 1.5: 8.7 us; before the words, with a K tail that waited for its loads one by one, and
//   with the first group alone at the end 10.7.  515 x 1001 x 1008 8.4 -> 7.8, x 64 5.2 -> 4.4, x 2003 16.9 -> 15.3.  Measured
//   earlier, 515 x 1001 x 1003 to f32: 671 us with the scalar kernel it replaces (one thread per output) -> 13.3 (one
//   group, four register sets) -> 12.1 (two groups) -> 11.5 (four groups, two register sets each; with four
//   12.7), the same with K = 1000 9.4; 500 x 500 x 2003 20.6 -> 18.0 -> 16.8;
//   12 x 333 x 64 x 333 as A.B 88 -> 6.6 us.  128 x 128 tiles were measured too: no faster even at
//   8000 x 1001 x 1003 (54 us against 51), half the speed on small grids.
//   THROUGH: f32 outputs are written through the L2s (see any_output_stays).
// ---------------------------------------------------------------------------
template <bool KN, int P, int KG, bool THROUGH, bool ODD>
__global__ void __launch_bounds__(256 * KG) any_kernel(GemmArgs g, int tiles_m, int tiles_n) {
  constexpr int BM = 64, BN = 64;
  constexpr int A_CH = BM * 8 / 256, B_CH = BN * 8 / 256;  // 16-byte chunks per thread and stage
  constexpr int WM = BM / 2, WN = BN / 2, TM = WM / 16, TN = WN / 16;
  constexpr int ELD = WN + 4;  // floats per row of a wave's output staging area
  constexpr int BUF = (BM + BN) * 8;
  __shared__ __attribute__((aligned(16))) uint4 smem_all[KG][2][BUF];
  static_assert(4 * 16 * ELD * 4 <= 2 * BUF * 16, "the output staging reuses the operand buffers");

  const int grp = KG > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0;
  uint4(*smem)[BUF] = smem_all[grp];
  const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int z = blockIdx.z;
  const int M = g.M, N = g.N, K = g.K;
  int tm, tn;
  tile_of_block(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, tiles_m < 4 ? tiles_m : 4, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const u16* __restrict__ A = (const u16*)g.a + (long long)z * g.sa;
  const u16* __restrict__ B = (const u16*)g.b + (long long)z * g.sb;

  const int ld_row = tid >> 3, ld_c = tid & 7;  // K-contiguous operands: chunk ld_c of rows ld_row + 32 i
  constexpr int NC = BN / 8;                    // KN: chunks per k row
  const u16* a_src[A_CH];
  const u16* b_src[B_CH];
#pragma unroll
  for (int i = 0; i < A_CH; ++i) {
    const int row = m0 + ld_row + 32 * i;
    a_src[i] = A + (long long)(row < M ? row : M - 1) * g.lda + ld_c * 8;
  }
#pragma unroll
  for (int i = 0; i < B_CH; ++i) {
    if (KN) {
      b_src[i] = B + n0 + (tid % NC) * 8;
    } else {
      const int row = n0 + ld_row + 32 * i;
      b_src[i] = B + (long long)(row < N ? row : N - 1) * g.ldb + ld_c * 8;
    }
  }
  const int n_left = N - (n0 + (tid % NC) * 8);  // KN: columns of this thread's chunk that exist

  // physical chunk of (row, chunk): rows are 8 chunks; for a KN tile (NC chunks per k row) pairs of
  // chunks stay together, spread so that the 8 rows a transposing read touches fall into different banks
  auto phys = [](int row, int c) { return row * 8 + (c ^ ((row >> 1) & 7)); };
  auto phys_kn = [](int k, int c) {
    const int f = ((k >> 1) & 1) | (((k >> 3) & 1) << 1);
    return k * NC + (c ^ (f << 1));
  };

  // ODD: some rows start at an odd element.  These are loaded from the element before, where a whole 32-bit word starts (a
  // 16-byte load whose address is not one takes three times as long), and moved down on their way to LDS, for which a
  // stage's last chunk needs the word behind it: shifts of this thread's rows, 0 or 16 bits.
  static_assert(!ODD || (!KN && KG > 1), "rows of a [K, N] operand, and those of one group, are loaded as they are");
  uint32_t sh_a[A_CH], sh_b[B_CH];
#pragma unroll
  for (int i = 0; i < A_CH; ++i) sh_a[i] = ODD ? ((uint32_t)(uintptr_t)a_src[i] & 2u) * 8u : 0u;
#pragma unroll
  for (int i = 0; i < B_CH; ++i) sh_b[i] = ODD ? ((uint32_t)(uintptr_t)b_src[i] & 2u) * 8u : 0u;
  uint4 ra[P][A_CH], rb[P][B_CH];
  uint32_t na[P][A_CH], nb[P][B_CH];
  const int KT_all = (K + 63) >> 6;
  const int KT = (KT_all - grp + KG - 1) / KG;  // stages of this group of four waves: grp, grp + KG, ...
  const int KT0 = (KT_all + KG - 1) / KG;       // of group 0, which has the most
  auto chunk_kn = [&](int i, int k0) {
    const int k = k0 + tid / NC + i * (256 / NC);
    const u16* src = b_src[i] + (long long)k * g.ldb;
    return k >= K || n_left <= 0 ? make_uint4(0, 0, 0, 0) : (n_left >= 8 ? load8_unaligned(src) : load8_tail(src, n_left, N));
  };
  auto load = [&](auto set_tag, int s) {
    constexpr int SET = decltype(set_tag)::value;
    const int k0 = (s * KG + grp) << 6;
    // K past the end is zeroed on the way to LDS: of a chunk that holds it the row's last eight elements are loaded.  (No branch:
    // where two loads meet in one register the compiler may copy, and wait for, what is meant to be on its way.)
    const bool whole = k0 + 64 <= K;  // (uniform)
    const int k = whole || k0 + ld_c * 8 <= K - 8 ? k0 : K - 8 - ld_c * 8;
    auto rows = [&](uint4* v, uint32_t* next, const u16* const* src, const uint32_t* sh, int n) {
#pragma unroll
      for (int i = 0; i < n; ++i) {
        const char* p = (const char*)(src[i] + k) - (ODD && whole ? sh[i] >> 3 : 0u);
        v[i] = load8_unaligned((const u16*)p);
        // (K is odd: the row goes on behind a whole stage)
        if (ODD && whole && ld_c == 7 && sh[i] != 0) next[i] = *(const uint32_t*)(p + 16);
      }
    };
    rows(ra[SET], na[SET], a_src, sh_a, A_CH);
    if (!KN) rows(rb[SET], nb[SET], b_src, sh_b, B_CH);
    if (KN) {
#pragma unroll
      for (int i = 0; i < B_CH; ++i) rb[SET][i] = chunk_kn(i, k0);
    }
  };
  // Chunks of stage s as they go to LDS.  (The tail is told apart once for all of them: chunk by chunk every one waited for its own load
  // behind a branch, 2 % of launches of more tiles than compute units.)
  auto store = [&](auto set_tag, int buf, int s) {
    constexpr int SET = decltype(set_tag)::value;
    const int k0 = (s * KG + grp) << 6, left = K - (k0 + ld_c * 8), n = left < 0 ? 0 : left > 8 ? 8 : left;
    auto rows = [&](auto tail) {
      auto settle = [&](const uint4& v, uint32_t next, uint32_t sh) {
        if constexpr (decltype(tail)::value) return keep_first8(v, n);
        return ODD ? shift8(v, next, sh, ld_c == 7) : v;
      };
#pragma unroll
      for (int i = 0; i < A_CH; ++i) smem[buf][phys(ld_row + 32 * i, ld_c)] = settle(ra[SET][i], na[SET][i], sh_a[i]);
      if (!KN) {
#pragma unroll
        for (int i = 0; i < B_CH; ++i) smem[buf][BM * 8 + phys(ld_row + 32 * i, ld_c)] = settle(rb[SET][i], nb[SET][i], sh_b[i]);
      }
    };
    if (k0 + 64 > K) rows(std::true_type());
    else rows(std::false_type());
    if (KN) {
#pragma unroll
      for (int i = 0; i < B_CH; ++i) smem[buf][BM * 8 + phys_kn(tid / NC + i * (256 / NC), tid % NC)] = rb[SET][i];
    }
  };

  const int r = lane & 15, gq = lane >> 4;
  // One group: the bias of this lane's columns, ahead of the operands.  (Behind the products, one guarded load after the other, it was a
  // trip to memory at the end of every tile: 804 x 1465 x 91 to f32 with a bias 7.4 us, so 5.9.)
  uint32_t bias16[TN][4] = {};
  if (KG == 1 && g.epilogue != NIMBLE_EPI_NONE) {
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int n = n0 + wn * WN + i * 16 + gq * 4 + v;
        bias16[i][v] = ((const u16*)g.bias)[n < N ? n : N - 1];
      }
  }
  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](int buf) {
    const uint4* as = &smem[buf][0];
    const uint4* bs = as + BM * 8;
    const uint32_t bs_lds = lds_addr_of(bs);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      bf16x8 xa[TM], wb[TN];
#pragma unroll
      for (int j = 0; j < TM; ++j) xa[j] = as_bf16x8(as[phys(wm * WM + j * 16 + r, h * 4 + gq)]);
#pragma unroll
      for (int i = 0; i < TN; ++i) {
        if (KN) {
          // lane group gq: k rows 8 gq .. 8 gq + 7 of this half, 16 columns of tile i, four rows at a time
          const int k = h * 32 + gq * 8 + (r >> 2);
          const int c = (wn * WN + i * 16) / 8 + ((r & 3) >> 1);
          const uint2 lo = lds_read_tr16(bs_lds + phys_kn(k, c) * 16 + (r & 1) * 8);
          const uint2 hi = lds_read_tr16(bs_lds + phys_kn(k + 4, c) * 16 + (r & 1) * 8);
          wb[i] = as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y));
        } else {
          wb[i] = as_bf16x8(bs[phys(wn * WN + i * 16 + r, h * 4 + gq)]);
        }
      }
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wb[i], xa[j], acc[i][j], 0, 0, 0);
    }
  };

  // stage s: its operands lie in LDS buffer s & 1; register set s % P is free and takes stage s + P
  auto stage = [&](int s, auto u_tag) {
    constexpr int U = decltype(u_tag)::value;
    if (s + P < KT) load(u_tag, s + P);
    if (KG == 1 || s < KT) multiply(U & 1);
    if (s + 1 < KT) store(std::integral_constant<int, (U + 1) % P>{}, (U + 1) & 1, s + 1);
    __syncthreads();
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  using S2 = std::integral_constant<int, 2 % P>;
  using S3 = std::integral_constant<int, 3 % P>;
  if (K >= 8) {
    if (KT > 0) load(S0{}, 0);
    if (KT > 1) load(S1{}, 1);
    if (P > 2 && KT > 2) load(S2{}, 2);
    if (P > 2 && KT > 3) load(S3{}, 3);
    if (KT > 0) store(S0{}, 0, 0);
  } else if (KT > 0) {  // one stage, of one chunk per row that no load of eight elements fits
    auto row = [&](const u16* p) { return ld_c == 0 ? load8_tail(p, K, K) : make_uint4(0, 0, 0, 0); };
#pragma unroll
    for (int i = 0; i < A_CH; ++i) smem[0][phys(ld_row + 32 * i, ld_c)] = row(a_src[i]);
#pragma unroll
    for (int i = 0; i < B_CH; ++i)
      smem[0][BM * 8 + (KN ? phys_kn(tid / NC + i * (256 / NC), tid % NC) : phys(ld_row + 32 * i, ld_c))] =
          KN ? chunk_kn(i, 0) : row(b_src[i]);
  }
  __syncthreads();
  for (int s = 0; s < KT0; s += P) {  // (every group walks KT0 stages: the barriers are the workgroup's)
    stage(s, S0{});
    if (s + 1 < KT0) stage(s + 1, S1{});
    if (P > 2 && s + 2 < KT0) stage(s + 2, S2{});
    if (P > 2 && s + 3 < KT0) stage(s + 3, S3{});
  }
  if constexpr (KG > 1) {
    // Each group leaves its sums in its first operand buffer, then group g adds those of sub-tile g of every wave in the order
    // of the groups and finishes it; the finished tile meets in group 0's second buffer, from where all waves store whole rows
    // of it.  (Added and finished by the first group alone this took 2.2 us of 9.6 at 515 x 1001 x 1003.)
    static_assert(TM * TN == KG && 4 * TM * TN * 64 <= BUF && BM * BN * 4 <= BUF * 16, "sums and tile reuse the operand buffers");
    f32x4* mine = (f32x4*)&smem[0][0] + wave * (KG * 64) + lane;
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j) mine[(i * TM + j) * 64] = acc[i][j];
    const int row = wm * WM + (grp % TM) * 16 + r, col = wn * WN + (grp / TM) * 16 + gq * 4;  // of the tile
    float bias[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) bias[v] = g.epilogue != NIMBLE_EPI_NONE && n0 + col + v < N ? bf2f(((const u16*)g.bias)[n0 + col + v]) : 0.f;
    __syncthreads();
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g2 = 0; g2 < KG; ++g2) {
      const f32x4 part = ((const f32x4*)&smem_all[g2][0][0])[wave * (KG * 64) + grp * 64 + lane];
      sum = g2 == 0 ? part : sum + part;
    }
    float4* tile = (float4*)&smem_all[0][1][0];  // 16 pieces of 4 columns per row, spread over the banks
    tile[row * 16 + ((col >> 2) ^ (row & 15))] =
        make_float4(epilogue(sum[0], g.alpha, bias[0], g.epilogue), epilogue(sum[1], g.alpha, bias[1], g.epilogue),
                    epilogue(sum[2], g.alpha, bias[2], g.epilogue), epilogue(sum[3], g.alpha, bias[3], g.epilogue));
    __syncthreads();
    constexpr int ROWS = BM / (4 * KG);
    const int row0 = (grp * 4 + wave) * ROWS;
    if (g.out_f32) {
      float* C = (float*)g.c + (long long)z * g.sc;
#pragma unroll
      for (int p = 0; p < ROWS; ++p) {
        const int m = row0 + p, n = n0 + lane;
        const float v = ((const float*)&tile[m * 16 + ((lane >> 2) ^ (m & 15))])[lane & 3];
        if (m0 + m < M && n < N) {
          if (THROUGH)
            store_through(&C[(long long)(m0 + m) * g.ldc + n], v);
          else
            C[(long long)(m0 + m) * g.ldc + n] = v;
        }
      }
    } else {
      u16* C = (u16*)g.c + (long long)z * g.sc;
      const bool pairs = (g.ldc & 1) == 0;  // rows start at whole 32-bit words
#pragma unroll
      for (int p = 0; p < ROWS / 2; ++p) {
        const int m = row0 + 2 * p + (lane >> 5), pair = lane & 31, n = n0 + 2 * pair;
        const float2 v = ((const float2*)&tile[m * 16 + ((pair >> 1) ^ (m & 15))])[pair & 1];
        const uint32_t pk = pack_bf16x2(v.x, v.y);
        if (m0 + m < M && n < N) {
          u16* dst = C + (long long)(m0 + m) * g.ldc + n;
          if (pairs) {  // (N even: both columns exist)
            *(uint32_t*)dst = pk;
          } else {
            dst[0] = (u16)(pk & 0xffff);
            if (n + 1 < N) dst[1] = (u16)(pk >> 16);
          }
        }
      }
    }
    return;
  }

  // epilogue: 16 rows at a time through the wave's own staging area, written back row by row so that a
  // wave's stores cover contiguous memory whatever the alignment of the output rows
  const int epi = g.epilogue;
  const float alpha = g.alpha;
  float* out_lds = (float*)&smem[0][0] + wave * (16 * ELD);
  const int n_base = n0 + wn * WN;
  float bias4[TN][4];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) bias4[i][v] = bf2f((u16)bias16[i][v]);
  const bool pairs = (g.ldc & 1) == 0;  // bf16 rows start at whole 32-bit words
#pragma unroll
  for (int j = 0; j < TM; ++j) {
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      float4 o;
      o.x = epilogue(acc[i][j][0], alpha, bias4[i][0], epi);
      o.y = epilogue(acc[i][j][1], alpha, bias4[i][1], epi);
      o.z = epilogue(acc[i][j][2], alpha, bias4[i][2], epi);
      o.w = epilogue(acc[i][j][3], alpha, bias4[i][3], epi);
      *(float4*)(out_lds + r * ELD + i * 16 + gq * 4) = o;
    }
    // (wave-private: a wave's LDS accesses execute in order)
    if (g.out_f32) {
      constexpr int RP = 64 / WN;  // rows per store
      float* C = (float*)g.c + (long long)z * g.sc;
#pragma unroll
      for (int p = 0; p < 16 / RP; ++p) {
        const int row = p * RP + lane / WN, col = lane % WN;
        const int m = m0 + wm * WM + j * 16 + row, n = n_base + col;
        const float v = out_lds[row * ELD + col];
        if (m < M && n < N) {
          if (THROUGH)
            store_through(&C[(long long)m * g.ldc + n], v);
          else
            C[(long long)m * g.ldc + n] = v;
        }
      }
    } else {
      constexpr int LW = WN / 2, RP = 64 / LW;  // lanes per row (two columns each), rows per store
      u16* C = (u16*)g.c + (long long)z * g.sc;
#pragma unroll
      for (int p = 0; p < 16 / RP; ++p) {
        const int row = p * RP + lane / LW, col = (lane % LW) * 2;
        const int m = m0 + wm * WM + j * 16 + row, n = n_base + col;
        const float2 v = *(const float2*)(out_lds + row * ELD + col);
        const uint32_t pk = pack_bf16x2(v.x, v.y);
        if (m < M && n < N) {
          u16* dst = C + (long long)m * g.ldc + n;
          if (pairs) {  // (N even: both columns exist)
            *(uint32_t*)dst = pk;
          } else {
            dst[0] = (u16)(pk & 0xffff);
            if (n + 1 < N) dst[1] = (u16)(pk >> 16);
          }
        }
      }
    }
  }
}

}  // namespace nimble
#endif
