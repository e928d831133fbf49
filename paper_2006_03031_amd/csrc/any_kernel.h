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
//   KG = 4: four groups of four waves take the stages in turn and add their sums at the end.
//   What bounds it: a few hundred tiles of some ten stages are the whole launch, so the chain load ->
//   LDS -> MFMA per stage (0.32 us at 64 x 64, 0.5 with rows that start at odd addresses: a 16-byte load
//   then spans two pieces of a line).  Measured, 515 x 1001 x 1003 to f32: 671 us with the scalar kernel
//   it replaces (one thread per output) -> 13.3 (one group, four register sets) -> 12.1 (two groups) -> 11.5 (four
//   groups, two register sets each; with four 12.7), the same with K = 1000 9.4; 500 x 500 x 2003 20.6 -> 18.0 -> 16.8;
//   12 x 333 x 64 x 333 as A.B 88 -> 6.6 us.  128 x 128 tiles were measured too: no faster even at
//   8000 x 1001 x 1003 (54 us against 51), half the speed on small grids.
//   THROUGH: f32 outputs are written through the L2s (see any_output_stays).
// ---------------------------------------------------------------------------
template <bool KN, int P, int KG, bool THROUGH>
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

  uint4 ra[P][A_CH], rb[P][B_CH];
  const int KT_all = (K + 63) >> 6;
  const int KT = (KT_all - grp + KG - 1) / KG;  // stages of this group of four waves: grp, grp + KG, ...
  const int KT0 = (KT_all + KG - 1) / KG;       // of group 0, which has the most
  auto load = [&](auto set_tag, int s) {
    constexpr int SET = decltype(set_tag)::value;
    const int k0 = (s * KG + grp) << 6;
    if (k0 + 64 <= K) {  // uniform
#pragma unroll
      for (int i = 0; i < A_CH; ++i) ra[SET][i] = load8_unaligned(a_src[i] + k0);
      if (!KN) {
#pragma unroll
        for (int i = 0; i < B_CH; ++i) rb[SET][i] = load8_unaligned(b_src[i] + k0);
      }
    } else {
      const int left = K - (k0 + ld_c * 8);
#pragma unroll
      for (int i = 0; i < A_CH; ++i)
        ra[SET][i] = left >= 8 ? load8_unaligned(a_src[i] + k0)
                               : (left > 0 ? load8_tail(a_src[i] + k0, left, K) : make_uint4(0, 0, 0, 0));
      if (!KN) {
#pragma unroll
        for (int i = 0; i < B_CH; ++i)
          rb[SET][i] = left >= 8 ? load8_unaligned(b_src[i] + k0)
                                 : (left > 0 ? load8_tail(b_src[i] + k0, left, K) : make_uint4(0, 0, 0, 0));
      }
    }
    if (KN) {
#pragma unroll
      for (int i = 0; i < B_CH; ++i) {
        const int k = k0 + tid / NC + i * (256 / NC);
        const u16* src = b_src[i] + (long long)k * g.ldb;
        rb[SET][i] = k >= K || n_left <= 0 ? make_uint4(0, 0, 0, 0)
                                           : (n_left >= 8 ? load8_unaligned(src) : load8_tail(src, n_left, N));
      }
    }
  };
  auto store = [&](auto set_tag, int buf) {
    constexpr int SET = decltype(set_tag)::value;
#pragma unroll
    for (int i = 0; i < A_CH; ++i) smem[buf][phys(ld_row + 32 * i, ld_c)] = ra[SET][i];
#pragma unroll
    for (int i = 0; i < B_CH; ++i)
      smem[buf][BM * 8 + (KN ? phys_kn(tid / NC + i * (256 / NC), tid % NC) : phys(ld_row + 32 * i, ld_c))] = rb[SET][i];
  };

  const int r = lane & 15, gq = lane >> 4;
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
    if (s + 1 < KT) store(std::integral_constant<int, (U + 1) % P>{}, (U + 1) & 1);
    __syncthreads();
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  using S2 = std::integral_constant<int, 2 % P>;
  using S3 = std::integral_constant<int, 3 % P>;
  if (KT > 0) load(S0{}, 0);
  if (KT > 1) load(S1{}, 1);
  if (P > 2 && KT > 2) load(S2{}, 2);
  if (P > 2 && KT > 3) load(S3{}, 3);
  if (KT > 0) store(S0{}, 0);
  __syncthreads();
  for (int s = 0; s < KT0; s += P) {  // (every group walks KT0 stages: the barriers are the workgroup's)
    stage(s, S0{});
    if (s + 1 < KT0) stage(s + 1, S1{});
    if (P > 2 && s + 2 < KT0) stage(s + 2, S2{});
    if (P > 2 && s + 3 < KT0) stage(s + 3, S3{});
  }
  if constexpr (KG > 1) {  // the other groups hand their sums to the first, which adds them in order and finishes the tile
    static_assert(4 * TM * TN * 64 <= 2 * BUF, "the partial sums reuse a group's operand buffers");
    if (grp > 0) {
      f32x4* part = (f32x4*)&smem_all[grp][0][0] + wave * (TM * TN * 64) + lane;
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) part[(i * TM + j) * 64] = acc[i][j];
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g2 = 1; g2 < KG; ++g2) {
      const f32x4* part = (const f32x4*)&smem_all[g2][0][0] + wave * (TM * TN * 64) + lane;
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] += part[(i * TM + j) * 64];
    }
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
    for (int v = 0; v < 4; ++v) {
      const int n = n_base + i * 16 + gq * 4 + v;
      bias4[i][v] = (epi != NIMBLE_EPI_NONE && n < N) ? bf2f(((const u16*)g.bias)[n]) : 0.f;
    }
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
