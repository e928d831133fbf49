// Device-side helpers shared by every kernel: bf16 conversion, the dense epilogue, direct
// global->LDS loads, the workgroup-to-tile map.
#ifndef NIMBLE_DEVICE_COMMON_H_
#define NIMBLE_DEVICE_COMMON_H_
#include <hip/hip_runtime.h>

#include <cstdint>

#include "nimble_internal.h"

namespace nimble {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16;

__device__ __forceinline__ float bf2f(u16 b) { return __uint_as_float(((uint32_t)b) << 16); }

// float32 -> bfloat16, round to nearest, ties to even.
__device__ __forceinline__ u16 f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
  u += 0x7fffu + ((u >> 16) & 1u);
  return (u16)(u >> 16);
}

// gelu(v) = v/2 (1 + erf(v / sqrt 2)), evaluated as v * sigmoid(a v + b v^3 + c v^5) with
// a = 1.5950, b = 0.074011, c = -0.00070303 (a least-squares fit of the odd quintic to the erf form
// on |v| <= 9, the constants below being -log2(e) times these; largest deviation 2.5e-5, an order of
// magnitude below the bfloat16 spacing of the result; v^2 is clamped at 81, beyond which the
// sigmoid is 0 or 1): seven ordinary instructions plus the hardware exp2 and reciprocal.  The
// epilogue of a GELU layer is bound by exactly these instructions (128 outputs per lane with
// nothing to overlap them): the three-term rational-times-Gaussian erf of Abramowitz & Stegun
// 7.1.25 (same accuracy, eleven instructions) was the previous form, 7.1.26 and the library erff
// cost more still.  Reading the function from a 1024-segment table of chords in LDS (five ordinary
// instructions and one data-dependent 8-byte read per element) was measured too: 2-6 % slower per
// kernel, the reads' bank conflicts cost more than the arithmetic they replace.
__device__ __forceinline__ float gelu_exponent(float v) {
  const float t = fminf(v * v, 81.0f);
  float p = fmaf(0.0010142630f, t, -0.10677572f);  // -log2(e) (a + b t + c t^2)
  p = fmaf(p, t, -2.3011212f);
  return p * v;
}
__device__ __forceinline__ float gelu_erf(float v) {
  const float e = __builtin_amdgcn_exp2f(gelu_exponent(v));  // exp(-(a v + b v^3 + c v^5))
  return v * __builtin_amdgcn_rcpf(1.0f + e);
}

// The LSTM cell's nonlinearities on the hardware's exp2 and reciprocal (about 1 ulp each):
// sigma(z) = 1 / (1 + 2^(-z log2 e)), tanh(z) = 1 - 2 / (1 + 2^(2 z log2 e)); both saturate correctly
// (2^x -> inf gives 1/inf = 0).  The absolute error is a few 1e-7: far inside the bf16 rounding of h
// and the f32 bar of c.  The library forms (a division sequence, a branching tanh) are 150-250
// dependent instructions per cell, which is most of what a one-row step does after its last MFMA.
__device__ __forceinline__ float sigmoidf(float z) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}
__device__ __forceinline__ float tanh_fast(float z) {
  return fmaf(-2.0f, __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(2.8853900817779268f * z)), 1.0f);
}
// One cell update from the four gate pre-activations (i, f, g, o): returns h, writes c.  Every LSTM
// kernel goes through this one function, with the fused multiply-add spelled out, so that they agree
// bit for bit.
__device__ __forceinline__ float lstm_cell(const float (&gate)[4], float c_prev, float& c_new) {
  const float a_i = sigmoidf(gate[0]), a_f = sigmoidf(gate[1]), a_g = tanh_fast(gate[2]), a_o = sigmoidf(gate[3]);
  c_new = fmaf(a_f, c_prev, a_i * a_g);
  return a_o * tanh_fast(c_new);
}
// Makes a value opaque to the compiler at this point: what was loaded before a loop stays in its
// registers instead of being loaded again inside the loop.
__device__ __forceinline__ void keep_in_registers(uint4& v) {
  asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
}

// `bias` is 0 when the epilogue has none, so one fused multiply-add serves every case.
__device__ __forceinline__ float epilogue(float acc, float alpha, float bias, int epi) {
  const float v = fmaf(alpha, acc, bias);
  return epi == NIMBLE_EPI_BIAS_GELU_ERF ? gelu_erf(v) : v;
}
// The same for N values at a time with the choice made outside.  With a choice per value there is a branch per value, and
// left to itself the compiler computes one or two values at a time, each a chain of a dozen dependent instructions; here
// N chains go side by side (the empty statements keep the N results of a step together).  Eight at a time, with their
// choice outside, as graph replays on the eight-wave kernels: the feed-forward pair of 4500 / 8069 tokens 83.1 / 124.0 ->
// 80.2 / 121.6 us (16129 tokens 224 / 223, within the spread of the runs), 800 x 3072 x 768 with GELU 10.05 -> 9.9.
template <bool GELU, int N>
__device__ __forceinline__ void epilogue_of(float (&v)[N]) {
  if (!GELU) return;
  float e[N];
  auto together = [&](float (&x)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]));
  };
#pragma unroll
  for (int i = 0; i < N; ++i) e[i] = gelu_exponent(v[i]);
  together(e);
#pragma unroll
  for (int i = 0; i < N; ++i) e[i] = __builtin_amdgcn_exp2f(e[i]);
  together(e);
#pragma unroll
  for (int i = 0; i < N; ++i) e[i] = 1.0f + e[i];
  together(e);
#pragma unroll
  for (int i = 0; i < N; ++i) e[i] = __builtin_amdgcn_rcpf(e[i]);
  together(e);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] *= e[i];
}

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// Eight bf16 from an address that is only known to be 2-byte aligned (one global_load_dwordx4: the
// hardware takes unaligned vector loads from global memory).
__device__ __forceinline__ uint4 load8_unaligned(const u16* p) {
  uint4 v;
  __builtin_memcpy(&v, p, 16);
  return v;
}
// The first `left` (1..7) of them, the rest zero: the last chunk of a row of `len` elements, past which
// nothing may be read.  The row's last eight elements are loaded instead and shifted down (element by
// element, each load behind a branch, this chunk alone took 3.5 us at K = 1003).
__device__ __forceinline__ uint4 load8_tail(const u16* p, int left, int len) {
  if (len < 8) {
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < 7; ++e)
      if (e < left) w[e >> 1] |= (uint32_t)p[e] << (16 * (e & 1));
    return make_uint4(w[0], w[1], w[2], w[3]);
  }
  const uint4 v = load8_unaligned(p + left - 8);
  const uint64_t lo = ((uint64_t)v.y << 32) | v.x, hi = ((uint64_t)v.w << 32) | v.z;
  const int sh = 16 * (8 - left);  // 16 .. 112 bits
  const uint64_t rlo = sh < 64 ? (lo >> sh) | (hi << (64 - sh)) : hi >> (sh - 64);
  const uint64_t rhi = sh < 64 ? hi >> sh : 0;
  return make_uint4((uint32_t)rlo, (uint32_t)(rlo >> 32), (uint32_t)rhi, (uint32_t)(rhi >> 32));
}

// The first `n` (0 .. 8) elements of a chunk of which the row's last eight have been loaded, the rest zero.
__device__ __forceinline__ uint4 keep_first8(uint4 v, int n) {
  const uint64_t lo = ((uint64_t)v.y << 32) | v.x, hi = ((uint64_t)v.w << 32) | v.z;
  const int sh = 16 * (8 - n);  // 0 .. 128 bits
  const uint64_t rlo = sh == 0 ? lo : sh < 64 ? (lo >> sh) | (hi << (64 - sh)) : sh < 128 ? hi >> (sh - 64) : 0;
  const uint64_t rhi = sh < 64 ? hi >> sh : 0;
  return make_uint4((uint32_t)rlo, (uint32_t)(rlo >> 32), (uint32_t)rhi, (uint32_t)(rhi >> 32));
}
// A chunk whose row starts at an odd element, loaded from the element before, moved down by it (sh = 16; 0: left as it is).
// `next` is the word behind the chunk; where a lane's neighbour holds that chunk (!own) it is taken from there.
__device__ __forceinline__ uint4 shift8(uint4 v, uint32_t next, uint32_t sh, bool own) {
  const uint32_t neighbour = (uint32_t)__builtin_amdgcn_mov_dpp((int)v.x, 0x101, 0xf, 0xf, true);
  next = own ? next : neighbour;
  return make_uint4(__builtin_amdgcn_alignbit(v.y, v.x, sh), __builtin_amdgcn_alignbit(v.z, v.y, sh),
                    __builtin_amdgcn_alignbit(v.w, v.z, sh), __builtin_amdgcn_alignbit(next, v.w, sh));
}

// Two float32 -> two bfloat16 (round to nearest even) in one v_cvt_pk_bf16_f32; lo in bits 0..15.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// Output stores of device scope: they go through the L2 to the memory side at once.  Plain stores leave the output dirty
// in the L2s, which are written back when the kernel ends, in front of whatever waits for it; these are on their way
// while the rest of the kernel runs, and the next kernel still finds them in the memory-side cache (non-temporal stores,
// which do not stay there, cost it as much as they gain).  4096 x 4096 bf16 at K = 64 13.3 -> 10.7 us, at K = 1024 34.0 ->
// 31.9; the feed-forward pair 2113 / 16129 x (1024 -> 4096 -> 1024) 54.1 / 235 -> 52.8 / 230.  What goes to memory this way has to be
// whole 64-byte pieces, better whole lines: pieces do not meet in the L2 any more (attention from registers, 16 bytes of a row
// at a time: 48 heads of 512 10.0 -> 10.9; the streaming kernel's 2-byte ones, 509 x 768 x 768, 5.65 -> 5.95; rows that start
// anywhere, see output_stays and any_output_stays).
// (The two wait states keep the next vector instruction, which the compiler does not know to be near a store, off the
// data registers until the store has read them.)
__device__ __forceinline__ void store_through(void* p, uint4 v) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 w = {v.x, v.y, v.z, v.w};
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(w));
}
template <typename T>
__device__ __forceinline__ void store_through(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_through(void* p, uint2 v) {
  store_through((unsigned long long*)p, ((unsigned long long)v.y << 32) | v.x);
}

// Whether the partial sums of a K-split launch stay in the L2s for the reduction behind it (plain stores).  Beside weights
// that come from memory, which are the bound then, they do better there: layers of 5120 and 8192 columns, several in turn,
// 50 / 100 / 128 rows 217 / 166 / 251 us a pass, 222 / 173 / 264 with the sums through the L2; small layers do not: 400 x 1024 x
// 4096 13.4 / 12.9, 509 x 768 x 3072 12.7 / 11.9.  The line is what the L2s hold together.
__device__ __forceinline__ bool partial_sums_stay(const GemmArgs& g, unsigned slices) {
  return slices > 1 && (long long)g.N * g.K * 2 >= (32ll << 20);
}

// An output store, plain or through the L2 (see output_stays).
template <bool STAYS>
__device__ __forceinline__ void store_out(void* p, uint4 v) {
  if (STAYS)
    *(uint4*)p = v;
  else
    store_through(p, v);
}

// Direct global -> LDS load of 16 bytes per lane: lane i's data lands at LDS byte
// address lds_addr + 16 i (lds_addr is wave-uniform and goes through M0).  It is
// tracked by vmcnt only; the caller waits with s_waitcnt vmcnt before a barrier
// makes the data visible to the other waves.  Written as inline assembly so that
// the compiler does not serialise it against LDS reads of the other ring slots.
__device__ __forceinline__ void dma16(const void* g, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off\n" ::"v"(g), "s"(lds_addr)
               : "memory", "m0");
}
// acc += a . b on the matrix core with the accumulator held in place in the accumulation
// registers.  Written as a volatile statement: the order in the source is the order issued, and
// the register allocator cannot decide to shuffle accumulators between register files.
__device__ __forceinline__ void mfma_acc(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// The compiler does not know that the statement above is a matrix instruction, so it adds none of
// the wait states a matrix result needs before anything else reads its registers (a copy, a
// spill store, the epilogue's arithmetic), and it may place such a reader directly behind the
// statement.  The last MFMA of a tile's last stage therefore carries the wait states itself, in
// the same statement so that nothing can come in between: `last` (wave-uniform) != 0 runs 32 idle
// cycles, by the end of which this result and those of all earlier MFMAs have been written.
__device__ __forceinline__ void mfma_acc_last(f32x4& acc, const bf16x8& a, const bf16x8& b, int last) {
  asm volatile(
      "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\t"
      "s_cmp_eq_u32 %3, 0\n\t"
      "s_cbranch_scc1 .Lnimble_mfma_done_%=\n\t"
      "s_nop 15\n\t"
      "s_nop 15\n"
      ".Lnimble_mfma_done_%=:"
      : "+a"(acc)
      : "v"(a), "v"(b), "s"(__builtin_amdgcn_readfirstlane(last))
      : "scc");
}

// The direct global -> LDS load addressed as a wave-uniform 64-bit base (in SGPRs) plus a 32-bit
// per-lane byte offset, which keeps per-lane 64-bit pointers out of the vector registers.
__device__ __forceinline__ void dma16_so(uint32_t voff, const void* sbase, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n" ::"v"(voff), "s"(sbase),
               "s"(lds_addr)
               : "memory", "m0");
}
// The same for data that nobody reads again: non-temporal, it passes the caches by.
__device__ __forceinline__ void dma16_so_once(uint32_t voff, const void* sbase, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt\n" ::"v"(voff), "s"(sbase),
               "s"(lds_addr)
               : "memory", "m0");
}
// A matrix product with a direct global -> LDS load behind it, at LDS byte lds_base + lds_off (the product is also the
// wait state between writing M0 and the load).
__device__ __forceinline__ void mfma_acc_load(f32x4& acc, const bf16x8& a, const bf16x8& b, uint32_t voff, const void* sbase,
                                              uint32_t lds_base, uint32_t lds_off) {
  asm volatile(
      "s_add_u32 m0, %5, %6\n\t"
      "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\t"
      "global_load_lds_dwordx4 %3, %4"
      : "+a"(acc)
      : "v"(a), "v"(b), "v"(voff), "s"(sbase), "s"(lds_base), "s"(lds_off)
      : "memory", "m0", "scc");
}
// One dword per lane: a wave instruction fills 256 contiguous bytes of LDS.
__device__ __forceinline__ void dma4_so(uint32_t voff, const void* sbase, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1\n" ::"v"(voff), "s"(sbase),
               "s"(lds_addr)
               : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_addr_of(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

typedef short s16x4_t __attribute__((ext_vector_type(4)));
// Transposing LDS read: the 16 lanes of a group each name 8 bytes; they are taken as 4 rows of 16
// 16-bit values (lanes 4 r .. 4 r + 3 hold row r) and lane i of the group receives column i.
__device__ __forceinline__ uint2 lds_read_tr16(uint32_t lds_addr) {
  typedef __attribute__((address_space(3))) s16x4_t* ptr;
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((ptr)(uintptr_t)lds_addr));
}

// ---------------------------------------------------------------------------
// Workgroup id -> macro tile.  Workgroups are handed to the 8 XCDs round robin;
// give each XCD a contiguous run of tile ids so that the tiles sharing rows of
// A and B meet in that XCD's L2, and walk the tiles in groups of `group_m`
// tile rows so that the set in flight is a compact block.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void tile_of_block(int bid, int nblocks, int tiles_m, int tiles_n,
                                              int group_m, int& tm, int& tn) {
  const int q = nblocks >> 3, rem = nblocks & 7;
  const int xcd = bid & 7, local = bid >> 3;
  const int pid = xcd * q + (xcd < rem ? xcd : rem) + local;
  const int in_group = group_m * tiles_n;
  const int gid = pid / in_group;
  const int first_m = gid * group_m;
  const int gsize = (tiles_m - first_m) < group_m ? (tiles_m - first_m) : group_m;
  const int rest = pid - gid * in_group;
  tm = first_m + rest % gsize;
  tn = rest / gsize;
}

}  // namespace nimble
#endif
