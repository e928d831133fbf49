// Row softmax, transpose.
#ifndef NIMBLE_MISC_KERNELS_H_
#define NIMBLE_MISC_KERNELS_H_
#include "device_common.h"

namespace nimble {

// ---------------------------------------------------------------------------
// Row softmax, f32 in, bf16 out; one wave per row, four rows per workgroup.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// b [T, K, N] -> bt [T, N, K] (bf16), 32 x 32 tiles through LDS: the NN batch_matmul is run as
// the NT one on the transposed operand, which lives in the caller's workspace.
__global__ void __launch_bounds__(256)
    transpose_kn_kernel(const u16* __restrict__ b, u16* __restrict__ bt, int K, int N) {
  __shared__ u16 tile[32][33];
  const long long plane = (long long)K * N;
  const u16* src = b + blockIdx.z * plane;
  u16* dst = bt + blockIdx.z * plane;
  const int k0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int k = k0 + ty + 8 * r, n = n0 + tx;
    if (k < K && n < N) tile[ty + 8 * r][tx] = src[(long long)k * N + n];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int n = n0 + ty + 8 * r, k = k0 + tx;
    if (n < N && k < K) dst[(long long)n * K + k] = tile[tx][ty + 8 * r];
  }
}

__global__ void __launch_bounds__(256)
    softmax_rows_kernel(const float* __restrict__ s, u16* __restrict__ p, long long rows, int cols) {
  const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int lane = threadIdx.x & 63;
  const float* sr = s + row * cols;
  u16* pr = p + row * cols;
  float mx = -INFINITY;
  for (int j = lane; j < cols; j += 64) mx = fmaxf(mx, sr[j]);
  mx = wave_max(mx);
  float sum = 0.f;
  for (int j = lane; j < cols; j += 64) sum += expf(sr[j] - mx);
  sum = wave_sum(sum);
  const float inv = 1.0f / sum;
  for (int j = lane; j < cols; j += 64) pr[j] = f2bf(expf(sr[j] - mx) * inv);
}

}  // namespace nimble
#endif
