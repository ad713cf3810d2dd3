// Fold of a dense layer's constants into the start value of its accumulator.
#include "conv_params.h"

namespace f8 {

namespace {

constexpr int NT = 256;          // threads per workgroup (4 waves)

// acc0[n] = bias[n] + rnd + (unsigned x ? 128 * sum_k w[n][k] : 0); one wave per channel.
__global__ __launch_bounds__(NT) void fold_acc0_kernel(const int8_t *w, const int32_t *bias, int32_t *acc0,
                                                       int N, int n_pad, int K, int x_unsigned, int rnd) {
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * (NT / 64) + (threadIdx.x >> 6);
  if (n >= n_pad) return;
  int sum = 0;
  if (n < N) {
    if (x_unsigned) {
      const int8_t *row = w + (size_t)n * K;
      for (int k = lane; k < K; k += 64) sum += (int)row[k];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
      sum *= 128;
    }
    sum += rnd + (bias ? bias[n] : 0);
  }
  if (lane == 0) acc0[n] = sum;
}

}  // namespace

int launch_fold_acc0(const int8_t *w, const int32_t *bias, int32_t *acc0, int N, int n_pad, int K,
                     int x_unsigned, int rnd, hipStream_t stream) {
  if (n_pad <= 0) return 0;
  dim3 grid((unsigned)((n_pad + NT / 64 - 1) / (NT / 64))), block(NT);
  hipLaunchKernelGGL(fold_acc0_kernel, grid, block, 0, stream, w, bias, acc0, N, n_pad, K, x_unsigned, rnd);
  return (int)hipGetLastError();
}

}  // namespace f8
