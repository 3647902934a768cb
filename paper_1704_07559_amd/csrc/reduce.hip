// Second pass of the deterministic FP64 reductions: slot k of the result is the fold of
// slot k over the per-block partials, in an order fixed by their number: thread t folds slot
// t mod 8 of the partials t / 8, t / 8 + 128, ..., then the threads of one slot are folded by a
// fixed tree. A chain of latencies bounds it, so one block of 1024 threads reads eight values
// at a time, coalesced over the slots (4096 partials: 5 us; one thread per partial with 256
// threads, each reading the eight slots in turn, 10 us).
#include <hip/hip_runtime.h>

#include "internal.h"
#include "launch.h"
#include "reduce.h"

namespace lbm {

constexpr int kFinalThreads = 1024;

// rho0 > 0: slot 6 holds the largest |j|^2 and becomes max |u| = sqrt(max |j|^2) / rho0 (one
// square root and one division instead of one per node; both are correctly rounded and
// monotone, so this is the maximum of the per-node values bit for bit).
__global__ __launch_bounds__(kFinalThreads) void reduce_final_kernel(const double* __restrict__ partials, int nblocks,
                                                                     double* __restrict__ out, double rho0) {
  const int k = threadIdx.x % kReduceVals, n = nblocks * kReduceVals;
  constexpr int kAhead = 8;
  double a = 0.0;  // max slot: |j|^2 >= 0
  for (int i = threadIdx.x; i < n; i += kAhead * kFinalThreads) {
    double p[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int j = i + u * kFinalThreads;
      p[u] = j < n ? partials[j] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) a = combine(k, a, p[u]);
  }
#pragma unroll
  for (int off = 32; off >= kReduceVals; off >>= 1) a = combine(k, a, __shfl_xor(a, off, 64));
  __shared__ double sh[kFinalThreads / 64][kReduceVals];
  if ((threadIdx.x & 63) < kReduceVals) sh[threadIdx.x >> 6][k] = a;
  __syncthreads();
  if (threadIdx.x < kReduceVals) {
    a = sh[0][k];
    for (int w = 1; w < kFinalThreads / 64; ++w) a = combine(k, a, sh[w][k]);
    out[k] = (k == 6 && rho0 > 0.0) ? sqrt(a) / rho0 : a;
  }
}

hipError_t launch_reduce_final(const double* partials, int nblocks, double* out, hipStream_t st, double rho0) {
  hipLaunchKernelGGL(reduce_final_kernel, dim3(1), dim3(kFinalThreads), 0, st, partials, nblocks, out, rho0);
  return hipGetLastError();
}

}  // namespace lbm
