// Deterministic FP64 block reduction of kReduceVals values per thread. Slot 6 is reduced
// with max, every other slot with +. The order of every addition is fixed by the launch
// shape, so repeated runs give identical bits.
#pragma once
#include <hip/hip_runtime.h>

#include "internal.h"
#include "launch.h"

namespace lbm {

__device__ __forceinline__ double combine(int k, double a, double b) { return k == 6 ? fmax(a, b) : a + b; }

// Block of 256 threads (4 waves of 64). Thread 0 writes partials[blockIdx.x * 8 + k].
__device__ __forceinline__ void block_reduce_store(double (&v)[kReduceVals], double* partials) {
  __shared__ double sh[4][kReduceVals];
#pragma unroll
  for (int k = 0; k < kReduceVals; ++k) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v[k] = combine(k, v[k], __shfl_xor(v[k], off, 64));
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < kReduceVals; ++k) sh[wave][k] = v[k];
  }
  __syncthreads();
  if (threadIdx.x < kReduceVals) {
    const int k = threadIdx.x;
    double a = sh[0][k];
    for (int w = 1; w < 4; ++w) a = combine(k, a, sh[w][k]);
    partials[blockIdx.x * kReduceVals + k] = a;
  }
}

// n / d for n < 2^30 by a high multiply, an add and a shift: with l = ceil(log2 d) and
// m = floor(2^32 (2^l - d) / d) + 1, floor(n / d) = (hi(m n) + n) >> l for every 32-bit n
// (Granlund and Montgomery, division by invariant integers); the sum stays below 2^31 here.
struct FastDiv {
  unsigned m, l;
};
inline FastDiv fast_div(unsigned d) {
  unsigned l = 0;
  while ((1ull << l) < d) ++l;
  return FastDiv{static_cast<unsigned>((((1ull << l) - d) << 32) / d + 1), l};
}
__device__ __forceinline__ unsigned quotient(unsigned n, const FastDiv& f) { return (__umulhi(n, f.m) + n) >> f.l; }

// The reductions' threads walk over the nodes in their order in memory, a grid apart, so that
// every lane has a node whatever the row length (whole rows per block left 3 of 4 lanes idle at
// 64^3 and a ragged last round of blocks elsewhere).
struct NodeWalk {
  FastDiv nx, ny;
};
inline NodeWalk node_walk(const Geo& G) { return NodeWalk{fast_div(G.nx), fast_div(G.ny)}; }

struct Coord {
  int x, y, z;
};
__device__ __forceinline__ Coord coord_of(const Geo& G, const NodeWalk& W, unsigned n) {
  const unsigned r = quotient(n, W.nx);
  const unsigned z = quotient(r, W.ny);
  return Coord{static_cast<int>(n - r * G.nx), static_cast<int>(r - z * G.ny), static_cast<int>(z)};
}

// Blocks of a reduction: one node per thread up to 1280 blocks (5 per CU; the D3Q19 kernel's
// registers allow 7), then as many as leave a thread 16 nodes, up to kReduceBlocks. Both lines are
// measured: the fold at a block's end costs as much as a few nodes, so that at 128^3 1280 blocks
// take 35 us and 4096 take 41, while at 256^3 4096 blocks (16 nodes per thread) balance better than
// 1280 (51 per thread; 221 against 224 us).
constexpr unsigned kReduceFill = 1280;
inline unsigned reduce_blocks(const Geo& G) {
  const unsigned all = (G.N + 255) / 256;
  unsigned nb = G.N / (256 * 16);
  if (nb < kReduceFill) nb = kReduceFill;
  if (nb > static_cast<unsigned>(kReduceBlocks)) nb = kReduceBlocks;
  return nb < all ? nb : all;
}

}  // namespace lbm
