// Two steps per launch for the 3D lattices (FP32 storage, periodic or with walls, no body force, constant
// viscosity or Smagorinsky, lagged or implicit, with the Yu strain): the marching kernel, its launch rule and its launch.
// A lattice gives its node update as a type (Lat, kLagged, run).
#pragma once
#include <hip/hip_runtime.h>

#include "internal.h"
#include "launch.h"
#include "static_for.h"

namespace lbm {

constexpr unsigned kXcds = 8;

__device__ __forceinline__ float fma3(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// A block owns WX x HY columns of nodes and marches through `planes` planes of z. Per plane, one
// thread per node of the (WX + 2) x (HY + 2) level-1 tile takes the first step of that plane into
// LDS; the second step of the plane below needs three level-1 planes, of which LDS holds the newest:
// each thread has already gathered what its node pulls from the two before (the directions with
// cz > 0 wait two planes in hz and hzz, those with cz = 0 one plane in hn; each array uses only
// those elements). The next plane's loads are issued before the second step, and LDS holds two planes
// in turn, so that one barrier per plane is enough. Blocks that follow one another on an XCD are
// neighbours, whose tile edges meet in its L2.
// What it saves is HBM traffic: a node is read once (and re-read at tile edges, mostly out of the L2) and
// written once for two steps (D3Q19 160 bytes against 320). What is left is that traffic (178 bytes as
// counted, 5.0 TB/s) and the vector unit side by side (0.45 of its issue rate).
// us a step, against single steps, Smagorinsky: D3Q19 256^3 300 (418), 384^3 993 (1488), 128^3 44.3 (54.1),
// 96^3 18.6 (24.8), D3Q15 256^3 249 (325), 200^3 157 (180), 96^3 16.0 (21.0); constant viscosity at 256^3
// 278 (418) and 229 (323), implicit 296 (419) and 254 (320), Smagorinsky between walls 335 (446; its 64 x 13
// instance spills 28 bytes) and 246 (337). Measured on the way, D3Q19 256^3: blocks dealt out over the XCDs in turn 325,
// two barriers and one plane of LDS 310, without the early loads 304.
template <class Update, int B, int WX, int HY, bool WALLS, bool STREAM>
__global__ __launch_bounds__(B, B / 256) void pair_kernel(Geo G, PairPlan P, ModelF M, ViscF V,
                                                          const float* __restrict__ src, float* __restrict__ dst,
                                                          const float* __restrict__ snu_in,
                                                          float* __restrict__ snu_out) {
  using Lat = typename Update::Lat;
  constexpr int Q = Lat::Q;
  constexpr bool LAGGED = Update::kLagged;
  constexpr int W1 = WX + 2, H1 = HY + 2, N1 = W1 * H1;
  static_assert(N1 <= B && WX * HY <= B, "a thread per node of either level");
  __shared__ float planes[2][LAGGED ? Q + 1 : Q][N1];
  const int tile = (blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
  if (tile >= P.tiles) return;
  const int t = threadIdx.x;
  const int x0 = tile % P.tx * WX, y0 = tile / P.tx % P.ty * HY, z0 = tile / (P.tx * P.ty) * P.planes;
  const int nz2 = min(P.planes, G.nz - z0);
  // level 1: this thread's node, wrapped
  const int xa = x0 - 1 + t % W1, ya = y0 - 1 + t / W1;
  const bool on1 = t < N1 && xa <= G.nx && (WALLS ? ya >= 0 && ya < G.ny : ya <= G.ny);
  const int x1 = xa < 0 ? xa + G.nx : (xa >= G.nx ? xa - G.nx : xa);
  const int y1 = ya < 0 ? ya + G.ny : (ya >= G.ny ? ya - G.ny : ya);
  // level 2
  const int x2 = x0 + t % WX, y2 = y0 + t / WX;
  const bool on2 = t < WX * HY && x2 < G.nx && y2 < G.ny;
  const int q = (t / WX + 1) * W1 + t % WX + 1;

  float g[Q], rate = 0.0f;
  const auto load = [&](int k) {
    int z = z0 - 1 + k;
    z = z < 0 ? z + G.nz : (z >= G.nz ? z - G.nz : z);
    if (on1) {
      pull_rows<Lat, float, WALLS, true, true>(src, G, rows_of<Q, float>(G, x1, y1, z), y1, g);
      if constexpr (LAGGED) rate = snu_in[node_index(G, x1, y1, z)];
    }
  };
  float hn[Q], hz[Q], hzz[Q];
  float back[2] = {0.0f, 0.0f};
  float snu_l = 0.0f;
  load(0);
  for (int k = 0; k < nz2 + 2; ++k) {
    auto& sh = planes[k & 1];
    if (on1) {
      const float s1 = Update::run(g, M, V, rate);
      static_for<Q>([&](auto ii) {
        constexpr int i = ii;
        sh[i][t] = g[i];
      });
      if constexpr (LAGGED) sh[Q][t] = s1;
    }
    __syncthreads();
    float full[Q];
    const float snu_f = snu_l;
    if (on2) {
      static_for<Q>([&](auto ii) {
        constexpr int i = ii;
        constexpr int cx = Lat::cx(i), cy = Lat::cy(i), cz = Lat::cz(i);
        const float v = sh[i][q - cx - cy * W1];
        // a population that crosses a wall is the opposite one of the node itself, from the middle plane
        const bool bounce = WALLS && crosses_wall<cy>(G, y2);
        if constexpr (cz < 0) {
          full[i] = v;
          if constexpr (WALLS && cy != 0) {
            constexpr int w = cx > 0 ? 1 : 0;  // (a node has one wall: boxes of one row are not filled well enough)
            if (bounce) {
              full[i] = back[w];
              back[w] = sh[Lat::opp(i)][q];
            }
          }
        } else if constexpr (cz == 0) {
          full[i] = hn[i];
          hn[i] = v;
          if constexpr (WALLS && cy != 0) {
            if (bounce) hn[i] = sh[Lat::opp(i)][q];
          }
        } else {
          full[i] = hzz[i];
          hzz[i] = hz[i];
          if constexpr (WALLS && cy != 0) {
            if (bounce) hzz[i] = sh[Lat::opp(i)][q];
          }
          hz[i] = v;
        }
      });
      if constexpr (LAGGED) snu_l = sh[Q][q];
    }
    if (k < nz2 + 1) load(k + 1);
    if (on2 && k >= 2) {
      const int z2 = z0 + k - 2;
      const float s2 = Update::run(full, M, V, snu_f);
      if constexpr (LAGGED) snu_out[node_index(G, x2, y2, z2)] = s2;
      const Rows<Q, float> r = rows_of<Q, float>(G, x2, y2, z2);
      char* to = reinterpret_cast<char*>(dst) + r.zb[1] + r.self;
      const size_t run = static_cast<size_t>(G.nx) * sizeof(float);
      static_for<Q>([&](auto ii) {
        constexpr int i = ii;
        plane_store<STREAM>(reinterpret_cast<float*>(to + i * run), full[i]);
      });
    }
  }
}

// Stores go through the caches where both population buffers fit the 256 MB last-level cache, which
// then holds the state from one launch to the next, and where tiles meet inside lines in boxes far
// beyond it (us a step, constant viscosity, streamed and cached: 96^3 21.3 and 16.2, 120^3 37.9 and 27.6,
// but 128^3, 159 MB a buffer, 40.9 and 44.3; rows of 16 n + r floats: 150^3, 245 MB a buffer, 85 and 87,
// 180^3 130 and 117, 250^3 319 and 286).
inline bool pair_fits(const Geo& G, int q) { return !packed_stream(G, q, sizeof(float)); }
inline bool pair_stream(const Geo& G, int q) {
  if (pair_fits(G, q)) return false;
  return runs_aligned(G, sizeof(float), 64) || size_t(G.N) * sizeof(float) * q <= (size_t(1) << 28);
}

// One block per CU (LDS): 64 x 13 columns in 1024 threads (990 level-1 nodes), or 64 x 9 in 768 (726).
constexpr int kPairCols = 64, kPairRowsBig = 13, kPairRowsSmall = 9;

template <class Update, int B, int HY>
hipError_t launch_tile(const PairPlan& P, hipStream_t st, const Geo& G, const ModelF& M, const ViscF& V, const float* src,
                       float* dst, const float* snu_in, float* snu_out) {
  const bool stream = pair_stream(G, Update::Lat::Q);
  const auto k = G.walls ? (stream ? pair_kernel<Update, B, kPairCols, HY, true, true>
                                   : pair_kernel<Update, B, kPairCols, HY, true, false>)
                         : (stream ? pair_kernel<Update, B, kPairCols, HY, false, true>
                                   : pair_kernel<Update, B, kPairCols, HY, false, false>);
  hipLaunchKernelGGL(k, dim3((P.tiles + kXcds - 1) / kXcds * kXcds), dim3(B), 0, st, G, P, M, V, src, dst, snu_in, snu_out);
  return hipGetLastError();
}

template <class Update>
hipError_t launch_march(const PairPlan& P, hipStream_t st, const Geo& G, const ModelF& M, const ViscF& V,
                        const void* src, void* dst, const float* snu_in, float* snu_out) {
  if (Update::kLagged != (snu_in != nullptr) || (snu_in != nullptr) != (snu_out != nullptr) ||
      (snu_in && snu_in == snu_out))
    return hipErrorInvalidValue;
  const float* s = static_cast<const float*>(src);
  float* d = static_cast<float*>(dst);
  if (P.rows == kPairRowsBig) return launch_tile<Update, 1024, kPairRowsBig>(P, st, G, M, V, s, d, snu_in, snu_out);
  if (P.rows == kPairRowsSmall) return launch_tile<Update, 768, kPairRowsSmall>(P, st, G, M, V, s, d, snu_in, snu_out);
  return hipErrorInvalidValue;
}

// The tile and the planes per block that cost the least: rounds of blocks over the CUs, times the planes
// that one marches through (two more than it stores), times the nodes of its tile (the small one costs 5 %
// more a node: 128^3 45.2 us a step against 44.3). `fill` is the box's share of that product. A node of it
// takes 32 ps of the chip for two steps and a node of a single step 26, so pairs need a fill of 0.6
// (us a step, single and pairs, Smagorinsky: 171x133x95, fill 0.66, 58.8 and 54.2, 150^3, 0.68, 90 and 90,
// 144^3, 0.62, 84 and 75, but 130^3, 0.54, 60.7 and 65.3). In the last-level cache a plane of a tile takes
// half of that, and 0.38 is enough (80^3, 0.41, 17.7 and 13.4, D3Q15 15.0 and 11.9; 72^3, 0.34, 12.2 and
// 11.6, D3Q15 9.9 and 10.4; 66^3, 0.27, 11.1 and 11.2). Up to 64^3 single steps run out of the L2s (7.1 and
// 7.6 us). The implicit rate's solve hides under the memory time of single steps, not of pairs: 0.7 and
// 0.45 (D3Q15 between walls 150^3, 0.68, 71.4 and 74.3, 80^3, 0.41, 14.3 and 14.6; 200^3, 0.72, 167 and 153).
inline PairPlan plan_pairs(int q, int storage, const Geo& G, const ViscF& V, const ForceF& Fo) {
  PairPlan best{};
  if (storage != 0 || Fo.mode || Fo.strain_corr) return best;
  if (V.kind == 2 || (V.kind != 0 && V.drive_chai)) return best;
  constexpr long long kCus = 256;
  long long least = 0;
  for (const int rows : {kPairRowsBig, kPairRowsSmall}) {
    const long long tx = (G.nx + kPairCols - 1) / kPairCols, ty = (G.ny + rows - 1) / rows;
    for (int chunks = 1; chunks <= 64 && chunks <= G.nz; ++chunks) {
      const int planes = (G.nz + chunks - 1) / chunks;
      const long long tiles = tx * ty * ((G.nz + planes - 1) / planes);
      long long cost = (tiles + kCus - 1) / kCus * kCus * (planes + 2) * kPairCols * rows;
      if (rows == kPairRowsSmall) cost += cost / 20;
      if (best.planes && cost >= least) continue;
      least = cost;
      best = PairPlan{rows, planes, static_cast<int>(tx), static_cast<int>(ty), static_cast<int>(tiles)};
    }
  }
  const long long fill = V.kind == 3 ? (pair_fits(G, q) ? 45 : 70) : (pair_fits(G, q) ? 38 : 60);
  const bool use = 100ll * G.N >= fill * least && G.N > (1u << 18);
  if (!use) return PairPlan{};
  return best;
}

}  // namespace lbm
