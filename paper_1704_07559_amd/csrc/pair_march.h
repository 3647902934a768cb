// Two steps per launch for the 3D lattices (FP32 storage, periodic or with walls, no body force, constant
// viscosity or Smagorinsky, lagged or implicit, with the Yu strain): the marching kernel, its launch rule
// and its launch.
// A lattice gives its node update as a type (Lat, kLagged, run).
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.h"
#include "launch.h"
#include "static_for.h"

namespace lbm {

constexpr unsigned kXcds = 8;
constexpr int kPairNodes = 1024;  // most level-1 nodes, a thread each, of a tile

__device__ __forceinline__ float fma3(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// A block owns cols x rows (WX x HY) columns of nodes and marches through `planes` planes of z. Per plane, one
// thread per node of the (WX + 2) x (HY + 2) level-1 tile takes the first step of that plane into
// LDS; the second step of the plane below needs three level-1 planes, of which LDS holds the newest:
// each thread has already gathered what its node pulls from the two before (the directions with
// cz > 0 wait two planes in hz and hzz, those with cz = 0 one plane in hn; each array uses only
// those elements). The next plane's loads are issued before the second step, and LDS holds two planes
// in turn, so that one barrier per plane is enough. Blocks that follow one another on an XCD are
// neighbours, whose tile edges meet in its L2.
// What it saves is HBM traffic: a node is read once (and re-read at tile edges, mostly out of the L2) and
// written once for two steps (D3Q19 160 bytes against 320). What is left is that traffic (166 bytes as
// counted, 4.7 TB/s) and the vector unit side by side (0.48 of its issue rate).
// us a step, against single steps, Smagorinsky: D3Q19 256^3 297 (418), 384x384x128 316 (490), 200^3 153 (217),
// 128^3 42 (54), 96^3 17.0 (24.8), D3Q15 256^3 252 (325), 200^3 125 (180), 96^3 14.7 (21.0); constant viscosity
// at 256^3 270 (418) and 231 (323), implicit 299 (419) and 262 (320), Smagorinsky between walls 335 (446; that
// D3Q19 instance fills 128 VGPRs and spills 44 bytes) and 246 (337). One block runs on a CU: its two LDS planes are
// sized for 1024 nodes whatever the tile. At 256^3 a block has 704 threads (11 of the 16 waves that 126 VGPRs
// allow) and uses 103 of its 160 KB. Measured on the way, D3Q19 256^3: blocks dealt out over the XCDs in
// turn 325, two barriers and one plane of LDS 310, without the early loads 304.
template <class Update, bool WALLS, bool STREAM>
__global__ __launch_bounds__(kPairNodes, 4) void pair_kernel(Geo G, PairPlan P, ModelF M, ViscF V,
                                                          const float* __restrict__ src, float* __restrict__ dst,
                                                          const float* __restrict__ snu_in,
                                                          float* __restrict__ snu_out) {
  using Lat = typename Update::Lat;
  constexpr int Q = Lat::Q;
  constexpr bool LAGGED = Update::kLagged;
  const int WX = P.cols, HY = P.rows, W1 = WX + 2, N1 = W1 * (HY + 2);
  __shared__ float planes[2][LAGGED ? Q + 1 : Q][kPairNodes];
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

template <class Update>
hipError_t launch_march(const PairPlan& P, hipStream_t st, const Geo& G, const ModelF& M, const ViscF& V,
                        const void* src, void* dst, const float* snu_in, float* snu_out) {
  if (Update::kLagged != (snu_in != nullptr) || (snu_in != nullptr) != (snu_out != nullptr) ||
      (snu_in && snu_in == snu_out))
    return hipErrorInvalidValue;
  if (P.tiles <= 0 || (P.cols + 2) * (P.rows + 2) > P.threads || P.threads > kPairNodes) return hipErrorInvalidValue;
  const bool stream = pair_stream(G, Update::Lat::Q);
  const auto k = G.walls ? (stream ? pair_kernel<Update, true, true> : pair_kernel<Update, true, false>)
                         : (stream ? pair_kernel<Update, false, true> : pair_kernel<Update, false, false>);
  hipLaunchKernelGGL(k, dim3((P.tiles + kXcds - 1) / kXcds * kXcds), dim3(P.threads), 0, st, G, P, M, V,
                     static_cast<const float*>(src), static_cast<float*>(dst), snu_in, snu_out);
  return hipGetLastError();
}

// What the kernel computes.
inline bool march_takes(int storage, const ViscF& V, const ForceF& Fo) {
  return storage == 0 && !Fo.mode && V.kind != 2 && !(V.kind != 0 && V.drive_chai);
}

// The plan of tiles of cols x rows columns and `planes` planes, empty where the kernel does not take it.
inline PairPlan march_tiles(int storage, const Geo& G, const ViscF& V, const ForceF& Fo, int cols, int rows,
                            int planes) {
  if (!march_takes(storage, V, Fo) || cols < 1 || rows < 1 || planes < 1) return PairPlan{};
  if (cols > kPairNodes || rows > kPairNodes || (cols + 2) * (rows + 2) > kPairNodes) return PairPlan{};
  const int tx = (G.nx - 1) / cols + 1, ty = (G.ny - 1) / rows + 1, tz = (G.nz - 1) / planes + 1;
  const long long tiles = static_cast<long long>(tx) * ty * tz;
  if (tiles > (1 << 20)) return PairPlan{};  // (far more than a plan takes)
  return PairPlan{cols, rows, planes, tx, ty, static_cast<int>(tiles), ((cols + 2) * (rows + 2) + 63) / 64 * 64};
}

// The tile and the planes per block that take the least: rounds of blocks over the CUs (one block each,
// for its LDS), times the planes one marches through (two more than it stores), times ns a plane.
// A plane takes 217 ns per wave and 80 per 128-byte line of its tile's rows (64 x 13 6.9 us, 64 x 9 5.0,
// 32 x 28 8.4); rows are cut into equal tiles, so that boxes of any width fill theirs (us a step against
// tiles of 64 x 13 and 64 x 9 only, Smagorinsky: 200^3 153 and 195, 220^3 203 and 277, 171x133x95 51 and 54,
// 96^3 17.0 and 18.9, 256^3 297 and 301). Streamed stores need tiles that meet between lines (256^3 in
// three tiles of 86 columns 443). A single step takes about 26 ps a node out of HBM, in the last-level cache
// 28 to 38 where runs are aligned and up to 50 where not, a pair there 0.6 to 0.8 of its estimate: pairs are
// taken where the estimate is at most 26, 37 or 60 ps a node and step (us, single and pairs, estimate:
// 512x24x24 9.0 and 8.7, 36 ps; 66^3 11.1 and 8.5, 38; 17x17x1000 14.8 and 9.7, 57; 150^3 90 and 83, 20).
// Up to 2^18 nodes single steps run out of the L2s (64^3 7.1, two 64 x 9 tiles' planes 7.6).
inline PairPlan plan_pairs(int q, int storage, const Geo& G, const ViscF& V, const ForceF& Fo) {
  PairPlan best{};
  if (!march_takes(storage, V, Fo) || G.N <= (1u << 18)) return best;
  constexpr long long kCus = 256;
  long long least = 0;
  const bool whole = runs_aligned(G, sizeof(float), 64) && pair_stream(G, q);  // tiles meet between lines
  const int tx0 = (G.nx + 125) / 126;
  for (int tx = tx0; tx < tx0 + 6; ++tx) {
    int cols = (G.nx + tx - 1) / tx;
    if (whole && tx > 1) cols = (cols + 15) / 16 * 16;
    if (cols > 126) continue;
    const int most = kPairNodes / (cols + 2) - 2;
    for (int rows = most; rows >= 4 && rows > most / 2; --rows) {
      const long long ty = (G.ny + rows - 1) / rows, columns = ((G.nx + cols - 1) / cols) * ty;
      const int waves = ((cols + 2) * (rows + 2) + 63) / 64;
      const long long plane = 217 * waves + (rows + 2) * (78 + (cols + 2) * 5 / 2);
      const long long first = (columns + kCus - 1) / kCus;
      for (long long rounds = first; rounds < first + 8; ++rounds) {
        const long long chunks = std::min<long long>(kCus * rounds / columns, G.nz);
        const int planes = static_cast<int>((G.nz + chunks - 1) / chunks);
        const long long tiles = columns * ((G.nz + planes - 1) / planes);
        const long long cost = (tiles + kCus - 1) / kCus * (planes + 2) * plane;
        if (best.planes && cost >= least) continue;
        least = cost;
        best = PairPlan{cols, rows, planes, static_cast<int>((G.nx + cols - 1) / cols), static_cast<int>(ty),
                        static_cast<int>(tiles), waves * 64};
      }
    }
  }
  // least / N is 2 steps' ns a node
  const long long ps = !pair_fits(G, q) ? 26 : ragged_rows(G, sizeof(float)) ? 60 : 37;
  if (500 * least > ps * G.N) return PairPlan{};
  return best;
}

}  // namespace lbm
