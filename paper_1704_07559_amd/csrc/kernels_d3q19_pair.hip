// D3Q19, two steps per launch: FP32 storage, periodic boxes, no body force, constant viscosity or
// the lagged Smagorinsky model with the Yu strain. Reference: the pipeline of two ordinary steps.
#include <hip/hip_runtime.h>

#include "d3q19.h"
#include "d3q19_node.h"
#include "internal.h"
#include "launch.h"

namespace lbm {
namespace d3q19 {

namespace {

constexpr unsigned kXcds = 8;

__device__ __forceinline__ float fma3(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// The node update of kernels_d3q19_step.hip (moments, Yu strain, lagged viscosity, relaxation,
// back-transform) for the cases above, with every fused product written out. The step kernels leave
// to the compiler which product of a sum is fused; what it picks there depends on the code around
// the sum, so the same source in this kernel rounds differently. The picks below are theirs:
// all pull modes share them but the LDS exchange (XCHG), whose instances differ in two sums (o[3],
// o[4]). Two steps of this kernel therefore equal two single steps bit for bit.
template <int KIND, bool XCHG>
__device__ __forceinline__ float pair_update(float (&g)[Q], const ModelF& M, const ViscF& V, float snu_prev) {
#pragma clang fp contract(off)
  const Pairs P = make_pairs(g);
  const float (&s)[NP] = P.s;
  const float (&d)[NP] = P.d;
  const float A = s[3] + s[4], B = s[5] + s[6], C = s[7] + s[8], AB = A + B, dg = AB + C;
  const float s12 = s[1] + s[2], ax = s[0] + s12;
  const float drho = (P.g0 + ax) + dg;
  const float m1 = fma3(-30.0f, P.g0, fma3(8.0f, dg, -11.0f * ax));
  const float m2 = fma3(12.0f, P.g0, fma3(-4.0f, ax, dg));
  const float T1 = fma3(-2.0f, C, AB);
  const float D12 = s[1] - s[2], AmB = A - B;
  const float X1 = d[3] - d[4], X2 = d[5] - d[6], Y1 = d[3] + d[4], Y2 = d[7] - d[8], Z1 = d[5] + d[6],
              Z2 = d[7] + d[8];
  const float Xs = X1 + X2, Ys = Y1 + Y2, Zs = Z1 + Z2;
  const float jx = d[0] + Xs, jy = d[1] + Ys, jz = d[2] + Zs;
  const float m16 = X1 - X2, m17 = Y2 - Y1, m18 = Z1 - Z2;

  // non-equilibrium moments (noneq_moments)
  const float ir = M.inv_rho0;
  const float jx2 = jx * jx, jy2 = jy * jy, jz2 = jz * jz;
  const float jj = fma3(jz, jz, fma3(jy, jy, jx2));
  const float pxx = fma3(-jz, jz, fma3(2.0f, jx2, -jy2));
  const float pww = fma3(jy, jy, -jz2);
  const float pxx_r = pxx * ir, pww_r = pww * ir;
  const float n1 = m1 - fma3(19.0f * jj, ir, -11.0f * drho);
  const float n2 = m2 - fma3(M.om_eps, drho, M.om_epsj * jj * ir);
  const float n4 = fma3(2.0f / 3.0f, jx, fma3(-4.0f, d[0], Xs));
  const float n6 = fma3(2.0f / 3.0f, jy, fma3(-4.0f, d[1], Ys));
  const float n8 = fma3(2.0f / 3.0f, jz, fma3(-4.0f, d[2], Zs));
  const float n9 = fma3(-pxx, ir, fma3(2.0f, s[0], T1) - s12);
  const float n10 = fma3(-M.om_xx, pxx_r, fma3(-4.0f, s[0], fma3(2.0f, s12, T1)));
  const float n11 = fma3(-pww, ir, D12 + AmB);
  const float n12 = fma3(-M.om_xx, pww_r, fma3(-2.0f, D12, AmB));
  const float n13 = fma3(-(jx * jy), ir, s[3] - s[4]);
  const float n14 = fma3(-(jy * jz), ir, s[7] - s[8]);
  const float n15 = fma3(-(jx * jz), ir, s[5] - s[6]);

  float snu = M.s[9];
  if constexpr (KIND == 1) {
    // strain_yu, strain_sq and viscous_rate
    const float a = M.s[1] * n1, b = snu_prev * n9, c = snu_prev * n11;
    const float Sxx = -fma3(19.0f, b, a) * (ir * (1.0f / 38.0f));
    const float Syy = -fma3(-19.0f, fma3(-3.0f, c, b), 2.0f * a) * (ir * (1.0f / 76.0f));
    const float Szz = -fma3(-19.0f, fma3(3.0f, c, b), 2.0f * a) * (ir * (1.0f / 76.0f));
    const float Sxy = -1.5f * snu_prev * n13 * ir;
    const float Syz = -1.5f * snu_prev * n14 * ir;
    const float Sxz = -1.5f * snu_prev * n15 * ir;
    const float diag = fma3(Szz, Szz, fma3(Syy, Syy, Sxx * Sxx));
    const float off = fma3(Sxz, Sxz, fma3(Syz, Syz, Sxy * Sxy));
    const float gamma = fast_sqrt(2.0f * fma3(2.0f, off, diag));
    snu = fast_rcp(fma3(3.0f, fma3(V.csmag2, gamma, V.nu0), 0.5f));
  }

  // relaxation, as w_k = dm_k / D_k
  const float w1 = M.sd[1] * n1, w2 = M.sd[2] * n2;
  const float w4 = M.sd[4] * n4, w6 = M.sd[6] * n6, w8 = M.sd[8] * n8;
  const float w9 = -snu * (1.0f / 36.0f) * n9, w11 = -snu * (1.0f / 12.0f) * n11;
  const float w10 = M.sd[10] * n10, w12 = M.sd[12] * n12;
  const float c13 = -snu * (1.0f / 4.0f);
  const float w13 = c13 * n13, w14 = c13 * n14, w15 = c13 * n15;
  const float s16 = M.sd[16], s17 = M.sd[17], s18 = M.sd[18];
  const float w16 = s16 * m16, w17 = s17 * m17;

  // back_transform
  const float dg0 = fma3(12.0f, w2, -30.0f * w1);
  const float Eax = fma3(-11.0f, w1, -4.0f * w2);
  const float Edg = fma3(8.0f, w1, w2);
  const float U = fma3(2.0f, w10, -w9), W = fma3(-2.0f, w12, w11);
  const float EU = Eax + U;
  const float W9 = w9 + w10, W11 = w11 + w12;
  const float EW = Edg + W9, Exy = EW + W11, Exz = EW - W11, Eyz = fma3(-2.0f, W9, Edg);
  const float e[NP] = {fma3(-2.0f, U, Eax), EU + W,    EU - W,    Exy + w13, Exy - w13,
                       Exz + w15,           Exz - w15, Eyz + w14, Eyz - w14};
  const float a3 = XCHG ? fma3(-s17, m17, w16) : fma3(s16, m16, -w17);
  const float a4 = XCHG ? fma3(s17, m17, w16) : fma3(s16, m16, w17);
  const float o[NP] = {-4.0f * w4,
                       -4.0f * w6,
                       -4.0f * w8,
                       (w4 + w6) + a3,
                       (w6 - w4) - a4,
                       (w4 + w8) + fma3(-s16, m16, s18 * m18),
                       (w8 - w4) + fma3(s16, m16, s18 * m18),
                       (w6 + w8) + fma3(s17, m17, -(s18 * m18)),
                       (w8 - w6) - fma3(s17, m17, s18 * m18)};
  g[0] += dg0;
  static_for<NP>([&](auto pi) {
#pragma clang fp contract(off)
    constexpr int p = pi;
    g[DV.pa[p]] += e[p] + o[p];
    g[DV.pb[p]] += e[p] - o[p];
  });
  return snu;
}

// A block owns WX x HY columns of nodes and marches through `planes` planes of z. Per plane, one
// thread per node of the (WX + 2) x (HY + 2) level-1 tile takes the first step of that plane into
// LDS; the second step of the plane below needs three level-1 planes, of which LDS holds the newest:
// each thread has already gathered what its node pulls from the two before (the directions with
// cz > 0 wait two planes in hz and hzz, those with cz = 0 one plane in hn; each array uses only
// those elements). The next plane's loads are issued before the second step, and LDS holds two planes
// in turn, so that one barrier per plane is enough. Blocks that follow one another on an XCD are
// neighbours, whose tile edges meet in its L2.
// What it saves is HBM traffic: a node is read once (and re-read at tile edges, out of the L2) and
// written once for two steps, 160 bytes against 320. What is left is that traffic and the vector unit
// side by side (540 instructions a thread and plane, half of the 6.9 us that a 64 x 13 plane takes).
// us a step, against single steps: 256^3 Smagorinsky 300 (418), constant viscosity 278 (418), 384^3
// 993 (1488), 128^3 44.3 (54.1), 96^3 18.6 (24.8). Measured on the way, 256^3 Smagorinsky: blocks dealt out over the XCDs in turn 325,
// two barriers and one plane of LDS 310, without the early loads 304.
template <int B, int WX, int HY, int KIND, bool XCHG, bool STREAM>
__global__ __launch_bounds__(B, B / 256) void pair_kernel(Geo G, PairPlan P, ModelF M, ViscF V,
                                                          const float* __restrict__ src, float* __restrict__ dst,
                                                          const float* __restrict__ snu_in,
                                                          float* __restrict__ snu_out) {
  constexpr int W1 = WX + 2, H1 = HY + 2, N1 = W1 * H1;
  static_assert(N1 <= B && WX * HY <= B, "a thread per node of either level");
  constexpr bool LAGGED = KIND != 0;
  __shared__ float planes[2][LAGGED ? Q + 1 : Q][N1];
  const int tile = (blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
  if (tile >= P.tiles) return;
  const int t = threadIdx.x;
  const int x0 = tile % P.tx * WX, y0 = tile / P.tx % P.ty * HY, z0 = tile / (P.tx * P.ty) * P.planes;
  const int nz2 = min(P.planes, G.nz - z0);
  // level 1: this thread's node, wrapped
  const int xa = x0 - 1 + t % W1, ya = y0 - 1 + t / W1;
  const bool on1 = t < N1 && xa <= G.nx && ya <= G.ny;
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
      pull_rows<Lat, float, false, true, true>(src, G, rows_of<Q, float>(G, x1, y1, z), y1, g);
      if constexpr (LAGGED) rate = snu_in[node_index(G, x1, y1, z)];
    }
  };
  float hn[Q], hz[Q], hzz[Q];
  float snu_l = 0.0f;
  load(0);
  for (int k = 0; k < nz2 + 2; ++k) {
    auto& sh = planes[k & 1];
    if (on1) {
      const float s1 = pair_update<KIND, XCHG>(g, M, V, rate);
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
        if constexpr (cz < 0) {
          full[i] = v;
        } else if constexpr (cz == 0) {
          full[i] = hn[i];
          hn[i] = v;
        } else {
          full[i] = hzz[i];
          hzz[i] = hz[i];
          hz[i] = v;
        }
      });
      if constexpr (LAGGED) snu_l = sh[Q][q];
    }
    if (k < nz2 + 1) load(k + 1);
    if (on2 && k >= 2) {
      const int z2 = z0 + k - 2;
      const float s2 = pair_update<KIND, XCHG>(full, M, V, snu_f);
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
bool pair_fits(const Geo& G) { return !packed_stream(G, Q, sizeof(float)); }
bool pair_stream(const Geo& G) {
  if (pair_fits(G)) return false;
  return runs_aligned(G, sizeof(float), 64) || size_t(G.N) * sizeof(float) * Q <= (size_t(1) << 28);
}

// One block per CU (LDS): 64 x 13 columns in 1024 threads (990 level-1 nodes), or 64 x 9 in 768 (726).
constexpr int kPairCols = 64, kPairRowsBig = 13, kPairRowsSmall = 9;

template <int B, int HY>
hipError_t launch_tile(const PairPlan& P, bool xchg, hipStream_t st, const Geo& G, const ModelF& M, const ViscF& V,
                       const float* src, float* dst, const float* snu_in, float* snu_out) {
  constexpr int WX = kPairCols;
  decltype(&pair_kernel<B, WX, HY, 0, false, false>) k;
  switch ((V.kind ? 1 : 0) + (pair_stream(G) ? 2 : 0) + (xchg ? 4 : 0)) {
    case 0: k = pair_kernel<B, WX, HY, 0, false, false>; break;
    case 1: k = pair_kernel<B, WX, HY, 1, false, false>; break;
    case 2: k = pair_kernel<B, WX, HY, 0, false, true>; break;
    case 3: k = pair_kernel<B, WX, HY, 1, false, true>; break;
    case 4: k = pair_kernel<B, WX, HY, 0, true, false>; break;
    case 5: k = pair_kernel<B, WX, HY, 1, true, false>; break;
    case 6: k = pair_kernel<B, WX, HY, 0, true, true>; break;
    default: k = pair_kernel<B, WX, HY, 1, true, true>; break;
  }
  const unsigned blocks = (P.tiles + kXcds - 1) / kXcds * kXcds;
  hipLaunchKernelGGL(k, dim3(blocks), dim3(B), 0, st, G, P, M, V, src, dst, snu_in, snu_out);
  return hipGetLastError();
}

}  // namespace

// The tile and the planes per block that cost the least: rounds of blocks over the CUs, times the planes
// that one marches through (two more than it stores), times the nodes of its tile (the small one costs 5 %
// more a node: 128^3 45.2 us a step against 44.3). `fill` is the box's share of that product. A node of it
// takes 32 ps of the chip for two steps and a node of a single step 26, so pairs need a fill of 0.6
// (us a step, single and pairs, Smagorinsky: 171x133x95, fill 0.66, 58.8 and 54.2, 150^3, 0.68, 90 and 90,
// 144^3, 0.62, 84 and 75, but 130^3, 0.54, 60.7 and 65.3). In the last-level cache a plane of a tile takes
// half of that: 72^3, fill 0.34, 12.2 and 11.6, 80^3, 0.41, 17.7 and 13.4, 66^3, 0.27, 11.1 and 11.2.
// Up to 64^3 single steps run out of the L2s (7.1 and 7.6 us).
PairPlan pair_plan(int storage, const Geo& G, const ViscF& V, const ForceF& Fo) {
  PairPlan best{};
  if (storage != 0 || G.walls || Fo.mode || Fo.strain_corr) return best;
  if (V.kind != 0 && !(V.kind == 1 && !V.drive_chai)) return best;
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
  const bool use = pair_fits(G) ? G.N > (1u << 18) && 10ll * G.N >= 3 * least : 10ll * G.N >= 6 * least;
  if (!use) return PairPlan{};
  return best;
}

hipError_t launch_pair(const PairPlan& P, const Geo& G, const ModelF& M, const ViscF& V, const void* src, void* dst,
                       const float* snu_in, float* snu_out, hipStream_t st) {
  if ((V.kind != 0) != (snu_in != nullptr) || (snu_in != nullptr) != (snu_out != nullptr) ||
      (snu_in && snu_in == snu_out))
    return hipErrorInvalidValue;
  const bool xchg = !packed_rows(G, sizeof(float)) && pull_mode(G, node_launch(G).block) == 2;
  const float* s = static_cast<const float*>(src);
  float* d = static_cast<float*>(dst);
  if (P.rows == kPairRowsBig) return launch_tile<1024, kPairRowsBig>(P, xchg, st, G, M, V, s, d, snu_in, snu_out);
  if (P.rows == kPairRowsSmall) return launch_tile<768, kPairRowsSmall>(P, xchg, st, G, M, V, s, d, snu_in, snu_out);
  return hipErrorInvalidValue;
}

}  // namespace d3q19
}  // namespace lbm
