// D3Q19 kernels around the step: initial state, the strain query, canonical gather/scatter
// and the diagnostics reduction. One thread per node (the reduction: one x-row per block at
// a time).
#include <hip/hip_runtime.h>

#include "d3q19.h"
#include "d3q19_node.h"
#include "internal.h"
#include "launch.h"
#include "reduce.h"

namespace lbm {
namespace d3q19 {

// ------------------------------------------------------------------------------------------
// Strain of the current state (read only)
// ------------------------------------------------------------------------------------------
// CACHED: the loads go through the caches (cached_strain); STREAM: streaming stores (plane_stream).
template <typename S, bool CACHED, bool STREAM>
__global__ __launch_bounds__(kMaxBlock) void strain_kernel(Geo G, ModelF M, ViscF V, ForceF Fo, const S* buf,
                                                     const float* snu_f, int kind, float* S_out) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y * blockDim.y + threadIdx.y;
  const int z = blockIdx.z;
  if (x >= G.nx || y >= G.ny) return;
  const Node<Q, S> nb = node_at<Q, S>(G, x, y, z);
  float g[Q];
  pull_rows<Lat, S, true, true, CACHED>(buf, G, nb.rows, y, g);
  const Pairs P = make_pairs(g);
  const float drho = delta_rho(P);
  float jx = momentum<0>(P), jy = momentum<1>(P), jz = momentum<2>(P);
  float Fx, Fy, Fz;
  load_force(Fo, G.N, nb.self, Fx, Fy, Fz);
  jx += 0.5f * Fx;
  jy += 0.5f * Fy;
  jz += 0.5f * Fz;
  const Neq n = noneq_moments(P, drho, jx, jy, jz, M);
  const StrainIn<true> si = strain_in_state(n, jx, jy, jz, Fx, Fy, Fz, M, Fo);
  const float snu = V.kind == 3 ? implicit_rate(P, drho, jx, jy, jz, si, M, V) : (snu_f ? snu_f[nb.self] : M.s[9]);
  float S6[6];
  if (kind == 2) {
    float r[Q];
    rates_with(M, snu, r);
    strain_chai_in(P, drho, jx, jy, jz, r, si, M.inv_rho0, S6);
  } else {
    strain_yu(si.ns, M.s[1], snu, M.inv_rho0, S6);
  }
#pragma unroll
  for (int c = 0; c < 6; ++c) plane_store<STREAM>(&S_out[static_cast<size_t>(c) * G.N + nb.self], S6[c]);
}

// ------------------------------------------------------------------------------------------
// Initial state g^eq(delta_rho, rho0 u) [+ Chapman-Enskog non-equilibrium part]
// ------------------------------------------------------------------------------------------
template <typename S>
__global__ __launch_bounds__(kMaxBlock) void init_kernel(Geo G, ModelF M, S* buf, float* snu, const float* rho_u,
                                                   const float* grad_u) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y * blockDim.y + threadIdx.y;
  const int z = blockIdx.z;
  if (x >= G.nx || y >= G.ny) return;
  const Node<Q, S> nb = node_at<Q, S>(G, x, y, z);
  const unsigned self = nb.self;
  float drho = 0.f, ux = 0.f, uy = 0.f, uz = 0.f;
  if (rho_u) {
    drho = rho_u[self];
    ux = rho_u[G.N + self];
    uy = rho_u[2 * static_cast<size_t>(G.N) + self];
    uz = rho_u[3 * static_cast<size_t>(G.N) + self];
  }
  float g[Q];
  equilibrium(drho, M.rho0 * ux, M.rho0 * uy, M.rho0 * uz, M.inv_rho0, g);
  if (grad_u) {
    // d[a*3+b] = d j_b / d x_a; non-equilibrium moments of the Chapman-Enskog relations
    // (Eq. YuLuobasis), every other row zero.
    float d[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) d[k] = M.rho0 * grad_u[static_cast<size_t>(k) * G.N + self];
    const float div = d[0] + d[4] + d[8];
    const float s1 = M.s[1], sn = M.s[9];
    float mn[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) mn[k] = 0.0f;
    mn[1] = -38.0f * div / (3.0f * s1);
    mn[9] = -2.0f * (3.0f * d[0] - div) / (3.0f * sn);
    mn[11] = -2.0f * (d[4] - d[8]) / (3.0f * sn);
    mn[13] = -(d[1] + d[3]) / (3.0f * sn);
    mn[14] = -(d[5] + d[7]) / (3.0f * sn);
    mn[15] = -(d[2] + d[6]) / (3.0f * sn);
    add_neq_from_moments(mn, g);
  }
  scatter_rows<Lat, S>(buf, G, nb.rows, y, g);
  if (snu) snu[self] = M.s[9];
}

// CACHED: loads and stores through the caches (cached_get).
template <typename S, bool CACHED>
__global__ __launch_bounds__(kMaxBlock) void get_kernel(Geo G, const S* buf, float* canon) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y * blockDim.y + threadIdx.y;
  const int z = blockIdx.z;
  if (x >= G.nx || y >= G.ny) return;
  const Node<Q, S> nb = node_at<Q, S>(G, x, y, z);
  float g[Q];
  pull_rows<Lat, S, true, true, CACHED>(buf, G, nb.rows, y, g);
  store_local<Q, !CACHED>(canon, G, nb.self * 4u, g);
}

template <typename S>
__global__ __launch_bounds__(kMaxBlock) void set_kernel(Geo G, S* buf, const float* canon) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y * blockDim.y + threadIdx.y;
  const int z = blockIdx.z;
  if (x >= G.nx || y >= G.ny) return;
  const Node<Q, S> nb = node_at<Q, S>(G, x, y, z);
  float g[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) g[i] = canon[static_cast<size_t>(i) * G.N + nb.self];
  scatter_rows<Lat, S>(buf, G, nb.rows, y, g);
}

// ------------------------------------------------------------------------------------------
// Diagnostics: mass, momentum, kinetic energy, sum S:S (Yu), max |u|, non-finite count
// ------------------------------------------------------------------------------------------
// Bound by HBM in FP32 (256^3: 0.222 ms = 6.05 TB/s, 0.231 with whole rows per block; 128^3 35 us
// against 56) and by instruction issue with 16-bit storage (256^3 FP16 0.150 ms against 0.169).
template <typename S, bool CORR, bool IMPLICIT>
__global__ __launch_bounds__(256) void reduce_kernel(Geo G, ModelF M, ViscF V, ForceF Fo, NodeWalk W, const S* buf,
                                                     const float* snu_f, double* partials) {
  double acc[kReduceVals] = {0, 0, 0, 0, 0, 0, 0, 0};
  const double per_jj = 0.5 / M.rho0;
  for (unsigned self = blockIdx.x * 256 + threadIdx.x; self < G.N; self += gridDim.x * 256) {
    const Coord c = coord_of(G, W, self);
    // (loaded ahead of the populations: behind them its latency would stand alone)
    float snu = (!IMPLICIT && snu_f) ? snu_f[self] : M.s[9];
    float g[Q];
    pull_rows<Lat, S, true, false>(buf, G, rows_of<Q, S>(G, c.x, c.y, c.z), c.y, g);
    const Pairs P = make_pairs(g);
    const float drho = delta_rho(P);
    // (their sum is non-finite where a population is, so that finite nodes pay one test)
    if (!isfinite(drho)) {
      int bad = 0;
#pragma unroll
      for (int i = 0; i < Q; ++i) bad += !isfinite(g[i]);
      acc[7] += bad;
    }
    float jx = momentum<0>(P), jy = momentum<1>(P), jz = momentum<2>(P);
    float Fx, Fy, Fz;
    load_force(Fo, G.N, self, Fx, Fy, Fz);
    jx += 0.5f * Fx;
    jy += 0.5f * Fy;
    jz += 0.5f * Fz;
    const Neq n = noneq_moments(P, drho, jx, jy, jz, M);
    float SF[Q];
    if constexpr (CORR) force_moments(jx, jy, jz, Fx, Fy, Fz, M.inv_rho0, SF);
    const StrainIn<CORR> si = strain_in<CORR>(n, SF);
    if constexpr (IMPLICIT) snu = implicit_rate(P, drho, jx, jy, jz, si, M, V);
    float S6[6];
    strain_yu(si.ns, M.s[1], snu, M.inv_rho0, S6);
    const double jj = static_cast<double>(jx) * jx + static_cast<double>(jy) * jy + static_cast<double>(jz) * jz;
    acc[0] += drho;
    acc[1] += jx;
    acc[2] += jy;
    acc[3] += jz;
    acc[4] += jj * per_jj;
    double ss = 0.0;
#pragma unroll
    for (int k = 0; k < 6; ++k) ss += (k < 3 ? 1.0 : 2.0) * static_cast<double>(S6[k]) * S6[k];
    acc[5] += ss;
    acc[6] = fmax(acc[6], jj);  // max |j|^2: the final pass takes sqrt(.) / rho0 once
  }
  block_reduce_store(acc, partials);
}

// ------------------------------------------------------------------------------------------
// Launchers
// ------------------------------------------------------------------------------------------
template <typename S>
static const S* cbuf(const void* p) {
  return static_cast<const S*>(p);
}

template <typename S>
static void launch_strain_t(const Launch& L, size_t lds, hipStream_t st, const Geo& G, const ModelF& M,
                            const ViscF& V, const ForceF& Fo, const void* buf, const float* snu, int kind, float* S_out) {
  // (rows whose runs are aligned are multiples of 8 nodes)
  const auto k = !cached_strain(G, Q, sizeof(S)) ? strain_kernel<S, false, true>
                 : plane_stream(G)               ? strain_kernel<S, true, true>
                                                 : strain_kernel<S, true, false>;
  hipLaunchKernelGGL(k, L.grid, L.block, lds, st, G, M, V, Fo, cbuf<S>(buf), snu, kind, S_out);
}

hipError_t launch_strain(int storage, const Geo& G, const ModelF& M, const ViscF& V, const ForceF& Fo, const void* buf,
                         const float* snu, int kind, float* S_out, hipStream_t st) {
  const Launch L = node_launch(G);
  // whole 256-node rows: 5 blocks per CU instead of 8 (+1.9 % at 256^3; 4 blocks lost 0.6 %)
  const size_t lds = (storage == 0 && L.block.x == 256 && L.block.y == 1) ? lds_cap_bytes(5, 0) : 0;
  switch (storage) {
    case 0: launch_strain_t<float>(L, lds, st, G, M, V, Fo, buf, snu, kind, S_out); break;
    case 1: launch_strain_t<_Float16>(L, lds, st, G, M, V, Fo, buf, snu, kind, S_out); break;
    case 2: launch_strain_t<__bf16>(L, lds, st, G, M, V, Fo, buf, snu, kind, S_out); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_init(int storage, const Geo& G, const ModelF& M, void* buf, float* snu, const float* rho_u,
                       const float* grad_u, hipStream_t st) {
  const Launch L = node_launch(G);
  switch (storage) {
    case 0: hipLaunchKernelGGL(init_kernel<float>, L.grid, L.block, 0, st, G, M, static_cast<float*>(buf), snu, rho_u, grad_u); break;
    case 1: hipLaunchKernelGGL(init_kernel<_Float16>, L.grid, L.block, 0, st, G, M, static_cast<_Float16*>(buf), snu, rho_u, grad_u); break;
    case 2: hipLaunchKernelGGL(init_kernel<__bf16>, L.grid, L.block, 0, st, G, M, static_cast<__bf16*>(buf), snu, rho_u, grad_u); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename S>
static void launch_get_t(hipStream_t st, const Geo& G, const void* buf, float* canon) {
  const Launch L = node_launch(G);
  const auto k = cached_get(G, Q, sizeof(S)) ? get_kernel<S, true> : get_kernel<S, false>;
  hipLaunchKernelGGL(k, L.grid, L.block, 0, st, G, cbuf<S>(buf), canon);
}

hipError_t launch_get(int storage, const Geo& G, const void* buf, float* canon, hipStream_t st) {
  switch (storage) {
    case 0: launch_get_t<float>(st, G, buf, canon); break;
    case 1: launch_get_t<_Float16>(st, G, buf, canon); break;
    case 2: launch_get_t<__bf16>(st, G, buf, canon); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_set(int storage, const Geo& G, void* buf, const float* canon, hipStream_t st) {
  const Launch L = node_launch(G);
  switch (storage) {
    case 0: hipLaunchKernelGGL(set_kernel<float>, L.grid, L.block, 0, st, G, static_cast<float*>(buf), canon); break;
    case 1: hipLaunchKernelGGL(set_kernel<_Float16>, L.grid, L.block, 0, st, G, static_cast<_Float16*>(buf), canon); break;
    case 2: hipLaunchKernelGGL(set_kernel<__bf16>, L.grid, L.block, 0, st, G, static_cast<__bf16*>(buf), canon); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// The force-corrected strain and the implicit rate are instances of their own: their code costs
// the plain diagnostics 10 VGPRs and a tenth of its instructions.
template <typename S>
static void launch_reduce_t(unsigned nb, hipStream_t st, const Geo& G, const ModelF& M, const ViscF& V,
                            const ForceF& Fo, const S* buf, const float* snu, double* partials) {
  // FP32 with more blocks than fit at once: 4 blocks per CU instead of the 7 its registers allow
  // (3.5 % less time per call at 256^3; 3 blocks 7 % more)
  const size_t cap = sizeof(S) == 4 && nb > kReduceFill ? lds_cap_bytes(4, 4 * kReduceVals * sizeof(double)) : 0;
  decltype(&reduce_kernel<S, false, false>) f;
  switch ((Fo.strain_corr ? 1 : 0) + (V.kind == 3 ? 2 : 0)) {
    case 0: f = reduce_kernel<S, false, false>; break;
    case 1: f = reduce_kernel<S, true, false>; break;
    case 2: f = reduce_kernel<S, false, true>; break;
    default: f = reduce_kernel<S, true, true>; break;
  }
  hipLaunchKernelGGL(f, dim3(nb), dim3(256), cap, st, G, M, V, Fo, node_walk(G), buf, snu, partials);
}

hipError_t launch_reduce(int storage, const Geo& G, const ModelF& M, const ViscF& V, const ForceF& Fo, const void* buf,
                         const float* snu, double* partials, double* out, hipStream_t st) {
  const unsigned nb = reduce_blocks(G);
  switch (storage) {
    case 0: launch_reduce_t<float>(nb, st, G, M, V, Fo, cbuf<float>(buf), snu, partials); break;
    case 1: launch_reduce_t<_Float16>(nb, st, G, M, V, Fo, cbuf<_Float16>(buf), snu, partials); break;
    case 2: launch_reduce_t<__bf16>(nb, st, G, M, V, Fo, cbuf<__bf16>(buf), snu, partials); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_reduce_final(partials, static_cast<int>(nb), out, st, static_cast<double>(M.rho0));
}

}  // namespace d3q19
}  // namespace lbm
