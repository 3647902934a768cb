// D3Q15, two steps per launch: FP32 storage, periodic or with walls, no body force, constant viscosity or the
// Smagorinsky model, lagged or implicit, with the Yu-type strain.
#include <hip/hip_runtime.h>

#include "d3q15.h"
#include "pair_march.h"

namespace lbm {
namespace d3q15 {

// The node update of kernels_d3q15.hip for the cases above, with every fused product written out as the
// step kernels' instances (of every pull mode alike) fuse it, so that two steps of this kernel equal two
// single steps bit for bit. The moments are small whole-number sums and round alike however fused.
template <int KIND>
struct PairUpdate {
  using Lat = d3q15::Lat;
  static constexpr bool kLagged = KIND == 1;
  static __device__ __forceinline__ float run(float (&g)[Q], const ModelF& M, const ViscF& V, float snu_prev) {
#pragma clang fp contract(off)
    const Pairs P = make_pairs(g);
    const float drho = delta_rho(P);
    const float jx = momentum<0>(P), jy = momentum<1>(P), jz = momentum<2>(P);

    // non-equilibrium moments (noneq_moments)
    const float ir = M.inv_rho0;
    const float jx2 = jx * jx, jy2 = jy * jy, jz2 = jz * jz;
    const float j2 = fma3(jz, jz, fma3(jy, jy, jx2));
    const float n1 = moment<1>(P) - fma3(j2, ir, -drho);
    const float n2 = moment<2>(P) - fma3(-5.0f, j2 * ir, drho);
    const float n4 = fma3(7.0f / 3.0f, jx, moment<4>(P));
    const float n6 = fma3(7.0f / 3.0f, jy, moment<6>(P));
    const float n8 = fma3(7.0f / 3.0f, jz, moment<8>(P));
    const float n9 = fma3(-fma3(-jz, jz, fma3(2.0f, jx2, -jy2)), ir, moment<9>(P));
    const float n10 = fma3(-fma3(jy, jy, -jz2), ir, moment<10>(P));
    const float n11 = fma3(-(jx * jy), ir, moment<11>(P));
    const float n12 = fma3(-(jy * jz), ir, moment<12>(P));
    const float n13 = fma3(-(jx * jz), ir, moment<13>(P));
    const float n14 = moment<14>(P);

    float snu = M.s[9];
    if constexpr (KIND == 1) {
      // strain_yu, strain_sq and viscous_rate
      const float a = M.s[1] * n1, b = snu_prev * n9, c3 = 3.0f * snu_prev;
      const float t = fma3(2.0f, a, -b);
      const float Sxx = -fma3(M.s[1], n1, b) * (0.5f * ir);
      const float Syy = -fma3(c3, n10, t) * (0.25f * ir);
      const float Szz = -fma3(-c3, n10, t) * (0.25f * ir);
      const float Sxy = -1.5f * snu_prev * n11 * ir;
      const float Syz = -1.5f * snu_prev * n12 * ir;
      const float Sxz = -1.5f * snu_prev * n13 * ir;
      const float diag = fma3(Szz, Szz, fma3(Sxx, Sxx, Syy * Syy));
      const float off = fma3(Sxz, Sxz, fma3(Sxy, Sxy, Syz * Syz));
      const float gamma = fast_sqrt(2.0f * fma3(2.0f, off, diag));
      snu = fast_rcp(fma3(3.0f, fma3(V.csmag2, gamma, V.nu0), 0.5f));
    }
    if constexpr (KIND == 3) {
      // implicit_rate: strain_yu at (s_e, 0) and at (0, 1)
      const float a = M.s[1] * n1;
      const float Pm[6] = {-a * (0.5f * ir), -(2.0f * a) * (0.25f * ir), -(2.0f * a) * (0.25f * ir), 0.0f, 0.0f,
                           0.0f};
      const float A[6] = {-n9 * (0.5f * ir), -fma3(3.0f, n10, -n9) * (0.25f * ir), fma3(3.0f, n10, n9) * (0.25f * ir),
                          -1.5f * n11 * ir,  -1.5f * n12 * ir,                    -1.5f * n13 * ir};
      snu = implicit_smagorinsky(Pm, A, V.nu0, V.csmag2);
    }

    // relaxation and back-transform (add_back_transform), w_k = dm_k / D_k
    constexpr float i4 = 1.0f / 40.0f, i9 = 1.0f / 12.0f;
    const float d2 = -M.s[2] * n2, d6 = -M.s[6] * n6, d8 = -M.s[8] * n8, d9 = -snu * n9;
    const float w1 = -M.s[1] * n1 * (1.0f / 18.0f), w2 = d2 * (1.0f / 360.0f), w4 = -M.s[4] * n4 * i4;
    const float w10 = -snu * n10 * 0.25f, w11 = -snu * n11 * 0.125f, w12 = -snu * n12 * 0.125f,
                w13 = -snu * n13 * 0.125f, w14 = -M.s[14] * n14 * 0.125f;
    const float ax = fma3(-4.0f, w2, -w1), yz = fma3(-d9, i9, ax);
    const float corner = fma3(d2, 1.0f / 360.0f, w1);
    const float c_p = corner + w11, c_m = corner - w11;
    const float e[NP] = {fma3(2.0f, d9 * i9, ax), yz + w10,        yz - w10,       c_p + w12 + w13,
                         c_p - w12 - w13,          c_m - w12 + w13, c_m + w12 - w13};
    const float p46 = fma3(d6, i4, w4), m46 = fma3(-d6, i4, w4);
    const float o[NP] = {-4.0f * w4,
                         -4.0f * (d6 * i4),
                         -4.0f * (d8 * i4),
                         fma3(d8, i4, p46) + w14,
                         fma3(-d8, i4, p46) - w14,
                         fma3(d8, i4, m46) - w14,
                         fma3(d8, i4, -m46) - w14};
    g[0] += fma3(16.0f, w2, -2.0f * w1);
    static_for<NP>([&](auto pi) {
#pragma clang fp contract(off)
      constexpr int p = pi;
      g[DV.pa[p]] += e[p] + o[p];
      g[DV.pb[p]] += e[p] - o[p];
    });
    return snu;
  }
};

PairPlan pair_plan(int storage, const Geo& G, const ViscF& V, const ForceF& Fo) {
  return plan_pairs(Q, storage, G, V, Fo);
}

PairPlan pair_tiles(int storage, const Geo& G, const ViscF& V, const ForceF& Fo, int cols, int rows, int planes) {
  return march_tiles(storage, G, V, Fo, cols, rows, planes);
}

hipError_t launch_pair(const PairPlan& P, const Geo& G, const ModelF& M, const ViscF& V, const void* src, void* dst,
                       const float* snu_in, float* snu_out, hipStream_t st) {
  switch (V.kind) {
    case 0: return launch_march<PairUpdate<0>>(P, st, G, M, V, src, dst, snu_in, snu_out);
    case 1: return launch_march<PairUpdate<1>>(P, st, G, M, V, src, dst, snu_in, snu_out);
    case 3: return launch_march<PairUpdate<3>>(P, st, G, M, V, src, dst, snu_in, snu_out);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace d3q15
}  // namespace lbm
