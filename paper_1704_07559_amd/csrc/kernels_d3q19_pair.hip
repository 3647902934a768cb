// D3Q19, two steps per launch: FP32 storage, periodic or with walls, no body force, constant viscosity or the
// Smagorinsky model, lagged or implicit, with the Yu strain. Reference: the pipeline of two ordinary steps.
#include <hip/hip_runtime.h>

#include "d3q19.h"
#include "d3q19_node.h"
#include "pair_march.h"

namespace lbm {
namespace d3q19 {

// The node update of kernels_d3q19_step.hip (moments, Yu strain, lagged viscosity, relaxation,
// back-transform) for the cases above, with every fused product written out. The step kernels leave
// to the compiler which product of a sum is fused; what it picks there depends on the code around
// the sum, so the same source in this kernel rounds differently. The picks below are theirs:
// all pull modes share them but the LDS exchange (XCHG), whose instances differ in two sums (o[3],
// o[4]). Two steps of this kernel therefore equal two single steps bit for bit. That holds for the compiler
// these picks were read from: another may fuse the step kernels' sums differently, which the tests of pairs
// against single steps (every pull mode, law and lattice) then show, and the picks are to be renewed.
template <int KIND, bool XCHG>
struct PairUpdate {
  using Lat = d3q19::Lat;
  static constexpr bool kLagged = KIND == 1;
  static __device__ __forceinline__ float run(float (&g)[Q], const ModelF& M, const ViscF& V, float snu_prev) {
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
    if constexpr (KIND == 3) {
      // implicit_rate: strain_yu at (s_1, 0) and at (0, 1)
      const float a = M.s[1] * n1, r76 = ir * (1.0f / 76.0f);
      const float Pm[6] = {-a * (ir * (1.0f / 38.0f)), -(2.0f * a) * r76, -(2.0f * a) * r76, 0.0f, 0.0f, 0.0f};
      const float A[6] = {-(19.0f * n9) * (ir * (1.0f / 38.0f)), (19.0f * fma3(-3.0f, n11, n9)) * r76,
                          (19.0f * fma3(3.0f, n11, n9)) * r76,   -1.5f * n13 * ir,
                          -1.5f * n14 * ir,                      -1.5f * n15 * ir};
      snu = implicit_smagorinsky(Pm, A, V.nu0, V.csmag2);
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
};

PairPlan pair_plan(int storage, const Geo& G, const ViscF& V, const ForceF& Fo) {
  return plan_pairs(Q, storage, G, V, Fo);
}

PairPlan pair_tiles(int storage, const Geo& G, const ViscF& V, const ForceF& Fo, int cols, int rows, int planes) {
  return march_tiles(storage, G, V, Fo, cols, rows, planes);
}

template <bool XCHG>
static hipError_t launch_kind(const PairPlan& P, const Geo& G, const ModelF& M, const ViscF& V, const void* src,
                              void* dst, const float* snu_in, float* snu_out, hipStream_t st) {
  switch (V.kind) {
    case 0: return launch_march<PairUpdate<0, XCHG>>(P, st, G, M, V, src, dst, snu_in, snu_out);
    case 1: return launch_march<PairUpdate<1, XCHG>>(P, st, G, M, V, src, dst, snu_in, snu_out);
    case 3: return launch_march<PairUpdate<3, XCHG>>(P, st, G, M, V, src, dst, snu_in, snu_out);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_pair(const PairPlan& P, const Geo& G, const ModelF& M, const ViscF& V, const void* src, void* dst,
                       const float* snu_in, float* snu_out, hipStream_t st) {
  const bool xchg = !packed_rows(G, Q, sizeof(float), V) && pull_mode(G, node_launch(G).block) == 2;
  return xchg ? launch_kind<true>(P, G, M, V, src, dst, snu_in, snu_out, st)
              : launch_kind<false>(P, G, M, V, src, dst, snu_in, snu_out, st);
}

}  // namespace d3q19
}  // namespace lbm
