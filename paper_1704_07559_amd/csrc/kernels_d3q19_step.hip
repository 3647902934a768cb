// D3Q19 fused collide-stream-strain step.
//
// One thread owns one node. The step pulls the 19 post-collision populations of the
// previous step from the neighbours (Eq. mrteq read backwards), forms the moments
// m = T g (Section 2), the equilibrium moments (Eq. meq), the strain of this pre-collision
// state by the Yu formula (Eq. LuoS) and/or the Chai formula (Eq. ChaiS), the new s_nu of
// the viscosity model, relaxes in moment space (Eq. mrteqvT) and stores the 19
// post-collision populations at the node itself. Loads are coalesced along x (shifted by
// at most one element), stores are aligned and coalesced.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "d3q19.h"
#include "d3q19_node.h"
#include "internal.h"
#include "launch.h"

namespace lbm {
namespace d3q19 {

// Everything one node does between the pull and the store: moments, strain of the incoming
// state (Yu and/or Chai, with the lagged s_nu or the implicitly solved one), viscosity
// model, relaxation with the Guo term, back-transform. g holds the pulled pre-collision
// populations on entry and the post-collision populations on exit; `self` is the node's
// element offset in the fields. PACK: g was converted from FP16 on load; the FP16 values are
// kept packed (pack_pairs) and both their uses, the pair sums and the final sums, read them
// through mixed-precision FMAs. snu_ahead (AHEAD): the node's lagged rate (read only where io.snu is
// given), which the caller loads along with the populations, so that its latency hides behind theirs
// (ahead of the exchange's barrier, else right after their loads: in front of them its branch drags
// every kernel argument's load there, 0.3 us more in a small box): at its use it cost 7 % of the BF16
// 384 x 384 x 48 step (105 us against 97.5) and 9 % of FP16 200^3 (139 against 126). It is taken over inside
// the branch, and opaque, because merging that branch into the code around changes which products of a sum the
// compiler fuses. Whole rows pulled directly (small ragged boxes) keep the late load: 60^3 8.1 us a step
// against 8.8; so do exchanged rows in launches of a middle size (route_of).
template <bool CORR, bool PACK, bool AHEAD>
__device__ __forceinline__ void node_update(float (&g)[Q], unsigned self, const Geo& G, const ModelF& M,
                                            const ViscF& V, const ForceF& Fo, const StepIO& io, float snu_ahead) {
  HalfPairs hp;
  Pairs P_;
  if constexpr (PACK) {
    hp = pack_pairs(g);
    P_ = make_pairs_packed(hp);
  } else {
    P_ = make_pairs(g);
  }
  const float drho = delta_rho(P_);
  float jx = momentum<0>(P_), jy = momentum<1>(P_), jz = momentum<2>(P_);
  float Fx, Fy, Fz;
  load_force(Fo, G.N, self, Fx, Fy, Fz);
  if (Fo.mode) {
    jx = __builtin_fmaf(0.5f, Fx, jx);
    jy = __builtin_fmaf(0.5f, Fy, jy);
    jz = __builtin_fmaf(0.5f, Fz, jz);
  }
  const Neq n = noneq_moments(P_, drho, jx, jy, jz, M);
  // the Guo source in moment space (the relaxation's forcing term); with CORR it is formed
  // here, before the strain, since half of it joins the non-equilibrium part
  float SF[Q];
  if constexpr (CORR) force_moments(jx, jy, jz, Fx, Fy, Fz, M.inv_rho0, SF);
  const StrainIn<CORR> si = strain_in<CORR>(n, SF);

  float Syu[6], Sch[6];
  float snu = M.s[9];
  float s_strain;  // the s_nu this step's strain is taken with
  if (V.kind == 3) {
    // implicit coupling: the strain at the rate of this very collision
    snu = implicit_rate(P_, drho, jx, jy, jz, si, M, V);
    s_strain = snu;
    if (io.S_out) {
      if (io.emit == 2) {
        float r[Q];
        rates_with(M, snu, r);
        strain_chai_in(P_, drho, jx, jy, jz, r, si, M.inv_rho0, Sch);
      } else {
        strain_yu(si.ns, M.s[1], snu, M.inv_rho0, Syu);
      }
#pragma unroll
      for (int c = 0; c < 6; ++c)
        stream_store(&io.S_out[static_cast<size_t>(c) * G.N + self], io.emit == 2 ? Sch[c] : Syu[c]);
    }
  } else {
    // lagged coupling: the strain of the incoming state with the rates of the previous collision
    float snu_prev = M.s[9];
    if (io.snu) {
      if constexpr (AHEAD) {
        asm volatile("" : "+v"(snu_ahead));
        snu_prev = snu_ahead;
      } else {
        snu_prev = io.snu[self];
      }
    }
    s_strain = snu_prev;
    const bool need_yu = io.emit == 1 || (V.kind != 0 && !V.drive_chai);
    const bool need_chai = io.emit == 2 || (V.kind != 0 && V.drive_chai);
    if (need_yu) strain_yu(si.ns, M.s[1], snu_prev, M.inv_rho0, Syu);
    if (need_chai) {
      float r[Q];
      rates_with(M, snu_prev, r);
      strain_chai_in(P_, drho, jx, jy, jz, r, si, M.inv_rho0, Sch);
    }
    if (io.S_out) {
#pragma unroll
      for (int c = 0; c < 6; ++c)
        stream_store(&io.S_out[static_cast<size_t>(c) * G.N + self], io.emit == 2 ? Sch[c] : Syu[c]);
    }
    // viscosity model -> s_nu of this collision (kept for the next step's strain)
    if (V.kind != 0) {
      snu = viscous_rate(V.drive_chai ? strain_sq(Sch) : strain_sq(Syu), V);
      io.snu[self] = snu;
    }
  }

  // Relaxation in moment space, dm_k = -s_k (m_k - m_k^eq) + (1 - s_k/2) S_F,k, taken
  // directly as w_k = dm_k / D_k for the back-transform g += T^T w: the row norms are folded
  // into the rates (M.sd, M.fd; per node for the s_nu rows).
  float w[Q];
  w[0] = 0.0f;
  constexpr float iD3 = 1.0f / static_cast<float>(DV.D[3]);
  w[3] = Fx * iD3;
  w[5] = Fy * iD3;
  w[7] = Fz * iD3;
  static_for<Q>([&](auto ki) {
    constexpr int k = ki;
    if constexpr (k != 0 && k != 3 && k != 5 && k != 7) {
      constexpr float iD = 1.0f / static_cast<float>(DV.D[k]);
      const float c = is_nu_slot(k) ? -snu * iD : M.sd[k];
      w[k] = c * n.m[k];
    }
  });
  if (Fo.mode) {
    if constexpr (!CORR) force_moments(jx, jy, jz, Fx, Fy, Fz, M.inv_rho0, SF);
    static_for<Q>([&](auto ki) {
      constexpr int k = ki;
      if constexpr (k != 0 && k != 3 && k != 5 && k != 7 && k < 16) {
        constexpr float iD = 1.0f / static_cast<float>(DV.D[k]);
        const float c = is_nu_slot(k) ? __builtin_fmaf(-0.5f * iD, snu, iD) : M.fd[k];
        w[k] = __builtin_fmaf(c, SF[k], w[k]);
      }
    });
  }
  if constexpr (PACK) add_scaled_back_transform_packed(w, hp, g);
  else add_scaled_back_transform(w, g);

  if (io.save) {
    // what the adjoint of this step needs: j, and for a strain-dependent viscosity the
    // moments the strain took (Eq. LuoS rows; force-corrected when it is) and its rate
    const size_t N = G.N;
    stream_store(&io.save[self], jx);
    stream_store(&io.save[N + self], jy);
    stream_store(&io.save[2 * N + self], jz);
    if (V.kind != 0) {
      stream_store(&io.save[3 * N + self], si.ns.m[1]);
      stream_store(&io.save[4 * N + self], si.ns.m[9]);
      stream_store(&io.save[5 * N + self], si.ns.m[11]);
      stream_store(&io.save[6 * N + self], si.ns.m[13]);
      stream_store(&io.save[7 * N + self], si.ns.m[14]);
      stream_store(&io.save[8 * N + self], si.ns.m[15]);
      stream_store(&io.save[9 * N + self], s_strain);
    }
  }
}

// ------------------------------------------------------------------------------------------
// The fused step: one thread per node
// ------------------------------------------------------------------------------------------
// XMODE: how a block pulls along x (pull_mode: 0 part rows, 1 whole rows, 2 whole rows with
// the LDS exchange, 3 whole rows, cached loads and packed stores), 4 as 2 with the lagged rate
// loaded at its use. CORR: the force-corrected strain (a separate instance, so that the plain
// step keeps its register budget).
// FP16 storage without the LDS exchange (whose x-shifted values arrive through LDS as FP32)
// keeps the pulled values packed; that instance fits 80 VGPRs without spilling and is asked
// for 6 waves per SIMD (the 16-bit step moves half the bytes per wave, so it needs the extra
// wave in flight: 4 instead of 5 waves cost it 6.5 %, 6 instead of 5 gained 3.7 %).
template <typename S, int XMODE>
constexpr bool kPackHalves = Codec<S>::kMixedFma && XMODE != 2 && XMODE != 4;
// Where the lagged rate is loaded ahead of its use (see node_update). FP16 part rows gain nothing from it and lose
// on ragged rows (1000x200x40 153 us a step against 144, 384x384x96 188 and 187).
template <typename S, int XMODE>
constexpr bool kRateAhead = XMODE == 2 || XMODE == 3 || (XMODE == 0 && !kPackHalves<S, XMODE>);
template <typename S, int XMODE, bool CORR>
constexpr int kMinWavesPerEU = (kPackHalves<S, XMODE> && !CORR && XMODE != 3) ? 6 : 1;

template <typename S, bool WALLS, int XMODE, bool CORR>
__global__ __launch_bounds__(XMODE == 3 ? kMaxPackedBlock : kMaxBlock, (kMinWavesPerEU<S, XMODE, CORR>))
void step_kernel(Geo G, ModelF M, ViscF V, ForceF Fo, StepIO io) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y * blockDim.y + threadIdx.y;
  const int z = blockIdx.z;
  if constexpr (XMODE == 3) {
    extern __shared__ __align__(16) char chunk[];
    const bool on = y < G.ny;
    float g[Q];
    if (on) {
      pull_rows<Lat, S, WALLS, true, true>(static_cast<const S*>(io.src), G, rows_of<Q, S>(G, x, y, z), y, g);
      const unsigned self = node_index(G, x, y, z);
      const float snu_ahead = io.snu ? io.snu[self] : 0.0f;
      node_update<CORR, kPackHalves<S, XMODE>, true>(g, self, G, M, V, Fo, io, snu_ahead);
    }
    store_rows_packed<Q>(static_cast<S*>(io.dst), G, reinterpret_cast<S*>(chunk), on, z, io.stream, g);
  } else {
    if (x >= G.nx || y >= G.ny) return;
    const Rows<Q, S> r = rows_of<Q, S>(G, x, y, z);
    const unsigned self = node_index(G, x, y, z);
    float g[Q], snu_ahead = 0.0f;
    constexpr bool ahead = kRateAhead<S, XMODE>;
    if constexpr (XMODE == 2 || XMODE == 4) {
      if (ahead && io.snu) snu_ahead = io.snu[self];
      pull_rows_staged<Lat, S, WALLS>(static_cast<const S*>(io.src), G, r, y, g);
    } else {
      pull_rows<Lat, S, WALLS, XMODE == 1>(static_cast<const S*>(io.src), G, r, y, g);
      if (ahead && io.snu) snu_ahead = io.snu[self];
    }
    node_update<CORR, kPackHalves<S, XMODE>, ahead>(g, self, G, M, V, Fo, io, snu_ahead);
    store_rows<Q>(static_cast<S*>(io.dst), G, r, g);
  }
}

// Blocks per CU, 0 for as many as the registers allow (5 in FP32). FP32: fewer in the two shapes where that was
// measured faster. Whole 256-node rows, us a step: 4 blocks (256^3 Smagorinsky 423 and 429 with 5; power law
// between walls 422 and 415, but 3 blocks 465), in large boxes without walls or force 3 (256^3 416, constant
// viscosity 414 and 422 with 4; but 256 x 256 x 4, 4 blocks to a CU, 10.2 and 7.4, and between walls with a
// force 5 % more at every size). 128 x 2 part rows: 4 blocks, +1.8 % at 384^3. Whole 128-node rows (the 128 x
// 128 x 512 channel) ran as fast uncapped and 4.4 % slower capped, so other shapes keep their occupancy. The
// 16-bit steps want more waves, not fewer.
static StepRoute route_of(size_t elem, const Launch& L, const Geo& G, const ViscF& V, const ForceF& Fo) {
  if (packed_rows(G, Q, elem, V)) return StepRoute{3, 0, false};
  StepRoute r{pull_mode(G, L.block), 0, false};
  if (elem == 4) {
    if (r.mode == 2 && L.block.x == 256 && L.block.y == 1)
      r.blocks = G.N >= (1u << 23) && !G.walls && !Fo.mode && V.kind != 2 ? 3 : 4;
    else if (r.mode == 0 && L.block.x == 128 && L.block.y == 2)
      r.blocks = 4;
  }
  // The exchange's kernel loads the rate ahead in small launches and in large ones (128x128x96 FP16 22.5 us a step
  // and 24.7 at its use), but at its use between 4 and 9 blocks per CU, in every storage type (64x64x128 FP16 9.9
  // ahead and 9.1, 128x108x20 FP32 9.7 and 8.5), and so it does where there is no rate, from fewer blocks on
  // (128x128x20 implicit 10.4 and 8.4, 64x64x48 const 6.3 and 6.1; 64x64x16 4.4 and 4.8). The lines are measured:
  // registers (87 and 90) and blocks per CU (5) are the same either way.
  const bool lagged = V.kind == 1 || V.kind == 2;
  const unsigned blocks = L.grid.x * L.grid.y * L.grid.z;
  r.late = r.mode == 2 && blocks > (lagged ? 1024 : 640) && blocks <= (r.blocks ? r.blocks * 256u : 2304);
  return r;
}

template <typename S, bool CORR>
static void launch_step_c(bool walls, const Launch& L, hipStream_t st, const Geo& G, const ModelF& M, const ViscF& V,
                          const ForceF& Fo, const StepIO& io) {
  const StepRoute route = route_of(sizeof(S), L, G, V, Fo);
  if (route.mode == 3) {
    const Launch R = packed_launch(G);
    StepIO pio = io;
    pio.stream = packed_stream(G, Q, sizeof(S));
    // FP32 streaming blocks of four waves: 3 per CU (250^3 429 us against 445, 200^3 214 against 224;
    // three-wave blocks lose, 171x200x200 187 against 207, and so does FP16, 128 against 166)
    const unsigned threads = R.block.x * R.block.y;
    const size_t cap = (sizeof(S) == 4 && pio.stream && threads > 192 && threads <= 256) ? lds_cap_bytes(3, 0) : 0;
    const size_t chunk = std::max(packed_lds_bytes<Q, S>(R.block.x, R.block.y), cap);
    if (walls) hipLaunchKernelGGL((step_kernel<S, true, 3, CORR>), R.grid, R.block, chunk, st, G, M, V, Fo, pio);
    else hipLaunchKernelGGL((step_kernel<S, false, 3, CORR>), R.grid, R.block, chunk, st, G, M, V, Fo, pio);
    return;
  }
  const size_t lds = lds_cap_bytes(route.blocks, route.mode == 2 ? staged_lds_bytes<Lat>() : 0);
  switch (route.mode + (walls ? 3 : 0)) {
    case 0: hipLaunchKernelGGL((step_kernel<S, false, 0, CORR>), L.grid, L.block, lds, st, G, M, V, Fo, io); break;
    case 1: hipLaunchKernelGGL((step_kernel<S, false, 1, CORR>), L.grid, L.block, lds, st, G, M, V, Fo, io); break;
    case 2: {
      const auto k = route.late ? step_kernel<S, false, 4, CORR> : step_kernel<S, false, 2, CORR>;
      hipLaunchKernelGGL(k, L.grid, L.block, lds, st, G, M, V, Fo, io);
      break;
    }
    case 3: hipLaunchKernelGGL((step_kernel<S, true, 0, CORR>), L.grid, L.block, lds, st, G, M, V, Fo, io); break;
    case 4: hipLaunchKernelGGL((step_kernel<S, true, 1, CORR>), L.grid, L.block, lds, st, G, M, V, Fo, io); break;
    default: {
      const auto k = route.late ? step_kernel<S, true, 4, CORR> : step_kernel<S, true, 2, CORR>;
      hipLaunchKernelGGL(k, L.grid, L.block, lds, st, G, M, V, Fo, io);
    }
  }
}

template <typename S>
static void launch_step_t(bool walls, const Launch& L, hipStream_t st, const Geo& G, const ModelF& M, const ViscF& V,
                          const ForceF& Fo, const StepIO& io) {
  if (Fo.strain_corr) launch_step_c<S, true>(walls, L, st, G, M, V, Fo, io);
  else launch_step_c<S, false>(walls, L, st, G, M, V, Fo, io);
}

static Launch step_launch(int storage, const Geo& G) {
  Launch L = node_launch(G);
  // 16-bit storage: part-row blocks hold one row segment (128 x 1 ran 1 % faster than 128 x 2
  // in FP16 and BF16 at 384^3, while FP32 runs 3 % faster with two rows)
  if (storage != 0 && pull_mode(G, L.block) == 0 && L.block.y > 1) {
    L.block.y = 1;
    L.grid.y = G.ny;
  }
  return L;
}

StepRoute step_route(int storage, const Geo& G, const ViscF& V, const ForceF& Fo) {
  return route_of(storage == 0 ? 4 : 2, step_launch(storage, G), G, V, Fo);
}

hipError_t launch_step(int storage, const Geo& G, const ModelF& M, const ViscF& V, const ForceF& Fo, const StepIO& io,
                       hipStream_t st) {
  const Launch L = step_launch(storage, G);
  switch (storage) {
    case 0: launch_step_t<float>(G.walls != 0, L, st, G, M, V, Fo, io); break;
    case 1: launch_step_t<_Float16>(G.walls != 0, L, st, G, M, V, Fo, io); break;
    case 2: launch_step_t<__bf16>(G.walls != 0, L, st, G, M, V, Fo, io); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace d3q19
}  // namespace lbm
