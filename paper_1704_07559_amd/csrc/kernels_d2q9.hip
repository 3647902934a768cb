// D2Q9 kernels: the same fused pull-stream / collide / strain step as D3Q19 on the
// nine-velocity lattice (Sections 5.3 and 5.4 of the paper), plus initial state, strain
// query, canonical gather/scatter and the diagnostics reduction. One thread per node.
#include <hip/hip_runtime.h>

#include <algorithm>

// Contraction of a product and a sum into an FMA only within one expression of the source
// (for this file and the headers it includes): left to the code generator, which product of
// a sum gets fused depends on the code around it, and the two-step kernel below must round
// every operation as the single step does.
#pragma clang fp contract(on)

#include "d2q9.h"
#include "internal.h"
#include "launch.h"
#include "reduce.h"

namespace lbm {
namespace d2q9 {

__device__ __forceinline__ void load_force(const ForceF& Fo, unsigned N, unsigned self, float& Fx, float& Fy) {
  if (Fo.mode == 1) {
    Fx = Fo.F[0];
    Fy = Fo.F[1];
  } else if (Fo.mode == 2) {
    Fx = Fo.field[self];
    Fy = Fo.field[N + self];
  } else {
    Fx = Fy = 0.0f;
  }
}

__device__ __forceinline__ void rates_with(const ModelF& M, float snu, float (&r)[Q]) {
  static_for<Q>([&](auto ki) {
    constexpr int k = ki;
    r[k] = is_nu_slot(k) ? snu : M.s[k];
  });
}

// S:S (the off-diagonal component counts twice) in one fixed order of operations. Written as
// plain products and sums, the compiler may fuse either product of a sum into an FMA, and
// which one it picks depends on the code around it, so the same strain could round to two
// different rates in two kernels; the two-step kernel must round exactly as the single step.
__device__ __forceinline__ float strain_sq(const float (&S)[3]) {
  return __builtin_fmaf(S[0], S[0], __builtin_fmaf(S[1], S[1], 2.0f * S[2] * S[2]));
}

// The force-corrected strain (optional) takes the non-equilibrium part plus half the Guo
// source, m - m^eq + S_F/2. StrainIn holds the moments the Yu-type formula reads (ns) and,
// with CORR, h = S_F/2, which the Chai formula adds as the Yu-type contraction of h with the
// same rates (the Chai contraction of F-bar/2 in moment space). Without CORR only the plain
// moments are held.
template <bool CORR>
struct StrainIn {
  Neq ns;
  Neq h;
};

template <bool CORR>
__device__ __forceinline__ StrainIn<CORR> strain_in(const Neq& n, const float (&SF)[Q]) {
  StrainIn<CORR> si;
  if constexpr (CORR) {
    static_for<Q>([&](auto ki) {
      constexpr int k = ki;
      si.h.m[k] = 0.5f * SF[k];
      si.ns.m[k] = n.m[k] + si.h.m[k];
    });
  } else {
    si.ns = n;
  }
  return si;
}

// The read-only kernels take the corrected form always, with a zero source when the
// correction is off.
__device__ __forceinline__ StrainIn<true> strain_in_state(const Neq& n, float jx, float jy, float Fx, float Fy,
                                                          const ModelF& M, const ForceF& Fo) {
  float SF[Q];
  if (Fo.strain_corr) {
    force_moments(jx, jy, Fx, Fy, M.inv_rho0, SF);
  } else {
#pragma unroll
    for (int k = 0; k < Q; ++k) SF[k] = 0.0f;
  }
  return strain_in<true>(n, SF);
}

template <bool CORR>
__device__ __forceinline__ void strain_chai_in(const Pairs& P, float drho, float jx, float jy, const float (&rates)[Q],
                                               const StrainIn<CORR>& si, float inv_rho0, float (&S)[3]) {
  strain_chai(P, drho, jx, jy, rates, inv_rho0, S);
  if constexpr (CORR) {
    float Sh[3];
    strain_yu(si.h, rates[1], rates[7], inv_rho0, Sh);
#pragma unroll
    for (int c = 0; c < 3; ++c) S[c] += Sh[c];
  }
}

// s_nu of the implicit Smagorinsky coupling at one node, from the formula V selects (both
// are affine in s_nu: split into the part at the other rates and the s_nu rows).
template <bool CORR>
__device__ __forceinline__ float implicit_rate(const Pairs& P_, float drho, float jx, float jy,
                                               const StrainIn<CORR>& si, const ModelF& M, const ViscF& V) {
  float P[3], A[3];
  if (V.drive_chai) {
    float rb[Q], rn[Q];
    rates_with(M, 0.0f, rb);
    static_for<Q>([&](auto ki) {
      constexpr int k = ki;
      rn[k] = is_nu_slot(k) ? 1.0f : 0.0f;
    });
    strain_chai_in(P_, drho, jx, jy, rb, si, M.inv_rho0, P);
    strain_chai_in(P_, drho, jx, jy, rn, si, M.inv_rho0, A);
  } else {
    strain_yu(si.ns, M.s[1], 0.0f, M.inv_rho0, P);
    strain_yu(si.ns, 0.0f, 1.0f, M.inv_rho0, A);
  }
  return implicit_smagorinsky(P, A, V.nu0, V.csmag2);
}

// One node's collision with its strain and viscosity (Eq. mrteq's right side with the rates
// of Eq. mrteqvT; the strain of Section 5.3, or the Yu-type formula of Section 5.4): g holds
// the pulled populations on entry and the post-collision ones on return. lagged() gives the
// node's lagged rate (read only where the lagged coupling needs it), store_lagged(s) keeps
// the rate a lagged viscosity law derived for the next step. (Fx, Fy): the node's force
// (load_force). S_out / emit: the optional strain output (emit 1 Yu, 2 Chai). Returns the
// rate of s_nu's rows this collision used.
template <bool CORR, class Lagged, class StoreLagged>
__device__ __forceinline__ float collide(const Geo& G, const ModelF& M, const ViscF& V, const ForceF& Fo,
                                         unsigned self, Lagged lagged, StoreLagged store_lagged, float Fx, float Fy,
                                         float* S_out, int emit, float (&g)[Q]) {
  const Pairs P = make_pairs(g);
  const float drho = delta_rho(P);
  float jx = momentum<0>(P), jy = momentum<1>(P);
  if (Fo.mode) {
    jx = __builtin_fmaf(0.5f, Fx, jx);
    jy = __builtin_fmaf(0.5f, Fy, jy);
  }
  const Neq n = noneq_moments(P, drho, jx, jy, M.inv_rho0);
  // the Guo source in moment space; with CORR formed before the strain (half of it joins the
  // non-equilibrium part the strain takes)
  float SF[Q];
  if constexpr (CORR) force_moments(jx, jy, Fx, Fy, M.inv_rho0, SF);
  const StrainIn<CORR> si = strain_in<CORR>(n, SF);
  float Syu[3], Sch[3];
  float snu = M.s[7];
  if (V.kind == 3) {
    // implicit coupling: the strain at the rate of this very collision
    snu = implicit_rate(P, drho, jx, jy, si, M, V);
    if (S_out) {
      if (emit == 2) {
        float r[Q];
        rates_with(M, snu, r);
        strain_chai_in(P, drho, jx, jy, r, si, M.inv_rho0, Sch);
      } else {
        strain_yu(si.ns, M.s[1], snu, M.inv_rho0, Syu);
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) stream_store(&S_out[static_cast<size_t>(c) * G.N + self], emit == 2 ? Sch[c] : Syu[c]);
    }
  } else {
    // lagged coupling: the strain of the incoming state with the rates of the previous collision
    const float snu_prev = lagged();
    const bool need_yu = emit == 1 || (V.kind != 0 && !V.drive_chai);
    const bool need_chai = emit == 2 || (V.kind != 0 && V.drive_chai);
    if (need_yu) strain_yu(si.ns, M.s[1], snu_prev, M.inv_rho0, Syu);
    if (need_chai) {
      float r[Q];
      rates_with(M, snu_prev, r);
      strain_chai_in(P, drho, jx, jy, r, si, M.inv_rho0, Sch);
    }
    if (S_out) {
#pragma unroll
      for (int c = 0; c < 3; ++c) stream_store(&S_out[static_cast<size_t>(c) * G.N + self], emit == 2 ? Sch[c] : Syu[c]);
    }
    if (V.kind != 0) {
      snu = viscous_rate(V.drive_chai ? strain_sq(Sch) : strain_sq(Syu), V);
      store_lagged(snu);
    }
  }
  float dm[Q];
  dm[0] = 0.0f;
  dm[3] = Fx;
  dm[5] = Fy;
  static_for<Q>([&](auto ki) {
    constexpr int k = ki;
    if constexpr (k != 0 && k != 3 && k != 5) dm[k] = -(is_nu_slot(k) ? snu : M.s[k]) * n.m[k];
  });
  if (Fo.mode) {
    if constexpr (!CORR) force_moments(jx, jy, Fx, Fy, M.inv_rho0, SF);
    static_for<Q>([&](auto ki) {
      constexpr int k = ki;
      if constexpr (k != 0 && k != 3 && k != 5) {
        const float sk = is_nu_slot(k) ? snu : M.s[k];
        dm[k] = __builtin_fmaf(1.0f - 0.5f * sk, SF[k], dm[k]);
      }
    });
  }
  add_back_transform(dm, g);
  return snu;
}

// XMODE: how a block pulls along x (pull_mode: 0 part rows, 1 whole rows, 2 whole rows with
// the LDS exchange). CORR: the force-corrected strain (a separate instance, so that the plain
// step keeps its register budget).
template <typename S, bool WALLS, int XMODE, bool CORR>
__global__ __launch_bounds__(kMaxBlock) void step_kernel(Geo G, ModelF M, ViscF V, ForceF Fo, StepIO io) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y * blockDim.y + threadIdx.y;
  if (x >= G.nx || y >= G.ny) return;
  const unsigned self = node_index(G, x, y, 0);
  const Rows<Q, S> r = rows_of<Q, S>(G, x, y, 0);
  // The rate is loaded ahead of the populations, its latency hidden behind theirs (us a step ahead and at its use:
  // FP16 64x16384 9.4 and 10.2, FP32 184x712 4.3 and 4.5, power law 1161x3328 57.8 and 61.3), but not in FP32
  // boxes whose buffers fill the L2s (100x3932 9.1 and 7.4, 3000x349 power law 5 % more ahead).
  const bool ahead = sizeof(S) == 2 || G.N < (11u << 14) || G.N >= (3u << 19);
  const float snu_prev = ahead && io.snu ? io.snu[self] : M.s[7];
  float g[Q];
  if constexpr (XMODE == 2) pull_rows_staged<Lat, S, WALLS>(static_cast<const S*>(io.src), G, r, y, g);
  else pull_rows<Lat, S, WALLS, XMODE == 1>(static_cast<const S*>(io.src), G, r, y, g);
  float Fx, Fy;
  load_force(Fo, G.N, self, Fx, Fy);
  collide<CORR>(
      G, M, V, Fo, self, [&] { return ahead || !io.snu ? snu_prev : io.snu[self]; },
      [&](float s) { io.snu[self] = s; }, Fx, Fy, io.S_out, io.emit, g);
  store_rows<Q>(static_cast<S*>(io.dst), G, r, g);
}

// Two steps per launch: the
// result is that of two launches of step_kernel, bit for bit, for the algorithmic HBM
// traffic of one (the rows at block edges are read twice).
// A block of B lanes owns a strip of B - 2 columns (lane l at column x0 - 1 + l, the two edge
// lanes a ring column on either side, wrapped periodically) and R rows of the result, and walks
// its rows upwards. At row t it pulls the incoming state from HBM and
// collides it (level 1, rounded to the storage type as a store would round it); the
// populations a neighbouring lane pulls at level 2 (c_x != 0) go to an LDS ring of rows,
// those the lane itself pulls (c_x = 0) stay in registers. After one barrier it pulls row
// t - 1 of level 1 (from rows t - 2, t - 1 and t), collides it again and stores it. The ring
// is deep enough that one barrier per row suffices: the slot written at row t + 1 is none of
// those read at row t. Level 1 is computed for the two ring columns and for
// one extra row below and above the block's rows, as the neighbouring blocks compute them
// too: B / (B - 2) more columns and (R + 2) / R more rows of level-1 work.
// The lagged rate s_nu cannot be updated in place (a neighbour still reads the old value of
// a ring node after this block has passed it), so it is read from snu_in and written to
// snu_out.
//
// Rows per block (pair_rows): fewer rows mean more level-1 rows computed twice, more rows fewer
// blocks to overlap one another's barriers and memory waits, and a longer chain of rows (about
// 2 us each) where the blocks do not fill the chip. Large boxes, 4096^2: FP32 160 us per step
// at 6 rows, 176 at 2, 163 at 8 and 162 at 12; FP16 111 at 12, 116 at 6, 143 at 2. Below 1280
// blocks of 256 lanes (5 per CU; 2560 of 128) every row fewer wins: 600 x 201 between walls 5.0 us per
// step at 1 row, 5.7 at 2, 8.7 at 6; 256^2 4.4, 5.0, 8.4; 1024^2 FP32 18.3 at 1, 13.6 at 4 (1280 blocks), 14.5
// at 6, FP16 15.5, 11.0, 12.1 and 16.3 at 12; 100 x 3000 (128 lanes) 6.3 at 1, 6.1 at 2, 6.4 at 3.
template <typename S>
constexpr int kPairMaxRows = sizeof(S) == 4 ? 6 : 12;
template <typename S>
inline int pair_rows(int strips, int ny, int B) {
  const long long all = static_cast<long long>(strips) * ny, fill = 1280 * 256 / B;
  const long long r = (all + fill - 1) / fill;
  return r < kPairMaxRows<S> ? static_cast<int>(r) : kPairMaxRows<S>;
}

// Lanes per block: 256, or 128 where that leaves at least a quarter fewer lanes without a column
// (rows up to 126 nodes, or 300 to 378): wide rows favour 256 (4096^2 160 us per step against 181,
// the strips' ends being partial lines), 100^2 takes 3.4 us either way.
constexpr int pair_strips(int nx, int B) { return (nx + B - 3) / (B - 2); }
inline int pair_lanes(int nx) { return 4 * 128 * pair_strips(nx, 128) <= 3 * 256 * pair_strips(nx, 256) ? 128 : 256; }

// LDS ring rows of the x-shifted populations: one with c_y = -1 is read in the row it was
// written (2 slots: a fast thread writes the next row while a slow one still reads this one),
// the others one or two rows later (4 slots); ring_row(i) is population i's first slot. With
// walls a population is also read one row later as the opposite of one that bounces back:
// 4 slots for all.
template <bool WALLS>
constexpr int ring_rows(int i) { return Lat::cx(i) == 0 ? 0 : (Lat::cy(i) < 0 && !WALLS ? 2 : 4); }
template <bool WALLS>
constexpr int ring_row(int i) { return i == 0 ? 0 : ring_row<WALLS>(i - 1) + ring_rows<WALLS>(i - 1); }

// WALLS: halfway bounce-back at y = -1/2 and ny - 1/2 (no wrap in y; level 1 is not computed
// for the rows beyond the walls, and a population of level 2 that crosses a wall is the
// opposite one of the node's own level-1 state). CORR: the force-corrected strain.
// EMIT: the strain output S_out (emit 1 Yu, 2 Chai), taken at level 2 only (the strain of
// the second step's incoming state, which single steps leave in S_out last); a template
// parameter, as its code costs the instances without it 15 VGPRs otherwise.
template <typename S, int B, bool WALLS, bool CORR, bool EMIT>
__global__ __launch_bounds__(B) void pair_kernel(Geo G, int R, ModelF M, ViscF V, ForceF Fo,
                                                 const S* __restrict__ src, S* __restrict__ dst,
                                                 const float* snu_in, float* snu_out, float* S_out, int emit) {
  // (in the storage type: level 1 is rounded to it anyway, and 16-bit rows halve the LDS)
  __shared__ S ring[ring_row<WALLS>(Q)][B];
  const int lane = threadIdx.x;
  const int x0 = blockIdx.x * (B - 2);
  const int xl = x0 - 1 + lane;  // this lane's column, unwrapped
  // (lanes past the ring column of a ragged last strip compute level 1 of a column no one reads,
  // so that every lane takes the same path through level 1)
  int x = xl < 0 ? xl + G.nx : (xl >= G.nx ? xl - G.nx : xl);
  if (x >= G.nx) x = 0;
  const bool kept = lane >= 1 && lane <= B - 2 && xl < G.nx;  // level 2 owned here
  const int y0 = blockIdx.y * R;
  const int rows = min(R, G.ny - y0);
  // The rate is loaded ahead of the populations, its latency hidden behind theirs (1024^2 FP32 13.0 us
  // per step against 13.5, 600 x 201 4.6 against 5.0, 4096^2 FP16 106 against 111), except in FP32
  // blocks of the full number of rows, which it costs 1 % (4096^2 161.6 us against 160.2).
  const bool ahead = sizeof(S) == 2 || R < kPairMaxRows<S>;
  // level-1 values of the c_x = 0 populations this lane pulls back one and two rows later
  float prev[Q], prev2[Q], snu_prev = 0.0f;
  constexpr auto slot = [](int i, int row) { return ring_row<WALLS>(i) + (row & (ring_rows<WALLS>(i) - 1)); };
  for (int k = 0; k < rows + 2; ++k) {
    int t = y0 - 1 + k;
    float g[Q], snu1 = 0.0f;
    if (!WALLS) t = t < 0 ? t + G.ny : (t >= G.ny ? t - G.ny : t);
    if (!WALLS || (t >= 0 && t < G.ny)) {  // (uniform over the block)
      const unsigned self1 = node_index(G, x, t, 0);
      const float snu0 = ahead && snu_in ? snu_in[self1] : M.s[7];
      pull_rows<Lat, S, WALLS, false>(src, G, rows_of<Q, S>(G, x, t, 0), t, g);
      float Fx, Fy;
      load_force(Fo, G.N, self1, Fx, Fy);
      snu1 = collide<CORR>(
          G, M, V, Fo, self1, [&] { return ahead || !snu_in ? snu0 : snu_in[self1]; }, [](float) {}, Fx, Fy,
          nullptr, 0, g);
      static_for<Q>([&](auto ii) {
        constexpr int i = ii;
        if constexpr (sizeof(S) == 2) g[i] = static_cast<float>(static_cast<S>(g[i]));
        // opaque: no operation of level 2 may be fused with the last one of level 1
        asm volatile("" : "+v"(g[i]));
        if constexpr (Lat::cx(i) != 0) ring[slot(i, k)][lane] = static_cast<S>(g[i]);
      });
      asm volatile("" : "+v"(snu1));
    } else {
      static_for<Q>([&](auto ii) { g[ii] = 0.0f; });  // a row beyond a wall: never pulled
    }
    __syncthreads();
    if (k >= 2 && kept) {
      const int y = y0 + k - 2;
      float h[Q];
      static_for<Q>([&](auto ii) {
        constexpr int i = ii;
        constexpr int cx = Lat::cx(i), cy = Lat::cy(i), o = Lat::opp(i);
        float v;
        if constexpr (cx != 0) v = static_cast<float>(ring[slot(i, k - 1 - cy)][lane - cx]);
        else if constexpr (cy == 0) v = prev[i];
        else if constexpr (cy > 0) v = prev2[i];
        else v = g[i];
        if constexpr (WALLS && cy != 0) {
          // bounce-back: the opposite population of this node's own level-1 state (row k - 1)
          float b;
          if constexpr (Lat::cx(o) != 0) b = static_cast<float>(ring[slot(o, k - 1)][lane]);
          else b = prev[o];
          if (crosses_wall<cy>(G, y)) v = b;
        }
        h[i] = v;
      });
      const unsigned self = node_index(G, x, y, 0);
      float Fx, Fy;
      load_force(Fo, G.N, self, Fx, Fy);
      collide<CORR>(
          G, M, V, Fo, self, [&] { return snu_prev; }, [&](float s) { snu_out[self] = s; }, Fx, Fy,
          EMIT ? S_out : nullptr, EMIT ? emit : 0, h);
      store_rows<Q>(dst, G, rows_of<Q, S>(G, x, y, 0), h);
    }
    static_for<Q>([&](auto ii) {
      constexpr int i = ii;
      if constexpr (Lat::cx(i) == 0) {
        prev2[i] = prev[i];
        prev[i] = g[i];
      }
    });
    snu_prev = snu1;
  }
}

// CACHED: the loads go through the caches (cached_strain); STREAM: streaming stores (plane_stream).
template <typename S, bool CACHED, bool STREAM>
__global__ __launch_bounds__(kMaxBlock) void strain_kernel(Geo G, ModelF M, ViscF V, ForceF Fo, const S* buf,
                                                           const float* snu_f, int kind, float* S_out) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y * blockDim.y + threadIdx.y;
  if (x >= G.nx || y >= G.ny) return;
  const Node<Q, S> nb = node_at<Q, S>(G, x, y, 0);
  float g[Q];
  pull_rows<Lat, S, true, true, CACHED>(buf, G, nb.rows, y, g);
  const Pairs P = make_pairs(g);
  const float drho = delta_rho(P);
  float Fx, Fy;
  load_force(Fo, G.N, nb.self, Fx, Fy);
  const float jx = momentum<0>(P) + 0.5f * Fx, jy = momentum<1>(P) + 0.5f * Fy;
  const Neq n = noneq_moments(P, drho, jx, jy, M.inv_rho0);
  const StrainIn<true> si = strain_in_state(n, jx, jy, Fx, Fy, M, Fo);
  const float snu = V.kind == 3 ? implicit_rate(P, drho, jx, jy, si, M, V) : (snu_f ? snu_f[nb.self] : M.s[7]);
  float S3[3];
  if (kind == 2) {
    float r[Q];
    rates_with(M, snu, r);
    strain_chai_in(P, drho, jx, jy, r, si, M.inv_rho0, S3);
  } else {
    strain_yu(si.ns, M.s[1], snu, M.inv_rho0, S3);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) plane_store<STREAM>(&S_out[static_cast<size_t>(c) * G.N + nb.self], S3[c]);
}

template <typename S>
__global__ __launch_bounds__(kMaxBlock) void init_kernel(Geo G, ModelF M, S* buf, float* snu, const float* rho_u,
                                                   const float* grad_u) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y * blockDim.y + threadIdx.y;
  if (x >= G.nx || y >= G.ny) return;
  const Node<Q, S> nb = node_at<Q, S>(G, x, y, 0);
  const unsigned self = nb.self;
  float drho = 0.f, ux = 0.f, uy = 0.f;
  if (rho_u) {
    drho = rho_u[self];
    ux = rho_u[G.N + self];
    uy = rho_u[2 * static_cast<size_t>(G.N) + self];
  }
  float g[Q];
  equilibrium(drho, M.rho0 * ux, M.rho0 * uy, M.inv_rho0, g);
  if (grad_u) {
    // d[a*3+b] = d j_b / d x_a; inverse of the Yu-type formula (Chapman-Enskog state).
    const size_t N = G.N;
    const float dxx = M.rho0 * grad_u[0 * N + self], dxy = M.rho0 * grad_u[1 * N + self];
    const float dyx = M.rho0 * grad_u[3 * N + self], dyy = M.rho0 * grad_u[4 * N + self];
    const float sn = M.s[7];
    float mn[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) mn[k] = 0.0f;
    mn[1] = -2.0f * (dxx + dyy) / M.s[1];
    mn[7] = -2.0f * (dxx - dyy) / (3.0f * sn);
    mn[8] = -(dxy + dyx) / (3.0f * sn);
    add_back_transform(mn, g);
  }
  scatter_rows<Lat, S>(buf, G, nb.rows, y, g);
  if (snu) snu[self] = M.s[7];
}

// CACHED: loads and stores through the caches (cached_get).
template <typename S, bool CACHED>
__global__ __launch_bounds__(kMaxBlock) void get_kernel(Geo G, const S* buf, float* canon) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y * blockDim.y + threadIdx.y;
  if (x >= G.nx || y >= G.ny) return;
  const Node<Q, S> nb = node_at<Q, S>(G, x, y, 0);
  float g[Q];
  pull_rows<Lat, S, true, true, CACHED>(buf, G, nb.rows, y, g);
  store_local<Q, !CACHED>(canon, G, nb.self * 4u, g);
}

template <typename S>
__global__ __launch_bounds__(kMaxBlock) void set_kernel(Geo G, S* buf, const float* canon) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y * blockDim.y + threadIdx.y;
  if (x >= G.nx || y >= G.ny) return;
  const Node<Q, S> nb = node_at<Q, S>(G, x, y, 0);
  float g[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) g[i] = canon[static_cast<size_t>(i) * G.N + nb.self];
  scatter_rows<Lat, S>(buf, G, nb.rows, y, g);
}

// ROWS: blocks take whole rows in turn instead of nodes in their order in memory (reduce_by_rows).
template <typename S, bool CORR, bool IMPLICIT, bool ROWS>
__global__ __launch_bounds__(256) void reduce_kernel(Geo G, ModelF M, ViscF V, ForceF Fo, NodeWalk W, const S* buf,
                                                     const float* snu_f, double* partials) {
  double acc[kReduceVals] = {0, 0, 0, 0, 0, 0, 0, 0};
  const double per_jj = 0.5 / M.rho0;
  const auto add = [&](unsigned self, int x, int y) {
    // (loaded ahead of the populations: behind them its latency would stand alone)
    float snu = (!IMPLICIT && snu_f) ? snu_f[self] : M.s[7];
    float g[Q];
    pull_rows<Lat, S, true, ROWS>(buf, G, rows_of<Q, S>(G, x, y, 0), y, g);
    const Pairs P = make_pairs(g);
    const float drho = delta_rho(P);
    // (their sum is non-finite where a population is, so that finite nodes pay one test)
    if (!isfinite(drho)) {
      int bad = 0;
#pragma unroll
      for (int i = 0; i < Q; ++i) bad += !isfinite(g[i]);
      acc[7] += bad;
    }
    float Fx, Fy;
    load_force(Fo, G.N, self, Fx, Fy);
    const float jx = momentum<0>(P) + 0.5f * Fx, jy = momentum<1>(P) + 0.5f * Fy;
    const Neq n = noneq_moments(P, drho, jx, jy, M.inv_rho0);
    float SF[Q];
    if constexpr (CORR) force_moments(jx, jy, Fx, Fy, M.inv_rho0, SF);
    const StrainIn<CORR> si = strain_in<CORR>(n, SF);
    if constexpr (IMPLICIT) snu = implicit_rate(P, drho, jx, jy, si, M, V);
    float S3[3];
    strain_yu(si.ns, M.s[1], snu, M.inv_rho0, S3);
    const double jj = static_cast<double>(jx) * jx + static_cast<double>(jy) * jy;
    acc[0] += drho;
    acc[1] += jx;
    acc[2] += jy;
    acc[4] += jj * per_jj;
    acc[5] += static_cast<double>(S3[0]) * S3[0] + static_cast<double>(S3[1]) * S3[1] +
              2.0 * static_cast<double>(S3[2]) * S3[2];
    acc[6] = fmax(acc[6], jj);  // max |j|^2: the final pass takes sqrt(.) / rho0 once
  };
  if constexpr (ROWS) {
    for (int y = blockIdx.x; y < G.ny; y += gridDim.x)
      for (int x = threadIdx.x; x < G.nx; x += 256) add(node_index(G, x, y, 0), x, y);
  } else {
    for (unsigned self = blockIdx.x * 256 + threadIdx.x; self < G.N; self += gridDim.x * 256) {
      const Coord c = coord_of(G, W, self);
      add(self, c.x, c.y);
    }
  }
  block_reduce_store(acc, partials);
}

template <typename S>
static const S* cb(const void* p) {
  return static_cast<const S*>(p);
}

template <typename S, bool CORR>
static void launch_step_c(bool walls, const Launch& L, hipStream_t st, const Geo& G, const ModelF& M, const ViscF& V,
                          const ForceF& Fo, const StepIO& io) {
  switch (pull_mode(G, L.block) + (walls ? 3 : 0)) {
    case 0: hipLaunchKernelGGL((step_kernel<S, false, 0, CORR>), L.grid, L.block, 0, st, G, M, V, Fo, io); break;
    case 1: hipLaunchKernelGGL((step_kernel<S, false, 1, CORR>), L.grid, L.block, 0, st, G, M, V, Fo, io); break;
    case 2: hipLaunchKernelGGL((step_kernel<S, false, 2, CORR>), L.grid, L.block, 0, st, G, M, V, Fo, io); break;
    case 3: hipLaunchKernelGGL((step_kernel<S, true, 0, CORR>), L.grid, L.block, 0, st, G, M, V, Fo, io); break;
    case 4: hipLaunchKernelGGL((step_kernel<S, true, 1, CORR>), L.grid, L.block, 0, st, G, M, V, Fo, io); break;
    default: hipLaunchKernelGGL((step_kernel<S, true, 2, CORR>), L.grid, L.block, 0, st, G, M, V, Fo, io); break;
  }
}

template <typename S>
static void launch_step_t(bool walls, const Launch& L, hipStream_t st, const Geo& G, const ModelF& M, const ViscF& V,
                          const ForceF& Fo, const StepIO& io) {
  if (Fo.strain_corr) launch_step_c<S, true>(walls, L, st, G, M, V, Fo, io);
  else launch_step_c<S, false>(walls, L, st, G, M, V, Fo, io);
}

hipError_t launch_step(int storage, const Geo& G, const ModelF& M, const ViscF& V, const ForceF& Fo, const StepIO& io,
                       hipStream_t st) {
  const Launch L = node_launch(G);
  switch (storage) {
    case 0: launch_step_t<float>(G.walls != 0, L, st, G, M, V, Fo, io); break;
    case 1: launch_step_t<_Float16>(G.walls != 0, L, st, G, M, V, Fo, io); break;
    case 2: launch_step_t<__bf16>(G.walls != 0, L, st, G, M, V, Fo, io); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename S, int B>
static void launch_pair_b(const PairPlan& P, hipStream_t st, const Geo& G, const ModelF& M, const ViscF& V,
                          const ForceF& Fo, const void* src, void* dst, const float* snu_in, float* snu_out,
                          float* S_out, int emit) {
  decltype(&pair_kernel<S, B, false, false, false>) k;
  switch ((G.walls ? 1 : 0) + (Fo.strain_corr ? 2 : 0) + (S_out ? 4 : 0)) {
    case 0: k = pair_kernel<S, B, false, false, false>; break;
    case 1: k = pair_kernel<S, B, true, false, false>; break;
    case 2: k = pair_kernel<S, B, false, true, false>; break;
    case 3: k = pair_kernel<S, B, true, true, false>; break;
    case 4: k = pair_kernel<S, B, false, false, true>; break;
    case 5: k = pair_kernel<S, B, true, false, true>; break;
    case 6: k = pair_kernel<S, B, false, true, true>; break;
    default: k = pair_kernel<S, B, true, true, true>; break;
  }
  hipLaunchKernelGGL(k, dim3(P.tx, P.ty, 1), dim3(B), 0, st, G, P.rows, M, V, Fo, cb<S>(src), static_cast<S*>(dst),
                     snu_in, snu_out, S_out, emit);
}

template <typename S>
static void launch_pair_s(const PairPlan& P, hipStream_t st, const Geo& G, const ModelF& M, const ViscF& V,
                          const ForceF& Fo, const void* src, void* dst, const float* snu_in, float* snu_out,
                          float* S_out, int emit) {
  if (P.threads == 128) launch_pair_b<S, 128>(P, st, G, M, V, Fo, src, dst, snu_in, snu_out, S_out, emit);
  else launch_pair_b<S, 256>(P, st, G, M, V, Fo, src, dst, snu_in, snu_out, S_out, emit);
}

// Whether two steps per launch beat two launches. `filled` is the share of lanes that own a column, `work` the
// level-1 nodes computed per node of the result; us per step below are single steps and pairs.
// Up to 2^14 nodes (2^15 where half of the lanes are filled) both are a launch's latency (64x64 3.3 and 3.1).
// Beyond, lanes without a column cost as much as the others (16x65536 18.6 and 34.9, 48x21845 15.9 and 19.6;
// 64x16384, half filled, 14.7 and 14.2), and so do rows computed twice, most in boxes of one row per block,
// whose single steps run out of the L2s (128x1024 3.8 and 4.5, 256x512 4.2 and 4.7, but 250x1048 6.2 and 5.2:
// rows of a multiple of 64 nodes exchange through LDS in a single step, others are half again as slow there;
// 250x16777 66 and 40). A 16-bit step has half the traffic to save (256x4096 12.2 and 14.9, 250x4194 15.6 and
// 11.4), the power law and the implicit rate more arithmetic to do twice (power law FP32 90x11650 20.3 and
// 19.7, 160x6553 17.0 and 20.2, FP16 250x1048 6.5 and 8.6; implicit FP16 64x16384 12.1 and 22.8).
static bool pair_pays(int storage, const Geo& G, const ViscF& V, const PairPlan& P) {
  const double lanes = static_cast<double>(P.threads) * P.tx, filled = G.nx / lanes;
  const double work = (P.rows + 2) / (P.rows * filled);
  const bool whole = G.nx % 64 == 0, wide = G.nx >= 256, half = storage != 0;
  if (V.kind == 2) {
    if (half) return !whole && work <= 1.5 && G.N >= (3u << 21);
    return work <= (runs_aligned(G, 4, 64) ? 1.9 : 2.2);
  }
  // (16-bit rows of 256 nodes and more that are no multiple of 64 are pulled in parts by single steps)
  const bool half_wide = half && wide && !whole && work <= 3.3;
  if (G.N <= (1u << 14)) return true;
  if (half && V.kind == 3) return half_wide || (!whole && work <= 1.5);
  if (G.N <= (1u << 15) && filled >= 0.5) return true;
  if (filled < (V.kind == 0 && !half ? 0.35 : 0.5)) return false;
  if (half) return half_wide || (G.N >= 300000 && work <= (whole ? 1.7 : 3.1));
  if (!wide && G.N < (11u << 14)) return false;
  return work <= (!whole ? 3.9 : V.kind == 3 ? 2.5 : 3.1);
}

// The plan of `cols` (126 or 254) columns and `rows` rows per block, empty where no launch covers the box
// with it (the grid's y extent is at most 65535).
PairPlan pair_tiles(const Geo& G, int cols, int rows) {
  if ((cols != 126 && cols != 254) || rows < 1 || G.nz != 1) return PairPlan{};
  const int strips = pair_strips(G.nx, cols + 2), ty = (G.ny - 1) / rows + 1;
  if (ty > 65535) return PairPlan{};
  return PairPlan{cols, rows, 1, strips, ty, strips * ty, cols + 2};
}

PairPlan pair_plan(int storage, const Geo& G, const ViscF& V) {
  const int B = pair_lanes(G.nx), strips = pair_strips(G.nx, B);
  const int R = storage == 0 ? pair_rows<float>(strips, G.ny, B) : pair_rows<_Float16>(strips, G.ny, B);
  const PairPlan P = pair_tiles(G, B - 2, R);
  return P.planes && pair_pays(storage, G, V, P) ? P : PairPlan{};
}

hipError_t launch_pair(const PairPlan& P, int storage, const Geo& G, const ModelF& M, const ViscF& V,
                       const ForceF& Fo, const void* src, void* dst, const float* snu_in, float* snu_out, float* S_out, int emit,
                       hipStream_t st) {
  if (P.planes != 1 || P.rows < 1 || (P.threads != 128 && P.threads != 256)) return hipErrorInvalidValue;
  if ((V.kind == 1 || V.kind == 2) != (snu_in != nullptr) || (snu_in != nullptr) != (snu_out != nullptr) ||
      (snu_in && snu_in == snu_out))
    return hipErrorInvalidValue;
  switch (storage) {
    case 0: launch_pair_s<float>(P, st, G, M, V, Fo, src, dst, snu_in, snu_out, S_out, emit); break;
    case 1: launch_pair_s<_Float16>(P, st, G, M, V, Fo, src, dst, snu_in, snu_out, S_out, emit); break;
    case 2: launch_pair_s<__bf16>(P, st, G, M, V, Fo, src, dst, snu_in, snu_out, S_out, emit); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename S>
static void launch_strain_t(const Launch& L, hipStream_t st, const Geo& G, const ModelF& M, const ViscF& V,
                            const ForceF& Fo, const void* buf, const float* snu, int kind, float* S_out) {
  // (rows whose runs are aligned are multiples of 8 nodes)
  const auto k = !cached_strain(G, Q, sizeof(S)) ? strain_kernel<S, false, true>
                 : plane_stream(G)               ? strain_kernel<S, true, true>
                                                 : strain_kernel<S, true, false>;
  hipLaunchKernelGGL(k, L.grid, L.block, 0, st, G, M, V, Fo, cb<S>(buf), snu, kind, S_out);
}

hipError_t launch_strain(int storage, const Geo& G, const ModelF& M, const ViscF& V, const ForceF& Fo, const void* buf,
                         const float* snu, int kind, float* S_out, hipStream_t st) {
  const Launch L = node_launch(G);
  switch (storage) {
    case 0: launch_strain_t<float>(L, st, G, M, V, Fo, buf, snu, kind, S_out); break;
    case 1: launch_strain_t<_Float16>(L, st, G, M, V, Fo, buf, snu, kind, S_out); break;
    case 2: launch_strain_t<__bf16>(L, st, G, M, V, Fo, buf, snu, kind, S_out); break;
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
  hipLaunchKernelGGL(k, L.grid, L.block, 0, st, G, cb<S>(buf), canon);
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

// Wide rows that fill their blocks' last 256 nodes and are many enough are taken whole: the division that finds a
// node's coordinates costs more there than a row's end (4096^2 FP16 67.6 us against 77.4, implicit 91 against 109,
// 961x737 FP32 14.0 against 15.5; but 920x4096 FP16 29.8 against 27.1, 4096x520 22.9 against 19.8, 300x10000 30.4
// against 23.5).
static bool reduce_by_rows(const Geo& G) {
  const int lanes = (G.nx + 255) / 256 * 256;
  return G.nx >= 900 && 25 * G.nx >= 23 * lanes && G.ny >= 512 && 5 * G.ny >= G.nx;
}

// The force-corrected strain and the implicit rate are instances of their own: their code costs
// the plain diagnostics 10 VGPRs and a tenth of its instructions.
template <typename S>
static void launch_reduce_t(unsigned nb, hipStream_t st, const Geo& G, const ModelF& M, const ViscF& V,
                            const ForceF& Fo, const S* buf, const float* snu, double* partials) {
  decltype(&reduce_kernel<S, false, false, false>) f;
  switch ((Fo.strain_corr ? 1 : 0) + (V.kind == 3 ? 2 : 0) + (reduce_by_rows(G) ? 4 : 0)) {
    case 0: f = reduce_kernel<S, false, false, false>; break;
    case 1: f = reduce_kernel<S, true, false, false>; break;
    case 2: f = reduce_kernel<S, false, true, false>; break;
    case 3: f = reduce_kernel<S, true, true, false>; break;
    case 4: f = reduce_kernel<S, false, false, true>; break;
    case 5: f = reduce_kernel<S, true, false, true>; break;
    case 6: f = reduce_kernel<S, false, true, true>; break;
    default: f = reduce_kernel<S, true, true, true>; break;
  }
  hipLaunchKernelGGL(f, dim3(nb), dim3(256), 0, st, G, M, V, Fo, node_walk(G), buf, snu, partials);
}

hipError_t launch_reduce(int storage, const Geo& G, const ModelF& M, const ViscF& V, const ForceF& Fo,
                         const void* buf, const float* snu, double* partials, double* out, hipStream_t st) {
  const unsigned nb = reduce_by_rows(G) ? static_cast<unsigned>(std::min(G.ny, kReduceBlocks)) : reduce_blocks(G);
  switch (storage) {
    case 0: launch_reduce_t<float>(nb, st, G, M, V, Fo, cb<float>(buf), snu, partials); break;
    case 1: launch_reduce_t<_Float16>(nb, st, G, M, V, Fo, cb<_Float16>(buf), snu, partials); break;
    case 2: launch_reduce_t<__bf16>(nb, st, G, M, V, Fo, cb<__bf16>(buf), snu, partials); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_reduce_final(partials, static_cast<int>(nb), out, st, static_cast<double>(M.rho0));
}

}  // namespace d2q9
}  // namespace lbm
