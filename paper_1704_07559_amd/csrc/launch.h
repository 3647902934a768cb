// Host-side launchers of the kernels (one translation unit per lattice), called by the C
// ABI, and the sizes of the reductions. Nothing here changes the code of the step kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "internal.h"

namespace lbm {

// Reductions: 8 doubles per block (at most kReduceBlocks blocks over the nodes in memory order),
// then one block folds the partials in a fixed order.
constexpr int kReduceBlocks = 4096;
constexpr int kReduceVals = 8;

// Two steps in one launch: src -> dst, the lagged s_nu field (if any) snu_in -> snu_out (distinct
// buffers). The result equals two launch_step calls bit for bit. The plan (how blocks of `cols` x `rows`
// columns and `planes` planes cover the box) is empty, planes = 0, where single steps are to be taken.
struct PairPlan {
  int cols, rows, planes, tx, ty, tiles, threads;
};

// How a single step is launched: the pull mode (pull_mode, 3 for packed rows), the blocks per CU (0: as many
// as the registers allow), and whether rows exchanged through LDS load the lagged rate at its use.
struct StepRoute {
  int mode, blocks;
  bool late;
};

namespace d3q19 {
StepRoute step_route(int storage, const Geo&, const ViscF&, const ForceF&);
int adjoint_mode(const Geo&, const ViscF&);
hipError_t launch_init(int storage, const Geo&, const ModelF&, void* buf, float* snu, const float* rho_u,
                       const float* grad_u, hipStream_t);
hipError_t launch_step(int storage, const Geo&, const ModelF&, const ViscF&, const ForceF&, const StepIO&,
                       hipStream_t);
hipError_t launch_strain(int storage, const Geo&, const ModelF&, const ViscF&, const ForceF&, const void* buf,
                         const float* snu, int kind, float* S_out, hipStream_t);
hipError_t launch_get(int storage, const Geo&, const void* buf, float* canon, hipStream_t);
hipError_t launch_set(int storage, const Geo&, void* buf, const float* canon, hipStream_t);
hipError_t launch_reduce(int storage, const Geo&, const ModelF&, const ViscF&, const ForceF&, const void* buf,
                         const float* snu, double* partials, double* out, hipStream_t);
// in_rows / out_rows: planes 0..18 of lam_in / lam_out row-interleaved (as the population
// buffers) instead of canonical planes; a multi-step sweep keeps its intermediate states so.
hipError_t launch_adjoint_step(const Geo&, const ModelF&, const ViscF&, const ForceF&, const float* rec,
                               const float* lam_in, float* lam_out, float* grad_force, hipStream_t,
                               bool in_rows = false, bool out_rows = false);
hipError_t launch_loss_seed(int storage, const Geo&, const ModelF&, const ViscF&, const ForceF&, const void* buf,
                            const float* snu, float* lam_out, float* grad_force, double* partials, double* out,
                            hipStream_t);
hipError_t launch_init_adjoint(const Geo&, const ModelF&, const float* rho_u, const float* lam0, float* grad_u0,
                               hipStream_t);
PairPlan pair_plan(int storage, const Geo&, const ViscF&, const ForceF&);
PairPlan pair_tiles(int storage, const Geo&, const ViscF&, const ForceF&, int cols, int rows, int planes);
hipError_t launch_pair(const PairPlan&, const Geo&, const ModelF&, const ViscF&, const void* src, void* dst,
                       const float* snu_in, float* snu_out, hipStream_t);
}  // namespace d3q19

namespace d2q9 {
hipError_t launch_init(int storage, const Geo&, const ModelF&, void* buf, float* snu, const float* rho_u,
                       const float* grad_u, hipStream_t);
hipError_t launch_step(int storage, const Geo&, const ModelF&, const ViscF&, const ForceF&, const StepIO&,
                       hipStream_t);
hipError_t launch_strain(int storage, const Geo&, const ModelF&, const ViscF&, const ForceF&, const void* buf,
                         const float* snu, int kind, float* S_out, hipStream_t);
hipError_t launch_get(int storage, const Geo&, const void* buf, float* canon, hipStream_t);
hipError_t launch_set(int storage, const Geo&, void* buf, const float* canon, hipStream_t);
hipError_t launch_reduce(int storage, const Geo&, const ModelF&, const ViscF&, const ForceF&, const void* buf,
                         const float* snu, double* partials, double* out, hipStream_t);
PairPlan pair_plan(int storage, const Geo&, const ViscF&);
PairPlan pair_tiles(const Geo&, int cols, int rows);
// S_out (or nullptr) receives the strain (emit 1 Yu, 2 Chai) of the second step.
hipError_t launch_pair(const PairPlan&, int storage, const Geo&, const ModelF&, const ViscF&, const ForceF&,
                       const void* src, void* dst, const float* snu_in, float* snu_out, float* S_out, int emit,
                       hipStream_t);
}  // namespace d2q9

namespace d3q15 {
StepRoute step_route(int storage, const Geo&, const ViscF&);
hipError_t launch_init(int storage, const Geo&, const ModelF&, void* buf, float* snu, const float* rho_u,
                       const float* grad_u, hipStream_t);
hipError_t launch_step(int storage, const Geo&, const ModelF&, const ViscF&, const ForceF&, const StepIO&,
                       hipStream_t);
hipError_t launch_strain(int storage, const Geo&, const ModelF&, const ViscF&, const ForceF&, const void* buf,
                         const float* snu, int kind, float* S_out, hipStream_t);
hipError_t launch_get(int storage, const Geo&, const void* buf, float* canon, hipStream_t);
hipError_t launch_set(int storage, const Geo&, void* buf, const float* canon, hipStream_t);
hipError_t launch_reduce(int storage, const Geo&, const ModelF&, const ViscF&, const ForceF&, const void* buf,
                         const float* snu, double* partials, double* out, hipStream_t);
PairPlan pair_plan(int storage, const Geo&, const ViscF&, const ForceF&);
PairPlan pair_tiles(int storage, const Geo&, const ViscF&, const ForceF&, int cols, int rows, int planes);
hipError_t launch_pair(const PairPlan&, const Geo&, const ModelF&, const ViscF&, const void* src, void* dst,
                       const float* snu_in, float* snu_out, hipStream_t);
}  // namespace d3q15

// Fixed device scratch of the allocation-free adjoint sweep: room for one adjoint state of up
// to 64 MiB (A planes of N floats), held by every device the library runs on.
constexpr size_t kNoAllocScratchBytes = size_t(64) << 20;

// Address of that scratch on the device of `stream` (looked up on the first call per device;
// no allocation).
hipError_t noalloc_scratch(hipStream_t stream, void** out);

// Fold nblocks partials into out[0..7]. rho0 > 0 (the diagnostics): slot 6 arrives as the
// largest |j|^2 and leaves as max |u| = sqrt(.) / rho0.
hipError_t launch_reduce_final(const double* partials, int nblocks, double* out, hipStream_t, double rho0 = 0.0);
hipError_t launch_stream_copy(const void* src, void* dst, size_t bytes, hipStream_t);
// The copies take a block of 256 threads per 4096 bytes, and a launch has fewer than 2^32 threads
// along x: just under 64 GiB. (A D3Q19 FP32 state with its rate field passes that at 859M nodes.)
inline size_t copy_blocks(size_t bytes) { return (bytes + 4095) / 4096; }
inline bool copy_fits_launch(size_t bytes1, size_t bytes2) {
  return copy_blocks(bytes1) + copy_blocks(bytes2) <= 0xffffffffu / 256;
}
// Two device-to-device copies (the second may be empty) in one launch, or by the runtime where one does not do.
hipError_t launch_copy2(const void* src1, void* dst1, size_t bytes1, const void* src2, void* dst2, size_t bytes2,
                        hipStream_t);

}  // namespace lbm
