// ng_launch.hpp -- host-callable launchers of the HIP kernels (ng_kernels.hip).
// dim: 1 or 2; prec: 0 = FP64, 1 = FP32, 2 = mixed.  All launches are
// asynchronous on s.  Optional events e0 / e1 receive the kernel's own start
// and end (timed launches; never under stream capture).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ng_internal.hpp"

namespace ng {

// variant: 0 for any set of solves; 1 + r when every solve of the launch is
// periodic with the HLLC flux and closure recipe r (a kernel with that path
// only); kVariantCsph (dim 1, FP64) when every solve takes the CSPH-TVD step.
// blocks == nullptr: the launch covers solve 0's workgroups 0..nblocks-1.
hipError_t launch_step(int dim, int prec, int variant, const InstDesc* descs, InstCtrl* ctrls,
                       const BlockRef* blocks, int64_t nblocks, int waves, int remap, int fused,
                       hipStream_t s, hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
// Priming pass: totals, checks and signal speed of the current state.  With
// blocks == nullptr the launch covers solve `inst`'s own workgroups 0..nblocks-1.
hipError_t launch_prime(int dim, int prec, const InstDesc* descs, InstCtrl* ctrls,
                        const BlockRef* blocks, int inst, int64_t nblocks, int waves,
                        hipStream_t s);
hipError_t launch_finalize(const InstDesc* descs, InstCtrl* ctrls, const int32_t* insts, int n,
                           int mode, hipStream_t s, hipEvent_t e0 = nullptr,
                           hipEvent_t e1 = nullptr);
hipError_t launch_small(int dim, int prec, const InstDesc* descs, InstCtrl* ctrls,
                        const int32_t* insts, int n, int waves, int64_t nsteps, hipStream_t s);
// Cells [i0, i0 + m) of a solve's current state as FP64 planes of m values at
// out (memory the device can write), conserved or primitive; status (may be
// null, likewise) receives the solve's status.
hipError_t launch_readout(int dim, int prec, const InstDesc* descs, const InstCtrl* ctrls, int inst,
                          int64_t i0, int64_t m, int prim, double* out, int32_t* status,
                          hipStream_t s);
hipError_t launch_set_limits(InstCtrl* ctrls, const int32_t* insts, int n, double t_end,
                             int64_t max_steps_from_now, hipStream_t s);

// Cooperative launch of 1D solves for up to nsteps <= kCoopMaxSteps steps each:
// grid workgroups of `waves` waves, all resident together (the runtime refuses
// a grid that does not fit).  s: 0..3 HLLC with closure recipe s, 4 HLL, 5 and
// 6 CSPH-TVD with the general closures and recipe 1 (3, 5, 6: FP64).  lds: the
// cells stay in LDS (lds_bytes of it), else in the state buffers.  One solve:
// `one`, groups and refs null; more: in groups, refs[w] the (group, workgroup of
// it) of workgroup w.  launch_resident_after has to follow.  resident_capacity
// gives the workgroups of that shape a CU holds at once.
constexpr int64_t kCoopMaxSteps = int64_t(1) << 16;
int resident_max_waves(int prec);
hipError_t resident_capacity(int prec, int s, bool lds, int waves, size_t lds_bytes,
                             int* blocks_per_cu);
hipError_t launch_resident(int prec, int s, bool lds, const InstDesc* descs, InstCtrl* ctrls,
                           const ResGroup* groups, const BlockRef* refs, const ResGroup& one,
                           const ResSync& sync, int grid, int waves, size_t lds_bytes,
                           int64_t nsteps, int32_t spin_limit, hipStream_t st);

// Clears the step number, the slots and the edges (bytes: res_space of them).
hipError_t launch_resident_clear(const ResSync& sync, size_t bytes, hipStream_t st);
// Folds the records of a cooperative launch into the control blocks of its
// solves and moves the step number on.
hipError_t launch_resident_after(const InstDesc* descs, InstCtrl* ctrls, const ResGroup* groups,
                                 int ngroups, const ResGroup& one, const ResSync& sync, int64_t nsteps,
                                 hipStream_t st);
// The cooperative launch of one 2D solve: every strip's rows in `chunks` runs, a
// wave each.  s: 0..2 periodic HLLC with closure recipe s, 3 HLLC with any ends,
// 4 the same with recipe 3 (FP64), 5 HLL.
int resident2d_max_waves(int prec);
hipError_t resident2d_capacity(int prec, int s, bool coh, int waves, int* blocks_per_cu);
hipError_t launch_resident2d(int prec, int s, const InstDesc* descs, InstCtrl* ctrls, int inst,
                             const ResSync& sync, int grid, int chunks, int waves, int64_t nsteps,
                             int32_t spin_limit, hipStream_t st);

// Static scratch of the entry point that allocates nothing: its device
// address on the current device (looked up once per device), and the priming
// pass that leaves one solve's descriptor, control block (one step from t, the
// first dt included)
// and finalize index list in it; nblocks <= kStaticPrimeBlocks workgroups,
// each with a record at d.partials.
constexpr size_t kStaticScratchBytes = size_t(2) << 20;
constexpr int64_t kStaticPrimeBlocks = 192;
constexpr int kMaxDevices = 64;
hipError_t static_scratch(void** ptr);
hipError_t launch_static_prime(int dim, const InstDesc& d, double t, double t_end, InstDesc* descs,
                               InstCtrl* ctrls, int32_t* insts, int64_t nblocks, hipStream_t s);

}  // namespace ng
