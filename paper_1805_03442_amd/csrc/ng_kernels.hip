// ng_kernels.hip -- HIP kernels (gfx950) of one MUSCL step, eq. (15), for
// batches of 1D and 2D periodic solves, plus the per-solve reduction of the
// step's global quantities (dt of eq. (16), FP64 totals and source budgets).
//
// Work decomposition.  A wavefront owns a strip of 64 consecutive x-cells: the
// 60 cells it updates plus 2 halo cells on each side, one cell per lane, so
// every x-neighbour (slopes, face states, fluxes) is one lane away and moves
// with a DPP lane shift, without LDS or barriers.
//   2D: a work item is (strip, chunk of rows).  The wave marches up the chunk
//       one row per iteration, keeping the rows it still needs (primitive
//       states of three rows, the half-step state and x-slopes of the row being
//       updated, the north face state and the y-flux below it) in registers, so
//       each y-face flux is computed once and each cell is loaded once (plus a
//       2-row halo per chunk).
//   1D: a work item is a group of consecutive 60-cell segments (58 cells and
//       3 halo lanes per side for the CSPH-TVD step of section 2.3, whose
//       particles reach three cells).
// Each cell's arithmetic does not depend on where it sits in a strip or chunk,
// so results are independent of the launch shape.
//
// The step kernel writes U^{n+1} into the other state buffer and, per
// workgroup, the max signal speed of U^{n+1}, the FP64 sums of U^{n+1}, the
// FP64 sums of the source increments, minima of rho and p and failure flags.
// The finalize kernel (one workgroup per solve) folds those records in a fixed
// order, accepts or rejects the step, advances t and computes the next dt.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <math.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "ng_device.hpp"
#include "ng_march2d.hpp"
#include "ng_launch.hpp"

namespace ng {

// Apply a folded step record v = (tot[5], src[2], smax, rho_min, p_min) with
// flags to a solve: reject (sticky NG_EPHYS, buffers not swapped) or accept
// (swap buffers, advance t, next dt from eq. (16)).  mode 1: priming (no step
// taken, only the totals and the first dt).
__device__ void accept_step(const InstDesc& d, InstCtrl& c, const StepCtl& sc, const double* v,
                            uint32_t flags, int mode)
{
    const double n = (double)d.ncell;
    const uint32_t bad = flags & 7u;
    if (bad) {
        c.status = -3;  // NG_EPHYS
        c.flags = bad;
        return;
    }
    if (mode == 0) {
        c.cur = sc.cur ^ 1;
        c.t = c.t + sc.dt;
        c.steps = c.steps + 1;
        c.dt_last = sc.dt;
        c.budget[0] += v[5];
        c.budget[1] += v[6];
    }
    for (int q = 0; q < 5; q++) c.total[q] = v[q] + n * d.uref[q];
    c.smax = v[7];
    c.rho_min = v[8];
    c.p_min = v[9];
    c.dt_cfl = d.cfl * d.h / v[7];
    c.flags = 0u;
    if (d.bc[0] == kBcSource) source_ghosts(d, c);
}

// ================================================================ finalize

// One workgroup per solve: fold the step's records in a fixed order, accept
// (swap buffers, advance t, next dt from eq. (16)) or reject (sticky NG_EPHYS,
// the state before the step is kept).  mode 0: after a step; 1: priming.
// Fold a solve's workgroup records in a fixed order with all threads of the
// calling workgroup (up to 16 waves): strided per-thread sums, then lanes
// (butterfly; lane 0's order is fixed), then waves in order.  The result is in
// out[10] / *oflags, valid in thread 0 after the call.
__device__ void fold_partials(const InstDesc& d, int64_t nb, double* out, uint32_t* oflags)
{
    __shared__ double sh[16][10];
    __shared__ uint32_t shf[16];
    const Partial* parts = (const Partial*)d.partials;
    double tot[5] = {0, 0, 0, 0, 0}, src0 = 0.0, src1 = 0.0, smax = 0.0, rmin = INFINITY,
           pmin = INFINITY;
    uint32_t flags = 0;
#pragma unroll 4
    for (int64_t b = threadIdx.x; b < nb; b += blockDim.x) {
        const Partial& p = parts[b];
        for (int q = 0; q < 5; q++) tot[q] += p.tot[q];
        src0 += p.src[0];
        src1 += p.src[1];
        smax = fmax(smax, p.smax);
        rmin = fmin(rmin, p.rho_min);
        pmin = fmin(pmin, p.p_min);
        flags |= p.flags;
    }
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    for (int m = 32; m >= 1; m >>= 1) {
        for (int q = 0; q < 5; q++) tot[q] += lane_xor(tot[q], lane, m);
        src0 += lane_xor(src0, lane, m);
        src1 += lane_xor(src1, lane, m);
        smax = fmax(smax, lane_xor(smax, lane, m));
        rmin = fmin(rmin, lane_xor(rmin, lane, m));
        pmin = fmin(pmin, lane_xor(pmin, lane, m));
        flags |= (uint32_t)__builtin_amdgcn_ds_bpermute(((lane ^ m) & 63) << 2, (int)flags);
    }
    if (lane == 0) {
        for (int q = 0; q < 5; q++) sh[wave][q] = tot[q];
        sh[wave][5] = src0;
        sh[wave][6] = src1;
        sh[wave][7] = smax;
        sh[wave][8] = rmin;
        sh[wave][9] = pmin;
        shf[wave] = flags;
    }
    __syncthreads();
    if (t == 0) {
        const int nw = blockDim.x >> 6;
        for (int w = 1; w < nw; w++) {
            for (int q = 0; q < 7; q++) sh[0][q] += sh[w][q];
            sh[0][7] = fmax(sh[0][7], sh[w][7]);
            sh[0][8] = fmin(sh[0][8], sh[w][8]);
            sh[0][9] = fmin(sh[0][9], sh[w][9]);
            shf[0] |= shf[w];
        }
        for (int q = 0; q < 10; q++) out[q] = sh[0][q];
        *oflags = shf[0];
    }
}

__global__ void __launch_bounds__(256) finalize_kernel(const InstDesc* __restrict__ descs,
                                                        InstCtrl* __restrict__ ctrls,
                                                        const int32_t* __restrict__ insts,
                                                        int mode)
{
    const int inst = insts[blockIdx.x];
    const InstDesc& d = descs[inst];
    InstCtrl& c = ctrls[inst];
    if (mode == 0 && d.fused) return;   // accepted by the step kernel itself
    const StepCtl sc = read_ctl(c);
    if (mode == 0 && !sc.active) return;
    if (mode == 1 && c.status != 0) return;
    double v[10];
    uint32_t flags;
    fold_partials(d, d.nblocks, v, &flags);
    if (threadIdx.x == 0) accept_step(d, c, sc, v, flags, mode);
}

// The last workgroup of a solve to finish a step folds the solve's records and
// accepts the step, so that a step is a single launch.  Each workgroup
// releases its record (agent-scope release fence) before it counts itself in;
// only the last one acquires (agent-scope acquire fence) before reading all
// records, so the other workgroups never invalidate their caches.  The counter
// is reset by the last one.
__device__ void last_block_accept(const InstDesc& d, InstCtrl& c, const StepCtl& sc)
{
    __shared__ int last;
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        const uint32_t prev =
            __hip_atomic_fetch_add(&c.arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = prev == (uint32_t)(d.nblocks - 1);
    }
    __syncthreads();
    if (!last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    double v[10];
    uint32_t flags;
    fold_partials(d, d.nblocks, v, &flags);
    if (threadIdx.x == 0) {
        accept_step(d, c, sc, v, flags, 0);
        c.arrive = 0u;
    }
}

// The workgroup's solve and its number there.  Without a table (the step of
// ng_step_static) the launch is solve 0's; it then zeroes the counter of the
// priming pass before it, which that pass left at zero unless overlapping
// calls raced: such a race does not outlive them.
__device__ __forceinline__ BlockRef block_ref(const BlockRef* blocks, int64_t bid, InstCtrl* ctrls)
{
    if (blocks) return blocks[bid];
    if (bid == 0 && threadIdx.x == 0) ctrls[0].primed = 0u;
    return BlockRef{0, (int32_t)bid};
}

// ================================================================ 2D step

// periodic solves take the plain wrap-around indexing; solves with a wall or
// outflow end the ghost mapping (a uniform choice per solve)
template <class P, int RS>
__device__ __forceinline__ void march2d_bc(const InstDesc& d, const typename P::K& k, int cur,
                                           const double* gsrc, int strip, int r0, int r1, int lane,
                                           Acc<typename P::R>& acc)
{
    if (d.any_bc)
        march2d<P, RS, true>(d, k, cur, gsrc, strip, r0, r1, lane, acc);
    else
        march2d<P, RS, false>(d, k, cur, gsrc, strip, r0, r1, lane, acc);
}

// One HLLC work item: a periodic solve whose closures match a compiled recipe
// (kRecipeCodes) takes that recipe's march, every other solve the general
// one.  Every kernel that steps a solve applies this same rule, so a solve's
// state is bitwise the same on every path.
template <class P, int CL = kRecipes>
__device__ __forceinline__ void march2d_hllc(const InstDesc& d, const typename P::K& k, int cur,
                                             const double* gsrc, int strip, int r0, int r1,
                                             int lane, Acc<typename P::R>& acc)
{
    if constexpr (P::kRecipes && CL > 0) {
        if (!d.any_bc && d.cl_recipe == CL) {
            march2d<P, 0, false, CL>(d, k, cur, gsrc, strip, r0, r1, lane, acc);
            return;
        }
        march2d_hllc<P, CL - 1>(d, k, cur, gsrc, strip, r0, r1, lane, acc);
    } else {
        march2d_bc<P, 0>(d, k, cur, gsrc, strip, r0, r1, lane, acc);
    }
}

// The strip and rows of work item `item`: strips fastest, then chunks of
// rows_per_item rows.
struct Item2d {
    int strip, r0, r1;
    __device__ Item2d(const InstDesc& d, int64_t item)
    {
        const int64_t chunk = item / d.nstrips;
        strip = (int)(item - chunk * d.nstrips);
        r0 = (int)(chunk * d.rows_per_item);
        r1 = r0 + d.rows_per_item < (int)d.ny ? r0 + d.rows_per_item : (int)d.ny;
    }
};

// V = 0: any solves (boundary kind, flux and closures per solve);
// V = 1 + r: every solve of the launch is periodic with the HLLC flux and its
// closures match recipe r (kRecipeCodes; r = 0: the general form) -- a kernel
// with only that path, and so fewer registers.
template <class P, int V>
__global__ void __launch_bounds__(256, P::kMinWaves) step2d_kernel(const InstDesc* __restrict__ descs,
                                                     InstCtrl* __restrict__ ctrls,
                                                     const BlockRef* __restrict__ blocks,
                                                     int remap, int fused)
{
    using R = typename P::R;
    const int64_t G = gridDim.x;
    const int64_t bid = remap ? xcd_remap(blockIdx.x, G) : (int64_t)blockIdx.x;
    const BlockRef br = block_ref(blocks, bid, ctrls);
    const InstDesc& d = descs[br.inst];
    const StepCtl sc = read_ctl(ctrls[br.inst]);
    if (!sc.active) return;
    const typename P::K k = P::make(d, sc.dt);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nwaves = d.waves_per_block;
    Acc<R> acc;
    acc_init(acc);
    const int64_t item = (int64_t)br.local * nwaves + wave;
    if (item < d.nitems) {
        const Item2d it(d, item);
        if constexpr (V > 0)
            march2d<P, 0, false, V - 1>(d, k, sc.cur, sc.gsrc, it.strip, it.r0, it.r1, lane, acc);
        else if (d.riemann == 1)
            march2d_bc<P, 1>(d, k, sc.cur, sc.gsrc, it.strip, it.r0, it.r1, lane, acc);
        else
            march2d_hllc<P>(d, k, sc.cur, sc.gsrc, it.strip, it.r0, it.r1, lane, acc);
    }
    acc_finish<P>(acc, k);
    Partial* parts = (Partial*)d.partials;
    block_reduce_store(acc, parts + br.local, wave, lane, nwaves);
    if (fused && d.fused) last_block_accept(d, ctrls[br.inst], sc);
}

// ================================================================ 1D step

// One work item of the 1D step: a group of consecutive 60-cell segments.  The
// next segment's load is issued before the current one is computed.
template <class P, int RS, bool BC, int CL = 0>
__device__ __forceinline__ void march1d(const InstDesc& d, const typename P::K& k, int cur,
                                        const double* gsrc, int64_t item, int lane,
                                        Acc<typename P::R>& acc)
{
    using R = typename P::R;
    constexpr int NC = 4;
    const int64_t n = d.nx;
    using St = typename P::St;
    const Planes<St, NC> src(d.buf[cur], n);
    const Planes<St, NC> dst(d.buf[cur ^ 1], n);
    const int64_t s0 = item * d.rows_per_item;
    const int64_t s1 = s0 + d.rows_per_item < d.nstrips ? s0 + d.rows_per_item : d.nstrips;
    auto boff = [&](int64_t sg) -> uint32_t {
        bool f;
        const int64_t x = BC ? axis_cell(sg * kInterior - kHalo + lane, n, d.bc[0], d.bc[1], f)
                             : wrap_axis(sg * kInterior - kHalo + lane, n);
        return (uint32_t)(x * (int64_t)sizeof(St));
    };
    St UA[NC], UB[NC];
    src.load(boff(s0), UA);
    auto seg = [&](int64_t sg, St* Uc, St* Ux) {
        const uint32_t o = boff(sg);
        // issued on every segment (the last one fetches itself again, from
        // cache, into the unused buffer), so that the compiler's wait counts
        // let the load stay in flight
        src.load(boff(sg + 1 < s1 ? sg + 1 : sg), Ux);
        if (BC) {
            // the lanes before a forced source take its wave; wall ghosts
            // carry the mirrored momentum
            bool f;
            const int64_t xr = sg * kInterior - kHalo + lane;
            (void)axis_cell(xr, n, d.bc[0], d.bc[1], f);
            if (d.bc[0] == kBcSource && xr < 0) source_cell<St, NC, P::kSplitE>(d, gsrc + (xr == -1 ? 0 : 5), Uc);
            if (f) Uc[1] = -Uc[1];
        }
        St Uo[NC];
        R Wn[NC + 1], s, sE, sV;
        seg1d<P, RS, CL>(k, Uc, Uo, Wn, s, sE, sV);
        const bool inner =
            lane >= kHalo && lane < kWave - kHalo && sg * kInterior + (lane - kHalo) < n;
        if (inner) {
            dst.store(o, Uo);
            acc_cell<P, NC>(acc, k, Uo, Wn, s, sE, sV);
        }
    };
    int64_t sg = s0;
    for (; sg + 1 < s1; sg += 2) {
        seg(sg, UA, UB);
        seg(sg + 1, UB, UA);
    }
    if (sg < s1) seg(sg, UA, UB);
}

template <class P, int RS>
__device__ __forceinline__ void march1d_bc(const InstDesc& d, const typename P::K& k, int cur,
                                           const double* gsrc,
                                           int64_t item, int lane, Acc<typename P::R>& acc)
{
    if (d.any_bc)
        march1d<P, RS, true>(d, k, cur, gsrc, item, lane, acc);
    else
        march1d<P, RS, false>(d, k, cur, gsrc, item, lane, acc);
}

// the 1D counterpart of march2d_hllc
template <class P, int CL = kRecipes>
__device__ __forceinline__ void march1d_hllc(const InstDesc& d, const typename P::K& k, int cur,
                                             const double* gsrc, int64_t item, int lane,
                                             Acc<typename P::R>& acc)
{
    if constexpr (P::kRecipes && CL > 0) {
        if (!d.any_bc && d.cl_recipe == CL) {
            march1d<P, 0, false, CL>(d, k, cur, gsrc, item, lane, acc);
            return;
        }
        march1d_hllc<P, CL - 1>(d, k, cur, gsrc, item, lane, acc);
    } else {
        march1d_bc<P, 0>(d, k, cur, gsrc, item, lane, acc);
    }
}

// CSPH-TVD step (section 2.3) of the segments of work item `item`, each 58
// cells and three halo lanes per side (seg_csph; ghost particles by the
// boundary rule, a wall ghost with its momentum negated, the three before a
// forced source with its wave at the step's start time, gsrc).
// FP64 only (the state is stored whole).
template <class P, bool BC>
__device__ __forceinline__ void march_csph(const InstDesc& d, const K64& k, int cur,
                                           const double* gsrc, int64_t item, int lane,
                                           Acc<double>& acc)
{
    static_assert(std::is_same<typename P::K, K64>::value, "CSPH-TVD runs on the FP64 state");
    constexpr int NC = 4;
    const int64_t n = d.nx;
    const Planes<double, NC> src(d.buf[cur], n);
    const Planes<double, NC> dst(d.buf[cur ^ 1], n);
    const int64_t s0 = item * d.rows_per_item;
    const int64_t s1 = s0 + d.rows_per_item < d.nstrips ? s0 + d.rows_per_item : d.nstrips;
    const CsphGrid g = csph_grid(d);
    auto coord = [&](int64_t sg) { return sg * kCsphInterior - kCsphHalo + lane; };
    auto boff = [&](int64_t sg) -> uint32_t {
        bool f;
        const int64_t x = BC ? axis_cell(coord(sg), n, d.bc[0], d.bc[1], f) : wrap_axis(coord(sg), n);
        return (uint32_t)(x * (int64_t)sizeof(double));
    };
    double UA[NC], UB[NC];
    src.load(boff(s0), UA);
    auto seg = [&](int64_t sg, double* Un, double* Ux) {
        const uint32_t o = boff(sg);
        src.load(boff(sg + 1 < s1 ? sg + 1 : sg), Ux);
        if (BC) {
            bool f;
            const int64_t xr = coord(sg);
            (void)axis_cell(xr, n, d.bc[0], d.bc[1], f);
            if (d.bc[0] == kBcSource && xr < 0 && xr >= -kCsphHalo)
                source_cell<double, NC, false>(d, gsrc + 5 * (-1 - xr), Un);
            if (f) Un[1] = -Un[1];
        }
        double Uo[NC], Wn[NC + 1], sv, sE, sV;
        seg_csph<0>(k, g, Un, Uo, Wn, sv, sE, sV);
        const bool inner = lane >= kCsphHalo && lane < kWave - kCsphHalo &&
                           sg * kCsphInterior + (lane - kCsphHalo) < n;
        if (inner) {
            dst.store(o, Uo);
            acc_cell<P, NC>(acc, k, Uo, Wn, sv, sE, sV);
        }
    };
    int64_t sg = s0;
    for (; sg + 1 < s1; sg += 2) {
        seg(sg, UA, UB);
        seg(sg + 1, UB, UA);
    }
    if (sg < s1) seg(sg, UA, UB);
}

// the FP64 1D step of a solve under its scheme (the MUSCL step on the other
// arithmetic)
template <class P>
__device__ __forceinline__ void march1d_any(const InstDesc& d, const typename P::K& k, int cur,
                                            const double* gsrc, int64_t item, int lane,
                                            Acc<typename P::R>& acc)
{
    if constexpr (std::is_same<typename P::K, K64>::value) {
        if (d.scheme == kSchemeCsph) {
            if (d.any_bc)
                march_csph<P, true>(d, k, cur, gsrc, item, lane, acc);
            else
                march_csph<P, false>(d, k, cur, gsrc, item, lane, acc);
            return;
        }
    }
    if (d.riemann == 1)
        march1d_bc<P, 1>(d, k, cur, gsrc, item, lane, acc);
    else
        march1d_hllc<P>(d, k, cur, gsrc, item, lane, acc);
}

// V as for step2d_kernel, or kVariantCsph: every solve of the launch takes the
// CSPH-TVD step (a kernel with that path only)
template <class P, int V>
__global__ void __launch_bounds__(256, P::kMinWaves1D) step1d_kernel(const InstDesc* __restrict__ descs,
                                                     InstCtrl* __restrict__ ctrls,
                                                     const BlockRef* __restrict__ blocks,
                                                     int remap, int fused)
{
    using R = typename P::R;
    const int64_t G = gridDim.x;
    const int64_t bid = remap ? xcd_remap(blockIdx.x, G) : (int64_t)blockIdx.x;
    const BlockRef br = block_ref(blocks, bid, ctrls);
    const InstDesc& d = descs[br.inst];
    const StepCtl sc = read_ctl(ctrls[br.inst]);
    if (!sc.active) return;
    const typename P::K k = P::make(d, sc.dt);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nwaves = d.waves_per_block;
    Acc<R> acc;
    acc_init(acc);
    const int64_t item = (int64_t)br.local * nwaves + wave;
    if (item < d.nitems) {
        if constexpr (V == kVariantCsph) {
            if (d.any_bc)
                march_csph<P, true>(d, k, sc.cur, sc.gsrc, item, lane, acc);
            else
                march_csph<P, false>(d, k, sc.cur, sc.gsrc, item, lane, acc);
        } else if constexpr (V > 0) {
            march1d<P, 0, false, V - 1>(d, k, sc.cur, sc.gsrc, item, lane, acc);
        } else {
            march1d_any<P>(d, k, sc.cur, sc.gsrc, item, lane, acc);
        }
    }
    acc_finish<P>(acc, k);
    Partial* parts = (Partial*)d.partials;
    block_reduce_store(acc, parts + br.local, wave, lane, nwaves);
    if (fused && d.fused) last_block_accept(d, ctrls[br.inst], sc);
}

// ============================================================ priming pass

// Signal speed, sums and checks of the current state (no step): the records
// from which the finalize kernel derives the first dt and the totals.
template <class P, int NC>
__global__ void __launch_bounds__(256) prime_kernel(const InstDesc* __restrict__ descs,
                                                    InstCtrl* __restrict__ ctrls,
                                                    const BlockRef* __restrict__ blocks, int inst)
{
    using R = typename P::R;
    // without a workgroup table the launch covers the workgroups of one solve
    const BlockRef br = blocks ? blocks[blockIdx.x] : BlockRef{inst, (int32_t)blockIdx.x};
    const InstDesc& d = descs[br.inst];
    const InstCtrl& cc = ctrls[br.inst];
    if (cc.status != 0) return;
    const typename P::K k = P::make(d, 0.0);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nwaves = d.waves_per_block;
    Acc<R> acc;
    acc_init(acc);
    const int64_t item = (int64_t)br.local * nwaves + wave;
    if (item < d.nitems) {
        using St = typename P::St;
        const St* __restrict__ src = (const St*)d.buf[cc.cur];
        const int64_t nx = d.nx, ncell = d.ncell;
        int64_t xs, rows0, rows1, seg0, seg1;
        if (NC == 5) {
            const int64_t strip = item % d.nstrips, chunk = item / d.nstrips;
            xs = strip * kInterior;
            rows0 = chunk * d.rows_per_item;
            rows1 = rows0 + d.rows_per_item < d.ny ? rows0 + d.rows_per_item : d.ny;
            seg0 = 0;
            seg1 = 1;
        } else {
            xs = 0;
            rows0 = 0;
            rows1 = 1;
            seg0 = item * d.rows_per_item;
            seg1 = seg0 + d.rows_per_item < d.nstrips ? seg0 + d.rows_per_item : d.nstrips;
        }
        const int w = NC == 5 ? kInterior : seg_cells(d.scheme);
        for (int64_t sg = seg0; sg < seg1; sg++) {
            const int64_t xbase = NC == 5 ? xs : sg * w;
            const int64_t xo = xbase + (lane - kHalo);
            const bool inner = lane >= kHalo && lane < kHalo + w && xo < nx;
            if (!inner) continue;
            for (int64_t r = rows0; r < rows1; r++) {
                St U[NC];
                R W[NC + 1];
                load_cell_cached<St, NC>(src, ncell, r * nx + xo, U);
                P::prim(k, U, W);
                R s = P::speed(k, W);
                acc_cell<P, NC>(acc, k, U, W, s, (R)0, (R)0);
            }
        }
    }
    acc_finish<P>(acc, k);
    Partial* parts = (Partial*)d.partials;
    block_reduce_store(acc, parts + br.local, wave, lane, nwaves);
}

// ============================================================== read-out

// Cells [i0, i0 + m) of a solve's current state as full FP64 planes of m values
// at out (pinned host memory: the kernel's stores cross the bus themselves):
// conserved, or primitive by eq. (5).  The reference of a deviation state is
// added back and its energy slot made E again; every operation is one IEEE
// operation in a fixed order.  status (null: none): receives the solve's.
template <class St, int NC, bool Split>
__global__ void __launch_bounds__(256) readout_kernel(const InstDesc* __restrict__ descs,
                                                      const InstCtrl* __restrict__ ctrls, int inst,
                                                      int64_t i0, int64_t m, int prim,
                                                      double* __restrict__ out,
                                                      int32_t* __restrict__ status)
{
    const InstDesc& d = descs[inst];
    const int32_t cur = ctrls[inst].cur, left = ctrls[inst].status;
    const St* __restrict__ src = (const St*)d.buf[cur];
    constexpr int iE = NC == 5 ? 3 : 2, iV = NC - 1;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * blockDim.x) {
        double U[NC];
        for (int c = 0; c < NC; c++) U[c] = (double)src[c * d.ncell + i0 + i];
        if (Split) {
            for (int c = 0; c < NC; c++)
                U[c] = U[c] + (c == 0 ? d.uref[0] : (c == iE ? d.e1_r : (c == iV ? d.uref[4] : 0.0)));
            U[iE] = U[iE] + U[iV];
        }
        if (prim) {
            const double rho = U[0], u = U[1] / rho;
            const double v = NC == 5 ? U[2] / rho : 0.0;
            const double ke = 0.5 * rho * (NC == 5 ? u * u + v * v : u * u);
            U[1] = u;
            if (NC == 5) U[2] = v;
            U[iE] = d.gm1 * (U[iE] - ke - U[iV]);
        }
        for (int c = 0; c < NC; c++) __builtin_nontemporal_store(U[c], out + c * m + i);
    }
    if (status && blockIdx.x == 0 && threadIdx.x == 0) *status = left;
}

// Set the stop condition of a set of solves (a kernel, so that it can sit in
// the stream between captured graphs without a host copy).
__global__ void set_limits_kernel(InstCtrl* __restrict__ ctrls, const int32_t* __restrict__ insts,
                                  int n, double t_end, int64_t max_steps_from_now)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    InstCtrl& c = ctrls[insts[i]];
    c.t_end = t_end;
    c.max_steps = max_steps_from_now < 0 ? INT64_MAX : c.steps + max_steps_from_now;
}

// ====================================================== small solves

// One workgroup advances one small solve through up to nsteps steps without
// returning to the host: its waves share the solve's work items, fold their
// records through LDS in wave order, and wave 0 accepts the step before the
// next one starts.  Per-cell arithmetic is that of the step kernels, so the
// state is bitwise the same as with one launch per step.
template <class P, int NC>
__global__ void __launch_bounds__(512) run_small_kernel(const InstDesc* __restrict__ descs,
                                                        InstCtrl* __restrict__ ctrls,
                                                        const int32_t* __restrict__ insts,
                                                        int64_t nsteps)
{
    using R = typename P::R;
    const int inst = insts[blockIdx.x];
    const InstDesc& d = descs[inst];
    InstCtrl& c = ctrls[inst];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nw = blockDim.x >> 6;
    __shared__ double sh[kMaxWaves][10];
    __shared__ uint32_t shf[kMaxWaves];
    for (int64_t st = 0; st < nsteps; st++) {
        const StepCtl sc = read_ctl(c);
        if (!sc.active) break;
        const typename P::K k = P::make(d, sc.dt);
        Acc<R> acc;
        acc_init(acc);
        for (int64_t item = wave; item < d.nitems; item += nw) {
            if constexpr (NC == 5) {
                const Item2d it(d, item);
                if (d.riemann == 1)
                    march2d_bc<P, 1>(d, k, sc.cur, sc.gsrc, it.strip, it.r0, it.r1, lane, acc);
                else
                    march2d_hllc<P>(d, k, sc.cur, sc.gsrc, it.strip, it.r0, it.r1, lane, acc);
            } else {
                march1d_any<P>(d, k, sc.cur, sc.gsrc, item, lane, acc);
            }
        }
        acc_finish<P>(acc, k);
        uint32_t flags = acc_flags(acc);
        double smax = (double)acc.smax, rmin = (double)acc.rmin, pmin = (double)acc.pmin;
        for (int m = 32; m >= 1; m >>= 1) {
            for (int q = 0; q < 5; q++) acc.tot[q] += lane_xor(acc.tot[q], lane, m);
            acc.src[0] += lane_xor(acc.src[0], lane, m);
            acc.src[1] += lane_xor(acc.src[1], lane, m);
            smax = fmax(smax, lane_xor(smax, lane, m));
            rmin = fmin(rmin, lane_xor(rmin, lane, m));
            pmin = fmin(pmin, lane_xor(pmin, lane, m));
            flags |= (uint32_t)__builtin_amdgcn_ds_bpermute(((lane ^ m) & 63) << 2, (int)flags);
        }
        if (lane == 0) {
            for (int q = 0; q < 5; q++) sh[wave][q] = acc.tot[q];
            sh[wave][5] = acc.src[0];
            sh[wave][6] = acc.src[1];
            sh[wave][7] = smax;
            sh[wave][8] = rmin;
            sh[wave][9] = pmin;
            shf[wave] = flags;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < nw; w++) {
                for (int q = 0; q < 7; q++) sh[0][q] += sh[w][q];
                sh[0][7] = fmax(sh[0][7], sh[w][7]);
                sh[0][8] = fmin(sh[0][8], sh[w][8]);
                sh[0][9] = fmin(sh[0][9], sh[w][9]);
                shf[0] |= shf[w];
            }
            accept_step(d, c, sc, sh[0], shf[0], 0);
        }
        __syncthreads();
    }
}

// ======================================================= static scratch

// Device memory of the entry point for callers that cannot allocate
// (ng_step_static): the solve's descriptor and control block, the index list
// of the finalize kernel and the per-workgroup reduction records, in one
// file-scope array of kStaticScratchBytes that each GPU holds
// until the process ends.  Host code never uses the array's name as an
// address: static_scratch() takes each device's own address of it once.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

hipError_t static_scratch(void** ptr)
{
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

// Priming pass of the entry point that allocates nothing.  The solve's
// descriptor and control come as arguments and are left in the scratch for the
// step's launch.  Each thread takes cells a launch apart (a record needs no
// strips or rows), and the last workgroup folds the records (as
// last_block_accept, with a counter of its own that it leaves at zero): two
// launches where setting up, priming, folding, stepping and folding were five.
// Latency bounds it on small grids, the read of the state on large ones (a call
// back to back, before and now: 150x150 cells 32.2 and 23.1 us, 380x400 35.4
// and 31.6, 10^6 cells in 1D 58.0 and 49.7).
template <class P, int NC>
__global__ void __launch_bounds__(256) static_prime_kernel(InstDesc d, double t, double t_end,
                                                           InstDesc* __restrict__ descs,
                                                           InstCtrl* __restrict__ ctrls,
                                                           int32_t* __restrict__ insts)
{
    using R = typename P::R;
    using St = typename P::St;
    __shared__ int last;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        descs[0] = d;
        insts[0] = 0;
    }
    const typename P::K k = P::make(d, 0.0);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const St* __restrict__ src = (const St*)d.buf[0];
    Acc<R> acc;
    acc_init(acc);
    const int64_t step = (int64_t)gridDim.x * 256;
#pragma unroll 2
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < d.ncell; i += step) {
        St U[NC];
        R W[NC + 1];
        load_cell_cached<St, NC>(src, d.ncell, i, U);
        P::prim(k, U, W);
        const R s = P::speed(k, W);
        acc_cell<P, NC>(acc, k, U, W, s, (R)0, (R)0);
    }
    acc_finish<P>(acc, k);
    block_reduce_store(acc, (Partial*)d.partials + blockIdx.x, wave, lane, 4);
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        const uint32_t prev = __hip_atomic_fetch_add(&ctrls[0].primed, 1u, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
        last = prev == gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    double v[10];
    uint32_t flags;
    // descs[0], which workgroup 0 released with its record: a late use of the
    // argument puts a copy of it into every thread's scratch memory at entry
    // (380x400 cells: 38 to 61 us per call)
    fold_partials(descs[0], gridDim.x, v, &flags);
    if (threadIdx.x == 0) {
        InstCtrl& c = ctrls[0];
        c = InstCtrl{};
        c.t = t;
        c.t_end = t_end;
        c.max_steps = 1;
        accept_step(descs[0], c, read_ctl(c), v, flags, 1);
    }
}

hipError_t launch_static_prime(int dim, const InstDesc& d, double t, double t_end, InstDesc* descs,
                               InstCtrl* ctrls, int32_t* insts, int64_t nblocks, hipStream_t s)
{
    if (nblocks < 1 || nblocks > kStaticPrimeBlocks) return hipErrorInvalidValue;
    dim3 g((unsigned)nblocks), b(256);
    if (dim == 2)
        hipLaunchKernelGGL((static_prime_kernel<Plain64<5>, 5>), g, b, 0, s, d, t, t_end, descs, ctrls,
                           insts);
    else
        hipLaunchKernelGGL((static_prime_kernel<Plain64<4>, 4>), g, b, 0, s, d, t, t_end, descs, ctrls,
                           insts);
    return hipGetLastError();
}

// ================================================================ launchers

static inline bool grid_ok(int64_t nblocks) { return nblocks > 0 && nblocks < (1LL << 31); }

// Launch on s; with events, through the AMD extension that records the
// kernel's own start and end in them (no separate event packets on the
// stream, so timing adds no gaps between launches).  Untimed launches use the
// plain form, which stream capture records as a kernel node.
template <class... A>
static void launch(void (*kernel)(A...), dim3 g, dim3 b, hipStream_t s, hipEvent_t e0,
                   hipEvent_t e1, A... a)
{
    if (e0 || e1)
        hipExtLaunchKernelGGL(kernel, g, b, 0, s, e0, e1, 0, a...);
    else
        hipLaunchKernelGGL(kernel, g, b, 0, s, a...);
}

// Step kernel of a policy for variant v.
template <template <int> class Pol, int NC>
static void launch_variant(int v, dim3 g, dim3 b, hipStream_t s, hipEvent_t e0, hipEvent_t e1,
                           const InstDesc* descs, InstCtrl* ctrls, const BlockRef* blocks,
                           int remap, int fused)
{
    using P = Pol<NC>;
    if constexpr (NC == 5) {
        if (v == 0) launch(step2d_kernel<P, 0>, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
        else if (v == 1) launch(step2d_kernel<P, 1>, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
        else if (v == 2) launch(step2d_kernel<P, 2>, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
        else launch(step2d_kernel<P, 3>, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
    } else {
        if (v == 0) launch(step1d_kernel<P, 0>, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
        else if (v == 1) launch(step1d_kernel<P, 1>, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
        else if (v == 2) launch(step1d_kernel<P, 2>, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
        else if (v == 3) launch(step1d_kernel<P, 3>, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
        else if constexpr (std::is_same<typename P::K, K64>::value)
            launch(step1d_kernel<P, kVariantCsph>, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
    }
}

hipError_t launch_step(int dim, int prec, int variant, const InstDesc* descs, InstCtrl* ctrls,
                       const BlockRef* blocks, int64_t nblocks, int waves, int remap, int fused,
                       hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    static_assert(kRecipes == 2, "launch_variant instantiates variants 0..3");
    if (!grid_ok(nblocks) || waves < 1 || waves > 4) return hipErrorInvalidValue;
    if (variant < 0 || (variant > kRecipes + 1 &&
                        !(variant == kVariantCsph && dim == 1 && prec == 0)))
        return hipErrorInvalidValue;
    dim3 g((unsigned)nblocks), b((unsigned)(64 * waves));
    if (dim == 2) {
        if (prec == 0)
            launch_variant<Plain64, 5>(variant, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
        else if (prec == 1)
            launch_variant<Dev32, 5>(variant, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
        else
            launch_variant<Mix32, 5>(variant, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
    } else {
        if (prec == 0)
            launch_variant<Plain64, 4>(variant, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
        else if (prec == 1)
            launch_variant<Dev32, 4>(variant, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
        else
            launch_variant<Mix32, 4>(variant, g, b, s, e0, e1, descs, ctrls, blocks, remap, fused);
    }
    return hipGetLastError();
}

hipError_t launch_prime(int dim, int prec, const InstDesc* descs, InstCtrl* ctrls,
                        const BlockRef* blocks, int inst, int64_t nblocks, int waves,
                        hipStream_t s)
{
    if (!grid_ok(nblocks) || waves < 1 || waves > 4) return hipErrorInvalidValue;
    dim3 g((unsigned)nblocks), b((unsigned)(64 * waves));
    if (dim == 2) {
        if (prec == 0)
            hipLaunchKernelGGL((prime_kernel<Plain64<5>, 5>), g, b, 0, s, descs, ctrls, blocks, inst);
        else if (prec == 1)
            hipLaunchKernelGGL((prime_kernel<Dev32<5>, 5>), g, b, 0, s, descs, ctrls, blocks, inst);
        else
            hipLaunchKernelGGL((prime_kernel<Mix32<5>, 5>), g, b, 0, s, descs, ctrls, blocks, inst);
    } else {
        if (prec == 0)
            hipLaunchKernelGGL((prime_kernel<Plain64<4>, 4>), g, b, 0, s, descs, ctrls, blocks, inst);
        else if (prec == 1)
            hipLaunchKernelGGL((prime_kernel<Dev32<4>, 4>), g, b, 0, s, descs, ctrls, blocks, inst);
        else
            hipLaunchKernelGGL((prime_kernel<Mix32<4>, 4>), g, b, 0, s, descs, ctrls, blocks, inst);
    }
    return hipGetLastError();
}

hipError_t launch_finalize(const InstDesc* descs, InstCtrl* ctrls, const int32_t* insts, int n,
                           int mode, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    if (n <= 0) return hipSuccess;
    // four waves per solve: enough to fold a few thousand records with one
    // load in flight per lane, and a quarter of the dispatch work of 1024
    // threads when a batch finalizes hundreds of solves (512 solves: 108 ->
    // 99 us per step; 4096^2 alone: 10.8 -> 8.0 us)
    launch(finalize_kernel, dim3((unsigned)n), dim3(256), s, e0, e1, descs, ctrls, insts, mode);
    return hipGetLastError();
}

hipError_t launch_small(int dim, int prec, const InstDesc* descs, InstCtrl* ctrls,
                        const int32_t* insts, int n, int waves, int64_t nsteps, hipStream_t s)
{
    if (n <= 0 || nsteps <= 0) return hipSuccess;
    if (waves < 1 || waves > kMaxWaves) return hipErrorInvalidValue;
    dim3 g((unsigned)n), b((unsigned)(64 * waves));
    if (dim == 2) {
        if (prec == 0)
            hipLaunchKernelGGL((run_small_kernel<Plain64<5>, 5>), g, b, 0, s, descs, ctrls, insts, nsteps);
        else if (prec == 1)
            hipLaunchKernelGGL((run_small_kernel<Dev32<5>, 5>), g, b, 0, s, descs, ctrls, insts, nsteps);
        else
            hipLaunchKernelGGL((run_small_kernel<Mix32<5>, 5>), g, b, 0, s, descs, ctrls, insts, nsteps);
    } else {
        if (prec == 0)
            hipLaunchKernelGGL((run_small_kernel<Plain64<4>, 4>), g, b, 0, s, descs, ctrls, insts, nsteps);
        else if (prec == 1)
            hipLaunchKernelGGL((run_small_kernel<Dev32<4>, 4>), g, b, 0, s, descs, ctrls, insts, nsteps);
        else
            hipLaunchKernelGGL((run_small_kernel<Mix32<4>, 4>), g, b, 0, s, descs, ctrls, insts, nsteps);
    }
    return hipGetLastError();
}

hipError_t launch_readout(int dim, int prec, const InstDesc* descs, const InstCtrl* ctrls, int inst,
                          int64_t i0, int64_t m, int prim, double* out, int32_t* status,
                          hipStream_t s)
{
    if (m <= 0) return hipErrorInvalidValue;
    const int64_t g = (m + 255) / 256;
    dim3 gr((unsigned)(g < 1024 ? g : 1024)), b(256);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, gr, b, 0, s, descs, ctrls, inst, i0, m, prim, out, status);
    };
    if (dim == 2) {
        if (prec == 0) go(readout_kernel<double, 5, false>);
        else if (prec == 1) go(readout_kernel<float, 5, true>);
        else go(readout_kernel<double, 5, true>);
    } else {
        if (prec == 0) go(readout_kernel<double, 4, false>);
        else if (prec == 1) go(readout_kernel<float, 4, true>);
        else go(readout_kernel<double, 4, true>);
    }
    return hipGetLastError();
}

hipError_t launch_set_limits(InstCtrl* ctrls, const int32_t* insts, int n, double t_end,
                             int64_t max_steps_from_now, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(set_limits_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       ctrls, insts, n, t_end, max_steps_from_now);
    return hipGetLastError();
}

}  // namespace ng
