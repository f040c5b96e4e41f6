// ng_device.hpp -- device code shared by the kernels of ng_kernels.hip and
// ng_resident.hip: lane shifts, boundary rules, the arithmetic policies, the
// per-lane accumulators and their reduction, the control word of a step, the
// forced source, state planes, and one segment of either 1D step.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "ng_cell.hpp"
#include "ng_csph.hpp"
#include "ng_internal.hpp"

namespace ng {

// ------------------------------------------------------------ cross-lane

// Whole-wavefront DPP shifts: from_left gives lane l the value of lane l-1,
// from_right the value of lane l+1 (the end lanes get 0 through bound_ctrl;
// they are halo lanes whose results are never used).
__device__ __forceinline__ int dpp_l(int v) { return __builtin_amdgcn_mov_dpp(v, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int dpp_r(int v) { return __builtin_amdgcn_mov_dpp(v, 0x130, 0xf, 0xf, true); }
__device__ __forceinline__ float from_left(float v) { return __int_as_float(dpp_l(__float_as_int(v))); }
__device__ __forceinline__ float from_right(float v) { return __int_as_float(dpp_r(__float_as_int(v))); }
__device__ __forceinline__ double from_left(double v)
{
    return __hiloint2double(dpp_l(__double2hiint(v)), dpp_l(__double2loint(v)));
}
__device__ __forceinline__ double from_right(double v)
{
    return __hiloint2double(dpp_r(__double2hiint(v)), dpp_r(__double2loint(v)));
}

// face value W + s/2 of a limited linear profile (eq. (14)) as one fused
// multiply-add: the product by 1/2 is exact, so this is the correctly rounded
// W + s/2, the value of the separate multiply and add
__device__ __forceinline__ float face(float w, float s) { return __builtin_fmaf(0.5f, s, w); }
__device__ __forceinline__ double face(double w, double s) { return __builtin_fma(0.5, s, w); }

// keep a value computed here (stops it from being sunk into a later block,
// away from the DPP move it combines with)
__device__ __forceinline__ void pin(float& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void pin(double& v) { asm volatile("" : "+v"(v)); }

// lane permute through the LDS crossbar (reductions only)
__device__ __forceinline__ double lane_xor(double v, int lane, int m)
{
    const int addr = ((lane ^ m) & 63) << 2;
    int lo = __builtin_amdgcn_ds_bpermute(addr, __double2loint(v));
    int hi = __builtin_amdgcn_ds_bpermute(addr, __double2hiint(v));
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float lane_xor(float v, int lane, int m)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(((lane ^ m) & 63) << 2, __float_as_int(v)));
}

// index of a cell coordinate in [-3, n + 62) on a periodic axis of n >= 4
// cells (one wrap suffices when n >= 64; short axes wrap several times)
__device__ __forceinline__ int64_t wrap_axis(int64_t x, int64_t n)
{
    if (x < 0) x += n;
    if (n >= kWave) return x >= n ? x - n : x;
    while (x >= n) x -= n;
    return x;
}

// Cell of coordinate j in [-3, n + 62) on an axis of n >= 4 cells whose ends
// have boundary kinds lo and hi, and whether the normal momentum of the value
// loaded there is to be negated.  Ghosts of a periodic end wrap around, of a
// wall mirror the edge cells (-1 -> 0, -2 -> 1, -3 -> 2), of an outflow end copy the
// edge cell; coordinates beyond the ghost layer (lanes that feed no interior
// cell) are clamped into the axis.
__device__ __forceinline__ int64_t axis_cell(int64_t j, int64_t n, int lo, int hi, bool& flip)
{
    flip = false;
    if (j >= 0 && j < n) return j;
    const int bc = j < 0 ? lo : hi;
    if (bc == kBcPeriodic) return wrap_axis(j, n);
    if (bc == kBcOutflow || bc == kBcSource) return j < 0 ? 0 : n - 1;
    flip = true;
    const int64_t m = j < 0 ? -1 - j : 2 * n - 1 - j;
    return m < 0 ? 0 : (m >= n ? n - 1 : m);
}

// Workgroups are dispatched round-robin over the 8 XCDs; hand each XCD a
// contiguous range of logical workgroups so that neighbouring tiles (which
// share halo rows and columns) meet in the same L2.
__device__ __forceinline__ int64_t xcd_remap(int64_t b, int64_t G)
{
    int64_t x = b & 7, i = b >> 3;
    int64_t q = G >> 3, r = G & 7;
    return (x < r) ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

// ------------------------------------------------------------- policies

template <int NC>
struct Plain64 {
    using R = double;
    // the FP64 step needs more than 128 registers; asking for two waves per
    // SIMD trades a few spills for latency hiding (13 % faster at 4096^2)
    static constexpr int kMinWaves = 2;
    static constexpr int kMinWaves1D = 3;
    // largest workgroup of a resident launch
    static constexpr int kResThreads = 768;
    static constexpr int kRes2Threads = 512;
    // U^n of the updated row is re-read from cache (no registers to spare)
    static constexpr bool kKeepRows = false;
    // the energy slot holds E itself
    static constexpr bool kSplitE = false;
    // the general kernels take the closure recipe in the closures themselves
    static constexpr bool kRecipes = false;
    using St = double;
    using K = K64;
    static __device__ K make(const InstDesc& d, double dt)
    {
        K k;
        k.gam = d.gamma;
        k.gm1 = d.gm1;
        k.R = d.R;
        k.Cv = d.Cv;
        k.rho0 = d.rho0;
        k.T0 = d.T0;
        k.tau0 = d.tau0;
        k.Q0 = d.Q0;
        k.I0 = d.I0;
        k.d = &d;
        k.fx = d.fx;
        k.fy = d.fy;
        k.igm1 = d.igm1;
        k.iR = d.iR;
        k.irho0 = d.irho0;
        k.iT0 = d.iT0;
        k.cl = d.cl_recipe;
        k.stiff_z = d.stiff_z;
        k.dt = dt;
        k.dtdx = quot64(dt, d.h, d.ih);
        k.hdtdx = 0.5 * k.dtdx;
        k.hdt = 0.5 * dt;
        k.riemann = d.riemann;
        return k;
    }
    static __device__ void prim(const K& k, const R* U, R* W) { prim64<NC>(k, U, W); }
    static __device__ R speed(const K& k, const R* W) { return speed64<NC>(k, W); }
    template <bool FR = false, int CL = 0>
    static __device__ void predict(const K& k, const R* W, const R* sx, const R* sy, R* Wh,
                                   R act = 1)
    {
        predict64<NC, CL>(k, W, sx, sy, Wh, act);
    }
    template <int RS>
    static __device__ void flux(const K& k, const R* L, const R* Rr, R* F)
    {
        flux64<NC, RS>(k, L, Rr, F);
    }
    template <bool FR = false, int CL = 0>
    static __device__ void update(const K& k, const R* Un, const R* dF, const R* dG, const R* Wh,
                                  R* Unew, R& sE, R& sV, R act = 1)
    {
        update64<NC, CL>(k, Un, dF, dG, Wh, Unew, sE, sV, act);
    }
    static __device__ R full_rho(const K&, R r) { return r; }
    static __device__ R full_p(const K&, R p) { return p; }
};

template <int NC>
struct Dev32 {
    using R = float;
    using St = float;   // stored state: FP32 deviations
    using K = K32;
    static constexpr int kMinWaves = 1;
    static constexpr int kMinWaves1D = 1;
    // twelve waves (three per SIMD at up to 168 registers, one workgroup per
    // CU): 2^20 cells 12.3 against 13.2 us per step with eight; sixteen-wave
    // workgroups, which force 128 registers, spill and were slower
    static constexpr int kResThreads = 768;
    // (twelve waves, at 168 registers, spill: 1024^2 20.0 against 19.1 us per step)
    static constexpr int kRes2Threads = 512;
    // the raw rows stay in registers until their update
    static constexpr bool kKeepRows = true;
    // the energy slot holds e = E - E_nu (deviation from e_r)
    static constexpr bool kSplitE = true;
    static constexpr bool kRecipes = true;
    static __device__ K make(const InstDesc& d, double dt)
    {
        K k;
        k.gam = (float)d.gamma;
        k.gm1 = (float)d.gm1;
        k.igm1 = (float)(1.0 / d.gm1);
        k.CvR = (float)(d.Cv / d.R);
        k.rho_r = (float)d.uref[0];
        k.p_r = (float)d.p_r;
        k.ev_r = (float)d.uref[4];
        k.H_r = (float)d.H_r;
        k.D_r = (float)d.D_r;
        for (int i = 0; i < 3; i++) {
            k.cl_c[i] = (float)d.cl_c[i];
            k.cl_a[i] = (float)d.cl_a[i];
            k.cl_b[i] = (float)d.cl_b[i];
        }
        k.gp_r = (float)(d.gamma * d.p_r);
        k.fx = (float)d.fx;
        k.fy = (float)d.fy;
        k.stiff_z = (float)d.stiff_z;
        k.hstiff_z = 0.5f * k.stiff_z;
        k.dt = (float)dt;
        k.dtdx = (float)(dt / d.h);
        k.hdtdx = 0.5f * k.dtdx;
        k.hdt = 0.5f * k.dt;
        k.hdtfx = k.hdt * k.fx;
        k.hdtfy = k.hdt * k.fy;
        k.force = d.fx != 0.0 || d.fy != 0.0;
        k.dt64 = (double)k.dt;
        k.hdt64 = (double)k.hdt;
        k.riemann = d.riemann;
        return k;
    }
    static __device__ void prim(const K& k, const R* U, R* W) { prim32<NC>(k, U, W); }
    static __device__ R speed(const K& k, const R* W) { return speed32<NC>(k, W); }
    // FR: the half-step state carries the full density (HLLC faces);
    // CL: closure recipe
    template <bool FR = false, int CL = 0>
    static __device__ void predict(const K& k, const R* W, const R* sx, const R* sy, R* Wh,
                                   R act = 1)
    {
        predict32<NC, FR, CL>(k, W, sx, sy, Wh, act);
    }
    template <int RS>
    static __device__ void flux(const K& k, const R* L, const R* Rr, R* F)
    {
        flux32<NC, RS>(k, L, Rr, F);
    }
    template <bool FR = false, int CL = 0>
    static __device__ void update(const K& k, const R* Un, const R* dF, const R* dG, const R* Wh,
                                  R* Unew, R& sE, R& sV, R act = 1)
    {
        update32<NC, FR, CL>(k, Un, dF, dG, Wh, Unew, sE, sV, act);
    }
    static __device__ R full_rho(const K& k, R r) { return k.rho_r + r; }
    static __device__ R full_p(const K& k, R p) { return k.p_r + p; }
};

// FP32 arithmetic on an FP64 state: the deviations from the reference are
// stored in FP64 and rounded to FP32 where the stencil reads them; the step's
// FP32 increment is added in FP64, so rounding no longer accumulates in the
// stored state (the FP32 store loses ~1e-8 of a perturbation per step).
template <int NC>
struct Mix32 {
    using R = float;
    using St = double;
    using K = K32;
    static constexpr int kMinWaves = 1;
    static constexpr int kMinWaves1D = 1;
    static constexpr int kResThreads = 768;
    static constexpr int kRes2Threads = 512;
    static constexpr bool kKeepRows = true;
    static constexpr bool kSplitE = true;
    static constexpr bool kRecipes = true;
    static __device__ K make(const InstDesc& d, double dt) { return Dev32<NC>::make(d, dt); }
    static __device__ void prim(const K& k, const St* U, R* W)
    {
        R D[NC];
        for (int c = 0; c < NC; c++) D[c] = (R)U[c];
        prim32<NC>(k, D, W);
    }
    static __device__ R speed(const K& k, const R* W) { return speed32<NC>(k, W); }
    // FR: the half-step state carries the full density (HLLC faces);
    // CL: closure recipe
    template <bool FR = false, int CL = 0>
    static __device__ void predict(const K& k, const R* W, const R* sx, const R* sy, R* Wh,
                                   R act = 1)
    {
        predict32<NC, FR, CL>(k, W, sx, sy, Wh, act);
    }
    template <int RS>
    static __device__ void flux(const K& k, const R* L, const R* Rr, R* F)
    {
        flux32<NC, RS>(k, L, Rr, F);
    }
    template <bool FR = false, int CL = 0>
    static __device__ void update(const K& k, const St* Un, const R* dF, const R* dG, const R* Wh,
                                  St* Unew, R& sE, R& sV, R act = 1)
    {
        R dU[NC];
        increment32<NC, FR, CL>(k, (R)Un[NC == 5 ? 4 : 3], dF, dG, Wh, dU, sE, sV, act);
        for (int c = 0; c < NC; c++) Unew[c] = Un[c] + (St)dU[c];
    }
    static __device__ R full_rho(const K& k, R r) { return k.rho_r + r; }
    static __device__ R full_p(const K& k, R p) { return k.p_r + p; }
};

// ------------------------------------------------------ reduction records

// Per-lane accumulators of one work item: FP64 sums of the updated conserved
// values and source increments, and the extrema in the working precision.
template <class R>
struct Acc {
    double tot[5];
    double src[2];
    R smax, rmin, pmin;
};

template <class R>
__device__ __forceinline__ void acc_init(Acc<R>& a)
{
    for (int c = 0; c < 5; c++) a.tot[c] = 0.0;
    a.src[0] = a.src[1] = 0.0;
    a.smax = (R)0;
    a.rmin = (R)INFINITY;
    a.pmin = (R)INFINITY;
}

// Record one updated cell: NC conserved values (as stored), its primitives
// and signal speed, and its source increments.  The minima of rho and p are
// kept in the primitives' own form (deviations for FP32) and made full by
// acc_finish: rounding is monotone, so the minimum of the full values is the
// reference plus the minimum deviation.  A split energy slot holds E - E_nu;
// its sum is made the sum of E by acc_finish.
template <class P, int NC>
__device__ __forceinline__ void acc_cell(Acc<typename P::R>& a, const typename P::K& k,
                                         const typename P::St* U, const typename P::R* W,
                                         typename P::R s, typename P::R sE, typename P::R sV)
{
    constexpr int iE = NC == 5 ? 3 : 2, iV = NC - 1;
    a.tot[0] += (double)U[0];
    a.tot[1] += (double)U[1];
    if (NC == 5) a.tot[2] += (double)U[2];
    a.tot[3] += (double)U[iE];
    a.tot[4] += (double)U[iV];
    a.src[0] += (double)sE;
    a.src[1] += (double)sV;
    a.smax = fmax(a.smax, s);
    a.rmin = fmin(a.rmin, W[0]);
    a.pmin = fmin(a.pmin, W[NC == 5 ? 3 : 2]);
}

// Per-lane accumulators as the records expect them: the sum of E (a split
// energy slot summed E - E_nu) and full minima of rho and p.
template <class P>
__device__ __forceinline__ void acc_finish(Acc<typename P::R>& a, const typename P::K& k)
{
    if (P::kSplitE) a.tot[3] += a.tot[4];
    a.rmin = P::full_rho(k, a.rmin);
    a.pmin = P::full_p(k, a.pmin);
}

// Failure flags of a lane: a non-finite value anywhere makes its sums
// non-finite; min/max ignore NaN, so positivity is checked on the extrema.
template <class R>
__device__ __forceinline__ uint32_t acc_flags(const Acc<R>& a)
{
    double all = a.tot[0] + a.tot[1] + a.tot[2] + a.tot[3] + a.tot[4] + a.src[0] + a.src[1];
    uint32_t f = 0u;
    if (!isfinite(all)) f |= 1u;
    if (!(a.rmin > (R)0)) f |= 2u;
    if (!(a.pmin > (R)0)) f |= 4u;
    return f;
}

// Fold the lanes of each wave (lane 0 keeps a fixed-order result), then the
// waves of the workgroup in wave order, and store the workgroup's record
// (WT: with agent-scope stores, which write through to memory).
template <class R, int MaxW = kMaxWaves, bool WT = false>
__device__ __forceinline__ void block_reduce_store(Acc<R>& a, Partial* out, int wave, int lane,
                                                   int nwaves)
{
    __shared__ double sh[MaxW][11];
    __shared__ uint32_t shf[MaxW];
    uint32_t flags = acc_flags(a);
    double smax = (double)a.smax, rmin = (double)a.rmin, pmin = (double)a.pmin;
    for (int m = 32; m >= 1; m >>= 1) {
        for (int c = 0; c < 5; c++) a.tot[c] += lane_xor(a.tot[c], lane, m);
        a.src[0] += lane_xor(a.src[0], lane, m);
        a.src[1] += lane_xor(a.src[1], lane, m);
        smax = fmax(smax, lane_xor(smax, lane, m));
        rmin = fmin(rmin, lane_xor(rmin, lane, m));
        pmin = fmin(pmin, lane_xor(pmin, lane, m));
        flags |= (uint32_t)__builtin_amdgcn_ds_bpermute(((lane ^ m) & 63) << 2, (int)flags);
    }
    if (lane == 0) {
        for (int c = 0; c < 5; c++) sh[wave][c] = a.tot[c];
        sh[wave][5] = a.src[0];
        sh[wave][6] = a.src[1];
        sh[wave][7] = smax;
        sh[wave][8] = rmin;
        sh[wave][9] = pmin;
        shf[wave] = flags;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        Partial r;
        for (int c = 0; c < 5; c++) r.tot[c] = 0.0;
        r.src[0] = r.src[1] = 0.0;
        r.smax = 0.0;
        r.rho_min = INFINITY;
        r.p_min = INFINITY;
        r.flags = 0u;
        r.pad = 0u;
        for (int w = 0; w < nwaves; w++) {
            for (int c = 0; c < 5; c++) r.tot[c] += sh[w][c];
            r.src[0] += sh[w][5];
            r.src[1] += sh[w][6];
            r.smax = fmax(r.smax, sh[w][7]);
            r.rho_min = fmin(r.rho_min, sh[w][8]);
            r.p_min = fmin(r.p_min, sh[w][9]);
            r.flags |= shf[w];
        }
        if constexpr (WT) {
            auto put = [](double* p, double x) {
                __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            };
            for (int c = 0; c < 5; c++) put(&out->tot[c], r.tot[c]);
            put(&out->src[0], r.src[0]);
            put(&out->src[1], r.src[1]);
            put(&out->smax, r.smax);
            put(&out->rho_min, r.rho_min);
            put(&out->p_min, r.p_min);
            __hip_atomic_store(&out->flags, r.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            *out = r;
        }
    }
}

// Control word of a solve as seen by the kernels of one step.
struct StepCtl {
    double dt;
    int cur;
    bool active;
    const double* gsrc;   // forced source: ghost states at the step's start time
};

__device__ __forceinline__ StepCtl read_ctl(const InstCtrl& c)
{
    StepCtl s;
    double t = c.t, t_end = c.t_end;
    s.active = c.status == 0 && t < t_end && c.steps < c.max_steps;
    double dt = c.dt_cfl;
    if (t + dt > t_end) dt = t_end - t;
    s.dt = dt;
    s.cur = c.cur;
    s.gsrc = &c.src_ghost[0][0];
    return s;
}

// A forced-source ghost in the stored form: the full FP64 conserved state
// (5 components; the 1D planes skip rho v) minus the reference (zero in FP64),
// with E - E_nu in the energy slot of a split state.
template <class St, int NC, bool Split>
__device__ __forceinline__ void source_cell(const InstDesc& d, const double* g, St* U)
{
    for (int c = 0; c < NC; c++) {
        const int q = NC == 5 ? c : (c < 2 ? c : c + 1);
        U[c] = (St)(g[q] - d.uref[q]);
    }
    if (Split) U[NC == 5 ? 3 : 2] = (St)((g[3] - g[4]) - d.e1_r);
}

template <class R, int NC>
__device__ __forceinline__ void load_cell_cached(const R* __restrict__ base, int64_t ncell,
                                                 int64_t idx, R* U)
{
    for (int c = 0; c < NC; c++) U[c] = base[c * ncell + idx];
}

// ==================================================== accepting a step

// Ghost g (cell -1 - g, centre x = -h/2 - g h) of a forced source at the
// x-low end for the time t: the plane sound wave s = a sin(omega t - k x)
// about the background (section 3's forced oscillations), as conserved FP64
// values (eq. (5)).  The step kernels take it from the control block, the
// cooperative kernel computes it itself: the same arithmetic in both.
__device__ __forceinline__ void source_ghost(const InstDesc& d, double t, int g, double* U)
{
    const double x = ((double)(-1 - g) + 0.5) * d.h;
    const double s = d.src_amp * sin(d.src_omega * t - d.src_k * x);
    const double rho = d.src_rho + s;
    const double u = d.src_uc * s;
    const double v = 0.0;
    const double p = d.src_p + d.src_c2 * s;
    const double e = d.src_ev + d.src_er * s;
    U[0] = rho;
    U[1] = rho * u;
    U[2] = rho * v;
    U[3] = p / d.gm1 + 0.5 * rho * (u * u + v * v) + e;
    U[4] = e;
}

// the three ghosts for the time c.t, into the control block
__device__ __noinline__ void source_ghosts(const InstDesc& d, InstCtrl& c)
{
    for (int g = 0; g < 3; g++) source_ghost(d, c.t, g, c.src_ghost[g]);
}
// one ghost, out of line: inlined, the sine's registers would count against
// the cooperative kernel's step loop
__device__ __noinline__ void source_ghost_at(const InstDesc& d, double t, int g, double* U)
{
    source_ghost(d, t, g, U);
}

// After a cooperative launch of G workgroups of a solve (one workgroup of up to
// 256 threads): the most advanced view of the control (most steps accepted; a
// rejection over a wait that ran out at the same step) becomes the solve's
// control, with the FP64 totals and extrema of the last accepted step and the
// source budgets of every accepted step folded from the records in workgroup
// order.  A launch whose wait ran out leaves the solve stopped with
// kStatusStall.
__device__ __forceinline__ void coop_fold(const InstDesc& d, InstCtrl& c, int G,
                                          const CoopRec* recs, const CoopView* views, int nwg)
{
    __shared__ uint64_t s_key[4];
    __shared__ double sh[4][10];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    // key of a view: steps accepted, then rejection, then the lowest index
    uint64_t key = 0;
    int stall = 0;
    for (int j = t; j < G; j += blockDim.x) {
        const CoopView& a = views[j];
        const uint64_t kj = ((uint64_t)a.nacc << 33) | ((uint64_t)(a.status != 0) << 32) |
                            (uint64_t)(0xffffffffu - (uint32_t)j);
        key = kj > key ? kj : key;
        stall |= a.stalled != 0u;
    }
    stall = __syncthreads_or(stall);
    for (int m = 32; m >= 1; m >>= 1) {
        const int src = ((lane ^ m) & 63) << 2;
        const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)(uint32_t)key);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)(uint32_t)(key >> 32));
        const uint64_t o = ((uint64_t)hi << 32) | lo;
        key = o > key ? o : key;
    }
    if (lane == 0) s_key[wave] = key;
    __syncthreads();
    for (int x = 0; x < (int)(blockDim.x >> 6); x++) key = s_key[x] > key ? s_key[x] : key;
    const CoopView w = views[0xffffffffu - (uint32_t)key];
    const int p = (int)((w.nacc - 1) & 1);
    double v[10] = {0, 0, 0, 0, 0, 0, 0, 0, INFINITY, INFINITY};
    if (w.nacc > 0) {
        for (int j = t; j < G; j += blockDim.x) {
            const CoopRec& r = recs[(size_t)p * nwg + j];
            for (int q = 0; q < 5; q++) v[q] += r.tot[q];
            v[5] += r.src[0];
            v[6] += r.src[1];
            v[7] = fmax(v[7], r.smax);
            v[8] = fmin(v[8], r.rho_min);
            v[9] = fmin(v[9], r.p_min);
        }
        for (int m = 32; m >= 1; m >>= 1) {
            for (int q = 0; q < 7; q++) v[q] += lane_xor(v[q], lane, m);
            v[7] = fmax(v[7], lane_xor(v[7], lane, m));
            v[8] = fmin(v[8], lane_xor(v[8], lane, m));
            v[9] = fmin(v[9], lane_xor(v[9], lane, m));
        }
        if (lane == 0)
            for (int q = 0; q < 10; q++) sh[wave][q] = v[q];
    }
    __syncthreads();
    if (t != 0) return;
    if (w.nacc > 0) {
        for (int x = 1; x < (int)(blockDim.x >> 6); x++) {
            for (int q = 0; q < 7; q++) v[q] += sh[x][q];
            v[7] = fmax(v[7], sh[x][7]);
            v[8] = fmin(v[8], sh[x][8]);
            v[9] = fmin(v[9], sh[x][9]);
        }
        const double n = (double)d.ncell;
        for (int q = 0; q < 5; q++) c.total[q] = v[q] + n * d.uref[q];
        c.budget[0] += v[5];
        c.budget[1] += v[6];
        c.smax = v[7];
        c.rho_min = v[8];
        c.p_min = v[9];
        c.t = w.t;
        c.steps = w.steps;
        c.cur = w.cur;
        c.dt_cfl = w.dt_cfl;
        c.dt_last = w.dt_last;
        c.flags = 0u;
        if (d.bc[0] == kBcSource) source_ghosts(d, c);
    }
    // a solve that had failed before the launch keeps its status and flags
    if (c.status != 0) return;
    if (w.status != 0) {
        c.status = w.status;
        c.flags = w.flags;
    } else if (stall != 0) {
        c.status = kStatusStall;
    }
}

// The NC conserved planes of one state buffer: uniform base addresses and a
// 32-bit byte offset per cell (planes are < 4 GiB).  Coh: agent-scope loads
// and stores (the cooperative launch, where the next step's loads must see
// what workgroups on other XCDs stored: the stores write through to memory
// and the loads never take a stale line from this XCD's L2).
typedef __attribute__((address_space(1))) char gchar;

template <class R, int NC, bool Coh = false>
struct Planes {
    typedef __attribute__((address_space(1))) R gR;
    gchar* base[NC];
    __device__ Planes(uint64_t buf, int64_t ncell)
    {
        for (int c = 0; c < NC; c++) base[c] = (gchar*)(buf + (uint64_t)(c * ncell * (int64_t)sizeof(R)));
    }
    __device__ __forceinline__ void load(uint32_t boff, R* U) const
    {
        for (int c = 0; c < NC; c++) {
            if constexpr (Coh)
                U[c] = __hip_atomic_load((gR*)(base[c] + (uint64_t)boff), __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
            else
                U[c] = *(const gR*)(base[c] + (uint64_t)boff);
        }
    }
    __device__ __forceinline__ void store(uint32_t boff, const R* U) const
    {
        for (int c = 0; c < NC; c++) {
            if constexpr (Coh)
                __hip_atomic_store((gR*)(base[c] + (uint64_t)boff), U[c], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            else
                __builtin_nontemporal_store(U[c], (gR*)(base[c] + (uint64_t)boff));
        }
    }
    // a store that stays in the cache for the next step's load
    __device__ __forceinline__ void store_cached(uint32_t boff, const R* U) const
    {
        for (int c = 0; c < NC; c++) *(gR*)(base[c] + (uint64_t)boff) = U[c];
    }
};

// One 60-cell segment of the 1D MUSCL step: lane l holds the stored values Uc
// of its cell (two ghost lanes per side) and gets the cell's next values Uo,
// their primitives, signal speed and source increments (of the middle lanes).
template <class P, int RS, int CL>
__device__ __forceinline__ void seg1d(const typename P::K& k, const typename P::St* Uc,
                                      typename P::St* Uo, typename P::R* Wn, typename P::R& s,
                                      typename P::R& sE, typename P::R& sV)
{
    using R = typename P::R;
    constexpr int NC = 4;
    constexpr bool FR = RS == 0;
    R W[NC + 1], sx[NC], h[NC];
    P::prim(k, Uc, W);
    for (int c = 0; c < NC; c++) {
        R l = from_left(W[c]), r = from_right(W[c]);
        R a = W[c] - l, b = r - W[c];
        pin(a);
        pin(b);
        sx[c] = minmod(a, b);
    }
    P::template predict<FR, CL>(k, W, sx, sx, h);
    R E[NC], Wr[NC], Fx[NC], dF[NC];
    for (int c = 0; c < NC; c++) {
        E[c] = face(h[c], sx[c]);
        Wr[c] = from_right(face(h[c], -sx[c]));
    }
    P::template flux<RS>(k, E, Wr, Fx);
    for (int c = 0; c < NC; c++) {
        dF[c] = Fx[c] - from_left(Fx[c]);
        pin(dF[c]);
    }
    P::template update<FR, CL>(k, Uc, dF, dF, h, Uo, sE, sV);
    P::prim(k, Uo, Wn);
    s = P::speed(k, Wn);
}

// The run-constant geometry of the CSPH-TVD step: the cell size, its rounded
// reciprocal, the kernel's factor and its gradients at +-h (the predictor's
// particles sit at the centres).
struct CsphGrid {
    double h, ih, wn, g1, g2;
};
__device__ __forceinline__ CsphGrid csph_grid(const InstDesc& d)
{
    CsphGrid g;
    g.h = d.h;
    g.ih = d.ih;
    g.wn = 2.0 / (3.0 * (g.h * g.h));
    g.g1 = csph_grad_w(g.h, g.h, g.ih, g.wn);
    g.g2 = csph_grad_w(-g.h, g.h, g.ih, g.wn);
    return g;
}

// One 58-cell segment of the CSPH-TVD step (section 2.3): lane l holds the
// particle of its cell, Un (three ghost lanes per side).  Neighbours are one
// lane away, so each stage is one DPP shift per quantity:
//   predictor (eq. (10)) on lanes 1..62: U* = U^n + dt Y(U^n), xi* = dt (u^n +
//     u*)/2, with every particle at its cell centre;
//   corrector (eq. (11)) on lanes 2..61: U~ = (U^n + U*)/2 + dt/2 Y(U*, xi*),
//     xi~ = xi*/2 + dt/2 (u^n + u~)/2;
//   face j+1/2 on lanes 2..60: HLL (eq. (13)) between U^L = U^{n+1/2}_j +
//     (h - xi~_j) Theta_j / 2 and U^R = U^{n+1/2}_{j+1} - (h + xi~_{j+1})
//     Theta_{j+1} / 2 (eq. (14)), U^{n+1/2} = (U^n + U~)/2;
//   update (eq. (9)) on lanes 3..60: U^{n+1} = U~ - dt/h (F_{j+1/2} - F_{j-1/2}).
template <int CL>
__device__ __forceinline__ void seg_csph(const K64& k, const CsphGrid& g, const double* Un,
                                         double* Uo, double* Wn, double& s, double& sE, double& sV)
{
    constexpr int NC = 4;
    const double h = g.h, ih = g.ih, wn = g.wn, g1 = g.g1, g2 = g.g2;
    const double dt = k.dt, hdt = k.hdt, dtdx = k.dtdx;
    // predictor
    double un, pn, phin, yn;
    csph_prim(k, Un, un, pn, phin, yn);
    double Y[NC], sEp, sVp, sEc, sVc;
    csph_y<CL>(k, h, g1, g2, from_left(phin), from_left(un), from_right(phin), from_right(un),
               Un[0], yn, un, pn, Un[3], phin, Y, sEp, sVp);
    double Us[NC];
    for (int c = 0; c < NC; c++) Us[c] = Un[c] + dt * Y[c];
    double us, ps, phis, ys;
    csph_prim(k, Us, us, ps, phis, ys);
    const double xs = dt * (0.5 * (un + us));
    // corrector, at the predicted positions
    const double ga = csph_grad_w(h + (xs - from_left(xs)), h, ih, wn);
    const double gb = csph_grad_w(-h + (xs - from_right(xs)), h, ih, wn);
    csph_y<CL>(k, h, ga, gb, from_left(phis), from_left(us), from_right(phis), from_right(us),
               Us[0], ys, us, ps, Us[3], phis, Y, sEc, sVc);
    double Ut[NC];
    for (int c = 0; c < NC; c++) Ut[c] = 0.5 * (Un[c] + Us[c]) + hdt * Y[c];
    const double ut = div64(Ut[1], Ut[0]);
    const double xt = 0.5 * xs + hdt * (0.5 * (un + ut));
    // face j+1/2: this particle's profile gives U^L, the right neighbour's U^R
    const double al = 0.5 * (h - xt), ar = 0.5 * (h + xt);
    double UL[NC], UR[NC], F[NC];
    for (int c = 0; c < NC; c++) {
        const double l = from_left(Un[c]), r = from_right(Un[c]);
        double a = Un[c] - l, b = r - Un[c];
        pin(a);
        pin(b);
        const double th = quot64(minmod(a, b), h, ih);
        const double hl = 0.5 * (Un[c] + Ut[c]);
        UL[c] = hl + al * th;
        UR[c] = from_right(hl - ar * th);
    }
    csph_flux(k, UL, UR, F);
    for (int c = 0; c < NC; c++) {
        double dF = F[c] - from_left(F[c]);
        pin(dF);
        Uo[c] = Ut[c] - dtdx * dF;
    }
    prim64<NC>(k, Uo, Wn);
    s = speed64<NC>(k, Wn);
    sE = hdt * sEp + hdt * sEc;
    sV = hdt * sVp + hdt * sVc;
}

}  // namespace ng
