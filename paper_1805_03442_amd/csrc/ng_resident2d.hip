// ng_resident2d.hip -- the cooperative path of the 2D MUSCL step: one launch
// advances a grid through many steps.
//
// The grid is dealt to the waves of G workgroups that stay resident together,
// each a strip (60 columns) by a run of rows.  The state stays in the
// two state buffers; loads and stores are agent-scope (a step's loads must see
// what workgroups on other XCDs stored), and a wave's stores have reached memory
// before its workgroup publishes the step's signal speed.  All workgroups then
// take the next dt of eq. (16) alike (ng_exchange.hpp).  A grid alone in one
// workgroup (60x4 at most) needs none of that and has a form of its own (Coh =
// false): us per step at 60x4 and, in the others' form, at 48x40 and 600^2, FP32,
// 2.79, 3.98, 8.62; with one form whose exchange a test skips 2.88, 4.03, 8.68;
// with one form that always exchanges 3.53, 3.98, 8.62.
//
// It replaces two launches per step (the step and its acceptance) on grids that
// do not fill the chip for long: kCoopCells in ng_api.cpp says where the line
// lies and what both cost.
//
// Per-cell arithmetic, t and dt follow the step kernels and the finalize kernel
// operation for operation, so the state, t and dt are bitwise those of one
// launch per step; only the summation order of the FP64 totals differs.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "ng_exchange.hpp"
#include "ng_launch.hpp"
#include "ng_march2d.hpp"

namespace ng {

// every store of this wave has reached memory
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// S: 0..2 the periodic HLLC step with closure recipe S (0: general), 3 the HLLC
// step with any ends and the general closures, 4 the same with recipe 3 (FP64),
// 5 the HLL step with any ends.
template <class P, int S, bool Coh>
__global__ void __launch_bounds__(P::kRes2Threads) run_resident2d_kernel(
    const InstDesc* __restrict__ descs, const InstCtrl* __restrict__ ctrls, int inst, int chunks,
    const uint32_t* __restrict__ base, uint64_t* __restrict__ slots, CoopRec* __restrict__ recs,
    CoopView* __restrict__ views, int32_t nwg, int64_t nsteps, int32_t spin_limit)
{
    using R = typename P::R;
    using St = typename P::St;
    // (two rows more in flight pay in FP32 on periodic grids, 600^2 9.4 to 8.9 us
    // per step; the mixed step loses 8 % at 1024^2, the FP64 step has no registers)
    constexpr int NC = 5, kRing = std::is_same<P, Dev32<5>>::value && S <= 2 ? 6 : 4;
    const InstDesc& d = descs[inst];
    const InstCtrl& c = ctrls[inst];
    const uint32_t G = gridDim.x, b = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nw = blockDim.x >> 6, tid = threadIdx.x;
    const uint32_t gen0 = *base;
    __shared__ double s_sum[kCoopMaxWaves][10];
    __shared__ double s_sm[kCoopMaxWaves];
    __shared__ uint32_t s_fl[kCoopMaxWaves];
    __shared__ ResCtl s_c;
    __shared__ double s_gsrc[2][5];   // a forced source's ghosts
    // this wave's share: chunk g % chunks of the rows of strip g / chunks
    const int g = (int)b * nw + wave;
    const int strip = g / chunks, chunk = g % chunks;
    const int64_t ny = d.ny;
    const bool work = strip < d.nstrips;
    const int r0 = (int)(chunk * ny / chunks), r1 = (int)((chunk + 1) * ny / chunks);
    const int cur0 = c.cur;
    if (tid == 0) s_c.start(c);
    __syncthreads();
    const bool src = S >= 3 && d.bc[0] == kBcSource;
    const double* gsrc = &s_gsrc[0][0];
    if (src) {
        if (tid < 2) source_ghost_at(d, s_c.t, tid, s_gsrc[tid]);
        __syncthreads();
    }
    // Per lane, the sums of the last computed step (acc) and the source
    // increments of every accepted step (bud).
    Acc<R> acc;
    acc_init(acc);
    double bud0 = 0.0, bud1 = 0.0;
    int st = 0;
    for (; st < (int)nsteps && s_c.go; st++) {
        const uint32_t gen = gen0 + 1u + (uint32_t)st;
        const typename P::K k = P::make(d, s_c.dt);
        const double t_new = src ? s_c.t + s_c.dt : 0.0;   // where the step leads
        const int cur = cur0 ^ (st & 1);
        acc_init(acc);
        if (work && r0 < r1) {
            if constexpr (S <= 2)
                march2d<P, 0, false, S, Coh, kRing>(d, k, cur, gsrc, strip, r0, r1, lane, acc);
            else
                march2d<P, S == 5 ? 1 : 0, true, S == 4 ? 3 : 0, Coh, kRing>(d, k, cur, gsrc, strip, r0, r1,
                                                                     lane, acc);
        }
        acc_finish<P>(acc, k);
        {
            const double sm = wave_max((double)acc.smax);
            const uint32_t fl = wave_flags(acc_flags(acc));
            if (lane == 0) {
                s_sm[wave] = sm;
                s_fl[wave] = fl;
            }
        }
        if constexpr (Coh) stores_done();
        __syncthreads();
        if (wave == 0) {
            double m = wave_max(lane < nw ? s_sm[lane] : 0.0);
            uint32_t f = wave_flags(lane < nw ? s_fl[lane] : 0u);
            bool out = false;
            if constexpr (Coh)
                out = exchange_slots<R>(slots + (size_t)(st & 1) * nwg * kResSlot, G, b, gen, lane,
                                        spin_limit, m, f);
            if (lane == 0) s_c.decide(d, c, out, m, f);
        } else if (wave == 1 && src && lane < 2) {
            // a forced source's ghosts for the time the step leads to (every
            // wave has marched this step)
            source_ghost_at(d, t_new, lane, s_gsrc[lane]);
        }
        __syncthreads();
        if (s_c.ok) {
            bud0 += acc.src[0];
            bud1 += acc.src[1];
        }
    }
    // the last computed step, and whether this workgroup saw it accepted
    const int st_c = st - 1, nacc = s_c.nacc;
    const bool cur_ok = s_c.ok != 0;
    if (st_c >= 0) {
        auto put = [&](double b0, double b1, int step) {
            put_record(acc, b0, b1, step, recs + (size_t)(step & 1) * nwg + b, s_sum, wave, lane, nw);
        };
        if (cur_ok) {
            put(bud0, bud1, st_c);
        } else {
            put(bud0 + acc.src[0], bud1 + acc.src[1], st_c);
            if (st_c >= 1) {
                // the sums of the accepted state, from its cells
                const typename P::K k = P::make(d, 0.0);
                const Planes<St, NC, Coh> pl(d.buf[cur0 ^ (nacc & 1)], d.ncell);
                const int x0 = strip * kInterior;
                const int w = (int)d.nx - x0 < kInterior ? (int)d.nx - x0 : kInterior;
                acc_init(acc);
                for (int r = r0; work && r < r1 && lane < w; r++) {
                    St U[NC];
                    R Wn[NC + 1];
                    pl.load((uint32_t)(((int64_t)r * d.nx + x0 + lane) * (int64_t)sizeof(St)), U);
                    P::prim(k, U, Wn);
                    acc_cell<P, NC>(acc, k, U, Wn, P::speed(k, Wn), (R)0, (R)0);
                }
                acc_finish<P>(acc, k);
                put(bud0, bud1, st_c - 1);
            }
        }
    }
    if (tid == 0) s_c.view(cur0, views[b]);
}

// ================================================================ launchers

template <template <int> class Pol, bool Coh>
static const void* kernel2d_of(int s)
{
    using P = Pol<5>;
    switch (s) {
    case 0: return (const void*)run_resident2d_kernel<P, 0, Coh>;
    case 1: return (const void*)run_resident2d_kernel<P, 1, Coh>;
    case 2: return (const void*)run_resident2d_kernel<P, 2, Coh>;
    case 3: return (const void*)run_resident2d_kernel<P, 3, Coh>;
    case 5: return (const void*)run_resident2d_kernel<P, 5, Coh>;
    default: break;
    }
    if constexpr (std::is_same<typename P::K, K64>::value)
        if (s == 4) return (const void*)run_resident2d_kernel<P, 4, Coh>;
    return nullptr;
}

static const void* kernel2d_of(int prec, int s, bool coh)
{
    if (prec == 0) return coh ? kernel2d_of<Plain64, true>(s) : kernel2d_of<Plain64, false>(s);
    if (prec == 1) return coh ? kernel2d_of<Dev32, true>(s) : kernel2d_of<Dev32, false>(s);
    if (prec == 2) return coh ? kernel2d_of<Mix32, true>(s) : kernel2d_of<Mix32, false>(s);
    return nullptr;
}

int resident2d_max_waves(int prec)
{
    return (prec == 0 ? Plain64<5>::kRes2Threads
                      : (prec == 1 ? Dev32<5>::kRes2Threads : Mix32<5>::kRes2Threads)) / kWave;
}

hipError_t resident2d_capacity(int prec, int s, bool coh, int waves, int* blocks_per_cu)
{
    const void* k = kernel2d_of(prec, s, coh);
    if (!k || waves < 2 || waves > resident2d_max_waves(prec)) return hipErrorInvalidValue;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k, waves * kWave, 0);
}

hipError_t launch_resident2d(int prec, int s, const InstDesc* descs, InstCtrl* ctrls, int inst,
                             const ResSync& sync, int grid, int chunks, int waves, int64_t nsteps,
                             int32_t spin_limit, hipStream_t st)
{
    const void* k = kernel2d_of(prec, s, grid > 1);
    // (grid * waves covers strips * chunks: waves beyond them idle)
    if (!k || grid < 1 || grid > sync.nwg || grid > kCoopFlat || chunks < 1 || waves < 2 ||
        waves > resident2d_max_waves(prec) || nsteps < 1 || nsteps > kCoopMaxSteps || spin_limit < 0)
        return hipErrorInvalidValue;
    void* args[] = {(void*)&descs,     (void*)&ctrls,      (void*)&inst,
                    (void*)&chunks,    (void*)&sync.base,  (void*)&sync.slots,
                    (void*)&sync.recs, (void*)&sync.views, (void*)&sync.nwg,
                    (void*)&nsteps,    (void*)&spin_limit};
    return hipLaunchCooperativeKernel(k, dim3((unsigned)grid), dim3((unsigned)(waves * kWave)), args,
                                      0, st);
}

}  // namespace ng
