// ng_resident.hip -- the cooperative path of the 1D steps: one launch advances
// a solve, or many solves side by side, through many steps (MUSCL, eq. (15), or
// CSPH-TVD, section 2.3).
//
// A solve's cells are dealt to G workgroups that stay resident together, each
// one run of consecutive segments, and a workgroup keeps its cells in LDS (160
// KB per CU: 4900 FP32 or 2400 FP64 cells with the two copies a step needs) for
// the whole launch.  A step then moves no state through memory: its latency is
// the arithmetic of the segments, one exchange and two workgroup barriers.
// The exchange carries what the others need and nothing else: each workgroup
// writes its largest signal speed and failure flags, and its first and last
// two (CSPH-TVD: three) cells, as 8-byte words (step number << 32 | 32 bits of
// payload) in device memory.  A reader that sees the step number in a word has
// its payload, so no ordering between words, no cache write-back and no wait
// for stores is needed.  One wave polls the speeds of all the solve's
// workgroups and takes the next dt of eq. (16), alike in each; a second wave
// polls the neighbours' edge cells, or fills the ghosts of a domain end.
// A solve too large for LDS keeps its cells in the two state buffers instead
// (InLds = false): each workgroup still reads and writes only its own cells
// there, so plain cached loads and stores serve, and the edges travel as above.
//
// What it measured (us per step; before: a kernel that kept the state in memory,
// with agent-scope loads and stores, and met at a barrier of 24-byte messages):
//   cells            200        1024       16384      2^17       2^20
//   FP32          2.81 1.35   2.92 2.18  3.27 2.48  5.37 3.68  11.97 8.7
//   FP64          5.46 1.96   5.60 2.85  5.90 3.27 11.03 5.75  40.2  22.6
//   CSPH-TVD      6.02 2.1    6.19 3.2   6.67 3.6  12.5  6.6   47.0  27
// (the FP64 rows with the new divisions too; 2^20 FP64 cells are beyond LDS).
// What is left at 200 cells is one segment's chain of dependent operations, at
// 2^20 the vector ALUs (5.7 segments per wave, three waves per SIMD).
//
// Per-cell arithmetic, t and dt follow the step kernels and the finalize kernel
// operation for operation, so the state, t and dt are bitwise those of one
// launch per step; only the summation order of the FP64 totals differs.  Those
// sums never cross the barrier: each lane keeps those of its last computed
// step, each workgroup folds them into its records when the launch ends, and resident_after_kernel folds the records of the last
// accepted step into the control block.
//
// Every wait is bounded by spin_limit polls: a workgroup whose wait runs out
// leaves, the others leave when their own next wait runs out, and the solve
// keeps the last step a barrier accepted.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "ng_device.hpp"
#include "ng_exchange.hpp"
#include "ng_launch.hpp"

namespace ng {

// One cell as LDS holds it: its components side by side, so that a lane loads
// or stores it in one or two 16-byte operations.
template <class St>
struct alignas(16) ResCell {
    St u[4];
};

// S: 0..3 the HLLC step with closure recipe S (0: general), 4 the HLL step,
// 5 and 6 the CSPH-TVD step with the general closures and recipe 1.
// groups/refs: the launch's solves and the (group, local workgroup) of each
// workgroup; null: one solve, `one`.
// T: largest workgroup.  The FP64 kernels with calls or both HLL sides spill at
// the 168 registers that twelve waves leave, so they have a form for eight.
template <class P, int S, bool InLds, int T>
__global__ void __launch_bounds__(T) run_resident_kernel(
    const InstDesc* __restrict__ descs, const InstCtrl* __restrict__ ctrls,
    const ResGroup* __restrict__ groups, const BlockRef* __restrict__ refs, ResGroup one,
    const uint32_t* __restrict__ base, uint64_t* __restrict__ slots, uint64_t* __restrict__ edges,
    CoopRec* __restrict__ recs, CoopView* __restrict__ views, int32_t nwg, int64_t nsteps,
    int32_t spin_limit)
{
    using R = typename P::R;
    using St = typename P::St;
    constexpr bool csph = S >= 5;
    constexpr int NC = 4, H = csph ? kCsphHalo : kHalo, W = kWave - 2 * H;
    constexpr int CL = S < 4 ? S : (S == 6 ? 1 : 0), RS = S == 4 ? 1 : 0;
    constexpr int kHalves = (int)sizeof(St) / 4;     // 32-bit payloads per value
    constexpr int kSide = H * NC * kHalves;          // edge words per side
    static_assert(2 * kSide <= kWave && kSide <= kResEdge, "one wave exchanges both edges");

    const BlockRef ref = refs ? refs[blockIdx.x] : BlockRef{0, (int32_t)blockIdx.x};
    const ResGroup gr = groups ? groups[ref.inst] : one;
    const InstDesc& d = descs[gr.inst];
    const InstCtrl& c = ctrls[gr.inst];
    const uint32_t G = (uint32_t)gr.G, b = (uint32_t)ref.local;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nw = blockDim.x >> 6, tid = threadIdx.x, nthr = blockDim.x;
    const uint32_t gen0 = *base;

    extern __shared__ __align__(16) unsigned char dyn[];
    __shared__ double s_sum[kCoopMaxWaves][10];
    __shared__ double s_sm[kCoopMaxWaves];
    __shared__ uint32_t s_fl[kCoopMaxWaves];
    __shared__ ResCtl s_c;
    __shared__ int s_edge_out;        // the wait for the edges ran out
    __shared__ double s_gsrc[3][5];   // a forced source's ghosts
    // cells of this workgroup: segments [g0, g1), cells [c0, c0 + len)
    const int64_t n = d.nx;
    const int g0 = (int)((int64_t)b * d.nstrips / G), g1 = (int)((int64_t)(b + 1) * d.nstrips / G);
    const int64_t c0 = (int64_t)g0 * W;
    const int len = (int)((int64_t)g1 * W < n ? (int64_t)(g1 - g0) * W : n - c0);
    const int f0 = wave * (g1 - g0) / nw, f1 = (wave + 1) * (g1 - g0) / nw;

    // Storage.  In LDS: two copies of the cells with H ghosts per side, copy q
    // at q * pitch, cell c0 + i at H + i.  Else only the ghosts are there, H per
    // side and copy, and the cells are in the state buffers.
    ResCell<St>* lds = (ResCell<St>*)dyn;
    const int pitch = InLds ? gr.pitch : 2 * H;
    const int cur0 = c.cur;
    const Planes<St, NC> pl0(d.buf[cur0], n), pl1(d.buf[cur0 ^ 1], n);
    // the LDS slot of ghost i (0..H-1: left, H..2H-1: right) of copy q, and of
    // the edge cell of the workgroup that neighbour's ghost i holds
    auto ghost_at = [&](int q, int i) -> ResCell<St>& {
        return lds[q * pitch + (InLds && i >= H ? len + i : i)];
    };
    // a cell's value by its index in [0, len), from copy q
    auto own = [&](int q, int i, St* U) {
        if constexpr (InLds) {
            const ResCell<St> t = lds[q * pitch + H + i];
            for (int x = 0; x < NC; x++) U[x] = t.u[x];
        } else {
            (q ? pl1 : pl0).load((uint32_t)((c0 + i) * (int64_t)sizeof(St)), U);
        }
    };

    const bool src = d.bc[0] == kBcSource;
    // neighbours of this workgroup; ends without one have ghosts by the
    // boundary rule (a lone workgroup's periodic ghosts too)
    const bool periodic = d.bc[0] == kBcPeriodic;
    const bool has_l = G > 1u && (b > 0u || periodic), has_r = G > 1u && (b + 1u < G || periodic);
    const uint32_t nb_l = (uint32_t)gr.first + (b > 0u ? b - 1u : G - 1u);
    const uint32_t nb_r = (uint32_t)gr.first + (b + 1u < G ? b + 1u : 0u);
    const uint32_t me = (uint32_t)gr.first + b;

    if (tid == 0) {
        s_c.start(c);
        s_edge_out = 0;
    }
    __syncthreads();
    // copy 0 from the state buffer, ghosts by the boundary rule
    if (s_c.go) {
        if (src && tid < H) source_ghost_at(d, s_c.t, tid, s_gsrc[tid]);
        __syncthreads();
        auto fetch = [&](int64_t j, ResCell<St>& out) {
            bool flip;
            const int64_t x = axis_cell(j, n, d.bc[0], d.bc[1], flip);
            St U[NC];
            pl0.load((uint32_t)(x * (int64_t)sizeof(St)), U);
            if (flip) U[1] = -U[1];
            if (src && j < 0) source_cell<St, NC, P::kSplitE>(d, s_gsrc[-1 - j], U);
            for (int x2 = 0; x2 < NC; x2++) out.u[x2] = U[x2];
        };
        if constexpr (InLds) {
            for (int i = tid; i < len + 2 * H; i += nthr) fetch(c0 - H + i, lds[i]);
        } else {
            if (tid < 2 * H) fetch(tid < H ? c0 - H + tid : c0 + len + tid - H, ghost_at(0, tid));
        }
        __syncthreads();
    }

    CsphGrid cg{};
    if constexpr (csph) cg = csph_grid(d);
    // Per lane, the sums of the last computed step (acc) and the source
    // increments of every accepted step (bud); they are folded into the
    // workgroup's records once, when the launch ends, not at every step.
    Acc<R> acc;
    acc_init(acc);
    double bud0 = 0.0, bud1 = 0.0;
    int st = 0;

    for (; st < (int)nsteps && s_c.go; st++) {
        const uint32_t gen = gen0 + 1u + (uint32_t)st;
        const int q = st & 1;   // U^n is in copy q
        const typename P::K k = P::make(d, s_c.dt);
        const double t_new = src ? s_c.t + s_c.dt : 0.0;   // where the step leads
        acc_init(acc);
        // this wave's segments; the next segment's cells are fetched before
        // the current one is computed
        if (f0 < f1) {
            const Planes<St, NC>& src_pl = q ? pl1 : pl0;
            const Planes<St, NC>& dst_pl = q ? pl0 : pl1;
            auto get = [&](int sg, St* U) {
                const int i = sg * W + lane;     // cell c0 - H + i
                if constexpr (InLds) {
                    const ResCell<St> v = lds[q * pitch + (i < len + 2 * H ? i : len + 2 * H - 1)];
                    for (int x = 0; x < NC; x++) U[x] = v.u[x];
                } else {
                    const int j = i < H ? 0 : (i < H + len ? i - H : len - 1);
                    src_pl.load((uint32_t)((c0 + j) * (int64_t)sizeof(St)), U);
                }
            };
            auto seg = [&](int sg, St* Uc, St* Ux) {
                get(sg + 1 < f1 ? sg + 1 : sg, Ux);
                const int i = sg * W + lane;
                if constexpr (!InLds) {
                    // ghosts of the workgroup's ends come from LDS (the right
                    // ones may reach into the last segment but one)
                    if (i < H || i >= H + len) {
                        const int gi = i < H ? i : i - len;
                        const ResCell<St> v = lds[q * pitch + (gi < 2 * H ? gi : 2 * H - 1)];
                        for (int x = 0; x < NC; x++) Uc[x] = v.u[x];
                    }
                }
                St Uo[NC];
                R Wn[NC + 1], sp, sE, sV;
                if constexpr (csph)
                    seg_csph<CL>(k, cg, Uc, Uo, Wn, sp, sE, sV);
                else
                    seg1d<P, RS, CL>(k, Uc, Uo, Wn, sp, sE, sV);
                if (lane >= H && lane < kWave - H && i < H + len) {
                    if constexpr (InLds) {
                        ResCell<St> v;
                        for (int x = 0; x < NC; x++) v.u[x] = Uo[x];
                        lds[(q ^ 1) * pitch + i] = v;
                    } else {
                        dst_pl.store_cached((uint32_t)((c0 + i - H) * (int64_t)sizeof(St)), Uo);
                    }
                    acc_cell<P, NC>(acc, k, Uo, Wn, sp, sE, sV);
                }
            };
            St UA[NC], UB[NC];
            get(f0, UA);
            int sg = f0;
            for (; sg + 1 < f1; sg += 2) {
                seg(sg, UA, UB);
                seg(sg + 1, UB, UA);
            }
            if (sg < f1) seg(sg, UA, UB);
        }
        acc_finish<P>(acc, k);
        // the exchange needs only the signal speed and the failure flags
        {
            const double sm = wave_max((double)acc.smax);
            const uint32_t fl = wave_flags(acc_flags(acc));
            if (lane == 0) {
                s_sm[wave] = sm;
                s_fl[wave] = fl;
            }
        }
        __syncthreads();
        if (wave == 0) {
            double m = wave_max(lane < nw ? s_sm[lane] : 0.0);
            uint32_t f = wave_flags(lane < nw ? s_fl[lane] : 0u);
            bool out = false;
            if (G > 1u) {
                out = exchange_slots<R>(slots + ((size_t)q * nwg + gr.first) * kResSlot, G, b, gen,
                                        lane, spin_limit, m, f);
            }
            if (lane == 0) s_c.decide(d, c, out, m, f);
        } else if (wave == 1) {
            // Ghosts of the next step, copy q ^ 1.  Lane w of a side carries
            // 32 bits of one value of one edge cell: it publishes this
            // workgroup's, and takes the neighbour's (or the boundary rule's)
            // into the ghosts.
            const int side = lane >= kSide ? 1 : 0, w = lane - side * kSide;
            const bool mine = lane < 2 * kSide;
            const int g = w / (NC * kHalves), x = (w / kHalves) % NC, hf = w % kHalves;
            auto half_of = [&](int i) -> uint32_t {
                if constexpr (InLds) {
                    return ((const uint32_t*)&lds[(q ^ 1) * pitch + H + i].u[x])[hf];
                } else {
                    St U[NC];
                    own(q ^ 1, i, U);
                    uint32_t r = 0;
                    for (int y = 0; y < NC; y++)
                        if (y == x) {
                            uint32_t bits[kHalves];
                            __builtin_memcpy(bits, &U[y], sizeof(St));
                            r = kHalves == 2 && hf ? bits[kHalves - 1] : bits[0];
                        }
                    return r;
                }
            };
            bool out = false;
            if (G > 1u && mine) {
                const uint32_t v = half_of(side ? len - H + g : g);
                __hip_atomic_store(edges + (((size_t)q * nwg + me) * 2 + side) * kResEdge + w,
                                   ((uint64_t)gen << 32) | v, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            const bool take = mine && (side ? has_r : has_l);
            uint32_t v = 0;
            if (mine && !take) {
                const int kind = d.bc[side];
                const int i = kind == kBcPeriodic ? (side ? g : len - H + g)
                              : kind == kBcWall   ? (side ? len - 1 - g : H - 1 - g)
                                                  : (side ? len - 1 : 0);
                v = half_of(i);
                if (kind == kBcWall && x == 1 && hf == kHalves - 1) v ^= 0x80000000u;
            }
            const uint64_t* const from =
                edges + (((size_t)q * nwg + (side ? nb_r : nb_l)) * 2 + (side ? 0 : 1)) * kResEdge + w;
            if (G > 1u)
                for (int32_t it = 0;; it++) {
                    uint64_t word = (uint64_t)gen << 32;
                    if (take)
                        word = __hip_atomic_load(from, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const bool have = (uint32_t)(word >> 32) == gen;
                    if (__builtin_amdgcn_ballot_w64(!have) == 0ull) {
                        if (take) v = (uint32_t)word;
                        break;
                    }
                    if (it >= spin_limit) {
                        out = true;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            if (mine && !(src && side == 0 && !has_l))
                ((uint32_t*)&ghost_at(q ^ 1, side * H + g).u[x])[hf] = v;
            if (out && lane == 0) s_edge_out = 1;
        } else if (wave == 2 && src && b == 0u && lane < H) {
            // a forced source's ghosts for the time the step leads to
            source_ghost_at(d, t_new, lane, s_gsrc[lane]);
            St U[NC];
            source_cell<St, NC, P::kSplitE>(d, s_gsrc[lane], U);
            for (int x = 0; x < NC; x++) ghost_at(q ^ 1, H - 1 - lane).u[x] = U[x];
        }
        __syncthreads();
        if (s_edge_out) break;
        if (s_c.ok) {
            bud0 += acc.src[0];
            bud1 += acc.src[1];
        }
    }
    // st_c: the last computed step; cur_ok: this workgroup saw it accepted.
    // (Edges that did not come stop the workgroup like slots that did not, but
    // with the step accepted: its next one is what it cannot compute.)
    const int nacc = s_c.nacc;
    const bool cur_ok = s_c.ok != 0;
    const int st_c = s_edge_out ? st : st - 1;
    if (s_edge_out && cur_ok) {
        bud0 += acc.src[0];
        bud1 += acc.src[1];
    }
    const bool stalled = s_c.stalled != 0;
    auto put_rec = [&](const Acc<R>& a, double b0, double b1, int step) {
        put_record(a, b0, b1, step, recs + (size_t)(step & 1) * nwg + me, s_sum, wave, lane, nw);
    };
    if (st_c >= 0) {
        if (cur_ok) {
            put_rec(acc, bud0, bud1, st_c);
        } else {
            put_rec(acc, bud0 + acc.src[0], bud1 + acc.src[1], st_c);
            if (st_c >= 1) {
                // the sums of the accepted state, from its cells
                const typename P::K k = P::make(d, 0.0);
                acc_init(acc);
                for (int i = tid; i < len; i += nthr) {
                    St U[NC];
                    R Wn[NC + 1];
                    own(nacc & 1, i, U);
                    P::prim(k, U, Wn);
                    acc_cell<P, NC>(acc, k, U, Wn, P::speed(k, Wn), (R)0, (R)0);
                }
                acc_finish<P>(acc, k);
                put_rec(acc, bud0, bud1, st_c - 1);
            }
        }
    }
    // The state: U after a accepted steps goes to the buffer of parity a.  A
    // workgroup whose wait ran out does not know whether the others accepted
    // its last computed step, so it leaves that one too (in the other buffer);
    // after zero accepted steps buffer 0 still holds the start.
    if constexpr (InLds) {
        auto dump = [&](int a) {
            const Planes<St, NC>& pl = (a & 1) ? pl1 : pl0;
            for (int i = tid; i < len; i += nthr) {
                const ResCell<St> v = lds[(a & 1) * pitch + H + i];
                St U[NC];
                for (int x = 0; x < NC; x++) U[x] = v.u[x];
                pl.store((uint32_t)((c0 + i) * (int64_t)sizeof(St)), U);
            }
        };
        if (nacc > 0) dump(nacc);
        if (stalled) dump(nacc + 1);
    }
    // and its view of the control
    if (tid == 0) {
        if (s_edge_out) s_c.stalled = 1;
        s_c.view(cur0, views[me]);
    }
}

// One workgroup per solve of a resident launch (coop_fold); the first moves
// the step number on past every number this launch can have used.
__global__ void __launch_bounds__(256) resident_after_kernel(const InstDesc* __restrict__ descs,
                                                             InstCtrl* __restrict__ ctrls,
                                                             const ResGroup* __restrict__ groups,
                                                             ResGroup one,
                                                             const CoopRec* __restrict__ recs,
                                                             const CoopView* __restrict__ views,
                                                             int32_t nwg,
                                                             uint32_t* __restrict__ base,
                                                             uint32_t nsteps)
{
    const ResGroup gr = groups ? groups[blockIdx.x] : one;
    coop_fold(descs[gr.inst], ctrls[gr.inst], gr.G, recs + gr.first, views + gr.first, nwg);
    if (blockIdx.x == 0 && threadIdx.x == 0) *base += nsteps + 1u;
}

// ================================================================ launchers

template <template <int> class Pol, bool InLds, int T>
static const void* kernel_of(int s)
{
    using P = Pol<4>;
    switch (s) {
    case 0: return (const void*)run_resident_kernel<P, 0, InLds, T>;
    case 4: return (const void*)run_resident_kernel<P, 4, InLds, T>;
    default: break;
    }
    if constexpr (T == P::kResThreads) {
        if (s == 1) return (const void*)run_resident_kernel<P, 1, InLds, T>;
        if (s == 2) return (const void*)run_resident_kernel<P, 2, InLds, T>;
    }
    if constexpr (std::is_same<typename P::K, K64>::value) {
        if (s == 5) return (const void*)run_resident_kernel<P, 5, InLds, T>;
        if constexpr (T == P::kResThreads) {
            if (s == 3) return (const void*)run_resident_kernel<P, 3, InLds, T>;
            if (s == 6) return (const void*)run_resident_kernel<P, 6, InLds, T>;
        }
    }
    return nullptr;
}

// (FP64, up to eight waves: the form with registers to spare where there is one)
template <template <int> class Pol>
static const void* kernel_of(int s, bool lds, int waves)
{
    constexpr int T = Pol<4>::kResThreads;
    if constexpr (std::is_same<typename Pol<4>::K, K64>::value)
        if (waves <= kResEight && (s == 0 || s == 4 || s == 5))
            return lds ? kernel_of<Pol, true, kResEight * kWave>(s)
                       : kernel_of<Pol, false, kResEight * kWave>(s);
    return lds ? kernel_of<Pol, true, T>(s) : kernel_of<Pol, false, T>(s);
}

static const void* kernel_of(int prec, int s, bool lds, int waves)
{
    if (prec == 0) return kernel_of<Plain64>(s, lds, waves);
    if (prec == 1) return kernel_of<Dev32>(s, lds, waves);
    if (prec == 2) return kernel_of<Mix32>(s, lds, waves);
    return nullptr;
}

int resident_max_waves(int prec)
{
    return (prec == 0 ? Plain64<4>::kResThreads
                      : (prec == 1 ? Dev32<4>::kResThreads : Mix32<4>::kResThreads)) / kWave;
}

hipError_t resident_capacity(int prec, int s, bool lds, int waves, size_t lds_bytes,
                             int* blocks_per_cu)
{
    const void* k = kernel_of(prec, s, lds, waves);
    if (!k || waves < kResMinWaves || waves > resident_max_waves(prec)) return hipErrorInvalidValue;
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)kResLdsBytes);
    if (e != hipSuccess) return e;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k, waves * kWave, lds_bytes);
}

hipError_t launch_resident(int prec, int s, bool lds, const InstDesc* descs, InstCtrl* ctrls,
                           const ResGroup* groups, const BlockRef* refs, const ResGroup& one,
                           const ResSync& sync, int grid, int waves, size_t lds_bytes,
                           int64_t nsteps, int32_t spin_limit, hipStream_t st)
{
    const void* k = kernel_of(prec, s, lds, waves);
    if (!k || grid < 1 || grid > sync.nwg || waves < kResMinWaves ||
        waves > resident_max_waves(prec) || nsteps < 1 || nsteps > kCoopMaxSteps ||
        spin_limit < 0 || lds_bytes > kResLdsBytes)
        return hipErrorInvalidValue;
    void* args[] = {(void*)&descs,      (void*)&ctrls,      (void*)&groups,
                    (void*)&refs,       (void*)&one,        (void*)&sync.base,
                    (void*)&sync.slots, (void*)&sync.edges, (void*)&sync.recs,
                    (void*)&sync.views, (void*)&sync.nwg,   (void*)&nsteps,
                    (void*)&spin_limit};
    return hipLaunchCooperativeKernel(k, dim3((unsigned)grid), dim3((unsigned)(waves * kWave)), args,
                                      (unsigned)lds_bytes, st);
}

// (a kernel and not a memset, so that a caller's stream capture can hold it)
__global__ void resident_clear_kernel(uint64_t* __restrict__ p, size_t words)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < words;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

hipError_t launch_resident_clear(const ResSync& sync, size_t bytes, hipStream_t st)
{
    hipLaunchKernelGGL(resident_clear_kernel, dim3(64), dim3(256), 0, st, (uint64_t*)sync.base,
                       bytes / 8);
    return hipGetLastError();
}

hipError_t launch_resident_after(const InstDesc* descs, InstCtrl* ctrls, const ResGroup* groups,
                                 int ngroups, const ResGroup& one, const ResSync& sync, int64_t nsteps,
                                 hipStream_t st)
{
    if (ngroups < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(resident_after_kernel, dim3((unsigned)ngroups), dim3(256), 0, st, descs,
                       ctrls, groups, one, sync.recs, sync.views, sync.nwg, sync.base, (uint32_t)nsteps);
    return hipGetLastError();
}

}  // namespace ng
