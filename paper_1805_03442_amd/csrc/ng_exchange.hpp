// ng_exchange.hpp -- how the workgroups of a cooperative launch agree on a step
// (ng_resident.hip, ng_resident2d.hip): the wave's reduction of the signal
// speed and failure flags, the slots they are published in and polled from,
// and the workgroup's record of a step's sums.
#pragma once

#include "ng_device.hpp"

namespace ng {

// largest value of the wave, in every lane (NaN lanes ignored): row shifts,
// then the two row broadcasts, leave it in lane 63
template <int Ctrl, int RowMask>
__device__ __forceinline__ double dpp_max(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(v), __double2loint(v), Ctrl, RowMask,
                                               0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(v), __double2hiint(v), Ctrl, RowMask,
                                               0xf, false);
    return fmax(v, __hiloint2double(hi, lo));
}
__device__ __forceinline__ double wave_max(double v)
{
    v = dpp_max<0x111, 0xf>(v);   // row_shr:1
    v = dpp_max<0x112, 0xf>(v);   // row_shr:2
    v = dpp_max<0x114, 0xf>(v);   // row_shr:4
    v = dpp_max<0x118, 0xf>(v);   // row_shr:8
    v = dpp_max<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_max<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}
// union of three flag bits over the wave
__device__ __forceinline__ uint32_t wave_flags(uint32_t f)
{
    return (__builtin_amdgcn_ballot_w64(f & 1u) ? 1u : 0u) |
           (__builtin_amdgcn_ballot_w64(f & 2u) ? 2u : 0u) |
           (__builtin_amdgcn_ballot_w64(f & 4u) ? 4u : 0u);
}

// Wave-wide wait for the slots of step gen of G <= kCoopFlat workgroups: lane j
// reads slots j, j + 64, ... (NQ of them; past the last, the last again), at
// most spin_limit polls after the first; true when they ran out.  m, f: the
// largest signal speed and the union of the flags of this lane's slots.  R:
// the speed's type.  What the exchange costs is set by the slots' spacing:
// stores of different XCDs into one 128-byte line wait for each other, and
// every poll moves all slots' sectors to every workgroup.  Us per step at 16,
// 32, 64 and 128 bytes per slot: 16384 FP32 cells (69 workgroups) 3.03, 2.67,
// 2.48, 2.51; 262144 FP64 cells (256 workgroups) 8.19, 8.03, 8.10, 8.36; three
// words per slot at 32 bytes made it 8.5.  So 64 bytes up to 128 workgroups,
// then 32.  (A second poll in flight, and no sleep between polls, changed
// nothing or cost 0.1 us.)
constexpr int slot_words(uint32_t G) { return G <= 128u ? 8 : 4; }
template <class R, int NQ>
struct SlotPoll {
    static constexpr int kWords = (int)sizeof(R) / 4;
    uint64_t w[NQ][kWords];
    __device__ __forceinline__ void issue(const uint64_t* slots, uint32_t G, int lane)
    {
#pragma unroll
        for (int q = 0; q < NQ; q++) {
            const uint32_t j = (uint32_t)lane + 64u * q;
#pragma unroll
            for (int x = 0; x < kWords; x++)
                w[q][x] = __hip_atomic_load(slots + (j < G ? j : G - 1u) * slot_words(NQ <= 2 ? 1u : 256u) + x,
                                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __device__ __forceinline__ bool have(uint32_t gen) const
    {
        bool h = true;
#pragma unroll
        for (int q = 0; q < NQ; q++)
#pragma unroll
            for (int x = 0; x < kWords; x++) h = h && (uint32_t)(w[q][x] >> 32) == gen;
        return __builtin_amdgcn_ballot_w64(!h) == 0ull;
    }
    __device__ __forceinline__ void fold(double& m, uint32_t& f) const
    {
        m = 0.0;
        f = 0u;
#pragma unroll
        for (int q = 0; q < NQ; q++) {
            const uint32_t hi = (uint32_t)w[q][kWords - 1];
            if (hi & 0x80000000u)
                f |= hi & 7u;
            else if (kWords == 2)
                m = fmax(m, __hiloint2double((int)hi, (int)(uint32_t)w[q][0]));
            else
                m = fmax(m, (double)__int_as_float((int)hi));
        }
    }
};
template <class R, int NQ>
__device__ __forceinline__ bool poll_slots(const uint64_t* slots, uint32_t G, uint32_t gen,
                                           int lane, int32_t spin_limit, double& m, uint32_t& f)
{
    static_assert(kCoopFlat <= 4 * kWave, "at most four slots per lane");
    SlotPoll<R, NQ> a;
    a.issue(slots, G, lane);
    for (int32_t n = 0;; n++) {
        if (a.have(gen)) {
            a.fold(m, f);
            return false;
        }
        if (n >= spin_limit) {
            m = 0.0;
            f = 0u;
            return true;
        }
        __builtin_amdgcn_s_sleep(1);
        a.issue(slots, G, lane);
    }
}

// The solve's control as a workgroup of a cooperative launch tracks it, alike in
// all of them; in LDS, kept by lane 0 of wave 0, so that it costs the marching
// lanes no registers.
struct ResCtl {
    double t, dt_cfl, dt_last;
    double dt;          // the step to take
    int64_t steps;
    int32_t nacc;       // steps this launch accepted
    int32_t status;
    uint32_t bad;       // failure flags of a rejected step
    int32_t go;         // a further step is to be taken
    int32_t ok;         // the last computed step was accepted
    int32_t stalled;    // the wait for the slots ran out

    // the dt of the step to take, and whether one is
    __device__ __forceinline__ void next(const InstCtrl& c)
    {
        go = status == 0 && t < c.t_end && steps < c.max_steps;
        dt = dt_cfl;
        if (t + dt > c.t_end) dt = c.t_end - t;
    }
    __device__ __forceinline__ void start(const InstCtrl& c)
    {
        t = c.t;
        dt_cfl = c.dt_cfl;
        dt_last = c.dt_last;
        steps = c.steps;
        nacc = 0;
        status = c.status;
        bad = 0u;
        ok = 0;
        stalled = 0;
        next(c);
    }
    // the outcome of a step, from the largest signal speed m and the union of
    // the flags f, as accept_step advances the control block
    __device__ __forceinline__ void decide(const InstDesc& d, const InstCtrl& c, bool out, double m,
                                           uint32_t f)
    {
        ok = 0;
        if (out) {
            stalled = 1;
            go = 0;
        } else if (f & 7u) {
            bad = f & 7u;
            status = -3;   // NG_EPHYS
            go = 0;
        } else {
            t = t + dt;
            steps = steps + 1;
            dt_last = dt;
            dt_cfl = d.cfl * d.h / m;
            nacc++;
            ok = 1;
            next(c);
        }
    }
    __device__ __forceinline__ void view(int cur0, CoopView& w) const
    {
        w.t = t;
        w.dt_cfl = dt_cfl;
        w.dt_last = dt_last;
        w.steps = steps;
        w.nacc = nacc;
        w.cur = cur0 ^ (nacc & 1);
        w.status = status;
        w.flags = bad;
        w.stalled = stalled ? 1u : 0u;
    }
};

// One wave's part of a step's end: publish workgroup b's signal speed m and
// flags f (the same in every lane) in its slot, wait for the slots of all G
// workgroups, and return the largest speed and the union of the flags in m
// and f.  True when the wait ran out.
template <class R>
__device__ __forceinline__ bool exchange_slots(uint64_t* sl, uint32_t G, uint32_t b, uint32_t gen,
                                               int lane, int32_t spin_limit, double& m, uint32_t& f)
{
    constexpr int kWords = (int)sizeof(R) / 4;
    if (lane < kWords) {
        // lane 0: the low half in FP64, the whole in FP32
        const uint32_t lo = kWords == 2 ? (uint32_t)__double2loint(m)
                                        : (uint32_t)__float_as_int((float)m);
        const uint32_t hi = (uint32_t)__double2hiint(m);
        uint32_t v = lane == 0 ? lo : hi;
        if (f && lane == kWords - 1) v = 0x80000000u | f;
        __hip_atomic_store(sl + (size_t)slot_words(G) * b + lane, ((uint64_t)gen << 32) | v,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    bool out;
    if (G <= 64u)
        out = poll_slots<R, 1>(sl, G, gen, lane, spin_limit, m, f);
    else if (G <= 128u)
        out = poll_slots<R, 2>(sl, G, gen, lane, spin_limit, m, f);
    else
        out = poll_slots<R, 4>(sl, G, gen, lane, spin_limit, m, f);
    m = wave_max(m);
    f = wave_flags(f);
    return out;
}

// A workgroup's record of step `step` (lanes, then waves in order): the sums of
// that step and the source increments b0, b1 up to it.  The after-kernel folds
// the records of the last step the most advanced workgroup accepted, found by
// its parity.
template <class R>
__device__ __forceinline__ void put_record(const Acc<R>& a, double b0, double b1, int step,
                                           CoopRec* out, double (*s_sum)[10], int wave, int lane,
                                           int nw)
{
    double v[10];
    for (int x = 0; x < 5; x++) v[x] = a.tot[x];
    v[5] = b0;
    v[6] = b1;
    v[7] = (double)a.smax;
    v[8] = (double)a.rmin;
    v[9] = (double)a.pmin;
    for (int m = 32; m >= 1; m >>= 1) {
        for (int x = 0; x < 7; x++) v[x] += lane_xor(v[x], lane, m);
        v[7] = fmax(v[7], lane_xor(v[7], lane, m));
        v[8] = fmin(v[8], lane_xor(v[8], lane, m));
        v[9] = fmin(v[9], lane_xor(v[9], lane, m));
    }
    __syncthreads();
    if (lane == 0)
        for (int x = 0; x < 10; x++) s_sum[wave][x] = v[x];
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < nw; w++) {
            for (int x = 0; x < 7; x++) v[x] += s_sum[w][x];
            v[7] = fmax(v[7], s_sum[w][7]);
            v[8] = fmin(v[8], s_sum[w][8]);
            v[9] = fmin(v[9], s_sum[w][9]);
        }
        CoopRec r;
        for (int x = 0; x < 5; x++) r.tot[x] = v[x];
        r.src[0] = v[5];
        r.src[1] = v[6];
        r.smax = v[7];
        r.rho_min = v[8];
        r.p_min = v[9];
        r.flags = 0u;
        r.step = (uint32_t)step;
        *out = r;
    }
}

}  // namespace ng
