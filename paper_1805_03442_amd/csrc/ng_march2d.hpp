// ng_march2d.hpp -- one work item of the 2D MUSCL step: a wavefront marches up
// the rows of a strip (ng_kernels.hip, ng_resident2d.hip).
#pragma once

#include "ng_device.hpp"

namespace ng {

// y-face flux: the normal velocity is v, so the Riemann solver sees
// (rho, v, u, p, E_nu) and returns (., G_v, G_u, ., .)
template <class P, int RS>
__device__ __forceinline__ void flux_y(const typename P::K& k, const typename P::R* N,
                                       const typename P::R* S, typename P::R* G)
{
    using R = typename P::R;
    R a[5] = {N[0], N[2], N[1], N[3], N[4]};
    R b[5] = {S[0], S[2], S[1], S[3], S[4]};
    R f[5];
    P::template flux<RS>(k, a, b, f);
    G[0] = f[0];
    G[1] = f[2];
    G[2] = f[1];
    G[3] = f[3];
    G[4] = f[4];
}

// One work item of the 2D step: rows [r0, r1) of a strip (60 columns + halo).
// CL: closure recipe of the FP32 arithmetic (0: general).  Coh: agent-scope
// state loads and stores (Planes).
template <class P, int RS, bool BC, int CL = 0, bool Coh = false, int Ring = 4>
__device__ __forceinline__ void march2d(const InstDesc& d, const typename P::K& k, int cur,
                                        const double* gsrc, int strip, int r0, int r1, int lane,
                                        Acc<typename P::R>& acc)
{
    using R = typename P::R;
    constexpr int NC = 5;
    // the HLLC flux takes the full density in its face states
    constexpr bool FR = RS == 0;
    const int64_t nx = d.nx, ny = d.ny;
    const int64_t x0 = (int64_t)strip * kInterior;
    bool flipx = false;
    const int64_t x = BC ? axis_cell(x0 - kHalo + lane, nx, d.bc[0], d.bc[1], flipx)
                         : wrap_axis(x0 - kHalo + lane, nx);
    const bool inner = lane >= kHalo && lane < kWave - kHalo && x0 + (lane - kHalo) < nx;
    // rows in 32 bits (a grid has fewer than 2^30 cells): the row arithmetic
    // is the same for every lane and stays on the scalar unit
    const int nyi = (int)ny;
    using St = typename P::St;
    const Planes<St, NC, Coh> src(d.buf[cur], d.ncell);
    const Planes<St, NC, Coh> dst(d.buf[cur ^ 1], d.ncell);
    const uint32_t rowb = (uint32_t)(nx * (int64_t)sizeof(St));
    const uint32_t xb = (uint32_t)(x * (int64_t)sizeof(St));
    // byte offset of (row r, this lane's column); r within two rows of [0, ny)
    auto boff = [&](int r) -> uint32_t {
        int rr;
        if (BC) {
            bool f;
            rr = (int)axis_cell(r, ny, d.bc[2], d.bc[3], f);
        } else {
            rr = r < 0 ? r + nyi : (r >= nyi ? r - nyi : r);
        }
        return (uint32_t)rr * rowb + xb;
    };
    // a loaded row r as ghost values: the lanes before a forced source take
    // its wave, wall ghosts carry the mirrored normal momentum (x ends: rho u,
    // y ends: rho v)
    const int64_t xr = x0 - kHalo + lane;
    const bool srcx = BC && d.bc[0] == kBcSource && xr < 0;
    const double* gs = gsrc + (xr == -1 ? 0 : 5);
    // the source drives the ghosts of the rows of its segment (all rows when
    // the segment's half-width is not positive)
    auto src_row = [&](int64_t r) -> bool {
        if (!(d.src_hw > 0.0)) return true;
        const double y = ((double)r + 0.5) * d.h;
        return fabs(y - d.src_yc) <= d.src_hw;
    };
    auto ghost = [&](int64_t r, St* U) {
        if (BC) {
            bool fy;
            (void)axis_cell(r, ny, d.bc[2], d.bc[3], fy);
            if (srcx && src_row(r)) source_cell<St, NC, P::kSplitE>(d, gs, U);
            if (flipx) U[1] = -U[1];
            if (fy) U[2] = -U[2];
        }
    };
    // pump and sink only inside an active wedge (the 2D sector run of section
    // 3): 1 or 0 for this lane's cell centre in row r, ghost cells included
    const bool wedge = BC && d.wedge_tan > 0.0;
    const double xc = ((double)xr + 0.5) * d.h;
    auto active = [&](int64_t r) -> R {
        if (!wedge) return (R)1;
        const double y = ((double)r + 0.5) * d.h;
        const double dx = xc - d.wedge_x0;
        return (dx >= 0.0 && fabs(y - d.wedge_y0) <= dx * d.wedge_tan) ? (R)1 : (R)0;
    };
    auto slopes_x = [&](const R* W, R* sx) {
        for (int c = 0; c < NC; c++) {
            R l = from_left(W[c]), r = from_right(W[c]);
            R a = W[c] - l, b = r - W[c];
            pin(a);
            pin(b);
            sx[c] = minmod(a, b);
        }
    };

    // Rolling state, in two register sets that swap roles every row:
    //   Wd/We  primitive state of rows i+1 / i+2 (and, FP32, 1/rho)
    //   Dp/Dn  y-differences W(i+1) - W(i) / W(i+2) - W(i+1)
    //   h0/h1  half-step state of rows i / i+1;  x0s/x1s their x-slopes
    //   Np/Nn  north face states of rows i / i+1
    //   Gp/Gn  y-fluxes at faces i-1/2 / i+1/2
    //   Uc/Ux  raw row i+2 (arrived) / row i+3 (in flight)
    // Policies that keep the raw rows hold Ring of them (rows i .. i+Ring-1, the
    // last Ring - 3 in flight) in U[row - r0 mod Ring], so U^n of row i is still
    // in registers at its update; the others re-read it and use U[2], U[3] only.
    R WA[NC + 1], WB[NC + 1], DA[NC], DB[NC], HA[NC], HB[NC], XA[NC], XB[NC];
    R NA[NC], NB[NC], GA[NC], GB[NC];
    static_assert(Ring == 4 || (Ring == 6 && P::kKeepRows), "the unrolled loops below");
    St U[Ring][NC];

    // prologue: rows r0-2 .. r0+1
    {
        R Wa[NC + 1], Wb[NC + 1], Wc[NC + 1], sy[NC], sx[NC], hb[NC], S[NC];
        St t[NC];
        St* t0 = P::kKeepRows ? U[0] : t;
        St* t1 = P::kKeepRows ? U[1] : t;
        src.load(boff(r0 - 2), t);
        ghost(r0 - 2, t);
        P::prim(k, t, Wa);
        src.load(boff(r0 - 1), t);
        ghost(r0 - 1, t);
        P::prim(k, t, Wb);
        src.load(boff(r0), t0);
        ghost(r0, t0);
        P::prim(k, t0, Wc);
        src.load(boff(r0 + 1), t1);
        ghost(r0 + 1, t1);
        P::prim(k, t1, WA);
        src.load(boff(r0 + 2), U[2]);
        if constexpr (Ring == 6) {
            src.load(boff(r0 + 3 < r1 + 1 ? r0 + 3 : r1 + 1), U[3]);
            src.load(boff(r0 + 4 < r1 + 1 ? r0 + 4 : r1 + 1), U[4]);
        }
        // row r0-1: its north face state
        slopes_x(Wb, sx);
        for (int c = 0; c < NC; c++) sy[c] = minmod(Wb[c] - Wa[c], Wc[c] - Wb[c]);
        P::template predict<FR, CL>(k, Wb, sx, sy, hb, active(r0 - 1));
        for (int c = 0; c < NC; c++) hb[c] = face(hb[c], sy[c]);
        // row r0
        slopes_x(Wc, XA);
        for (int c = 0; c < NC; c++) {
            R dp = Wc[c] - Wb[c];
            DA[c] = WA[c] - Wc[c];
            sy[c] = minmod(dp, DA[c]);
        }
        P::template predict<FR, CL>(k, Wc, XA, sy, HA, active(r0));
        for (int c = 0; c < NC; c++) {
            S[c] = face(HA[c], -sy[c]);
            NA[c] = face(HA[c], sy[c]);
        }
        flux_y<P, RS>(k, hb, S, GA);
    }

    auto row = [&](int i, R* Wd, R* We, R* Dp, R* Dn, R* h0, R* h1, R* x0s, R* x1s,
                   R* Np, R* Nn, R* Gp, R* Gn, St* Uk, St* Uc, St* Ux) {
        // U^n of row i: kept in the ring (Uk), or else re-read from cache
        // for the update (it was loaded two rows ago).  Loads complete in
        // order, so an FP64 state asks for it before row i+3 and waiting for
        // it does not also wait for the row in flight; an FP32 state asks late
        // and keeps the registers free meanwhile
        constexpr bool reread = !P::kKeepRows;
        constexpr bool early = reread && sizeof(St) == 8;
        St Ul[NC];
        St* Un = reread ? Ul : Uk;
        if (early) src.load(boff(i), Ul);
        // row i+2 has arrived in Uc; put row i+Ring-1 in flight.  The load is
        // issued on every row (on the chunk's last rows it fetches row r1+1
        // again, from cache, into an unused buffer): a load on one path only
        // makes the compiler's wait counts assume the other path, so each row
        // would wait for the loads it has just issued
        ghost(i + 2, Uc);
        P::prim(k, Uc, We);
        src.load(boff(i + Ring - 1 < r1 + 1 ? i + Ring - 1 : r1 + 1), Ux);
        // predictor of row i+1
        R sy[NC];
        slopes_x(Wd, x1s);
        for (int c = 0; c < NC; c++) {
            Dn[c] = We[c] - Wd[c];
            sy[c] = minmod(Dp[c], Dn[c]);
        }
        P::template predict<FR, CL>(k, Wd, x1s, sy, h1, active(i + 1));
        // y-face i+1/2 between the north state of row i and the south state
        // of row i+1
        {
            R S[NC];
            for (int c = 0; c < NC; c++) {
                S[c] = face(h1[c], -sy[c]);
                Nn[c] = face(h1[c], sy[c]);
            }
            flux_y<P, RS>(k, Np, S, Gn);
        }
        // x-faces of row i: lane j computes face j+1/2 from its east state and
        // lane j+1's west state; face j-1/2 comes from lane j-1
        R dF[NC], dG[NC];
        {
            R E[NC], Wr[NC], Fx[NC];
            for (int c = 0; c < NC; c++) {
                E[c] = face(h0[c], x0s[c]);
                Wr[c] = from_right(face(h0[c], -x0s[c]));
            }
            P::template flux<RS>(k, E, Wr, Fx);
            for (int c = 0; c < NC; c++) {
                dF[c] = Fx[c] - from_left(Fx[c]);
                pin(dF[c]);
                dG[c] = Gn[c] - Gp[c];
            }
        }
        // update of row i
        St Uo[NC];
        R Wn[NC + 1], sE, sV;
        const uint32_t o = boff(i);
        if (reread && !early) src.load(o, Ul);
        P::template update<FR, CL>(k, Un, dF, dG, h0, Uo, sE, sV, active(i));
        P::prim(k, Uo, Wn);
        R s = P::speed(k, Wn);
        if (inner) {
            dst.store(o, Uo);
            acc_cell<P, NC>(acc, k, Uo, Wn, s, sE, sV);
        }
    };

    int i = r0;
    if constexpr (P::kKeepRows && Ring == 6) {
        for (; i < r1; i += 6) {
            row(i, WA, WB, DA, DB, HA, HB, XA, XB, NA, NB, GA, GB, U[0], U[2], U[5]);
            if (i + 1 >= r1) break;
            row(i + 1, WB, WA, DB, DA, HB, HA, XB, XA, NB, NA, GB, GA, U[1], U[3], U[0]);
            if (i + 2 >= r1) break;
            row(i + 2, WA, WB, DA, DB, HA, HB, XA, XB, NA, NB, GA, GB, U[2], U[4], U[1]);
            if (i + 3 >= r1) break;
            row(i + 3, WB, WA, DB, DA, HB, HA, XB, XA, NB, NA, GB, GA, U[3], U[5], U[2]);
            if (i + 4 >= r1) break;
            row(i + 4, WA, WB, DA, DB, HA, HB, XA, XB, NA, NB, GA, GB, U[4], U[0], U[3]);
            if (i + 5 >= r1) break;
            row(i + 5, WB, WA, DB, DA, HB, HA, XB, XA, NB, NA, GB, GA, U[5], U[1], U[4]);
        }
    } else if constexpr (P::kKeepRows) {
        for (; i < r1; i += 4) {
            row(i, WA, WB, DA, DB, HA, HB, XA, XB, NA, NB, GA, GB, U[0], U[2], U[3]);
            if (i + 1 >= r1) break;
            row(i + 1, WB, WA, DB, DA, HB, HA, XB, XA, NB, NA, GB, GA, U[1], U[3], U[0]);
            if (i + 2 >= r1) break;
            row(i + 2, WA, WB, DA, DB, HA, HB, XA, XB, NA, NB, GA, GB, U[2], U[0], U[1]);
            if (i + 3 >= r1) break;
            row(i + 3, WB, WA, DB, DA, HB, HA, XB, XA, NB, NA, GB, GA, U[3], U[1], U[2]);
        }
    } else {
        for (; i + 1 < r1; i += 2) {
            row(i, WA, WB, DA, DB, HA, HB, XA, XB, NA, NB, GA, GB, U[0], U[2], U[3]);
            row(i + 1, WB, WA, DB, DA, HB, HA, XB, XA, NB, NA, GB, GA, U[0], U[3], U[2]);
        }
        if (i < r1) row(i, WA, WB, DA, DB, HA, HB, XA, XB, NA, NB, GA, GB, U[0], U[2], U[3]);
    }
}

}  // namespace ng
