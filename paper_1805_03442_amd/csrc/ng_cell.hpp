// ng_cell.hpp -- per-cell and per-face arithmetic of the MUSCL step for the
// vibrationally excited gas (Khrapov & Khoperskov, J. Phys.: Conf. Ser. 973
// (2018) 012007), in the two precisions of the library.
//
// FP64 ("Plain64"): the full conserved state U = (rho, rho u, rho v, E, E_nu)
// and the formulas exactly as eqs. (5), (13)-(15) state them, each written in
// one fixed evaluation order; the library is built without multiply-add
// contraction so that these are the IEEE results of that order.
//
// FP32 ("Dev32"): the state is stored as deviations from a uniform reference
// at rest, and the energy slot holds e = E - E_nu (the thermal and kinetic
// part) instead of E: (d rho, rho u, rho v, de = e - e_r, dEv = E_nu - Ev_r)
// with e_r = p_r/(gamma - 1).  Pressure then needs no difference of E and
// E_nu (eq. (5): p = (gamma - 1)(e - rho|v|^2/2)), so a medium whose E_nu lies
// far from the reference (the passive part of the sector run) keeps its
// pressure accurate.  e obeys the energy equation minus the E_nu equation:
// flux u (e + p), source rho (Q - I) + rho v.f minus the E_nu source.  Every
// flux and source is evaluated in a form in which the reference part cancels
// exactly:
//   p - p_r       = (gamma - 1)(de - rho|v|^2/2)                 (eq. (5))
//   F - F(U_ref)  = (rho u, rho u^2 + dp, rho u v, u (H_r + de + dp), u Ev),
//                   H_r = e_r + p_r
//   E_nue - E_nu  = (Cv/R) dp - dEv + (Cv/R p_r - Ev_r)          (eq. (7))
//   U*_K - U_K    = q_K (rho, rho S_K, rho v, e + p + rho (S_K - u) S*, Ev)_K,
//                   q_K = (S* - u_K)/(S_K - S*)                 (HLLC star jump)
// so that the O(1) background never enters a difference of two fluxes.  FP32
// rounding then acts on the perturbation, not on the background.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "ng_internal.hpp"

namespace ng {

// ------------------------------------------------------------- limiter

// minmod of two undivided differences (slopes of eq. (14)): zero unless both
// have the same strict sign, else the one of smaller magnitude.
__device__ __forceinline__ double minmod(double a, double b)
{
    // the smaller of two positive differences, the larger of two negative
    // ones; the other term is zero, so the sum is exact (five operations
    // instead of six compares and their selections)
    return fmax(0.0, fmin(a, b)) + fmin(0.0, fmax(a, b));
}
__device__ __forceinline__ float minmod(float a, float b)
{
    // the median of (a, b, 0) is exactly that selection
    return __builtin_amdgcn_fmed3f(a, b, 0.0f);
}

// ===================================================================== FP64

struct K64 {
    double gam, gm1, R, Cv, rho0, T0, tau0, Q0, I0, fx, fy;
    const InstDesc* d;             // exponents of a gas without a recipe
    double igm1, iR, irho0, iT0;   // correctly rounded reciprocals (quot64)
    double stiff_z;
    double dt, dtdx, hdtdx, hdt;
    int riemann;
    int cl;                        // closure recipe of the solve (kRecipe64)
};

// Division and square root.  The FP64 step is bound by vector ALU issue and
// about half of its instructions were the compiler's IEEE division (ten
// operations and a reciprocal for each quotient: scaling of both operands,
// two Newton steps, the quotient, its correction, special cases) and square
// root.  The operands here are densities, pressures, speeds and times, far
// from the ends of the exponent range, so the scaling and the special cases are
// left out; quotients with one denominator share its reciprocal; and
// denominators constant over a run have theirs rounded on the host.  The last
// operation adds the exact remainder, times the reciprocal, to a quotient that
// is off by less than two units in the last place, which gives the correctly
// rounded one while operands, quotient and remainder are normal numbers: whole
// steps equal the oracle's, with IEEE divisions, bit for bit.  Outside that the
// last bit may differ, a negative zero as numerator gives a positive one, and a
// zero denominator NaN, where a flux discards the quotient or the step fails
// either way; the exceptions, which a step survives, are a relaxation time of
// zero or infinity (quot64_any) and a temperature of zero (powh64).  With the
// closures compiled per exponent set and one side's state in the HLLC flux this
// takes half of the step's instructions away.  Us per step before and after:
// 1000x601 cells 60 and 36, 1024 cells 5.6 and 4.4, CSPH-TVD on 100003 cells 9.7
// and 7.6, section 3's gas (its -3/2 power by pow before) on 1600 cells 7.6 and
// 5.3.

// 1/b to about half a unit in the last place: the hardware's approximation
// (2^-23) and one third-order Newton step (error 2^-69 before the rounding)
__device__ __forceinline__ double recip64(double b)
{
    const double y = __builtin_amdgcn_rcp(b);
    const double e = __builtin_fma(-b, y, 1.0);
    return __builtin_fma(__builtin_fma(e, e, e), y, y);
}
// a/b, correctly rounded, from y = recip64(b) or the rounded 1/b
__device__ __forceinline__ double quot64(double a, double b, double y)
{
    const double q = a * y;
    return __builtin_fma(__builtin_fma(-b, q, a), y, q);
}
__device__ __forceinline__ double div64(double a, double b) { return quot64(a, b, recip64(b)); }
// quot64 that keeps the IEEE result of a zero or infinite denominator (a
// relaxation time that over- or underflows)
__device__ __forceinline__ double quot64_any(double a, double b, double y)
{
    return __builtin_amdgcn_div_fixup(quot64(a, b, y), b, a);
}
// 1/b, correctly rounded; Any: also for b zero or infinite
template <bool Any>
__device__ __forceinline__ double inv64(double b)
{
    const double y = recip64(b);
    const double q = __builtin_fma(__builtin_fma(-b, y, 1.0), y, y);
    return Any ? __builtin_amdgcn_div_fixup(q, b, 1.0) : q;
}
// recip64(a b) for b near a constant's multiple: from a first approximation
// y of relative error below 2^-50 (a product of two reciprocals)
__device__ __forceinline__ double recip64_from(double b, double y)
{
    return __builtin_fma(__builtin_fma(-b, y, 1.0), y, y);
}
// sqrt(x), correctly rounded: Goldschmidt's coupled iteration from the
// hardware's reciprocal root (2^-24): one step on the root and its half
// reciprocal (2^-47, from below), then two corrections by the exact remainder.
// (A third-order step instead, which may come from above, misrounds
// x = (1 - 2^-53) 4^n, whose root lies 2^-109 from a midpoint.)
// The addend keeps x = 0 (gas at rest) from 0 * infinity; it changes no x
// above 1e-284 and a zero gives 1e-150.  Negative x gives NaN.
__device__ __forceinline__ double sqrt64(double x)
{
    x = x + 1e-300;
    const double y = __builtin_amdgcn_rsq(x);
    double s = x * y, h = 0.5 * y;
    const double r = __builtin_fma(-h, s, 0.5);
    s = __builtin_fma(s, r, s);
    h = __builtin_fma(h, r, h);
    s = __builtin_fma(__builtin_fma(-s, s, x), h, s);
    return __builtin_fma(__builtin_fma(-s, s, x), h, s);
}

// pow for the exponents without a short form, kept out of line: inlined
// copies of pow would make the code many times larger than the path it runs
__device__ __noinline__ double pow_general(double x, double a) { return pow(x, a); }

// x^(C/2) of the power laws (6) for an exponent code C known at compile time:
// 0, 1, -1, 2 and 1/2 by the correctly rounded IEEE operations (the exact
// power rounded once); -3/2 (section 3's relaxation time) as the reciprocal
// of x sqrt(x) carried to twice the precision and rounded once (about 20
// operations against some 200 of pow).  Any: x may be zero, as the temperature of
// a half step whose sink takes all the pressure, and a relaxation time then
// infinite.
template <int C, bool Any>
__device__ __forceinline__ double powh64(double x)
{
    static_assert(C == 0 || C == 2 || C == -2 || C == 4 || C == 1 || C == -3,
                  "exponent code without a short form");
    if constexpr (C == 0) return 1.0;
    else if constexpr (C == 2) return x;
    else if constexpr (C == -2) return inv64<Any>(x);
    else if constexpr (C == 4) return x * x;
    else if constexpr (C == 1) return sqrt64(x);
    else {
        // sqrt(x) = s + ds, x sqrt(x) = m + dm, 1/(m + dm) = y + y (1 - y m - y dm)
        const double s = sqrt64(x);
        const double ds = __builtin_fma(-s, s, x) * (0.5 * recip64(s));
        const double m = x * s;
        const double dm = __builtin_fma(x, s, -m) + x * ds;
        const double y = recip64(m);
        const double e = __builtin_fma(-y, dm, __builtin_fma(-m, y, 1.0));
        const double q = __builtin_fma(e, y, y);
        return Any ? __builtin_amdgcn_div_fixup(q, x, 1.0) : q;
    }
}
// the same for an exponent a known at run time with its form (pow_form), the
// same for every lane: one scalar branch
template <bool Any>
__device__ __forceinline__ double powr64(double x, int form, double a)
{
    switch (form) {
    case 0: return 1.0;
    case 1: return x;
    case 2: return powh64<-2, Any>(x);
    case 3: return x * x;
    case 4: return powh64<1, Any>(x);
    case 5: return powh64<-3, Any>(x);
    default: return pow_general(x, a);
    }
}

// tau, Q and I of eq. (6)
struct Powers64 {
    double tau, Q, I;
};

// tau, Q and I of eq. (6) with the exponents of recipe CL (kRecipe64)
template <int CL>
__device__ __forceinline__ Powers64 powers64(const K64& k, double r, double t)
{
    constexpr const int* e = kRecipe64[CL];
    return {k.tau0 * powh64<e[0], false>(r) * powh64<e[1], true>(t),
            k.Q0 * powh64<e[2], false>(r) * powh64<e[3], true>(t),
            k.I0 * powh64<e[4], false>(r) * powh64<e[5], true>(t)};
}
// the same with the exponents known at run time; out of line, once per library.
// The descriptor's address and the forms are made scalar again (arguments of a
// call are not), so that the exponents are scalar loads and their selection
// scalar branches: compared lane by lane, 36 branches cost more than the pow
// (1024 cells with one general exponent 7.1 us per step, now 5.3).
__device__ __noinline__ Powers64 powers64_any(const InstDesc* dv, double r, double t)
{
    const uint64_t p = (uint64_t)(uintptr_t)dv;
    const uint64_t pu = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32)) << 32) |
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    typedef const __attribute__((address_space(4))) InstDesc CDesc;
    const CDesc* d = (const CDesc*)pu;
    const int f = d->pow_forms;
    return {d->tau0 * powr64<false>(r, f & 15, d->tau_rho) * powr64<true>(t, (f >> 4) & 15, d->tau_T),
            d->Q0 * powr64<false>(r, (f >> 8) & 15, d->Q_rho) * powr64<true>(t, (f >> 12) & 15, d->Q_T),
            d->I0 * powr64<false>(r, (f >> 16) & 15, d->I_rho) * powr64<true>(t, (f >> 20) & 15, d->I_T)};
}

// closures of eq. (6) at (rho, p), and T (eq. (7)); y = recip64(rho).  The
// predictor and corrector scale Q and I by act, 0 outside an active wedge (the
// 2D sector run of section 3).  A kernel without a recipe of its own (CL = 0)
// takes the compiled forms through one scalar branch on the solve's recipe.
template <int CL>
__device__ __forceinline__ void closures64(const K64& k, double rho, double p, double y, double& T,
                                           double& tau, double& Q, double& I)
{
    const double b = k.R * rho;
    T = quot64(p, b, recip64_from(b, y * k.iR));
    const double r = quot64(rho, k.rho0, k.irho0), t = quot64(T, k.T0, k.iT0);
    Powers64 f;
    if constexpr (CL > 0) {
        f = powers64<CL>(k, r, t);
    } else {
        if (k.cl == 3) f = powers64<3>(k, r, t);
        else if (k.cl == 1) f = powers64<1>(k, r, t);
        else if (k.cl == 2) f = powers64<2>(k, r, t);
        else f = powers64_any(k.d, r, t);
    }
    tau = f.tau;
    Q = f.Q;
    I = f.I;
}

// conserved -> primitive (eq. (5) solved for p), and 1/rho in W[NC]; NC = 4
// (1D) or 5 (2D)
template <int NC>
__device__ __forceinline__ void prim64(const K64& k, const double* U, double* W)
{
    double rho = U[0];
    double y = recip64(rho);
    double u = quot64(U[1], rho, y);
    W[NC] = y;
    if (NC == 5) {
        double v = quot64(U[2], rho, y);
        double ke = 0.5 * rho * (u * u + v * v);
        W[0] = rho;
        W[1] = u;
        W[2] = v;
        W[3] = k.gm1 * (U[3] - ke - U[4]);
        W[4] = U[4];
    } else {
        double ke = 0.5 * rho * (u * u);
        W[0] = rho;
        W[1] = u;
        W[2] = k.gm1 * (U[2] - ke - U[3]);
        W[3] = U[3];
    }
}

// signal speed of eq. (16): max(|v| + c, 2|v|)
template <int NC>
__device__ __forceinline__ double speed64(const K64& k, const double* W)
{
    double rho = W[0], u = W[1];
    double vel, p;
    if (NC == 5) {
        vel = sqrt64(u * u + W[2] * W[2]);
        p = W[3];
    } else {
        vel = fabs(u);   // the rounded sqrt(u * u)
        p = W[2];
    }
    double c = sqrt64(quot64(k.gam * p, rho, W[NC]));
    return fmax(vel + c, 2.0 * vel);
}

// Half-step predictor: quasi-linear primitive form of eqs. (1)-(5) with the
// sources at t^n (the "predictor" of the two-step scheme of section 2.3).
// W = (rho, u, v, p, E_nu) (2D) or (rho, u, p, E_nu) (1D), 1/rho in W[NC];
// sx, sy limited slopes.
template <int NC, int CL = 0>
__device__ __forceinline__ void predict64(const K64& k, const double* W, const double* sx,
                                          const double* sy, double* Wh, double act = 1.0)
{
    const double gam = k.gam, gm1 = k.gm1, hdtdx = k.hdtdx, hdt = k.hdt;
    constexpr int iP = NC == 5 ? 3 : 2, iV = NC == 5 ? 4 : 3;
    const double rho = W[0], u = W[1], p = W[iP], ev = W[iV], y = W[NC];
    const double sr = sx[0], su = sx[1], sp = sx[iP], se = sx[iV];
    double a_r = u * sr + rho * su;
    double a_u = u * su + quot64(sp, rho, y);
    double a_v = 0.0;
    double a_p = u * sp + gam * p * su;
    double a_e = u * se + ev * su;
    double v = 0.0;
    if (NC == 5) {
        v = W[2];
        a_v = u * sx[2];
        double tr = sy[0], tu = sy[1], tv = sy[2], tp = sy[3], te = sy[4];
        a_r = a_r + (v * tr + rho * tv);
        a_u = a_u + v * tu;
        a_v = a_v + (v * tv + quot64(tp, rho, y));
        a_p = a_p + (v * tp + gam * p * tv);
        a_e = a_e + (v * te + ev * tv);
    }
    double T, tau, Q, I;
    closures64<CL>(k, rho, p, y, T, tau, Q, I);
    Q = act * Q;
    I = act * I;
    const double Ee = rho * k.Cv * T;
    const double ytau = recip64(tau);
    Wh[0] = rho - hdtdx * a_r;
    Wh[1] = u - hdtdx * a_u + hdt * k.fx;
    if (NC == 5) Wh[2] = v - hdtdx * a_v + hdt * k.fy;
    if (quot64_any(k.dt, tau, ytau) > k.stiff_z) {
        // eq. (4) over dt/2 solved exactly with E_nue, tau, Q frozen
        double dEv = ((Ee + tau * (rho * Q)) - ev) * (-expm1(-(hdt / tau)));
        Wh[iP] = p - hdtdx * a_p - gm1 * (dEv - hdt * (rho * (Q - I)));
        Wh[iV] = ev - hdtdx * a_e + dEv;
    } else {
        double dEr = hdt * quot64_any(Ee - ev, tau, ytau);
        Wh[iP] = p - hdtdx * a_p - gm1 * (dEr + hdt * (rho * I));
        Wh[iV] = ev - hdtdx * a_e + (dEr + hdt * (rho * Q));
    }
}

// Interface flux along a normal.  Face states (rho, u_n, [u_t], p, E_nu);
// returns (mass, normal momentum, [tangential momentum], energy, E_nu) fluxes.
// HLL: eq. (13) with the wave speeds printed under it; HLLC: three waves, the
// middle one from equal pressure and normal velocity across the contact.
template <int NC, int RS>
__device__ __forceinline__ void flux64(const K64& k, const double* WL, const double* WR,
                                       double* F)
{
    const double gam = k.gam, gm1 = k.gm1;
    constexpr int iP = NC == 5 ? 3 : 2, iE = NC == 5 ? 3 : 2, iV = NC == 5 ? 4 : 3;
    const double rL = WL[0], uL = WL[1], pL = WL[iP];
    const double rR = WR[0], uR = WR[1], pR = WR[iP];
    const double yL = recip64(rL), yR = recip64(rR);
    const double cL = sqrt64(quot64(gam * pL, rL, yL));
    const double cR = sqrt64(quot64(gam * pR, rR, yR));
    const double SL = fmin(uL - cL, uR - cR);
    const double SR = fmax(uL + cL, uR + cR);
    // conserved state and physical flux of one side, component order (rho,
    // m_n, [m_t], E, E_nu)
    auto side = [&](double r, double u, double v, double p, double e, double* U, double* Fs) {
        const double E = quot64(p, gm1, k.igm1) +
                         0.5 * r * (NC == 5 ? u * u + v * v : u * u) + e;
        const double m = r * u;
        U[0] = r;
        U[1] = m;
        Fs[0] = m;
        Fs[1] = m * u + p;
        if (NC == 5) {
            U[2] = r * v;
            Fs[2] = m * v;
        }
        U[iE] = E;
        Fs[iE] = u * (E + p);
        U[iV] = e;
        Fs[iV] = u * e;
    };

    if (RS == 1) {
        // HLL, eq. (13)
        double UL[5], UR[5], FL[5], FR[5];
        side(rL, uL, NC == 5 ? WL[2] : 0.0, pL, WL[iV], UL, FL);
        side(rR, uR, NC == 5 ? WR[2] : 0.0, pR, WR[iV], UR, FR);
        const double dS = SR - SL, yS = recip64(dS);
        for (int c = 0; c < NC; c++) {
            double fh = quot64(SR * FL[c] - SL * FR[c] + SL * SR * (UR[c] - UL[c]), dS, yS);
            F[c] = (0.0 < SL) ? FL[c] : ((SR < 0.0) ? FR[c] : fh);
        }
        return;
    }
    const double dL = SL - uL, dR = SR - uR;
    const double Ss = div64(pR - pL + rL * uL * dL - rR * uR * dR, rL * dL - rR * dR);
    // Only one side K enters the flux: left if 0 < S_L (its flux alone) or
    // 0 < S* (the star state beside the contact), else right (its star state
    // if 0 <= S_R); selecting the five primitives of that side leaves one
    // conserved state and one physical flux to compute
    const bool sup = 0.0 < SL;
    const bool left = sup | (0.0 < Ss);
    const bool plain = sup | !(left | (0.0 <= SR));
    const double r = left ? rL : rR, u = left ? uL : uR, p = left ? pL : pR;
    const double v = NC == 5 ? (left ? WL[2] : WR[2]) : 0.0, e = left ? WL[iV] : WR[iV];
    const double S = left ? SL : SR, dS = left ? dL : dR, y = left ? yL : yR;
    double U[5], Fs[5], Us[5];
    side(r, u, v, p, e, U, Fs);
    const double rd = r * dS;
    const double fac = div64(rd, S - Ss);
    Us[0] = fac;
    Us[1] = fac * Ss;
    if (NC == 5) Us[2] = fac * v;
    Us[iE] = fac * (quot64(U[iE], r, y) + (Ss - u) * (Ss + div64(p, rd)));
    Us[iV] = fac * quot64(e, r, y);
    for (int c = 0; c < NC; c++) F[c] = plain ? Fs[c] : Fs[c] + S * (Us[c] - U[c]);
}

// Sources Y of eq. (15) at the half-step state and the conservative update.
// Un: conserved state at t^n; dF, dG: flux differences over the cell; Wh: the
// half-step primitive state.  Writes Unew and the cell's contributions to the
// source budget (dt * Y_E and the E_nu source increment).
template <int NC, int CL = 0>
__device__ __forceinline__ void update64(const K64& k, const double* Un, const double* dF,
                                         const double* dG, const double* Wh, double* Unew,
                                         double& srcE, double& srcV, double act = 1.0)
{
    const double dt = k.dt, dtdx = k.dtdx;
    constexpr int iP = NC == 5 ? 3 : 2, iE = NC == 5 ? 3 : 2, iV = NC == 5 ? 4 : 3;
    const double rho = Wh[0], u = Wh[1], v = NC == 5 ? Wh[2] : 0.0, p = Wh[iP], ev = Wh[iV];
    double T, tau, Q, I;
    closures64<CL>(k, rho, p, recip64(rho), T, tau, Q, I);
    Q = act * Q;
    I = act * I;
    double Ee = rho * k.Cv * T;
    const double ytau = recip64(tau);
    double Y[5];
    Y[0] = 0.0;
    Y[1] = rho * k.fx;
    if (NC == 5) {
        Y[2] = rho * k.fy;
        Y[iE] = rho * (u * k.fx + v * k.fy + Q - I);
    } else {
        Y[iE] = rho * (u * k.fx + Q - I);
    }
    Y[iV] = quot64_any(Ee - ev, tau, ytau) + rho * Q;
    for (int c = 0; c < NC; c++) {
        if (NC == 5)
            Unew[c] = Un[c] - dtdx * (dF[c] + dG[c]) + dt * Y[c];
        else
            Unew[c] = Un[c] - dtdx * dF[c] + dt * Y[c];
    }
    double de = dt * Y[iV];
    double z = quot64_any(dt, tau, ytau);
    if (z > k.stiff_z) {
        // eq. (4) over the whole step solved exactly from the start-of-step
        // E_nu, with E_nue, tau and Q frozen at t^{n+1/2}
        de = ((Ee + tau * (rho * Q)) - Un[iV]) * (-expm1(-z));
        if (NC == 5)
            Unew[iV] = Un[iV] - dtdx * (dF[iV] + dG[iV]) + de;
        else
            Unew[iV] = Un[iV] - dtdx * dF[iV] + de;
    }
    srcE = dt * Y[iE];
    srcV = de;
}

// ===================================================================== FP32

__device__ __forceinline__ float rcp32(float x) { return __builtin_amdgcn_rcpf(x); }

// Stiff branch: eq. (4) solved exactly over a time z tau with E_nue, tau and
// Q frozen, E_nu(z tau) - E_nu = (num + tau rhoQ)(1 - exp(-z)), num = E_nue -
// E_nu, evaluated in FP64 and returned less hq (the caller's explicit pump
// term, which it adds back).  Kept out of line: it runs only where dt/tau is
// large.
__device__ __noinline__ float relax_exact(float num, float rhoQ, float itau, double z, float hq)
{
    const double a = ((double)num + (double)rhoQ / (double)itau) * (-expm1(-z));
    return (float)(a - (double)hq);
}

struct K32 {
    float gam, gm1, igm1, CvR;
    float rho_r, p_r, ev_r, H_r, D_r;   // reference state and its cancelled constants
                                        // (H_r = e_r + p_r, e = E - E_nu)
    float cl_c[3], cl_a[3], cl_b[3];    // closures of eq. (6): c rho^a p^b
    float fx, fy;
    float gp_r;                         // gamma p_r
    float stiff_z, hstiff_z;            // stiffness threshold on dt/tau, and half of it
    float dt, dtdx, hdtdx, hdt;
    float hdtfx, hdtfy;                 // (dt/2) f, the body force of the predictor
    double dt64, hdt64;
    int riemann;
    bool force;                         // f != 0
};

// x^(C/2) for a half-integer exponent code C in [-4, 4] known at compile
// time, from x, 1/x and 1/sqrt(x)
template <int C>
__device__ __forceinline__ float pw_half(float x, float ix, float sx)
{
    static_assert(C >= -4 && C <= 4, "exponent code out of range");
    if constexpr (C == 0) return 1.0f;
    else if constexpr (C == 1) return x * sx;
    else if constexpr (C == 2) return x;
    else if constexpr (C == 3) return x * (x * sx);
    else if constexpr (C == 4) return x * x;
    else if constexpr (C == -1) return sx;
    else if constexpr (C == -2) return ix;
    else if constexpr (C == -3) return ix * sx;
    else return ix * ix;
}

// 1/tau, Q and I of eq. (6) at full (rho, p) in FP32, each c rho^a p^b
// (T = p / (R rho)).  Recipe CL > 0 (kRecipeCodes): the half-integer
// exponents are compile-time constants, so each power is a product of rho,
// p, 1/rho, 1/p and reciprocal square roots (at most one transcendental per
// base).  CL = 0: one exp2 of a log2(rho) + b log2(p) per closure.  HaveIr:
// irho is 1/rho; otherwise it is computed here when an exponent needs it.
template <bool HaveIr, int CL>
__device__ __forceinline__ void closures32(const K32& k, float rho, float p, float irho,
                                           float& itau, float& Q, float& I)
{
    if constexpr (CL == 0) {
        const float lr = __builtin_amdgcn_logf(rho), lp = __builtin_amdgcn_logf(p);
        itau = k.cl_c[0] * __builtin_amdgcn_exp2f(fmaf(k.cl_a[0], lr, k.cl_b[0] * lp));
        Q = k.cl_c[1] * __builtin_amdgcn_exp2f(fmaf(k.cl_a[1], lr, k.cl_b[1] * lp));
        I = k.cl_c[2] * __builtin_amdgcn_exp2f(fmaf(k.cl_a[2], lr, k.cl_b[2] * lp));
    } else {
        constexpr int a0 = kRecipeCodes[CL][0], b0 = kRecipeCodes[CL][1];
        constexpr int a1 = kRecipeCodes[CL][2], b1 = kRecipeCodes[CL][3];
        constexpr int a2 = kRecipeCodes[CL][4], b2 = kRecipeCodes[CL][5];
        constexpr bool odd_r = ((a0 | a1 | a2) & 1) != 0, neg_r = a0 < 0 || a1 < 0 || a2 < 0;
        constexpr bool odd_p = ((b0 | b1 | b2) & 1) != 0, neg_p = b0 < -1 || b1 < -1 || b2 < -1;
        float sr = 1.0f, ir = irho, ip = 1.0f, sp = 1.0f;
        if constexpr (odd_r) sr = __builtin_amdgcn_rsqf(rho);
        if constexpr (!HaveIr && neg_r) ir = odd_r ? sr * sr : rcp32(rho);
        if constexpr (neg_p) ip = rcp32(p);
        if constexpr (odd_p) sp = __builtin_amdgcn_rsqf(p);
        itau = k.cl_c[0] * (pw_half<a0>(rho, ir, sr) * pw_half<b0>(p, ip, sp));
        Q = k.cl_c[1] * (pw_half<a1>(rho, ir, sr) * pw_half<b1>(p, ip, sp));
        I = k.cl_c[2] * (pw_half<a2>(rho, ir, sr) * pw_half<b2>(p, ip, sp));
    }
}

// deviation primitives (d rho, u, [v], dp, dEv) from deviation conserved,
// and 1/rho in W[NC] for the predictor and the signal speed; rho |v|^2 is
// formed as m.v, the momentum times the velocity
template <int NC>
__device__ __forceinline__ void prim32(const K32& k, const float* D, float* W)
{
    float rho = k.rho_r + D[0];
    float ir = rcp32(rho);
    float u = D[1] * ir;
    W[NC] = ir;
    W[0] = D[0];
    W[1] = u;
    if (NC == 5) {
        float v = D[2] * ir;
        float m2 = fmaf(D[1], u, D[2] * v);
        W[2] = v;
        W[3] = k.gm1 * fmaf(-0.5f, m2, D[3]);
        W[4] = D[4];
    } else {
        W[2] = k.gm1 * fmaf(-0.5f, D[1] * u, D[2]);
        W[3] = D[3];
    }
}

// signal speed of eq. (16) in FP32, max(|v| + c, 2|v|) = |v| + max(c, |v|)
// (the same rounded value); c = sqrt(gamma p / rho) from the 1/rho that prim32
// leaves in W[NC]; square roots by the hardware (about 1 ulp; the speed only
// bounds dt)
template <int NC>
__device__ __forceinline__ float speed32(const K32& k, const float* W)
{
    float u = W[1];
    float v2 = NC == 5 ? W[2] * W[2] : 0.0f;
    float gp = fmaf(k.gam, W[NC == 5 ? 3 : 2], k.gp_r);
    float vel = __builtin_amdgcn_sqrtf(fmaf(u, u, v2));
    float c = __builtin_amdgcn_sqrtf(gp * W[NC]);
    return vel + fmaxf(c, vel);
}

// half-step predictor in primitive form: W + (dt/2)(-A_x dW/dx - A_y dW/dy + S(W))
// with undivided slopes sx, sy and the divergence su + tv shared by the
// density, pressure and E_nu rows.  FullRho: Wh[0] is the full density (the
// HLLC flux and the corrector use only that), else its deviation.
template <int NC, bool FullRho = false, int CL = 0>
__device__ __forceinline__ void predict32(const K32& k, const float* W, const float* sx,
                                          const float* sy, float* Wh, float act = 1.0f)
{
    const float hdtdx = k.hdtdx, hdt = k.hdt;
    constexpr int iP = NC == 5 ? 3 : 2, iV = NC == 5 ? 4 : 3;
    float dr = W[0], u = W[1], dp = W[iP], de = W[iV];
    float rho = k.rho_r + dr, p = k.p_r + dp, ev = k.ev_r + de;
    float irho = W[NC];
    float gp = fmaf(k.gam, dp, k.gp_r);
    float sr = sx[0], su = sx[1], sp = sx[iP], se = sx[iV];
    float a_r, a_u, a_v = 0.0f, a_p, a_e, v = 0.0f;
    if (NC == 5) {
        v = W[2];
        float sv = sx[2];
        float tr = sy[0], tu = sy[1], tv = sy[2], tp = sy[3], te = sy[4];
        float dv = su + tv;
        a_r = fmaf(u, sr, fmaf(v, tr, rho * dv));
        a_u = fmaf(u, su, fmaf(v, tu, sp * irho));
        a_v = fmaf(u, sv, fmaf(v, tv, tp * irho));
        a_p = fmaf(u, sp, fmaf(v, tp, gp * dv));
        a_e = fmaf(u, se, fmaf(v, te, ev * dv));
    } else {
        a_r = fmaf(u, sr, rho * su);
        a_u = fmaf(u, su, sp * irho);
        a_p = fmaf(u, sp, gp * su);
        a_e = fmaf(u, se, ev * su);
    }
    float itau, Q, I;
    closures32<true, CL>(k, rho, p, irho, itau, Q, I);
    Q = act * Q;
    I = act * I;
    float relax_num = fmaf(k.CvR, dp, k.D_r - de);   // E_nue - E_nu
    // (dt/2)/tau against half the threshold: the same decision as dt/tau
    // against the threshold (both sides scaled by exactly 1/2)
    float z = hdt * itau;
    float dEr;
    if (z > k.hstiff_z)
        dEr = relax_exact(relax_num, rho * Q, itau, k.hdt64 * (double)itau, hdt * (rho * Q));
    else
        dEr = relax_num * z;
    Wh[0] = fmaf(-hdtdx, a_r, FullRho ? rho : dr);
    Wh[1] = fmaf(-hdtdx, a_u, u);
    if (NC == 5) Wh[2] = fmaf(-hdtdx, a_v, v);
    if (k.force) {
        Wh[1] += k.hdtfx;
        if (NC == 5) Wh[2] += k.hdtfy;
    }
    Wh[iP] = fmaf(-k.gm1, fmaf(hdt, rho * I, dEr), fmaf(-hdtdx, a_p, dp));
    Wh[iV] = fmaf(hdt, rho * Q, dEr) + fmaf(-hdtdx, a_e, de);
}

// Interface flux minus the flux of the reference state, face states in
// deviation primitives.  HLLC is evaluated on one side only: the side K whose
// flux the face takes (L if 0 < S_L or 0 < S*, else R) gives
// F = F_K + S_K (U*_K - U_K), with the star jump zero on supersonic faces.
// With sq = S_K q_K the components factor as
//   rho (u + sq) = F_rho,  F_rho v,  (E + p)(u + sq) + sq rho (S_K - u) S*,
//   E_nu (u + sq).
// The HLLC flux takes face states with the full density in [0] (it uses the
// density only in products), HLL the deviation (its jump U_R - U_L).
template <int NC, int RS>
__device__ __forceinline__ void flux32(const K32& k, const float* WL, const float* WR, float* F)
{
    constexpr int iP = NC == 5 ? 3 : 2, iV = NC == 5 ? 4 : 3;
    float rL = RS == 1 ? k.rho_r + WL[0] : WL[0], rR = RS == 1 ? k.rho_r + WR[0] : WR[0];
    float uL = WL[1], uR = WR[1];
    float dpL = WL[iP], dpR = WR[iP];
    float gpL = fmaf(k.gam, dpL, k.gp_r), gpR = fmaf(k.gam, dpR, k.gp_r);
    float cL = gpL * __builtin_amdgcn_rsqf(gpL * rL);
    float cR = gpR * __builtin_amdgcn_rsqf(gpR * rR);
    float SL = fminf(uL - cL, uR - cR);
    float SR = fmaxf(uL + cL, uR + cR);
    float mL = rL * uL, mR = rR * uR;
    if (RS == 1) {
        // HLL, eq. (13), with both physical fluxes
        float vL = NC == 5 ? WL[2] : 0.0f, vR = NC == 5 ? WR[2] : 0.0f;
        float deL = WL[iV], deR = WR[iV];
        float m2L = NC == 5 ? fmaf(mL, uL, (rL * vL) * vL) : mL * uL;
        float m2R = NC == 5 ? fmaf(mR, uR, (rR * vR) * vR) : mR * uR;
        float dEL = fmaf(0.5f, m2L, dpL * k.igm1);   // de = e - e_r
        float dER = fmaf(0.5f, m2R, dpR * k.igm1);
        float HL = k.H_r + (dEL + dpL), HR = k.H_r + (dER + dpR);
        float UL[5], UR[5], FL[5], FR[5];
        UL[0] = WL[0];
        UR[0] = WR[0];
        UL[1] = mL;
        UR[1] = mR;
        FL[0] = mL;
        FR[0] = mR;
        FL[1] = fmaf(mL, uL, dpL);
        FR[1] = fmaf(mR, uR, dpR);
        if (NC == 5) {
            UL[2] = rL * vL;
            UR[2] = rR * vR;
            FL[2] = mL * vL;
            FR[2] = mR * vR;
        }
        UL[iP] = dEL;
        UR[iP] = dER;
        UL[iV] = deL;
        UR[iV] = deR;
        FL[iP] = uL * HL;
        FR[iP] = uR * HR;
        FL[iV] = uL * (k.ev_r + deL);
        FR[iV] = uR * (k.ev_r + deR);
        float inv = rcp32(SR - SL);
        float SLR = SL * SR;
        for (int c = 0; c < NC; c++) {
            float fh = fmaf(SLR, UR[c] - UL[c], fmaf(SR, FL[c], -(SL * FR[c]))) * inv;
            F[c] = (0.0f < SL) ? FL[c] : ((SR < 0.0f) ? FR[c] : fh);
        }
        return;
    }
    float dL = SL - uL, dR = SR - uR;
    float Ss = fmaf(mL, dL, fmaf(-mR, dR, dpR - dpL)) * rcp32(fmaf(rL, dL, -(rR * dR)));
    // bitwise on the comparison masks (no branch)
    const bool supL = 0.0f < SL, supR = SR < 0.0f;
    const bool left = supL | (!supR & (0.0f < Ss));
    float rK = left ? rL : rR, uK = left ? uL : uR, dpK = left ? dpL : dpR;
    float deK = left ? WL[iV] : WR[iV];
    float vK = NC == 5 ? (left ? WL[2] : WR[2]) : 0.0f;
    float SK = left ? SL : SR, dK = left ? dL : dR, mK = left ? mL : mR;
    float m2K = NC == 5 ? fmaf(mK, uK, (rK * vK) * vK) : mK * uK;   // rho |v|^2
    float dEK = fmaf(0.5f, m2K, dpK * k.igm1);   // de = e - e_r
    float HK = k.H_r + (dEK + dpK);   // e + p
    float evK = k.ev_r + deK;
    float q = (supL | supR) ? 0.0f : (Ss - uK) * rcp32(SK - Ss);
    float sq = SK * q, sqr = sq * rK;
    float us = uK + sq;
    float F0 = fmaf(sq, rK, mK);
    F[0] = F0;
    F[1] = fmaf(sqr, SK, fmaf(mK, uK, dpK));
    if (NC == 5) F[2] = F0 * vK;
    F[iP] = fmaf(HK, us, sqr * (dK * Ss));
    F[iV] = evK * us;
}

// corrector of eq. (15): U^n - dt/h (dF + dG) + dt Y(W^{n+1/2}); the source
// rows without a body force reduce to rho (Q - I) and (E_nue - E_nu)/tau + rho Q
template <int NC, bool FullRho = false, int CL = 0>
__device__ __forceinline__ void update32(const K32& k, const float* Un, const float* dF,
                                         const float* dG, const float* Wh, float* Unew,
                                         float& srcE, float& srcV, float act = 1.0f)
{
    constexpr int iP = NC == 5 ? 3 : 2, iV = NC == 5 ? 4 : 3;
    const float dt = k.dt, dtdx = k.dtdx;
    float u = Wh[1], dp = Wh[iP], de = Wh[iV];
    float v = NC == 5 ? Wh[2] : 0.0f;
    float rho = FullRho ? Wh[0] : k.rho_r + Wh[0], p = k.p_r + dp;
    float itau, Q, I;
    closures32<false, CL>(k, rho, p, 0.0f, itau, Q, I);
    Q = act * Q;
    I = act * I;
    float yE = rho * (Q - I);
    float relax_num = fmaf(k.CvR, dp, k.D_r - de);
    float yV = fmaf(relax_num, itau, rho * Q);
    float div[NC];
    for (int c = 0; c < NC; c++) div[c] = NC == 5 ? dF[c] + dG[c] : dF[c];
    for (int c = 0; c < NC; c++) Unew[c] = fmaf(-dtdx, div[c], Un[c]);
    if (k.force) {
        Unew[1] = fmaf(dt, rho * k.fx, Unew[1]);
        if (NC == 5) Unew[2] = fmaf(dt, rho * k.fy, Unew[2]);
        yE = fmaf(rho, fmaf(u, k.fx, v * k.fy), yE);
    }
    float dv = dt * yV;
    if (k.dt * itau > k.stiff_z) {
        // eq. (4) solved exactly from the start-of-step E_nu, FP64 factor
        float num = fmaf(k.CvR, dp, k.D_r - Un[iV]);
        float dEr = relax_exact(num, rho * Q, itau, k.dt64 * (double)itau, dt * (rho * Q));
        dv = fmaf(dt, rho * Q, dEr);
        Unew[iV] = dv + Unew[iV];
    } else {
        Unew[iV] = fmaf(dt, yV, Unew[iV]);
    }
    // e = E - E_nu gains the energy source less what E_nu gains
    Unew[iP] = fmaf(dt, yE, Unew[iP]) - dv;
    srcE = dt * yE;
    srcV = dv;
}

// The change of one step, -dt/h (dF + dG) + dt Y(W^{n+1/2}) (eq. (15)), for a
// state kept in another precision: the same sources and stiff branch as
// update32; ev_n is the start-of-step E_nu deviation the stiff branch relaxes.
template <int NC, bool FullRho = false, int CL = 0>
__device__ __forceinline__ void increment32(const K32& k, float ev_n, const float* dF,
                                            const float* dG, const float* Wh, float* dU,
                                            float& srcE, float& srcV, float act = 1.0f)
{
    constexpr int iP = NC == 5 ? 3 : 2, iV = NC == 5 ? 4 : 3;
    const float dt = k.dt, dtdx = k.dtdx;
    float u = Wh[1], dp = Wh[iP], de = Wh[iV];
    float v = NC == 5 ? Wh[2] : 0.0f;
    float rho = FullRho ? Wh[0] : k.rho_r + Wh[0], p = k.p_r + dp;
    float itau, Q, I;
    closures32<false, CL>(k, rho, p, 0.0f, itau, Q, I);
    Q = act * Q;
    I = act * I;
    float yE = rho * (Q - I);
    float relax_num = fmaf(k.CvR, dp, k.D_r - de);
    float yV = fmaf(relax_num, itau, rho * Q);
    for (int c = 0; c < NC; c++) dU[c] = -dtdx * (NC == 5 ? dF[c] + dG[c] : dF[c]);
    if (k.force) {
        dU[1] = fmaf(dt, rho * k.fx, dU[1]);
        if (NC == 5) dU[2] = fmaf(dt, rho * k.fy, dU[2]);
        yE = fmaf(rho, fmaf(u, k.fx, v * k.fy), yE);
    }
    float dv = dt * yV;
    if (k.dt * itau > k.stiff_z) {
        float num = fmaf(k.CvR, dp, k.D_r - ev_n);
        float dEr = relax_exact(num, rho * Q, itau, k.dt64 * (double)itau, dt * (rho * Q));
        dv = fmaf(dt, rho * Q, dEr);
        dU[iV] = dv + dU[iV];
    } else {
        dU[iV] = fmaf(dt, yV, dU[iV]);
    }
    dU[iP] = fmaf(dt, yE, dU[iP]) - dv;
    srcE = dt * yE;
    srcV = dv;
}

}  // namespace ng
