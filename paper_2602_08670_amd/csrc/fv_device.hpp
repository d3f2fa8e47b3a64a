// Device-side physics of the finite-volume step: face-state reconstruction,
// normal-frame numerical fluxes and the hydrostatic bed treatment.
//
// Thesis "A Machine Learning accelerated geophysical fluid solver":
//   shallow-water flux, eq 2.3; Euler flux with the ideal-gas law, eq 2.4 and
//   section 4.2; MINMOD face states, eq 2.18; HLLE, eq 2.16; Rusanov, eq 2.12;
//   Roe, eq 2.13/2.14; axis-aligned rotation into the face frame, eq 2.24.
// The bed source follows the hydrostatic reconstruction of Audusse et al.
// (2004), the reading taken where the thesis leaves the discretisation open.
//
// The step is bound by vector-ALU issue, so the code is written branch-free:
// min/max/abs map to single instructions (v_min3/v_max3, |x| source
// modifiers), MINMOD is one v_med3_f32, guards are selects, and every face
// evaluates one reciprocal per side, one for the Roe weight and one for the
// HLLE denominator, plus three square roots.
#pragma once

#include <hip/hip_runtime.h>

namespace fvk {

enum { SWE = 0, EULER = 1 };
enum { HLLE = 0, RUSANOV = 1, ROE = 2 };
enum { MINMOD = 0, FIRST = 1 };

// ---------------------------------------------------------------- arithmetic
// Single precision uses the hardware reciprocal and square root (about 1 ulp);
// double precision keeps IEEE division and square root.
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp(double x) { return 1.0 / x; }
__device__ __forceinline__ float fsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double fsqrt(double x) { return __builtin_sqrt(x); }
__device__ __forceinline__ float tmin(float a, float b) { return __builtin_fminf(a, b); }
__device__ __forceinline__ double tmin(double a, double b) { return __builtin_fmin(a, b); }
__device__ __forceinline__ float tmax(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ __forceinline__ double tmax(double a, double b) { return __builtin_fmax(a, b); }
__device__ __forceinline__ float tabs(float a) { return __builtin_fabsf(a); }
__device__ __forceinline__ double tabs(double a) { return __builtin_fabs(a); }

// a b + c, rounded once
__device__ __forceinline__ float tfma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double tfma(double a, double b, double c) { return __builtin_fma(a, b, c); }

// MINMOD(a, b): 0 unless a and b share a sign, else the one of smaller
// magnitude -- which is the median of (a, b, 0).
__device__ __forceinline__ float minmod(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, 0.0f); }
__device__ __forceinline__ double minmod(double a, double b)
{
    return __builtin_fmax(__builtin_fmin(a, b), __builtin_fmin(__builtin_fmax(a, b), 0.0));
}

// 1/x nearly rounded: the hardware's with one Newton step.
__device__ __forceinline__ float rcp_near(float x)
{
    const float r = rcp(x);
    return __builtin_fmaf(__builtin_fmaf(-x, r, 1.0f), r, r);
}
__device__ __forceinline__ double rcp_near(double x) { return 1.0 / x; }

// 1/x for x > 0, else 0 (a dry state has zero velocity).
template <typename T> __device__ __forceinline__ T rcp_pos(T x) { return x > T(0) ? rcp(x) : T(0); }

// A positive power of two far below any wave speed or sqrt(h) of interest:
// the floor that keeps HLLE's denominator and the Roe weight positive.
template <typename T> __device__ __forceinline__ T tiny() { return T(0x1p-60f); }

template <typename T> struct Phys {
    T g;      // gravity
    T sqg;    // sqrt(g)
    T gamma;  // ratio of specific heats
    T h0;     // reference depth: the SWE pressure is carried as g (h^2 - h0^2) / 2
};

// ------------------------------------------------------------ shallow water
// Normal-frame state given by depth and velocities: (h, u normal, v tangential).
template <typename T> struct SweV { T h, u, v; };

// Numerical flux of two normal-frame shallow-water states.  The pressure
// g h^2/2 is carried relative to the constant g c/2, c = h0^2 rounded to the
// working precision: every flux below is affine in (F_L, F_R) with weights
// summing to one (and equal to F_L when both sides are dry), so the constant
// shifts all face fluxes equally and cancels in every cell's divergence,
// while h^2 - c, formed as one fused multiply-add, carries a rounding error
// that scales with |h^2 - h0^2| instead of h^2.
template <typename T, int FLUX>
__device__ __forceinline__ void swe_numflux(const SweV<T> &L, const SweV<T> &R, const Phys<T> &ph, T F[3])
{
    const T hg = T(0.5) * ph.g;
    const T c0 = ph.h0 * ph.h0;
    T ml = L.h * L.u, mr = R.h * R.u;
    T fl[3] = {ml, ml * L.u + hg * (L.h * L.h - c0), ml * L.v};
    T fr[3] = {mr, mr * R.u + hg * (R.h * R.h - c0), mr * R.v};
    T dq[3] = {R.h - L.h, mr - ml, R.h * R.v - L.h * L.v};
    T wl = fsqrt(L.h), wr = fsqrt(R.h);
    T cl = ph.sqg * wl, cr = ph.sqg * wr;
    if (FLUX == RUSANOV) {
        T a = tmax(tabs(L.u) + cl, tabs(R.u) + cr);
#pragma unroll
        for (int k = 0; k < 3; k++) F[k] = T(0.5) * (fl[k] + fr[k]) - T(0.5) * a * dq[k];
        return;
    }
    // Roe averages: sqrt(h)-weighted velocities (zero when both sides are
    // dry), c~ = sqrt(g (hL + hR) / 2)
    T iw = rcp(tmax(wl + wr, tiny<T>()));
    T ua = (wl * L.u + wr * R.u) * iw;
    T ca = fsqrt(hg * (L.h + R.h));
    if (FLUX == HLLE) {
        // sR is floored at a tiny power of two instead of 0.  The denominator
        // is then never zero: where it would be (both sides dry, sL = sR = 0)
        // the formula returns F_L exactly, which equals (F_L + F_R)/2 there;
        // elsewhere the floor moves the flux by a relative 2^-60 at most.
        // (sR F_L - sL F_R + sL sR dQ) / (sR - sL) = F_L + t (sR dQ - (F_R - F_L)),
        // t = sL / (sR - sL)
        T sL = tmin(tmin(L.u - cl, ua - ca), T(0));
        T sR = tmax(tmax(R.u + cr, ua + ca), tiny<T>());
        T t = sL * rcp(sR - sL);
#pragma unroll
        for (int k = 0; k < 3; k++) F[k] = fl[k] + t * (sR * dq[k] - (fr[k] - fl[k]));
        return;
    }
    // Roe: three waves u-c, u (shear), u+c
    T va = (wl * L.v + wr * R.v) * iw;
    T i2c = rcp_pos(T(2) * ca);
    T a1 = ((ua + ca) * dq[0] - dq[1]) * i2c;
    T a3 = (dq[1] - (ua - ca) * dq[0]) * i2c;
    T a2 = dq[2] - va * dq[0];
    T l1 = tabs(ua - ca) * a1, l2 = tabs(ua) * a2, l3 = tabs(ua + ca) * a3;
    F[0] = T(0.5) * (fl[0] + fr[0]) - T(0.5) * (l1 + l3);
    F[1] = T(0.5) * (fl[1] + fr[1]) - T(0.5) * (l1 * (ua - ca) + l3 * (ua + ca));
    F[2] = T(0.5) * (fl[2] + fr[2]) - T(0.5) * (l1 * va + l2 + l3 * va);
}

// ----------------------------------------------------------------- Euler
template <typename T> struct EulS { T r, m, t, E; };

template <typename T> __device__ __forceinline__ T eul_p(const EulS<T> &s, T gamma)
{
    return (gamma - T(1)) * (s.E - T(0.5) * (s.m * s.m + s.t * s.t) * rcp(s.r));
}

template <typename T, int FLUX>
__device__ __forceinline__ void eul_numflux(const EulS<T> &L, const EulS<T> &R, T gamma, T F[4])
{
    T irl = rcp(L.r), irr = rcp(R.r);
    T ul = L.m * irl, ur = R.m * irr;
    T vl = L.t * irl, vr = R.t * irr;
    T pl = (gamma - T(1)) * (L.E - T(0.5) * (L.m * ul + L.t * vl));
    T pr = (gamma - T(1)) * (R.E - T(0.5) * (R.m * ur + R.t * vr));
    T fl[4] = {L.m, L.m * ul + pl, L.t * ul, ul * (L.E + pl)};
    T fr[4] = {R.m, R.m * ur + pr, R.t * ur, ur * (R.E + pr)};
    T dq[4] = {R.r - L.r, R.m - L.m, R.t - L.t, R.E - L.E};
    T cl = fsqrt(gamma * pl * irl), cr = fsqrt(gamma * pr * irr);
    if (FLUX == RUSANOV) {
        T a = tmax(tabs(ul) + cl, tabs(ur) + cr);
#pragma unroll
        for (int k = 0; k < 4; k++) F[k] = T(0.5) * (fl[k] + fr[k]) - T(0.5) * a * dq[k];
        return;
    }
    T wl = fsqrt(L.r), wr = fsqrt(R.r);
    T iw = rcp(wl + wr);
    T ua = (wl * ul + wr * ur) * iw;
    T va = (wl * vl + wr * vr) * iw;
    T Ha = (wl * ((L.E + pl) * irl) + wr * ((R.E + pr) * irr)) * iw;
    T c2 = (gamma - T(1)) * (Ha - T(0.5) * (ua * ua + va * va));
    T ca = fsqrt(tmax(c2, T(0)));
    if (FLUX == HLLE) {
        T sL = tmin(tmin(ul - cl, ua - ca), T(0));
        T sR = tmax(tmax(ur + cr, ua + ca), T(0));
        T id = rcp(sR - sL), ss = sL * sR;  // sR - sL >= c~ > 0 for admissible states
#pragma unroll
        for (int k = 0; k < 4; k++) F[k] = (sR * fl[k] - sL * fr[k] + ss * dq[k]) * id;
        return;
    }
    // Roe: acoustic u-c, entropy u, shear u, acoustic u+c (normal frame)
    T gm1 = gamma - T(1);
    T a3 = dq[2] - va * dq[0];
    T d5 = dq[3] - a3 * va;
    T a2 = gm1 * rcp(ca * ca) * (dq[0] * (Ha - ua * ua) + ua * dq[1] - d5);
    T a1 = (dq[0] * (ua + ca) - dq[1] - ca * a2) * rcp(T(2) * ca);
    T a4 = dq[0] - (a1 + a2);
    T w1 = tabs(ua - ca) * a1, w2 = tabs(ua) * a2, w3 = tabs(ua) * a3, w4 = tabs(ua + ca) * a4;
    F[0] = T(0.5) * (fl[0] + fr[0]) - T(0.5) * (w1 + w2 + w4);
    F[1] = T(0.5) * (fl[1] + fr[1]) - T(0.5) * (w1 * (ua - ca) + w2 * ua + w4 * (ua + ca));
    F[2] = T(0.5) * (fl[2] + fr[2]) - T(0.5) * (w1 * va + w2 * va + w3 + w4 * va);
    F[3] = T(0.5) * (fl[3] + fr[3]) -
           T(0.5) * (w1 * (Ha - ua * ca) + w2 * T(0.5) * (ua * ua + va * va) + w3 * va + w4 * (Ha + ua * ca));
}

// --------------------------------------------------------- face states

// Face states on both sides of face i+1/2 from the four cells i-1, i, i+1, i+2
// along the face normal, for one scalar: MINMOD (eq 2.18, right state taken
// towards the face) or first order.
template <typename T, int RECON>
__device__ __forceinline__ void recon_pair(T m1, T c0, T c1, T p2, T &ql, T &qr)
{
    if (RECON == FIRST) {
        ql = c0;
        qr = c1;
    } else {
        ql = c0 + T(0.5) * minmod(c0 - m1, c1 - c0);
        qr = c1 - T(0.5) * minmod(c1 - c0, p2 - c1);
    }
}

template <typename T> __device__ __forceinline__ bool eul_admissible(T r, T m, T t, T E, T gamma)
{
    T p = (gamma - T(1)) * (E - T(0.5) * (m * m + t * t) * rcp(r));
    return r > T(0) && p > T(0);
}

// CFL rate (|u|+c)/dx + (|v|+c)/dy of a cell and whether the cell is
// admissible (finite, h > 0; or rho > 0 and p > 0).  A non-finite or
// non-positive depth, or a non-finite momentum or energy, makes the rate NaN
// or infinite, so one comparison of the rate covers finiteness; the
// comparison is false for NaN.  (A positive depth so small that the rate
// overflows is reported inadmissible too: it would stall Delta t at 0.)
// Fused multiply-adds are written out, so that every kernel computes the
// same bits.
template <typename T, int EQN>
__device__ __forceinline__ bool cell_rate_ok(const T *s, const Phys<T> &ph, T rdx, T rdy, T &rate)
{
#pragma clang fp contract(off)
    const T ir = rcp(s[0]);
    const T u = s[1] * ir, v = s[2] * ir;
    if (EQN == SWE) {
        const T w = fsqrt(s[0]);
        rate = tfma(tfma(ph.sqg, w, tabs(v)), rdy, tfma(ph.sqg, w, tabs(u)) * rdx);
        return rate < T(__builtin_inf());
    }
    const T p = (ph.gamma - T(1)) * tfma(T(-0.5), tfma(s[2], v, s[1] * u), s[3]);
    const T c = fsqrt(ph.gamma * p * ir);
    rate = tfma(tabs(v) + c, rdy, (tabs(u) + c) * rdx);
    return s[0] > T(0) && p > T(0) && rate < T(__builtin_inf());
}

// Full face computation of a flat bottom, for the exported fluxes.  Inputs:
// the four cells along the normal for each variable, in Cartesian order.
// Output: the flux (NV values, Cartesian order).
// AXIS 0: x face (normal momentum is variable 1), AXIS 1: y face (variable 2).
template <typename T, int EQN, int FLUX, int RECON, int AXIS>
__device__ __forceinline__ void face_flux(const T (*st)[4], const Phys<T> &ph, T *F)
{
    constexpr int NV = EQN == SWE ? 3 : 4;
    constexpr int NM = AXIS == 0 ? 1 : 2, TM = AXIS == 0 ? 2 : 1;
    T QL[NV], QR[NV];
#pragma unroll
    for (int v = 0; v < NV; v++) recon_pair<T, RECON>(st[v][0], st[v][1], st[v][2], st[v][3], QL[v], QR[v]);
    if (EQN == EULER) {
        // face states that are not admissible fall back to the cell average
        const bool okl = eul_admissible(QL[0], QL[1], QL[2], QL[3], ph.gamma);
        const bool okr = eul_admissible(QR[0], QR[1], QR[2], QR[3], ph.gamma);
#pragma unroll
        for (int v = 0; v < NV; v++) {
            QL[v] = okl ? QL[v] : st[v][1];
            QR[v] = okr ? QR[v] : st[v][2];
        }
        EulS<T> L{QL[0], QL[NM], QL[TM], QL[3]}, R{QR[0], QR[NM], QR[TM], QR[3]};
        T G[4];
        eul_numflux<T, FLUX>(L, R, ph.gamma, G);
        F[0] = G[0];
        F[NM] = G[1];
        F[TM] = G[2];
        F[3] = G[3];
        return;
    }
    T il = rcp(QL[0]), ir = rcp(QR[0]);  // face depths are positive here
    SweV<T> L{QL[0], QL[NM] * il, QL[TM] * il}, R{QR[0], QR[NM] * ir, QR[TM] * ir};
    T G[3];
    swe_numflux<T, FLUX>(L, R, ph, G);
    F[0] = G[0];
    F[NM] = G[1];
    F[TM] = G[2];
}

// ------------------------------------------------ faces of the stage kernels
// The stage kernels are bound by vector-ALU issue, so their faces use fewer
// operations than the formulas above, and write every fused multiply-add out
// (contraction off), so that a face has the same bits wherever it is
// evaluated: in any tile shape, at a tile's edge or inside.
//
// Euler's HLLE weighs the two sides, a F_L + b F_R + c dQ with a = s_R w,
// b = -s_L w, c = s_L s_R w, w = 1 / (s_R - s_L): where all waves run to one
// side the other side's flux drops out with its rounding, however strong the
// jump, and a face and its mirror image have the same bits (at a wall the mass
// flux is exactly zero), so the sums of the two sides are not fused.  Anchored
// on one side (a_L F_0 + (a_R - a_L) b per transported quantity, 16 steps of
// 1000 x 700 cells 319 us instead of 334) an FP32 cell's energy update was off
// from double precision by 5.3e-8 rms where it is 2.9e-8 so (contrasts of
// e^0.1, Mach 0.5), by up to 1.1e-3 where it is 1.5e-4 (e^3, Mach 5).
//
// Shallow water's HLLE is F_L + t (s_R dQ - (F_R - F_L)), t = s_L / (s_R - s_L).
// With the mass flux F_0 and b = t (s_R h_R - m_R), a velocity a is transported
// as a_L F_0 + (a_R - a_L) b, which is the same value rearranged.  Its Roe
// average is a_L + k (a_R - a_L), k = sqrt(h_R) / (sqrt(h_L) + sqrt(h_R)).
//
// Shallow water carries the normal momentum flux relative to the pressure
// g h^2 / 2 of each side's own face state, since a cell's two face states
// along an axis are h -+ s/2: the pressures (and with a bed the hydrostatic
// terms and the centred source) of the two faces sum to -g h s_eta, s_eta the
// limited slope of the free surface, which the cell adds by itself.  No large
// pressure is then formed and subtracted, and a face hands over three values.

// MINMOD values of a cell at its low and high face, and its slope, from the
// differences to its two neighbours along the axis.
template <typename T, int RECON>
__device__ __forceinline__ void cell_ends(T c, T dl, T dh, T &lo, T &hi, T &slope)
{
#pragma clang fp contract(off)
    if (RECON == FIRST) {
        lo = hi = c;
        slope = T(0);
        return;
    }
    slope = minmod(dl, dh);
    lo = tfma(T(-0.5), slope, c);
    hi = tfma(T(0.5), slope, c);
}

// Difference of the two face values between cells whose averages differ by d
// and whose slopes are sl and sr.
template <typename T, int RECON> __device__ __forceinline__ T face_jump(T d, T sl, T sr)
{
    if (RECON == FIRST) return d;
    return tfma(T(-0.5), sl + sr, d);
}

template <typename T> __device__ __forceinline__ T clamp0(T x, T hi) { return tmax(tmin(x, hi), T(0)); }
template <> __device__ __forceinline__ float clamp0(float x, float hi) { return __builtin_amdgcn_fmed3f(x, 0.0f, hi); }

// Shallow water: face values QL, QR (Cartesian order, the free surface last
// with a bed) and the jump of the free surface across the face -> F (the flux
// as the low cell sees it, normal momentum relative to its own pressure) and
// nr (the normal momentum flux as the high cell sees it).  The jump is formed
// from the cells' differences and slopes, which are exact or nearly so, and
// carries none of the face values' rounding into the pressure.  With a bed
// the depths are limited against the higher bed side (velocities kept):
// h_L* = h_R - jump within [0, h_L], h_R* = h_L + jump within [0, h_R], and
// h_R* - h_L* is the jump within [-h_L, h_R].
template <typename T, bool BATHY, int FLUX, int AXIS>
__device__ __forceinline__ void swe_face(const T *QL, const T *QR, T jump, const Phys<T> &ph, T *F, T &nr)
{
#pragma clang fp contract(off)
    constexpr int NM = AXIS == 0 ? 1 : 2, TM = AXIS == 0 ? 2 : 1;
    T hl = QL[0], hr = QR[0];
    const T il = rcp(hl), ir = rcp(hr);  // face depths are positive here
    const T ul = QL[NM] * il, vl = QL[TM] * il, ur = QR[NM] * ir, vr = QR[TM] * ir;
    T ml = QL[NM], mr = QR[NM];
    T dh = jump;
    if constexpr (BATHY) {
        dh = tmax(tmin(jump, hr), -hl);
        const T a = clamp0(hr - jump, hl), b = clamp0(hl + jump, hr);
        hl = a;
        hr = b;
        ml = hl * ul;
        mr = hr * ur;
    }
    const T du = ur - ul, dv = vr - vl, dm = BATHY ? tfma(hr, ur, -ml) : mr - ml;
    const T gs = (T(0.5) * ph.g) * (hl + hr);
    const T hp = gs * dh;  // pressure difference
    const T wl = fsqrt(hl), wr = fsqrt(hr);
    if constexpr (FLUX == RUSANOV) {
        const T a = T(0.5) * tmax(tfma(ph.sqg, wl, tabs(ul)), tfma(ph.sqg, wr, tabs(ur)));
        F[0] = tfma(-a, dh, T(0.5) * (ml + mr));
        F[NM] = tfma(-a, dm, T(0.5) * (tfma(mr, ur, ml * ul) + hp));
        F[TM] = tfma(-a, tfma(hr, vr, -(hl * vl)), T(0.5) * tfma(mr, vr, ml * vl));
        nr = F[NM] - hp;
        return;
    }
    const T ws = wl + wr;
    const T k = wr * rcp(BATHY ? tmax(ws, tiny<T>()) : ws);
    const T ua = tfma(k, du, ul), ca = fsqrt(gs);
    if constexpr (FLUX == HLLE) {
        // s_R is floored at a tiny power of two instead of 0: where both
        // sides are dry the formula then returns F_L = 0
        const T sL = tmin(tmin(tfma(-ph.sqg, wl, ul), ua - ca), T(0));
        const T sR = tmax(tmax(tfma(ph.sqg, wr, ur), ua + ca), tiny<T>());
        const T t = sL * rcp(sR - sL);
        const T f0 = tfma(t, tfma(sR, dh, -dm), ml);
        const T b = t * tfma(sR, hr, -mr);
        F[0] = f0;
        F[NM] = tfma(du, b, tfma(ul, f0, -(t * hp)));
        F[TM] = tfma(dv, b, vl * f0);
        nr = F[NM] - hp;
        return;
    }
    // Roe: three waves u-c, u (shear), u+c
    const T va = tfma(k, dv, vl);
    const T i2c = rcp_pos(T(2) * ca);
    const T a1 = tabs(ua - ca) * (tfma(ua + ca, dh, -dm) * i2c);
    const T a3 = tabs(ua + ca) * (tfma(-(ua - ca), dh, dm) * i2c);
    const T a2 = tabs(ua) * (tfma(hr, vr, -(hl * vl)) - va * dh);
    F[0] = T(0.5) * ((ml + mr) - (a1 + a3));
    F[NM] = T(0.5) * (tfma(mr, ur, ml * ul) + hp - tfma(a3, ua + ca, a1 * (ua - ca)));
    F[TM] = T(0.5) * (tfma(mr, vr, ml * vl) - tfma(a1 + a3, va, a2));
    nr = F[NM] - hp;
}

// Euler: face values QL, QR and the cell averages CL, CR that replace them
// where they are not admissible -> F (Cartesian order).  The replacement is
// rare: it runs only in waves that need it.
template <typename T> __device__ __forceinline__ T eul_prim(const T *Q, int nm, int tm, T gm1, T &ir, T &u, T &v)
{
#pragma clang fp contract(off)
    ir = rcp(Q[0]);
    u = Q[nm] * ir;
    v = Q[tm] * ir;
    return gm1 * tfma(T(-0.5), tfma(Q[tm], v, Q[nm] * u), Q[3]);
}

template <typename T, int FLUX, int AXIS>
__device__ __forceinline__ void eul_face(T *QL, T *QR, const T *CL, const T *CR, const Phys<T> &ph, T *F)
{
#pragma clang fp contract(off)
    constexpr int NM = AXIS == 0 ? 1 : 2, TM = AXIS == 0 ? 2 : 1;
    const T gm1 = ph.gamma - T(1);
    T irl, ul, vl, irr, ur, vr;
    T pl = eul_prim(QL, NM, TM, gm1, irl, ul, vl), pr = eul_prim(QR, NM, TM, gm1, irr, ur, vr);
    const bool okl = QL[0] > T(0) && pl > T(0), okr = QR[0] > T(0) && pr > T(0);
    if (__any(!(okl && okr))) {
#pragma unroll
        for (int v = 0; v < 4; v++) {
            QL[v] = okl ? QL[v] : CL[v];
            QR[v] = okr ? QR[v] : CR[v];
        }
        pl = eul_prim(QL, NM, TM, gm1, irl, ul, vl);
        pr = eul_prim(QR, NM, TM, gm1, irr, ur, vr);
    }
    const T cl = fsqrt((ph.gamma * pl) * irl), cr = fsqrt((ph.gamma * pr) * irr);
    const T Hl = (QL[3] + pl) * irl, Hr = (QR[3] + pr) * irr;
    const T dr = QR[0] - QL[0], dm = QR[NM] - QL[NM];
    const T ml = QL[NM], mr = QR[NM], dt = QR[TM] - QL[TM], dE = QR[3] - QL[3];
    // twice the mean flux of the two states
    const T s0 = ml + mr, s1 = tfma(mr, ur, ml * ul) + (pl + pr), s2 = tfma(mr, vr, ml * vl), s3 = tfma(mr, Hr, ml * Hl);
    if constexpr (FLUX == RUSANOV) {
        const T a = tmax(tabs(ul) + cl, tabs(ur) + cr);
        F[0] = T(0.5) * tfma(-a, dr, s0);
        F[NM] = T(0.5) * tfma(-a, dm, s1);
        F[TM] = T(0.5) * tfma(-a, dt, s2);
        F[3] = T(0.5) * tfma(-a, dE, s3);
        return;
    }
    const T wl = fsqrt(QL[0]), wr = fsqrt(QR[0]);
    const T iw = rcp(wl + wr), kl = wl * iw, kr = wr * iw;
    const T ua = kl * ul + kr * ur, va = kl * vl + kr * vr, Ha = kl * Hl + kr * Hr;
    const T ca = fsqrt(tmax(gm1 * tfma(T(-0.5), tfma(va, va, ua * ua), Ha), T(0)));
    if constexpr (FLUX == ROE) {
        // acoustic u - c, entropy u, shear u, acoustic u + c
        const T a3 = tfma(-va, dr, dt);
        const T d5 = tfma(-a3, va, dE);
        const T a2 = gm1 * rcp(ca * ca) * (tfma(dr, tfma(-ua, ua, Ha), ua * dm) - d5);
        const T a1 = (tfma(dr, ua + ca, -dm) - ca * a2) * rcp(T(2) * ca);
        const T a4 = dr - (a1 + a2);
        const T w1 = tabs(ua - ca) * a1, w2 = tabs(ua) * a2, w3 = tabs(ua) * a3, w4 = tabs(ua + ca) * a4;
        const T w = w1 + w2 + w4;
        F[0] = T(0.5) * (s0 - w);
        F[NM] = T(0.5) * (s1 - tfma(w, ua, ca * (w4 - w1)));
        F[TM] = T(0.5) * (s2 - tfma(w, va, w3));
        F[3] = T(0.5) * (s3 - tfma(w1, tfma(-ua, ca, Ha), tfma(w4, tfma(ua, ca, Ha),
                                   tfma(w2, T(0.5) * tfma(ua, ua, va * va), w3 * va))));
        return;
    }
    const T sL = tmin(tmin(ul - cl, ua - ca), T(0));
    const T sR = tmax(tmax(ur + cr, ua + ca), T(0));
    const T w = rcp_near(sR - sL);  // sR - sL >= c~ > 0 for admissible states
    const T a = sR * w, b = -sL * w, c = (sL * sR) * w;
    const T x = a * ml, y = b * mr;
    F[0] = tfma(c, dr, x + y);
    F[NM] = tfma(c, dm, a * tfma(ml, ul, pl) + b * tfma(mr, ur, pr));
    F[TM] = tfma(c, dt, x * vl + y * vr);
    F[3] = tfma(c, dE, x * Hl + y * Hr);
}

// The face between two cells from its two face values, for either system;
// nr is the normal momentum flux as the high cell sees it (Euler: F's), jump
// the free surface's (shallow water).
template <typename T, int EQN, bool BATHY, int FLUX, int AXIS>
__device__ __forceinline__ void stage_face(T *QL, T *QR, const T *CL, const T *CR, T jump, const Phys<T> &ph,
                                           T *F, T &nr)
{
    if constexpr (EQN == EULER) {
        eul_face<T, FLUX, AXIS>(QL, QR, CL, CR, ph, F);
        nr = F[AXIS == 0 ? 1 : 2];
    } else {
        swe_face<T, BATHY, FLUX, AXIS>(QL, QR, jump, ph, F, nr);
    }
}

// The same from the four cells c[v][0..3] around it (the free surface as the
// last variable with a bed); slope: the free surface's slope in cell 2.
template <typename T, int EQN, bool BATHY, int FLUX, int RECON, int AXIS>
__device__ __forceinline__ void line_face(const T (*c)[4], const Phys<T> &ph, T *F, T &nr, T &slope)
{
#pragma clang fp contract(off)
    constexpr int NL = (EQN == SWE ? 3 : 4) + (BATHY ? 1 : 0);
    T ql[NL], qr[NL], cl[NL], cr[NL], jump = T(0);
#pragma unroll
    for (int v = 0; v < NL; v++) {
        const T d = c[v][2] - c[v][1];
        T x, sl, sr;
        cell_ends<T, RECON>(c[v][1], c[v][1] - c[v][0], d, x, ql[v], sl);
        cell_ends<T, RECON>(c[v][2], d, c[v][3] - c[v][2], qr[v], x, sr);
        cl[v] = c[v][1];
        cr[v] = c[v][2];
        if (v == (BATHY ? NL - 1 : 0)) {
            slope = sr;
            jump = face_jump<T, RECON>(d, sl, sr);
        }
    }
    stage_face<T, EQN, BATHY, FLUX, AXIS>(ql, qr, cl, cr, jump, ph, F, nr);
}

}  // namespace fvk
