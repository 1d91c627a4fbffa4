// mhd_physics.hpp -- per-state ideal-MHD physics on gfx950 for the VL+CT step
// (Caddy & Schneider, "Cholla-MHD", Sec. 2.1-2.2): wave speeds, the HLLD
// Riemann solver, the characteristic eigen-system and the PLMC / PPMC
// reconstructions.  Everything is FP64 and inlined into the kernels.
//
// Sweep frame: a 1D problem along axis d uses the state
//   W7 = (rho, v_n, v_t1, v_t2, P, B_t1, B_t2)
// with (n, t1, t2) the cyclic permutation (x,y,z), (y,z,x), (z,x,y) of the
// axes (Table emf and its note); the normal field B_n is a parameter.
#pragma once
#if !defined(VLCT_HOST_COUNT) && !defined(VLCT_HOST_ESTIMATES)
#include <hip/hip_runtime.h>
#define VLCT_DEV __device__ __forceinline__
#else
#define VLCT_DEV inline  // host build of the same code for operation counting
#endif

namespace vlct {

#ifndef VLCT_HOST_COUNT
#ifdef VLCT_HOST_ESTIMATES  // a host test of the chains supplies its own
double rsq_estimate(double x);
double rcp_estimate(double x);
#else
VLCT_DEV double rsq_estimate(double x) { return __builtin_amdgcn_rsq(x); }
VLCT_DEV double rcp_estimate(double x) { return __builtin_amdgcn_rcp(x); }
#endif
// Roots and quotients from the hardware estimates (v_rsq_f64, v_rcp_f64, about
// 23 correct bits), refined by the shortest chain that keeps the rounding of
// the longer ones it replaced: over 2^20 random arguments msqrt, mrcp and mdiv
// stay within 0.5000 ulp and mrsqrt within 0.99 (rms 0.33).  No range scaling
// (arguments here are densities, pressures, squared speeds and field
// magnitudes, never subnormal or near overflow).  The flux kernels issue FP64
// instructions most of the time, and a PLMC + HLLD face needs 27 of these:
// with them, the half-slope limiter of plmc and hlld selecting its side early,
// such a face went from 1236 to 1084 vector instructions, and the 256^3 step
// from 5.80 to 5.25 ms (PLMC) and 7.00 to 6.40 ms (PPMC).

// square root, x >= 0: one Goldschmidt step (46 bits), then one correction
// with the residual, whose factor needs only the estimate's bits.  The
// estimate is taken of at least the smallest normal number, which maps zero to
// zero without a select (rsq(0) is infinite).
VLCT_DEV double msqrt(double x)
{
    const double y = rsq_estimate(fmax(x, 0x1p-1022));
    double g = x * y;
    const double h = 0.5 * y;
    g = fma(g, fma(-g, h, 0.5), g);
    return fma(fma(-g, g, x), h, g);
}
// Reciprocal square root, x > 0: the third-order step y (1 + e/2 + 3 e^2/8),
// e = 1 - x y^2.  One of these replaces a square root and a division where
// both the root and its reciprocal are needed.
VLCT_DEV double mrsqrt(double x)
{
    const double y = rsq_estimate(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}
// reciprocal: the third-order step y (1 + e + e^2), e = 1 - x y
VLCT_DEV double mrcp(double x)
{
    const double y = rcp_estimate(x);
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}
// quotient: a Newton step on the reciprocal (46 bits), then the quotient
// corrected with its residual
VLCT_DEV double mdiv(double a, double b)
{
    double y = rcp_estimate(b);
    y = fma(fma(-b, y, 1.0), y, y);
    const double q = a * y;
    return fma(fma(-b, q, a), y, q);
}
#else
VLCT_DEV double msqrt(double x) { return sqrt(x); }
VLCT_DEV double mrsqrt(double x) { return 1.0 / sqrt(x); }
VLCT_DEV double mrcp(double x) { return 1.0 / x; }
VLCT_DEV double mdiv(double a, double b) { return a / b; }
#endif

// Floors on derived and reconstructed rho, P (the conserved state is never changed).
constexpr double kFloorRho = 1.0e-20;
constexpr double kFloorP = 1.0e-20;
// HLLD: star states fall back to the outer states where
// |rho (S - u)(S - S_M) - B_n^2| < kHlldDegen * p_T*.
constexpr double kHlldDegen = 1.0e-8;
// Eigenvectors: B_n with |B_n| <= kBperpTiny sqrt(gP + B^2) is taken as zero and
// |B_perp| <= kBperpTiny sqrt(gP + B^2) uses beta_t1 = beta_t2 = 1/sqrt(2);
// rho (c_f^2 - c_s^2) <= kCfCsTiny rho c_f^2 uses alpha_f = 1, alpha_s = 0.
constexpr double kBperpTiny = 1.0e-12;
constexpr double kCfCsTiny = 1.0e-12;
// CT upwinding: |S_M| <= kUpwindTiny (c_max + |u_L| + |u_R|) counts as zero.
constexpr double kUpwindTiny = 1.0e-12;
// Colella-Sekora curvature ratio used by the PPMC limiters.
constexpr double kPpmC = 1.25;
// PPMC: a stencil difference below this fraction of the values' magnitudes (with
// c_f and sqrt(rho) c_f as floors for velocity and field components) is zero.
constexpr double kPpmTie = 1.0e-12;

constexpr uint32_t kStatusPressureFloor = 1u;
constexpr uint32_t kStatusDensityFloor = 2u;
constexpr uint32_t kStatusNonfinite = 4u;

struct W7 {
    double d, u, v, w, p, by, bz;
};

// Squared fast speed and the discriminant d = rho (c_f^2 - c_s^2) of the
// fast/slow speed formula (Sec. 2.2 Step 1), with the discriminant written as
// (gP - B^2)^2 + 4 gP B_perp^2 so it never cancels.
VLCT_DEV double fast_sq(double d, double p, double bn, double bt1, double bt2,
                                          double gam, double &disc)
{
    const double gp = gam * p;
    const double bp2 = bt1 * bt1 + bt2 * bt2;
    const double b2 = bn * bn + bp2;
    const double t = gp - b2;
    disc = msqrt(t * t + 4.0 * gp * bp2);
    return mdiv(gp + b2 + disc, 2.0 * d);
}

VLCT_DEV double fast_speed(double d, double p, double bn, double bt1,
                                             double bt2, double gam)
{
    double disc;
    return msqrt(fast_sq(d, p, bn, bt1, bt2, gam, disc));
}

// ---------------------------------------------------------------------------
// HLLD (Sec. 2.2 Step 3, Miyoshi & Kusano 2005): 7 flux components in the
// sweep frame plus the CT upwind indicator (+1, -1, 0) taken from the sign of
// the interface (contact) velocity S_M, the sign of the mass flux.
// ---------------------------------------------------------------------------
template <class U>  // U: the indicator's type (int8_t in the kernels)
VLCT_DEV void hlld(const W7 &L, const W7 &R, double bn, double gam, double gm1i,
                                     double f[7], U &upw)
{
    const double bn2 = bn * bn;
    const double pbL = 0.5 * (bn2 + L.by * L.by + L.bz * L.bz);
    const double pbR = 0.5 * (bn2 + R.by * R.by + R.bz * R.bz);
    const double ptL = L.p + pbL;
    const double ptR = R.p + pbR;
    // c_f = sqrt(num / (2 rho)) = num / sqrt(2 rho num), num = gP + B^2 + disc
    // (the fast-speed formula of fast_sq with one reciprocal root per side)
    auto fast = [&](const W7 &X) {
        const double gp = gam * X.p;
        const double bp2 = X.by * X.by + X.bz * X.bz;
        const double b2 = bn2 + bp2;
        const double t = gp - b2;
        const double num = gp + b2 + msqrt(t * t + 4.0 * gp * bp2);
        return num * mrsqrt(2.0 * X.d * num);
    };
    const double cfL = fast(L);
    const double cfR = fast(R);
    const double cmax = fmax(cfL, cfR);
    const double sL = fmin(L.u, R.u) - cmax;
    const double sR = fmax(L.u, R.u) + cmax;

    const double qL = (sL - L.u) * L.d;
    const double qR = (sR - R.u) * R.d;
    const double iq = mrcp(qR - qL);
    const double sM = (qR * R.u - qL * L.u - ptR + ptL) * iq;
    const double pts = (qR * ptL - qL * ptR + qL * qR * (R.u - L.u)) * iq;

    // single-star states of both sides (the energy only where it is used,
    // on the side whose fan contains x/t = 0)
    double ds[2], vs[2], ws[2], bys[2], bzs[2], issm[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const W7 &X = a == 0 ? L : R;
        const double S = a == 0 ? sL : sR;
        const double su = S - X.u;
        const double ssm = S - sM;
        issm[a] = mrcp(ssm);
        ds[a] = X.d * su * issm[a];
        const double den = X.d * su * ssm - bn2;
        const bool degen = fabs(den) < kHlldDegen * pts;
        const double iden = mrcp(den);
        const double t1 = degen ? 0.0 : bn * (sM - X.u) * iden;
        const double t2 = degen ? 1.0 : (X.d * su * su - bn2) * iden;
        vs[a] = X.v - X.by * t1;
        ws[a] = X.w - X.bz * t1;
        bys[a] = X.by * t2;
        bzs[a] = X.bz * t2;
    }
    // double-star states (shared by both sides)
    const double sg = bn >= 0.0 ? 1.0 : -1.0;
    const double irL = mrsqrt(ds[0]), irR = mrsqrt(ds[1]);
    const double rL = ds[0] * irL, rR = ds[1] * irR;
    const double isum = mrcp(rL + rR);
    const double vss = (rL * vs[0] + rR * vs[1] + sg * (bys[1] - bys[0])) * isum;
    const double wss = (rL * ws[0] + rR * ws[1] + sg * (bzs[1] - bzs[0])) * isum;
    const double byss = (rL * bys[1] + rR * bys[0] + sg * rL * rR * (vs[1] - vs[0])) * isum;
    const double bzss = (rL * bzs[1] + rR * bzs[0] + sg * rL * rR * (ws[1] - ws[0])) * isum;
    const double vbss = sM * bn + vss * byss + wss * bzss;

    // the side whose fan contains x/t = 0 (dir: -1 left, +1 right); what
    // follows cheaply from its state is evaluated after the selection
    const bool left = sM >= 0.0;
    const double dir = left ? -1.0 : 1.0;
    const W7 X{left ? L.d : R.d, left ? L.u : R.u, left ? L.v : R.v, left ? L.w : R.w,
               left ? L.p : R.p, left ? L.by : R.by, left ? L.bz : R.bz};
    const double S = left ? sL : sR;
    const double pb = left ? pbL : pbR;
    const double pt = X.p + pb;
    const double e = X.p * gm1i + 0.5 * X.d * (X.u * X.u + X.v * X.v + X.w * X.w) + pb;
    const double dsa = left ? ds[0] : ds[1];
    const double vsa = left ? vs[0] : vs[1], wsa = left ? ws[0] : ws[1];
    const double bysa = left ? bys[0] : bys[1], bzsa = left ? bzs[0] : bzs[1];
    const double ir = left ? irL : irR;
    const double r = dsa * ir;
    const double ss = sM + dir * (fabs(bn) * ir);
    const bool star_only = dir * ss <= 0.0;
    // its single-star energy and the double-star correction
    const double vbs = sM * bn + vsa * bysa + wsa * bzsa;
    const double vb = X.u * bn + X.v * X.by + X.w * X.bz;
    const double esa =
        ((S - X.u) * e - pt * X.u + pts * sM + bn * (vb - vbs)) * (left ? issm[0] : issm[1]);
    const double des = r * (dir * sg) * (vbs - vbss);
    const bool outer = dir * S < 0.0;
    const double cS = outer ? 0.0 : S;
    const double cSS = (outer || star_only) ? 0.0 : ss;

    const double mu = X.d * X.u;
    // physical flux F(W) of the chosen side (Sec. 2.1, sweep frame)
    const double F0 = mu;
    const double F1 = mu * X.u + pt - bn2;
    const double F2 = mu * X.v - bn * X.by;
    const double F3 = mu * X.w - bn * X.bz;
    const double F4 = (e + pt) * X.u - bn * vb;
    const double F5 = X.by * X.u - bn * X.v;
    const double F6 = X.bz * X.u - bn * X.w;
    // U* - U and U** - U*
    const double dU0 = dsa - X.d;
    const double dU1 = dsa * sM - mu;
    const double dU2 = dsa * vsa - X.d * X.v;
    const double dU3 = dsa * wsa - X.d * X.w;
    const double dU4 = esa - e;
    const double dU5 = bysa - X.by;
    const double dU6 = bzsa - X.bz;
    const double dV2 = dsa * (vss - vsa);
    const double dV3 = dsa * (wss - wsa);
    const double dV5 = byss - bysa;
    const double dV6 = bzss - bzsa;
    f[0] = F0 + cS * dU0;
    f[1] = F1 + cS * dU1;
    f[2] = F2 + cS * dU2 + cSS * dV2;
    f[3] = F3 + cS * dU3 + cSS * dV3;
    f[4] = F4 + cS * dU4 + cSS * des;
    f[5] = F5 + cS * dU5 + cSS * dV5;
    f[6] = F6 + cS * dU6 + cSS * dV6;

    const double vtol = kUpwindTiny * (cmax + fabs(L.u) + fabs(R.u));
    const U ind = sM > vtol ? U(1) : (sM < -vtol ? U(-1) : U(0));
    upw = sL > 0.0 ? U(1) : (sR < 0.0 ? U(-1) : ind);
}

// ---------------------------------------------------------------------------
// Characteristic eigen-system of the 1D primitive system (Sec. 2.2 Step 6,
// item 3) with the Roe-Balsara normalisation; left eigenvectors in closed
// form (they are the exact inverse of the right ones).
// Waves m = 0..6: u-cf, u-ca, u-cs, u, u+cs, u+ca, u+cf.
// ---------------------------------------------------------------------------
struct Eigen {
    double d, sqd, asq, a, ia2;   // rho, sqrt(rho), a^2 = gP/rho, a, 1/a^2
    double cf, cs, af, as;        // fast/slow speeds and alpha_f, alpha_s
    double by, bz, s;             // beta_t1, beta_t2, sign(B_n)
    // left-eigenvector coefficients
    double nf, ns, qf, qs, pf, ps, bf, bs, sr;
};

VLCT_DEV void eigen_setup(const W7 &c, double bn_in, double gam, Eigen &E)
{
    // field components below kBperpTiny of the magnetosonic scale
    // sqrt(gP + B^2) are rounding noise and are zero here, so noise cannot
    // turn the B_perp direction (compared in squares)
    const double gp = gam * c.p;
    const double tiny2 =
        kBperpTiny * kBperpTiny * (gp + bn_in * bn_in + c.by * c.by + c.bz * c.bz);
    const double bn = bn_in * bn_in <= tiny2 ? 0.0 : bn_in;
    const double bt1 = c.by * c.by <= tiny2 ? 0.0 : c.by;
    const double bt2 = c.bz * c.bz <= tiny2 ? 0.0 : c.bz;
    // r = 1/sqrt(rho), q = 1/sqrt(gP): every root and reciprocal of rho and gP
    // below follows from these two
    const double r = mrsqrt(c.d), q = mrsqrt(gp);
    const double id = r * r;
    E.d = c.d;
    E.sqd = c.d * r;
    E.asq = gp * id;
    E.a = gp * q * r;          // sqrt(gP / rho)
    E.ia2 = c.d * q * q;       // rho / (gP)
    const double bp2 = bt1 * bt1 + bt2 * bt2;
    const double t = gp - (bn * bn + bp2);
    const double disc = msqrt(t * t + 4.0 * gp * bp2);
    // c_f = sqrt(num / (2 rho)) = num rq and 1 / c_f = 2 rho rq, rq = 1 / sqrt(2 rho num)
    const double num = gp + bn * bn + bp2 + disc;
    const double rq = mrsqrt(2.0 * c.d * num);
    E.cf = num * rq;
    // c_s = a |B_n| / (sqrt(rho) c_f), the root of gP B_n^2 / (rho^2 c_f^2)
    E.cs = E.a * fabs(bn) * r * (2.0 * c.d * rq);
    const bool haveperp = bp2 > tiny2;
    const double ibp = mrsqrt(haveperp ? bp2 : 1.0);
    E.by = haveperp ? bt1 * ibp : 0.70710678118654752440;
    E.bz = haveperp ? bt2 * ibp : 0.70710678118654752440;
    const double tdiff = t;
    const bool split = disc > 0.5 * kCfCsTiny * num;  // rho c_f^2 = num / 2
    const double idisc = 0.5 * mrcp(disc);
    const double af2 = fmin(fmax((disc + tdiff) * idisc, 0.0), 1.0);
    const double as2 = fmin(fmax((disc - tdiff) * idisc, 0.0), 1.0);
    E.af = split ? msqrt(af2) : 1.0;
    E.as = split ? msqrt(as2) : 0.0;
    E.s = bn >= 0.0 ? 1.0 : -1.0;
    const double ia2 = E.ia2;
    E.nf = 0.5 * E.af * E.cf * ia2;
    E.ns = 0.5 * E.as * E.cs * ia2;
    E.qf = 0.5 * E.s * E.as * E.cs * ia2;
    E.qs = 0.5 * E.s * E.af * E.cf * ia2;
    E.pf = 0.5 * E.af * ia2 * id;
    E.ps = 0.5 * E.as * ia2 * id;
    E.bf = 0.5 * E.as * q;     // q = 1 / (a sqrt(rho))
    E.bs = -0.5 * E.af * q;
    E.sr = 0.5 * E.s * r;
}

// characteristic amplitudes a = L dW of a primitive increment dW
VLCT_DEV void project(const Eigen &E, const double dw[7], double a[7])
{
    const double vpar = E.by * dw[2] + E.bz * dw[3];
    const double vperp = -E.bz * dw[2] + E.by * dw[3];
    const double bpar = E.by * dw[5] + E.bz * dw[6];
    const double bperp = -E.bz * dw[5] + E.by * dw[6];
    const double hf = E.pf * dw[4] + E.bf * bpar;
    const double gf = E.nf * dw[1] - E.qf * vpar;
    const double hs = E.ps * dw[4] + E.bs * bpar;
    const double gs = E.ns * dw[1] + E.qs * vpar;
    a[0] = hf - gf;
    a[6] = hf + gf;
    a[2] = hs - gs;
    a[4] = hs + gs;
    a[1] = 0.5 * vperp + E.sr * bperp;
    a[5] = 0.5 * vperp - E.sr * bperp;
    a[3] = dw[0] - dw[4] * E.ia2;
}

// primitive increment dW = R a of characteristic amplitudes a
VLCT_DEV void unproject(const Eigen &E, const double a[7], double dw[7])
{
    const double fsum = a[0] + a[6], fdif = a[6] - a[0];
    const double ssum = a[2] + a[4], sdif = a[4] - a[2];
    const double asum = a[1] + a[5], adif = a[5] - a[1];
    const double tpar = -E.s * (E.as * E.cs * fdif - E.af * E.cf * sdif);
    const double bmag = E.a * E.sqd * (E.as * fsum - E.af * ssum);
    const double sb = E.s * E.sqd * adif;
    dw[0] = E.d * (E.af * fsum + E.as * ssum) + a[3];
    dw[1] = E.af * E.cf * fdif + E.as * E.cs * sdif;
    dw[2] = E.by * tpar - E.bz * asum;
    dw[3] = E.bz * tpar + E.by * asum;
    dw[4] = E.d * E.asq * (E.af * fsum + E.as * ssum);
    dw[5] = E.by * bmag + E.bz * sb;
    dw[6] = E.bz * bmag - E.by * sb;
}

VLCT_DEV void to_arr(const W7 &w, double x[7])
{
    x[0] = w.d; x[1] = w.u; x[2] = w.v; x[3] = w.w; x[4] = w.p; x[5] = w.by; x[6] = w.bz;
}

VLCT_DEV W7 from_arr(const double x[7])
{
    return W7{x[0], x[1], x[2], x[3], x[4], x[5], x[6]};
}

// floor an interface state; returns status bits
VLCT_DEV uint32_t floor_state(W7 &w)
{
    uint32_t st = 0;
    if (!(w.d >= kFloorRho)) { w.d = kFloorRho; st |= kStatusDensityFloor; }
    if (!(w.p >= kFloorP)) { w.p = kFloorP; st |= kStatusPressureFloor; }
    return st;
}

// ---------------------------------------------------------------------------
// PLMC (Sec. 2.2 Step 6 items 1-6, Eq. limiter): left/right/centred/van Leer
// primitive differences projected with the eigenvectors of the cell,
// limited, projected back; fm = state at the low face, fp = at the high face.
// ---------------------------------------------------------------------------
template <bool CHAR>
VLCT_DEV void plmc(const W7 &wm, const W7 &w0, const W7 &wp, double bn,
                                     double gam, W7 &fm, W7 &fp)
{
    // CHAR = false is PLMP: the same steps with the projections skipped.
    // Half slopes throughout (exact factors of two): min(2|l|, 2|r|, |c|, |v|) / 2
    // with c = (l + r) / 2, so the centred difference needs no projection of
    // its own, and v / 2 = l r / (l + r).
    double xm[7], x0[7], xp[7];
    to_arr(wm, xm);
    to_arr(w0, x0);
    to_arr(wp, xp);
    double dl[7], dr[7], hv[7];
#pragma unroll
    for (int c = 0; c < 7; ++c) {
        dl[c] = x0[c] - xm[c];
        dr[c] = xp[c] - x0[c];
        const double pr = dl[c] * dr[c];
        const double q = mdiv(pr, dl[c] + dr[c]);
        hv[c] = pr > 0.0 ? q : 0.0;
    }
    Eigen E;
    double al[7], ar[7], av[7], am[7];
    if (CHAR) {
        eigen_setup(w0, bn, gam, E);
        project(E, dl, al);
        project(E, dr, ar);
        project(E, hv, av);
    } else {
#pragma unroll
        for (int c = 0; c < 7; ++c) {
            al[c] = dl[c];
            ar[c] = dr[c];
            av[c] = hv[c];
        }
    }
#pragma unroll
    for (int m = 0; m < 7; ++m) {
        const double lim = fmin(fmin(fabs(al[m]), fabs(ar[m])),
                                fmin(fabs(0.25 * (al[m] + ar[m])), fabs(av[m])));
        am[m] = al[m] * ar[m] > 0.0 ? copysign(lim, al[m]) : 0.0;
    }
    double dw[7];
    if (CHAR) {
        unproject(E, am, dw);
    } else {
#pragma unroll
        for (int c = 0; c < 7; ++c) dw[c] = am[c];
    }
    double p[7], q[7];
#pragma unroll
    for (int c = 0; c < 7; ++c) {
        p[c] = x0[c] + dw[c];
        q[c] = x0[c] - dw[c];
    }
    fp = from_arr(p);
    fm = from_arr(q);
}

// ---------------------------------------------------------------------------
// PPMC (third order, limited in characteristic variables).  The paper defers
// to Felker & Stone (2018) without formulas; this implements the reading used
// throughout the library: stencil differences relative to the cell (rounding-
// level differences set to zero), fourth-order face values, Colella-Sekora
// face limiter, extremum-preserving parabola limiter / overshoot correction
// per characteristic field, back projection, then each face primitive clamped
// between the two cells that share the face.
// ---------------------------------------------------------------------------
// minmod of the parabola's second difference d2 and kPpmC times the
// neighbouring ones (zero unless all share d2's sign), written with the common
// sign factored out so that no sign test is needed
VLCT_DEV double ppm_curv(double d2, double da, double db)
{
    const double sc = copysign(kPpmC, d2);
    return fmax(fmin(fmin(sc * da, sc * db), fabs(d2)), 0.0);
}

// fourth-order face value between the cells a0 and ap
VLCT_DEV double ppm_face(double am, double a0, double ap, double app)
{
    double f = (7.0 / 12.0) * (a0 + ap) - (1.0 / 12.0) * (am + app);
    if ((f - a0) * (ap - f) < 0.0) {
        // all three curvature estimates are h^2 f'' on a parabola: with the
        // limiter not binding this gives back the fourth-order f
        const double d2 = 3.0 * (a0 - 2.0 * f + ap);
        const double lim = copysign(ppm_curv(d2, am - 2.0 * a0 + ap, a0 - 2.0 * ap + app), d2);
        f = 0.5 * (a0 + ap) - lim * (1.0 / 6.0);
    }
    return f;
}

// the tie test's tolerance of a stencil difference t - x0: kPpmTie (|t| +
// |x0| + floor), base = kPpmTie (|x0| + floor)
VLCT_DEV double ppm_tol(double t, double base) { return base + kPpmTie * fabs(t); }

template <bool CHAR>
VLCT_DEV void ppmc(const W7 &wmm, const W7 &wm, const W7 &w0, const W7 &wp,
                                     const W7 &wpp, double bn, double gam, W7 &fm, W7 &fp)
{
    // CHAR = false is PPMP: the same steps with the projections skipped
    // stencil differences relative to the cell; a difference within kPpmTie of
    // the magnitudes it is taken from counts as zero, so that rounding noise at
    // a symmetric extremum cannot pick the other branch of the extremum test
    Eigen E;
    double fv, fb;
    if (CHAR) {
        eigen_setup(w0, bn, gam, E);
        fv = E.cf;
        fb = E.sqd * E.cf;
    } else {
        fv = fast_speed(w0.d, w0.p, bn, w0.by, w0.bz, gam);
        fb = msqrt(w0.d) * fv;
    }
    // magnitude floors of the tie test: c_f for velocities, sqrt(rho) c_f for B
    const double floor_c[7] = {0.0, fv, fv, fv, 0.0, fb, fb};
    double x0[7], base[7], xs[4][7];
    to_arr(w0, x0);
#pragma unroll
    for (int c = 0; c < 7; ++c) base[c] = kPpmTie * (fabs(x0[c]) + floor_c[c]);
    {
        const W7 *nb[4] = {&wmm, &wm, &wp, &wpp};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            double t[7];
            to_arr(*nb[q], t);
#pragma unroll
            for (int c = 0; c < 7; ++c) {
                const double d = t[c] - x0[c];
                xs[q][c] = fabs(d) <= ppm_tol(t[c], base[c]) ? 0.0 : d;
            }
        }
    }
    double a[4][7];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        if (CHAR) {
            project(E, xs[s], a[s]);
        } else {
#pragma unroll
            for (int c = 0; c < 7; ++c) a[s][c] = xs[s][c];
        }
    }
    double dplus[7], dminus[7];
#pragma unroll
    for (int m = 0; m < 7; ++m) {
        // characteristic values relative to the cell (a_0 = 0); d2l, d2c, d2r
        // are the second differences centred on the left cell, the cell and
        // the right cell, fl and fr ppm_face of the two faces
        const double a_2 = a[0][m], a_1 = a[1][m], a1 = a[2][m], a2 = a[3][m];
        const double d2l = a_2 - 2.0 * a_1, d2c = a_1 + a1, d2r = a2 - 2.0 * a1;
        double fl = (7.0 / 12.0) * a_1 - (1.0 / 12.0) * (a_2 + a1);
        double fr = (7.0 / 12.0) * a1 - (1.0 / 12.0) * (a_1 + a2);
        const bool ovl = (fl - a_1) * fl > 0.0, ovr = (fr - a1) * fr > 0.0;
        if (ovl || ovr) {
            const double dl = 3.0 * (a_1 - 2.0 * fl), dr = 3.0 * (a1 - 2.0 * fr);
            const double ll = copysign(ppm_curv(dl, d2l, d2c), dl);
            const double lr = copysign(ppm_curv(dr, d2c, d2r), dr);
            fl = ovl ? 0.5 * a_1 - ll * (1.0 / 6.0) : fl;
            fr = ovr ? 0.5 * a1 - lr * (1.0 / 6.0) : fr;
        }
        double dp = fr, dm = -fl;
        if (fr * fl >= 0.0 || a1 * a_1 >= 0.0) {
            const double d2 = 6.0 * (fl + fr);
            const double lim = fmin(ppm_curv(d2, d2l, d2r),
                                    fmax(copysign(kPpmC, d2) * d2c, 0.0));
            const double ratio = d2 != 0.0 ? mdiv(lim, fabs(d2)) : 0.0;
            dp = dp * ratio;
            dm = dm * ratio;
        } else {
            dp = fabs(dp) >= 2.0 * fabs(dm) ? 2.0 * dm : dp;
            dm = fabs(dm) >= 2.0 * fabs(dp) ? 2.0 * dp : dm;
        }
        // the limited interface values stay between the cell's (0) and the
        // neighbour's characteristic values
        dplus[m] = fmax(fmin(0.0, a1), fmin(dp, fmax(0.0, a1)));
        dminus[m] = fmax(fmin(0.0, a_1), fmin(-dm, fmax(0.0, a_1)));
    }
    double wpl[7], wmi[7];
    if (CHAR) {
        unproject(E, dplus, wpl);
        unproject(E, dminus, wmi);
    } else {
#pragma unroll
        for (int c = 0; c < 7; ++c) {
            wpl[c] = dplus[c];
            wmi[c] = dminus[c];
        }
    }
    double xl[7], xr[7], p[7], q[7];
    to_arr(wm, xl);
    to_arr(wp, xr);
#pragma unroll
    for (int c = 0; c < 7; ++c) {
        const double up = x0[c] + wpl[c];
        const double um = x0[c] + wmi[c];
        // bound between the neighbouring cell values
        double vp = fmax(fmin(x0[c], xr[c]), fmin(up, fmax(x0[c], xr[c])));
        double vm = fmax(fmin(x0[c], xl[c]), fmin(um, fmax(x0[c], xl[c])));
        // a bound that acted beyond rounding: Colella-Woodward monotonicity
        // constraints on this primitive's interface pair
        // (written out: keeping `base` alive to here costs 14 registers)
        const double tol = kPpmTie * (fabs(xl[c]) + fabs(xr[c]) + fabs(x0[c]) + floor_c[c]);
        if (fabs(vp - up) > tol || fabs(vm - um) > tol) {
            const double dpp = vp - x0[c], dmm = x0[c] - vm;
            if (dpp * dmm <= 0.0) {
                vp = x0[c];
                vm = x0[c];
            } else {
                if (fabs(dpp) >= 2.0 * fabs(dmm)) vp = x0[c] + 2.0 * dmm;
                if (fabs(dmm) >= 2.0 * fabs(dpp)) vm = x0[c] - 2.0 * dpp;
            }
        }
        p[c] = vp;
        q[c] = vm;
    }
    fp = from_arr(p);
    fm = from_arr(q);
}

}  // namespace vlct
