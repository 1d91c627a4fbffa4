// Host build of the device physics header (mhd_physics.hpp) with the device's
// own root and quotient chains (VLCT_HOST_ESTIMATES: the hardware estimates
// stood in for by the exact value moved by up to 2^-24 of itself) or with the
// library's roots and quotients (VLCT_HOST_COUNT).  The first argument names
// the form; each line of input is one case:
//   plmc, plmp: 3 cells of 7 primitives, bn, gamma -> low, high face state
//   ppmc, ppmp: 5 cells                            -> low, high face state
//   hlld:       2 states                           -> 7 fluxes, upwind indicator
//   curv:       d2, da, db                         -> ppm_curv(d2, da, db)
// Test infrastructure only.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#define __host__
#define __device__
#define __forceinline__ inline
#include "mhd_physics.hpp"

#ifdef VLCT_HOST_ESTIMATES
static std::mt19937_64 rng(2);
static double moved(long double v)
{
    return (double)(v * (1.0L + std::uniform_real_distribution<double>(-1.0, 1.0)(rng) * 0x1p-24L));
}
namespace vlct {
double rsq_estimate(double x) { return moved(1.0L / sqrtl((long double)x)); }
double rcp_estimate(double x) { return moved(1.0L / (long double)x); }
}
#endif

using vlct::W7;
static W7 w7(const double *c) { return W7{c[0], c[1], c[2], c[3], c[4], c[5], c[6]}; }

int main(int argc, char **argv)
{
    const char *form = argc > 1 ? argv[1] : "";
    auto is = [&](const char *s) { return std::strcmp(form, s) == 0; };
    const bool plm = is("plmc") || is("plmp"), ppm = is("ppmc") || is("ppmp");
    const int n = plm ? 23 : (ppm ? 37 : (is("hlld") ? 16 : 3));
    double a[37];
    while (true) {
        for (int q = 0; q < n; ++q)
            if (scanf("%lf", &a[q]) != 1) return 0;
        if (is("curv")) {
            printf("%.17g\n", vlct::ppm_curv(a[0], a[1], a[2]));
            continue;
        }
        if (is("hlld")) {
            double f[7];
            int8_t up;
            vlct::hlld(w7(a), w7(a + 7), a[14], a[15], 1.0 / (a[15] - 1.0), f, up);
            for (int q = 0; q < 7; ++q) printf("%.17g ", f[q]);
            printf("%d\n", (int)up);
            continue;
        }
        W7 m, p;
        const double bn = a[n - 2], gam = a[n - 1];
        if (is("plmc")) vlct::plmc<true>(w7(a), w7(a + 7), w7(a + 14), bn, gam, m, p);
        if (is("plmp")) vlct::plmc<false>(w7(a), w7(a + 7), w7(a + 14), bn, gam, m, p);
        if (is("ppmc"))
            vlct::ppmc<true>(w7(a), w7(a + 7), w7(a + 14), w7(a + 21), w7(a + 28), bn, gam, m, p);
        if (is("ppmp"))
            vlct::ppmc<false>(w7(a), w7(a + 7), w7(a + 14), w7(a + 21), w7(a + 28), bn, gam, m, p);
        const double o[14] = {m.d, m.u, m.v, m.w, m.p, m.by, m.bz, p.d, p.u, p.v, p.w, p.p, p.by, p.bz};
        for (int q = 0; q < 14; ++q) printf("%.17g%c", o[q], q == 13 ? '\n' : ' ');
    }
}
