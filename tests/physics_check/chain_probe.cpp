// The root and quotient chains of the device physics header (mhd_physics.hpp)
// on the host: the hardware estimates are stood in for by the exact value moved
// by up to +-2^-23 of itself (worse than the hardware's), the refinement is
// the header's own.  Prints, per function, the largest error in units of the
// last place of the exact result over the arguments of each range, and then the
// chains' values at zero, infinity and NaN.  Test infrastructure only.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#define __host__
#define __device__
#define __forceinline__ inline
#define VLCT_HOST_ESTIMATES
#include "mhd_physics.hpp"

static std::mt19937_64 rng(1);
static double uniform(double lo, double hi)
{
    return std::uniform_real_distribution<double>(lo, hi)(rng);
}
// one in four at either end of the error's range
static double moved(long double v)
{
    const int q = (int)(rng() & 3);
    const double d = q == 0 ? 1.0 : (q == 1 ? -1.0 : uniform(-1.0, 1.0));
    return (double)(v * (1.0L + (long double)d * 0x1p-23L));
}
namespace vlct {
double rsq_estimate(double x) { return moved(1.0L / sqrtl((long double)x)); }
double rcp_estimate(double x) { return moved(1.0L / (long double)x); }
}

static double ulps(double got, long double want)
{
    int e;
    frexpl(want, &e);
    return (double)(fabsl((long double)got - want) / ldexpl(1.0L, e - 53));
}

int main(int argc, char **argv)
{
    const int n = argc > 1 ? atoi(argv[1]) : 1000000;
    const double lo[3] = {1.0, 1e-30, 1e-150}, hi[3] = {4.0, 1e30, 1e150};
    for (int r = 0; r < 3; ++r) {
        double m[4] = {0, 0, 0, 0};
        for (int i = 0; i < n; ++i) {
            const double x = r == 0 ? uniform(lo[r], hi[r]) : exp(uniform(log(lo[r]), log(hi[r])));
            const double a = r == 0 ? uniform(lo[r], hi[r]) : exp(uniform(log(lo[r]), log(hi[r])));
            const long double X = x, A = a;
            m[0] = fmax(m[0], ulps(vlct::msqrt(x), sqrtl(X)));
            m[1] = fmax(m[1], ulps(vlct::mrsqrt(x), 1.0L / sqrtl(X)));
            m[2] = fmax(m[2], ulps(vlct::mrcp(x), 1.0L / X));
            m[3] = fmax(m[3], ulps(vlct::mdiv(a, x), A / X));
        }
        printf("%.17g %.17g %.17g %.17g\n", m[0], m[1], m[2], m[3]);
    }
    // roots of the smallest normal numbers
    double m = 0.0;
    for (int i = 0; i < n; ++i) {
        const double x = exp(uniform(log(2.3e-308), log(1e-290)));
        m = fmax(m, ulps(vlct::msqrt(x), sqrtl((long double)x)));
    }
    printf("%.17g\n", m);
    printf("%.17g %d %.17g\n", vlct::msqrt(0.0), (int)std::isnan(vlct::msqrt(NAN)), vlct::mdiv(0.0, 3.0));
}
