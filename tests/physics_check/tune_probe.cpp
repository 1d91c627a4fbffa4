// Host build of the batch tuner's search (batch_tune.hpp) on made-up times:
// reads "seed noise drift gain_class gain" lines and prints the plan found for
// runs of 16, 32, 64 and 128 cells.  A step takes 1 ms, or (1 - gain) of it
// under a plan that gives the runs of that size class CT tile 1 (class < 0:
// none does); every timing is off by up to +-noise, and the machine gets faster
// by `drift` per timing.  Test infrastructure only.
#include <cstdio>
#include <random>

#include "batch_tune.hpp"

int main()
{
    unsigned seed;
    double noise, drift, gain;
    int cls;
    while (scanf("%u %lf %lf %d %lf", &seed, &noise, &drift, &cls, &gain) == 5) {
        std::mt19937 rng(seed);
        std::uniform_real_distribution<double> u(-noise, noise);
        double speed = 1.0;
        const std::vector<int> nx{16, 32, 64, 128};
        std::vector<uint8_t> plan;
        const int rc = vlct::tune_plan(nx, 3, 3, [&](const std::vector<uint8_t> &p, float &ms) {
            const bool fast = cls >= 0 && (p[cls] & 15) == 1;
            speed *= 1.0 - drift;
            ms = (float)(speed * (fast ? 1.0 - gain : 1.0) * (1.0 + u(rng)));
            return 0;
        }, plan);
        printf("%d %d %d %d %d\n", rc, plan[0], plan[1], plan[2], plan[3]);
    }
}
