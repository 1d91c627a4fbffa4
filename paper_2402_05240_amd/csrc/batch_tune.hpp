// batch_tune.hpp -- the search of vlct_batch_tune over tile plans, apart from
// what it times (host code only).
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

namespace vlct {

// Size classes by the x extent (the CT tile's long side): <= 24, <= 48, <= 96,
// larger.  Each class's CT tile (low nibble of the plan bytes), then its march
// segment (high nibble), is changed while the rest of the batch keeps its
// current choice.  time(plan, ms) times one step under a plan; a value other
// than 0 that it returns ends the search and is returned.
//
// The variants differ by a few percent at most and single timings by as much,
// so one that looks at least 1% faster is timed in turn with the current plan
// and replaces it only if its slowest time beats the fastest of the other by
// 1%; the whole plan has to win against the untuned one in the same way, or the
// untuned one is returned.  (64 runs of 16..96 cells: the plan accepted on
// single timings took 3.58 ms a step against 3.48 untuned.)
template <class Time>
int tune_plan(const std::vector<int> &nx, int ct_variants, int march_variants, Time time,
              std::vector<uint8_t> &plan)
{
    const size_t n = nx.size();
    std::vector<int> cls(n);
    for (size_t i = 0; i < n; ++i) cls[i] = nx[i] <= 24 ? 0 : (nx[i] <= 48 ? 1 : (nx[i] <= 96 ? 2 : 3));
    constexpr float kGain = 0.99f;
    // is plan b at least 1% faster than plan a, in kRounds timings of each?  (By
    // chance 6e-4 of equal plans are with timings that vary by 3%.)
    constexpr int kRounds = 5;
    auto beats = [&](const std::vector<uint8_t> &a, const std::vector<uint8_t> &b,
                     bool &yes) -> int {
        float least_a = 0.0f, most_b = 0.0f;
        yes = true;
        for (int r = 0; r < kRounds && yes; ++r) {
            float ta = 0.0f, tb = 0.0f;
            if (int rc = time(a, ta)) return rc;
            if (int rc = time(b, tb)) return rc;
            least_a = r == 0 ? ta : std::min(least_a, ta);
            most_b = std::max(most_b, tb);
            yes = most_b < kGain * least_a;
        }
        return 0;
    };
    const std::vector<uint8_t> untuned(n, 0);
    std::vector<uint8_t> cur = untuned;
    for (int c = 0; c < 4; ++c) {
        if (std::find(cls.begin(), cls.end(), c) == cls.end()) continue;
        for (int field = 0; field < 2; ++field) {
            const int nv = field == 0 ? ct_variants : march_variants;
            for (int v = 0; v < nv; ++v) {
                std::vector<uint8_t> trial = cur;
                for (size_t i = 0; i < n; ++i) {
                    if (cls[i] != c) continue;
                    trial[i] = field == 0 ? (uint8_t)((trial[i] & 0xF0) | v)
                                          : (uint8_t)((trial[i] & 0x0F) | (v << 4));
                }
                if (trial == cur) continue;
                bool yes = false;
                if (int rc = beats(cur, trial, yes)) return rc;
                if (yes) cur = trial;
            }
        }
    }
    if (cur != untuned) {
        bool yes = false;
        if (int rc = beats(untuned, cur, yes)) return rc;
        if (!yes) cur = untuned;
    }
    plan = cur;
    return 0;
}

}  // namespace vlct
