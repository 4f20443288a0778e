// Sizes of a per-trial run's workspace over the whole range of graphs and
// trial counts, run by tests/test_trial_space.py: what is asked for stays
// within the budgets, is used, and covers every trial.  Prints "trial_space ok".
#include <cstdio>
#include <cstdlib>

#include "plan.hpp"

using namespace imsim_plan;

#define CHECK(c)                                                                                               \
    do {                                                                                                       \
        if (!(c)) {                                                                                            \
            std::fprintf(stderr, "check failed: %s (line %d): n %llu T %llu row %llu blocks %llu lanes %llu\n", #c, __LINE__, \
                         (unsigned long long)n, (unsigned long long)T, (unsigned long long)row, (unsigned long long)blocks, \
                         (unsigned long long)lanes);                                                           \
            std::exit(1);                                                                                      \
        }                                                                                                      \
    } while (0)

int main()
{
    const uint64_t nodes[] = {1, 63, 64, 1000, 65535, 65536, 148000, 1u << 18, 500000, 1u << 20};
    const uint64_t trials[] = {1, 63, 64, 65, 1000, 4096, 10000, 1u << 18};
    for (uint64_t n : nodes)
        for (uint64_t T : trials)
            // lazy coins; 8-bit and 32-bit states with bitmaps; the coin row of 2^24 arcs
            for (uint64_t row : {uint64_t(0), n, 4 * n + n / 8, uint64_t(1) << 21})
                for (uint64_t blocks : {uint64_t(1), uint64_t(256), uint64_t(2048), uint64_t(8192)})
                    for (uint64_t lanes = 1; lanes <= 4; ++lanes) {
                        const TrialSpace s = trial_space(n, T, row, blocks, lanes);
                        CHECK(s.trials >= 64 && s.trials % 64 == 0 && s.trials < T + 64);
                        CHECK(lanes * s.trials * row <= kTrialRowBudget || s.trials == 64);
                        CHECK(s.lists >= 1 && s.lists <= blocks && s.lists <= s.trials && s.lists <= T);
                        CHECK(lanes * s.lists * 4 * n <= kTrialListBudget);
                        CHECK(s.lists <= trial_lists(n, lanes));
                        // nothing is given away: a run is cut only where a budget or its size says so
                        CHECK(s.lists == blocks || s.lists == s.trials || s.lists == T || lanes * (s.lists + 1) * 4 * n > kTrialListBudget);
                        CHECK(s.trials >= T || lanes * (s.trials + 64) * (row + 1) > kTrialRowBudget);
                    }
    std::puts("trial_space ok");
    return 0;
}
