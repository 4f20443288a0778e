// CPU model of a batch's tagged slot state over a sequence of plans, run by
// tests/test_batch_replan.py under the sanitizers.  Slots write (slot, tag)
// into their words of one buffer, as the tasks do, and no task may meet its
// own tag in a word that it has not written since the plan began or that its
// own slot did not write.  With an argument the clears are left out (a planted
// mistake): the model must then find such a word.  Prints "slot_tags ok".
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "plan.hpp"

static uint64_t rng_state = 0x9E3779B97F4A7C15ull;
static uint64_t below(uint64_t k)
{
    rng_state ^= rng_state << 13;
    rng_state ^= rng_state >> 7;
    rng_state ^= rng_state << 17;
    return rng_state % k;
}

struct Word {
    uint64_t tag = 0, slot = ~0ull;
};

int main(int argc, char**)
{
    const bool planted = argc > 1;
    uint64_t met = 0;
    for (int batch = 0; batch < 200; ++batch) {
        imsim_plan::SlotTags tags;
        std::vector<Word> words;
        std::vector<uint64_t> steps;
        for (int plan = 0; plan < 6; ++plan) {
            const uint64_t stride = 1 + below(3) * 7, slots = 1 + below(12);
            // buffers only grow, and a grown buffer starts clear
            if (steps.size() < slots) steps.assign(slots, 0);
            if (words.size() < slots * stride) words.assign(slots * stride, Word{});
            if (tags.replan(stride, slots) && !planted) {
                words.assign(words.size(), Word{});
                steps.assign(steps.size(), 0);
            }
            for (int task = 0; task < 40; ++task) {
                const uint64_t slot = below(slots), tag = steps[slot] + 1;
                std::vector<bool> own(stride, false);
                uint64_t n = below(stride) + 1;
                for (uint64_t k = 0; k < 2 * n; ++k) {
                    const uint64_t v = below(n);
                    Word& w = words[slot * stride + v];
                    if (w.tag == tag && !own[v]) ++met;
                    w = Word{tag, slot};
                    own[v] = true;
                }
                steps[slot] += 1 + below(3);
            }
        }
    }
    if ((met != 0) != planted) {
        std::fprintf(stderr, "%llu words taken for a task's own\n", (unsigned long long)met);
        return 1;
    }
    std::puts("slot_tags ok");
    return 0;
}
