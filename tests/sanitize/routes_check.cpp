// Prints which form the rules of csrc/routes.hpp choose for the calls that
// tests/test_routes.py describes, one a line on standard input.
#include <iostream>
#include <string>

#include "routes.hpp"

using namespace imsim_plan;

int main()
{
    std::string what;
    while (std::cin >> what) {
        RouteGraph g;
        g.records = true;
        if (what == "lt") {
            uint64_t arcs, left;
            uint32_t trials;
            std::cin >> g.n >> g.m >> g.max_out >> g.lt_uniform >> g.lt_max_in >> arcs >> left >> trials;
            std::cout << (lt_run_pays(g, arcs, left, trials) ? "trials" : "sweeps") << "\n";
        } else if (what == "ic") {
            uint64_t arcs;
            uint32_t trials;
            bool bits;
            std::cin >> g.n >> g.m >> g.max_out >> g.ic_pbar >> g.ic_growth >> arcs >> trials >> bits;
            g.ic_in_m = g.m;
            const IcForm f = ic_run_form(g, arcs, trials, bits);
            std::cout << (f == IcForm::kTasks ? "tasks" : f == IcForm::kMet ? "met" : "drawn") << "\n";
        } else if (what == "sets") {
            uint64_t sets, size, arcs;
            uint32_t trials;
            bool base;
            std::cin >> g.n >> g.m >> g.max_out >> g.ic_pbar >> g.ic_growth >> g.ic_spread >> g.ic_fresh >> base >> sets >> size >> arcs >> trials;
            g.ic_in_m = g.m;
            std::vector<uint32_t> off;
            for (uint64_t i = 0; i <= sets; ++i) off.push_back((uint32_t)(i * size));
            std::cout << (live_sets_pay(g, base, off, arcs, trials) ? "drawn" : "tasks") << "\n";
        } else if (what == "sweeps") {
            uint64_t arcs;
            uint32_t words;
            std::cin >> g.n >> g.m >> arcs >> words;
            std::cout << (lt_sliced_pays(g, arcs, words) ? "sliced" : "table") << "\n";
        } else if (what == "levels") {
            uint64_t arcs;
            uint32_t trials;
            std::cin >> g.n >> g.m >> g.max_out >> g.ic_pbar >> g.ic_growth >> arcs >> trials;
            g.ic_in_m = g.m;
            std::cout << (live_levels_pay(g, arcs, trials) ? "drawn" : "tasks") << "\n";
        } else if (what == "graph") {
            // offsets, targets and thresholds follow: the measures of locality
            std::cin >> g.n >> g.m;
            std::vector<int64_t> off((size_t)g.n + 1);
            std::vector<uint32_t> idx((size_t)g.m), thr((size_t)g.m);
            for (auto& x : off) std::cin >> x;
            for (auto& x : idx) std::cin >> x;
            for (auto& x : thr) std::cin >> x;
            ic_locality(g, off.data(), idx.data(), thr.data());
            std::cout << g.ic_spread << " " << g.ic_fresh << "\n";
        }
    }
    return 0;
}
