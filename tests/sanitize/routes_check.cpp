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
        }
    }
    return 0;
}
