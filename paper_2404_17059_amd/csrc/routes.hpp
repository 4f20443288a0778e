// Which form a call runs in: plain C++ (no HIP) over what is known of the graph
// and the call before it starts, so that the rules can be checked on the CPU.
// Every form gives the same results; the lines stand where the measured times
// beside them cross.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <vector>

namespace imsim_plan {

// Largest graph of the IC per-trial forms (their visited bitmap is 32 KB of LDS).
constexpr uint64_t kLiveNodes = 1u << 18;
constexpr uint64_t kTinySeeds = 4;  // larger seed sets of a many-sets call go to a wavefront at once

// What the rules know of a graph.
struct RouteGraph {
    int64_t n = 0, m = 0;
    uint64_t max_out = 0;    // most out-arcs of a node
    bool records = false;    // the graph has the arc records of the per-trial forms
    int64_t ic_in_m = 0;     // IC: in-arcs (arcs whose threshold is not 0)
    double ic_pbar = 0.0;    // IC: mean firing probability of those arcs
    double ic_growth = 0.0;  // IC: live out-arcs of the target of a live arc, on average
    // IC: the two-step targets of a node, as a part of those that as many arcs
    // to random nodes would have (rings 0.1 to 0.6, grids 0.56, random, power-
    // law and preferential-attachment graphs 0.84 to 1), and the part of the
    // two-step live arcs that lead back neither to the node nor to one it has
    // reached in one step
    double ic_spread = 1.0, ic_fresh = 1.0;
    // cascades stay among the seeds' neighbours' neighbours
    bool local() const { return ic_spread < 0.7; }
    bool lt_uniform = false; // LT: equal in-weights
    bool lt_zero = false;    // LT: some arc has weight 0
    uint64_t lt_max_in = 0;  // LT: most in-arc pieces of a node, and
    uint64_t lt_long = 0;    // those of all nodes with more than 64
};

// ic_spread and ic_fresh from at most 256 nodes, spread over the ids, and 32
// arcs a node (under 1 ms whatever the graph).
inline void ic_locality(RouteGraph& g, const int64_t* off, const uint32_t* idx, const uint32_t* thr)
{
    constexpr int64_t kNodes = 256, kArcs = 32;
    const int64_t n = g.n, samples = std::min(n, kNodes);
    std::vector<uint32_t> seen((size_t)n, 0);  // sample that met the node, counted from 1
    std::vector<float> reached((size_t)n, 0.0f);  // probability that the sample's arc to the node is live
    double distinct = 0.0, random = 0.0, fresh = 0.0, all = 0.0;
    auto each = [&](int64_t u, auto use) {
        const int64_t d = off[u + 1] - off[u], k = std::min(d, kArcs);
        for (int64_t i = 0; i < k; ++i) {
            const int64_t e = off[u] + i * d / k;
            if (thr[e] != 0) use(idx[e], (float)((double)thr[e] * 0x1p-32));
        }
    };
    for (int64_t s = 0; s < samples; ++s) {
        const int64_t u = s * n / samples;
        each(u, [&](uint32_t v, float p) { reached[v] = std::max(reached[v], p); });
        int64_t arcs = 0, met = 0;
        each(u, [&](uint32_t v, float p) {
            each((int64_t)v, [&](uint32_t w, float q) {
                ++arcs;
                met += seen[w] != (uint32_t)s + 1 ? 1 : 0;
                seen[w] = (uint32_t)s + 1;
                all += (double)p * q;
                if ((int64_t)w != u) fresh += (double)p * q * (1.0 - reached[w]);
            });
        });
        each(u, [&](uint32_t v, float) { reached[v] = 0.0f; });
        distinct += (double)met;
        random += (double)n * (1.0 - std::exp(-(double)arcs / (double)n));
    }
    g.ic_spread = random > 0.0 ? distinct / random : 1.0;
    g.ic_fresh = all > 0.0 ? fresh / all : 1.0;
}

// Whether a one-set run takes the drawn-coins form.  It draws all m * T coins
// (`draw`, us) where the other forms draw those of the arcs they meet, so it
// pays unless the cascades stay in a small part of the graph; growth (live
// out-arcs of the target of a live arc) tells how far they go.  Measured on
// Erdos-Renyi, preferential-attachment and small-world graphs of 500 to
// 100,000 nodes, 64 to 10,000 trials, probabilities 0.01 to 0.1, TV, UR, WC:
// - growth below 0.7: the other forms end sooner, but for level counts, which
//   cost them 0.2 ms.
// - up to 1.3: 1.1 to 3x faster up to a draw of 110 us (20,000-node ring, WC,
//   300 trials 0.114 against 0.178 ms; 1,000 trials, draw 167 us, 0.24
//   against 0.18).  With 16 arcs a node and more the other forms meet that
//   many more: 1.7 to 3x faster up to the largest draw tried, 800 us (44 arcs,
//   4,000 nodes, WC, 1,000 trials 0.33 against 0.70; 24 arcs, 12,000 nodes,
//   3,000 trials 1.0 against 2.1), but not below growth 0.85.
//   Level counts: 2 to 12x at every size tried.
// - up to 2: 2 to 4x faster up to a draw of 400 us, slower from about 650;
//   from 16 arcs a node 7 to 10x faster at 600 us.
// - above: 1.5 to 13x faster at every size tried, but for skewed graphs with
//   many live arcs per node, or hubs, whose pull steps end early: there only
//   with fewer than 20,000 nodes and 4,000 trials, and up to 90 million live
//   arcs (16 arcs, 12,000 nodes, UR, 1,000 trials 0.99 against 1.08 ms, 3,000
//   trials 2.4 against 1.6), 50 million on directed graphs with hubs (3,000-node preferential
//   attachment, UR, 4,000 trials 1.24 against 0.77 ms; 300 trials 0.24
//   against 0.49).  From eight live arcs a node every graph but a ring is
//   covered in three or four levels, whose pull steps meet few arcs of a node:
//   the walk over all live arcs pays up to 40 million of them, 100,000 a
//   trial and 2,000 trials (44 arcs, 1,000 nodes, UR, 1,000 trials 0.26 against 0.39 ms; 4,000
//   nodes 0.97 against 0.52; 12,000 nodes, 128 trials 1.1 against 0.63).
inline bool live_single_pays(const RouteGraph& g, uint32_t n_trials, bool levels)
{
    const double n = (double)g.n, growth = g.ic_growth;
    const double draw = (double)g.m * (double)((n_trials + 7) / 8) / 150e3;
    if ((uint64_t)g.n > kLiveNodes || g.n == 0 || !g.records) return false;
    if (growth < 0.7) return levels && draw <= 80.0;
    const bool dense = (double)g.m >= 16.0 * n;
    if (growth < 1.3) return draw <= (levels ? 2000.0 : !dense || growth < 0.85 ? 110.0 : 800.0);
    if (levels) return true;
    if (growth < 2.0) return draw <= (dense ? 800.0 : 400.0);
    const double live_degree = g.ic_pbar * (double)g.ic_in_m / n;
    if (live_degree >= 8.0) return n_trials <= 2000 && live_degree * n <= 100e3 && live_degree * n * n_trials <= 40e6;
    const bool skewed = growth >= 1.5 * live_degree, hubs = (double)g.max_out * n >= 20.0 * (double)g.m;
    if (live_degree >= 3.0 && (skewed || hubs))
        return n < 20000.0 && n_trials < 4000 && live_degree * n * n_trials <= (skewed ? 90e6 : 50e6);
    return true;
}

// Whether a run with level counts does: not where most trials end at once and
// the others soon (10,000-node directed power law, TV, one node, 1,000 trials
// 0.062 against 0.115 ms; near growth 1 some go on: 10,000-node Erdos-Renyi, WC,
// one node, 1,000 trials 0.73 against 0.24, 80,000 nodes, 100 trials 0.92 against
// 0.37; ten nodes of an 11,000-node ring, TV, 586 trials 0.23 against 0.16).
inline bool live_levels_pay(const RouteGraph& g, uint64_t arcs, uint32_t n_trials)
{
    if (!live_single_pays(g, n_trials, true)) return false;
    const double m = (double)g.m;
    const bool few = (double)arcs * g.ic_pbar < 0.5 && m < 16.0 * (double)g.n && g.ic_growth < 0.7;
    return !few || m * (double)((n_trials + 7) / 8) / 150e3 <= 15.0;
}

// Whether an IC item of a batch does: the tasks share the chip there, so the
// lines lie lower than for a run alone (batches of 8 items, ms, tasks / this:
// 60,000 to 300,000 arcs, WC, 2,000 trials 2.7 / 2.9, at draws up to 40 us 0.94
// / 0.37; 44 arcs a node, WC, draws of 300 us and more 4.4 / 6.0, up to 150 us
// 1.5 / 0.9; 44 arcs a node, UR 0.59 / 0.80; 40 arcs, Erdos-Renyi, UR, 200
// trials 1.05 / 0.42, 2,000 trials 2.1 / 2.3; hubs and 2.5 live
// arcs a node, 8,000 to 30,000 nodes, 100 hubs, 200 trials 2.6 / 3.3, 1,000 to
// 3,000 nodes 0.28 / 0.34, one node 0.77 / 0.34; under one live seed arc, 2,000
// trials 0.35 / 0.47; rings, 8,000 to 30,000 nodes, one node 0.15 / 0.28, 100
// 0.33 / 0.47, a tenth of 1,000 to 3,000 0.36 / 0.17).
inline bool live_item_pays(const RouteGraph& g, uint64_t arcs, uint32_t n_trials)
{
    if (!live_single_pays(g, n_trials, false)) return false;
    const double n = (double)g.n, m = (double)g.m, draw = m * (double)((n_trials + 7) / 8) / 150e3;
    const double live = (double)arcs * g.ic_pbar, live_degree = g.ic_pbar * (double)g.ic_in_m / n;
    if (g.ic_growth < 1.3 && g.local() && live < n / 50.0) return false;
    if (g.ic_growth < 2.0 && live < 0.8 && m < 16.0 * n && n_trials > 1000 && draw > 10.0) return false;
    if (g.ic_growth < 1.3) return draw <= (m >= 16.0 * n ? 150.0 : 45.0);
    if (live_degree >= 2.5 && (g.ic_growth >= 1.5 * live_degree || (double)g.max_out * n >= 20.0 * m)) return n < 5000.0 && live < 200.0;
    return live_degree < 8.0 || (g.ic_growth < 1.5 * live_degree && n_trials <= 500 && live_degree * n <= 60e3);
}

// The form of a one-set IC run.  `arcs`: out-arcs of the seeds; `live` of them
// live in a trial, on average.
// - kDrawn: all coins drawn densely, then a workgroup per trial.
// - kMet: a workgroup per trial draws an arc's coin when it meets the arc, a
//   whole hash block of which it uses an eighth; up to 1,500 trials (the tasks
//   of 4 to 16 trials share the blocks) and hubs of 4,000 out-arcs (one
//   workgroup walks them).
// - kTasks: word-local tasks or grid-wide levels.
// Growth below 0.7 (cascades stay small; ms, tasks / met / drawn):
// - a hundred live seed arcs, and a part of all arcs that grows with the
//   trials (0.5% at 100, 5% at 1,000): drawn (200,000-node Erdos-Renyi, 30
//   arcs, p 0.01, 66,666 seeds, 100 trials 2.9 / 19.7 / 0.96; 100,000 nodes, 4
//   arcs, p 0.01, 2,000 seeds with 5%, 1,000 trials 0.25 / 0.34 / 0.41)
// - up to 200,000 arcs met over all trials, or 300 trials on graphs of up to
//   12 arcs a node: met, half to all of the tasks' time; beyond, 0.4 to 3 times;
//   without hubs 100 arcs a node, up to 2 million, and 750 trials (medians up to
//   1.2 million arcs: 0.75 to 0.86 of the tasks' time at 100 to 750 trials, beyond
//   0.9 on 10,000 nodes and more, 1.2 on 1,000; 28,000-node ring, p 0.07, 91 seeds,
//   624 trials 0.099 / 0.070; 96,000 nodes, 60 seeds, 1,184 trials 0.15 / 0.12)
// Above:
// - under two live seed arcs, a mean below 1.1 a node, and a draw of over 10
//   us: most trials end at once (200,000-node preferential attachment, p 0.05,
//   one node, 100 trials 0.035 / 0.024 / 0.133)
// - rings and other local graphs below growth 1.3, live seed arcs fewer than
//   0.3% of the nodes: likewise (40,000-node ring, WC, 100 nodes, 1,000 trials
//   0.19 / 0.12 / 0.40; 12,000 nodes, 10 nodes, 5,000 trials 0.14 / 0.22 / 0.59)
// - where the draw does not pay, met up to 300 live seed arcs below growth 1.3
//   and 16 arcs a node (100,000-node Erdos-Renyi, WC, 1,000 trials 2.3 / 1.3;
//   60 arcs, 12,000 nodes 2.0 / 2.6), drawn above (100,000-node preferential
//   attachment, WC, 33,333 hubs, 1,000 trials 1.8 / 5.8 / 1.9)
// - hubs and 2.5 live arcs a node, 13,000 live seed arcs: two or three pull
//   steps end it (100,000-node directed power law, UR, 100 hubs, 100 trials
//   0.62 / 5.1 / 2.6)
// With active bits (`bits`) the tasks run whole words and take 2 to 6 times as
// long, so the arcs met do not count there.
// (8,064 runs, 1 to a third of the nodes as seeds: slower than the tasks by
// more than 15% in 90, at most 2.0 times; 667, at most 6.9 times, by growth
// and trial count alone.  With bits 15 of 4,320, at most 1.8 times; 66, at most
// 6.6 times.)
enum class IcForm { kTasks, kDrawn, kMet };
inline IcForm ic_run_form(const RouteGraph& g, uint64_t arcs, uint32_t n_trials, bool bits)
{
    if (g.n == 0 || (uint64_t)g.n > kLiveNodes || !g.records) return IcForm::kTasks;
    const double n = (double)g.n, m = (double)g.m, growth = g.ic_growth, trials = (double)n_trials;
    const double live = (double)arcs * g.ic_pbar, live_degree = g.ic_pbar * (double)g.ic_in_m / n;
    const double draw = m * (double)((n_trials + 7) / 8) / 150e3;
    const double met = trials * std::min(m, (double)arcs / (1.0 - std::min(growth, 0.9)));  // arcs met over all trials
    const bool dense = m >= 16.0 * n, meets = n_trials <= 1500 && g.max_out <= 4000;
    if (growth < 0.7) {
        if (n_trials <= 1500 && live >= 100.0 && (double)arcs >= 5e-5 * m * trials) return IcForm::kDrawn;
        const bool flat = (double)g.max_out * n <= 8.0 * m;
        const double most = flat ? std::max(2e5, std::min(100.0 * n, 2e6)) : 2e5;
        const bool small = n_trials <= (flat ? 750u : 300u) && m <= 12.0 * n && live < 100.0;
        return meets && (bits || met <= most || small) ? IcForm::kMet : IcForm::kTasks;
    }
    if (growth < 2.0 && live < 2.0 && live_degree < 1.1 && !dense && draw > 10.0)
        return growth < 1.3 && meets && (bits || met <= 2e5) ? IcForm::kMet : IcForm::kTasks;
    if (growth < 1.3 && g.local() && live < 0.003 * n) return meets ? IcForm::kMet : IcForm::kTasks;
    if (growth >= 2.0 && live_degree >= 2.5 && (double)g.max_out * n >= 20.0 * m && live >= 13000.0) return IcForm::kTasks;
    if (live_single_pays(g, n_trials, false)) return IcForm::kDrawn;
    if (growth >= 1.3 || dense) return IcForm::kTasks;
    return live >= 300.0 ? IcForm::kDrawn : meets ? IcForm::kMet : IcForm::kTasks;
}

// Per-trial LT form: element width of a graph's states, and whether a trial's
// fit the LDS beside the kernel's own arrays.
constexpr uint64_t kLtTrialLds = 160 * 1024 - 12 * 1024;
inline uint32_t lt_trial_bits(const RouteGraph& g)
{
    return !g.lt_uniform || g.lt_zero || g.lt_max_in >= 32767 ? 32 : g.lt_max_in >= 127 ? 16 : 8;
}
inline bool lt_trial_lds(const RouteGraph& g)
{
    const uint64_t n = (uint64_t)g.n, bits = lt_trial_bits(g);
    return n * bits / 8 + (bits == 32 ? n / 8 : 0) + 64 <= kLtTrialLds;
}

// Whether an item of a batch takes it, and a run of few seeds.  It touches every arc once per trial, in as many
// rounds of one workgroup as the cascade has steps; the grid-wide sweeps read
// everything pending at every step but share it between 64 trials.  Measured
// (1,000 trials, ms, this against the sweeps; Erdos-Renyi, preferential-
// attachment and directed power-law graphs of 1,000 to 500,000 nodes, 64 to
// 4,000 trials): 20,000-node Erdos-Renyi 1.6 / 13.7, preferential attachment
// 0.6 / 53, power law 0.75 / 1.8; state outside the LDS: 100,000-node
// Erdos-Renyi with random weights 12.7 / 123, 200,000-node preferential
// attachment 1.4 / 127.  The sweeps win where a hub holding a notable part of
// all arcs makes the cascade dense within few steps (and no node has more
// in-arcs than a sweep stages): with hub seeds above about 200,000 arcs
// (36,000 nodes 2.2 / 1.55), 90,000 with 32-bit states at 1,000 trials (87,000
// arcs 0.90 / 0.90, 175,000 2.3 / 1.5) and more at fewer trials (100 trials:
// 264,000 arcs 0.87 / 1.42), any number with the state outside the LDS (45,000
// nodes 14.5 / 2.1); with other seeds above about a million (140,000 nodes,
// 15 arcs each: 7.6 / 4.4; where few trials leave the chip idle, half of
// that: 800,000 arcs, 128 trials 2.0 / 1.7, 256 trials 2.0 / 1.9, 320 trials
// 2.0 / 2.0), 300,000 outside the LDS (222,000 arcs 2.3 / 2.9,
// 346,000 3.7 / 3.0).
inline bool lt_trials_pay(const RouteGraph& g, uint64_t arcs, uint32_t n_trials)
{
    if (!g.records) return false;
    if (g.max_out * 64 < (uint64_t)g.m || g.lt_max_in > 64) return true;
    const bool dense = arcs * 16 >= (uint64_t)g.m;
    if (!lt_trial_lds(g)) return !dense && g.m <= 300000;
    if (!dense) return g.m <= (n_trials < 320 ? 500000u : 1060000u);
    return lt_trial_bits(g) == 32 ? (double)g.m * std::min(1000.0, (double)n_trials) <= 90e6 : g.m <= 200000;
}

// Whether a one-set run does.  The more out-arcs the seeds have (`arcs`), the
// fewer sweeps a cascade takes, while every trial still pushes along all it
// reaches, so the line is a number of seed arcs over all trials: 1.1e8 with the
// states in the LDS (scaled by the square root of a state's size, as larger
// ones leave fewer trials a compute unit), 1.4e7 outside it; below 512 and 256
// trials a workgroup's chain decides, not their number, and beyond the 1,024
// trials that sweep together both forms' times grow with it.  Directed graphs with
// a hub holding a notable part of all arcs reach far from any seed, and their
// sweeps are few: 5e7 there, 1.5e7 where a compute unit holds one trial and they
// take turns, and up to 1.1 million arcs (outside the LDS 300,000, and no
// seeds with a sixteenth of the arcs).  The sweeps draw the hashes of rows
// above 64 in-arcs anew each time, so those that no seed covers (`long_left`)
// move the line up.  ms, this against the sweeps:
// - 300,000-node Erdos-Renyi, 3 arcs, 320 trials: 300 seeds 0.7 / 5.5, 6,000
//   3.8 / 6.3, 30,000 8.3 / 3.6, 100,000 11.9 / 2.3; 60,000 nodes, 8 arcs,
//   random weights, 1,000 trials: 300 seeds 16.6 / 41, 1,200 20.4 / 21.6,
//   6,000 20.6 / 5.8
// - 130,000-node preferential attachment, 1,000 trials: the 50 largest hubs
//   2.7 / 3.2, 300 5.1 / 1.6; 13,000 random nodes 8.0 / 16
// - in the LDS, 60,000-node preferential attachment, 1,000 trials: 1,200 hubs
//   1.1 / 1.2, 20,000 2.0 / 0.5
// - directed power-law graphs, 8 arcs, 1,000 trials: 60,000 nodes, the largest
//   hub 2.5 / 3.5, ten 2.6 / 2.7; 100,000 nodes (one trial a compute unit), 50
//   random nodes 2.2 / 4.1, 2,000 6.1 / 4.5, the largest hub 7.8 / 4.5, at
//   256 trials 2.1 / 3.9
// (5,100 runs: slower than the sweeps by more than 15% in 47, at most 2.6
// times; 371, at most 30 times, by the rule above.)
inline bool lt_run_pays(const RouteGraph& g, uint64_t arcs, uint64_t long_left, uint32_t n_trials)
{
    if (!g.records) return false;
    const bool lds = lt_trial_lds(g), hub = g.max_out * 64 >= (uint64_t)g.m && g.lt_max_in <= 64;
    if (hub && (lds ? g.m > 1100000 : g.m > 300000 || arcs * 16 >= (uint64_t)g.m)) return false;
    const double state = (double)g.n * lt_trial_bits(g) / 8;
    const double pushed = (double)arcs * std::min(std::max<double>(n_trials, lds ? 512 : 256), 1024.0) * (lds ? std::sqrt(state / 65536.0) : 1.0);
    const double most = !lds ? 1.4e7 : !hub ? 1.1e8 : state > 70e3 && n_trials > 256 ? 1.5e7 : 5e7;
    const double left = (double)long_left / (double)std::max<int64_t>(g.m, 1);
    return pushed <= most * (1.0 + 35.0 * left + 700.0 * left * left);
}

// Whether sweeps over unequal weights take the bit-sliced sums.  Those give a
// lane to each word of a row, so below six words most lanes idle (100,000-node
// power-law graph, random weights, ms, threshold table / sliced: 1.2 / 2.1 at 2
// words, 3.0 / 3.4 at 5, 3.6 / 3.5 at 7, 7.3 / 3.1 at 16), and they sum every
// in-arc of a pending node, where the table's sweep looks only at the words in
// which one is active: cascades that stay small on graphs of eight arcs a node
// and more take it up to 0.85% of the arcs at the seeds, over the words (10 arcs,
// 55,000 nodes, 34 random seeds, 6 words 2.4 / 4.6, 9 words 3.7 / 5.8, 16 words
// 6.4 / 6.7; 250,000 nodes, 16 arcs, 10 seeds, 16 words 8.7 / 16.2; 70,000 nodes, 100
// seeds, 6 words 3.3 / 3.8, 11 words 5.4 / 5.0, 16 words 8.1 / 5.3; 60,000 nodes,
// 16 arcs, 1,000 seeds, 8 words 8.0 / 7.0).
inline bool lt_sliced_pays(const RouteGraph& g, uint64_t arcs, uint32_t words)
{
    return words >= 6 && (g.m < 8 * g.n || (double)arcs * words >= 0.0085 * (double)g.m);
}

// Whether a many-sets call takes the drawn-coins form.  It draws every arc's
// coin once, m * T / 8 hash blocks at about 150 a nanosecond; the tasks draw
// the coins of the arcs their cascades meet, set by set, at least those of
// the seeds' out-arcs in every trial, and where the target of a live arc has
// about one live out-arc or more a cascade goes on to meet many times that (it
// is heavy tailed: on the 200k-node weighted-cascade graph at 1,000 trials the forms
// break even at about 100 random single nodes, m / 2,000 seed out-arcs; one
// hub already takes 1.7 against 4.4 ms, a set of 25 nodes 2.4 against 21).
// Below that the factor is the geometric sum of that growth times what a
// dense draw gains per block.  From eight sets on draws of up to 20 us pay
// whatever the sets' arcs, where none of the exceptions below applies.
// Sets on top of a base meet an unknown part of their arcs.  The measured
// times there (graphs of 5,000 to 200,000 nodes with weighted-cascade
// probabilities, 100 to 10,000 trials, 1 to 128 hubs on bases of 3 to 20) are
// about 250 us + the draw + 2.5 ns per (trial, set) for the drawn-coins form,
// and for the tasks at least 150 us + 15 ns per node (one task's chain of
// steps) and 50 times the draw of the sets' own out-arcs; growth above 2
// leaves little outside the base (0.07 ms for the tasks), below 0.8 little at
// all.  A few nodes with under five live arcs each often lie in the base already,
// so up to eight the estimates have to lie a factor of two apart (60,000-node
// preferential attachment, TV, a base of 20 hubs, four nodes 0.16 / 0.45 ms);
// more of them reach past it (20,000-node Erdos-Renyi, 30 arcs, TV, a base of
// one node, 16 sets of 30 43 / 1.9).  (14,930 calls: 30 slower than the tasks by
// more than 15%, but for one at most 3.5 times.)
inline bool live_sets_pay(const RouteGraph& g, bool base, const std::vector<uint32_t>& off, uint64_t arcs, uint32_t n_trials)
{
    if ((uint64_t)g.n > kLiveNodes || g.n == 0 || !g.records || off.size() > (1u << 24)) return false;
    const double blocks = (double)((n_trials + 7) / 8);
    const double draw = (double)g.m * blocks / 150e3;  // us
    if (base) {
        const double live = 250.0 + draw + 0.0025 * (double)n_trials * (double)(off.size() - 1);
        // the chain only where the sets are hubs (40,000-node preferential
        // attachment, 8 random nodes, 1,000 trials: tasks 0.40, drawn 0.64 ms)
        const bool hubs = (double)arcs * (double)g.n >= 4.0 * (double)g.m * (double)off.back();
        const double tasks = std::max(hubs ? 150.0 + 0.015 * (double)g.n : 0.0, 50.0 * (double)arcs * blocks / 150e3);
        const double apart = off.back() <= 8 && (double)arcs * g.ic_pbar < 5.0 * (double)off.back() ? 2.0 : 1.0;
        return g.ic_growth >= 0.8 && g.ic_growth <= 2.0 && apart * live < tasks;
    }
    // Where the tasks stay faster (whole calls in ms, tasks / drawn; random sets
    // on graphs of 1,000 to 40,000 nodes, 5 to 44 arcs a node):
    // - small cascades of many seeds, which a lane does not follow alone, and
    //   of few sets (growth 0.16, 1,000 trials, 64 sets of 30 0.25 / 0.87, 16
    //   single nodes 0.100 / 0.107; 256 single nodes 0.36 / 0.17); up to growth
    //   0.9 with fewer than 16 arcs a node and many trials (64 sets of 30,
    //   1,000 trials 0.69 / 0.92, 100 trials 0.44 / 0.21);
    // - under four sets near growth 1 (0.14 / 0.16);
    // - cascades that cover the graph in three levels, whose pull steps end
    //   early, but for few walks (growth 39, 16 sets, 1,000 trials 0.85 / 1.68,
    //   100 trials 0.81 / 0.44);
    // - below growth 0.6, hubs of small graphs: eight live seed arcs a set, up to
    //   5,000 nodes (directed power law, TV, 1,000 trials, 200 hubs in sets of 4:
    //   1,000 nodes 0.80 / 1.25, 5,000 nodes 2.2 / 2.5, 20,000 nodes 5.2 / 3.2);
    // - sets that mostly light nothing, and a long draw: below growth 1.25
    //   with under one live seed arc in all per 1,700 nodes (100,000-node
    //   preferential attachment, p 0.02, 1,000 trials, 64 nodes 0.39 / 0.92; 60,000
    //   nodes, p 0.05, 4,000 trials, 64 nodes 0.78 / 1.40, 200 nodes 2.0 / 1.5);
    // - rings and other local graphs with less than 1.1 new live arcs per live
    //   arc: a cascade's steps meet the same nodes again and a task's few steps
    //   end it, unless there is much to walk per set and little to draw
    //   (degree 4, WC, 1,000 trials, 40 sets of 30: 200,000 nodes 0.30 / 2.4, 1,000
    //   nodes 0.28 / 0.56; degree 20, 8 sets of 30, 5,000 nodes 0.95 / 0.29,
    //   200,000 nodes 1.6 / 4.6), or many single nodes (degree 4, 20,000 nodes, WC, 8
    //   nodes 0.11 / 0.17, 1,000 nodes 1.8 / 0.30).  Small calls (sets times
    //   trials up to 4,000, draws up to 45 us) and sets of 64 live seed arcs and
    //   more are as on other graphs.
    //   Of 21,923 calls 672 were slower than the tasks by more than 15%, at most
    //   8 times, without the last three lines; 126, at most 2.1 times, with them,
    //   and 80 calls stay with tasks that are slower, at most 2.8 times.
    const uint64_t sets = off.size() - 1;
    uint64_t large = 0;
    for (uint64_t i = 0; i < sets; ++i) large += off[i + 1] - off[i] > kTinySeeds ? 1u : 0u;
    const bool dense = (double)g.m >= 16.0 * (double)g.n;
    if (g.ic_growth < 0.6 && (large || sets < 64)) return false;
    if (g.ic_growth < 0.9 && !dense && large * n_trials > 8000) return false;
    if (sets < 4 && g.ic_growth < (dense ? 0.85 : 1.4)) return false;
    if (g.ic_growth >= 8.0 && sets * n_trials > 8000) return false;
    const double live = (double)arcs * g.ic_pbar / (double)sets, renewed = g.ic_growth * g.ic_fresh;
    const double walked = (double)arcs / (double)sets / (1.0 - std::min(renewed, 0.97));  // by a set's cascade
    if (g.ic_growth < 0.6 && g.n <= 5000 && live > 8.0) return false;
    if (g.ic_growth < 1.25 && live < 0.6 && draw >= 100.0 && (double)arcs * g.ic_pbar * 1700.0 < (double)g.n) return false;
    if (g.local() && renewed < 1.1 && live < 64.0 && !(sets * n_trials <= 4000 && draw <= 45.0) &&
        (live > 2.0 ? walked < 1500.0 || draw > walked / 12.0 : (double)arcs * 200.0 < (double)g.m))
        return false;
    const double reach = g.ic_growth >= 0.8 ? 2000.0 : 8.0 / (1.0 - g.ic_growth);
    return (double)arcs * reach >= (double)g.m || (draw <= 20.0 && off.size() > 8);
}

}  // namespace imsim_plan
