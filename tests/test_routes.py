"""The rules that choose a call's form (csrc/routes.hpp), compiled for the CPU:
calls on which the two forms' measured times lie far apart take the faster."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("routes") / "routes_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2404_17059_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "sanitize", "routes_check.cpp")], check=True, capture_output=True, text=True)

    def ask(*call):
        res = subprocess.run([exe], input=" ".join(str(x) for x in call), capture_output=True, text=True, timeout=60)
        assert res.returncode == 0, res.stdout + res.stderr
        return res.stdout.strip()

    return ask


@pytest.mark.parametrize("n,m,max_out,equal,max_in,arcs,left,trials,form", [
    # Erdos-Renyi graphs: few seeds, then a tenth and a third of the nodes (ms, per-trial form / sweeps)
    (300000, 899995, 13, 1, 15, 906, 0, 320, "trials"),         # 0.7 / 5.5
    (300000, 899995, 13, 1, 15, 90000, 0, 320, "sweeps"),       # 8.3 / 3.6
    (300000, 899995, 13, 1, 15, 300000, 0, 320, "sweeps"),      # 11.9 / 2.3
    (60000, 479966, 22, 0, 23, 480, 0, 1000, "trials"),         # 8.3 / 48
    (60000, 479966, 22, 0, 23, 48000, 0, 1000, "sweeps"),       # 20.6 / 5.8
    (130000, 2079853, 36, 1, 36, 885802, 0, 64, "sweeps"),      # in the LDS, 3.3 / 1.3
    (12000, 35992, 12, 1, 12, 11997, 0, 1000, "trials"),        # in the LDS, 0.19 / 0.65
    # preferential attachment: hubs, with the long rows that are left to draw, and as many random nodes
    (130000, 519926, 1115, 1, 1115, 13206, 25000, 1000, "trials"),   # 50 hubs 2.7 / 3.2
    (130000, 519926, 1115, 1, 1115, 188000, 0, 1000, "sweeps"),      # 13,000 hubs 16.5 / 1.0
    (130000, 519926, 1115, 1, 1115, 10400, 25000, 1000, "trials"),   # 2,600 random 2.4 / 17
    (60000, 239932, 762, 1, 762, 149821, 0, 1000, "sweeps"),         # a third of the nodes, in the LDS, 2.0 / 0.5
    # directed power-law graphs: the largest hub where two trials and one share a compute unit, 50 random nodes
    (60000, 471669, 20195, 1, 20, 20195, 0, 1000, "trials"),         # 2.5 / 3.5
    (100000, 789128, 32128, 1, 23, 32128, 0, 1000, "sweeps"),        # 7.8 / 4.5
    (100000, 789128, 32128, 1, 23, 32128, 0, 256, "trials"),         # 2.1 / 3.9
    (100000, 789128, 32128, 1, 23, 236, 0, 1000, "trials"),          # 2.2 / 4.1
])
def test_lt_runs_of_many_seeds_take_the_sweeps(routes, n, m, max_out, equal, max_in, arcs, left, trials, form):
    assert routes("lt", n, m, max_out, equal, max_in, arcs, left, trials) == form


@pytest.mark.parametrize("n,m,max_out,equal,max_in,arcs,left,trials,form", [
    # beyond the 1,024 trials that sweep together both forms' times grow with the trials (ms, per-trial form / sweeps)
    (20000, 200000, 12, 1, 12, 67360, 0, 4096, "trials"),        # a ring, a third of the nodes 1.0 / 3.3
    (20000, 155757, 7601, 1, 20, 27241, 0, 4096, "trials"),      # directed power law, the ten largest hubs 2.1 / 6.6
    (20000, 159949, 16, 1, 21, 74312, 0, 4096, "trials"),        # Erdos-Renyi, a third of the nodes 1.5 / 3.2
    # rows above 64 in-arcs that no seed covers: 10,000 random nodes 16 / 54
    (100000, 799582, 2343, 1, 2343, 79638, 54000, 1000, "trials"),
])
def test_lt_runs_of_many_seeds_and_trials(routes, n, m, max_out, equal, max_in, arcs, left, trials, form):
    assert routes("lt", n, m, max_out, equal, max_in, arcs, left, trials) == form


@pytest.mark.parametrize("n,m,max_out,pbar,growth,arcs,trials,bits,form", [
    # ms: tasks / coins met / coins drawn
    (200000, 5999568, 57, 0.01, 0.3, 2400761, 100, 0, "drawn"),     # a third of the nodes 2.86 / 19.7 / 0.96
    (200000, 1599965, 24, 0.037, 0.295, 532583, 100, 0, "drawn"),   # 1.87 / 4.46 / 0.58
    (100000, 399988, 16, 0.01, 0.04, 8052, 1000, 0, "tasks"),       # 2,000 nodes
    (40000, 319956, 22, 0.05, 0.4, 9, 1000, 0, "met"),              # one node
    (12000, 95962, 21, 0.05, 0.4, 2400, 1000, 1, "met"),            # 240 nodes, bits wanted 0.78 / 0.13 / 0.13
    (200000, 1199730, 3330, 0.05, 1.643, 7, 100, 0, "tasks"),       # one leaf 0.035 / 0.024 / 0.133
    (200000, 1188837, 3000, 0.16783, 0.998, 3, 100, 0, "met"),      # 0.032 / 0.021 / 0.132
    (100000, 599754, 2346, 0.16674, 1.0, 366395, 1000, 0, "drawn"),  # 33,333 hubs 1.8 / 5.8 / 1.9
    (100000, 591739, 24895, 0.49954, 2.925, 173195, 100, 0, "tasks"),  # 100 hubs, two in three arcs live 0.62 / 5.1 / 2.6
    (100000, 591739, 24895, 0.49954, 2.925, 600, 100, 0, "drawn"),  # 100 random nodes
    (10000, 100000, 12, 0.5, 5.0, 1000, 1000, 0, "drawn"),          # a ring, UR 2.2 / - / 0.39
    (100000, 999000, 3000, 0.01, 0.6, 500, 10000, 0, "tasks"),      # beyond 1,500 trials
    (300000, 900000, 20, 0.1, 0.3, 30, 100, 0, "tasks"),            # more nodes than the per-trial forms take
    # small cascades without hubs, tens of seeds, hundreds of trials
    (28460, 227680, 12, 0.0716, 0.573, 728, 624, 0, "met"),         # a ring 0.099 / 0.070
    (51979, 467811, 24, 0.037, 0.33, 540, 364, 0, "met"),           # Erdos-Renyi, TV 0.076 / 0.058
    (95702, 574212, 8, 0.0848, 0.51, 360, 1184, 0, "met"),          # a ring 0.15 / 0.12
    (1900, 15200, 20, 0.05, 0.4, 800, 1400, 0, "tasks"),            # 2 million arcs met
])
def test_ic_runs_choose_by_their_seeds(routes, n, m, max_out, pbar, growth, arcs, trials, bits, form):
    assert routes("ic", n, m, max_out, pbar, growth, arcs, trials, bits) == form


RING = (1.0, 0.22, 0.84)      # growth, spread, fresh of a ring with ten neighbours, WC
LATTICE = (1.0, 0.57, 0.66)   # with four
RANDOM = (1.0, 1.0, 1.0)
POWER = (1.0, 0.93, 0.80)


@pytest.mark.parametrize("n,m,pbar,shape,base,sets,size,arcs,trials,form", [
    # ms: tasks / drawn
    (200000, 2000000, 0.1, RING, 0, 40, 4, 1602, 1000, "tasks"),     # 0.25 / 1.9
    (200000, 800000, 0.25, LATTICE, 0, 40, 30, 4807, 1000, "tasks"),  # 0.30 / 2.4
    (20000, 200000, 0.1, RING, 0, 16, 1, 160, 1000, "tasks"),        # 0.14 / 0.31
    (20000, 200000, 0.1, RING, 0, 16, 30, 4800, 1000, "tasks"),      # 0.43 / 0.48
    (20000, 80000, 0.25, LATTICE, 0, 1000, 1, 3992, 1000, "drawn"),  # 1.8 / 0.30
    (20000, 200000, 0.1, RING, 0, 8, 1000, 80000, 1000, "drawn"),    # a twentieth of the nodes a set
    (20000, 200000, 0.1, RANDOM, 0, 16, 1, 160, 1000, "drawn"),      # the same arcs to random nodes
    (200000, 1969000, 0.1, POWER, 0, 128, 25, 300000, 1000, "drawn"),
    (200000, 1969000, 0.1, POWER, 1, 64, 1, 150000, 10000, "drawn"),
    (60000, 359768, 0.037, (1.14, 0.93, 0.83), 1, 4, 1, 470, 1000, "tasks"),   # four nodes on a base of 20 hubs 0.16 / 0.45
    (100000, 1000000, 0.02, (1.2, 0.93, 0.9), 0, 64, 1, 640, 1000, "tasks"),   # 0.39 / 0.92
    (1000, 10000, 0.037, (0.31, 1.0, 1.0), 0, 1000, 4, 280000, 1000, "tasks"),  # hubs 3.3 / 5.2
])
def test_sets_on_local_graphs_keep_the_tasks(routes, n, m, pbar, shape, base, sets, size, arcs, trials, form):
    assert routes("sets", n, m, m // n * 20, pbar, *shape, base, sets, size, arcs, trials) == form


@pytest.mark.parametrize("n,m,max_out,pbar,growth,spread,fresh,sets,size,arcs,trials,form", [
    # ms: tasks / drawn.  A random regular graph, TV: the draw is shared by the sets
    (5000, 34981, 7, 0.0368, 0.2572, 1.0, 1.0, 64, 1, 448, 10000, "tasks"),       # 0.52 / 0.57
    (5000, 34981, 7, 0.0368, 0.2572, 1.0, 1.0, 5000, 1, 34981, 10000, "drawn"),   # 36 / 1.6
    (20000, 318844, 1780, 0.0370, 1.94, 1.0, 1.0, 1000, 1, 15356, 1000, "drawn"),  # preferential attachment, TV, 77 / 4.0
    # hubs of directed power-law graphs, and sets of four on an Erdos-Renyi graph
    (200000, 1969424, 70707, 0.0370, 0.3633, 1.0, 1.0, 200, 1, 1544502, 100, "drawn"),  # 9.6 / 0.72
    (60000, 585800, 23602, 0.02, 0.1923, 1.0, 1.0, 200, 4, 1931047, 100, "drawn"),      # 3.3 / 0.49
    (5000, 49941, 23, 0.0370, 0.3719, 1.0, 1.0, 1000, 4, 76559, 1000, "drawn"),         # 1.7 / 0.55
    (1000, 8913, 394, 0.0365, 0.3099, 1.0, 1.0, 200, 4, 57037, 1000, "tasks"),          # 0.80 / 1.25
    # rings: much to walk and little to draw, and the other way round
    (5000, 99996, 22, 0.05, 1.0, 0.12, 0.92, 8, 30, 4807, 1000, "drawn"),      # 0.95 / 0.29
    (200000, 3999998, 23, 0.05, 1.0, 0.11, 0.92, 8, 30, 4799, 1000, "tasks"),  # 1.0 / 3.2
    (60000, 599980, 17, 0.1, 1.0, 0.46, 0.86, 200, 30, 60091, 100, "drawn"),   # a quarter rewired, 0.97 / 0.60
    (20000, 80000, 6, 0.25, 1.0, 0.57, 0.66, 200, 1, 797, 1000, "drawn"),      # 0.45 / 0.21
    (60000, 600000, 12, 0.1, 1.0, 0.22, 0.84, 40, 1, 401, 1000, "tasks"),      # 0.19 / 0.61
    # light sets: the live seed arcs in all count
    (60000, 359768, 1500, 0.05, 1.16, 0.93, 0.85, 64, 1, 384, 4000, "tasks"),      # preferential attachment, p 0.05, 0.78 / 1.40
    (60000, 359768, 1500, 0.05, 1.16, 0.93, 0.85, 200, 1, 1200, 4000, "drawn"),    # 2.0 / 1.5
    (20000, 194000, 3000, 0.1, 1.0, 0.9, 0.8, 200, 1, 536, 1000, "drawn"),         # directed power law, WC, 0.83 / 0.50
    (151922, 1032316, 9000, 0.137, 1.0, 0.93, 0.8, 284, 1, 1215, 760, "drawn"),    # 1.35 / 1.07
])
def test_many_sets_share_the_drawn_coins(routes, n, m, max_out, pbar, growth, spread, fresh, sets, size, arcs, trials, form):
    assert routes("sets", n, m, max_out, pbar, growth, spread, fresh, 0, sets, size, arcs, trials) == form


@pytest.mark.parametrize("n,m,max_out,pbar,growth,sets,size,arcs,trials,form", [
    # ms: tasks / drawn
    (20000, 599977, 55, 0.037, 1.11, 16, 30, 21900, 1000, "drawn"),    # Erdos-Renyi, TV, a base of one node 43 / 1.9
    (5000, 149950, 50, 0.0333, 1.0, 16, 30, 14300, 1000, "drawn"),     # WC, a base of 20 random nodes 3.8 / 0.56
    (60000, 359768, 1500, 0.037, 1.14, 4, 1, 470, 1000, "tasks"),      # four nodes on a base of 20 hubs 0.16 / 0.45
])
def test_marginal_sets_of_many_nodes_take_the_drawn_coins(routes, n, m, max_out, pbar, growth, sets, size, arcs, trials, form):
    assert routes("sets", n, m, max_out, pbar, growth, 1.0, 1.0, 1, sets, size, arcs, trials) == form


@pytest.mark.parametrize("n,m,max_out,pbar,growth,arcs,trials,form", [
    # one node, ms: tasks / drawn
    (10000, 79990, 22, 0.125, 1.0, 8, 1000, "drawn"),      # Erdos-Renyi, WC 0.73 / 0.24
    (80000, 639980, 24, 0.125, 1.0, 8, 100, "drawn"),      # 0.92 / 0.37
    (10000, 99945, 800, 0.1, 1.0, 5, 1000, "drawn"),       # preferential attachment, WC 0.53 / 0.23
    (10000, 94500, 4000, 0.037, 0.34, 2, 1000, "tasks"),   # directed power law, TV 0.062 / 0.115
    (80000, 639980, 24, 0.02, 0.16, 8, 100, "tasks"),      # 0.069 / 0.081
    (11173, 44692, 7, 0.037, 0.15, 40, 586, "drawn"),      # ten nodes of a ring, TV 0.23 / 0.16
])
def test_level_counts_from_one_node(routes, n, m, max_out, pbar, growth, arcs, trials, form):
    assert routes("levels", n, m, max_out, pbar, growth, arcs, trials) == form


@pytest.mark.parametrize("n,m,arcs,words,form", [
    # directed power-law graphs, unequal weights, ms: threshold table / bit-sliced sums
    (54860, 534000, 220, 6, "table"),       # 34 random seeds 2.4 / 4.6
    (54860, 534000, 220, 9, "table"),       # 3.7 / 5.8
    (250000, 3885325, 40, 16, "table"),     # ten random seeds 8.7 / 16.2
    (70000, 685129, 541, 16, "sliced"),     # 100 random seeds 8.1 / 5.3
    (54860, 534000, 90000, 6, "sliced"),    # the largest hubs 2.8 / 2.5
    (100000, 591739, 20, 16, "sliced"),     # six arcs a node
    (100000, 591739, 60000, 5, "table"),    # under six words
])
def test_sweeps_over_unequal_weights(routes, n, m, arcs, words, form):
    assert routes("sweeps", n, m, arcs, words) == form


@pytest.mark.parametrize("kind,low,high", [("ring", 0.1, 0.6), ("random", 0.95, 1.05)])
def test_locality_tells_rings_from_random_graphs(routes, kind, low, high):
    n = 3000
    if kind == "ring":
        u = np.repeat(np.arange(n), 10)
        v = (u + np.tile([-5, -4, -3, -2, -1, 1, 2, 3, 4, 5], n)) % n
        off, idx = np.arange(0, 10 * n + 1, 10), v
    else:
        g = synth.erdos_renyi_directed(n, 10.0, seed=4)
        off, idx = g.offsets, g.indices
    thr = np.full(len(idx), 1 << 28)
    spread, fresh = (float(x) for x in routes("graph", n, len(idx), *off.tolist(), *idx.tolist(), *thr.tolist()).split())
    assert low <= spread <= high and (kind == "random") == (fresh > 0.95)
    # arcs that never fire are no arcs, and a graph without any is not local
    assert routes("graph", n, len(idx), *off.tolist(), *idx.tolist(), *[0] * len(idx)).split() == ["1", "1"]
