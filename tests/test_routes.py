"""The rules that choose a call's form (csrc/routes.hpp), compiled for the CPU:
calls on which the two forms' measured times lie far apart take the faster."""
import os
import shutil
import subprocess

import pytest

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
