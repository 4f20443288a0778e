"""Device memory of the per-trial forms: bounded at the largest graphs and
trial counts they take."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_sizes_stay_within_their_budgets(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "trial_space_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2404_17059_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "sanitize", "trial_space_check.cpp")], check=True, capture_output=True, text=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr


@pytest.mark.gpu
def test_large_lt_run_keeps_a_bounded_workspace():
    """1M nodes at 10,000 trials: 4 GiB of states and bitmaps and 4 GiB of lists at most, and the same counts."""
    import torch

    import oracle
    import paper_2404_17059_amd as ims
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    g = np.random.default_rng(6)
    n, T = 1000000, 10000
    key = np.unique(g.integers(0, n * n, 3 * n))
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=off[1:])
    idx = (key % n).astype(np.uint32)
    w = 1.0 / np.bincount(idx, minlength=n)[idx]
    seeds = g.choice(n, 50, replace=False).astype(np.uint32)
    G = ims.Graph(n, off, idx, "lt", w)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    r = ims.simulate(G, seeds, T, 5, opts=ims.Opts(test_flags=16))
    held = before - torch.cuda.mem_get_info()[0]
    assert held <= (17 << 29), f"{held >> 20} MB"  # 8.5 GiB: both budgets and the outputs
    tc = r["trial_counts"].cpu().numpy().view(np.uint32)
    assert int(tc.astype(np.int64).sum()) == r["total"] == int(r["node_counts"].sum(dtype=torch.int64).item())
    enc = oracle.encode("lt", w)
    for t0, count in ((0, 64), (4992, 16), (9984, 16)):
        ref = oracle.simulate("lt", n, off, idx, enc, seeds, count, 5, t_begin=t0, threads=8, want_bits=False)
        assert (tc[t0:t0 + count] == ref["trial_counts"]).all(), t0
    G.close()
