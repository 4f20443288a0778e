"""A batch planned again: task timing switched on and off and autotune move
items between the task list and the per-trial forms, and with them the place
of every slot's tagged state.  A CPU model of that state, and on the GPU every
output of every launch against single runs."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_task_meets_another_plans_tags(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "slot_tags_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2404_17059_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "sanitize", "slot_tags_check.cpp")], check=True, capture_output=True, text=True)
    for args in ([], ["planted"]):
        res = subprocess.run([exe, *args], capture_output=True, text=True, timeout=120)
        assert res.returncode == 0, res.stdout + res.stderr


def csr(n, src, dst):
    key = np.unique(src * np.int64(n) + dst)
    key = key[key // n != key % n]
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=off[1:])
    return off, (key % n).astype(np.uint32)


def in_deg_weights(n, idx):
    return 1.0 / np.bincount(idx, minlength=n)[idx]


@pytest.mark.gpu
def test_replanned_batch_equals_single_runs():
    """An LT item that stays on the task list (hub seeds on a directed power-law
    graph of over 200,000 arcs), a larger one in a per-trial form, and many
    quick IC tasks ahead of both, which spread the LT tasks over the slots."""
    import torch

    import paper_2404_17059_amd as ims
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    g = np.random.default_rng(11)

    n = 36000
    w = np.arange(1, n + 1, dtype=np.float64) ** (-1.0 / 1.1)
    d = np.minimum(g.poisson(w * (8 * n / w.sum())), n // 2)
    off, idx = csr(n, np.repeat(np.arange(n), d), g.integers(0, n, int(d.sum())))
    hubs = np.argsort(-np.diff(off), kind="stable")[:50].astype(np.uint32)
    # what keeps it on the list: a hub, no long in-rows, seeds holding much of all arcs, over 200,000 of them
    assert np.diff(off).max() * 64 >= idx.size > 200000 and np.bincount(idx).max() <= 64 and np.diff(off)[hubs].sum() * 16 >= idx.size
    listed = (ims.Graph(n, off, idx, "lt", in_deg_weights(n, idx)), hubs, 400, 21)

    n = 60000
    off, idx = csr(n, g.integers(0, n, 2 * n), g.integers(0, n, 2 * n))
    assert np.diff(off).max() * 64 < idx.size  # no hub: a per-trial form
    aside = (ims.Graph(n, off, idx, "lt", in_deg_weights(n, idx)), g.choice(n, 40, replace=False).astype(np.uint32), 200, 22)

    n = 20000
    off, idx = csr(n, g.integers(0, n, 4 * n), g.integers(0, n, 4 * n))
    quick = (ims.Graph(n, off, idx, "ic", np.full(idx.size, 0.05)), g.choice(n, 5, replace=False).astype(np.uint32), 8192, 23)

    items = [listed, aside, quick]
    want = [ims.simulate(*it, opts=ims.Opts(shape=2)) for it in items]
    want = [(r["trial_counts"].cpu().numpy().view(np.uint32), r["node_counts"].cpu().numpy().view(np.uint32), r["total"]) for r in want]
    B = ims.Batch(items)

    def launch(what):
        B.launch()
        for i, (got, ref) in enumerate(zip(B.results(), want)):
            assert got["total"] == ref[2], (what, i)
            assert (got["trial_counts"] == ref[0]).all(), (what, i)
            assert (got["node_counts"] == ref[1]).all(), (what, i)

    launch("as created")
    for k in range(3):
        B.task_timing(True)
        launch(f"timed {k}")
        codes, _ = B.task_times()
        assert set((codes >> np.uint64(32)).tolist()) == {0, 1, 2}  # timed: every item on the list
        B.task_timing(False)
        launch(f"timed and back {k}")
    for k in range(2):
        B.autotune(1)
        launch(f"autotuned {k}")
        launch(f"autotuned, replayed {k}")
    B.close()
    for it in items:
        it[0].close()
