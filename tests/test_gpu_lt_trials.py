"""LT runs in the per-trial form (a workgroup per trial, thresholds counted
down in LDS) against the oracle: active bits, per-trial and per-node counts,
whole numbers, so equal.  One case per element width (8 bits: equal in-weights
and at most 126 in-arcs; 16: more in-arcs; 32: unequal or zero weights), at the
edges of its range, and trial counts around a hash block, a 64-trial word and
the wavefront counts."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

FORCED = 16  # Opts.test_flags: the per-trial form whatever the sizes say


@pytest.fixture(scope="module")
def ims():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2404_17059_amd as m
    return m


def graph(n, m, rng, into):
    """m random distinct arcs and `into` arcs into node 1, rows in id order."""
    keys = np.concatenate([rng.integers(0, n * n, size=m), np.arange(into, dtype=np.int64) * n + 1])
    keys = np.unique(keys)
    keys = keys[keys // n != keys % n]
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(keys // n, minlength=n), out=off[1:])
    return off, (keys % n).astype(np.uint32)


def weights(kind, n, idx, rng):
    ind = np.bincount(idx, minlength=n)
    if kind == "equal":
        return 1.0 / ind[idx]  # in-degree 1: a weight of exactly 1
    w = rng.random(idx.size) + 0.01
    if kind == "zeros":
        w[rng.random(idx.size) < 0.3] = 0.0
    s = np.bincount(idx, weights=w, minlength=n)
    w = np.where(s[idx] > 0, w / np.maximum(s[idx], 1e-30), 0.0)
    return w * 0.999999


@pytest.mark.parametrize("kind,n,m,trials,seeds,into", [
    ("equal", 15, 30, 1, 1, 0),
    ("equal", 64, 120, 7, 2, 0),
    ("equal", 65, 300, 64, 3, 0),
    ("equal", 300, 900, 65, 5, 120),       # 8-bit states, in-degrees near their limit
    ("equal", 300, 900, 200, 5, 200),      # 16-bit states
    ("equal", 3000, 12000, 1100, 300, 40),  # more seeds than travel with the launch
    ("equal", 500, 1500, 4100, 4, 0),      # one wavefront per trial
    ("equal", 40000, 90000, 65, 30, 300),  # 16-bit states, 80 KB of LDS
    ("random", 63, 200, 9, 2, 0),
    ("random", 300, 1500, 130, 6, 250),
    ("random", 300, 1500, 321, 6, 40),     # six words: the fewest that the sweeps sum bit-sliced
    ("zeros", 300, 1500, 65, 6, 100),
    ("zeros", 300, 1500, 1025, 6, 100),    # sixteen words and one more
    ("random", 30000, 60000, 65, 40, 0),   # 32-bit states, 124 KB of LDS
    ("equal", 500, 1500, 10, 0, 0),        # no seed
    ("random", 45000, 90000, 65, 40, 0),   # state outside the LDS, at each width
    ("equal", 80000, 160000, 9, 40, 300),
    ("equal", 160000, 320000, 9, 400, 0),  # more joins in one round than the ring keeps
    ("equal", 20000, 400000, 9, 3000, 0),
])
def test_per_trial_runs_match_the_oracle(ims, kind, n, m, trials, seeds, into):
    rng = np.random.default_rng([n, m, trials, into])
    off, idx = graph(n, m, rng, into)
    w = weights(kind, n, idx, rng)
    sd = rng.choice(n, seeds, replace=False).astype(np.uint32)
    G = ims.Graph(n, off, idx, "lt", w)
    ref = oracle.simulate("lt", n, off, idx, oracle.encode("lt", w), sd, trials, 77)
    forced = ims.Opts(test_flags=FORCED)
    for want_bits in (True, False):
        got = ims.simulate(G, np.concatenate([sd, sd[:1]]), trials, 77, want_bits=want_bits, opts=forced)
        assert got["total"] == ref["total"]
        assert (got["trial_counts"].cpu().numpy().view(np.uint32) == ref["trial_counts"]).all()
        assert (got["node_counts"].cpu().numpy().view(np.uint32) == ref["node_counts"]).all()
        if want_bits:
            assert (got["active_bits"].cpu().numpy().view(np.uint64) == ref["active_bits"]).all()
    sweeps = ims.simulate(G, sd, trials, 77, opts=ims.Opts(shape=2))
    assert sweeps["total"] == ref["total"]
    again = ims.simulate(G, sd, trials, 77, opts=forced)
    assert again["total"] == ref["total"]
    G.close()


def test_default_batch_mixes_forms_and_replays(ims):
    """A default batch runs items in per-trial forms beside the task list (a
    subcritical IC item on a large trial count stays there); every output of
    every launch equals the single runs', replays with work in between too."""
    import torch
    rng = np.random.default_rng(5)
    items, singles = [], []
    for i, (n, m, T) in enumerate([(300, 1500, 200), (2000, 9000, 130), (300, 900, 4200), (700, 4000, 65), (45000, 90000, 70), (40, 60, 3)] * 2):
        off, idx = graph(n, m, rng, 150 if i == 3 else 0)
        lt = i % 2 == 0 or i == 4
        p = weights("random" if i in (2, 4) else "equal", n, idx, rng) if lt else np.full(idx.size, 0.01 if i == 7 else 0.3)
        g = ims.Graph(n, off, idx, "lt" if lt else "ic", p)
        sd = rng.choice(n, min(n, 300 if i == 1 else 8), replace=False).astype(np.uint32)
        items.append((g, sd, T, 1000 + i))
        r = ims.simulate(g, sd, T, 1000 + i, opts=ims.Opts(shape=2))
        singles.append([r["trial_counts"].cpu().numpy().view(np.uint32), r["node_counts"].cpu().numpy().view(np.uint32), r["total"]])
    B = ims.Batch(items)

    def check(what):
        for i, (got, want) in enumerate(zip(B.results(), singles)):
            assert got["total"] == want[2], (what, i)
            assert (got["trial_counts"] == want[0]).all(), (what, i)
            assert (got["node_counts"] == want[1]).all(), (what, i)

    for k in range(3):
        B.launch()
        check(f"launch {k}")
        # other work on the device and on the graphs between the replays
        ims.simulate(items[k][0], items[k][1], items[k][2], 3)
        torch.ones(1 << 20, device="cuda").sum().item()
    B.autotune(1)
    for k in range(2):
        B.launch()
        check(f"after autotune {k}")
    B.close()
