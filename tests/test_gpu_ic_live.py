"""IC many-sets calls in the drawn-coins form (every arc's coins drawn once
into bit rows, the cascades walked over them) against the oracle: totals and
per-node counts, whole numbers, so equal.  Sizes sit at the edges of the form:
trial counts around a hash block, a 64-trial word and the coin rows' tail;
node and arc counts around a bitmap word, a 64-arc chunk and a 512-arc line;
sets on both sides of the sizes a lane follows alone, cascades that outgrow
its list, nodes with more arcs than one lane takes, enough large sets for the
packed live graphs."""
import numpy as np
import pytest

import oracle

FORCED = 16  # Opts.test_flags: the drawn-coins form whatever the sizes say
LAZY = 32    # the per-trial form that draws coins as it meets arcs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ims():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2404_17059_amd as m
    return m


def graph(n, m, rng, hub=0):
    """m distinct arcs, `hub` of them (or as many as fit) out of node 0."""
    keys = rng.choice(n * n, size=m, replace=False)
    if hub:
        keys = np.concatenate([np.arange(min(hub, n)), keys[keys >= n]])[:max(m, 1)]
    keys = np.sort(keys)
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(keys // n, minlength=n), out=off[1:])
    return off, (keys % n).astype(np.uint32)


CASES = [
    # n, m, trials, p, sets, most nodes per set, hub arcs
    (31, 40, 1, 0.3, 12, 3, 0),
    (32, 64, 7, 0.3, 12, 3, 0),
    (33, 65, 8, 0.3, 12, 6, 0),
    (63, 511, 9, 0.2, 40, 2, 60),
    (64, 512, 63, 0.2, 10, 1, 64),
    (65, 513, 64, "mixed", 10, 6, 65),
    (700, 3000, 65, 0.3, 300, 1, 600),
    (700, 3000, 130, "mixed", 40, 30, 600),  # packed live graphs, live rows above a lane's share
    (3000, 9000, 127, "one", 40, 8, 2500),
    (3000, 9000, 70, 0.0, 12, 8, 0),
    (400, 40000, 9, "one", 12, 8, 0),       # every node reached with arcs left to walk
    (400, 40000, 9, "one", 100, 8, 0),      # the same, packed
]


@pytest.mark.parametrize("n,m,trials,p,count,most,hub", CASES)
@pytest.mark.parametrize("based", [False, True])
def test_drawn_coin_sets_match_the_oracle(ims, n, m, trials, p, count, most, hub, based):
    rng = np.random.default_rng([n, m, trials])
    off, idx = graph(n, m, rng, hub)
    k = idx.size
    prob = {"mixed": rng.choice([0.0, 0.02, 0.5, 1.0], k), "one": np.ones(k)}.get(p, None)
    prob = np.full(k, float(p)) if prob is None else prob
    G = ims.Graph(n, off, idx, "ic", prob)
    enc = oracle.encode("ic", prob)
    sets = [rng.choice(n, size=rng.integers(1, min(most, n) + 1), replace=False).astype(np.uint32) for _ in range(count)]
    sets[1] = np.zeros(0, dtype=np.uint32)
    sets[2] = np.array([0, 0, n - 1], dtype=np.uint32)  # the hub, and a repeat
    rs = 4242
    state = np.zeros((-(-trials // 64), n), dtype=np.uint64)
    base = np.array([1, n // 2], dtype=np.uint32)
    if based:
        ref = oracle.simulate("ic", n, off, idx, enc, base, trials, rs)
        bits = ims.simulate(G, base, trials, rs, want_bits=True)["active_bits"]
        state = ref["active_bits"].copy()
        got = ims.simulate_sets_from(G, bits, sets, trials, rs, want_node_counts=True, opts=ims.Opts(test_flags=FORCED))
        totals = got["new_totals"]
    else:
        got = ims.simulate_sets(G, sets, trials, rs, want_node_counts=True, opts=ims.Opts(test_flags=FORCED))
        totals = got["totals"]
    for i, st in enumerate(sets):
        full = oracle.simulate("ic", n, off, idx, enc, np.unique(np.concatenate([st, base])) if based else np.unique(st), trials, rs)
        # new activations only: what the base alone leaves inactive
        new = np.zeros(n, dtype=np.int64)
        diff = full["active_bits"] & ~state
        for w in range(diff.shape[0]):
            new += np.array([bin(int(x)).count("1") for x in diff[w]], dtype=np.int64)
        assert (got["node_counts"][i].astype(np.int64) == new).all(), f"set {i}"
        assert int(totals[i]) == int(new.sum()), f"set {i}"
    # shape 1 asks for the tasks that draw their own coins: same totals, same steps
    a = G.last_status()
    again = (ims.simulate_sets_from(G, bits, sets, trials, rs, opts=ims.Opts(shape=1)) if based
             else ims.simulate_sets(G, sets, trials, rs, opts=ims.Opts(shape=1)))
    assert (again["new_totals" if based else "totals"] == totals).all()
    assert a == G.last_status()
    G.close()


@pytest.mark.parametrize("n,m,trials,p,seeds,hub", [
    (31, 40, 1, 0.3, 2, 0),
    (32, 64, 7, 0.3, 3, 0),
    (65, 513, 64, "mixed", 4, 65),
    (700, 3000, 65, 0.3, 1, 600),
    (700, 3000, 300, "one", 300, 600),      # more seeds than travel with the launch; eight wavefronts per cascade
    (700, 3000, 513, 0.1, 0, 600),          # no seed; four wavefronts
    (700, 3000, 1100, "mixed", 256, 600),   # two blocks of words in the node counts
    (3000, 30000, 70, 0.3, 10, 2500),
    (20000, 60000, 65, 0.5, 5, 9000),       # sixteen wavefronts
    (129, 700, 4096, 0.2, 3, 100),          # one wavefront
    (400, 40000, 65, 0.3, 3, 0),            # every node reached with arcs left to walk
    (400, 40000, 4096, 0.3, 400, 0),        # the seeds are all nodes; one wavefront
])
@pytest.mark.parametrize("form", [FORCED, LAZY])
def test_per_trial_run_matches_the_oracle(ims, n, m, trials, p, seeds, hub, form):
    rng = np.random.default_rng([n, m, trials, 1])
    off, idx = graph(n, m, rng, hub)
    k = idx.size
    prob = {"mixed": rng.choice([0.0, 0.02, 0.5, 1.0], k), "one": np.ones(k)}.get(p, None)
    prob = np.full(k, float(p)) if prob is None else prob
    sd = rng.choice(n, seeds, replace=False).astype(np.uint32)
    G = ims.Graph(n, off, idx, "ic", prob)
    ref = oracle.simulate("ic", n, off, idx, oracle.encode("ic", prob), sd, trials, 99)
    forced = ims.Opts(test_flags=form)
    for want_bits in (True, False):
        got = ims.simulate(G, np.concatenate([sd, sd[:2]]), trials, 99, want_bits=want_bits, opts=forced)
        assert got["total"] == ref["total"]
        assert (got["trial_counts"].cpu().numpy().view(np.uint32) == ref["trial_counts"]).all()
        assert (got["node_counts"].cpu().numpy().view(np.uint32) == ref["node_counts"]).all()
        if want_bits:
            assert (got["active_bits"].cpu().numpy().view(np.uint64) == ref["active_bits"]).all()
    # same steps as the grid shape takes; a tasks run on the same handle in between changes nothing
    grid = ims.simulate(G, sd, trials, 99, opts=ims.Opts(shape=2))
    assert grid["steps"] == got["steps"]
    again = ims.simulate(G, sd, trials, 99, opts=forced)
    assert again["total"] == ref["total"] and (again["node_counts"].cpu().numpy().view(np.uint32) == ref["node_counts"]).all()
    G.close()
