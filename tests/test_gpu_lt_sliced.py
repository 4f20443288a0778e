"""LT sweeps over unequal in-weights (bit-sliced sums of the weights' top
halves, exact sums where those leave a trial open) against the oracle: active
bits, per-trial and per-node counts, whole numbers, so equal.  Word counts at
the edges of the form (it starts at six) and of its padding to 8 and 16; rows
at the edge of the 64 pieces a sweep stages; sweeps that all mark and that
never mark; sums that fall on a threshold, beside it, and on either side of
its top half, so that the exact sums decide."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

RNG = 4711
LT_NODE = 2  # hash domain of the LT thresholds


@pytest.fixture(scope="module")
def ims():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2404_17059_amd as m
    return m


def check(ims, n, off, idx, w, seeds, T, alpha):
    pairs = np.unique(np.stack([idx.astype(np.uint64), w]), axis=1)
    assert pairs.shape[1] > len(np.unique(idx))  # equal weights at every node take another form
    ref = oracle.simulate("lt", n, off, idx, w, seeds, T, RNG, threads=8)
    G = ims.Graph(n, off, idx, "lt", w)
    for want_bits in (True, False):
        got = ims.simulate(G, seeds, T, RNG, want_bits=want_bits, opts=ims.Opts(shape=2, alpha=alpha))
        assert got["total"] == ref["total"]
        assert (got["trial_counts"].cpu().numpy().view(np.uint32) == ref["trial_counts"]).all()
        assert (got["node_counts"].cpu().numpy().view(np.uint32) == ref["node_counts"]).all()
        if want_bits:
            assert (got["active_bits"].cpu().numpy().view(np.uint64) == ref["active_bits"]).all()
    G.close()
    return ref


def csr(n, src, dst, w):
    order = np.lexsort((dst, src))
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(src, minlength=n), out=off[1:])
    return off, dst[order].astype(np.uint32), w[order].astype(np.uint64)


@pytest.mark.parametrize("alpha", [0.0, 1e-12, 2.0])  # by the rule, no sweep marks, every sweep marks
@pytest.mark.parametrize("T", [321, 384, 448, 450, 512, 577, 1000, 1024, 1088])
def test_rows_around_the_staged_length(ims, T, alpha):
    g = np.random.default_rng([T, 2])
    n = 400
    src, dst = [], []
    for v, d in enumerate([63, 64, 65, 130, 1, 2, 8, 32, 63, 1, 64, 0, 65]):
        src.append(g.choice(np.arange(20, n), d, replace=False))
        dst.append(np.full(d, v))
    src.append(g.integers(0, n, 3 * n))
    dst.append(g.integers(20, n, 3 * n))
    src, dst = np.concatenate(src), np.concatenate(dst)
    w = g.random(src.size) + 0.01
    w = (w / np.bincount(dst, weights=w, minlength=n)[dst] * 0.99999 * 2.0**32).astype(np.uint64)
    w[dst == 4] = 1 << 32  # one arc of the whole weight
    off, idx, w = csr(n, src, dst, w)
    check(ims, n, off, idx, w, g.choice(n, 12, replace=False).astype(np.uint32), T, alpha)


@pytest.mark.parametrize("T,pieces", [(384, 2), (512, 3), (1000, 8), (1024, 33), (700, 64)])
def test_sums_at_the_thresholds(ims, T, pieces):
    """Node v's in-weights, all from seeds, sum to a threshold of one of its trials (or to its top half) and a little."""
    g = np.random.default_rng([T, pieces])
    shifts = [-1, 0, 1, 2, -(1 << 16), 1 << 16]
    first = 64  # seeds 0 .. 63, then two nodes per shift and whole / top half for 20 trials
    targets = [(t, s, top) for t in g.choice(T, 20, replace=False) for s in shifts for top in (False, True)]
    n = first + len(targets)
    src, dst, w, joins = [], [], [], []
    for k, (t, s, top) in enumerate(targets):
        v = first + k
        h = oracle.hash32(RNG, LT_NODE, int(t), v)
        total = min(max(((h >> 16) << 16 if top else h) + s, pieces), 1 << 32)
        cut = np.sort(g.choice(np.arange(1, total), pieces - 1, replace=False)) if total < 1 << 20 else np.sort(g.integers(1, total, pieces - 1))
        parts = np.diff(np.concatenate([[0], cut, [total]]))
        src.append(g.choice(64, pieces, replace=False))
        dst.append(np.full(pieces, v))
        w.append(parts)
        joins.append((int(t), v, total > h))
    off, idx, w = csr(n, np.concatenate(src), np.concatenate(dst), np.concatenate(w))
    ref = check(ims, n, off, idx, w, np.arange(64, dtype=np.uint32), T, 0.0)
    for t, v, on in joins:
        assert bool(ref["active_bits"][t // 64, v] >> np.uint64(t % 64) & np.uint64(1)) == on
