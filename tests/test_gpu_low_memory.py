"""Calls made while little device memory is left: they run in the forms that
need less, or fail with the out-of-memory error and leave everything usable."""
import contextlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ims():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2404_17059_amd as m
    return m


@contextlib.contextmanager
def only(mib):
    """Hold all of the device's memory but about `mib` MiB."""
    import torch
    torch.cuda.empty_cache()
    held = []
    for chunk in (32768, 1024, 128, 12):
        while torch.cuda.mem_get_info()[0] - (chunk << 20) >= mib << 20:
            held.append(torch.empty(chunk << 20, dtype=torch.uint8, device="cuda"))
    print("left:", torch.cuda.mem_get_info()[0] >> 20, "MiB", flush=True)
    try:
        yield
    finally:
        torch.cuda.synchronize()
        held.clear()
        torch.cuda.empty_cache()


def sparse_graph(n, m, seed):
    g = np.random.default_rng(seed)
    key = np.unique(g.integers(0, n * n, m))
    off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=off[1:])
    return off, (key % n).astype(np.uint32)


def lt_graph(ims, n, m):
    off, idx = sparse_graph(n, m, 3)
    return ims.Graph(n, off, idx, "lt", 1.0 / np.bincount(idx, minlength=n)[idx])


def counts(r):
    return [x if isinstance(x, (int, np.ndarray)) else x.cpu().numpy().view(np.uint32) for x in (r["total"], r["trial_counts"], r["node_counts"])]


def equal(a, b):
    assert all(np.array_equal(x, y) for x, y in zip(counts(a), counts(b)))


def test_a_plan_without_room_leaves_the_batch_as_it_was(ims):
    """Task timing lists the item as tasks, whose slots find no room: the call fails, the batch goes on."""
    n, T = 20000, 1 << 14
    G, R = lt_graph(ims, n, 2 * n), lt_graph(ims, n, 2 * n)
    seeds = np.array([5, 77, 1234], dtype=np.uint32)
    want = ims.simulate(R, seeds, T, 9)
    B = ims.Batch([(G, seeds, T, 9)])
    B.launch()
    equal(B.results()[0], want)
    with only(700):  # the remainders of 512 slots alone take 1,250
        with pytest.raises(ims.ImsError) as e:
            B.task_timing(True)
        assert e.value.code == -5
        B.launch()
        equal(B.results()[0], want)
    B.task_timing(True)
    B.launch()
    equal(B.results()[0], want)
    assert len(B.task_times()[0]) == T // 8
    B.close()
    G.close()
    R.close()


def test_calls_without_room_for_per_trial_workspaces_take_the_general_forms(ims):
    """An LT run and a batch item (1 GiB of starting states), an IC run and seed sets (1.2 GiB of coin rows)."""
    n, T = 4000, 1 << 18
    off, idx = sparse_graph(n, 10 * n, 4)
    lt, ic = lt_graph(ims, n, 2 * n), ims.Graph(n, off, idx, "ic", np.full(idx.size, 0.02))
    seeds = np.array([5, 77, 1234], dtype=np.uint32)
    sets = [seeds, seeds[:1], seeds[1:]]
    forced = ims.Opts(test_flags=16)

    def calls(lt, ic, opts):
        batch = ims.Batch([(lt, seeds, T, 9)])
        batch.launch()
        out = [ims.simulate(lt, seeds, T, 9, opts=opts), ims.simulate(ic, seeds, T, 9, opts=opts), batch.results()[0]]
        totals = ims.simulate_sets(ic, sets, T, 9, opts=opts)["totals"]
        batch.close()
        return out, totals

    R = [lt_graph(ims, n, 2 * n), ims.Graph(n, off, idx, "ic", np.full(idx.size, 0.02))]
    want, want_totals = calls(*R, None)
    for g in R:
        g.close()
    for room in (850, None):
        with only(room) if room else contextlib.nullcontext():
            got, totals = calls(lt, ic, forced)
        for x, y in zip(got, want):
            equal(x, y)
        assert (totals == want_totals).all()
    lt.close()
    ic.close()


def test_graph_without_room_for_arc_records(ims):
    """4M arcs, whose records take 32 MiB beside the rest."""
    import torch
    n = 200000
    off, idx = sparse_graph(n, 20 * n, 5)
    w = 1.0 / np.bincount(idx, minlength=n)[idx]
    seeds = np.arange(0, n, 5000, dtype=np.uint32)
    R = ims.Graph(n, off, idx, "lt", w)
    want = ims.simulate(R, seeds, 64, 9, opts=ims.Opts(shape=2))
    torch.cuda.synchronize()
    R.close()
    free = torch.cuda.mem_get_info()[0]
    R = ims.Graph(n, off, idx, "lt", w)
    whole = (free - torch.cuda.mem_get_info()[0]) >> 20
    R.close()
    print("graph:", whole, "MiB", flush=True)
    with only(whole - 28):
        G = ims.Graph(n, off, idx, "lt", w)
    equal(ims.simulate(G, seeds, 64, 9), want)
    G.close()
