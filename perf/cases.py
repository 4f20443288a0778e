"""Workloads the framework is timed on: its public calls over the range of sizes they serve.

listed() names twelve of them, draw() gives more of the same ranges.  prepare() builds what a program holds
before the call (graph plan, seed sets, output tensors, network), run() makes one call, work() gives the bytes
and operations of one call that no implementation can avoid, exact() the float64 value of computed numbers
(the simulator's outputs are whole numbers fixed by the inputs, so it has none for them).
"""
import math

import numpy as np
import torch

import paper_2404_17059_amd as ims
from paper_2404_17059_amd import mpnn


def listed():
    return [
        # one notebook-sized call: a small random graph, a few seeds, outputs read by the caller (launch latency)
        {"name": "ic_er_1k", "kind": "ic", "graph": "er", "n": 1000, "deg": 10, "p": 0.1, "seeds": 10, "trials": 1000, "whole": True},
        # a medium scale-free graph at a low uniform probability, many trials
        {"name": "ic_ba_100k", "kind": "ic", "graph": "ba", "n": 100000, "deg": 5, "p": 0.01, "seeds": 50, "trials": 10000, "whole": False},
        # dense cascades (uniformly random probabilities) on a small-world ring: the paper's hardest weighting
        {"name": "ic_ws_ur_10k", "kind": "ic", "graph": "ws", "n": 10000, "deg": 10, "p": "ur", "seeds": 100, "trials": 1000, "whole": False},
        # active nodes per step, for plots of a cascade over time, on a graph of the paper's Facebook sizes
        {"name": "levels_ba_4k", "kind": "levels", "model": "ic", "graph": "ba", "n": 4039, "deg": 22, "p": "tv", "seeds": 100, "trials": 1000},
        # linear threshold on a small sparse graph: long, slow cascades
        {"name": "lt_er_5k", "kind": "lt", "graph": "er", "n": 5000, "deg": 8, "weights": "equal", "top": False, "seeds": 20, "trials": 1000, "whole": True},
        # linear threshold with unequal influence weights, each node's summing to 1
        {"name": "lt_random_100k", "kind": "lt", "graph": "cl", "n": 100000, "deg": 8, "weights": "random", "top": True, "seeds": 50, "trials": 1000, "whole": False},
        # the benchmark's large linear threshold run: nearly every node ends active
        {"name": "lt_chung_lu_1m", "kind": "lt", "graph": "cl", "n": 1000000, "deg": 16, "weights": "equal", "top": True, "seeds": 100, "trials": 1000, "whole": False},
        # a chunk of the first pass of greedy / CELF: single nodes in id order under common random numbers
        {"name": "sets_single_200k", "kind": "sets", "n": 200000, "deg": 10, "sets": 4096, "most": 1, "trials": 1000},
        # training pairs of the spread estimator: sets of 1 to 50 nodes, half drawn by degree (large cascades)
        {"name": "sets_mixed_200k", "kind": "sets", "n": 200000, "deg": 10, "sets": 128, "most": 50, "trials": 1000},
        # a later step of CELF: candidates added to a stored state of the seeds chosen so far
        {"name": "marginal_200k", "kind": "marginal", "n": 200000, "deg": 10, "base": 10, "sets": 64, "trials": 10000},
        # an uneven batch of graphs, IC and LT mixed, as one launch
        {"name": "batch_16", "kind": "batch", "items": 16, "low": 1000, "high": 50000, "trials": 2000},
        # one training pass of the spread estimator: forward, loss, every gradient
        {"name": "train_200k", "kind": "train", "n": 200000, "deg": 10, "batch": 32},
    ]


def _log(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    """One more case: sizes spread over the logarithm of their range."""
    kind = rng.choice(["ic", "ic", "ic", "levels", "lt", "lt", "lt", "sets", "sets", "marginal", "batch", "train"])
    if kind in ("ic", "levels"):
        graph = rng.choice(["er", "ba", "ws"])
        c = {"kind": kind, "graph": graph, "n": _log(rng, 500, 100000 if kind == "ic" else 20000),
             "deg": 2 * rng.randint(2, 6) if graph == "ws" else rng.randint(3, 12), "seeds": rng.randint(1, 120)}
        c["p"] = rng.choice(["tv", "ur", "wc", round(rng.uniform(0.005, 0.12), 4)])
        # the denser the cascades, the fewer trials: a drawn case costs no more than the largest listed one
        arcs = c["n"] * c["deg"] * (2 if graph == "ba" else 1)
        most = {"ur": 3e8, "tv": 1.5e9, "wc": 1.5e9}.get(c["p"], 1.5e9) / (4 if kind == "levels" else 1)
        c["trials"] = _log(rng, 64, max(128, min(10000, int(most / arcs))))
        if kind == "ic":
            c["whole"] = rng.random() < 0.3
        else:
            c["model"] = rng.choice(["ic", "lt"]) if c["n"] <= 5000 else "ic"
        return c
    if kind == "lt":
        c = {"kind": "lt", "graph": rng.choice(["er", "cl", "cl", "ba"]), "n": _log(rng, 1000, 500000), "deg": rng.randint(4, 16),
             "weights": rng.choice(["equal", "equal", "random"]), "top": rng.random() < 0.5, "seeds": rng.randint(5, 100)}
        if c["weights"] == "random":
            c["n"] = min(c["n"], _log(rng, 1000, 100000))
            c["deg"] = min(c["deg"], 10)
        arcs = c["n"] * c["deg"] * (2 if c["graph"] == "ba" else 1)
        c["trials"] = _log(rng, 64, max(128, min(4000, int((4e9 if c["weights"] == "equal" else 8e8) / arcs))))
        c["whole"] = rng.random() < 0.3
        return c
    if kind == "sets":
        most = rng.choice([1, 1, 50])
        n = _log(rng, 5000, 200000)
        return {"kind": "sets", "n": n, "deg": rng.randint(5, 10), "sets": _log(rng, 64, 4096) if most == 1 else _log(rng, 8, 96), "most": most,
                "trials": _log(rng, 100, 1000)}
    if kind == "marginal":
        return {"kind": "marginal", "n": _log(rng, 5000, 200000), "deg": rng.randint(5, 10), "base": rng.randint(1, 40), "sets": _log(rng, 8, 128),
                "trials": _log(rng, 500, 10000)}
    if kind == "batch":
        return {"kind": "batch", "items": rng.randint(4, 16), "low": 1000, "high": _log(rng, 4000, 40000), "trials": _log(rng, 200, 2000)}
    return {"kind": "train", "n": _log(rng, 3000, 150000), "deg": rng.randint(5, 10), "batch": rng.randint(4, 32)}


# ---------------------------------------------------------------- seeded inputs

def _csr(n, src, dst):
    """CSR of the arcs without loops and repeats, targets ascending."""
    keep = src != dst
    key = np.unique(src[keep] * np.int64(n) + dst[keep])
    offsets = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=offsets[1:])
    return offsets, (key % n).astype(np.uint32)


def _graph(kind, n, deg, g):
    """Arcs of an Erdos-Renyi ("er"), preferential-attachment ("ba"), small-world ("ws") or directed power-law ("cl") graph."""
    if kind == "er":
        m = n * deg
        return _csr(n, g.integers(0, n, m), g.integers(0, n, m))
    if kind == "ba":
        # arc end i copies a uniformly chosen earlier end; odd ends are themselves copies and are followed
        m = n * deg
        src = np.arange(m, dtype=np.int64) // deg
        pick = (g.random(m) * (2 * np.arange(m) + 1)).astype(np.int64)
        at = pick.copy()
        odd = np.flatnonzero(at & 1)
        while odd.size:
            at[odd] = pick[at[odd] >> 1]
            odd = odd[(at[odd] & 1) == 1]
        dst = src[at >> 1]
        return _csr(n, np.concatenate([src, dst]), np.concatenate([dst, src]))
    if kind == "ws":
        u = np.repeat(np.arange(n, dtype=np.int64), deg // 2)
        v = (u + np.tile(np.arange(1, deg // 2 + 1, dtype=np.int64), n)) % n
        far = g.random(v.size) < 0.007
        v[far] = g.integers(0, n, int(far.sum()))
        return _csr(n, np.concatenate([u, v]), np.concatenate([v, u]))
    w = np.arange(1, n + 1, dtype=np.float64) ** (-1.0 / 1.1)
    w *= deg * n / w.sum()
    d = np.minimum(g.poisson(w[g.permutation(n)]), n // 2).astype(np.int64)
    src = np.repeat(np.arange(n, dtype=np.int64), d)
    return _csr(n, src, g.integers(0, n, src.size))


def _undirected_power_law(n, deg, g):
    """Both arcs of every edge of a Chung-Lu graph, degree exponent 2.3."""
    w = np.arange(1, n + 1, dtype=np.float64) ** (-1.0 / 1.3)
    cdf = np.cumsum(w[g.permutation(n)])
    k = n * deg // 2
    a, b = (np.minimum(np.searchsorted(cdf, g.random(k) * cdf[-1], side="right"), n - 1) for _ in range(2))
    return _csr(n, np.concatenate([a, b]), np.concatenate([b, a]))


def _equal(n, idx):
    """1 / in-degree of the target: weighted-cascade probabilities, the usual LT weights."""
    return 1.0 / np.bincount(idx, minlength=n)[idx]


def _probabilities(p, n, idx, g):
    if p == "tv":
        return np.array([0.1, 0.01, 0.001])[g.integers(0, 3, idx.size)]
    if p == "ur":
        return g.random(idx.size)
    return _equal(n, idx) if p == "wc" else np.full(idx.size, float(p))


def _weights(kind, n, idx, g):
    if kind == "equal":
        return _equal(n, idx)
    w = g.random(idx.size) + 0.01
    return w / np.bincount(idx, weights=w, minlength=n)[idx]


def _seeds(n, k, off, top, g):
    k = min(k, n)
    s = np.argsort(-np.diff(off), kind="stable")[:k] if top else g.choice(n, k, replace=False)
    return np.sort(s).astype(np.uint32)


def _members(n, deg, count, most, g):
    """Seed sets of 1 to `most` nodes, each drawn uniformly or by degree; single nodes come in id order."""
    if most == 1:
        first = int(g.integers(0, max(1, n - count)))
        return [np.array([v % n], dtype=np.uint32) for v in range(first, first + count)]
    cdf = np.cumsum(deg + 1.0)
    out = []
    for k in g.integers(1, most + 1, count):
        by_deg = np.minimum(np.searchsorted(cdf, g.random(k) * cdf[-1], side="right"), n - 1)
        out.append(np.where(g.random(k) < 0.5, g.integers(0, n, k), by_deg).astype(np.uint32))
    return out


def _outputs(n, trials):
    return {"trial_counts": torch.empty(trials, dtype=torch.int32, device="cuda"), "node_counts": torch.empty(n, dtype=torch.int32, device="cuda"),
            "total": torch.empty(1, dtype=torch.int64, device="cuda")}


def _rng(case, seed):
    return np.random.Generator(np.random.PCG64([seed, case.get("n", 0), case.get("trials", 0)]))


def _batch_items(case, seed):
    g = _rng(case, seed)
    items = []
    for i in range(case["items"]):
        # sizes spread over the range, large and small ones in turn
        n = int(round(case["low"] * (case["high"] / case["low"]) ** ((i * 7 % case["items"]) / max(1, case["items"] - 1))))
        off, idx = _graph("er" if i % 2 == 0 else "ba", n, 8 if i % 2 == 0 else 4, g)
        items.append((ims.Graph(n, off, idx, "ic" if (i // 2) % 2 == 0 else "lt", _equal(n, idx)), _seeds(n, 20, off, False, g), case["trials"],
                      int(g.integers(1, 1 << 40))))
    return items


def _train_inputs(case, seed):
    g = _rng(case, seed)
    n, b = case["n"], case["batch"]
    off, idx = _undirected_power_law(n, case["deg"], g)
    a = _equal(n, idx).astype(np.float32)
    sets = _members(n, np.diff(off), b, 50, g)
    params = mpnn.init_params(int(g.integers(1, 1 << 40)))
    params[mpnn.OFF["bo"]] = math.log(0.03 / 0.97)
    target = np.exp(g.uniform(math.log(20.0), math.log(0.15 * n), b)).astype(np.float32)
    return n, off, idx, a, sets, params, target


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return {"case": case, "batch": ims.Batch(_batch_items(case, seed))}
    if kind == "train":
        n, off, idx, a, sets, params, target = _train_inputs(case, seed)
        offs, nodes = ims.pack_sets(sets)
        return {"case": case, "net": mpnn.Surrogate(n, off, idx, a, max_batch=case["batch"]), "offs": offs, "nodes": nodes,
                "params": torch.from_numpy(params).cuda(), "target": torch.from_numpy(target).cuda(),
                "grads": torch.empty(mpnn.NPARAMS, dtype=torch.float32, device="cuda"), "loss": torch.empty(1, dtype=torch.float32, device="cuda")}
    g = _rng(case, seed)
    n = case["n"]
    if kind in ("sets", "marginal"):
        off, idx = _undirected_power_law(n, case["deg"], g)
        s = {"case": case, "graph": ims.Graph(n, off, idx, "ic", _equal(n, idx)), "rng": int(g.integers(1, 1 << 40))}
        if kind == "sets":
            s["sets"] = _members(n, np.diff(off), case["sets"], case["most"], g)
            return s
        order = np.argsort(-np.diff(off), kind="stable").astype(np.uint32)
        s["bits"] = ims.simulate(s["graph"], order[:case["base"]], case["trials"], s["rng"], want_bits=True, want_node_counts=False)["active_bits"]
        s["sets"] = [order[k:k + 1] for k in range(case["base"], case["base"] + case["sets"])]
        return s
    off, idx = _graph(case["graph"], n, case["deg"], g)
    lt = kind == "lt" or case.get("model") == "lt"
    param = _weights(case.get("weights", "equal"), n, idx, g) if lt else _probabilities(case["p"], n, idx, g)
    s = {"case": case, "graph": ims.Graph(n, off, idx, "lt" if lt else "ic", param), "seeds": _seeds(n, case["seeds"], off, case.get("top", False), g),
         "rng": int(g.integers(1, 1 << 40))}
    if kind != "levels" and not case["whole"]:
        s["out"] = _outputs(n, case["trials"])
    return s


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        state["batch"].launch()
        return [out[:3] for out in state["batch"].outputs]
    if kind == "train":
        pred = state["net"].forward_packed(state["params"], state["offs"], state["nodes"])
        grads = state["net"].backward(state["params"], state["target"], grads=state["grads"], loss=state["loss"])
        return {"pred": pred, "loss": state["loss"], "grads": grads}
    if kind == "sets":
        return ims.simulate_sets(state["graph"], state["sets"], case["trials"], state["rng"])["totals"]
    if kind == "marginal":
        return ims.simulate_sets_from(state["graph"], state["bits"], state["sets"], case["trials"], state["rng"])["new_totals"]
    if kind == "levels":
        r = ims.simulate_levels(state["graph"], state["seeds"], case["trials"], state["rng"], max_levels=64)
        # one row per level of the axis the curves are drawn over
        return {"level_counts": np.pad(r["level_counts"], ((0, 64 - len(r["level_counts"])), (0, 0))), "trial_counts": r["trial_counts"],
                "total": r["total"]}
    if case["whole"]:
        r = ims.simulate(state["graph"], state["seeds"], case["trials"], state["rng"])
        return {k: r[k] for k in ("trial_counts", "node_counts", "total")}
    out = state["out"]
    ims.simulate_into(state["graph"], state["seeds"], case["trials"], state["rng"], out["trial_counts"], out["total"], out["node_counts"])
    return out


def work(case):
    """The graph, the seeds and the parameters read once, the outputs written once; the network's products."""
    kind = case["kind"]
    if kind == "batch":
        mean = (case["high"] - case["low"]) / math.log(case["high"] / case["low"])
        return {"bytes": case["items"] * (mean * (8 + 8 * 8 + 4) + 4 * case["trials"]), "flops": 0}
    n = case["n"]
    arcs = n * case["deg"] * (2 if case.get("graph") == "ba" else 1)
    if kind == "train":
        rows = n * case["batch"]
        dense = 2 * rows * 64 * (32 + 128 + 128)
        return {"bytes": 8 * (n + 1) + 8 * arcs + 12 * n + 3 * 4 * mpnn.NPARAMS,
                # forward, weight gradients (all layers), input gradients (two layers), five aggregations
                "flops": 2 * dense + 2 * rows * 64 * 256 + 2 * case["batch"] * arcs * (16 + 4 * 64)}
    graph = 8 * (n + 1) + 8 * arcs
    if kind in ("sets", "marginal"):
        state = 8 * n * ((case["trials"] + 63) // 64) if kind == "marginal" else 0
        return {"bytes": graph + state + case["sets"] * (2 * (case.get("most", 1) + 1) + 8), "flops": 0}
    return {"bytes": graph + 4 * case["seeds"] + 4 * case["trials"] + (4 * n if kind != "levels" else 0), "flops": 0}


def exact(case, seed):
    """The training pass in float64; the simulator's outputs are whole numbers."""
    if case["kind"] != "train":
        return None
    n, off, idx, a, sets, params, target = _train_inputs(case, seed)
    dev = "cuda"
    f64 = lambda x: torch.from_numpy(np.asarray(x, dtype=np.float64)).to(dev)  # noqa: E731
    src = torch.from_numpy(np.repeat(np.arange(n), np.diff(off))).to(dev)
    dst = torch.from_numpy(idx.astype(np.int64)).to(dev)
    w = f64(a)[:, None]
    asum = np.bincount(np.repeat(np.arange(n), np.diff(off)), weights=a.astype(np.float64), minlength=n)
    feat = f64(np.stack([np.log1p(np.diff(off)), np.log1p(np.bincount(idx, minlength=n)), np.log1p(asum)], axis=1))
    into = lambda h: torch.zeros_like(h).index_add_(0, dst, w * h[src])  # noqa: E731
    back = lambda h: torch.zeros_like(h).index_add_(0, src, w * h[dst])  # noqa: E731
    p = f64(params)
    sizes = [(mpnn.IN, "W0", "b0"), (64, "W1", "b1"), (64, "W2", "b2")]
    layers = [(p[mpnn.OFF[x]:mpnn.OFF[x] + 2 * d * 64].view(2 * d, 64), p[mpnn.OFF[y]:mpnn.OFF[y] + 64]) for d, x, y in sizes]
    wo, bo = p[mpnn.OFF["wo"]:mpnn.OFF["wo"] + 64], p[mpnn.OFF["bo"]]
    pred, grads = torch.zeros(len(sets), dtype=torch.float64, device=dev), torch.zeros_like(p)
    goal = f64(target)
    for b, members in enumerate(sets):
        x = torch.zeros(n, mpnn.IN, dtype=torch.float64, device=dev)
        x[:, 1:4] = feat
        hit = torch.from_numpy(np.unique(members).astype(np.int64)).to(dev)
        x[hit, 0] = 1.0
        h, ins = x, []
        for wl, bl in layers:
            ins.append(torch.cat([h, into(h)], dim=1))
            h = torch.relu(ins[-1] @ wl + bl)
        y = torch.sigmoid(h @ wo + bo)
        y[hit] = 1.0
        pred[b] = y.sum()
        dz = 2.0 * (pred[b] - goal[b]) / n / n / len(sets) * y * (1.0 - y)
        grads[mpnn.OFF["wo"]:mpnn.OFF["wo"] + 64] += h.t() @ dz
        grads[mpnn.OFF["bo"]] += dz.sum()
        d = dz[:, None] * wo
        for (wl, _), z, (width, wname, bname) in zip(reversed(layers), reversed(ins), reversed(sizes)):
            d = d * (h > 0)
            grads[mpnn.OFF[wname]:mpnn.OFF[wname] + 2 * width * 64] += (z.t() @ d).reshape(-1)
            grads[mpnn.OFF[bname]:mpnn.OFF[bname] + 64] += d.sum(0)
            h = z[:, :width]
            if wname != "W0":
                g = d @ wl.t()
                d = g[:, :width] + back(g[:, width:])
    return {"pred": pred, "loss": (((pred - goal) / n) ** 2).mean().reshape(1), "grads": grads}
