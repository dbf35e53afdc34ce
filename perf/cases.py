"""The work this library is measured on: calls of its public entry points as a program would make them.

A case is a dict of plain values; `op` names the entry point, the rest its sizes and the shape of its data.  Inputs
are synthetic, drawn on the GPU from a seed, with the distributions of the library's named workloads:

  equal   equal Gaussian blobs in a box, one spread for all of them
  spread  the same with a spread of its own for every blob, U[0.5, 2]
  zipf    blob sizes by Zipf's law with exponent 1.1 (a few blobs hold most rows)
  tight   tiny blobs far apart and 1 % of the rows bit-exact copies of others
  image   sparse non-negative rows made from 10 class templates, 80 % of the entries exactly 0

A program that clusters again and again keeps its workspace and its output tensors, so `prepare` makes both where the
call takes them.
"""
import math

import torch

import paper_2306_16354_amd as slhc

DEVICE = "cuda"


def listed():
    return [
        # -- the whole path: k-NN graph, spanning tree, dendrogram
        # interactive use: a few thousand rows, where launches, copies and host work are the time
        dict(name="slhc_4k_16", op="slhc", N=4096, d=16, k=16, data="equal", blobs=10, box=10.0),
        # an everyday table of embeddings
        dict(name="slhc_100k_64", op="slhc", N=100_000, d=64, k=32, data="spread", blobs=50, box=20.0),
        # the headline: a million descriptors, cluster sizes over three orders of magnitude
        dict(name="slhc_1m_128", op="slhc", N=1_000_000, d=128, k=32, data="zipf", blobs=1000, box=50.0),
        # images as rows: too many features for tiles to be skipped, so every pair is multiplied
        dict(name="slhc_250k_784", op="slhc", N=250_000, d=784, k=16, data="image", blobs=10, box=1.0),
        # many rows, few features, small k, duplicates: many rounds of connecting components
        dict(name="slhc_2m_32", op="slhc", N=2_000_000, d=32, k=8, data="tight", blobs=20_000, box=1000.0),
        # -- the neighbour graph alone
        # the headline's graph by brute force, the library's benchmark figure
        dict(name="knn_1m_128", op="knn", N=1_000_000, d=128, k=32, data="zipf", blobs=1000, box=50.0),
        # odd row count, a feature count that no tile likes
        dict(name="knn_20011_50", op="knn", N=20_011, d=50, k=10, data="equal", blobs=40, box=20.0),
        # the smallest call: a serving loop that may not allocate
        dict(name="knn_static_2k_32", op="knn_static", N=2048, d=32, k=8, data="equal", blobs=10, box=10.0),
        # -- nearest row of another matrix: few queries against an index
        dict(name="fused_1nn_1k_100k_128", op="fused_1nn", m=1000, n=100_000, d=128, data="equal", blobs=200, box=20.0),
        # nearest row of another colour, for a listed subset of rows
        dict(name="cross_1nn_10k_100k_64", op="cross_1nn", N=100_000, d=64, m=10_000, data="spread", blobs=50, box=20.0),
        # -- spanning forest of a road-like graph with a million vertices
        dict(name="csr_msf_1m", op="csr_msf", side=1024, integer_weights=False),
        # -- flat clusters from a finished dendrogram
        dict(name="flat_1m", op="flat", N=1_000_000, clusters=1000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _points(rng, N, d):
    """A data kind with parameters that suit N rows: clusters of a few dozen to a few thousand rows."""
    data = rng.choice(["equal", "spread", "zipf", "tight"])
    per_blob = _log_int(rng, 60, 3000) if data != "tight" else _log_int(rng, 60, 200)
    box = {"equal": 20.0, "spread": 20.0, "zipf": 50.0, "tight": 1000.0}[data]
    return dict(data=data, blobs=max(2, N // per_blob), box=box)


def draw(rng):
    op = rng.choice(["slhc", "slhc", "slhc", "slhc_wide", "knn", "knn", "knn_static", "fused_1nn", "fused_1nn",
                     "cross_1nn", "csr_msf", "flat"])
    if op == "slhc":
        N, d = _log_int(rng, 600, 1_000_000), _log_int(rng, 4, 128)
        return dict(op="slhc", N=N, d=d, k=_log_int(rng, 4, 64), **_points(rng, N, d))
    if op == "slhc_wide":
        return dict(op="slhc", N=_log_int(rng, 2000, 100_000), d=_log_int(rng, 150, 800), k=_log_int(rng, 4, 32),
                    data="image", blobs=10, box=1.0)
    if op == "knn":
        N, d = _log_int(rng, 1000, 300_000), _log_int(rng, 4, 300)
        return dict(op="knn", N=N, d=d, k=_log_int(rng, 1, 64), **_points(rng, N, d))
    if op == "knn_static":
        N, d = _log_int(rng, 500, 30_000), _log_int(rng, 4, 128)
        return dict(op="knn_static", N=N, d=d, k=_log_int(rng, 4, 32), **_points(rng, N, d))
    if op == "fused_1nn":
        n, d = _log_int(rng, 2000, 500_000), _log_int(rng, 4, 256)
        return dict(op="fused_1nn", m=_log_int(rng, 10, 20_000), n=n, d=d, **_points(rng, n, d))
    if op == "cross_1nn":
        N, d = _log_int(rng, 2000, 300_000), _log_int(rng, 4, 128)
        return dict(op="cross_1nn", N=N, d=d, m=_log_int(rng, 50, min(N, 20_000)), **_points(rng, N, d))
    if op == "csr_msf":
        return dict(op="csr_msf", side=_log_int(rng, 40, 3000), integer_weights=rng.random() < 0.3)
    N = _log_int(rng, 1000, 1_000_000)
    return dict(op="flat", N=N, clusters=_log_int(rng, 2, N // 4))


# ---- inputs

def _make_points(gen, N, d, data, blobs, box):
    """(X float32 [N, d], blob of every row int32 [N]), rows in random order."""
    if data == "image":
        templates = torch.rand((blobs, d), generator=gen, device=DEVICE) < 0.2
        label = torch.randint(blobs, (N,), generator=gen, device=DEVICE)
        X = torch.empty((N, d), dtype=torch.float32, device=DEVICE)
        for s in range(0, N, 65_536):
            on_template = templates[label[s:s + 65_536]]
            on = torch.rand(on_template.shape, generator=gen, device=DEVICE) < torch.where(on_template, 0.9, 0.025)
            X[s:s + 65_536] = on * (1.0 - torch.rand(on_template.shape, generator=gen, device=DEVICE))
        return X, label.to(torch.int32)
    share = torch.ones(blobs, dtype=torch.float64, device=DEVICE)
    if data == "zipf":
        share = torch.arange(1, blobs + 1, dtype=torch.float64, device=DEVICE) ** -1.1
    ends = torch.cumsum(share, 0) / share.sum() * N
    label = torch.searchsorted(ends, torch.arange(N, dtype=torch.float64, device=DEVICE), right=True).clamp_(max=blobs - 1)
    label = label[torch.randperm(N, generator=gen, device=DEVICE)]
    centres = (2.0 * torch.rand((blobs, d), generator=gen, device=DEVICE) - 1.0) * box
    std = torch.full((blobs, 1), 0.1 if data == "tight" else 1.0, device=DEVICE)
    if data == "spread":
        std = 0.5 + 1.5 * torch.rand((blobs, 1), generator=gen, device=DEVICE)
    X = torch.randn((N, d), generator=gen, device=DEVICE).mul_(std[label]).add_(centres[label])
    if data == "tight":
        copies = N // 100
        at = torch.randperm(N, generator=gen, device=DEVICE)[:2 * copies]
        X[at[:copies]] = X[at[copies:]]
        label[at[:copies]] = label[at[copies:]]
    return X, label.to(torch.int32)


def _make_road_graph(gen, side, integer_weights):
    """Symmetric CSR of side parallel streets of side vertices, connected by one road along their ends and by a
    quarter of the possible side roads (average degree 2.5, one component, as in road networks), vertex ids
    shuffled, weights U[1, 100) or whole numbers 1..10 (many ties)."""
    V = side * side
    ids = torch.arange(V, device=DEVICE).reshape(side, side)
    across = torch.rand((side - 1, side), generator=gen, device=DEVICE) < 0.25
    across[:, 0] = True
    a = torch.cat([ids[:, :-1].reshape(-1), ids[:-1, :][across]])
    b = torch.cat([ids[:, 1:].reshape(-1), ids[1:, :][across]])
    if integer_weights:
        w = torch.randint(1, 11, a.shape, generator=gen, device=DEVICE).to(torch.float32)
    else:
        w = 1.0 + 99.0 * torch.rand(a.shape, generator=gen, device=DEVICE)
    shuffled = torch.randperm(V, generator=gen, device=DEVICE)
    a, b = shuffled[a], shuffled[b]
    key, order = torch.sort(torch.cat([a * V + b, b * V + a]))
    offsets = torch.searchsorted(key, torch.arange(V + 1, device=DEVICE) * V)
    return (offsets.to(torch.int32), (key % V).to(torch.int32), torch.cat([w, w])[order].contiguous())


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    op, state = case["op"], dict(case)
    if op == "csr_msf":
        state["graph"] = _make_road_graph(gen, case["side"], case["integer_weights"])
        return state
    if op == "flat":
        X, _ = _make_points(gen, case["N"], 8, "equal", max(2, case["N"] // 300), 20.0)
        state["children"] = slhc.slhc(X, 8, prune=None)["children"]
        state["workspace"] = _bytes(slhc.flat_clusters_workspace_bytes(case["N"]))
        state["out"] = torch.empty(case["N"], dtype=torch.int32, device=DEVICE)
        return state
    kind = (case["data"], case["blobs"], case["box"])
    if op == "fused_1nn":
        XY, _ = _make_points(gen, case["m"] + case["n"], case["d"], *kind)
        state["Q"], state["Y"] = XY[:case["m"]].contiguous(), XY[case["m"]:].contiguous()
        state["out"] = _pair(case["m"])
        return state
    N, d = case["N"], case["d"]
    X, label = _make_points(gen, N, d, *kind)
    state["X"] = X
    if op == "cross_1nn":
        state["colour"] = label
        state["rows"] = torch.randperm(N, generator=gen, device=DEVICE)[:case["m"]].to(torch.int32)
    elif op == "slhc":
        state["workspace"] = _bytes(slhc.slhc_workspace_bytes(N, d, case["k"]))
        state["out"] = None
    else:
        state["out"] = _pair(N, case["k"])
        if op == "knn":
            state["workspace"] = _bytes(slhc.knn_workspace_bytes(N, d, case["k"]))
    return state


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device=DEVICE)


def _pair(*shape):
    return (torch.empty(shape, dtype=torch.int32, device=DEVICE), torch.empty(shape, dtype=torch.float32, device=DEVICE))


# ---- one pass

def run(state):
    op = state["op"]
    if op == "slhc":
        # prune=None is the library's plain entry point: it decides by size whether tiles are skipped
        state["out"] = slhc.slhc(state["X"], state["k"], workspace=state["workspace"], out=state["out"], prune=None)
        return {name: t for name, t in state["out"].items() if name != "stats"}
    if op == "knn":
        return slhc.knn_graph(state["X"], state["k"], out=state["out"], workspace=state["workspace"])
    if op == "knn_static":
        return slhc.knn_graph_static(state["X"], state["k"], state["out"])
    if op == "fused_1nn":
        return slhc.fused_1nn(state["Q"], state["Y"], out=state["out"])
    if op == "cross_1nn":
        return slhc.cross_1nn(state["X"], state["colour"], rows=state["rows"])
    if op == "csr_msf":
        forest = slhc.csr_msf(*state["graph"])
        return {name: forest[name] for name in ("mst_src", "mst_dst", "mst_w", "colours")}
    return slhc.flat_clusters(state["children"], state["clusters"], workspace=state["workspace"], out=state["out"])


# ---- what a pass cannot do without

def work(case):
    """Brute-force calls multiply every pair (2 d operations each).  The whole path prunes where it can (up to 128
    features, from 24 576 rows on): there only the k listed distances per row are counted, 3 d operations each."""
    op = case["op"]
    if op == "csr_msf":
        V = case["side"] ** 2
        E = 2 * 1.25 * case["side"] * (case["side"] - 1)
        return {"bytes": 4 * (V + 1) + 8 * E + 12 * (V - 1) + 4 * V, "flops": 0}
    if op == "flat":
        return {"bytes": 8 * (case["N"] - 1) + 4 * case["N"], "flops": 0}
    d = case["d"]
    if op == "fused_1nn":
        return {"bytes": 4 * d * (case["m"] + case["n"]) + 8 * case["m"], "flops": 2 * d * case["m"] * case["n"]}
    N = case["N"]
    if op == "cross_1nn":
        return {"bytes": 4 * d * N + 4 * N + 12 * case["m"], "flops": 2 * d * case["m"] * N}
    k = case["k"]
    every_pair = {"bytes": 4 * d * N + 8 * k * N, "flops": 2 * d * N * N}
    if op != "slhc":
        return every_pair
    flops = 3 * d * N * k if d <= 128 and N >= 24_576 else every_pair["flops"]
    return {"bytes": 4 * d * N + 28 * (N - 1), "flops": flops}


def tolerance(case):
    """Distances are float32 sums of d squares.  Rows at almost equal distance may change places in a list, and edges
    of almost equal weight in a tree (with the numbers of the merges they cause).  Graph weights are only copied."""
    if case["op"] in ("csr_msf", "flat"):
        return "exact"
    return {"rel": 1e-5, "max": 1e-4, "differ": 0.01 if case["op"] == "slhc" else 1e-3}
