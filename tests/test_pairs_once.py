"""Searches that multiply every pair of rows once (pairs_kernels.hip): lists and trees against the float32-product list kernels,
bit for bit, where blocks, offsets round the circle, bands and lists end."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2306_16354_amd as slhc
    slhc.load_library()
    assert torch.cuda.is_available()
    return slhc


def blobs(N, d, seed, spread=8.0, rows=400):
    g = torch.Generator(device="cuda").manual_seed(seed)
    centres = (2 * torch.rand((max(2, N // rows), d), generator=g, device="cuda") - 1) * spread
    label = torch.randint(len(centres), (N,), generator=g, device="cuda")
    return centres[label] + torch.randn((N, d), generator=g, device="cuda")


# the smallest search of its kind and, of both orders of every pair, the one of a row less; an odd and an even circle of blocks, the last of
# one to four tiles; every number of 16-column steps; whole and partial chunks beyond 128 columns; lists from 256 entries to 1024; one to
# several bands; the smallest search of 384 tiles
@pytest.mark.parametrize("N,d,k", [
    (3968, 33, 8), (3969, 33, 8), (4096, 48, 1), (4097, 49, 64), (4609, 64, 15), (5120, 65, 31), (6001, 81, 7), (7000, 97, 3), (8191, 113, 16),
    (9000, 128, 33), (9217, 128, 2), (4100, 129, 5), (4353, 192, 64), (5000, 321, 20), (12_545, 784, 9), (49_025, 66, 10), (50_000, 100, 50), (150_000, 80, 24),
    (70_000, 200, 12), (200_000, 128, 40),
])
def test_lists(lib, N, d, k):
    print(f"pairs once N={N} d={d} k={k}", flush=True)
    assert lib.probe_knn_products(N, d, k) == (0.5 if N > 3968 else 1.0)
    X = blobs(N, d, N + d)
    want, got = lib.knn_graph(X, k, fp32_filter=True), lib.knn_graph(X, k)
    torch.cuda.synchronize()
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])


# blocks of which every lane holds pairs that pass (one blob, long lists) or every pair does (half the rows one point): more than are looked through at a time, and
# than wait for their slots
@pytest.mark.parametrize("kind", ["blob", "point"])
@pytest.mark.parametrize("N,d,k", [(3969, 33, 64), (4500, 64, 50), (6500, 100, 64), (12_000, 128, 64), (4300, 129, 64), (4500, 320, 39)])
def test_crowded_blocks(lib, kind, N, d, k):
    print(f"pairs once, crowded, {kind}, N={N} d={d} k={k}", flush=True)
    assert lib.probe_knn_products(N, d, k) == 0.5
    X = torch.randn((N, d), generator=torch.Generator(device="cuda").manual_seed(N), device="cuda")
    if kind == "point":
        X[::2] = X[0]
    want, got = lib.knn_graph(X, k, fp32_filter=True), lib.knn_graph(X, k)
    torch.cuda.synchronize()
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])


# 9 to 13 steps of 16 columns: chunks of two with one step or two in the last, places of rows with up to three empty steps; both orders of
# every pair (fewer rows) and one, an odd number of tiles; 1-NN, of few queries with several segments
@pytest.mark.parametrize("d", [129, 145, 161, 177, 193, 208])
def test_chunks_of_columns(lib, d):
    print(f"chunks of columns d={d}", flush=True)
    for N in (2500, 4700):
        assert lib.probe_knn_products(N, d, 9) == (0.5 if N > 4000 else 1.0)
        X = blobs(N, d, d)
        want, got = lib.knn_graph(X, 9, fp32_filter=True), lib.knn_graph(X, 9)
        torch.cuda.synchronize()
        assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])
        # (a float32 sum of d squares is off by (d + 2) 2^-24 of its value at most, 1.3e-5)
        best = torch.cdist(X[:200].double().cpu(), X[200:].double().cpu()).square().min(1).values
        assert torch.allclose(lib.fused_1nn(X[:200], X[200:])[1].double().cpu(), best, rtol=2e-5, atol=0)
        colour = (torch.arange(N, device="cuda") < 200).to(torch.int32)
        rows = torch.arange(200, dtype=torch.int32, device="cuda")
        assert torch.allclose(lib.cross_1nn(X, colour, rows=rows)[1].double().cpu(), best, rtol=2e-5, atol=0)


# values beyond float16 on either side of a pair, rows with more ties than a list holds, one row that no other is near, rows in the
# order of their clusters
@pytest.mark.parametrize("kind", ["beyond_float16", "ties", "far_row", "sorted", "not_finite"])
@pytest.mark.parametrize("N,d,k", [(5000, 64, 12), (4500, 160, 12)])
def test_lists_of_unlike_rows(lib, kind, N, d, k):
    print(f"pairs once, {kind}, N={N} d={d}", flush=True)
    assert lib.probe_knn_products(N, d, k) == 0.5
    X = blobs(N, d, 7)
    if kind == "beyond_float16":
        X[::600] *= 1e7
    elif kind == "ties":
        X[::3] = X[0]
    elif kind == "far_row":
        X[N // 2] += 1e4
    elif kind == "sorted":
        X = X[torch.argsort(X[:, 0])].contiguous()
    elif kind == "not_finite":
        X[N // 3] = float("nan")
        X[N // 5, 2] = float("inf")
    want, got = lib.knn_graph(X, k, fp32_filter=True), lib.knn_graph(X, k)
    torch.cuda.synchronize()
    if kind == "not_finite":
        rows = torch.ones(N, dtype=torch.bool, device="cuda")
        rows[N // 3] = rows[N // 5] = False
        assert torch.equal(want[0][rows], got[0][rows]) and torch.equal(want[1][rows], got[1][rows])
        return
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])


# As many lanes of one block with something to keep as a wavefront keeps records of, one less, one more, and all of them
@pytest.mark.parametrize("many", [4, 15, 16, 17, 31, 64])
@pytest.mark.parametrize("N,d,k", [(4100, 40, 20), (4500, 160, 20), (50_000, 100, 20)])
def test_lanes_of_a_block(lib, many, N, d, k):
    print(f"pairs once, blocks of {many} lanes, N={N} d={d}", flush=True)
    assert lib.probe_knn_products(N, d, k) == 0.5
    X = blobs(N, d, many)
    X = X[torch.arange(N, device="cuda") % (N // many)].contiguous()
    want, got = lib.knn_graph(X, k, fp32_filter=True), lib.knn_graph(X, k)
    torch.cuda.synchronize()
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])


# Rows whose lists overflow are searched for on their own from 128 tiles on, in lists of 1024.  A row has to be met by all copies of its point
# and by all rows beyond float16, whatever its limit.  As many of them as a list holds and more, with the memory for lists of 1024
# (all of the workspace) and of 256 to 384 (40 % of it): none, some or all of the rows left over, in one to several batches; as
# many as the second list holds, and more, which the list kernels finish.  The two largest searches have several bands: more than half of the
# rows overflow before the last of them where all points have copies, and it is left out.
@pytest.mark.parametrize("share", [1.0, 0.4])
@pytest.mark.parametrize("kind,many", [("copies", 400), ("copies", 900), ("copies", 1030), ("copies", 5000), ("two_points", 450), ("all_points", 400), ("all_points", 700),
                                       ("beyond_float16", 400), ("beyond_float16", 1023), ("beyond_float16", 1200), ("both", 400)])
@pytest.mark.parametrize("N,d,k", [(16_257, 160, 12), (20_000, 129, 20), (50_000, 100, 12), (49_030, 65, 7), (150_000, 80, 12), (60_000, 300, 12)])
def test_rows_left_over(lib, kind, many, N, d, k, share):
    print(f"pairs once, rows left over, {many} {kind}, N={N} d={d} k={k}, {share} of the workspace", flush=True)
    assert lib.probe_knn_products(N, d, k) == 0.5 and 12 * (k + 1) <= 256
    X = blobs(N, d, many)
    at = torch.randperm(N, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    if kind in ("copies", "both"):
        X[at[:many]] = X[at[0]].clone()
    if kind == "two_points":
        X[at[:many]] = X[at[0]].clone()
        X[at[many:2 * many]] = X[at[many]].clone()
    if kind == "all_points":
        X = X[at % (N // many)].contiguous()
    if kind in ("beyond_float16", "both"):
        X[at[-many:]] *= 1e7
    workspace = torch.empty(int(lib.knn_workspace_bytes(N, d, k) * share), dtype=torch.uint8, device="cuda")
    want, got = lib.knn_graph(X, k, fp32_filter=True), lib.knn_graph(X, k, workspace=workspace)
    torch.cuda.synchronize()
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])


def least_ms(call):
    least = float("inf")
    for _ in range(6):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        out = call()
        end.record()
        end.synchronize()
        least = min(least, begin.elapsed_time(end))
    return out, least


# Every point 300 times: lists that hold 300 rows for k = 12, in two to three and a half times the time of a search without copies (6 to 20 times where rows
# overflowed lists of 256)
@pytest.mark.parametrize("N,d", [(5000, 200), (12_800, 48), (60_000, 128), (100_000, 400)])
def test_time_of_copies(lib, N, d):
    print(f"pairs once, copies, N={N} d={d}", flush=True)
    X = blobs(N, d, N)
    copies = X[torch.arange(N, device="cuda") % (N // 300)].contiguous()
    workspace = torch.empty(lib.knn_workspace_bytes(N, d, 12), dtype=torch.uint8, device="cuda")
    ms, ms_copies = (least_ms(lambda: lib.knn_graph(rows, 12, workspace=workspace))[1] for rows in (X, copies))
    assert ms_copies < 5 * ms, (ms_copies, ms)


# Rows in the order of their clusters, one of every cluster in turn, rows along a path: the same lists as in no order, in about the same time
# (up to 60 times as long where the places of the rows in the copy went by their numbers alone)
@pytest.mark.parametrize("kind", ["in_order", "in_turn", "path"])
@pytest.mark.parametrize("N,d,k", [(12_800, 48, 12), (25_000, 160, 12), (60_000, 128, 12), (60_000, 128, 50), (150_000, 80, 50)])
def test_rows_in_some_order(lib, kind, N, d, k):
    print(f"pairs once, rows {kind}, N={N} d={d} k={k}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N)
    row = torch.arange(N, device="cuda")
    X = torch.randn((N, d), generator=g, device="cuda")
    if kind == "path":
        X += torch.cumsum(0.1 * torch.randn((N, d), generator=g, device="cuda"), 0)
    else:
        clusters = N // 500 if kind == "in_order" else 50
        centres = (2 * torch.rand((clusters, d), generator=g, device="cuda") - 1) * 20
        X += centres[row * clusters // N if kind == "in_order" else row % clusters]
    order = torch.randperm(N, generator=g, device="cuda")
    workspace = torch.empty(lib.knn_workspace_bytes(N, d, k), dtype=torch.uint8, device="cuda")

    search = lambda rows: least_ms(lambda: lib.knn_graph(rows, k, workspace=workspace))
    got, ms = search(X)
    shuffled, ms_shuffled = search(X[order].contiguous())
    assert torch.equal(got[1][order], shuffled[1])
    assert (got[0][order] == order[shuffled[0].long()]).float().mean() > 0.999          # (else: ties)
    assert ms < 1.6 * ms_shuffled, (ms, ms_shuffled)


# the first connection round asks for most rows; few and many components, copies, a far row
@pytest.mark.parametrize("kind", ["clusters", "pairs", "copies", "far_row"])
@pytest.mark.parametrize("N,d", [(4097, 130), (6000, 256), (20_001, 300)])
def test_trees(lib, kind, N, d):
    print(f"pairs once, trees, {kind}, N={N} d={d}", flush=True)
    X = blobs(N, d, N, spread=30.0, rows=N // 8 if kind != "pairs" else 3)
    if kind == "copies":
        X = X[torch.arange(N, device="cuda") // 30].contiguous()
    if kind == "far_row":
        X[N // 3] *= 1e5
    want, got = lib.slhc(X, 4, prune=False, fp32_filter=True), lib.slhc(X, 4, prune=False)
    torch.cuda.synchronize()
    for key in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(want[key], got[key]), key
