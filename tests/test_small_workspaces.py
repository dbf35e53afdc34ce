"""Calls whose workspace is smaller than the size functions report: the half-precision engine in smaller batches, and, where it
does not fit at all, the list kernels.  Same outputs, bit for bit, and the list kernels' against the oracle."""
import ctypes

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
from workspaces import cross_1nn_in, least_bytes, scratch  # noqa: E402

pytestmark = pytest.mark.gpu

TREE = ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes")


@pytest.fixture(scope="module")
def lib():
    import paper_2306_16354_amd as slhc
    slhc.load_library()
    assert torch.cuda.is_available()
    return slhc


def same_for_all_sizes(lib, call, full, between=(0.1, 0.5)):
    """call(workspace) -> tensors.  Least, a share of the way to the full size, full, and one byte too few."""
    least = least_bytes(lib, call)
    assert least < full
    want = None
    for nbytes in [full] + [int(least + f * (full - least)) // 256 * 256 for f in between] + [least]:
        ws, guard = scratch(nbytes)
        got = [t.clone() for t in call(ws)]
        torch.cuda.synchronize()
        assert (guard == 0x5a).all()
        print(f"  {nbytes} bytes of {full}", flush=True)
        if want is None:
            want = got
        for a, b in zip(want, got):
            assert torch.equal(a, b), nbytes
    with pytest.raises(lib.SlhcError):
        call(scratch(least - 1)[0])
    return want


def blobs(N, d, seed, clusters=None, spread=20.0):
    rng = np.random.default_rng(seed)
    centres = rng.uniform(-spread, spread, size=(clusters or max(2, N // 500), d))
    X = (centres[rng.integers(0, len(centres), N)] + rng.standard_normal((N, d))).astype(np.float32)
    X[rng.integers(0, N, N // 50)] = X[rng.integers(0, N, N // 50)]
    return X


# list kernels by size: candidate ranges, one panel per item, ranges carried through the outputs (from 262 144 rows on), the
# streaming kernel; products from split bfloat16 halves wherever the width allows them.  The engine in batches of one panel and
# of several.
@pytest.mark.parametrize("N,d,k", [(2, 1, 1), (3000, 64, 16), (9000, 100, 33), (40_000, 128, 64), (270_000, 64, 8), (263_000, 30, 5),
                                   (5000, 200, 7), (66_500, 132, 20), (5000, 131, 64)])
def test_knn_lists(lib, N, d, k):
    print(f"k-NN in small workspaces N={N} d={d} k={k}", flush=True)
    X = blobs(N, d, N + d)
    Xd = torch.from_numpy(X).cuda()
    idx, dist = same_for_all_sizes(lib, lambda ws: lib.knn_graph(Xd, k, workspace=ws), lib.knn_workspace_bytes(N, d, k), (0.02, 0.5))
    fp = lib.knn_graph(Xd, k, fp32_filter=True)
    assert torch.equal(fp[0], idx) and torch.equal(fp[1], dist)
    rows = np.random.default_rng(N).choice(N, size=min(N, 96), replace=False)
    oi, od = oracle.knn_rows(X, rows, k)
    assert np.allclose(dist.cpu().numpy()[rows], od, rtol=1e-5, atol=1e-30)


@pytest.mark.parametrize("N,d,k", [(700, 4, 3), (30_000, 50, 16), (60_000, 128, 32)])
def test_pruned_knn_lists(lib, N, d, k):
    print(f"pruned k-NN in small workspaces N={N} d={d} k={k}", flush=True)
    Xd = torch.from_numpy(blobs(N, d, N + d, clusters=max(2, N // 3000))).cuda()
    same_for_all_sizes(lib, lambda ws: lib.knn_graph(Xd, k, workspace=ws, prune=True), lib.knn_workspace_bytes(N, d, k))


# with and without a row order, one workgroup's forests and larger ones, components that have to be connected
@pytest.mark.parametrize("N,d,k", [(2, 3, 1), (600, 4, 3), (6000, 32, 8), (20_000, 96, 5), (30_000, 16, 8), (70_000, 128, 16), (8000, 300, 6)])
def test_trees(lib, N, d, k):
    print(f"trees in small workspaces N={N} d={d} k={k}", flush=True)
    Xd = torch.from_numpy(blobs(N, d, N + d, clusters=max(1, N // 4000), spread=60.0)).cuda()

    def call(ws):
        out = lib.slhc(Xd, k, workspace=ws, prune=None)
        return [out[key] for key in TREE]
    same_for_all_sizes(lib, call, lib.slhc_workspace_bytes(N, d, k))


# the list kernels in one launch and in segments (few queries), the engine in one batch and several
@pytest.mark.parametrize("m,n,d", [(1000, 60_000, 64), (20_000, 9000, 128), (40, 300_000, 30), (3000, 20_000, 257), (3, 400_000, 128)])
def test_nearest_rows_of_another_matrix(lib, m, n, d):
    print(f"1-NN in small workspaces m={m} n={n} d={d}", flush=True)
    Y = blobs(n, d, n)
    Q = np.concatenate([blobs(m, d, m)[: m - 1], Y[n // 2:n // 2 + 1]])
    Qd, Yd = torch.from_numpy(Q).cuda(), torch.from_numpy(Y).cuda()
    out = ctypes.c_size_t(0)
    assert lib.load_library().slhc_fused_1nn_workspace_bytes(m, n, d, ctypes.byref(out)) == 0
    idx, dist = same_for_all_sizes(lib, lambda ws: lib.fused_1nn(Qd, Yd, workspace=ws), out.value)
    take = np.unique(np.r_[m - 1, np.random.default_rng(m).integers(0, m, 20)])
    oi, od = oracle.cross_1nn(np.concatenate([Q, Y]), np.r_[np.zeros(m, np.int32), np.ones(n, np.int32)], take.astype(np.int64))
    assert np.allclose(dist.cpu().numpy()[take], od, rtol=1e-5, atol=1e-30)
    assert (idx.cpu().numpy()[take] == oi - m).mean() >= 0.9


# all rows, listed rows, and searches small enough to evaluate every pair, on both sides of the lines where these end (100 and 200
# million operations, 65 536 candidates)
@pytest.mark.parametrize("N,d,m,listed", [(30_000, 64, 30_000, False), (60_000, 33, 5000, True), (20_000, 200, 900, True), (1500, 8, 1400, True),
                                          (60_000, 14, 82, True), (60_000, 14, 86, True), (65_536, 12, 45, True), (65_537, 12, 45, True),
                                          (9000, 250, 42, True)])
def test_nearest_rows_of_another_colour(lib, N, d, m, listed):
    print(f"1-NN by colours in small workspaces N={N} d={d} m={m}", flush=True)
    rng = np.random.default_rng(N)
    X = blobs(N, d, N)
    colour = rng.integers(0, 5, N).astype(np.int32)
    rows = rng.choice(N, m, replace=False).astype(np.int32)
    if listed:
        rows[3], rows[7] = -1, N                            # not rows: answered with nothing
    Xd, cd = torch.from_numpy(X).cuda(), torch.from_numpy(colour).cuda()
    out = ctypes.c_size_t(0)
    assert lib.load_library().slhc_cross_1nn_workspace_bytes(N, d, m, ctypes.byref(out)) == 0
    idx, dist = same_for_all_sizes(lib, cross_1nn_in(lib, Xd, cd, torch.from_numpy(rows).cuda() if listed else None, m), out.value)
    idx, dist = idx.cpu().numpy(), dist.cpu().numpy()
    if listed:
        assert idx[3] == idx[7] == -1 and np.isinf(dist[[3, 7]]).all()
    take = np.arange(10, 40)
    oi, od = oracle.cross_1nn(X, colour, (rows if listed else np.arange(N))[take].astype(np.int64))
    assert np.allclose(dist[take], od, rtol=1e-5, atol=1e-30)


def test_several_batches_of_nearest_row_queries(lib):
    """More queries than one batch holds (131 072): the scratch of a batch is used again by the next, among it the list of
    queries that are left over, which rows with many near neighbours of another colour fill in every batch."""
    rng = np.random.default_rng(5)
    m, n, d = 300_000, 4000, 20
    Y = np.repeat(rng.uniform(-50, 50, size=(n // 40, d)), 40, axis=0) + 1e-4 * rng.standard_normal((n, d))
    Q = Y[rng.integers(0, n, m)] + 1e-4 * rng.standard_normal((m, d))
    Qd, Yd = torch.from_numpy(Q.astype(np.float32)).cuda(), torch.from_numpy(Y.astype(np.float32)).cuda()
    out = ctypes.c_size_t(0)
    assert lib.load_library().slhc_fused_1nn_workspace_bytes(m, n, d, ctypes.byref(out)) == 0
    same_for_all_sizes(lib, lambda ws: lib.fused_1nn(Qd, Yd, workspace=ws), out.value, (0.3,))
    both = torch.cat([Yd, Qd[:200_000]]).contiguous()
    colour = torch.from_numpy(rng.integers(0, 7, n + 200_000).astype(np.int32)).cuda()
    assert lib.load_library().slhc_cross_1nn_workspace_bytes(n + 200_000, d, n + 200_000, ctypes.byref(out)) == 0
    same_for_all_sizes(lib, cross_1nn_in(lib, both, colour, None, n + 200_000), out.value, ())
