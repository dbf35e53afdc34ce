"""Minimum spanning forests and flat clusters where their small-input kernels end and where chains are longest."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2306_16354_amd as slhc
    slhc.load_library()
    assert torch.cuda.is_available()
    return slhc


# a path: with rising weights every vertex hooks onto its predecessor in round one (one chain of N - 1 links); with weights
# in random order there are many rounds.  Sizes: one-workgroup forests and the single-key edge sort end inside these.
@pytest.mark.parametrize("rising", [True, False])
@pytest.mark.parametrize("N", [2, 1000, 12_288, 12_289, 65_536, 65_537])
def test_forest_of_a_path(lib, N, rising):
    print(f"path forest N={N} rising={rising}", flush=True)
    w = np.arange(1, N, dtype=np.float32)
    if not rising:
        np.random.default_rng(N).shuffle(w)
    a = np.arange(N - 1)
    src, dst, ww = np.r_[a, a + 1], np.r_[a + 1, a], np.r_[w, w]
    order = np.lexsort((dst, src))
    offsets = np.r_[0, np.cumsum(np.bincount(src, minlength=N))].astype(np.int32)
    got = lib.csr_msf(torch.from_numpy(offsets).cuda(), torch.from_numpy(dst[order].astype(np.int32)).cuda(),
                      torch.from_numpy(ww[order]).cuda())
    torch.cuda.synchronize()
    by_weight = np.argsort(w, kind="stable")
    assert np.array_equal(got["mst_w"].cpu().numpy(), w[by_weight])
    assert np.array_equal(got["mst_src"].cpu().numpy(), by_weight)
    assert np.array_equal(got["mst_dst"].cpu().numpy(), by_weight + 1)


# forests whose rounds run in one workgroup: one to twelve vertices a thread, lists shorter than a load of four entries and of every
# remainder, clusters smaller than the lists (walked to their end, several rounds of queries) and larger, rows at equal distances
@pytest.mark.parametrize("N,k", [(2, 1), (5, 3), (600, 1), (1023, 2), (1025, 3), (4096, 4), (4097, 5), (8192, 7), (8193, 18), (12_288, 6), (12_289, 6)])
@pytest.mark.parametrize("rows_per_cluster", [3, 300])
def test_forest_of_points(lib, N, k, rows_per_cluster):
    print(f"forest of points N={N} k={k} clusters of {rows_per_cluster}", flush=True)
    rng = np.random.default_rng(N + k)
    centres = rng.integers(-50, 50, size=(max(1, N // rows_per_cluster), 3))
    X = (centres[rng.integers(0, len(centres), N)] + rng.integers(0, 8, size=(N, 3)) / 16).astype(np.float32)
    out = lib.slhc(torch.from_numpy(X).cuda(), k)
    torch.cuda.synchronize()
    ref = oracle.slhc(X)
    # (distances of such points are exact in float32, so the weights are)
    assert np.array_equal(np.sort(out["mst_w"].cpu().numpy()).astype(np.float64), np.sort(np.asarray(ref["heights"], dtype=np.float64)))
    lo, hi = out["mst_src"].cpu().numpy(), out["mst_dst"].cpu().numpy()
    assert np.array_equal(((X[lo].astype(np.float64) - X[hi]) ** 2).sum(1), out["mst_w"].cpu().numpy())


def cuts(N):
    return sorted({k for k in (0, 1, 2, 7, 8, 9, 63, 64, 65, 512, 4096, N // 2, N - 2, N - 1) if 0 <= k < N})


# one chain of N - 1 merges, row i joining rows 0 .. i - 1: after `kept` merges those up to row `kept` are one cluster, which
# is numbered last, and every other row is its own.  Cuts at a power of the links followed per pass and its neighbours.
@pytest.mark.parametrize("N", [2, 65, 1025, 8191, 8192, 8193, 40_000, 300_000])
def test_cuts_of_a_chain(lib, N):
    children = np.stack([np.r_[0, N + np.arange(N - 2)], np.arange(1, N)], 1).astype(np.int32)
    dev = torch.from_numpy(children).cuda()
    for kept in cuts(N):
        print(f"cut chain N={N} kept={kept}", flush=True)
        want = np.arange(N) - kept - 1
        want[:kept + 1] = N - kept - 1
        if kept == 0:
            want = np.arange(N)
        if N <= 1025:
            assert np.array_equal(want, oracle.flat_clusters(children, N - kept))
        assert np.array_equal(lib.flat_clusters(dev, N - kept).cpu().numpy(), want), kept


@pytest.mark.parametrize("N", [3, 1000, 8192, 8193, 40_000])
def test_cuts_of_random_joins(lib, N):
    rng = np.random.default_rng(N)
    children = np.empty((N - 1, 2), np.int32)
    alive = list(range(N))
    for i in range(N - 1):
        for side in (0, 1):
            j = int(rng.integers(len(alive)))
            alive[j], alive[-1] = alive[-1], alive[j]
            children[i, side] = alive.pop()
        alive.append(N + i)
    dev = torch.from_numpy(children).cuda()
    for kept in cuts(N):
        print(f"cut joins N={N} kept={kept}", flush=True)
        assert np.array_equal(lib.flat_clusters(dev, N - kept).cpu().numpy(), oracle.flat_clusters(children, N - kept)), kept
