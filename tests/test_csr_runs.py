"""The two sorts of a spanning forest's edges and the rounds without lists (csr_kernels.hip), against the oracle's Kruskal: runs of equal weights
about the longest one that is ordered in place, and vertices without edges about the line from which the first rounds go over all of them."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def check(V, a, b, w):
    import paper_2306_16354_amd as slhc
    src, dst, ww = np.r_[a, b], np.r_[b, a], np.r_[w, w].astype(np.float32)
    order = np.argsort(src, kind="stable")
    offsets = np.r_[0, np.cumsum(np.bincount(src, minlength=V))].astype(np.int32)
    indices, weights = dst[order].astype(np.int32), ww[order]
    lo, hi, want_w, _ = oracle.csr_msf(offsets, indices, weights)
    graph = [torch.from_numpy(x).cuda() for x in (offsets, indices, weights)]
    for _ in range(2):                     # the second in memory that the first has used
        got = slhc.csr_msf(*graph)
        torch.cuda.synchronize()
        assert np.array_equal(got["mst_src"].cpu().numpy(), lo) and np.array_equal(got["mst_dst"].cpu().numpy(), hi)
        assert np.array_equal(got["mst_w"].cpu().numpy(), np.abs(want_w.astype(np.float32)))
        c = got["colours"].cpu().numpy()
        assert len(np.unique(c)) == V - len(lo) and np.array_equal(c[lo], c[hi])


# `run` edges of one weight among others that differ: the lightest, the heaviest, or between
@pytest.mark.parametrize("run", [2, 63, 64, 65, 200])
@pytest.mark.parametrize("where", ["first", "last", "between"])
def test_runs(run, where):
    V = 70_001
    print(f"csr run of {run} equal weights, {where}", flush=True)
    rng = np.random.default_rng(run)
    ends = rng.permutation(V)
    w = rng.permutation(V - 1).astype(np.float32) + 1
    at = np.argsort(w)
    pick = {"first": at[:run], "last": at[-run:], "between": at[1000:1000 + run]}[where]
    w[pick] = {"first": 0.0, "last": w.max(), "between": w[pick[0]]}[where]
    w[pick[: run // 2]] *= np.float32(-1 if where == "first" else 1)       # (-0 is 0)
    check(V, ends[:-1], ends[1:], w)


@pytest.mark.parametrize("V", [131_072, 131_073, 140_001])
@pytest.mark.parametrize("part", [0.001, 0.5, 1.0])        # of the vertices that have edges
@pytest.mark.parametrize("values", [3, 30_000, 1 << 24])
def test_vertices_without_edges(V, part, values):
    print(f"csr V={V}, {part} with edges, {values} weights", flush=True)
    rng = np.random.default_rng(V)
    some = rng.permutation(V)[:max(2, int(part * V))]
    m = len(some)
    a, b = some[rng.integers(0, m, 2 * m)], some[rng.integers(0, m, 2 * m)]
    pairs = np.unique(np.c_[np.minimum(a, b), np.maximum(a, b)][a != b], axis=0)
    check(V, pairs[:, 0], pairs[:, 1], rng.integers(0, values, len(pairs)).astype(np.float32))
