"""The dendrogram on the device (dendrogram_kernels.hip): from 19 000 rows on, with levels in one workgroup from 4096 vertices down and
sums along chains in one workgroup for the last 8192 merges.  Children and sizes are whole numbers and follow from the sorted edges alone, so they
have to equal the oracle's sequential relabelling of the same edges."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rows(kind, N, rng):
    X = np.zeros((N, 4), np.float64)
    if kind == "rising":             # one chain: every merge adds the next row
        X[:, 0] = np.arange(N) ** 1.5
    elif kind == "rising, shuffled":
        X[:, 0] = rng.permutation(N) ** 1.5
    elif kind == "lattice":          # all gaps equal: order by row number alone
        X[:, 0] = np.arange(N)
    elif kind == "doubling":         # gaps 1, 2, 1, 4, 1, 2, 1, 8, ..: a level per doubling, all merges between chains
        X[1:, 0] = np.cumsum(np.arange(1, N) & -np.arange(1, N))
    elif kind == "copies":           # most merges at distance 0
        X[:] = rng.integers(0, 40, size=(N, 4))
    else:                            # clusters of 3 .. 300 rows
        centre = rng.uniform(-100, 100, size=(N // 60, 4))
        X[:] = centre[np.minimum(rng.integers(0, N // 60, N), rng.integers(0, N // 60, N))] + 0.3 * rng.standard_normal((N, 4))
    return X.astype(np.float32)


@pytest.mark.parametrize("N", [18_999, 19_000, 20_481, 65_537])
@pytest.mark.parametrize("kind", ["rising", "rising, shuffled", "lattice", "doubling", "copies", "clusters"])
def test_children_and_sizes(N, kind):
    import paper_2306_16354_amd as slhc
    print(f"dendrogram N={N} {kind}", flush=True)
    X = rows(kind, N, np.random.default_rng(N))
    out = slhc.slhc(torch.from_numpy(X).cuda(), 6)
    src, dst, w = (out[n].cpu().numpy() for n in ("mst_src", "mst_dst", "mst_w"))
    want = oracle.dendrogram(src, dst, w.astype(np.float64), N)
    assert np.array_equal(out["children"].cpu().numpy(), want["children"])
    assert np.array_equal(out["sizes"].cpu().numpy(), want["sizes"])


# arrays that begin at any word; the host's dendrogram and the device's
@pytest.mark.parametrize("N", [600, 18_999, 19_000, 40_000])
@pytest.mark.parametrize("word", [1, 3])
def test_arrays_at_odd_words(N, word):
    import paper_2306_16354_amd as slhc
    print(f"dendrogram into arrays at odd words N={N} word={word}", flush=True)
    X = torch.from_numpy(rows("clusters", N, np.random.default_rng(N))).cuda()
    want = slhc.slhc(X, 6)
    types = {"mst_src": torch.int32, "mst_dst": torch.int32, "mst_w": torch.float32, "children": torch.int32, "heights": torch.float32, "sizes": torch.int32}
    whole = {n: torch.full((2 * N + 8,), -7, dtype=t, device="cuda") for n, t in types.items()}
    out = {n: t[word:word + want[n].numel()].view(want[n].shape) for n, t in whole.items()}
    got = slhc.slhc(X, 6, out=out)
    for n in types:
        assert torch.equal(got[n], want[n]) and bool((whole[n][:word] == -7).all()) and bool((whole[n][word + want[n].numel():] == -7).all()), n


# one chain of more merges than 64 workgroups sum up: what comes before a span is looked for beyond the 64 spans before it
@pytest.mark.parametrize("kind,N", [("rising", 200_000), ("rising, shuffled", 300_001), ("doubling", 200_000)])
def test_long_chains(kind, N):
    test_children_and_sizes(N, kind)
