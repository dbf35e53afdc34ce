"""Entries that only one of the two rows has, spread over graphs of more workgroups than run at once (csr_kernels.hip): some workgroups report them while
others of the same launch start, and every workgroup either takes part in its barriers as a whole or leaves as a whole.  An error, never a forest, and
the next call is right."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rows(V, a, b, w):
    order = np.argsort(a, kind="stable")
    offsets = np.r_[0, np.cumsum(np.bincount(a, minlength=V))].astype(np.int32)
    return offsets, b[order].astype(np.int32), w[order].astype(np.float32)


def path(V):
    a, w = np.arange(V - 1), (np.arange(V - 1) % 7 + 1).astype(np.float32)
    return rows(V, np.r_[a, a + 1], np.r_[a + 1, a], np.r_[w, w])


# round 0 for four vertices a thread (beyond 131 072 vertices), and for one; the rounds without lists and the one behind them, whose edges are one-sided
# where a component's lightest edge out of it is
@pytest.mark.parametrize("V", [131_073, 140_000, 700_000, 3_000_000])
@pytest.mark.parametrize("kind", ["lightest, few", "lightest, many", "last vertices", "between pairs", "between fours"])
def test_one_sided_in_large_graphs(V, kind):
    import paper_2306_16354_amd as slhc
    print(f"csr one-sided V={V}, {kind}", flush=True)
    rng = np.random.default_rng(V)
    offsets, indices, weights = path(V)
    src = np.repeat(np.arange(V), np.diff(offsets))
    if kind in ("between pairs", "between fours"):                 # components of two (four) vertices first, one-sided edges between those
        n = 2 if kind == "between pairs" else 4
        a = np.arange(V - 1)[np.arange(V - 1) % n != n - 1]
        w = 1.0 + a % n % 2
        offsets, indices, weights = rows(V, np.r_[a, a + 1], np.r_[a + 1, a], np.r_[w, w].astype(np.float32))
        src = np.repeat(np.arange(V), np.diff(offsets))
        x = rng.permutation(V // n - 2)[:V // 50] * n
        y, v = x + n + 1, np.full(len(x), 3.0)
    else:
        x = {"lightest, few": rng.permutation(V - 9)[:3], "lightest, many": rng.permutation(V - 9)[:V // 3], "last vertices": np.arange(V - 4000, V - 9)}[kind]
        y, v = x + 5, np.full(len(x), 0.25)
    offsets, indices, weights = rows(V, np.r_[src, x], np.r_[indices, y], np.r_[weights, v].astype(np.float32))
    graph = [torch.from_numpy(t).cuda() for t in (offsets, indices, weights)]
    for _ in range(3):
        with pytest.raises(slhc.SlhcError, match="both rows"):
            slhc.csr_msf(*graph)
    offsets, indices, weights = path(V)
    got = slhc.csr_msf(*[torch.from_numpy(t).cuda() for t in (offsets, indices, weights)])
    order = np.argsort(np.arange(V - 1) % 7, kind="stable")
    assert np.array_equal(got["mst_src"].cpu().numpy(), order) and np.array_equal(got["mst_dst"].cpu().numpy(), order + 1)
