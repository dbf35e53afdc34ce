"""Flat clusters of more rows than one workgroup takes (cluster_kernels.hip): walks thinned by stages, roots counted in spans."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2306_16354_amd as slhc
    slhc.load_library()
    return slhc


def cut(children, N, kept):
    """The root of every row after `kept` merges, from the last of them down, and its number by ascending node id."""
    top = list(range(N + kept))
    for i in range(kept - 1, -1, -1):
        a, b = children[i]
        top[a] = top[b] = top[N + i]
    return np.unique(np.array(top[:N]), return_inverse=True)[1]


# rows and merges that end inside and at the end of a group, a wide load and a span; one and two turns per span
@pytest.mark.parametrize("N", [8193, 12_289, 65_536, 65_552, 131_073, 1_048_576 + 17])
def test_chains_side_by_side(lib, N):
    """Three chains that take their merges in turn, then joined: every third merge leads to the third after it."""
    third = N // 3
    starts = [0, third, 2 * third]
    ends = [third, 2 * third, N]
    children, last, at = [], list(starts), [s + 1 for s in starts]
    for i in range(N - 3):
        c = i % 3
        while at[c] >= ends[c]: c = (c + 1) % 3
        children.append((min(last[c], at[c]), max(last[c], at[c])))
        last[c] = N + i
        at[c] += 1
    children.append((min(last[:2]), max(last[:2])))
    children.append((min(last[2], 2 * N - 3), max(last[2], 2 * N - 3)))
    dev = torch.tensor(children, dtype=torch.int32, device="cuda")
    for kept in (1, 8, 255, 1025, 4097, N // 2, N - 4, N - 3, N - 2, N - 1) if N < 200_000 else (N // 2, N - 3, N - 1):
        print(f"chains side by side N={N} kept={kept}", flush=True)
        assert np.array_equal(lib.flat_clusters(dev, N - kept).cpu().numpy(), cut(children, N, kept)), kept


@pytest.mark.parametrize("N", [5_000_000, 34_000_001])
def test_long_chain(lib, N):
    """One chain: after `kept` merges the rows up to row `kept` are one cluster, numbered last.  The larger has a fourth stage."""
    children = torch.empty((N - 1, 2), dtype=torch.int32, device="cuda")
    children[:, 0] = torch.arange(N - 1, device="cuda") + (N - 1)
    children[0, 0] = 0
    children[:, 1] = torch.arange(1, N, device="cuda")
    for kept in (3, N // 2, N - 1):
        print(f"long chain N={N} kept={kept}", flush=True)
        want = torch.arange(N, device="cuda", dtype=torch.int32) - (kept + 1)
        want[:kept + 1] = N - kept - 1
        assert torch.equal(lib.flat_clusters(children, N - kept), want), kept


@pytest.mark.parametrize("N", [8193, 20_000])
def test_arrays_at_odd_words(lib, N):
    """Children and labels that start at any word."""
    children = np.stack([np.r_[0, N + np.arange(N - 2)], np.arange(1, N)], 1).astype(np.int32)
    dev = torch.empty(2 * N - 1, dtype=torch.int32, device="cuda")[1:].view(N - 1, 2)
    dev.copy_(torch.from_numpy(children))
    out = torch.empty(N + 1, dtype=torch.int32, device="cuda")[1:]
    lib.flat_clusters(dev, 100, out=out)
    assert np.array_equal(out.cpu().numpy(), cut(children.tolist(), N, N - 100))
