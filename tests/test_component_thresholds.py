"""Connection sweeps in the row order: components that lower their shared threshold as they are searched, and the evaluation of 32 queued
pairs at a time, against the sweeps of every tile, bit for bit."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2306_16354_amd as slhc
    slhc.load_library()
    assert torch.cuda.is_available()
    return slhc


# one row below and at the size from which small components lower theirs; up to 64 columns (a pass of 32 pairs) and beyond; clusters many
# radii apart (every row of one passes at first), overlapping ones, pairs of rows, and rows of few values (ties between clusters)
@pytest.mark.parametrize("N,d,k,rows,spread,steps", [
    (131_071, 32, 6, 100, 1000.0, 0), (131_072, 32, 6, 100, 1000.0, 0), (131_072, 4, 3, 40, 50.0, 0), (140_000, 64, 4, 60, 1000.0, 0),
    (140_000, 68, 4, 60, 1000.0, 0), (133_333, 24, 1, 2, 100.0, 0), (150_000, 8, 2, 300, 20.0, 4), (20_000, 64, 3, 50, 1000.0, 0), (5000, 36, 2, 7, 30.0, 2),
])
def test_trees(lib, N, d, k, rows, spread, steps):
    print(f"component thresholds N={N} d={d} k={k} rows={rows}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N + d)
    centres = (2 * torch.rand((N // rows, d), generator=g, device="cuda") - 1) * spread
    X = centres[torch.randint(len(centres), (N,), generator=g, device="cuda")] + torch.randn((N, d), generator=g, device="cuda")
    if steps:
        X = (X * steps).round() / steps
    want, got = lib.slhc(X, k, prune=False), lib.slhc(X, k, prune=True)
    assert got["stats"]["pruned"] == 1
    for name in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(want[name], got[name]), name
