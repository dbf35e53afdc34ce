"""Searches of narrow rows among themselves (pairs_kernels.hip): every pair in either order, for the row that asks, or once for both; workgroups of two, four and
twelve wavefronts; with and without the second search for rows whose lists overflow.  Lists against the float32-product list kernels, bit for bit."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2306_16354_amd as slhc
    slhc.load_library()
    return slhc


def check(lib, X, k):
    tiles, steps = -(-X.shape[0] // 128), -(-X.shape[1] // 16)
    assert lib.probe_knn_products(X.shape[0], X.shape[1], k) == (0.5 if steps >= 6 or steps >= 3 and tiles <= 100 or steps == 5 and tiles >= 384 else 1.0)
    want, got = lib.knn_graph(X, k, fp32_filter=True), lib.knn_graph(X, k)
    torch.cuda.synchronize()
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])


def blobs(N, d, seed, rows=300, spread=8.0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    centres = (2 * torch.rand((max(2, N // rows), d), generator=g, device="cuda") - 1) * spread
    return centres[torch.randint(len(centres), (N,), generator=g, device="cuda")] + torch.randn((N, d), generator=g, device="cuda")


# each number of 16-column steps, whole and partial; the largest search of two wavefronts' workgroups and the smallest of four; 100, 101, 255, 256, 383 and 384
# tiles; an odd tile at the end
@pytest.mark.parametrize("N,d,k", [
    (4481, 9, 6), (5000, 4, 5), (5001, 16, 30), (6001, 17, 12), (12_801, 81, 5), (25_000, 79, 40), (49_024, 96, 8), (5761, 32, 64), (5889, 31, 9), (12_801, 3, 10), (12_930, 128, 20), (13_000, 90, 15), (20_011, 50, 10), (32_640, 24, 7),
    (32_641, 65, 7), (33_000, 8, 1), (49_024, 48, 12), (49_025, 48, 12), (49_153, 64, 33), (49_153, 65, 33), (60_000, 16, 64), (150_001, 12, 8),
])
def test_lists(lib, N, d, k):
    print(f"pairs narrow N={N} d={d} k={k}", flush=True)
    check(lib, blobs(N, d, N + d), k)


# more copies of every point than the lists of the search hold, than those of the second one do (which then is left out), rows in the order of their
# clusters, rows whose norms differ by orders of magnitude (most are not told apart by their float16 copies), a lattice (ties at every distance)
@pytest.mark.parametrize("kind", ["copies300", "copies1500", "sorted", "radial", "lattice"])
@pytest.mark.parametrize("N,d,k", [(5000, 12, 12), (20_000, 30, 12), (40_000, 20, 12), (60_000, 100, 12)])
def test_lists_of_unlike_rows(lib, kind, N, d, k):
    print(f"pairs narrow, {kind}, N={N} d={d}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N)
    if kind.startswith("copies"):
        copies = int(kind[6:])
        X = torch.randn((N // copies + 1, d), generator=g, device="cuda").repeat(copies, 1)[:N][torch.randperm(N, generator=g, device="cuda")]
    elif kind == "sorted":
        X = blobs(N, d, 7)
        X = X[torch.argsort(X[:, 0])]
    elif kind == "radial":
        X = torch.randn((N, d), generator=g, device="cuda")
        X = X / X.norm(dim=1, keepdim=True) * torch.rand((N, 1), generator=g, device="cuda") ** 4 * 1000
    else:
        X = torch.randint(0, 3, (N, d), generator=g, device="cuda").float()
    check(lib, X.contiguous(), k)
