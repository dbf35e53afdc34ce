"""Exact distances and selection (near_kernels.hip) by how rows are read: quads at aligned addresses, quads at any word from 64 columns on, words below; rows and
matrices that begin at any word; few and many candidates per row.  Lists against the float32-product list kernels, bit for bit."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 9, 64])
@pytest.mark.parametrize("offset", [0, 1, 2])
@pytest.mark.parametrize("d", [3, 62, 63, 64, 65, 67, 127, 128, 129, 131, 258])
def test_rows_at_any_word(d, offset, k):
    import paper_2306_16354_amd as slhc
    print(f"rows at any word d={d} offset={offset} k={k}", flush=True)
    N = 4700
    g = torch.Generator(device="cuda").manual_seed(d + k)
    X = torch.empty(N * d + offset, device="cuda")[offset:].view(N, d)
    centre = 8 * torch.randn((12, d), generator=g, device="cuda")
    X.copy_(centre[torch.randint(12, (N,), generator=g, device="cuda")] + torch.randn((N, d), generator=g, device="cuda"))
    want, got = slhc.knn_graph(X.clone(), k, fp32_filter=True), slhc.knn_graph(X, k)
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])
    # nearest rows of another matrix: a float32 sum of d squares is off by (d + 2) 2^-24 of its value at most, on either side
    best = torch.cdist(X[:50].double().cpu(), X[50:].double().cpu()).square().min(1).values
    got = slhc.fused_1nn(X[:50], X[50:])[1].double().cpu()
    assert torch.allclose(got, best, rtol=2 * (d + 2) * 2.0 ** -24, atol=1e-9)


# nearest rows of another matrix and of another colour on both sides of the line up to which every pair is evaluated: twelve queries whatever the candidates are,
# and so many more as are 240 million operations
@pytest.mark.parametrize("n,d,more", [(300_000, 30, 11), (65_537, 64, 26), (20_000, 16, 272), (200_001, 5, 54)])
def test_few_queries_in_many_rows(n, d, more):
    import paper_2306_16354_amd as slhc
    assert more * n * (2 * d + 12) <= 240_000_000 < (more + 1) * n * (2 * d + 12)
    g = torch.Generator(device="cuda").manual_seed(n)
    Y = 20 * torch.randn((n, d), generator=g, device="cuda")
    Q = Y[torch.randint(n, (13 + more,), generator=g, device="cuda")] + torch.randn((13 + more, d), generator=g, device="cuda")
    colour = torch.randint(3, (n,), dtype=torch.int32, generator=g, device="cuda")
    rows = torch.randperm(n, generator=g, device="cuda")[:13 + more].to(torch.int32)
    for m in (12, 13, 12 + more, 13 + more):
        print(f"few queries in many rows m={m} n={n} d={d}", flush=True)
        D = torch.cdist(Q[:m].double(), Y.double()).square()
        idx, dist = slhc.fused_1nn(Q[:m], Y)
        assert torch.allclose(dist.double(), D.min(1).values, rtol=1e-5, atol=0) and torch.equal(idx.long(), D.argmin(1))
        D = torch.cdist(Y[rows[:m].long()].double(), Y.double()).square()
        D[colour[rows[:m].long(), None] == colour[None, :]] = float("inf")
        idx, dist = slhc.cross_1nn(Y, colour, rows=rows[:m])
        assert torch.allclose(dist.double(), D.min(1).values, rtol=1e-5, atol=0) and torch.equal(idx.long(), D.argmin(1))
