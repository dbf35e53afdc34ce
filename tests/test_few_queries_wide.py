"""Nearest rows of few queries where every pair is evaluated (direct_1nn): workgroups of four slabs of 64 candidates, so of one to four steps by the rows' width."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def distances(A, B):
    """In 64 bits, every pair's sum in the same order, so that copies of a row are as far as the row itself."""
    a, b = A.double().cpu().numpy(), B.double().cpu().numpy()
    return torch.from_numpy(np.stack([((x - b) ** 2).sum(1) for x in a])).cuda()


def first_least(D):
    """The first column of the least value (torch's argmin may name any of them)."""
    return torch.from_numpy(D.cpu().numpy().argmin(1)).cuda()


# one slab to five of a row; candidates about the ends of a step and of a share
@pytest.mark.parametrize("d", [64, 65, 128, 129, 192, 193, 256, 300, 1025])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 129, 255, 257, 1000])
def test_shares_meet_at_a_row(d, n):
    import paper_2306_16354_amd as slhc
    print(f"shares meet d={d} n={n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(d + n)
    Y = torch.randn((n, d), generator=g, device="cuda")
    Y[n // 2:] = Y[:n - n // 2].clone()                              # a row and its copy in another share: the first one counts
    Q = Y[torch.randint(n, (21,), generator=g, device="cuda")] + 0.1 * torch.randn((21, d), generator=g, device="cuda")
    D = distances(Q, Y)
    colour = torch.randint(3, (n,), dtype=torch.int32, generator=g, device="cuda")
    idx, dist = slhc.fused_1nn(Q, Y)
    # (a float32 sum of d squares is off by (d + 2) 2^-24 of its value at most)
    assert torch.equal(idx.long(), first_least(D)) and torch.allclose(dist.double(), D.min(1).values, rtol=(d + 2) * 2.0 ** -24, atol=0)
    if n < 2: return                                                 # (a search by colours takes two rows and more)
    rows = torch.randint(n, (9,), dtype=torch.int32, generator=g, device="cuda")
    D = distances(Y[rows.long()], Y)
    D[colour[rows.long(), None] == colour[None]] = float("inf")
    idx, dist = slhc.cross_1nn(Y, colour, rows=rows)
    none = D.min(1).values == float("inf")
    assert torch.equal(idx.long(), torch.where(none, -1, first_least(D))) and torch.allclose(dist.double(), D.min(1).values, rtol=(d + 2) * 2.0 ** -24, atol=0)


def least_us(f):
    f()
    least = float("inf")
    for _ in range(10):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        for _ in range(5): f()
        end.record()
        end.synchronize()
        least = min(least, begin.elapsed_time(end) * 200)
    return least


# some queries, and a few more, which the half-precision engine searches for: 57 and 105 us, 137 and 220, 596 and 1672 (202, 581 and 2683 of the first with
# shares of at least four steps)
@pytest.mark.parametrize("m,more,n,d", [(16, 48, 10_000, 784), (12, 24, 10_000, 2000), (12, 20, 10_000, 8000)])
def test_wide_rows_of_few_candidates(m, more, n, d):
    import paper_2306_16354_amd as slhc
    Y = torch.randn((n, d), device="cuda")
    Q = torch.randn((more, d), device="cuda")
    few, many = (least_us(lambda q=Q[:c].contiguous(): slhc.fused_1nn(q, Y)) for c in (m, more))
    print(f"{m} and {more} x {n} x {d}: {few:.0f} and {many:.0f} us", flush=True)
    assert few < many
