"""The half-precision engine (near_kernels.hip) where its tiles, segments, buffers and fallbacks end: its lists against the
float32-product list kernels bit for bit, its nearest rows against the oracle."""
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


def same_lists(lib, X, k):
    Xd = torch.from_numpy(np.ascontiguousarray(X)).cuda()
    a = lib.knn_graph(Xd, k, fp32_filter=True)
    b = lib.knn_graph(Xd, k)
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


# one tile and its edges, the workgroup sizes' edges, one wavefront's 64 queries, 16-column steps, both kernels (128 / 129
# columns), whole and partial chunks of 64, every list width, one- and two-stage plans; the fewest rows of every width that the engine
# sees (the pairs of fewer are all evaluated, in direct_kernels.hip)
@pytest.mark.parametrize("N,d,k", [
    (2, 3, 1), (64, 16, 63), (127, 17, 5), (128, 1, 8), (129, 15, 64), (255, 31, 9), (257, 33, 2), (385, 112, 64),
    (1025, 113, 16), (2047, 127, 33), (3000, 128, 1), (3001, 129, 7), (2500, 192, 64), (2600, 193, 17), (700, 321, 3),
    (8193, 64, 12), (33_000, 48, 40), (40_000, 200, 1), (66_001, 20, 31), (140_000, 130, 16),
    (4480, 8, 64), (3841, 16, 9), (3073, 31, 33), (2689, 48, 2), (2305, 63, 64), (2049, 96, 17), (1793, 112, 5), (1793, 113, 16),
])
def test_lists_at_the_edges(lib, N, d, k):
    print(f"half-precision lists N={N} d={d} k={k}", flush=True)
    rng = np.random.default_rng(N + d)
    centres = rng.uniform(-8, 8, size=(max(2, N // 400), d))
    same_lists(lib, (centres[rng.integers(0, len(centres), N)] + rng.standard_normal((N, d))).astype(np.float32), k)


@pytest.mark.parametrize("kind", ["one_point", "few_points", "far_rows", "beyond_float16", "sorted", "one_column"])
@pytest.mark.parametrize("d", [24, 150])
def test_lists_that_overflow_or_leave_float16(lib, kind, d):
    """Masses of ties fill every buffer and go to the list kernels; rows 10^3 to 10^30 times larger than the rest do not fit
    float16 after scaling; rows sorted by cluster."""
    rng = np.random.default_rng(d)
    N = 5000
    X = rng.standard_normal((N, d))
    if kind == "one_point":
        X[:] = X[0]
    elif kind == "few_points":
        X = X[rng.integers(0, 3, N)]
    elif kind == "far_rows":
        X[::700] *= 1.0e3
    elif kind == "beyond_float16":
        X[::900] *= 1.0e7
        X[5] = 3.0e17
    elif kind == "sorted":
        X = X * 0.1 + np.repeat(rng.uniform(-50, 50, size=(10, d)), N // 10, axis=0)
    elif kind == "one_column":
        X[:, 1:] = 0.0
    print(f"half-precision lists, {kind}, d={d}", flush=True)
    same_lists(lib, X.astype(np.float32), 12)


@pytest.mark.parametrize("m,n,d", [(1, 2, 1), (63, 129, 16), (65, 5000, 17), (130, 128, 128), (300, 9000, 129), (1500, 3000, 40),
                                   (4, 40_000, 260)])
def test_nearest_row_of_another_matrix(lib, m, n, d):
    print(f"half-precision 1-NN m={m} n={n} d={d}", flush=True)
    rng = np.random.default_rng(m + n + d)
    Q, Y = rng.standard_normal((m, d)).astype(np.float32), rng.standard_normal((n, d)).astype(np.float32)
    Y[n // 2] = Q[m // 2]
    gi, gd = lib.fused_1nn(torch.from_numpy(Q).cuda(), torch.from_numpy(Y).cuda())
    torch.cuda.synchronize()
    rows = np.unique(np.r_[0, m // 2, m - 1, rng.integers(0, m, 60)])
    colour = np.r_[np.zeros(m, np.int32), np.ones(n, np.int32)]
    oi, od = oracle.cross_1nn(np.concatenate([Q, Y]), colour, rows.astype(np.int64))
    assert np.allclose(gd.cpu().numpy()[rows], od, rtol=1e-5, atol=1e-30)
    assert (gi.cpu().numpy()[rows] == oi - m).mean() >= 0.99


@pytest.mark.parametrize("N,d,m,colours", [(130, 16, 5, 2), (4000, 64, 129, 7), (4000, 129, 600, 3), (20_000, 33, 64, 5000), (3000, 8, 3000, 1)])
def test_nearest_row_of_another_colour(lib, N, d, m, colours):
    """Rows in tight clusters of one colour each, so that a query's nearest foreign rows lie within the copies' rounding
    of each other by the hundred."""
    print(f"half-precision cross 1-NN N={N} d={d} m={m} colours={colours}", flush=True)
    rng = np.random.default_rng(N + m)
    label = rng.integers(0, max(colours, 12), N)
    X = (rng.uniform(-1000, 1000, size=(max(colours, 12), d))[label] + 0.1 * rng.standard_normal((N, d))).astype(np.float32)
    colour = (label % colours).astype(np.int32)
    rows = rng.integers(0, N, m).astype(np.int32)
    gi, gd = lib.cross_1nn(torch.from_numpy(X).cuda(), torch.from_numpy(colour).cuda(), torch.from_numpy(rows).cuda())
    torch.cuda.synchronize()
    gi, gd = gi.cpu().numpy(), gd.cpu().numpy()
    take = rng.integers(0, m, 50)
    if colours == 1:
        assert (gi == -1).all() and np.isinf(gd).all()
        return
    oi, od = oracle.cross_1nn(X, colour, rows[take].astype(np.int64))
    assert np.allclose(gd[take], od, rtol=1e-5)
    assert (gi[take] == oi).mean() >= 0.99


# connection rounds: components far apart, rows equally far from hundreds (a lattice; copies of rows), values beyond float16;
# few and many columns, one-workgroup forests and others
@pytest.mark.parametrize("kind", ["clusters", "lattice", "copies", "one_far_row", "all_far"])
@pytest.mark.parametrize("N,d", [(300, 3), (5000, 64), (13_000, 24), (4000, 129), (3000, 300), (20_000, 128)])
def test_trees_by_components(lib, kind, N, d):
    print(f"half-precision trees, {kind}, N={N} d={d}", flush=True)
    rng = np.random.default_rng(N + d)
    if kind == "lattice":
        X = rng.integers(0, 3, size=(N, d)) + 1000.0 * (rng.integers(0, 5, N) > 2)[:, None]
    else:
        X = 50.0 * rng.standard_normal((7, d))[rng.integers(0, 7, N)] + rng.standard_normal((N, d))
        if kind == "copies":
            X = X[rng.integers(0, N // 20 + 2, N)]
        if kind == "one_far_row":
            X[N // 3] *= 1e5
        if kind == "all_far":
            X *= 10.0 ** rng.uniform(0, 5, size=(N, 1))
    Xd = torch.from_numpy(X.astype(np.float32)).cuda()
    want = lib.slhc(Xd, 4, prune=False, fp32_filter=True)
    got = lib.slhc(Xd, 4, prune=False)
    torch.cuda.synchronize()
    for key in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(want[key], got[key]), key


# searches in the row order: panels of two, four and eight wavefronts (tiles from 256 and from 1024 on), clusters of more and of
# fewer rows than neighbours asked for, on both sides of the shortest region, one cluster, and clusters far apart for their size
@pytest.mark.parametrize("N,d,k,rows,spread", [
    (700, 4, 3, 700, 8), (5000, 128, 16, 20, 8), (20_000, 40, 31, 900, 8), (33_000, 100, 64, 1100, 40), (34_000, 12, 5, 8000, 8),
    (60_000, 64, 12, 2500, 5000), (64_000, 48, 9, 1000, 3000), (64_000, 48, 9, 850, 8), (110_000, 8, 20, 110_000, 0), (133_000, 20, 15, 9000, 8), (140_000, 128, 8, 30_000, 30),
])
def test_lists_and_trees_in_the_row_order(lib, N, d, k, rows, spread):
    print(f"half-precision row order N={N} d={d} k={k} rows={rows} spread={spread}", flush=True)
    rng = np.random.default_rng(N + d)
    centres = rng.uniform(-spread, spread, size=(max(1, N // rows), d))
    X = centres[rng.integers(0, len(centres), N)] + rng.standard_normal((N, d))
    X[: N // 50] = X[rng.integers(0, N, N // 50)] * (1.0 + 1e-3 * (rows > 5000))
    X[:3] = 40.0 * spread + rng.standard_normal((3, d))                       # fewer rows than neighbours, far from all others
    Xd = torch.from_numpy(X.astype(np.float32)).cuda()
    a, b = lib.knn_graph(Xd, k), lib.knn_graph(Xd, k, prune=True)
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    want, got = lib.slhc(Xd, min(k, 16), prune=False), lib.slhc(Xd, min(k, 16), prune=True)
    torch.cuda.synchronize()
    assert got["stats"]["pruned"] == 1
    for key in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(want[key], got[key]), key


# searches small enough to evaluate every pair: parts of a wavefront's queries, of a step of 64 candidates and of a slab of 64
# features, one and many shares of the candidates, rows that are not finite or close to it, rows outside the matrix
@pytest.mark.parametrize("m,n,d", [(1, 1, 1), (7, 63, 4), (9, 65, 31), (64, 1000, 64), (65, 1025, 65), (3, 30_000, 130), (2000, 700, 12)])
def test_small_nearest_row_searches(lib, m, n, d):
    print(f"small 1-NN m={m} n={n} d={d}", flush=True)
    rng = np.random.default_rng(m + n + d)
    Q, Y = rng.standard_normal((m, d)).astype(np.float32), rng.standard_normal((n, d)).astype(np.float32)
    Y[n // 3] = Y[n // 2] = Q[m // 2]
    if n > 100:
        Y[5] = np.nan
        Y[6] = 3e19
        Q[0] = 1e19 if m > 5 else Q[0]
    gi, gd = lib.fused_1nn(torch.from_numpy(Q).cuda(), torch.from_numpy(Y).cuda())
    colour = np.r_[np.zeros(m, np.int32), np.ones(n, np.int32)]
    both = torch.from_numpy(np.concatenate([Q, Y])).cuda()
    rows = torch.tensor(list(range(m)) + [-1, m + n], dtype=torch.int32, device="cuda")
    ci, cd = lib.cross_1nn(both, torch.from_numpy(colour).cuda(), rows)
    torch.cuda.synchronize()
    assert ci[m:].tolist() == [-1, -1] and torch.isinf(cd[m:]).all()
    assert torch.equal(ci[:m], torch.where(gi >= 0, gi + m, gi)) and torch.equal(cd[:m], gd)
    fine = np.flatnonzero(np.isfinite(Y).all(1) & (np.abs(Y).max(1) < 1e19))
    D = ((Q[:, None, :].astype(np.float64) - Y[None, fine, :]) ** 2).sum(2) if m * len(fine) * d < 5e7 else None
    if D is not None:
        take = np.arange(1 if n > 100 and m > 5 else 0, m)
        assert np.allclose(gd.cpu().numpy()[take], D.min(1)[take], rtol=1e-5, atol=1e-30)
        exact = gi.cpu().numpy()[take] == fine[D.argmin(1)[take]]
        assert exact.mean() >= 0.99


def test_f16_mfma_error_stays_within_the_budget(lib):
    """near_e budgets 9 x 2^-23 (18 x 2^-24) of the largest partial sum per v_mfma_f32_32x32x16_f16, and everything the engine
    discards rests on that: one unit of 2^-24 for each of 16 products and the accumulator that are aligned to the largest term
    and cut off, one for the rounding of the sum.  Checked against exact float64 sums, relative to the largest of the 17 terms
    (which no partial sum of the sweeps' values exceeds): the error must stay below half the budget.  Values as the copies hold
    them (2^-14 and above, or 0; products down to 2^-28 and up to 2^24), of equal and of widely different magnitude, of one sign
    and of both, the accumulator far above, at and far below the products; and one large product beside fifteen small ones."""
    g = torch.Generator().manual_seed(78)
    T = 1 << 18
    worst = 0.0
    for spread in (0, 2, 4, 10, 18, 26):
        for sign in ("plus", "both"):
            def draw(shape):
                v = (1.0 + torch.rand(shape, generator=g)) * torch.exp2(12.0 - torch.randint(0, spread + 1, shape, generator=g).float())
                v = v.to(torch.float16).float()
                assert v.min() >= 2.0 ** -14
                if sign == "both":
                    v = torch.where(torch.rand(shape, generator=g) < 0.5, -v, v)
                return torch.where(torch.rand(shape, generator=g) < 0.05, torch.zeros(()), v)
            A, B = draw((T, 16)), draw((T, 16))
            C = (1.0 + torch.rand((T,), generator=g)) * torch.exp2(torch.randint(-8, 33, (T,), generator=g).float())
            C = torch.where(torch.arange(T) % 7 == 0, torch.zeros(()), -C if sign == "both" else C)
            D = lib.probe_f16_mfma_values(A.cuda(), B.cuda(), C.cuda()).cpu().double()
            prod = A.double() * B.double()                             # 22 bits each: exact
            exact = C.double() + prod.sum(dim=1)
            largest = torch.maximum(torch.maximum(C.double().abs(), prod.abs().max(dim=1).values), exact.abs())
            fine = largest > 0
            rel = ((D - exact).abs()[fine] / (largest[fine] * 2.0 ** -24)).max().item()
            print(f"f16 MFMA, exponent spread {spread}, {sign}: worst error {rel:.3f} x 2^-24 of the largest", flush=True)
            worst = max(worst, rel)
    for small in (2.0 ** -24, 2.0 ** -25, 2.0 ** -26):
        A = torch.full((1, 16), 2.0 ** -12)
        B = torch.full((1, 16), small * 2.0 ** 12)
        A[0, 0] = B[0, 0] = 1.0
        assert B.min() >= 2.0 ** -14
        D = lib.probe_f16_mfma_values(A.cuda(), B.cuda(), torch.zeros(1).cuda()).cpu().double().item()
        err = abs(D - (1.0 + 15 * small)) / 2.0 ** -24
        print(f"one product of 1 and fifteen of {small:.3g}: off by {err:.3f} x 2^-24", flush=True)
        worst = max(worst, err)
    assert worst <= 9.0
