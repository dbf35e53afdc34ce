"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same seeded
inputs.  Tolerances are the ones the task fixes: k-NN distances rel 1e-5, neighbour indices
exact except among ties inside that band, MST total weight rel 1e-6, merge heights rel 1e-5,
dendrogram topology identical on tie-free data."""
import numpy as np
import pytest

import oracle
import slhc_inputs as gen

torch = pytest.importorskip("torch")
from workspaces import by_list_kernels, cross_1nn_in  # noqa: E402

pytestmark = pytest.mark.gpu

RTOL_DIST = 1e-5
RTOL_TOTAL = 1e-6
ATOL0 = 1e-30


@pytest.fixture(scope="module")
def lib():
    import paper_2306_16354_amd as slhc
    slhc.load_library()            # raises when libslhc.so is missing: no fallback exists
    assert torch.cuda.is_available()
    return slhc


def close(a, b, rtol):
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    return np.abs(a - b) <= rtol * np.maximum(np.abs(a), np.abs(b)) + ATOL0


def pair_dist64(X, i, j):
    """float64 sum_t (x_it - x_jt)^2 for broadcast index arrays i, j (chunked over rows)."""
    i, j = np.broadcast_arrays(np.asarray(i), np.asarray(j))
    out = np.empty(i.shape, dtype=np.float64)
    flat_i, flat_j, flat_o = i.reshape(-1), j.reshape(-1), out.reshape(-1)
    step = max(1024, (1 << 24) // max(1, X.shape[1]))          # ~128 MB of float64 per gathered operand
    for s in range(0, flat_i.size, step):
        diff = X[flat_i[s:s + step]].astype(np.float64) - X[flat_j[s:s + step]].astype(np.float64)
        flat_o[s:s + step] = np.einsum("nt,nt->n", diff, diff)
    return out


def check_knn(X, k, gi, gd, rows=None, min_exact=0.0):
    """gi/gd: GPU lists of the given query rows (all rows when rows is None)."""
    N = X.shape[0]
    rows = np.arange(N) if rows is None else np.asarray(rows)
    oi, od = oracle.knn_rows(X, rows, k)
    assert gi.shape == oi.shape and gd.shape == od.shape
    assert gi.min() >= 0 and gi.max() < N
    assert not (gi == rows[:, None]).any(), "a row lists itself"
    srt = np.sort(gi, axis=1)
    assert (srt[:, 1:] != srt[:, :-1]).all(), "a row lists a neighbour twice"
    assert (np.diff(gd.astype(np.float64), axis=1) >= 0).all(), "list not ascending"
    # every reported distance is the distance of the reported pair
    true_d = pair_dist64(X, rows[:, None], gi)
    assert close(gd, true_d, RTOL_DIST).all()
    # the selection is right: position by position the distances are the oracle's
    bad = ~close(gd, od, RTOL_DIST)
    assert not bad.any(), f"{bad.sum()} distances off, first at {np.argwhere(bad)[:3]}"
    # indices: exact, except where the oracle's own distances tie within the band
    diff = gi != oi
    if diff.any():
        r, c = np.nonzero(diff)
        assert close(true_d[r, c], od[r, c], RTOL_DIST).all()
    exact = 1.0 - diff.mean()
    assert exact >= min_exact, f"only {exact:.4f} of indices agree exactly"
    return exact


def gpu_knn(lib, X, k):
    Xd = torch.from_numpy(X).cuda()
    idx, dist = lib.knn_graph(Xd, k)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), dist.cpu().numpy()


def knn_by_list_kernels(lib, Xd, k, **flags):
    """The k-NN graph without the half-precision engine, which the smallest workspace leaves no room for."""
    return by_list_kernels(lib, lambda ws: lib.knn_graph(Xd, k, workspace=ws, **flags))


def slhc_by_list_kernels(lib, Xd, k, **flags):
    return by_list_kernels(lib, lambda ws: lib.slhc(Xd, k, workspace=ws, **flags))


# ----------------------------------------------------------------------------- k-NN graph
KNN_CASES = [
    ("c1", None, 0.999),      # full small workload: 4096 x 16, k=16
    ("c2", 5000, 0.999),      # 64 features, k=32
    ("c3", 6000, 0.999),      # 128 features, k=32 (headline shape, scaled)
    ("c4", 1500, 0.999),      # 784 features (K tail: 784 = 24*32 + 16), k=16
    ("c5", 9000, 0.90),       # duplicates and mass ties, k=8
]


@pytest.mark.parametrize("name,n,min_exact", KNN_CASES)
def test_knn_workloads(lib, name, n, min_exact):
    X, _, k = gen.make(name, n=n)
    print(f"knn {name} N={X.shape[0]} d={X.shape[1]} k={k}", flush=True)
    gi, gd = gpu_knn(lib, X, k)
    check_knn(X, k, gi, gd, min_exact=min_exact)


@pytest.mark.parametrize("N,d,k", [
    (2, 1, 1), (3, 5, 2), (65, 4, 64), (129, 33, 7), (130, 19, 1), (1037, 20, 33),
    (257, 36, 16), (640, 128, 32), (1000, 3, 5),
])
def test_knn_ragged_shapes(lib, N, d, k):
    print(f"knn ragged N={N} d={d} k={k}", flush=True)
    X = np.random.default_rng(N * 1000 + d).standard_normal((N, d)).astype(np.float32)
    gi, gd = gpu_knn(lib, X, k)
    check_knn(X, k, gi, gd, min_exact=0.999)


def test_knn_lattice_ties_exact(lib):
    # all distances are small integers, exact in fp32: the (dist, idx) order must match exactly
    X = gen.integer_lattice(9, 3, seed=4)
    k = 20
    gi, gd = gpu_knn(lib, X, k)
    oi, od = oracle.knn_graph(X, k)
    assert np.array_equal(gi, oi)
    assert np.array_equal(gd.astype(np.float64), od)


def test_knn_duplicates_are_neighbours_at_zero(lib):
    X, _, k = gen.make("c5", n=4000)
    gi, gd = gpu_knn(lib, X, k)
    _, od = oracle.knn_graph(X, k)
    zero_rows = np.where(od[:, 0] == 0.0)[0]
    assert zero_rows.size > 0
    assert (gd[zero_rows, 0] == 0.0).all()
    assert (gi[zero_rows, 0] != zero_rows).all()
    assert np.array_equal(X[zero_rows], X[gi[zero_rows, 0]])


def test_knn_distance_symmetry_bitwise(lib):
    X, _, k = gen.make("c2", n=3000)
    gi, gd = gpu_knn(lib, X, k)
    table = {}
    for i in range(X.shape[0]):
        for j, dv in zip(gi[i].tolist(), gd[i].tolist()):
            table[(i, j)] = dv
    both = [(a, b) for (a, b) in table if (b, a) in table]
    assert len(both) > 1000
    assert all(table[(a, b)] == table[(b, a)] for a, b in both)


def test_knn_large_norm_small_distance(lib):
    # far from the origin the expanded form loses every digit of the distance in fp32; the
    # reported values must still be right
    rng = np.random.default_rng(7)
    X = (rng.standard_normal((3000, 32)) * 0.05 + 3000.0).astype(np.float32)
    gi, gd = gpu_knn(lib, X, 8)
    check_knn(X, 8, gi, gd, min_exact=0.99)


def test_knn_full_size_sampled_rows(lib):
    # c2 at its full size (100k x 64, k=32) in the launch configuration bench.py uses; the
    # oracle checks a seeded sample of rows one by one, and every reported pair is recomputed
    X, _, k = gen.make("c2")
    N = X.shape[0]
    gi, gd = gpu_knn(lib, X, k)
    true_d = pair_dist64(X, np.arange(N)[:, None], gi)
    assert close(gd, true_d, RTOL_DIST).all()
    rows = np.random.default_rng(1).choice(N, size=512, replace=False)
    check_knn(X, k, gi[rows], gd[rows], rows=rows, min_exact=0.999)


# ----------------------------------------------------------------------------- argument errors
def test_error_codes(lib):
    X = torch.zeros((10, 4), dtype=torch.float32, device="cuda")
    with pytest.raises(lib.SlhcError) as e:
        lib.knn_graph(X, 10)
    assert e.value.status == 1
    X = torch.zeros((100, 4), dtype=torch.float32, device="cuda")
    with pytest.raises(lib.SlhcError) as e:
        lib.knn_graph(X, 65)
    assert e.value.status == 2
    with pytest.raises(lib.SlhcError) as e:
        lib.knn_graph(X, 4, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
    assert e.value.status == 3


# ----------------------------------------------------------------------------- cross-colour 1-NN
# c5: the nearest foreign blob is ~1e7 away and 0.1 wide, so its points tie within fp32 rounding;
# there only the distance (and that the answer is a foreign point at that distance) is unique.
@pytest.mark.parametrize("name,n,ncol,min_exact", [("c1", 3000, 7, 0.99), ("c3", 2500, 3, 0.99),
                                                   ("c5", 5000, 50, 0.9)])
def test_cross_1nn(lib, name, n, ncol, min_exact):
    X, labels, _ = gen.make(name, n=n)
    N = X.shape[0]
    colour = (labels % ncol).astype(np.int32)
    rows = np.random.default_rng(3).choice(N, size=min(N, 700), replace=False).astype(np.int32)
    print(f"cross_1nn {name} N={N} colours={ncol}", flush=True)
    gi, gd = lib.cross_1nn(torch.from_numpy(X).cuda(), torch.from_numpy(colour).cuda(),
                           torch.from_numpy(rows).cuda())
    torch.cuda.synchronize()
    gi, gd = gi.cpu().numpy(), gd.cpu().numpy()
    oi, od = oracle.cross_1nn(X, colour, rows.astype(np.int64))
    assert close(gd, od, RTOL_DIST).all()
    assert (colour[gi] != colour[rows]).all()
    assert close(pair_dist64(X, rows, gi), od, RTOL_DIST).all()
    assert (gi == oi).mean() >= min_exact


def test_cross_1nn_single_colour_and_all_rows(lib):
    X, labels, _ = gen.make("c1", n=500)
    Xd = torch.from_numpy(X).cuda()
    one = torch.zeros(500, dtype=torch.int32, device="cuda")
    gi, gd = lib.cross_1nn(Xd, one)
    torch.cuda.synchronize()
    assert (gi.cpu().numpy() == -1).all() and np.isinf(gd.cpu().numpy()).all()
    colour = labels.astype(np.int32)
    gi, gd = lib.cross_1nn(Xd, torch.from_numpy(colour).cuda())
    torch.cuda.synchronize()
    oi, od = oracle.cross_1nn(X, colour, np.arange(500))
    assert np.array_equal(gi.cpu().numpy(), oi)
    assert close(gd.cpu().numpy(), od, RTOL_DIST).all()


# ----------------------------------------------------------------------------- MST + dendrogram
def cluster_signatures(children, N, seed=0):
    """One 64-bit sum-hash per merged cluster (independent of the order of the merges)."""
    h = np.random.default_rng(seed).integers(1, 2 ** 62, size=2 * N - 1, dtype=np.uint64)
    with np.errstate(over="ignore"):
        for i, (a, b) in enumerate(children):
            h[N + i] = h[a] + h[b]          # wraps modulo 2^64; fine for a signature
    return h[N:]


def isolated_heights(heights, rtol):
    """True where a merge height has no neighbour (in sorted order) within the tolerance band:
    only there is the cluster formed by the merge uniquely defined across arithmetic."""
    h = np.asarray(heights, dtype=np.float64)
    gap_ok = np.ones(h.size, dtype=bool)
    near = np.abs(np.diff(h)) <= rtol * np.maximum(np.abs(h[1:]), np.abs(h[:-1]))
    gap_ok[1:] &= ~near
    gap_ok[:-1] &= ~near
    return gap_ok


def check_slhc(X, out, tie_free):
    N = X.shape[0]
    ref = oracle.slhc(X)
    src, dst, w = (out[n].cpu().numpy() for n in ("mst_src", "mst_dst", "mst_w"))
    children, heights, sizes = (out[n].cpu().numpy() for n in ("children", "heights", "sizes"))
    assert src.shape == (N - 1,) and (src < dst).all()
    # spanning tree
    parent = np.arange(N)

    def find(a):
        while parent[a] != a:
            parent[a] = parent[parent[a]]
            a = parent[a]
        return a

    for a, b in zip(src.tolist(), dst.tolist()):
        ra, rb = find(a), find(b)
        assert ra != rb, "cycle in returned tree"
        parent[ra] = rb
    # weights are the weights of the returned pairs, ascending
    assert close(w, pair_dist64(X, src, dst), RTOL_DIST).all()
    key = list(zip(w.tolist(), src.tolist(), dst.tolist()))
    assert key == sorted(key)
    total = float(np.sum(w.astype(np.float64)))
    assert abs(total - ref["total_weight"]) <= RTOL_TOTAL * ref["total_weight"] + ATOL0, \
        f"total weight {total} vs oracle {ref['total_weight']}"
    assert close(heights, ref["heights"], RTOL_DIST).all()
    assert np.array_equal(heights, w)
    # linkage invariants
    assert sizes[-1] == N
    assert sorted(children.ravel().tolist()) == list(range(2 * N - 2))
    assert (children[:, 0] < children[:, 1]).all()
    assert (children < (N + np.arange(N - 1))[:, None]).all()
    if tie_free:
        # Topology: every cluster that the oracle forms at a height with no near-tie next to it
        # must be formed by the GPU hierarchy too, and the other way round.  (Two merges whose
        # heights differ by less than float32 resolves may legitimately swap.)
        sig_g, sig_o = cluster_signatures(children, N), cluster_signatures(ref["children"], N)
        # band: a few float32 ulps, the accuracy of a directly summed squared distance
        iso_o, iso_g = isolated_heights(ref["heights"], 1e-6), isolated_heights(heights, 1e-6)
        n_tied = int((~iso_o).sum())
        # (how many heights have a neighbour within the band grows like N^2 x band on any continuous data:
        # it says where clusters may legitimately differ, not how much the trees do; that is the edge
        # comparison below, whose budget is absolute)
        print(f"  merge heights with a neighbour within 1e-6 relative (oracle): {n_tied} of {N - 1}", flush=True)
        assert np.isin(sig_o[iso_o], sig_g).all(), "an oracle cluster is missing from the GPU hierarchy"
        assert np.isin(sig_g[iso_g], sig_o).all(), "a GPU cluster is missing from the oracle hierarchy"
        assert np.array_equal(np.sort(sizes[iso_g & iso_o]), np.sort(ref["sizes"][iso_g & iso_o]))
        # Edge sets: the two trees may differ only by exchanging edges whose float64 weights agree
        # within what float32 resolves (each exchanged pair closes a cycle in which both are the heaviest
        # edge up to rounding), and only a handful of such exchanges can exist on tie-free data.
        eg = {(a, b) for a, b in zip(src.tolist(), dst.tolist())}
        eo = {(a, b) for a, b in zip(ref["src"].tolist(), ref["dst"].tolist())}
        only_g, only_o = sorted(eg - eo), sorted(eo - eg)
        print(f"  tree edges not shared with the oracle's tree: {len(only_g)}", flush=True)
        assert len(only_g) == len(only_o) <= max(2, N // 20000)
        if only_g:
            wg = np.sort(pair_dist64(X, [a for a, _ in only_g], [b for _, b in only_g]))
            wo = np.sort(pair_dist64(X, [a for a, _ in only_o], [b for _, b in only_o]))
            assert close(wg, wo, 2e-6).all(), "trees differ by more than an exchange of equal-weight edges"
    return out["stats"]


def check_tree_properties(X, k, gi, out, rng, n_nn=20_000, n_pairs=300, n_weights=300_000):
    """Checks of a returned tree and dendrogram that hold at any size, for inputs the oracle cannot
    finish: the edges span without a cycle (the sizes must be those of a union over the returned
    children), sampled weights are the float64 distances of their pairs, the nearest neighbour of
    every sampled vertex is a tree edge (the first Boruvka round is exact), and no sampled near pair
    is closer than the merge height of its lowest common ancestor (the cycle property)."""
    N = X.shape[0]
    src, dst, w = (out[n].cpu().numpy() for n in ("mst_src", "mst_dst", "mst_w"))
    children, heights, sizes = (out[n].cpu().numpy() for n in ("children", "heights", "sizes"))
    assert (src < dst).all() and (np.diff(w.astype(np.float64)) >= 0).all()
    es = rng.choice(N - 1, size=min(n_weights, N - 1), replace=False)
    assert close(w[es], pair_dist64(X, src[es], dst[es]), RTOL_DIST).all()
    assert np.array_equal(heights, w)
    # every tree edge joins two different clusters of the dendrogram built so far: replay the merges
    assert sizes[-1] == N
    counts = np.bincount(children.ravel(), minlength=2 * N - 1)
    assert (counts[:2 * N - 2] == 1).all() and counts[2 * N - 2] == 0
    assert (children[:, 0] < children[:, 1]).all()
    assert (children < (N + np.arange(N - 1))[:, None]).all()
    parent = np.arange(2 * N - 1)
    sz = np.ones(2 * N - 1, dtype=np.int64)
    parent[children[:, 0]] = N + np.arange(N - 1)
    parent[children[:, 1]] = N + np.arange(N - 1)
    for i in range(N - 1):
        sz[N + i] = sz[children[i, 0]] + sz[children[i, 1]]
    assert np.array_equal(sz[N:], sizes.astype(np.int64))
    # the dendrogram is the one of the returned edges: edge i must join the two children of merge i.
    # Checked on a sample by walking up from both end points to the first node created at or after i.
    def node_at(v, i):
        x = int(v)
        while parent[x] != x and parent[x] < N + i:
            x = int(parent[x])
        return x
    for i in rng.choice(N - 1, size=min(2000, N - 1), replace=False).tolist():
        a, b = node_at(src[i], i), node_at(dst[i], i)
        assert {a, b} == {int(children[i, 0]), int(children[i, 1])}, f"merge {i} does not join the ends of edge {i}"
    # distinct edges (with N-1 of them and the union replay above: a spanning tree)
    assert np.unique(src.astype(np.int64) * N + dst).size == N - 1
    # every vertex's nearest neighbour is a tree edge, unless another tree edge of the same weight
    # may stand in for it (exact duplicates: zero-weight ties)
    edge_keys = set((src.astype(np.int64) * N + dst).tolist())
    vs = rng.choice(N, size=min(n_nn, N), replace=False)
    nn = gi[vs, 0].astype(np.int64)
    lo, hi = np.minimum(vs, nn), np.maximum(vs, nn)
    missing = [(int(a), int(b)) for a, b in zip(lo, hi) if int(a) * N + int(b) not in edge_keys]
    if missing:
        # allowed only among ties: then v has a tree edge of exactly the same weight
        tree_min = np.full(N, np.inf)
        np.minimum.at(tree_min, src, w)
        np.minimum.at(tree_min, dst, w)
        for a, b in missing:
            dab = float(pair_dist64(X, [a], [b])[0])
            assert tree_min[a] <= dab * (1 + 1e-6) + ATOL0 and tree_min[b] <= dab * (1 + 1e-6) + ATOL0, \
                f"nearest-neighbour pair ({a},{b}) at {dab} is not covered by the tree"
    # cycle property on sampled near pairs: d(a,b) >= height of the lowest common ancestor
    def lca_height(a, b):
        seen = set()
        x = int(a)
        while True:
            seen.add(x)
            if parent[x] == x:
                break
            x = int(parent[x])
        y = int(b)
        while y not in seen:
            y = int(parent[y])
        return float(heights[y - N])

    pa = rng.integers(0, N, size=n_pairs)
    pb = gi[pa, rng.integers(0, k, size=n_pairs)]          # near pairs are the ones that could violate it
    d_ab = pair_dist64(X, pa, pb)
    for a, b, dab in zip(pa, pb, d_ab):
        assert lca_height(a, b) <= dab * (1 + 1e-5) + ATOL0


SLHC_CASES = [
    ("c1", None, True),
    ("c2", 4000, True),
    ("c3", 5000, True),
    ("c4", 1200, True),
    ("c5", 6000, False),
]


@pytest.mark.parametrize("name,n,tie_free", SLHC_CASES)
def test_slhc_workloads(lib, name, n, tie_free):
    X, _, k = gen.make(name, n=n)
    print(f"slhc {name} N={X.shape[0]} d={X.shape[1]} k={k}", flush=True)
    out = lib.slhc(torch.from_numpy(X).cuda(), k)
    stats = check_slhc(X, out, tie_free)
    print("stats", stats, flush=True)
    assert stats["boruvka_rounds"] >= 1


def test_slhc_connected_knn_graph_that_misses_an_mst_edge(lib):
    # two triples half a unit apart and a far point: the 2-NN graph is connected but lacks the
    # edge between the triples; the exact tree must still contain it
    X = np.array([[0, 0], [0, -.1], [0, -.2], [.5, 0], [.5, -.1], [.5, -.2], [.2, 10]], dtype=np.float32)
    out = lib.slhc(torch.from_numpy(X).cuda(), 2)
    check_slhc(X, out, tie_free=False)
    edges = set(zip(out["mst_src"].cpu().tolist(), out["mst_dst"].cpu().tolist()))
    assert (0, 3) in edges
    assert out["stats"]["connect_rounds"] >= 1


def test_slhc_increasing_gaps_line(lib):
    # closed form: consecutive points, weights (i+1)^2; also a worst case for hook chains
    N = 600
    X, pos = gen.increasing_gaps_line(N, 3, seed=2)
    out = lib.slhc(torch.from_numpy(X).cuda(), 4)
    check_slhc(X, out, tie_free=True)
    assert out["mst_w"].cpu().tolist() == [float((i + 1) ** 2) for i in range(N - 1)]


def test_slhc_hook_chain_longer_than_the_device_passes(lib):
    # every point's lightest edge leads to its left neighbour, so the first round hooks all N components into
    # one chain; beyond ~1000 hooks the two device passes of pointer jumping do not reach its end and the host
    # has to finish the chain before the relabelling (weights (i+1)^2 stay exact in float32 up to N = 4096)
    N = 3000
    X, pos = gen.increasing_gaps_line(N, 2, seed=5)
    out = lib.slhc(torch.from_numpy(X).cuda(), 3)
    check_slhc(X, out, tie_free=True)
    assert out["mst_w"].cpu().tolist() == [float((i + 1) ** 2) for i in range(N - 1)]


def test_slhc_unit_lattice_all_ties(lib):
    X = gen.integer_lattice(12, 2, seed=8)
    out = lib.slhc(torch.from_numpy(X).cuda(), 4)
    check_slhc(X, out, tie_free=False)
    assert (out["mst_w"].cpu().numpy() == 1.0).all()


def test_slhc_two_far_blobs(lib):
    rng = np.random.default_rng(11)
    X = np.concatenate([rng.standard_normal((300, 5)), rng.standard_normal((200, 5)) + 40.0]).astype(np.float32)
    out = lib.slhc(torch.from_numpy(X).cuda(), 8)
    stats = check_slhc(X, out, tie_free=True)
    assert stats["connect_rounds"] >= 1
    assert out["sizes"].cpu().tolist()[-1] == 500


def test_slhc_tiny(lib):
    for N, k in [(2, 1), (3, 2), (5, 1)]:
        X = np.random.default_rng(N).standard_normal((N, 2)).astype(np.float32)
        out = lib.slhc(torch.from_numpy(X).cuda(), k)
        check_slhc(X, out, tie_free=True)


# ----------------------------------------------------------------------------- tile pruning
# Pruning (SLHC_PRUNE) only skips work that cannot change a list, and ties are ordered by the
# caller's row ids in both modes, so its results must be bit-identical to the unpruned sweep.
@pytest.mark.parametrize("name,n", [("c1", None), ("c2", 20000), ("c3", 12000), ("c5", 30000)])
def test_pruned_knn_is_identical(lib, name, n):
    X, _, k = gen.make(name, n=n)
    print(f"pruned knn {name} N={X.shape[0]} d={X.shape[1]} k={k}", flush=True)
    Xd = torch.from_numpy(X).cuda()
    i0, d0 = lib.knn_graph(Xd, k, prune=False)
    i1, d1 = lib.knn_graph(Xd, k, prune=True)
    torch.cuda.synchronize()
    assert torch.equal(i0, i1) and torch.equal(d0, d1)
    rows = np.random.default_rng(5).choice(X.shape[0], size=300, replace=False)
    check_knn(X, k, i1.cpu().numpy()[rows], d1.cpu().numpy()[rows], rows=rows, min_exact=0.9)


# Whatever path fills a list (the first tile's seeding pass, the batched queue, the deferred queue),
# every neighbour appears once and the entries ascend in (distance, id): data with many exact
# duplicates and equal distances, both modes, several k.
@pytest.mark.parametrize("k", [2, 8, 33])
def test_knn_lists_are_strictly_ordered(lib, k):
    X, _, _ = gen.make("c5", n=20000)
    print(f"list order c5 N={X.shape[0]} d={X.shape[1]} k={k}", flush=True)
    Xd = torch.from_numpy(X).cuda()
    for prune in (False, True):
        idx, dist = lib.knn_graph(Xd, k, prune=prune)
        torch.cuda.synchronize()
        i, d = idx.cpu().numpy().astype(np.int64), dist.cpu().numpy()
        assert (i >= 0).all() and (i < X.shape[0]).all()
        assert (i != np.arange(X.shape[0])[:, None]).all()                  # self excluded
        dd, di = np.diff(d, axis=1), np.diff(i, axis=1)
        assert (dd >= 0).all()
        assert ((dd > 0) | (di > 0)).all()                                  # strict (distance, id) order: no repeats


def test_pruned_knn_lattice_and_ragged(lib):
    X = gen.integer_lattice(9, 3, seed=4)                      # ties everywhere
    Xd = torch.from_numpy(X).cuda()
    i0, d0 = lib.knn_graph(Xd, 20, prune=False)
    i1, d1 = lib.knn_graph(Xd, 20, prune=True)
    torch.cuda.synchronize()
    assert torch.equal(i0, i1) and torch.equal(d0, d1)
    oi, od = oracle.knn_graph(X, 20)
    assert np.array_equal(i1.cpu().numpy(), oi)
    for N, d, k in [(2, 4, 1), (130, 20, 7), (1037, 36, 33), (5000, 128, 64)]:
        X = np.random.default_rng(N).standard_normal((N, d)).astype(np.float32)
        Xd = torch.from_numpy(X).cuda()
        i0, d0 = lib.knn_graph(Xd, k, prune=False)
        i1, d1 = lib.knn_graph(Xd, k, prune=True)
        torch.cuda.synchronize()
        assert torch.equal(i0, i1) and torch.equal(d0, d1), (N, d, k)


@pytest.mark.parametrize("name,n", [("c1", None), ("c2", 15000), ("c3", 10000), ("c5", 20000)])
def test_pruned_slhc_is_identical(lib, name, n):
    X, _, k = gen.make(name, n=n)
    print(f"pruned slhc {name} N={X.shape[0]} d={X.shape[1]} k={k}", flush=True)
    Xd = torch.from_numpy(X).cuda()
    a = lib.slhc(Xd, k, prune=False)
    b = lib.slhc(Xd, k, prune=True)
    assert a["stats"]["pruned"] == 0 and b["stats"]["pruned"] == 1
    for name_ in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(a[name_], b[name_]), name_
    T = (X.shape[0] + 127) // 128
    assert a["stats"]["knn_tile_steps"] == T * T
    Ts = (b["stats"]["order_padded_rows"] + 127) // 128       # the reordered copy has padding rows
    assert X.shape[0] <= b["stats"]["order_padded_rows"] <= X.shape[0] + X.shape[0] // 2 + 256
    assert b["stats"]["knn_tile_steps"] <= Ts * Ts
    print("tile steps", b["stats"]["knn_tile_steps"], "of", T * T, "connect", b["stats"]["connect_tile_steps"],
          "vs", a["stats"]["connect_tile_steps"], "pivots", b["stats"]["order_pivots"], "padded rows",
          b["stats"]["order_padded_rows"], "order ms", round(b["stats"]["ms_order"], 2), flush=True)


def _pruned_equals_every_tile(lib, X, k):
    Xd = torch.from_numpy(np.ascontiguousarray(X, dtype=np.float32)).cuda()
    i0, d0 = lib.knn_graph(Xd, k, prune=False)
    i1, d1 = lib.knn_graph(Xd, k, prune=True)
    torch.cuda.synchronize()
    assert torch.equal(i0, i1) and torch.equal(d0, d1)
    a = lib.slhc(Xd, k, prune=False)
    b = lib.slhc(Xd, k, prune=True)
    for name_ in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(a[name_], b[name_]), name_
    return b


def test_pruned_with_outliers_uniform_and_duplicates(lib):
    rng = np.random.default_rng(11)
    # blobs plus 5 % uniform noise: the noise rows end up far from every pivot
    X, _, _ = gen.make("c1", n=19000)
    noise = rng.uniform(-12, 12, size=(1000, X.shape[1])).astype(np.float32)
    Xn = np.concatenate([X, noise])[rng.permutation(20000)]
    print("pruned: blobs + outliers", flush=True)
    b = _pruned_equals_every_tile(lib, Xn, 16)
    assert b["stats"]["pruned"] == 1
    check_slhc(Xn[:3000], lib.slhc(torch.from_numpy(np.ascontiguousarray(Xn[:3000])).cuda(), 16), tie_free=True)
    # no cluster structure at all
    print("pruned: uniform cube", flush=True)
    _pruned_equals_every_tile(lib, gen.uniform_cube(15000, 8, seed=5), 8)
    # half of the rows are exact copies of other rows (zero distances, mass ties)
    print("pruned: duplicates", flush=True)
    base = rng.standard_normal((4000, 12)).astype(np.float32)
    Xdup = np.concatenate([base, base[rng.integers(0, 4000, size=4000)]])[rng.permutation(8000)]
    _pruned_equals_every_tile(lib, Xdup, 4)
    # one single point repeated: every distance is zero
    print("pruned: one point", flush=True)
    _pruned_equals_every_tile(lib, np.ones((700, 8), dtype=np.float32), 3)


@pytest.mark.parametrize("N,d,k", [(512, 4, 3), (513, 36, 7), (1000, 128, 64), (2049, 20, 1), (6000, 100, 32)])
def test_pruned_ragged_shapes(lib, N, d, k):
    print(f"pruned ragged N={N} d={d} k={k}", flush=True)
    rng = np.random.default_rng(N + d)
    centres = rng.uniform(-20, 20, size=(7, d))
    X = (centres[rng.integers(0, 7, size=N)] + rng.standard_normal((N, d))).astype(np.float32)
    b = _pruned_equals_every_tile(lib, X, k)
    assert b["stats"]["pruned"] == 1
    check_slhc(X, b, tie_free=True)


def test_pruned_random_shapes(lib):
    """Seeded random shapes (rows, features, k, number and spread of blobs, duplicates, quantised
    coordinates): pruned and every-tile paths agree bit for bit, twice in a row with the same
    query counts, and the small cases also match the oracle."""
    rng = np.random.default_rng(2023)
    for case in range(24):
        N = int(rng.integers(520, 30000)) if case % 4 else int(rng.integers(520, 3000))
        d = int(rng.choice([4, 8, 12, 16, 20, 32, 36, 64, 100, 128]))
        k = int(rng.integers(1, 65))
        nb = int(rng.integers(1, 200))
        spread = float(rng.choice([3.0, 20.0, 1000.0]))
        sigma = float(rng.choice([0.05, 1.0, 3.0]))
        centres = rng.uniform(-spread, spread, size=(nb, d))
        X = (centres[rng.integers(0, nb, size=N)] + sigma * rng.standard_normal((N, d))).astype(np.float32)
        ties = False
        if case % 6 == 5:
            # a common offset (the split copy is taken relative to the column means) on rows that come sorted along
            # one axis (regions of the row order that follow the input order)
            X = (X + np.float32(1.0e4))[np.argsort(X[:, 0], kind="stable")]
        if rng.random() < 0.3:
            m = N // 10
            X[rng.integers(0, N, size=m)] = X[rng.integers(0, N, size=m)]
            ties = True
        if rng.random() < 0.3:
            X = (np.round(X * 2) / 2).astype(np.float32)
            ties = True
        print(f"random case {case}: N={N} d={d} k={k} blobs={nb} spread={spread} sigma={sigma} ties={ties}", flush=True)
        b = _pruned_equals_every_tile(lib, X, k)
        Xd = torch.from_numpy(np.ascontiguousarray(X)).cuda()
        b2 = lib.slhc(Xd, k)
        # which rows are queried is a function of the forest state alone; how many tiles their panels skip
        # depends on which panel lowers a component's threshold first, so tile steps may differ
        assert b2["stats"]["connect_query_rows"] == b["stats"]["connect_query_rows"]
        # the sweeps' own lower bounds (what row orders of more than 32768 tiles get) instead of the table
        b3 = lib.slhc(Xd, k, tile_table=False, split_scans=bool(case % 2))
        for name_ in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
            assert torch.equal(b[name_], b3[name_]), name_
        i3, d3 = lib.knn_graph(Xd, k, prune=True, tile_table=False)
        i0, d0 = lib.knn_graph(Xd, k)
        assert torch.equal(i0, i3) and torch.equal(d0, d3)
        if N <= 3000:
            check_slhc(np.ascontiguousarray(X), b, tie_free=not ties)


# ----------------------------------------------------------------------------- zero columns appended by the library
@pytest.mark.parametrize("N,d,k", [(700, 1, 3), (3000, 7, 5), (5000, 50, 16), (4000, 100, 32), (2100, 127, 64),
                                   (3000, 130, 8), (2500, 301, 16)])
def test_padded_columns_change_nothing(lib, N, d, k):
    """The list kernels of slhc_knn_graph and slhc_slhc work on a copy of X with zero columns appended (whole chunks of 32 up to
    128 features, a multiple of 4 beyond), which opens the register-resident-query kernel, split products and tile
    pruning to every d.  A zero column adds nothing to a distance, so their lists (float32 products, and those of the smallest
    workspace) must equal, bit for bit, those of the half-precision engine, which reads the rows as they are, with and without
    a workspace (slhc_knn_graph_static), the pruned path those of the every-tile path, and both the oracle's."""
    rng = np.random.default_rng(N + 7 * d)
    centres = rng.uniform(-15, 15, size=(9, d))
    X = (centres[rng.integers(0, 9, size=N)] + rng.standard_normal((N, d))).astype(np.float32)
    print(f"padded columns N={N} d={d} k={k}", flush=True)
    Xd = torch.from_numpy(X).cuda()
    plain = (torch.empty((N, k), dtype=torch.int32, device="cuda"), torch.empty((N, k), dtype=torch.float32, device="cuda"))
    lib.knn_graph_static(Xd, k, plain)
    i0, d0 = lib.knn_graph(Xd, k)
    torch.cuda.synchronize()
    assert torch.equal(plain[0], i0) and torch.equal(plain[1], d0)
    for padded in (lib.knn_graph(Xd, k, fp32_filter=True), knn_by_list_kernels(lib, Xd, k)):
        assert torch.equal(padded[0], i0) and torch.equal(padded[1], d0)
    check_knn(X, k, i0.cpu().numpy(), d0.cpu().numpy(), min_exact=0.999)
    b = _pruned_equals_every_tile(lib, X, k)
    assert b["stats"]["pruned"] == (1 if d <= 128 else 0)
    check_slhc(X, b, tie_free=True)


# ----------------------------------------------------------------------------- tile products from split bfloat16 halves
@pytest.mark.parametrize("kind", ["offset", "mantissa", "mixed_scale", "duplicates", "lattice", "tiny"])
@pytest.mark.parametrize("d", [32, 64, 96, 128, 132, 260, 784])
def test_split_bf16_filter_loses_nothing(lib, kind, d):
    """From 32 to 128 features (multiples of 32, register-resident queries) and beyond 128 features (multiples of
    4, streaming kernel, split copy padded to whole chunks) the every-tile sweeps of the list kernels (panel order; the
    smallest workspace) form their tile products from bfloat16 halves (hi*hi + hi*lo + lo*hi) and widen the filter's slack by
    what that drops; the half-precision engine, which runs otherwise, multiplies float16 copies under a bound of its own.  The
    filter only decides which pairs are evaluated exactly, so lists and trees of all three must equal those of the float32
    products bit for bit, and the oracle's on sampled rows, also where the slack is put to the test: a common offset far
    larger than the distances, values that use all 24 bits, rows of very different scale, duplicates, a
    lattice with many exact ties, tiny values."""
    rng = np.random.default_rng(len(kind) * 1000 + d)
    N = int(rng.integers(3000, 9000))
    k = int(rng.choice([1, 5, 16, 32, 64]))
    X = rng.standard_normal((N, d))
    if kind == "offset":
        X = 0.01 * X + 1000.0 * rng.standard_normal((1, d))
    elif kind == "mantissa":
        X = X * (1.0 + 2.0 ** -23 * rng.integers(0, 2 ** 22, size=(N, d)))
    elif kind == "mixed_scale":
        X = X * np.where(rng.random((N, 1)) < 0.1, 3.0e3, 1.0)
    elif kind == "duplicates":
        X[rng.integers(0, N, size=N // 3)] = X[rng.integers(0, N, size=N // 3)]
    elif kind == "lattice":
        X = np.round(X)
    elif kind == "tiny":
        X = X * 1.0e-15
    X = np.ascontiguousarray(X.astype(np.float32))
    Xd = torch.from_numpy(X).cuda()
    print(f"split bf16 filter: {kind} N={N} d={d} k={k}", flush=True)
    a = lib.knn_graph(Xd, k, fp32_filter=True)
    b = lib.knn_graph(Xd, k)
    for c in (b, lib.knn_graph(Xd, k, panel_order=True), knn_by_list_kernels(lib, Xd, k)):
        torch.cuda.synchronize()
        assert torch.equal(a[0], c[0]) and torch.equal(a[1], c[1])
    rows = rng.choice(N, size=150, replace=False)
    check_knn(X, k, b[0].cpu().numpy()[rows], b[1].cpu().numpy()[rows], rows=rows,
              min_exact=0.0 if kind in ("duplicates", "lattice") else 0.9)
    kt = min(k, 16)
    ta = lib.slhc(Xd, kt, prune=False, fp32_filter=True)
    assert ta["stats"]["split_products"] == 0
    for half, tb in ((1, lib.slhc(Xd, kt, prune=False)), (0, lib.slhc(Xd, kt, prune=False, panel_order=True)),
                     (0, slhc_by_list_kernels(lib, Xd, kt, prune=False))):
        assert tb["stats"]["split_products"] == 1 and tb["stats"]["half_products"] == half
        for name_ in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
            assert torch.equal(ta[name_], tb[name_]), name_


@pytest.mark.parametrize("N,d,k,offset", [(30_000, 20, 8, 1.0e4), (26_000, 3, 4, 3.0e5), (25_000, 64, 16, 1.0e3),
                                          (6_000, 200, 8, 1.0e3)])
def test_common_offset_stays_out_of_the_filter(lib, N, d, k, offset):
    """The filter's slack is a fraction of the rows' squared norms.  The split copy is taken relative to the column
    means, so an offset shared by all rows (coordinates far from the origin, all-positive features) does not count
    towards it; below 64 features, where the pruned sweeps otherwise multiply the rows as they are in float32, they
    switch to the split copy when the means carry most of the norms.  Same lists and trees as with float32
    products and as the oracle on sampled rows, and about as few pairs passed on to the exact evaluation as for
    the same data without the offset (without the shift: every pair of every multiplied tile).  The copies of the half-precision
    engine are taken relative to a central value of every column likewise; both are looked at."""
    rng = np.random.default_rng(N + d)
    centres = rng.uniform(-10, 10, size=(30, d))
    base = centres[rng.integers(0, 30, size=N)] + rng.standard_normal((N, d))
    shift = offset * rng.standard_normal((1, d))
    print(f"common offset N={N} d={d} k={k} offset={offset}", flush=True)
    per_row = {}
    for name_, X in (("plain", base.astype(np.float32)), ("offset", (base + shift).astype(np.float32))):
        Xd = torch.from_numpy(np.ascontiguousarray(X)).cuda()
        a = lib.knn_graph(Xd, k, fp32_filter=True)
        b = lib.knn_graph(Xd, k)
        c = lib.knn_graph(Xd, k, prune=True)
        torch.cuda.synchronize()
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and torch.equal(a[0], c[0]) and torch.equal(a[1], c[1])
        rows = rng.choice(N, size=100, replace=False)
        check_knn(X, k, b[0].cpu().numpy()[rows], b[1].cpu().numpy()[rows], rows=rows, min_exact=0.9)
        every = lib.slhc(Xd, k, prune=False)
        pruned = lib.slhc(Xd, k, prune=True)
        for n_ in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
            assert torch.equal(every[n_], pruned[n_]), n_
        lists = [slhc_by_list_kernels(lib, Xd, k, prune=prune) for prune in (False, True)]
        for out in lists:
            assert torch.equal(every["children"], out["children"]) and torch.equal(every["mst_w"], out["mst_w"])
        per_row[name_] = [out["stats"]["knn_filter_survivors"] / N for out in (every, pruned, *lists)]
        print(f"  {name_}: pairs passed per row, every tile and pruned, engine and list kernels: {per_row[name_]}", flush=True)
    for offset_, plain_ in zip(per_row["offset"], per_row["plain"]):
        assert offset_ <= 3.0 * plain_ + 50


@pytest.mark.parametrize("kind", ["blobs", "one_cluster", "tiny_clusters", "uniform", "chain"])
@pytest.mark.parametrize("d", [64, 100, 128])
def test_pruned_knn_by_regions_is_identical(lib, kind, d):
    """From 64 to 128 features the pruned k-NN sweep of the list kernels (without the table of tile pairs; the smallest
    workspace) runs as two launches: the tiles of a panel's own region (a run
    of tiles of the row order whose centres stay close) from a split copy relative to a centre of that region,
    then all other tiles, starting from the lists of the first launch, from the copy relative to the column
    means.  The half-precision engine, which runs otherwise, has a copy relative to the regions as well.  Only the filter's
    slack differs, so the lists must equal, bit for bit, those of the single launch
    (SLHC_ONE_SHIFT), of the every-tile sweep and of the entry point that never reorders, on data with
    one region, with regions of a tile or two, with none to speak of, and with clusters strung along a line so
    that a region's first tile lies far from its last."""
    rng = np.random.default_rng(len(kind) * 100 + d)
    N = int(rng.integers(6000, 14000))
    k = int(rng.choice([1, 7, 32]))
    if kind == "blobs":
        centres = rng.uniform(-40, 40, size=(12, d))
        X = centres[rng.integers(0, 12, size=N)] + rng.standard_normal((N, d))
    elif kind == "one_cluster":
        X = 300.0 + rng.standard_normal((N, d))
    elif kind == "tiny_clusters":
        centres = rng.uniform(-500, 500, size=(N // 40, d))
        X = centres[rng.integers(0, N // 40, size=N)] + 0.05 * rng.standard_normal((N, d))
    elif kind == "uniform":
        X = rng.uniform(-1, 1, size=(N, d))
    else:
        t = rng.uniform(0, 400, size=(N, 1))
        X = t * np.ones((1, d)) / np.sqrt(d) + 0.5 * rng.standard_normal((N, d))
    X = np.ascontiguousarray(X.astype(np.float32))
    Xd = torch.from_numpy(X).cuda()
    print(f"pruned k-NN by regions: {kind} N={N} d={d} k={k}", flush=True)
    plain = (torch.empty((N, k), dtype=torch.int32, device="cuda"), torch.empty((N, k), dtype=torch.float32, device="cuda"))
    lib.knn_graph_static(Xd, k, plain)
    two = lib.knn_graph(Xd, k, prune=True)
    one = lib.knn_graph(Xd, k, prune=True, one_shift=True)
    lists = [lib.knn_graph(Xd, k, prune=True, tile_table=False), knn_by_list_kernels(lib, Xd, k, prune=True)]
    torch.cuda.synchronize()
    for got in (two, one, *lists):
        assert torch.equal(plain[0], got[0]) and torch.equal(plain[1], got[1])
    a = slhc_by_list_kernels(lib, Xd, min(k, 16), prune=True)
    b = lib.slhc(Xd, min(k, 16), prune=True, one_shift=True)
    c = lib.slhc(Xd, min(k, 16), prune=False)
    e = lib.slhc(Xd, min(k, 16), prune=True)
    for name_ in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(a[name_], b[name_]) and torch.equal(a[name_], c[name_]) and torch.equal(a[name_], e[name_]), name_
    print(f"  pairs passed per row: {a['stats']['knn_filter_survivors'] / N:.1f} by regions, "
          f"{b['stats']['knn_filter_survivors'] / N:.1f} in one launch", flush=True)


def test_far_outlier_does_not_drag_the_shift(lib):
    """The shift of the split copy, as that of the float16 copy, is a median of means, not a mean: one row at 1e12 among
    unit-scale rows would move a mean to 3e8 per column and put that into every row's norm, after which every pair passes the
    filter.  Same lists with float32 products of the rows as they are, and about as few pairs passed as without the row."""
    rng = np.random.default_rng(77)
    N, d, k = 4500, 40, 6                  # (more rows than have all their pairs evaluated)
    base = rng.standard_normal((N, d)).astype(np.float32)
    with_outlier = np.concatenate([base, np.full((1, d), 1.0e12, dtype=np.float32)])
    per_row = []
    for X in (base, with_outlier):
        Xd = torch.from_numpy(np.ascontiguousarray(X)).cuda()
        n = X.shape[0]
        plain = lib.knn_graph(Xd, k, fp32_filter=True)
        for got in (lib.knn_graph(Xd, k), lib.knn_graph(Xd, k, panel_order=True)):
            torch.cuda.synchronize()
            assert torch.equal(plain[0], got[0]) and torch.equal(plain[1], got[1])
        per_row.append([lib.slhc(Xd, k, prune=False, panel_order=p)["stats"]["knn_filter_survivors"] / n for p in (False, True)])
    print(f"  pairs passed per row, engine and list kernels: {per_row[0]} without the outlier, {per_row[1]} with it", flush=True)
    for without, with_it in zip(*per_row):
        assert k <= without < N / 8 and k <= with_it <= 2.0 * without + 20


def test_bf16_mfma_error_stays_within_what_the_slack_allows(lib):
    """split_slack_coefficient budgets 16 * 2^-24 of the sum of magnitudes per v_mfma_f32_32x32x16_bf16 (one unit
    per product).  Measured behaviour of the instruction: its 16 products and the accumulator are aligned to the
    largest of them, cut off half a unit below that one's last place, added exactly and rounded to nearest, i.e.
    at most 8.5 * 2^-23 of the sum of magnitudes in theory and about 2 in practice.  Checked here against exact
    float64 sums on values of equal and of widely different magnitudes, with and without cancellation, and on the
    worst pattern found by hand: the error must stay below half the budget of 8 * 2^-23."""
    g = torch.Generator().manual_seed(77)
    T = 1 << 18
    worst = 0.0
    for spread in (0, 2, 4, 10, 24, 30):
        def draw(shape):
            v = (1.0 + torch.rand(shape, generator=g)) * torch.exp2(-torch.randint(0, spread + 1, shape, generator=g).float())
            sign = torch.where(torch.rand(shape, generator=g) < 0.5, -1.0, 1.0) if spread != 2 else 1.0
            return (v * sign).to(torch.bfloat16).float()
        A, B = draw((T, 16)), draw((T, 16))
        C = (1.0 + torch.rand((T,), generator=g)) * torch.exp2(torch.randint(-4, 5, (T,), generator=g).float())
        C[::7] = 0.0
        D = lib.probe_bf16_mfma_values(A.cuda(), B.cuda(), C.cuda()).cpu().double()
        prod = A.double() * B.double()
        exact = C.double() + prod.sum(dim=1)                       # 17 terms of at most 24 bits each: exact in float64
        mags = C.double().abs() + prod.abs().sum(dim=1)
        rel = ((D - exact).abs() / (mags * 2.0 ** -23)).max().item()
        print(f"bf16 MFMA, exponent spread {spread}: worst error {rel:.3f} x 2^-23 x sum of magnitudes", flush=True)
        worst = max(worst, rel)
    # one product of 1 beside fifteen of 2^-25 (a quarter of a unit in its last place): the seven that share its
    # half of the instruction are cut off, the other eight add up to two units
    A = torch.full((1, 16), 2.0 ** -12); B = torch.full((1, 16), 2.0 ** -13)
    A[0, 0] = 1.0; B[0, 0] = 1.0
    D = lib.probe_bf16_mfma_values(A.cuda(), B.cuda(), torch.zeros(1).cuda()).cpu().double().item()
    err = abs(D - (1.0 + 15 * 2.0 ** -25)) / 2.0 ** -23
    print(f"one large product and fifteen small ones: off by {err:.3f} units", flush=True)
    assert worst <= 4.0 and err <= 4.0


# ----------------------------------------------------------------------------- default entry point
def test_default_entry_point_prunes_from_its_limit(lib):
    """slhc_slhc runs the every-tile path below SLHC_AUTO_PRUNE_MIN_ROWS rows and the pruned one from there
    on; the trees are those of the explicit flags either way."""
    for n in (3000, 24575, 24576):
        X, _, k = gen.make("c2", n=n)
        Xd = torch.from_numpy(X).cuda()
        auto = lib.slhc(Xd, k, prune=None)
        assert bool(auto["stats"]["pruned"]) == (n >= 24576)
        other = lib.slhc(Xd, k, prune=not auto["stats"]["pruned"])
        for name_ in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
            assert torch.equal(auto[name_], other[name_]), name_


# ----------------------------------------------------------------------------- k-NN sweeps split into candidate ranges
@pytest.mark.parametrize("N,d,k", [(4096, 16, 16), (777, 8, 5), (2000, 128, 64), (16384, 64, 32), (9000, 100, 33),
                                    (32768, 4, 2), (300, 4, 3)])
def test_knn_candidate_ranges_equal_unsplit(lib, N, d, k):
    """With fewer query panels than half the workgroup slots the every-tile k-NN sweep (k > 1) splits the
    candidate tiles into up to 16 ranges, one work item per (panel, range), and a merge kernel picks the k
    smallest of a row's lists (the paper's multi-block row epilogue, App. A, without its mutex): the list kernels with float32
    products, with split ones in panel order, and in the smallest workspace.  The lists must equal, bit for bit, those of the
    half-precision engine, which keeps none per range, with and without a workspace, and sampled rows must equal the oracle's."""
    rng = np.random.default_rng(N + d + k)
    X = rng.standard_normal((N, d)).astype(np.float32)
    X[rng.integers(0, N, size=N // 20)] = X[rng.integers(0, N, size=N // 20)]        # duplicates: ties by index
    Xd = torch.from_numpy(X).cuda()
    idx, dist = lib.knn_graph(Xd, k)
    ref = (torch.empty((N, k), dtype=torch.int32, device="cuda"), torch.empty((N, k), dtype=torch.float32, device="cuda"))
    lib.knn_graph_static(Xd, k, ref)
    torch.cuda.synchronize()
    assert torch.equal(idx, ref[0]) and torch.equal(dist, ref[1])
    for got in (lib.knn_graph(Xd, k, fp32_filter=True), lib.knn_graph(Xd, k, panel_order=True), knn_by_list_kernels(lib, Xd, k)):
        torch.cuda.synchronize()
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    rows = rng.choice(N, size=min(N, 200), replace=False)
    check_knn(X, k, idx.cpu().numpy()[rows], dist.cpu().numpy()[rows], rows=rows, min_exact=0.9)


# ----------------------------------------------------------------------------- 1-NN between two matrices
# The oracle has no two-matrix search of its own; its cross-colour 1-NN on the stacked matrix
# [Q; Y] with colour 0 for the query rows and 1 for the index rows is the same definition.
def check_fused_1nn(lib, Q, Y, min_exact):
    m, n = Q.shape[0], Y.shape[0]
    gi, gd = lib.fused_1nn(torch.from_numpy(Q).cuda(), torch.from_numpy(Y).cuda())
    torch.cuda.synchronize()
    gi, gd = gi.cpu().numpy(), gd.cpu().numpy()
    XY = np.concatenate([Q, Y])
    colour = np.concatenate([np.zeros(m, np.int32), np.ones(n, np.int32)])
    oi, od = oracle.cross_1nn(XY, colour, np.arange(m, dtype=np.int32))
    oi = oi - m
    assert gi.min() >= 0 and gi.max() < n
    assert close(gd, od, RTOL_DIST).all()
    true_d = pair_dist64(XY, np.arange(m), gi + m)
    assert close(gd, true_d, RTOL_DIST).all()
    assert (gi == oi).mean() >= min_exact


@pytest.mark.parametrize("m,n,d", [(100, 20000, 64), (1000, 20000, 128), (3000, 10000, 256), (1, 700, 8),
                                   (130, 129, 20), (257, 5, 33)])
def test_fused_1nn_few_queries(lib, m, n, d):
    # shapes of the paper's 1-NN benchmark, scaled: few queries against a large index (the index
    # rows are split over workgroups and merged), plus ragged and tiny cases
    print(f"fused 1-NN m={m} n={n} d={d}", flush=True)
    rng = np.random.default_rng(m * 7 + d)
    Y = rng.standard_normal((n, d)).astype(np.float32)
    Q = rng.standard_normal((m, d)).astype(np.float32)
    check_fused_1nn(lib, Q, Y, 0.999)


def test_fused_1nn_finds_itself_and_ties(lib):
    Y = gen.integer_lattice(7, 3, seed=2)                  # exact ties: smallest index must win
    Q = Y[::5].copy()
    gi, gd = lib.fused_1nn(torch.from_numpy(Q).cuda(), torch.from_numpy(Y).cuda())
    assert (gd.cpu().numpy() == 0.0).all()
    assert np.array_equal(gi.cpu().numpy(), np.arange(Y.shape[0])[::5])
    Q2 = (Q + np.float32(0.5)).astype(np.float32)          # equidistant from 8 lattice points
    XY = np.concatenate([Q2, Y])
    colour = np.concatenate([np.zeros(Q2.shape[0], np.int32), np.ones(Y.shape[0], np.int32)])
    oi, od = oracle.cross_1nn(XY, colour, np.arange(Q2.shape[0], dtype=np.int32))
    gi, gd = lib.fused_1nn(torch.from_numpy(Q2).cuda(), torch.from_numpy(Y).cuda())
    assert np.array_equal(gi.cpu().numpy(), oi - Q2.shape[0])
    assert np.array_equal(gd.cpu().numpy().astype(np.float64), od)


# ----------------------------------------------------------------------------- CSR spanning forest
# Under the strict edge order (w, lo, hi) the forest is unique: integer work, compared exactly.
def check_csr_msf(lib, offsets, indices, weights):
    got = lib.csr_msf(torch.from_numpy(offsets).cuda(), torch.from_numpy(indices).cuda(),
                      torch.from_numpy(weights).cuda())
    lo, hi, w, comp = oracle.csr_msf(offsets, indices, weights)
    assert np.array_equal(got["mst_src"].cpu().numpy(), lo)
    assert np.array_equal(got["mst_dst"].cpu().numpy(), hi)
    assert np.array_equal(got["mst_w"].cpu().numpy(), w)
    col = got["colours"].cpu().numpy()
    pairs = set(zip(col.tolist(), comp.tolist()))
    assert len(pairs) == len(set(comp.tolist())) == len(set(col.tolist()))
    assert (col[col] == col).all()                       # a colour is a vertex of its own component
    return got


@pytest.mark.parametrize("side,integer_weights", [(40, False), (300, False), (300, True), (700, False)])
def test_csr_msf_road_graphs(lib, side, integer_weights):
    print(f"csr msf side={side} integer_weights={integer_weights}", flush=True)
    offsets, indices, weights = gen.road_graph(side, seed=side, integer_weights=integer_weights)
    got = check_csr_msf(lib, offsets, indices, weights)
    assert 1 <= got["rounds"] <= int(np.ceil(np.log2(side * side))) + 2


def test_csr_msf_complete_graph_equals_point_mst(lib):
    # the complete squared-L2 graph of a point set, fed as CSR: same tree as the point pipeline
    X, _, k = gen.make("c1", n=600)
    N = X.shape[0]
    D = ((X[:, None, :].astype(np.float64) - X[None, :, :].astype(np.float64)) ** 2).sum(-1).astype(np.float32)
    src, dst = np.nonzero(~np.eye(N, dtype=bool))
    offsets = (np.arange(N + 1) * (N - 1)).astype(np.int32)
    got = check_csr_msf(lib, offsets, dst.astype(np.int32), D[src, dst])
    out = lib.slhc(torch.from_numpy(X).cuda(), k)
    assert np.array_equal(got["mst_src"].cpu().numpy(), out["mst_src"].cpu().numpy())
    assert np.array_equal(got["mst_dst"].cpu().numpy(), out["mst_dst"].cpu().numpy())


def test_csr_msf_degenerate_and_errors(lib):
    z = lambda a, dt: torch.tensor(a, dtype=dt, device="cuda")
    # no edges at all: every vertex its own component
    got = lib.csr_msf(z([0, 0, 0, 0], torch.int32), z([], torch.int32), z([], torch.float32))
    assert got["mst_src"].numel() == 0 and got["colours"].tolist() == [0, 1, 2]
    # self loops and parallel edges of different weight
    offsets = np.array([0, 3, 6], dtype=np.int32)
    indices = np.array([0, 1, 1, 0, 0, 1], dtype=np.int32)
    weights = np.array([0.5, 3.0, 2.0, 3.0, 2.0, 0.25], dtype=np.float32)
    got = check_csr_msf(lib, offsets, indices, weights)
    assert got["mst_w"].tolist() == [2.0]
    # zero weights and duplicates of them
    offsets, indices, weights = gen.road_graph(30, seed=9, integer_weights=True)
    check_csr_msf(lib, offsets, indices, (weights - 1.0).astype(np.float32) * (weights < 4))
    for bad_w in (-1.0, float("nan"), float("inf")):
        with pytest.raises(lib.SlhcError) as e:
            lib.csr_msf(z([0, 1, 2], torch.int32), z([1, 0], torch.int32), z([bad_w, bad_w], torch.float32))
        assert e.value.status == 1
    with pytest.raises(lib.SlhcError) as e:
        lib.csr_msf(z([0, 1, 2], torch.int32), z([1, 7], torch.int32), z([1.0, 1.0], torch.float32))
    assert e.value.status == 1
    with pytest.raises(lib.SlhcError) as e:
        lib.csr_msf(z([0, 2, 1], torch.int32), z([1, 0], torch.int32), z([1.0, 1.0], torch.float32))
    assert e.value.status == 1


# ----------------------------------------------------------------------------- flat clusters
# Integer work: labels must equal the oracle's exactly when both cut the same dendrogram.
@pytest.mark.parametrize("name,n", [("c1", None), ("c2", 20000), ("c5", 30000)])
def test_flat_clusters_match_oracle(lib, name, n):
    X, _, k = gen.make(name, n=n)
    N = X.shape[0]
    out = lib.slhc(torch.from_numpy(X).cuda(), k)
    children = out["children"].cpu().numpy()
    for nc in (1, 2, 3, 10, 777, N // 3, N - 1, N):
        print(f"flat clusters {name} N={N} n_clusters={nc}", flush=True)
        got = lib.flat_clusters(out["children"], nc)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), oracle.flat_clusters(children, nc)), nc


def test_flat_clusters_deep_chain_and_tiny(lib):
    # increasing gaps on a line: the dendrogram is one chain of depth N-1 (worst case for walking up)
    X, _ = gen.increasing_gaps_line(5000, 3, seed=1)
    out = lib.slhc(torch.from_numpy(X).cuda(), 4)
    children = out["children"].cpu().numpy()
    for nc in (1, 2, 50, 4999, 5000):
        got = lib.flat_clusters(out["children"], nc).cpu().numpy()
        assert np.array_equal(got, oracle.flat_clusters(children, nc)), nc
    ch = torch.tensor([[0, 1]], dtype=torch.int32, device="cuda")          # N = 2
    assert lib.flat_clusters(ch, 1).tolist() == [0, 0]
    assert lib.flat_clusters(ch, 2).tolist() == [0, 1]
    with pytest.raises(lib.SlhcError) as e:
        lib.flat_clusters(ch, 3)
    assert e.value.status == 1
    with pytest.raises(lib.SlhcError) as e:
        lib.flat_clusters(ch, 0)
    assert e.value.status == 1


def test_flat_clusters_recover_the_blobs(lib):
    # well separated blobs: cutting at the number of blobs gives back the generator's labels
    X, labels, k = gen.make("c1")
    out = lib.slhc(torch.from_numpy(X).cuda(), k)
    got = lib.flat_clusters(out["children"], int(labels.max()) + 1).cpu().numpy()
    pairs = set(zip(got.tolist(), labels.tolist()))
    assert len(pairs) == int(labels.max()) + 1


# ----------------------------------------------------------------------------- full size (c5)
def test_c5_full_size_pruned_equals_every_tile(lib):
    """c5 at its full size (2M x 32, k=8; 20 000 small blobs, exact duplicates): sampled rows of the
    k-NN graph against the oracle, and the pruned path against the every-tile path bit for bit."""
    X, _, k = gen.make("c5")
    N = X.shape[0]
    Xd = torch.from_numpy(X).cuda()
    print("c5 full: knn", flush=True)
    idx, dist = lib.knn_graph(Xd, k)
    idx_p, dist_p = lib.knn_graph(Xd, k, prune=True)
    torch.cuda.synchronize()
    assert torch.equal(idx, idx_p) and torch.equal(dist, dist_p)
    gi, gd = idx.cpu().numpy(), dist.cpu().numpy()
    rows = np.random.default_rng(55).choice(N, size=256, replace=False)
    check_knn(X, k, gi[rows], gd[rows], rows=rows, min_exact=0.9)
    del idx_p, dist_p
    print("c5 full: slhc", flush=True)
    a = lib.slhc(Xd, k, prune=False)
    b = lib.slhc(Xd, k, prune=True)
    for name_ in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(a[name_], b[name_]), name_
    w = b["mst_w"].cpu().numpy()
    src, dst = b["mst_src"].cpu().numpy(), b["mst_dst"].cpu().numpy()
    es = np.random.default_rng(56).choice(N - 1, size=200_000, replace=False)
    assert close(w[es], pair_dist64(X, src[es], dst[es]), RTOL_DIST).all()
    assert int(b["sizes"][-1]) == N
    # the 1 % exact copies give at least that many zero-weight tree edges
    assert int((w == 0.0).sum()) >= 15_000
    print("c5 full: tree properties", flush=True)
    check_tree_properties(X, k, gi, b, np.random.default_rng(57))


# ----------------------------------------------------------------------------- sweeps range by range
@pytest.mark.parametrize("N,d,k", [(270_000, 64, 8), (263_000, 32, 5), (300_001, 128, 33), (262_144, 96, 1)])
def test_range_order_equals_panel_order(lib, N, d, k):
    """Every-tile k-NN sweeps of the list kernels of at least four panels per workgroup slot hand out their work range by range
    and carry a panel's lists from range to range through the output arrays; the lists (split products in the smallest
    workspace, float32 products) must equal those of the sweep that takes one panel at a time (split and float32 products) and
    of the half-precision engine, and sampled rows must equal the oracle's."""
    rng = np.random.default_rng(N + d)
    centres = rng.uniform(-20, 20, size=(200, d))
    X = (centres[rng.integers(0, 200, size=N)] + rng.standard_normal((N, d))).astype(np.float32)
    X[rng.integers(0, N, size=500)] = X[rng.integers(0, N, size=500)]          # some exact copies
    Xd = torch.from_numpy(X).cuda()
    print("range order", N, d, k, flush=True)
    a = knn_by_list_kernels(lib, Xd, k)
    e = lib.knn_graph(Xd, k)
    torch.cuda.synchronize()
    assert torch.equal(a[0], e[0]) and torch.equal(a[1], e[1])
    for fp32 in (False, True):
        b = lib.knn_graph(Xd, k, panel_order=True, fp32_filter=fp32)
        torch.cuda.synchronize()
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    c = lib.knn_graph(Xd, k, fp32_filter=True)
    torch.cuda.synchronize()
    assert torch.equal(a[0], c[0]) and torch.equal(a[1], c[1])
    rows = rng.choice(N, size=96, replace=False)
    check_knn(X, k, a[0].cpu().numpy()[rows], a[1].cpu().numpy()[rows], rows=rows, min_exact=0.99)


# ----------------------------------------------------------------------------- full size (headline)
def test_headline_full_size_properties(lib):
    """c3 at its full size (1M x 128, k=32), in the launch configuration bench.py times.  The
    oracle cannot run the whole problem, so: sampled rows of the k-NN graph are checked one by one
    against it, sampled reported pairs are recomputed in float64, and the tree is checked through
    properties that hold at any size (spanning, weights of the returned pairs, the nearest
    neighbour of every sampled vertex is a tree edge, no sampled pair is closer than the largest
    edge on its tree path)."""
    X, _, k = gen.make("c3")
    N = X.shape[0]
    Xd = torch.from_numpy(X).cuda()
    print("headline: knn", flush=True)
    idx, dist = lib.knn_graph(Xd, k)
    torch.cuda.synchronize()
    gi, gd = idx.cpu().numpy(), dist.cpu().numpy()
    rng = np.random.default_rng(99)
    rows = rng.choice(N, size=192, replace=False)
    check_knn(X, k, gi[rows], gd[rows], rows=rows, min_exact=0.999)
    pr = rng.integers(0, N, size=400_000)
    pc = rng.integers(0, k, size=400_000)
    assert close(gd[pr, pc], pair_dist64(X, pr, gi[pr, pc]), RTOL_DIST).all()
    assert (np.diff(gd.astype(np.float64), axis=1) >= 0).all()
    assert not (gi == np.arange(N)[:, None]).any()

    print("headline: pruned knn", flush=True)
    idx_p, dist_p = lib.knn_graph(Xd, k, prune=True)
    torch.cuda.synchronize()
    assert torch.equal(idx, idx_p) and torch.equal(dist, dist_p)
    del idx_p, dist_p
    print("headline: knn panel by panel by the list kernels, split and float32 products", flush=True)
    for fp32 in (False, True):
        idx_p, dist_p = lib.knn_graph(Xd, k, panel_order=True, fp32_filter=fp32)
        torch.cuda.synchronize()
        assert torch.equal(idx, idx_p) and torch.equal(dist, dist_p)
        del idx_p, dist_p

    print("headline: slhc", flush=True)
    out = lib.slhc(Xd, k)                      # with tile pruning (the default)
    print("stats", out["stats"], flush=True)
    brute = lib.slhc(Xd, k, prune=False)       # every tile multiplied: what bench.py's roofline step times
    print("stats (every tile)", brute["stats"], flush=True)
    for name_ in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(out[name_], brute[name_]), name_
    del brute
    brute = lib.slhc(Xd, k, prune=False, panel_order=True)     # connection sweeps panel by panel as well
    for name_ in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(out[name_], brute[name_]), name_
    del brute
    check_tree_properties(X, k, gi, out, rng)


# ----------------------------------------------------------------------------- full size (c2, c4)
def test_c2_full_size_tree_against_prim(lib):
    """c2 at its full size (100k x 64, k=32): the whole tree and dendrogram against the oracle's dense
    Prim (about a minute of host time), through both the pruned and the every-tile path."""
    X, _, k = gen.make("c2")
    Xd = torch.from_numpy(X).cuda()
    print("c2 full: slhc on the GPU, then the oracle's Prim on the host", flush=True)
    out = lib.slhc(Xd, k)
    brute = lib.slhc(Xd, k, prune=False)
    for name_ in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(out[name_], brute[name_]), name_
    check_slhc(X, out, tie_free=True)


def test_c4_full_size_properties(lib):
    """c4 at its full size (250k x 784, k=16), the half-precision engine's widest case: sampled rows of the k-NN graph against the oracle, sampled
    reported pairs recomputed, and the tree checked through the properties that hold at any size."""
    X, _, k = gen.make("c4")
    N = X.shape[0]
    Xd = torch.from_numpy(X).cuda()
    print("c4 full: knn", flush=True)
    idx, dist = lib.knn_graph(Xd, k)
    torch.cuda.synchronize()
    gi, gd = idx.cpu().numpy(), dist.cpu().numpy()
    rng = np.random.default_rng(44)
    rows = rng.choice(N, size=256, replace=False)
    check_knn(X, k, gi[rows], gd[rows], rows=rows, min_exact=0.999)
    pr = rng.integers(0, N, size=200_000)
    pc = rng.integers(0, k, size=200_000)
    assert close(gd[pr, pc], pair_dist64(X, pr, gi[pr, pc]), RTOL_DIST).all()
    assert (np.diff(gd.astype(np.float64), axis=1) >= 0).all()
    assert not (gi == np.arange(N)[:, None]).any()
    assert gi.min() >= 0 and gi.max() < N
    print("c4 full: slhc", flush=True)
    out = lib.slhc(Xd, k)
    print("stats", out["stats"], flush=True)
    T = (N + 127) // 128
    assert out["stats"]["knn_tile_steps"] == T * T          # every pair of tiles is multiplied
    check_tree_properties(X, k, gi, out, rng, n_weights=100_000)


# ----------------------------------------------------------------------------- streaming kernel, many panels
# More than 512 query panels (65 536 rows): every workgroup of the streaming sweep kernel (d > 128; the list kernels' way, which
# the smallest workspace asks for) then loops over several work items.  All list widths of that kernel are instantiated.  The
# half-precision engine gives the same lists.
@pytest.mark.parametrize("N,d,k", [(70_000, 132, 16), (70_000, 132, 33), (66_500, 30, 20), (66_000, 30, 5),
                                   (66_000, 130, 1)])
def test_streaming_kernel_many_panels(lib, N, d, k):
    print(f"streaming sweep N={N} d={d} k={k}", flush=True)
    rng = np.random.default_rng(N + d + k)
    centres = rng.uniform(-10, 10, size=(40, d))
    X = (centres[rng.integers(0, 40, size=N)] + rng.standard_normal((N, d))).astype(np.float32)
    gi, gd = gpu_knn(lib, X, k)
    li, ld = knn_by_list_kernels(lib, torch.from_numpy(X).cuda(), k)
    assert np.array_equal(gi, li.cpu().numpy()) and np.array_equal(gd, ld.cpu().numpy())
    assert gi.min() >= 0 and gi.max() < N
    step = 10_000
    for s0 in range(0, N, step):                      # every reported pair, in float64
        r = np.arange(s0, min(N, s0 + step))
        assert close(gd[r], pair_dist64(X, r[:, None], gi[r]), RTOL_DIST).all()
    assert (np.diff(gd.astype(np.float64), axis=1) >= 0).all()
    rows = rng.choice(N, size=256, replace=False)
    rows[:4] = [0, 65_535, 65_536, N - 1]             # first and last panels of the first and second pass
    check_knn(X, k, gi[rows], gd[rows], rows=rows, min_exact=0.999)


def test_streaming_1nn_many_query_panels(lib):
    """The k = 1 variants of the streaming kernel with more than 512 query panels (in the smallest workspace), and the
    half-precision engine: the cross-colour 1-NN over all rows and the two-matrix 1-NN, sampled rows against the oracle."""
    N, d = 68_000, 132
    rng = np.random.default_rng(5)
    centres = rng.uniform(-10, 10, size=(30, d))
    lab = rng.integers(0, 30, size=N)
    X = (centres[lab] + rng.standard_normal((N, d))).astype(np.float32)
    colour = (lab % 7).astype(np.int32)
    print("streaming cross 1-NN, all rows", flush=True)
    Xd, cd = torch.from_numpy(X).cuda(), torch.from_numpy(colour).cuda()
    gi, gd = lib.cross_1nn(Xd, cd)
    li, ld = by_list_kernels(lib, cross_1nn_in(lib, Xd, cd, None, N))
    torch.cuda.synchronize()
    assert torch.equal(gi, li) and torch.equal(gd, ld)
    gi, gd = gi.cpu().numpy(), gd.cpu().numpy()
    assert gi.min() >= 0 and gi.max() < N and (colour[gi] != colour).all()
    assert close(gd, pair_dist64(X, np.arange(N), gi), RTOL_DIST).all()
    rows = rng.choice(N, size=300, replace=False)
    rows[:3] = [0, 65_536, N - 1]
    oi, od = oracle.cross_1nn(X, colour, rows.astype(np.int64))
    assert close(gd[rows], od, RTOL_DIST).all()
    assert (gi[rows] == oi).mean() >= 0.99
    print("streaming two-matrix 1-NN, 68 000 queries", flush=True)
    Y = (centres[rng.integers(0, 30, size=3000)] + rng.standard_normal((3000, d))).astype(np.float32)
    Yd = torch.from_numpy(Y).cuda()
    fi, fd = lib.fused_1nn(Xd, Yd)
    li, ld = by_list_kernels(lib, lambda ws: lib.fused_1nn(Xd, Yd, workspace=ws))
    torch.cuda.synchronize()
    assert torch.equal(fi, li) and torch.equal(fd, ld)
    fi, fd = fi.cpu().numpy(), fd.cpu().numpy()
    assert fi.min() >= 0 and fi.max() < 3000
    XY = np.concatenate([X, Y])
    assert close(fd, pair_dist64(XY, np.arange(N), fi + N), RTOL_DIST).all()
    col2 = np.concatenate([np.zeros(N, np.int32), np.ones(3000, np.int32)])
    oi, od = oracle.cross_1nn(XY, col2, rows.astype(np.int64))
    assert close(fd[rows], od, RTOL_DIST).all()
    assert (fi[rows] == oi - N).mean() >= 0.99


# ----------------------------------------------------------------------------- dendrogram on several host threads
def test_threaded_dendrogram_equals_oracle(lib):
    """From 200 000 rows on the library groups all but the heaviest sixteenth of the tree edges by the
    component they lie in without the heavy ones, and host threads work through the groups side by side.
    The result must be the sequential relabelling of the same sorted edges (paper Sec. 3.3.1), which is
    what the oracle computes: many blobs (many groups), one blob (one giant group), duplicates (ties)."""
    rng = np.random.default_rng(4242)
    cases = [dict(N=300_000, d=8, k=4, nb=500, spread=50.0, sigma=1.0, dup=0),
             dict(N=250_000, d=4, k=4, nb=1, spread=0.0, sigma=1.0, dup=0),
             dict(N=220_000, d=16, k=6, nb=40, spread=30.0, sigma=1.0, dup=30_000)]
    for c in cases:
        N, d, k = c["N"], c["d"], c["k"]
        centres = rng.uniform(-c["spread"], c["spread"], size=(c["nb"], d)) if c["nb"] > 1 else np.zeros((1, d))
        X = (centres[rng.integers(0, c["nb"], size=N)] + c["sigma"] * rng.standard_normal((N, d))).astype(np.float32)
        if c["dup"]:
            X[rng.integers(0, N, size=c["dup"])] = X[rng.integers(0, N, size=c["dup"])]
        print(f"threaded dendrogram: N={N} d={d} k={k} blobs={c['nb']} duplicates={c['dup']}", flush=True)
        out = lib.slhc(torch.from_numpy(np.ascontiguousarray(X)).cuda(), k)
        src, dst, w = (out[n].cpu().numpy() for n in ("mst_src", "mst_dst", "mst_w"))
        ref = oracle.dendrogram(src, dst, w.astype(np.float64), N)
        assert np.array_equal(ref["src"], src) and np.array_equal(ref["dst"], dst), "edge order differs from (w, lo, hi)"
        assert np.array_equal(out["children"].cpu().numpy(), ref["children"])
        assert np.array_equal(out["sizes"].cpu().numpy(), ref["sizes"])
        assert np.array_equal(out["heights"].cpu().numpy(), w)


# ----------------------------------------------------------------------------- two-phase connection rounds
def test_split_connection_rounds_are_identical(lib):
    """SLHC_SPLIT_ROUNDS runs every pruned connection round of 256 rows or more in two phases (a sample
    of the row panels first, the other rows under the thresholds that leaves): the tree must equal the
    every-tile path's bit for bit on seeded random shapes, and the oracle's on the small ones."""
    rng = np.random.default_rng(777)
    split_seen = 0
    for case in range(20):
        N = int(rng.integers(600, 25_000)) if case % 3 else int(rng.integers(600, 3000))
        d = int(rng.choice([4, 8, 16, 32, 64, 100, 128]))
        k = int(rng.integers(1, 33))
        nb = int(rng.integers(2, 120))
        spread = float(rng.choice([3.0, 20.0, 1000.0]))
        sigma = float(rng.choice([0.05, 1.0, 3.0]))
        centres = rng.uniform(-spread, spread, size=(nb, d))
        X = (centres[rng.integers(0, nb, size=N)] + sigma * rng.standard_normal((N, d))).astype(np.float32)
        ties = False
        if rng.random() < 0.3:
            m = N // 10
            X[rng.integers(0, N, size=m)] = X[rng.integers(0, N, size=m)]
            ties = True
        print(f"split rounds case {case}: N={N} d={d} k={k} blobs={nb} spread={spread} sigma={sigma} ties={ties}", flush=True)
        Xd = torch.from_numpy(np.ascontiguousarray(X)).cuda()
        a = lib.slhc(Xd, k, prune=False)
        b = lib.slhc(Xd, k, prune=True, split_rounds=True)
        c = lib.slhc(Xd, k, prune=True)
        for name_ in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
            assert torch.equal(a[name_], b[name_]), name_
            assert torch.equal(a[name_], c[name_]), name_
        # a split round drops the rows the first phase made unnecessary, so it queries fewer rows
        if b["stats"]["connect_query_rows"] != c["stats"]["connect_query_rows"]:
            split_seen += 1
        if N <= 3000:
            check_slhc(np.ascontiguousarray(X), b, tie_free=not ties)
    print("cases in which the split changed the number of queried rows:", split_seen, flush=True)
    assert split_seen >= 3


# ----------------------------------------------------------------------------- split panel scans
def test_split_panel_scans_are_identical(lib):
    """SLHC_SPLIT_SCANS splits every query panel's scan of the candidate tiles in the pruned connection
    sweeps into 5 work items that meet in a 64-bit atomic minimum and adopt each other's finds: the tree
    must equal the every-tile path's bit for bit on seeded random shapes (blobs, duplicates, 1 to 32
    neighbours, 4 to 128 features), together with the two-phase rounds too, and the oracle's on the small
    ones.  The split must really have run: its work items multiply a different number of tiles."""
    rng = np.random.default_rng(31337)
    changed = 0
    for case in range(20):
        N = int(rng.integers(600, 30_000)) if case % 3 else int(rng.integers(600, 3000))
        d = int(rng.choice([4, 8, 16, 32, 64, 100, 128]))
        k = int(rng.integers(1, 33))
        nb = int(rng.integers(2, 150))
        spread = float(rng.choice([3.0, 20.0, 1000.0]))
        sigma = float(rng.choice([0.05, 1.0, 3.0]))
        centres = rng.uniform(-spread, spread, size=(nb, d))
        X = (centres[rng.integers(0, nb, size=N)] + sigma * rng.standard_normal((N, d))).astype(np.float32)
        ties = False
        if rng.random() < 0.3:
            m = N // 10
            X[rng.integers(0, N, size=m)] = X[rng.integers(0, N, size=m)]
            ties = True
        print(f"split scans case {case}: N={N} d={d} k={k} blobs={nb} spread={spread} sigma={sigma} ties={ties}", flush=True)
        Xd = torch.from_numpy(np.ascontiguousarray(X)).cuda()
        a = lib.slhc(Xd, k, prune=False)
        b = lib.slhc(Xd, k, prune=True, split_scans=True)
        c = lib.slhc(Xd, k, prune=True, split_scans=True, split_rounds=True)
        plain = lib.slhc(Xd, k, prune=True)
        for name_ in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
            assert torch.equal(a[name_], b[name_]), name_
            assert torch.equal(a[name_], c[name_]), name_
        if b["stats"]["pruned"] and b["stats"]["connect_tile_steps"] != plain["stats"]["connect_tile_steps"]:
            changed += 1
        if N <= 3000:
            check_slhc(np.ascontiguousarray(X), b, tie_free=not ties)
    print("cases in which the split scans multiplied a different number of tiles:", changed, flush=True)
    assert changed >= 5


# ----------------------------------------------------------------------------- non-finite input, bad rows
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf"), 3e20])
def test_nonfinite_rows(lib, bad):
    """A row with a NaN, an infinity or a squared norm beyond float32: the synchronous entry points
    return SLHC_NONFINITE (5); the asynchronous k-NN never writes an index outside -1 .. N-1, never
    lists the bad row, and gives every other row the list it has without that row."""
    X, _, k = gen.make("c1", n=3000)
    N = X.shape[0]
    Xb = X.copy()
    Xb[1234, 3] = bad
    Xd = torch.from_numpy(Xb).cuda()
    for prune in (True, False):
        with pytest.raises(lib.SlhcError) as e:
            lib.slhc(Xd, k, prune=prune)
        assert e.value.status == 5
    with pytest.raises(lib.SlhcError) as e:
        lib.knn_graph(Xd, k, prune=True)
    assert e.value.status == 5
    idx, dist = lib.knn_graph(Xd, k)
    torch.cuda.synchronize()
    gi = idx.cpu().numpy()
    assert gi.min() >= -1 and gi.max() < N
    others = np.arange(N) != 1234
    assert not (gi[others] == 1234).any()
    Xf = X.copy()
    Xf[1234] = 1e4                                     # far from everything: in nobody's list either
    ri, rd = gpu_knn(lib, Xf, k)
    assert np.array_equal(gi[others], ri[others])
    assert np.array_equal(dist.cpu().numpy()[others], rd[others])
    # the library is unharmed: the clean input still works
    check_slhc(X, lib.slhc(torch.from_numpy(X).cuda(), k), tie_free=True)


def test_cross_1nn_rows_out_of_range(lib):
    """Entries of the device row list outside [0, N) are not dereferenced and are answered with -1, +inf;
    the other rows are answered as usual (both sweep kernels)."""
    for d in (16, 33):
        X = np.random.default_rng(d).standard_normal((2000, d)).astype(np.float32)
        colour = (np.arange(2000) % 5).astype(np.int32)
        rows = np.array([5, -1, 1999, 2000, 17, 2**31 - 1, -2**31, 700] + list(range(300)), dtype=np.int32)
        gi, gd = lib.cross_1nn(torch.from_numpy(X).cuda(), torch.from_numpy(colour).cuda(), torch.from_numpy(rows).cuda())
        torch.cuda.synchronize()
        gi, gd = gi.cpu().numpy(), gd.cpu().numpy()
        ok = (rows >= 0) & (rows < 2000)
        assert (gi[~ok] == -1).all() and np.isinf(gd[~ok]).all()
        oi, od = oracle.cross_1nn(X, colour, rows[ok].astype(np.int64))
        assert np.array_equal(gi[ok], oi) and close(gd[ok], od, RTOL_DIST).all()
