"""Rounds over lists of active vertices and roots, and the sort by the smaller ends (csr_kernels.hip), against the oracle's Kruskal:
graphs whose rounds, lists, hook chains and edge counts per vertex end differently."""
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


def csr(V, a, b, w, shuffled=None):
    src, dst, ww = np.r_[a, b], np.r_[b, a], np.r_[w, w].astype(np.float32)
    order = np.argsort(src, kind="stable") if shuffled is None else np.lexsort((shuffled.random(len(src)), src))
    offsets = np.r_[0, np.cumsum(np.bincount(src, minlength=V))].astype(np.int32)
    return offsets, dst[order].astype(np.int32), ww[order]


def check(lib, V, offsets, indices, weights):
    got = lib.csr_msf(*(torch.from_numpy(x).cuda() for x in (offsets, indices, weights)))
    torch.cuda.synchronize()
    lo, hi, w, comp = oracle.csr_msf(offsets, indices, weights)
    assert np.array_equal(got["mst_src"].cpu().numpy(), lo) and np.array_equal(got["mst_dst"].cpu().numpy(), hi)
    assert np.array_equal(got["mst_w"].cpu().numpy(), w.astype(np.float32))
    c = got["colours"].cpu().numpy()
    assert len(np.unique(c)) == V - len(lo) and np.array_equal(c[lo], c[hi]) and np.array_equal(c[c], c)


# one vertex with all tree edges, as the smaller and as the larger end, with ties and without
@pytest.mark.parametrize("V", [2, 33, 34, 35, 300, 70_000])
@pytest.mark.parametrize("hub", ["first", "last"])
@pytest.mark.parametrize("ties", [True, False])
def test_stars(lib, V, hub, ties):
    print(f"csr star V={V} hub={hub} ties={ties}", flush=True)
    rng = np.random.default_rng(V)
    a = np.zeros(V - 1, np.int64) if hub == "first" else np.full(V - 1, V - 1)
    b = np.arange(1, V) if hub == "first" else np.arange(V - 1)
    w = rng.integers(1, 4, V - 1) if ties else rng.permutation(V - 1) + 0.5
    check(lib, V, *csr(V, a, b, w, rng))


# vertices with as many tree edges to larger ones as are ordered in place, one less and one more, on both sides of the line from which on the
# sort takes the smaller ends first; the rest of the tree a chain between them
@pytest.mark.parametrize("V", [65_536, 65_537, 90_000])
@pytest.mark.parametrize("edges", [31, 32, 33])
@pytest.mark.parametrize("values", [1, 3, 1_000_000])
def test_edges_per_smaller_end(lib, V, edges, values):
    print(f"csr V={V}, {edges} edges per smaller end, {values} weights", flush=True)
    rng = np.random.default_rng(V + edges)
    n = V // (edges + 1)
    hubs, others = rng.permutation(n), n + rng.permutation(V - n)
    own = others[:n * (edges - 1)].reshape(n, edges - 1)
    link = others[n * (edges - 1):][:n]                          # the last edge of a hub; the next hub's, too, would be one too many
    a = np.r_[np.repeat(hubs, edges - 1), hubs, link[:-1]]
    b = np.r_[own.ravel(), link, own[1:, 0]]
    assert np.bincount(np.minimum(a, b), minlength=V)[:n].tolist() == [edges] * n
    check(lib, V, *csr(V, a, b, rng.integers(0, values, len(a)), rng))


# rows in no order, several edges between two vertices, self loops, vertices without edges, many trees; weights of few values and of many, 0 included;
# wavefronts with rows of 49 entries and more, from a few to all
@pytest.mark.parametrize("V,degree,values", [(1, 0, 1), (500, 0.4, 3), (3000, 1.0, 1), (5000, 3.0, 2), (20_000, 1.3, 1000), (100_000, 2.5, 10), (66_000, 8.0, 1_000_000),
                                             (60, 50.0, 1000), (300, 80.0, 3), (1500, 45.0, 1_000_000), (6000, 80.0, 1000), (70_000, 49.0, 10)])
def test_random_graphs(lib, V, degree, values):
    print(f"csr random V={V} degree={degree} values={values}", flush=True)
    rng = np.random.default_rng(V)
    E = int(V * degree / 2)
    a, b = rng.integers(0, V, E), rng.integers(0, V, E)
    w = rng.integers(0, values, E).astype(np.float32)
    a, b, w = np.r_[a, a[:E // 10]], np.r_[b, b[:E // 10]], np.r_[w, w[:E // 10] + 1]
    keep = a != b
    loops = rng.integers(0, V, V // 50)
    offsets, indices, weights = csr(V, np.r_[a[keep]], np.r_[b[keep]], w[keep], rng)
    if len(loops):                       # (one entry each)
        src = np.repeat(np.arange(V), np.diff(offsets))
        src, dst, ww = np.r_[src, loops], np.r_[indices, loops], np.r_[weights, np.full(len(loops), 0.0, np.float32)]
        order = np.argsort(src, kind="stable")
        offsets = np.r_[0, np.cumsum(np.bincount(src, minlength=V))].astype(np.int32)
        indices, weights = dst[order].astype(np.int32), ww[order].astype(np.float32)
    check(lib, V, offsets, indices, weights)


# rows that a thread reads and rows that a wavefront reads, side by side and far apart: lengths around the line between them and around the wavefront's
# steps; hubs whose tree edges are few, many and on either end.  (One launch, launches per round, the sort by the smaller ends.)
@pytest.mark.parametrize("V", [1500, 20_000, 90_000])
@pytest.mark.parametrize("spread", [1, 61])
@pytest.mark.parametrize("values", [3, 1_000_000])
def test_hubs(lib, V, spread, values):
    print(f"csr hubs V={V} spread={spread} values={values}", flush=True)
    rng = np.random.default_rng(V + spread)
    lengths = [0, 1, 3, 5, 31, 32, 33, 47, 48, 49, 51, 52, 53, 64, 128, 255, 256, 257, 260, 511, 1000, 1023, 1024, 1025, 1400]
    hubs = np.r_[np.arange(len(lengths)), V - 1 - np.arange(len(lengths))]
    hubs = np.where(hubs < V // 2, hubs * spread, V - 1 - (V - 1 - hubs) * spread)
    a = np.concatenate([np.full(n, h) for h, n in zip(hubs, lengths * 2)])
    b = np.concatenate([(h + 1 + rng.permutation(V - 1)[:n]) % V for h, n in zip(hubs, lengths * 2)])
    path = rng.permutation(V)[:V // 2]
    a, b = np.r_[a, path[:-1]], np.r_[b, path[1:]]
    check(lib, V, *csr(V, a, b, rng.integers(0, values, len(a)).astype(np.float32), rng))


# Entries that only one of the two rows has, or with another weight there: an error, never a forest that leaves a component in parts.
# A row of (neighbour, weight) per vertex.
ONE_SIDED = {
    "both edges of a tree's root": [[(3, 1), (1, 9)], [(2, 2)], [], []],
    "the only edge": [[(1, 1)], []],
    "a later round's": [[(1, .1), (2, 1)], [(0, .1)], [(3, .5)], [(2, .5)]],
    "two weights": [[(1, 1), (2, 2)], [(0, 3), (2, 4)], [(0, 2), (1, 4)]],
    "a cycle": [[(1, 1)], [(2, 2)], [(0, 3)]],
    "one of two with equal weights": [[(1, 1), (2, 1)], [(2, 1)], [(0, 1), (1, 1)]],
}


@pytest.mark.parametrize("case", ONE_SIDED)
@pytest.mark.parametrize("more", [0, 3000, 70_000])          # (as many vertices beside it: one launch, launches per round, the other sort)
def test_one_sided_entries(lib, case, more):
    print(f"csr one-sided: {case}, {more} more", flush=True)
    rows = ONE_SIDED[case]
    at = len(rows)
    a = np.arange(more - 1) if more else np.zeros(0, np.int64)
    offsets, indices, weights = csr(at + more, a + at, a + 1 + at, (a % 7 + 1).astype(np.float32)) if more else (np.zeros(at + 1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32))
    ends = np.cumsum([len(r) for r in rows])
    offsets = np.r_[0, ends, ends[-1] + offsets[at + 1:]].astype(np.int32)
    indices = np.r_[np.array([u for r in rows for u, _ in r]), indices].astype(np.int32)
    weights = np.r_[np.array([w for r in rows for _, w in r]), weights].astype(np.float32)
    with pytest.raises(lib.SlhcError, match="both rows"):
        lib.csr_msf(*(torch.from_numpy(x).cuda() for x in (offsets, indices, weights)))


def test_graph_stored_once(lib):
    rng = np.random.default_rng(5)
    V = 20_000
    a, b = rng.integers(0, V, 3 * V), rng.integers(0, V, 3 * V)
    lo, hi = np.minimum(a, b), np.maximum(a, b)
    order = np.argsort(lo, kind="stable")
    offsets = np.r_[0, np.cumsum(np.bincount(lo, minlength=V))].astype(np.int32)
    with pytest.raises(lib.SlhcError, match="both rows"):
        lib.csr_msf(*(torch.from_numpy(x).cuda() for x in (offsets, hi[order].astype(np.int32), rng.random(3 * V).astype(np.float32))))


# -0.0 is a weight of 0, also where the other row has +0.0
@pytest.mark.parametrize("V", [2, 40, 5000])
def test_negative_zero(lib, V):
    print(f"csr negative zero V={V}", flush=True)
    a = np.arange(V - 1)
    offsets, indices, weights = csr(V, a, a + 1, (a % 3).astype(np.float32))
    weights[np.flatnonzero(weights == 0)[::2]] = -0.0
    assert np.signbit(weights).any()
    check(lib, V, offsets, indices, weights)


# Rows of 80 entries cost the time of rows of 3 and a half more, twice or so in all (five times where few CUs read them, one thread a row)
def test_time_of_dense_graphs(lib):
    V, ms = 20_000, []
    rng = np.random.default_rng(3)
    for degree in (3, 80):
        a, b = rng.integers(0, V, V * degree // 2), rng.integers(0, V, V * degree // 2)
        keep = a != b
        graph = [torch.from_numpy(x).cuda() for x in csr(V, a[keep], b[keep], rng.random(keep.sum()).astype(np.float32))]
        least = float("inf")
        for _ in range(12):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            lib.csr_msf(*graph)
            end.record()
            end.synchronize()
            least = min(least, begin.elapsed_time(end))
        ms.append(least)
    assert ms[1] < 3.5 * ms[0], ms


# hook chains of a round from one to all vertices long: weights rising along paths of `run` vertices, which meet at their ends
@pytest.mark.parametrize("run", [2, 63, 64, 65, 66, 4097, 100_000])
def test_chains(lib, run):
    print(f"csr chains of {run}", flush=True)
    V = 100_000 // run * run
    a = np.arange(V - 1)
    w = np.where((a + 1) % run == 0, 1e6 + a, (a % run).astype(np.float64))
    check(lib, V, *csr(V, a, a + 1, w.astype(np.float32)))


# as many entries as the call takes: the last row ends on the last number of 32 bits.  A path whose edges are stored 256 times in every row, the
# weights in an order that makes chains of five vertices
def test_largest_entry_count(lib):
    V, L = 1 << 22, 512
    E = V * L - 1
    print(f"csr V={V} E={E}", flush=True)
    dev = torch.device("cuda")
    v = torch.arange(V, device=dev, dtype=torch.int32)
    path_w = (torch.arange(V - 1, device=dev, dtype=torch.int32) * 3 % 5 + 1).float()
    indices = torch.empty(V * L, dtype=torch.int32, device=dev)
    weights = torch.empty(V * L, dtype=torch.float32, device=dev)
    left, right = torch.where(v == 0, 1, v - 1), torch.where(v == V - 1, V - 2, v + 1)      # (the ends have one neighbour)
    for table, a, b in ((indices, left, right), (weights, path_w[left.minimum(v).long()], path_w[right.minimum(v).long()])):
        rows = table.view(V, L)
        rows[:, 0::2] = a[:, None]
        rows[:, 1::2] = b[:, None]
    offsets = (torch.arange(V + 1, device=dev, dtype=torch.int64) * L).clamp_(max=E).to(torch.int32)
    got = lib.csr_msf(offsets, indices[:E], weights[:E])
    torch.cuda.synchronize()
    order = torch.argsort(path_w, stable=True)
    assert torch.equal(got["mst_src"].long(), order) and torch.equal(got["mst_dst"].long(), order + 1) and torch.equal(got["mst_w"], path_w[order])
    assert bool((got["colours"] == got["colours"][0]).all())
