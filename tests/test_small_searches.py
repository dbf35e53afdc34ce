"""Searches small enough to evaluate every pair in registers (direct_kernels.hip): lists and trees against the float32-product list
kernels, bit for bit."""
import ctypes

import pytest

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    import paper_2306_16354_amd as slhc
    slhc.load_library()
    assert torch.cuda.is_available()
    return slhc


def rows(N, d, seed, spread=8.0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    centres = (2 * torch.rand((max(2, N // 300), d), generator=g, device="cuda") - 1) * spread
    return centres[torch.randint(len(centres), (N,), generator=g, device="cuda")] + torch.randn((N, d), generator=g, device="cuda")


def same_lists(lib, X, k, bad=()):
    """bad: rows that are not finite, which have no list and are in none."""
    want, got = lib.knn_graph(X, k, fp32_filter=True), lib.knn_graph(X, k)
    static = (torch.full_like(got[0], -7), torch.full_like(got[1], -7.0))
    lib.knn_graph_static(X, k, static)
    torch.cuda.synchronize()
    bad = torch.tensor(list(bad), dtype=torch.int64, device="cuda")
    fine = torch.ones(len(X), dtype=torch.bool, device="cuda")
    fine[bad] = False
    for idx, dist in (got, static):
        assert torch.equal(want[0][fine], idx[fine]) and torch.equal(want[1][fine], dist[fine])
        assert (idx[bad] == -1).all() and torch.isinf(dist[bad]).all() and not torch.isin(idx, bad.to(torch.int32)).any()


# every number of quads the kernel is made for, whole and in part, less than one quad; parts of a wavefront, of 512 rows and of the 1, 2 and 4
# times 512 a lane holds; one round of workgroups and several, one row per workgroup and eight; both ways to a limit (16 and 17 neighbours),
# all other rows; on both sides of the last search of its kind
@pytest.mark.gpu
@pytest.mark.parametrize("N,d,k", [
    (2, 1, 1), (3, 3, 2), (63, 4, 8), (65, 5, 64), (66, 2, 17), (255, 7, 16), (257, 8, 2), (511, 9, 30), (512, 15, 1), (513, 16, 16), (700, 17, 17), (769, 31, 40),
    (1024, 32, 9), (1025, 33, 3), (1100, 47, 12), (1281, 48, 64), (1535, 49, 5), (1537, 50, 10), (1300, 63, 7), (1793, 64, 33), (1000, 65, 4), (1409, 96, 21),
    (1025, 97, 6), (900, 127, 64), (1690, 128, 16), (2047, 36, 8), (2049, 20, 11), (2561, 24, 5), (3073, 12, 19), (3700, 6, 25), (4097, 1, 13), (4472, 8, 3), (4473, 8, 3),
])
def test_lists(lib, N, d, k):
    print(f"small k-NN N={N} d={d} k={k}", flush=True)
    assert lib.probe_knn_products(N, d, k) == (0.0 if N < 4473 else 1.0)
    same_lists(lib, rows(N, d, N + d), k)


# copies of a point by the tens and hundreds (as many as a row keeps and more, all rows equal), rows that are not finite or close to it, rows that do
# not begin on 16 bytes
@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["copies_30", "copies_130", "copies_600", "one_point", "lattice", "far_rows", "large", "not_finite", "out_of_reach", "odd_address"])
@pytest.mark.parametrize("N,d,k", [(900, 6, 20), (1700, 32, 8), (1300, 61, 64)])
def test_lists_of_unlike_rows(lib, kind, N, d, k):
    print(f"small k-NN, {kind}, N={N} d={d} k={k}", flush=True)
    assert lib.probe_knn_products(N, d, k) == 0.0
    X = rows(N, d, N)
    if kind.startswith("copies"):
        X = X[torch.arange(N, device="cuda") % (N // int(kind[7:]))].contiguous()
    elif kind == "one_point":
        X[:] = X[0].clone()
    elif kind == "lattice":
        X = (X / 4).round()
    elif kind == "far_rows":
        X[::70] *= 1e15
    elif kind == "large":
        X *= 3e17
        X[5] = 0.0
    elif kind == "not_finite":
        X[N // 3] = float("nan")
        X[N // 5, 2] = float("inf")
        X[N // 7] = 3e19
    elif kind == "out_of_reach":
        X *= 1e14
        X[:, 0] += 1.5e19
        X[:40:8, 0] -= 3e19                      # (five rows, each within reach of four others and of row 7: fewer than k)
        X[7] = 0.0
        X[9], X[N - 2] = float("nan"), 3e19
    elif kind == "odd_address":
        X = torch.cat([X.new_zeros(1), X.reshape(-1)])[1:].reshape(N, d)
        assert X.data_ptr() % 16 == 4
    bad = {"not_finite": [N // 3, N // 5, N // 7], "out_of_reach": [9, N - 2]}.get(kind, [])
    same_lists(lib, X, k, bad)
    assert kind != "out_of_reach" or torch.isinf(lib.knn_graph(X, k)[1][:40:8, 5:]).all()


# rows of large norms or one that is not finite cost a look at each row, not at each pair (which took 25 and 10 times as long)
@pytest.mark.gpu
@pytest.mark.parametrize("N,d,k", [(2048, 32, 8), (4000, 8, 8), (1300, 100, 8)])
def test_large_rows_take_no_longer(lib, N, d, k):
    print(f"small k-NN, time with large rows, N={N} d={d} k={k}", flush=True)
    X = rows(N, d, N)
    large, nan = X * 3e17, X.clone()
    large[5], nan[N // 2] = 0.0, float("nan")
    out = (torch.empty((N, k), dtype=torch.int32, device="cuda"), torch.empty((N, k), dtype=torch.float32, device="cuda"))

    def least(X):
        times = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(8):
                lib.knn_graph_static(X, k, out)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times[2:])
    plain, with_large, with_nan = least(X), least(large), least(nan)
    print(f"  {125 * plain:.1f} us, {125 * with_large:.1f} with large rows, {125 * with_nan:.1f} with a NaN", flush=True)
    assert with_large < 3 * plain and with_nan < 3 * plain


# the same where the pairs can be counted on the host: which searches go this way does not depend on a GPU
@pytest.mark.parametrize("N,d,k,products", [(2048, 32, 8, 0.0), (4472, 8, 3, 0.0), (4473, 8, 3, 1.0), (1690, 128, 16, 0.0), (1691, 128, 16, 1.0), (500, 129, 4, 1.0)])
def test_searches_that_multiply_nothing(N, d, k, products):
    import paper_2306_16354_amd as slhc
    lib = slhc.load_library()
    out = ctypes.c_double(-1.0)
    assert lib.slhc_probe_knn_products(N, d, k, ctypes.byref(out)) == 0 and out.value == products


# a workspace that is too small is one whichever search would run in it (refused before anything is launched)
@pytest.mark.parametrize("N,d,k", [(600, 4, 3), (1500, 50, 8), (2048, 32, 8), (4096, 15, 16), (1690, 127, 16)])
def test_small_trees_ask_for_no_less(N, d, k):
    import paper_2306_16354_amd as slhc
    lib = slhc.load_library()

    def refusal(flags):
        some = ctypes.c_void_p(256)
        rc = lib.slhc_slhc_opt(some, N, d, k, some, some, some, some, some, some, None, some, 256, None, flags)
        return rc, lib.slhc_last_error().decode()
    assert refusal(0)[0] == 3 and refusal(0) == refusal(slhc.binding.SLHC_FP32_FILTER)


# rounds of connecting components: clusters too far apart for the lists, several rounds, copies in other components, few and many queries; rows that
# are read as they are (16 columns) and with columns of zeros; a forest of one workgroup and of many
@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["clusters", "tight", "copies", "lattice", "large"])
@pytest.mark.parametrize("N,d,k", [(3, 2, 1), (70, 5, 3), (513, 16, 2), (1025, 33, 4), (1537, 64, 8), (2049, 7, 3), (3100, 16, 4), (3500, 30, 6), (1800, 128, 5), (12_500, 4, 6)])
def test_trees(lib, kind, N, d, k):
    print(f"small trees, {kind}, N={N} d={d} k={k}", flush=True)
    X = rows(N, d, N, 200.0)
    if kind == "tight":
        X = (X / 20).round() * 20 + 1e-2 * rows(N, d, N + 1, 0.0)
    elif kind == "copies":
        X = X[torch.arange(N, device="cuda") % (N // 9 + 2)].contiguous()
        X[::2] += 3000.0
    elif kind == "lattice":
        X = (X / 60).round()
    elif kind == "large":
        X *= 1e16
    want, got = lib.slhc(X, k, prune=False, fp32_filter=True), lib.slhc(X, k, prune=False)
    torch.cuda.synchronize()
    for key in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(want[key], got[key]), key


# pairs evaluated exactly, as they are reported: all of them, of rows with and without a copy in split halves; beyond the last such search
# the engine's few
@pytest.mark.gpu
@pytest.mark.parametrize("N,d,all_pairs", [(3, 1, True), (700, 16, True), (900, 50, True), (1100, 64, True), (600, 127, True), (9000, 50, False), (9000, 64, False)])
def test_evaluated_pairs_are_counted(lib, N, d, all_pairs):
    print(f"evaluated pairs N={N} d={d}", flush=True)
    count = lib.slhc(rows(N, d, N), 2, prune=False)["stats"]["knn_filter_survivors"]
    assert count == N * (N - 1) if all_pairs else 2 * N <= count < 100 * N


# the last clustering of a width that evaluates every pair, and the first that does not (4100 x 32 took 334 us instead of 275 with all pairs); where lists
# are long the engine takes longer (5000 x 16, k = 48, 402 us instead of 380)
@pytest.mark.gpu
@pytest.mark.parametrize("d,k,most", [(8, 4, 5120), (16, 4, 4608), (32, 4, 3072), (48, 4, 3072), (64, 4, 2560), (96, 4, 2048), (128, 4, 2048), (8, 23, 5120), (8, 24, 5632),
                                      (9, 39, 4608), (16, 40, 5120), (32, 39, 3072), (32, 64, 3840), (64, 40, 3072), (65, 64, 2048)])
def test_last_clusterings_of_all_pairs(lib, d, k, most):
    print(f"last clustering of all pairs, {most} x {d}, k={k}", flush=True)
    counts = [lib.slhc(rows(N, d, N), k, prune=False)["stats"]["knn_filter_survivors"] for N in (most, most + 1)]
    assert counts[0] == most * (most - 1) and counts[1] < most * most // 4


# rows so far from each other that the distance is no float32, and one row between them that both reach (lists of one such distance, of a quad and a part of
# one, of all rows but the far one)
@pytest.mark.gpu
@pytest.mark.parametrize("near,far,k", [(30, 1, 31), (30, 1, 8), (30, 1, 30), (29, 2, 3), (61, 2, 63), (4, 1, 5), (1, 1, 1)])
def test_trees_of_rows_out_of_reach(lib, near, far, k):
    print(f"rows out of reach, {near} + 1 + {far}, k={k}", flush=True)
    X = 1e14 * torch.randn((near + 1 + far, 4), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    X[:near, 0] += 1.5e19
    X[near + 1:, 0] -= 1.5e19
    want, got = lib.slhc(X, k, prune=False, fp32_filter=True), lib.slhc(X, k, prune=False)
    torch.cuda.synchronize()
    for key in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(want[key], got[key]), key
    assert torch.isfinite(got["mst_w"]).all()


def rows_and_groups(N, d, k, groups):
    """One blob that the lists connect, and groups of k + 1 rows far from it and from each other, which have to ask for their nearest other row."""
    g = torch.Generator(device="cuda").manual_seed(N + d)
    X = torch.randn((N, d), generator=g, device="cuda")
    away = torch.randn((groups, d), generator=g, device="cuda")
    away *= 60 * d ** 0.5 / away.norm(dim=1, keepdim=True)
    at = torch.randperm(N, generator=g, device="cuda")[:groups * (k + 1)]
    X[at] = away.repeat_interleave(k + 1, 0) + 0.01 * torch.randn((len(at), d), generator=g, device="cuda")
    return X


# rounds that ask for few rows: one workgroup's queries and several, candidates in segments of one step and of many, the last of them in part; every number of
# quads the kernel is made for
@pytest.mark.gpu
@pytest.mark.parametrize("N,d,k,groups", [(5000, 4, 2, 1), (5000, 12, 3, 9), (20_481, 30, 8, 4), (12_801, 48, 8, 16), (9000, 61, 8, 1), (7777, 90, 8, 30), (24_000, 128, 8, 1),
                                          (24_100, 128, 8, 16), (60_000, 100, 5, 2), (150_000, 7, 8, 20), (250_000, 16, 4, 3)])
def test_few_rows_that_have_to_be_connected(lib, N, d, k, groups):
    print(f"few queries, N={N} d={d} k={k} {groups} groups", flush=True)
    X = rows_and_groups(N, d, k, groups)
    want, got = lib.slhc(X, k, prune=False, fp32_filter=True), lib.slhc(X, k, prune=False)
    torch.cuda.synchronize()
    for key in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(want[key], got[key]), key
    assert groups * (k + 1) <= got["stats"]["connect_query_rows"]


# ... occupy the chip (with all candidates passing by each workgroup of a few queries the first took 3.8 ms, the second 9; 0.11 and 0.23 now)
@pytest.mark.gpu
@pytest.mark.parametrize("N,d,k,limit", [(100_000, 128, 8, 1.0), (300_000, 100, 16, 3.0)])
def test_few_queries_take_their_share(lib, N, d, k, limit):
    print(f"few queries, time, N={N} d={d}", flush=True)
    X = rows_and_groups(N, d, k, 1)
    took = [lib.slhc(X, k, prune=False)["stats"]["ms_connect_kernels"] for _ in range(4)]
    print("  ms", took, flush=True)
    assert 0 < min(took) < limit


# the segments of few queries' candidates queue for one line, not for eight words of it one by one (20 in 100 000 x 6 took 55 us, 2.7 times what the few segments
# of 1250 in 4000 x 4 take; 19 and 20 now)
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,d", [(20, 100_000, 6), (61, 50_000, 8)])
def test_segments_of_few_queries_meet_at_a_line(lib, m, n, d):
    print(f"small 1-NN, time, m={m} n={n} d={d}", flush=True)

    def least(m, n, d):
        Q, Y = rows(m, d, m), rows(n, d, n)
        out = (torch.empty(m, dtype=torch.int32, device="cuda"), torch.empty(m, dtype=torch.float32, device="cuda"))
        times = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(16):
                lib.fused_1nn(Q, Y, out=out)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        distances = ((Q[:, None, :] - Y[None]) ** 2).sum(2)
        assert torch.allclose(out[1], distances.min(1).values, rtol=1e-5) and (out[0] == distances.argmin(1)).float().mean() >= 0.95
        return min(times[2:])
    few_segments, many = least(1250, 4000, 4), least(m, n, d)
    print(f"  {62.5 * few_segments:.1f} us with few segments, {62.5 * many:.1f} with many", flush=True)
    assert many < 1.7 * few_segments
