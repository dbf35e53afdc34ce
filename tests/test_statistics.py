"""Counters and stage times of slhc(): what the caller is told about a call holds on every path."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import paper_2306_16354_amd as slhc
    slhc.load_library()
    assert torch.cuda.is_available()
    return slhc


def blobs(N, d, clusters, spread, seed):
    rng = np.random.default_rng(seed)
    centres = rng.uniform(-spread, spread, size=(clusters, d))
    return (centres[rng.integers(0, clusters, N)] + rng.standard_normal((N, d))).astype(np.float32)


# connection rounds in the row order by the half-precision engine and by the list kernels (whole rounds and rounds in two
# phases), without a row order in half precision and in float32, and of a forest that one workgroup holds
@pytest.mark.parametrize("N,flags", [(60_000, dict()), (60_000, dict(split_scans=True)), (60_000, dict(split_rounds=True)),
                                     (60_000, dict(prune=False)), (30_000, dict(prune=False, fp32_filter=True)), (3000, dict(prune=False))])
def test_stage_times_are_times(lib, N, flags):
    """Every stage time is positive where the stage ran, and no part exceeds the whole."""
    print(f"stage times N={N} {flags}", flush=True)
    Xd = torch.from_numpy(blobs(N, 64, 12, 20.0, N)).cuda()
    lib.slhc(Xd, 16, **flags)
    st = lib.slhc(Xd, 16, **flags)["stats"]
    assert st["connect_rounds"] >= 1
    for name in ("ms_knn", "ms_norm_kernel", "ms_knn_kernel", "ms_boruvka", "ms_connect", "ms_connect_kernels", "ms_sort", "ms_dendrogram"):
        assert 0.0 < st[name] <= st["ms_total"], (name, st[name], st["ms_total"])
    assert 0.0 <= st["ms_order"] <= st["ms_total"] and (st["ms_order"] > 0.0 or not st["pruned"])
    # HIP-event time of kernels inside a stage of host time: no longer than that stage
    assert st["ms_connect_kernels"] <= 1.05 * st["ms_connect"] + 0.05
    assert st["ms_knn_kernel"] <= 1.05 * st["ms_knn"] + 0.05


@pytest.mark.parametrize("d,far", [(16, 1), (64, 1), (64, 3), (128, 1)])
def test_far_pivots_do_not_hide_others(lib, d, far):
    """Every 64th row is a pivot of the row order, every row belongs to its nearest, and rows far from theirs get pivots of
    their own.  A pivot whose values lie beyond float16 (relative to the rest of the data) is nobody's nearest, and no row may
    lose its own by it.  The rows come in clusters with one pivot each: a far row in the middle of a cluster leaves the 63
    others of it (16 rows to a pivot, and the far row itself) without one, and nobody else."""
    N, k = 60_032, 8
    rng = np.random.default_rng(d)
    X = (np.repeat(rng.uniform(-50, 50, size=(N // 64, d)), 64, axis=0) + rng.standard_normal((N, d))).astype(np.float32)
    for i in range(far):
        X[64 * (7 + 100 * i)] = 1.0e9 * (1.0 + i)               # rows that are pivots
    out = lib.slhc(torch.from_numpy(X).cuda(), k)
    assert out["stats"]["pruned"] == 1
    print(f"d={d}, {far} far pivots: {out['stats']['order_pivots']} of {N // 64}", flush=True)
    want = lib.slhc(torch.from_numpy(X).cuda(), k, prune=False, fp32_filter=True)
    for key in ("mst_src", "mst_dst", "mst_w", "children", "heights", "sizes"):
        assert torch.equal(want[key], out[key]), key
    assert out["stats"]["order_pivots"] <= N // 64 + 5 * far + 4
