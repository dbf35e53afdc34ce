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
