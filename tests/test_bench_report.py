"""The benchmark's line says which kernels its times are of."""
import json
import sys

import pytest

torch = pytest.importorskip("torch")


# a workload whose pairs are all evaluated multiplies nothing; one more row than such a search may have goes to the engine
@pytest.mark.gpu
@pytest.mark.parametrize("rows,every_pair", [(4096, True), (4608, True), (4609, False)])
@pytest.mark.parametrize("knn_only", [False, True])
def test_small_workload(monkeypatch, capsys, rows, every_pair, knn_only):
    import bench
    monkeypatch.setattr(sys, "argv", ["bench.py", "--workload", "c1", "--rows", str(rows), "--steps", "2", "--warmup", "1", "--no-cpu-baseline", "--no-pruned-leg",
                                      "--no-fp32-leg"] + (["--knn-only"] if knn_only else []))
    bench.main()
    line = json.loads(capsys.readouterr().out.strip().splitlines()[-1])
    roof = line["roofline"]
    if every_pair and not knn_only:
        assert roof["kernel"] == "direct_knn_kernel" and roof["bound"] == "vector_fp32" and line["dtype"] == "f32"
        assert roof["executed_mfma_flop_per_launch"] == 0 and line["counters"]["knn_filter_survivors"] == rows * (rows - 1)
    else:
        assert "near_select_kernel" in roof["kernel"] and roof["bound"] == "mfma" and "float16 copies" in line["dtype"]
        assert roof["executed_mfma_flop_per_launch"] > 0
