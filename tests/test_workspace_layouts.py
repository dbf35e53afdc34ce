"""Workspace layouts, on the host: the layout code is compiled without its kernels and asked directly."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    from paper_2306_16354_amd import binding, build
    if not os.path.exists(binding.library_path()):
        build.build_library(verbose=False)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    out = tmp_path_factory.mktemp("layouts")
    obj, exe = str(out / "layouts.o"), str(out / "layouts")
    where = os.path.dirname(binding.library_path())
    subprocess.run([hipcc, "-O1", "--cuda-host-only", "--offload-arch=gfx950", "-std=c++17", "-w", "-c",
                    os.path.join(ROOT, "tests", "workspace_layouts.hip"), "-o", obj], check=True, capture_output=True)
    # (the device half of the file is not there)
    subprocess.run([hipcc, "-o", exe, obj, "-L" + where, "-lslhc", "-Wl,-rpath," + where, "-Wl,--unresolved-symbols=ignore-all"],
                   check=True, capture_output=True)
    return subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()


def test_layouts_keep_within_their_bytes(report):
    assert report[-1].startswith("checked ") and int(report[-1].split()[1]) > 1000
    assert report[:-1] == []
