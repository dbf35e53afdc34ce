"""Workspace layouts and mailboxes, on the host: their code is compiled without the kernels and asked directly."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def host_program(name, out):
    """The lines that tests/<name>.hip prints."""
    from paper_2306_16354_amd import binding, build
    if not os.path.exists(binding.library_path()):
        build.build_library(verbose=False)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    obj, exe = str(out / (name + ".o")), str(out / name)
    where = os.path.dirname(binding.library_path())
    subprocess.run([hipcc, "-O1", "--cuda-host-only", "--offload-arch=gfx950", "-std=c++17", "-w", "-c",
                    os.path.join(ROOT, "tests", name + ".hip"), "-o", obj], check=True, capture_output=True)
    # (the device half of the file is not there)
    subprocess.run([hipcc, "-o", exe, obj, "-L" + where, "-lslhc", "-Wl,-rpath," + where, "-Wl,--unresolved-symbols=ignore-all"],
                   check=True, capture_output=True)
    return subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    return host_program("workspace_layouts", tmp_path_factory.mktemp("layouts"))


# A mailbox that has carried one kind of message takes nothing of it for the other's sequence number.
def test_messages_of_two_kinds_in_one_mailbox(tmp_path):
    assert host_program("mailboxes", tmp_path) == ["checked 800"]


def test_layouts_keep_within_their_bytes(report):
    assert report[-1].startswith("checked ") and int(report[-1].split()[1]) > 1000
    assert [line for line in report[:-1] if not line.startswith("least ")] == []


# Bytes that programs with a fixed budget have passed since before the half-precision engine: they are still accepted.
BUDGETS = """
knn 700 4 3 10783488          slhc 700 4 3 10865664
knn 4096 16 16 20844032       slhc 4096 16 16 21745408
knn 20011 50 10 50231040      slhc 20011 50 10 53675264
knn 100000 64 32 169009664    slhc 100000 64 32 203812096
knn 250000 784 16 802212608   slhc 250000 784 16 857216512
knn 1000000 128 32 3545627392 slhc 1000000 128 32 3893627648
knn 2000000 32 8 3855899392   slhc 2000000 32 8 4167899648
knn 100000000 8 8 13934118400 slhc 100000000 8 8 29534118656
fused 10 2000000 64 8000512   fused 1000 100000 128 412416    fused 1000 4000 30 28416      fused 20000 500000 256 2240256
cross 100000 64 10000 400384  cross 1000000 64 10 4000256     cross 2000 8 50 8448          cross 300000 128 300000 1200384
""".split()


@pytest.mark.parametrize("i", range(0, len(BUDGETS), 5))
def test_the_least_workspace_is_what_it_was(report, i):
    call, budget = " ".join(BUDGETS[i:i + 4]), int(BUDGETS[i + 4])
    least = [int(line.split()[-1]) for line in report if line.startswith("least " + call + " ")]
    assert len(least) == 1 and least[0] <= budget, call
