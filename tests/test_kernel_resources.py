"""Registers of built kernels, where one more of them costs a workgroup per CU."""
import os
import re
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Mangled name -> (vector registers, bytes of scratch memory per lane), of the library's gfx950 code."""
    from paper_2306_16354_amd import binding, build
    if not os.path.exists(binding.library_path()):
        build.build_library(verbose=False)
    where = tmp_path_factory.mktemp("code")
    lib = where / "libslhc.so"
    os.symlink(binding.library_path(), lib)
    subprocess.run([LLVM + "/llvm-objdump", "--offloading", str(lib)], check=True, capture_output=True, cwd=where)
    out = {}
    for code in where.glob("*gfx950*"):
        notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", str(code)], check=True, capture_output=True, text=True).stdout
        for part in notes.split("- .agpr_count:")[1:]:
            value = {key: v for key, v in re.findall(r"^\s+\.(name|vgpr_count|private_segment_fixed_size):\s+(\S+)", part, re.M)}
            out[value["name"]] = (int(value["vgpr_count"]), int(value["private_segment_fixed_size"]))
    return out


# emission of up to 32 columns, in the row order and without: four wavefronts per SIMD
@pytest.mark.parametrize("steps", [1, 2])
@pytest.mark.parametrize("listed", [0, 1])
def test_narrow_emission(kernels, steps, listed):
    registers, scratch = kernels[f"_ZN4slhc17near_sweep_kernelILi{steps}ELi1ELb0ELb{listed}EEEvNS_9NearSweepE"]
    assert registers <= 128 and scratch <= 64


# blocks of pairs in registers: all a CU has for two wavefronts per SIMD, and no scratch
@pytest.mark.parametrize("quads", [2, 4, 8, 12, 16, 24, 32])
@pytest.mark.parametrize("name", ["17direct_knn_kernelILi{}EEEvNS_9DirectKnnE", "18direct_near_kernelILi{}EEEvNS_10DirectNearE"])
def test_blocks_of_pairs(kernels, name, quads):
    registers, scratch = kernels["_ZN4slhc" + name.format(quads)]
    assert registers <= (128 if quads == 2 else 256) and scratch == 0


# searches by colours of up to 48 columns: four wavefronts per SIMD, where their masks leave the registers
@pytest.mark.parametrize("steps", [1, 2, 3])
@pytest.mark.parametrize("mode", [2, 5])
def test_narrow_searches_by_colours(kernels, steps, mode):
    registers, scratch = kernels[f"_ZN4slhc17near_sweep_kernelILi{steps}ELi{mode}ELb1ELb0EEEvNS_9NearSweepE"]
    assert registers <= 128 and scratch == 0
