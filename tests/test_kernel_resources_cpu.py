"""What the compiled kernels keep outside registers, from the metadata of the code
objects in the built library. A ligand or a work item held in scratch memory is
read from there in every step of a search."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2410_10447_amd import build_lib

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
SPILLS = 64          # bytes a lane: sixteen registers


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """Scratch bytes a lane of every kernel, by its mangled name."""
    objdump, readelf = os.path.join(LLVM, "llvm-objdump"), os.path.join(LLVM, "llvm-readelf")
    if not (os.path.exists(objdump) and os.path.exists(readelf) and os.path.exists(build_lib.LIB)):
        pytest.skip("needs the built library and the ROCm tools")
    tmp = tmp_path_factory.mktemp("objects")
    shutil.copy(build_lib.LIB, tmp / "lib.so")
    subprocess.run([objdump, "--offloading", "lib.so"], cwd=tmp, check=True, capture_output=True)
    out = {}
    for name in sorted(os.listdir(tmp)):
        if "gfx950" not in name:
            continue
        notes = subprocess.run([readelf, "--notes", name], cwd=tmp, check=True, capture_output=True, text=True).stdout
        for kernel in notes.split("- .agpr_count:")[1:]:
            symbol = re.search(r"^\s*\.name:\s+(\S+)", kernel, re.M).group(1)
            out[symbol] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", kernel).group(1))
    assert out
    return out


def test_kernels_that_choose_the_reduction_at_run_time(scratch):
    """ls_kernel<mode, -1> and ls_kernel_mw<-1, waves>: searches on plain maps or of
    items with different reductions."""
    several = {k: v for k, v in scratch.items() if re.search(r"ls_kernelILi\d+ELin1E|ls_kernel_mwILin1E", k)}
    assert len(several) == 5
    assert all(v <= SPILLS for v in several.values()), several
