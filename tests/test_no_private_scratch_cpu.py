"""No kernel of the built library uses private scratch: an array that is indexed at run time, or registers that do not
suffice, would put some of it there, and each launch then begins with a trip to memory that nobody sees."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_21140_amd import build

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


@pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-readelf")), reason="no llvm-readelf")
def test_no_kernel_uses_private_scratch(tmp_path):
    if not os.path.exists(build.LIB_PATH):
        build.build(verbose=False)
    lib = shutil.copy(build.LIB_PATH, tmp_path)  # the code objects are written beside the file
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    found = {}
    for obj in sorted(tmp_path.glob("*gfx950*")):
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", str(obj)], check=True, capture_output=True, text=True).stdout
        names = re.findall(r"^\s*\.name:\s+(_Z\S+)", notes, re.M)
        sizes = [int(n) for n in re.findall(r"\.private_segment_fixed_size:\s+(\d+)", notes)]
        assert len(names) == len(sizes)
        found.update(zip(names, sizes))
    assert any("gemm_bf16_dma_kernel" in n for n in found) and any("route_topk_rows_kernel" in n for n in found)
    assert not {n: s for n, s in found.items() if s}
