"""Copies from global memory to LDS take their LDS address from M0, and an instruction that writes M0 must not stand
right in front of one: the hardware needs a wait state between the two.  The compiler keeps it between instructions
of its own but does not look into inline assembly, so the code in the built library is checked."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_21140_amd import build

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
WRITES_M0 = re.compile(r"s_\w+ m0\b")


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_a_wait_state_between_m0_and_the_copy(tmp_path):
    if not os.path.exists(build.LIB_PATH):
        build.build(verbose=False)
    lib = shutil.copy(build.LIB_PATH, tmp_path)  # the code objects are written beside the file
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    where, before, copies, bad = "", "", {}, []
    for obj in sorted(tmp_path.glob("*gfx950*")):
        r = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(obj)], check=True, capture_output=True, text=True)
        for line in r.stdout.splitlines():
            text = line.split("//")[0].strip()
            if text.startswith("<") and text.endswith(">:"):
                where = text[1:-2]
            elif "global_load_lds" in text or (text.startswith("buffer_load") and text.endswith(" lds")):
                copies[where] = copies.get(where, 0) + 1
                if WRITES_M0.match(before):
                    bad.append((where, before, text))
            if text:
                before = text
    for kernel in ("gemm_bf16_dma_kernel", "router_tile_kernel"):
        assert any(kernel in name for name in copies)
    assert not bad, (len(bad), bad[:3])
